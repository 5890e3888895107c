"""A few tokens from INT8 codes on the matrix cores (one or two chunks of eight per workgroup) against the oracle: integers exactly,
outputs to two fp32 roundings."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2512_06443_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
REL = 2.0 ** -23


@pytest.fixture(scope="module")
def B():
    from paper_2512_06443_amd import binding
    binding.lib()
    yield binding


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# one and two chunks per workgroup, several token tiles, a last chunk that is absent or partly filled; 16 to 128 rows per workgroup; K with one
# tile column, a partly filled last one, columns that do not fill a macro step, the largest K of one (14592) and of two chunks (7168), one
# beyond; rows that no tile divides
@pytest.mark.parametrize("M,K,N", [(1, 4, 1), (5, 60, 3), (33, 64, 8), (203, 68, 9), (203, 1020, 16), (77, 2560, 17), (640, 2560, 24), (640, 2564, 41),
                                   (4097, 516, 8), (4100, 300, 13), (8200, 260, 16), (16400, 132, 5), (32768, 68, 2), (32769, 64, 2), (50, 7168, 16),
                                   (50, 7172, 16), (64, 14592, 8), (64, 14592, 11), (40, 14596, 2), (100, 8196, 20)])
def test_few_tokens_from_codes(B, M, K, N):
    print(f"codes case M={M} K={K} N={N}", flush=True)
    W, s, x = wl.small_case(3000 + M + K + N, M, K, N)
    _, _, acc_ref, y_ref = O.mpgemm(W, s, x)
    a_q, a_s = B.quantize_act(dev(x))
    packed = B.pack_weights(dev(W))
    y, acc = B.mpgemm(packed, float(s), a_q, a_s, M, want_acc=True)
    rows = torch.full((M,), float(s), device="cuda")
    pad = torch.full((N, M + 3), -7.0, device="cuda")
    yr, accr = B.mpgemm_rows(packed, rows, a_q, a_s, M, y=pad[:, :M], want_acc=True)
    torch.cuda.synchronize()
    assert np.array_equal(acc.cpu().numpy(), acc_ref) and torch.equal(acc, accr)
    assert np.all(np.abs(y.cpu().numpy().astype(np.float64) - y_ref) <= REL * np.abs(y_ref))
    assert torch.equal(y, yr) and torch.all(pad[:, M:] == -7.0)


# the 1.60-bit and the mixed packing: no, one and four groups of four behind the last twenty values, in every column position of them; the
# sizes of a workgroup as above (the largest K of two chunks is 7360)
@pytest.mark.parametrize("M,K,N", [(1, 20, 1), (5, 24, 3), (33, 320, 8), (203, 336, 9), (203, 1036, 16), (77, 2560, 17), (640, 2564, 33), (4097, 516, 8),
                                   (8200, 276, 16), (16400, 136, 5), (50, 7360, 16), (50, 7364, 16), (64, 14592, 8), (40, 14596, 2), (100, 396, 70)])
def test_few_tokens_from_codes_five_weights_per_byte(B, M, K, N):
    print(f"codes5 case M={M} K={K} N={N}", flush=True)
    W, s, x = wl.small_case(3500 + M + K + N, M, K, N)
    _, _, acc_ref, y_ref = O.mpgemm(W, s, x)
    a_q, a_s = B.quantize_act(dev(x))
    out = [B.mpgemm_mixed(B.pack_weights_mixed(dev(W)), float(s), a_q, a_s, M, want_acc=True)]
    if K % 20 == 0:
        out.append(B.mpgemm_g5(B.pack_weights_g5(dev(W)), float(s), a_q, a_s, M, want_acc=True))
    for y, acc in out:
        assert np.array_equal(acc.cpu().numpy(), acc_ref)
        assert np.all(np.abs(y.cpu().numpy().astype(np.float64) - y_ref) <= REL * np.abs(y_ref))


# every byte of both packings in every position of a dword: all pairs of digits that the byte permutes look up
@pytest.mark.parametrize("g,N", [(4, 3), (4, 40), (5, 3), (5, 40)])
def test_every_packed_byte(B, g, N):
    values = 3 ** g
    idx = (np.arange(values)[:, None] + 37 * np.arange(16)[None, :]) % values           # row r, byte b of a tile column
    digits = (idx[:, :, None] // 3 ** np.arange(g - 1, -1, -1)) % 3 - 1
    W = np.ascontiguousarray(digits.reshape(values, 16 * g).astype(np.int8))
    assert all(len(set(idx[:, b])) == values for b in range(16))
    rng = np.random.default_rng(5)
    q = rng.integers(-127, 128, (N, W.shape[1])).astype(np.int8)
    chunks = (N + 7) // 8
    a_q = np.zeros((chunks, W.shape[1], 8), np.int8)
    for n in range(N):
        a_q[n // 8, :, n % 8] = q[n]
    pack, mm = (B.pack_weights, B.mpgemm) if g == 4 else (B.pack_weights_g5, B.mpgemm_g5)
    _, acc = mm(pack(dev(W)), 1.0, dev(a_q), torch.ones(N, device="cuda"), values, want_acc=True)
    assert np.array_equal(acc.cpu().numpy(), W.astype(np.int64) @ q.T.astype(np.int64))


# the tiles whose loads are spread over two groups of matrix instructions and those added
# to the table (two workgroups of four waves per compute unit; 128 rows x 64 tokens), at sizes with a partly filled last tile and macro step
@pytest.mark.parametrize("M,K,N", [(5400, 388, 1030), (5376, 128, 1024), (6912, 2564, 200), (1500, 5124, 500)])
def test_large_tiles(B, M, K, N):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + K)
    W = torch.randint(-1, 2, (M, K), dtype=torch.int8, generator=gen, device="cuda")
    a_q, a_s = B.quantize_act(torch.randn(N, K, generator=gen, device="cuda"))
    _, acc = B.mpgemm(B.pack_weights(W), 1.0, a_q, a_s, M, want_acc=True)
    q = B.act_chunked_to_kn(a_q, N).float()                    # products and sums of whole numbers below 2^24: exact in fp32
    assert torch.equal(acc, (W.float().cpu() @ q.cpu()).to(torch.int32).cuda())
