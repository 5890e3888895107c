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
# tile column, a partly filled last one, columns that do not fill a macro step, the largest K of one (14592) and of two chunks (7168 with
# 2560 and 1300 rows, where two are taken), one beyond; rows that no tile divides
FEW_TOKENS = [(1, 4, 1), (5, 60, 3), (33, 64, 8), (203, 68, 9), (203, 1020, 16), (77, 2560, 17), (640, 2560, 24), (640, 2564, 41),
              (4097, 516, 8), (4100, 300, 13), (8200, 260, 16), (16400, 132, 5), (32768, 68, 2), (32769, 64, 2), (50, 7168, 16),
                                   (50, 7172, 16), (64, 14592, 8), (64, 14592, 11), (40, 14596, 2), (100, 8196, 20),
              (2560, 7168, 16), (2560, 7172, 16), (1300, 7168, 41), (900, 7168, 35)]


@pytest.mark.parametrize("M,K,N", FEW_TOKENS)
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
FEW_TOKENS_FIVE = [(1, 20, 1), (5, 24, 3), (33, 320, 8), (203, 336, 9), (203, 1036, 16), (77, 2560, 17), (640, 2564, 33), (4097, 516, 8),
                   (8200, 276, 16), (16400, 136, 5), (50, 7360, 16), (50, 7364, 16), (64, 14592, 8), (40, 14596, 2), (100, 396, 70),
                   (2560, 7360, 16), (2560, 7364, 16), (1300, 7356, 41), (903, 7356, 35)]


@pytest.mark.parametrize("M,K,N", FEW_TOKENS_FIVE)
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


# some tiles whose loads are spread over two groups of matrix instructions (256 rows x 128 tokens, 128 x 64, 64 x 64), at sizes with a partly
# filled last tile and macro step; every tile: the next test
@pytest.mark.parametrize("M,K,N", [(5400, 388, 1030), (5376, 128, 1024), (6912, 2564, 200), (1500, 5124, 500)])
def test_large_tiles(B, M, K, N):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + K)
    W = torch.randint(-1, 2, (M, K), dtype=torch.int8, generator=gen, device="cuda")
    a_q, a_s = B.quantize_act(torch.randn(N, K, generator=gen, device="cuda"))
    _, acc = B.mpgemm(B.pack_weights(W), 1.0, a_q, a_s, M, want_acc=True)
    q = B.act_chunked_to_kn(a_q, N).float()                    # products and sums of whole numbers below 2^24: exact in fp32
    assert torch.equal(acc, (W.float().cpu() @ q.cpu()).to(torch.int32).cuda())


# every workgroup that is built, (rows, tokens, parts of K), at sizes that it does not divide: outputs with a scale per row and rows further
# apart than their length, accumulators, the K loop with a rest.  test_plans_host.py checks the list against the plans and the table of tiles
WORKGROUPS = [("codes", 17, 5328, 10, (16, 8, 16)), ("codes", 18, 5344, 1171, (16, 16, 16)), ("codes", 2455, 2668, 18, (32, 8, 8)),
              ("codes", 35, 2716, 1396, (32, 16, 8)), ("codes", 4819, 1380, 17, (64, 8, 4)), ("codes", 1654, 1348, 73, (64, 16, 4)),
              ("codes", 8862, 704, 19, (128, 8, 2)), ("codes", 6424, 684, 33, (128, 16, 2)), ("codes", 35, 15600, 217, (32, 32, 8)),
              ("codes", 149, 728, 1365, (64, 32, 4)), ("codes", 1893, 668, 348, (64, 64, 4)), ("codes", 5391, 3064, 352, (64, 128, 4)),
              ("codes", 14130, 1096, 66, (128, 64, 4)), ("codes", 6040, 336, 332, (128, 128, 2)), ("codes", 7776, 176, 1051, (256, 128, 1)),
              ("codes", 13830, 388, 1030, (256, 128, 1)), ("codes", 8067, 348, 545, (256, 128, 2)),
              ("g5", 18, 5420, 9, (16, 8, 16)), ("g5", 20, 6200, 1100, (16, 16, 16)), ("g5", 2075, 2980, 17, (32, 8, 8)),
              ("g5", 68, 2800, 820, (32, 16, 8)), ("g5", 5158, 1400, 18, (64, 8, 4)), ("g5", 5574, 1420, 17, (64, 16, 4)),
              ("g5", 8651, 760, 17, (128, 8, 2)), ("g5", 193, 680, 1030, (128, 16, 2)), ("g5", 36, 15460, 37, (32, 32, 8)),
              ("g5", 5706, 1220, 34, (64, 32, 4)), ("g5", 772, 680, 610, (64, 64, 4)), ("g5", 2564, 340, 680, (128, 128, 2)),
              ("g5", 11429, 340, 286, (256, 128, 2)),
              ("mixed", 17, 5536, 1179, (16, 16, 16)), ("mixed", 8584, 692, 20, (128, 8, 2)), ("mixed", 37, 15344, 40, (32, 32, 8)),
              ("mixed", 258, 728, 1377, (64, 32, 4)), ("mixed", 5513, 684, 87, (64, 64, 4)), ("mixed", 1521, 336, 907, (128, 128, 2)),
              ("mixed", 11750, 364, 261, (256, 128, 2))]


@pytest.mark.parametrize("form,M,K,N,workgroup", WORKGROUPS)
def test_every_workgroup(B, form, M, K, N, workgroup):
    assert B.query_matrix_plan(form, M, K, N)[:3] == workgroup
    print(f"workgroup case {form} M={M} K={K} N={N} {workgroup}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + K + N)
    W = torch.randint(-1, 2, (M, K), dtype=torch.int8, generator=gen, device="cuda")
    a_q, a_s = B.quantize_act(torch.randn(N, K, generator=gen, device="cuda"))
    q = B.act_chunked_to_kn(a_q, N).float().cpu()
    acc_ref = W.float().cpu() @ q                              # products and sums of whole numbers below 2^24: exact in fp32
    pad = torch.full((N, M + 3), -7.0, device="cuda")
    if form == "codes":
        scale = torch.rand(M, generator=gen, device="cuda") + 0.5
        y, acc = B.mpgemm_rows(B.pack_weights(W), scale, a_q, a_s, M, y=pad[:, :M], want_acc=True)
    else:
        scale = torch.full((M,), 0.375, device="cuda")
        pack, mm = (B.pack_weights_g5, B.mpgemm_g5) if form == "g5" else (B.pack_weights_mixed, B.mpgemm_mixed)
        y, acc = mm(pack(W), 0.375, a_q, a_s, M, y=pad[:, :M], want_acc=True)
    assert torch.equal(acc.cpu(), acc_ref.to(torch.int32))
    want = acc_ref.double().t() * scale.cpu().double() * a_s.cpu().double()[:, None]
    assert torch.all((y.cpu().double() - want).abs() <= REL * want.abs()) and torch.all(pad[:, M:] == -7.0)
