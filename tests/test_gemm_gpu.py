"""The matrix-core path against the oracle at the edges of its tiles: every packed byte value, rows and tokens next to multiples
of the tile shapes, K with an odd number of packed tile columns, fewer macro steps than groups, the 2-bit tail of the
mixed packing at each of its lengths.  Integers are compared exactly; an output is one whole number below 2^24 times two
fp32 scales, two roundings, hence 2 * 2^-24 < 1.2e-7 relative to the oracle's fp64 product."""
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
    binding.set_plan(0, 0, 0, 0)
    binding.set_plan_g5(0, 0)
    return binding


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def check(B, W, s, x, packings=("p4", "mixed"), tag=""):
    M, K = W.shape
    N = x.shape[0]
    print(f"gemm case {tag} M={M} K={K} N={N}", flush=True)
    _, _, acc_ref, y_ref = O.mpgemm(W, s, x)
    a_q, a_s = B.quantize_act(dev(x))
    calls = {"p4": (B.pack_weights, B.mpgemm), "g5": (B.pack_weights_g5, B.mpgemm_g5), "mixed": (B.pack_weights_mixed, B.mpgemm_mixed)}
    for name in packings:
        pack, mpgemm = calls[name]
        ybig = torch.full((N + 1, M + 3), -7.0, device="cuda")
        y, acc = mpgemm(pack(dev(W)), float(s), a_q, a_s, M, y=ybig[:N, :M], want_acc=True)
        torch.cuda.synchronize()
        assert np.array_equal(acc.cpu().numpy(), acc_ref), name
        yy = y.cpu().numpy().astype(np.float64)
        assert np.all(np.abs(yy - y_ref) <= REL * np.abs(y_ref)), name
        full = ybig.cpu().numpy()
        assert np.all(full[:, M:] == -7.0) and np.all(full[N:] == -7.0), name


@pytest.mark.parametrize("g,K", [(4, 324), (5, 1220)])
def test_every_packed_byte(B, g, K):
    # row r holds pattern r in its group r and zeros elsewhere; all patterns in one row as well
    n = 3 ** g
    digits = np.array([[(v // 3 ** (g - 1 - j)) % 3 - 1 for j in range(g)] for v in range(n)], np.int8)
    W = np.zeros((n + 1, K), np.int8)
    for v in range(n):
        W[v, v * g:(v + 1) * g] = digits[v]
    W[n, :n * g] = digits.reshape(-1)
    check(B, W, np.float32(0.5), wl.activations(11, 40, K), ("p4",) if g == 4 else ("g5",), tag=f"all bytes g={g}")


@pytest.mark.parametrize("M,K,N", [(31, 64, 33), (32, 128, 32), (65, 192, 31), (33, 4160, 65), (127, 516, 64), (129, 2564, 96),
                                   (3840, 260, 1000), (4099, 1028, 1030), (8193, 132, 520), (513, 9220, 515), (7000, 2580, 127), (16, 32768, 33), (64, 16384, 40),
                                   (200, 14336, 64)])
def test_tile_edges(B, M, K, N):
    # (the last three: next to the rule that leaves few rows with a long K to the lookup kernel, tested with the route asked for
    # in test_routes_gpu.py)
    W, s, x = wl.small_case(1200 + M + N, M, K, N)
    check(B, W, s, x, tag="edges")


@pytest.mark.parametrize("K", [20, 24, 28, 32, 36, 176, 336, 2564, 2576])
def test_tail_lengths_of_the_mixed_packing(B, K):
    W, s, x = wl.small_case(1300 + K, 70, K, 37)
    check(B, W, s, x, ("mixed", "g5") if K % 20 == 0 else ("mixed",), tag="tail")


def test_extremes_of_the_accumulator(B):
    W = np.ones((40, 8192), np.int8)
    W[1::2] = -1
    x = np.ones((35, 8192), np.float32)
    x[::3] = -1.0
    check(B, W, np.float32(1.0), x, tag="all +-127")


@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 8, 9, 15, 16])
def test_few_tokens_from_fp32(B, N):
    # one launch that quantises inside: every count of token slots, rows next to 16, 32, 64 and 128 per workgroup, K with
    # one to more than twelve passes of 256 values per wave, the last ones ragged; unaligned rows of x
    for M, K in ((1, 4), (17, 260), (4097, 1028), (8200, 512), (16400, 64), (130, 3844), (50, 65536 // N // 4 * 4)):
        W, s, x = wl.small_case(1400 + M + N, M, K, N)
        x[N // 2] *= 1e-3
        _, s_ref, acc_ref, y_ref = O.mpgemm(W, s, x)
        packed = B.pack_weights(dev(W))
        odd = torch.full((N, K + 3), 9e9, device="cuda")
        odd[:, 1:K + 1] = dev(x)
        for xd in (dev(x), odd[:, 1:K + 1]):
            print(f"decode case M={M} K={K} N={N}", flush=True)
            y, acc, sc = B.mpgemm_f32(packed, float(s), xd, M, want_acc=True, want_scales=True)
            torch.cuda.synchronize()
            assert np.array_equal(acc.cpu().numpy(), acc_ref)
            assert np.array_equal(sc.cpu().numpy().view(np.uint32), s_ref.view(np.uint32))
            assert np.all(np.abs(y.cpu().numpy().astype(np.float64) - y_ref) <= REL * np.abs(y_ref))


@pytest.mark.parametrize("N", [1, 13, 259, 767, 768, 771, 1030])
def test_quantiser_with_one_and_four_tokens_per_workgroup(B, N):
    # rows that fit each count of registers per thread and longer ones, ragged K, unaligned rows, a zero row
    for K in (4, 260, 4096, 4100, 8196, 14340, 16388):
        x = wl.activations(1500 + K, N, K)
        x[N - 2] = 0.0
        # below 127 / FLT_MAX = 3.7e-37 the reciprocal overflows and every nonzero value becomes +-127; 0 * inf has no defined
        # code, so the scale keeps nonzero values nonzero (FLT_TRUE_MIN = 1.4e-45)
        x[N // 2] *= 1e-38
        q_ref, s_ref = O.quantize(x)
        odd = torch.full((N, K + 3), 9e9, device="cuda")
        odd[:, 1:K + 1] = dev(x)
        for xd in (dev(x), odd[:, 1:K + 1]):
            a_q, a_s = B.quantize_act(xd, torch.full(((N + 7) // 8, K, 8), 99, dtype=torch.int8, device="cuda"))
            torch.cuda.synchronize()
            assert np.array_equal(B.act_chunked_to_kn(a_q, N).cpu().numpy(), q_ref)
            assert np.array_equal(a_s.cpu().numpy().view(np.uint32), s_ref.view(np.uint32))
            if N % 8:
                assert int(a_q[-1, :, N % 8:].abs().max()) == 0      # tokens past N hold zeros


def test_pack_unaligned_and_value_check(B):
    # matrices and blobs that start at any byte, ragged tails; a bad value anywhere is reported and the next call is clean
    M, K = 37, 340
    W = wl.ternary(1600, M, K, 0.4)
    L = B.lib()
    calls = ((L.vlut_pack_weights, B.pack_weights), (L.vlut_pack_weights_g5, B.pack_weights_g5),
             (L.vlut_pack_weights_mixed, B.pack_weights_mixed))
    for raw, wrapped in calls:
        want = wrapped(dev(W))
        for off in (1, 2, 7):
            src = torch.zeros(M * K + 16, dtype=torch.int8, device="cuda")
            src[off:off + M * K] = dev(W).flatten()
            blob = torch.full((want.numel() + 16,), 255, dtype=torch.uint8, device="cuda")
            assert raw(src.data_ptr() + off, M, K, blob.data_ptr() + off, want.numel(), None) == 0
            assert torch.equal(blob[off:off + want.numel()], want)
            assert int((blob == 255).sum()) == 16
        good = want.clone()                                 # (the calls with a bad value overwrite the blob they are given)
        for pos, value in ((0, 2), (5 * K + 33, -2), (M * K - 1, 3), (M * K // 2, -128), (17, 127)):
            bad = dev(W).flatten()
            bad[pos] = value
            assert raw(bad.data_ptr(), M, K, want.data_ptr(), want.numel(), None) == B.VLUT_ERR_VALUE
            assert torch.equal(wrapped(dev(W)), good)


def test_missing_matrix_is_a_status_code(B):
    with pytest.raises(B.VlutError) as e:
        B.mpgemm_f32(None, 1.0, torch.zeros((4, 64), device="cuda"), 64)
    assert e.value.status == B.VLUT_ERR_NULL


@pytest.mark.parametrize("N", [1535, 1541, 3583, 3590])
def test_quantiser_at_its_switch_over_points(B, N):
    # one, four and eight tokens per workgroup, one, four and eight waves; rows at the limits of what each keeps in registers
    for K in (4, 252, 256, 260, 1024, 1028, 1536, 1540, 2048, 2052, 3072, 3076):
        x = wl.activations(1700 + K, N, K)
        x[N - 2] = 0.0
        q_ref, s_ref = O.quantize(x)
        odd = torch.full((N, K + 3), 9e9, device="cuda")
        odd[:, 1:K + 1] = dev(x)
        for xd in (dev(x), odd[:, 1:K + 1]):
            print(f"quantiser case K={K} N={N} stride={xd.stride(0)}", flush=True)
            a_q, a_s = B.quantize_act(xd, torch.full(((N + 7) // 8, K, 8), 99, dtype=torch.int8, device="cuda"))
            torch.cuda.synchronize()
            assert np.array_equal(B.act_chunked_to_kn(a_q, N).cpu().numpy(), q_ref)
            assert np.array_equal(a_s.cpu().numpy().view(np.uint32), s_ref.view(np.uint32))
            if N % 8:
                assert int(a_q[-1, :, N % 8:].abs().max()) == 0


@pytest.mark.parametrize("N,K", [(4096, 64), (4096, 1024), (2000, 2560), (1000, 6912)])
def test_unaligned_rows_cost_the_quantiser_about_what_aligned_ones_do(B, N, K):
    # they were read twice, eight loads at a time: 2 to 3 times as long.  The same bytes, so the same time but for the
    # narrower loads (0.9 to 1.05 measured); half of it is left for a busy machine, the best of several runs is taken
    x = torch.randn((N, K + 1), device="cuda")
    out = B.quantize_act(x[:, 1:])
    sides = {"unaligned": x[:, 1:], "aligned": x[:, 1:].contiguous()}
    best = {}
    for rep in range(8):
        for name, xd in sides.items():
            B.quantize_act(xd, *out)
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda._sleep(200000)                       # the launches queue up behind it: their own time, not the host's
            e0.record()
            for _ in range(20):
                B.quantize_act(xd, *out)
            e1.record()
            torch.cuda.synchronize()
            best[name] = min(best.get(name, 1e9), e0.elapsed_time(e1))
    print(best)
    assert best["unaligned"] < 1.5 * best["aligned"]


def check_f32(B, W, s, x, kernel):
    """mpgemm_f32 on aligned and on unaligned rows against the oracle; `kernel` is the one the library must take."""
    M, K = W.shape
    N = x.shape[0]
    assert B.query_kernel("f32", M, K, N) == kernel
    _, s_ref, acc_ref, y_ref = O.mpgemm(W, s, x)
    packed = B.pack_weights(dev(W))
    odd = torch.full((N, K + 3), 9e9, device="cuda")
    odd[:, 1:K + 1] = dev(x)
    for xd in (dev(x), odd[:, 1:K + 1]):
        print(f"f32 case {kernel} M={M} K={K} N={N} stride={xd.stride(0)}", flush=True)
        y, acc, sc = B.mpgemm_f32(packed, float(s), xd, M, want_acc=True, want_scales=True)
        torch.cuda.synchronize()
        assert np.array_equal(acc.cpu().numpy(), acc_ref)
        assert np.array_equal(sc.cpu().numpy().view(np.uint32), s_ref.view(np.uint32))
        assert np.all(np.abs(y.cpu().numpy().astype(np.float64) - y_ref) <= REL * np.abs(y_ref))


@pytest.mark.parametrize("M,K,kernel", [(16384, 1024, "matrix_few_tokens"), (16385, 1024, "few_tokens"), (16385, 1020, "matrix_few_tokens"),
                                        (16401, 9220, "few_tokens"), (32768, 1028, "few_tokens"), (32769, 260, "few_tokens")])
def test_one_token_on_many_rows(B, M, K, kernel):
    check_f32(B, *wl.small_case(1800 + M + K, M, K, 1), kernel)


@pytest.mark.parametrize("M,K,N,kernel", [(4, 6552, 10, "few_tokens"), (33, 4096, 16, "few_tokens"), (100, 5040, 13, "few_tokens"),
                                          (1000, 4680, 14, "few_tokens"), (1000, 4096, 14, "matrix_few_tokens"), (33, 3072, 16, "matrix_few_tokens")])
def test_nine_to_sixteen_tokens_on_few_rows(B, M, K, N, kernel):
    check_f32(B, *wl.small_case(1900 + M + N, M, K, N), kernel)


# The tiles whose operands are loaded straight to LDS: one to eight passes of the K loop (three slots, two register sets), K that ends
# anywhere in a step, tiles that the matrix fills (stored without checks, past the caches from 16 MB on) and cuts.
TILES_LOADED_TO_LDS = [
    (3328, 4, 640, (128, 128, 2)), (8307, 260, 238, (128, 128, 2)), (8448, 516, 256, (128, 128, 2)), (11187, 780, 167, (128, 128, 2)),
    (3840, 1300, 1024, (128, 128, 2)), (3840, 1544, 1000, (128, 128, 2)), (11008, 4, 384, (256, 128, 2)), (11266, 260, 384, (256, 128, 2)),
    (11008, 516, 384, (256, 128, 2)), (14336, 1540, 512, (256, 128, 2)), (9628, 4, 793, (256, 128, 1)), (14592, 132, 640, (256, 128, 1)),
    (11264, 388, 768, (256, 128, 1)), (13429, 812, 518, (256, 128, 1)), (3840, 520, 384, (128, 64, 4)), (14336, 1032, 67, (128, 64, 4)),
    (10888, 1156, 65, (128, 64, 2)), (8448, 2592, 128, (128, 64, 2)), (11261, 3944, 65, (128, 64, 2)), (9804, 4920, 100, (128, 64, 4)),
    (4096, 9220, 512, (128, 64, 4)), (2052, 1336, 1000, (160, 64, 4)), (2560, 2560, 1024, (160, 64, 4)), (10881, 2180, 190, (160, 64, 4))]


@pytest.mark.parametrize("M,K,N,workgroup", TILES_LOADED_TO_LDS)
def test_tiles_loaded_to_lds(B, M, K, N, workgroup):
    assert B.query_matrix_plan("codes", M, K, N)[:3] == workgroup
    print(f"tile case {workgroup} M={M} K={K} N={N}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + K + N)
    W = torch.randint(-1, 2, (M, K), dtype=torch.int8, generator=gen, device="cuda")
    a_q, a_s = B.quantize_act(torch.randn(N, K, generator=gen, device="cuda"))
    packed = B.pack_weights(W)
    acc_ref = W.float().cpu() @ B.act_chunked_to_kn(a_q, N).float().cpu()      # whole numbers below 2^24: exact in fp32
    rows = torch.rand(M, device="cuda") + 0.5
    def right(y, scale):                                     # two fp32 roundings of the exact product
        want = acc_ref.double().t() * scale.cpu().double() * a_s.cpu().double()[:, None]
        return bool(torch.all((y.cpu().double() - want).abs() <= REL * want.abs()))
    y, _ = B.mpgemm(packed, 0.375, a_q, a_s, M)
    assert right(y, torch.full((M,), 0.375))
    pad = torch.full((N, M + 7), -7.0, device="cuda")        # rows that start at any float, and what lies beside them
    y, acc = B.mpgemm_rows(packed, rows, a_q, a_s, M, y=pad[:, 3:M + 3], want_acc=True)
    assert torch.equal(acc.cpu(), acc_ref.to(torch.int32)) and right(y, rows)
    B.mpgemm_rows(packed, rows, a_q, a_s, M, y=pad[:, 3:M + 3])
    assert right(pad[:, 3:M + 3], rows) and torch.all(pad[:, :3] == -7.0) and torch.all(pad[:, M + 3:] == -7.0)
