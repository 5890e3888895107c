"""The kernels behind a call that an ordinary call of the same shape does not take: the lookup kernels of the 1.60-bit and the
mixed packing (a forced plan, operands that are not 16-byte aligned, K that 4 does not divide), the lookup kernel where it is
the faster one, and the few-token table kernel from fp32 where the one-launch matrix-core kernel does not apply.  The kernel is
asked for first, then the numbers are compared with the oracle: integers exactly, outputs to two fp32 roundings."""
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
    binding.set_plan(0, 0, 0, 0)
    binding.set_plan_g5(0, 0)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def shifted(t, nbytes):
    """The same bytes, starting `nbytes` behind a 16-byte boundary."""
    buf = torch.zeros(t.numel() + 16, dtype=t.dtype, device="cuda")
    out = buf[nbytes:nbytes + t.numel()].view(t.shape)
    out.copy_(t)
    assert out.data_ptr() % 16 == nbytes
    return out


def same(y, acc, acc_ref, y_ref):
    torch.cuda.synchronize()
    assert np.array_equal(acc.cpu().numpy(), acc_ref)
    assert np.all(np.abs(y.cpu().numpy().astype(np.float64) - y_ref) <= REL * np.abs(y_ref))


# plan of the 2-bit part (its K < 20 is a single stage: no split), plan of the 1.60-bit part, shift of the blob
@pytest.mark.parametrize("plan,plan5,shift", [((16, 2, 0, 1), (0, 0), 0), ((4, 1, 14, 1), (0, 0), 0), ((0, 0, 0, 0), (2, 3), 0),
                                              ((0, 0, 0, 0), (9, 1), 0), ((8, 3, 0, 1), (1, 2), 0), ((0, 0, 0, 0), (0, 0), 4)])
@pytest.mark.parametrize("M,K,N", [(257, 116, 33), (300, 4096, 40), (64, 16, 8), (130, 2560, 17), (101, 6912, 1), (48, 1036, 130)])
def test_mixed_packing_through_the_lookup_kernels(B, M, K, N, plan, plan5, shift):
    print(f"mixed case M={M} K={K} N={N} plan={plan} plan5={plan5} shift={shift}", flush=True)
    W, s, x = wl.small_case(2200 + M + N, M, K, N)
    _, _, acc_ref, y_ref = O.mpgemm(W, s, x)
    blob = shifted(B.pack_weights_mixed(dev(W)), shift)
    a_q, a_s = B.quantize_act(dev(x))
    B.set_plan(*plan)
    B.set_plan_g5(*plan5)
    try:
        try:
            kernel = B.query_kernel("mixed", M, K, N)
        except B.VlutError as e:                            # a split or R that this K does not admit
            assert e.status == B.VLUT_ERR_UNSUPPORTED and plan5 != (0, 0)
            with pytest.raises(B.VlutError):
                B.mpgemm_mixed(blob, float(s), a_q, a_s, M)
            return
        assert kernel == ("matrix" if shift else "lookup")  # (the query speaks of aligned operands)
        y, acc = B.mpgemm_mixed(blob, float(s), a_q, a_s, M, want_acc=True)
    finally:
        B.set_plan(0, 0, 0, 0)
        B.set_plan_g5(0, 0)
    same(y, acc, acc_ref, y_ref)


@pytest.mark.parametrize("M,K,N", [(257, 260, 33), (70, 1020, 7), (5, 20, 1), (300, 5120, 40)])
@pytest.mark.parametrize("shift_w,shift_a", [(4, 0), (0, 8), (4, 8)])
def test_1_60_bit_packing_with_unaligned_operands(B, M, K, N, shift_w, shift_a):
    print(f"g5 case M={M} K={K} N={N} shifts {shift_w} {shift_a}", flush=True)
    W, s, x = wl.small_case(2300 + M + N, M, K, N)
    _, _, acc_ref, y_ref = O.mpgemm(W, s, x)
    a_q, a_s = B.quantize_act(dev(x))
    y, acc = B.mpgemm_g5(shifted(B.pack_weights_g5(dev(W)), shift_w), float(s), shifted(a_q, shift_a), a_s, M, want_acc=True)
    same(y, acc, acc_ref, y_ref)


@pytest.mark.parametrize("M,K,N", [(70, 5, 3), (257, 1285, 33), (33, 2555, 64)])
def test_1_60_bit_packing_with_k_that_four_does_not_divide(B, M, K, N):
    # (codes that did not come from the quantiser, which wants K % 4 == 0)
    print(f"g5 case M={M} K={K} N={N}", flush=True)
    assert B.query_kernel("g5", M, K, N) == "lookup"
    W = wl.ternary(2400 + M, M, K, 0.4)
    rng = np.random.default_rng(K)
    q = rng.integers(-127, 128, (K, N), dtype=np.int8)
    sc = rng.random(N, dtype=np.float32) + np.float32(0.5)
    chunked = np.zeros(((N + 7) // 8, K, 8), np.int8)
    for n in range(N):
        chunked[n // 8, :, n % 8] = q[:, n]
    acc_ref = O.gemm_acc(W, q)
    y, acc = B.mpgemm_g5(B.pack_weights_g5(dev(W)), 0.25, dev(chunked), dev(sc), M, want_acc=True)
    same(y, acc, acc_ref, O.epilogue(acc_ref, np.float32(0.25), sc))


@pytest.mark.parametrize("M,K,N,kernel", [(64, 16384, 40, "lookup"), (16, 32768, 33, "lookup"), (200, 16384, 48, "lookup"), (640, 30000, 33, "lookup"),
                                          (1027, 20480, 21, "lookup"), (200, 14336, 64, "matrix"), (640, 16384, 128, "matrix"), (640, 2560, 40, "matrix")])
def test_long_rows_of_few_outputs(B, M, K, N, kernel):
    # both sides of the rule that compares the lookup kernel (K split over workgroups) with the matrix cores
    print(f"codes case {kernel} M={M} K={K} N={N}", flush=True)
    assert B.query_kernel("codes", M, K, N) == kernel
    W, s, x = wl.small_case(2500 + M + N, M, K, N)
    _, _, acc_ref, y_ref = O.mpgemm(W, s, x)
    a_q, a_s = B.quantize_act(dev(x))
    packed = B.pack_weights(dev(W))
    y, acc = B.mpgemm(packed, float(s), a_q, a_s, M, want_acc=True)
    same(y, acc, acc_ref, y_ref)
    y1, acc1, _ = B.mpgemm_f32(packed, float(s), dev(x), M, want_acc=True)
    same(y1, acc1, acc_ref, y_ref)
    assert torch.equal(y, y1)


# 32 to 256 rows per workgroup: for pairs of more than sixteen tokens, and for two tokens with N * K beyond the matrix-core kernel's bound
@pytest.mark.parametrize("M,K,N,rows", [(700, 516, 20, 32), (1500, 516, 19, 64), (3000, 516, 20, 128), (6000, 516, 20, 256), (100, 1028, 32, 32),
                                        (130, 36864, 2, 32), (8201, 32772, 2, 64), (16390, 32772, 2, 128), (40001, 1028, 2, 256)])
def test_few_token_table_kernel_from_fp32(B, M, K, N, rows):
    print(f"few-token case M={M} K={K} N={N} rows={rows}", flush=True)
    assert B.query_kernel("f32", M, K, N) == "few_tokens" and B.query_plan_f32(M, K, N)[1] == rows
    gen = torch.Generator(device="cuda")
    gen.manual_seed(2600 + M)
    Wd = torch.randint(-1, 2, (M, K), dtype=torch.int8, generator=gen, device="cuda")
    x = wl.activations(2600 + N, N, K)
    _, s_ref, acc_ref, y_ref = O.mpgemm(Wd.cpu().numpy(), np.float32(0.5), x)
    packed = B.pack_weights(Wd)
    odd = torch.full((N, K + 3), 9e9, device="cuda")
    odd[:, 1:K + 1] = dev(x)
    for xd in (dev(x), odd[:, 1:K + 1]):
        y, acc, sc = B.mpgemm_f32(packed, 0.5, xd, M, want_acc=True, want_scales=True)
        same(y, acc, acc_ref, y_ref)
        assert np.array_equal(sc.cpu().numpy().view(np.uint32), s_ref.view(np.uint32))
