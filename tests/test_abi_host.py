"""Host-only checks of the C ABI: the library loads without a GPU, exports every symbol that
include/vlut.h declares, its size helpers match the closed forms the paper gives, and every
argument error is reported before any HIP call."""
import ctypes
import os
import re

import pytest

from tests.conftest import ROOT

i64, sz, vp, ci, cf = ctypes.c_int64, ctypes.c_size_t, ctypes.c_void_p, ctypes.c_int, ctypes.c_float


@pytest.fixture(scope="module")
def L(vlut_lib_path):
    lib = ctypes.CDLL(vlut_lib_path)
    lib.vlut_status_string.argtypes, lib.vlut_status_string.restype = [ci], ctypes.c_char_p
    lib.vlut_packed_weight_bytes.argtypes, lib.vlut_packed_weight_bytes.restype = [i64, i64], sz
    lib.vlut_packed_offset.argtypes, lib.vlut_packed_offset.restype = [i64, i64, i64, i64], sz
    lib.vlut_lut_bytes.argtypes, lib.vlut_lut_bytes.restype = [i64, i64], sz
    lib.vlut_act_bytes.argtypes, lib.vlut_act_bytes.restype = [i64, i64], sz
    lib.vlut_workspace_bytes.argtypes, lib.vlut_workspace_bytes.restype = [i64, i64, i64], sz
    lib.vlut_pack_weights.argtypes = [vp, i64, i64, vp, sz, vp]
    lib.vlut_quantize_act.argtypes = [vp, i64, i64, i64, vp, vp, vp]
    lib.vlut_build_lut.argtypes = [vp, i64, i64, vp, sz, vp]
    g = [vp, cf, vp, vp, vp, i64, i64, i64, vp, i64, vp, vp, sz, vp]
    lib.vlut_mpgemm.argtypes = g
    lib.vlut_mpgemm_mfma.argtypes = g
    lib.vlut_mpgemm_rows.argtypes = [vp, vp] + g[2:]
    lib.vlut_set_plan.argtypes = [ci, ci, ci, ci]
    lib.vlut_query_lookup_waves.argtypes = [i64, i64, i64]
    lib.vlut_packed_weight_bytes_g5.argtypes, lib.vlut_packed_weight_bytes_g5.restype = [i64, i64], sz
    lib.vlut_packed_offset_g5.argtypes, lib.vlut_packed_offset_g5.restype = [i64, i64, i64, i64], sz
    lib.vlut_workspace_bytes_g5.argtypes, lib.vlut_workspace_bytes_g5.restype = [i64, i64, i64], sz
    lib.vlut_pack_weights_g5.argtypes = [vp, i64, i64, vp, sz, vp]
    lib.vlut_mpgemm_g5.argtypes = [vp, cf, vp, vp, i64, i64, i64, vp, i64, vp, vp, sz, vp]
    lib.vlut_set_plan_g5.argtypes = [ci, ci]
    lib.vlut_query_plan_g5.argtypes = [i64, i64, i64, ctypes.POINTER(ci)]
    lib.vlut_query_plan.argtypes = [i64, i64, i64, ctypes.POINTER(ci)]
    lib.vlut_mixed_k5.argtypes, lib.vlut_mixed_k5.restype = [i64], i64
    lib.vlut_packed_weight_bytes_mixed.argtypes, lib.vlut_packed_weight_bytes_mixed.restype = [i64, i64], sz
    lib.vlut_workspace_bytes_mixed.argtypes, lib.vlut_workspace_bytes_mixed.restype = [i64, i64, i64], sz
    lib.vlut_pack_weights_mixed.argtypes = [vp, i64, i64, vp, sz, vp]
    lib.vlut_mpgemm_mixed.argtypes = [vp, cf, vp, vp, i64, i64, i64, vp, i64, vp, vp, sz, vp]
    lib.vlut_workspace_bytes_f32.argtypes, lib.vlut_workspace_bytes_f32.restype = [i64, i64, i64], sz
    lib.vlut_query_plan_f32.argtypes = [i64, i64, i64, ctypes.POINTER(ci)]
    lib.vlut_mpgemm_f32.argtypes = [vp, cf, vp, vp, i64, i64, i64, i64, vp, i64, vp, vp, vp, sz, vp]
    return lib


def test_every_declared_symbol_is_exported(L):
    header = open(os.path.join(ROOT, "include", "vlut.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    names = sorted(set(re.findall(r"\b(vlut_[a-z0-9_]+)\s*\(", header)))
    assert {"vlut_pack_weights", "vlut_quantize_act", "vlut_build_lut", "vlut_mpgemm"} <= set(names)
    for n in names:
        assert hasattr(L, n), f"{n} declared in vlut.h but not exported"
    from paper_2512_06443_amd import binding
    assert set(binding.EXPORTS) == set(names)


def test_status_strings(L):
    assert L.vlut_status_string(0) == b"VLUT_OK"
    seen = {L.vlut_status_string(c) for c in range(-6, 1)}
    assert len(seen) == 7 and all(s for s in seen)
    assert L.vlut_status_string(-99).startswith(b"VLUT_ERR")


def test_size_helpers(L, golden):
    # 2.00 bits per weight when the shape needs no padding (Sec. 4: I2 = b2.00)
    assert L.vlut_packed_weight_bytes(6912, 2560) == 6912 * 2560 // 4
    assert L.vlut_packed_weight_bytes(256, 256) == 16384
    # padding to 4 rows x 16 groups
    assert L.vlut_packed_weight_bytes(257, 260) == 65 * 5 * 64
    assert L.vlut_packed_weight_bytes(1, 4) == 64
    for bad in [(0, 4), (4, 0), (4, 6), (-1, 8), (1 << 24, 4)]:
        assert L.vlut_packed_weight_bytes(*bad) == 0
    # the paper's full-table example (Sec. 1): 4096 x 14436 x 512 -> 285.5 MiB
    K, N = int(golden["full_lut_K"][0]), int(golden["full_lut_N"][0])
    assert round(L.vlut_lut_bytes(K, N) / 2 ** 20, 1) == float(golden["full_lut_mib"][0])
    assert L.vlut_lut_bytes(256, 8) == 64 * 81 * 8 * 2
    assert L.vlut_act_bytes(2560, 128) == 2560 * 128 and L.vlut_act_bytes(64, 9) == 2 * 64 * 8
    assert L.vlut_act_bytes(6, 8) == 0
    assert L.vlut_lut_bytes(6, 8) == 0 and L.vlut_lut_bytes(8, 0) == 0
    assert L.vlut_workspace_bytes(0, 8, 8) == 0


def test_packed_offset_is_a_bijection(L):
    M, K = 10, 136            # 3 row tiles (padded), 34 groups -> 3 k-tiles (padded)
    total = L.vlut_packed_weight_bytes(M, K)
    assert total == 3 * 3 * 64
    offs = {L.vlut_packed_offset(M, K, m, kg) for m in range(M) for kg in range(K // 4)}
    assert len(offs) == M * (K // 4) and max(offs) < total
    # tile structure: 4 rows x 16 groups contiguous, a row's 16 groups are 16 consecutive bytes
    assert L.vlut_packed_offset(M, K, 0, 1) - L.vlut_packed_offset(M, K, 0, 0) == 1
    assert L.vlut_packed_offset(M, K, 1, 0) - L.vlut_packed_offset(M, K, 0, 0) == 16
    assert L.vlut_packed_offset(M, K, 0, 16) - L.vlut_packed_offset(M, K, 0, 0) == 64
    assert L.vlut_packed_offset(M, K, 4, 0) - L.vlut_packed_offset(M, K, 0, 0) == 3 * 64
    for bad in [(M, 0), (-1, 0), (0, 34), (0, -1)]:
        assert L.vlut_packed_offset(M, K, *bad) == ctypes.c_size_t(-1).value


def test_argument_errors_come_before_any_device_call(L):
    d = 0x1000  # a fake non-null, 16-byte aligned "device pointer": never dereferenced on these paths
    assert L.vlut_pack_weights(None, 8, 8, d, 64, None) == -1
    assert L.vlut_pack_weights(d, 8, 8, None, 64, None) == -1
    assert L.vlut_pack_weights(d, 8, 6, d, 64, None) == -2
    assert L.vlut_pack_weights(d, 0, 8, d, 64, None) == -2
    assert L.vlut_pack_weights(d, 8, 8, d, 63, None) == -3
    assert L.vlut_quantize_act(None, 4, 8, 8, d, d, None) == -1
    assert L.vlut_quantize_act(d, 4, 8, 8, None, d, None) == -1
    assert L.vlut_quantize_act(d, 4, 8, 8, d, None, None) == -1
    assert L.vlut_quantize_act(d, 4, 8, 7, d, d, None) == -2      # ldx < K
    assert L.vlut_quantize_act(d, 0, 8, 8, d, d, None) == -2
    assert L.vlut_quantize_act(d, 4, 10, 10, d, d, None) == -2    # K % 4 != 0
    assert L.vlut_build_lut(None, 8, 4, d, 1 << 20, None) == -1
    assert L.vlut_build_lut(d, 8, 4, None, 1 << 20, None) == -1
    assert L.vlut_build_lut(d, 8, 4, d, 2 * 81 * 4 * 2 - 1, None) == -3
    assert L.vlut_build_lut(d, 9, 4, d, 1 << 20, None) == -2
    L.vlut_mfma_workspace_bytes.argtypes, L.vlut_mfma_workspace_bytes.restype = [i64, i64, i64], sz
    assert L.vlut_mfma_workspace_bytes(8, 6, 4) == 0                      # invalid shape
    assert L.vlut_mfma_workspace_bytes(8, 8, 4) == 0                      # one K step: nothing to split
    need = L.vlut_mfma_workspace_bytes(640, 2560, 16)                     # few tiles, 40 K steps: K is split
    assert need > 0 and need % (640 * 16 * 4) == 0 and need // (640 * 16 * 4) <= 16
    assert L.vlut_mfma_workspace_bytes(14336, 4096, 512) == 0             # enough tiles without a split
    assert L.vlut_mpgemm_mfma(d, 1.0, d, d, None, 640, 2560, 16, d, 640, None, None, 0, None) == -1   # needs its workspace
    assert L.vlut_mpgemm_mfma(d, 1.0, d, d, None, 640, 2560, 16, d, 640, None, d, need - 1, None) == -3
    assert L.vlut_mpgemm_mfma(d, 1.0, d, d, d, 8, 8, 4, d, 8, None, d, 1 << 20, None) == -6        # no materialised table here
    for fn in (L.vlut_mpgemm, L.vlut_mpgemm_mfma):
        assert fn(None, 1.0, d, d, None, 8, 8, 4, d, 8, None, None, 0, None) == -1
        assert fn(d, 1.0, None, d, None, 8, 8, 4, d, 8, None, None, 0, None) == -1
        assert fn(d, 1.0, d, None, None, 8, 8, 4, d, 8, None, None, 0, None) == -1
        assert fn(d, 1.0, d, d, None, 8, 8, 4, None, 8, None, None, 0, None) == -1   # neither y nor acc
        assert fn(d, 1.0, d, d, None, 8, 8, 4, d, 7, None, None, 0, None) == -2      # ldy < M
        assert fn(d, 1.0, d, d, None, 8, 7, 4, d, 8, None, None, 0, None) == -2
        assert fn(d, 1.0, d, d, None, 8, 8, 0, d, 8, None, None, 0, None) == -2
    assert L.vlut_mpgemm_rows(d, None, d, d, None, 8, 8, 4, d, 8, None, None, 0, None) == -1      # row scales are required
    assert L.vlut_mpgemm_rows(None, d, d, d, None, 8, 8, 4, d, 8, None, None, 0, None) == -1
    assert L.vlut_mpgemm_rows(d, d, d, d, None, 8, 8, 4, d, 7, None, None, 0, None) == -2
    assert L.vlut_set_plan(3, 0, 0, 0) == -6 and L.vlut_set_plan(0, 17, 0, 0) == -6
    assert L.vlut_set_plan(0, 0, 7, 0) == -6 and L.vlut_set_plan(0, 0, 0, 99) == -6
    assert L.vlut_set_plan(0, 0, 12, 0) == 0 and L.vlut_set_plan(0, 0, 14, 0) == 0 and L.vlut_set_plan(0, 0, 16, 0) == 0
    assert L.vlut_set_plan(0, 0, 0, 0) == 0
    assert L.vlut_query_plan(8, 8, 8, None) == -1


def test_split_k_needs_a_workspace(L):
    d = 0x1000
    assert L.vlut_set_plan(16, 1, 0, 2) == 0
    try:
        M, K, N = 8, 512, 8
        need = L.vlut_workspace_bytes(M, K, N)
        assert need == 2 * M * N * 4
        assert L.vlut_mpgemm(d, 1.0, d, d, None, M, K, N, d, M, None, None, 0, None) == -1
        assert L.vlut_mpgemm(d, 1.0, d, d, None, M, K, N, d, M, None, d, need - 1, None) == -3
    finally:
        assert L.vlut_set_plan(0, 0, 0, 0) == 0


def test_workspace_size_serves_the_materialised_table_variant_too(L):
    """The size vlut_workspace_bytes reports is accepted by vlut_mpgemm for lut != NULL as well, also where the
    streamed path takes the few-token kernel and needs none (the call then reaches the device step: no GPU here)."""
    d = 0x1000
    for (M, K, N) in [(70, 4352, 9), (640, 2560, 1), (2560, 2560, 4), (300, 8192, 2), (6912, 2560, 16), (300, 4352, 40)]:
        need = L.vlut_workspace_bytes(M, K, N)
        ws = d if need else None
        for lut in (None, d):
            rc = L.vlut_mpgemm(d, 1.0, d, d, lut, M, K, N, d, M, None, ws, need, None)
            assert rc not in (-1, -2, -3, -6), (M, K, N, lut, rc)


def test_override_that_does_not_fit_the_shape_is_an_error(L):
    d = 0x1000
    out = (ci * 4)()
    try:
        # K = 16384: 4096 groups; J = 1 -> 4 groups per stage, 1024 stages x 4 lookups per lane > 64 -> R <= 6 only
        assert L.vlut_set_plan(1, 9, 0, 1) == 0
        assert L.vlut_query_plan(300, 16384, 40, out) == -6
        assert L.vlut_mpgemm(d, 1.0, d, d, None, 300, 16384, 40, d, 300, None, None, 0, None) == -6
        assert L.vlut_workspace_bytes(300, 16384, 40) == 0
        # more K splits than stages: K = 256 -> 64 groups = one stage at J = 16
        assert L.vlut_set_plan(16, 2, 0, 4) == 0
        assert L.vlut_query_plan(300, 256, 40, out) == -6
        assert L.vlut_mpgemm(d, 1.0, d, d, None, 300, 256, 40, d, 300, None, d, 1 << 20, None) == -6
        assert L.vlut_set_plan(16, 2, 0, 1) == 0
        assert L.vlut_query_plan(300, 256, 40, out) == 0 and tuple(out)[:3] == (16, 2, 1)
    finally:
        assert L.vlut_set_plan(0, 0, 0, 0) == 0
    out3 = (ci * 3)()
    try:
        assert L.vlut_set_plan_g5(2, 4) == 0
        assert L.vlut_query_plan_g5(300, 320, 40, out3) == -6                  # 64 groups = one stage, four splits asked
    finally:
        assert L.vlut_set_plan_g5(0, 0) == 0


def test_packed_blob_must_be_16_byte_aligned(L):
    d, odd = 0x1000, 0x1004
    assert L.vlut_mpgemm(odd, 1.0, d, d, None, 8, 64, 40, d, 8, None, None, 0, None) == -6
    assert L.vlut_mpgemm_rows(odd, d, d, d, None, 8, 64, 40, d, 8, None, None, 0, None) == -6
    assert L.vlut_mpgemm_f32(odd, 1.0, None, d, 64, 8, 64, 40, d, 8, None, None, d, 1 << 20, None) == -6


def test_plans_cover_all_benchmark_shapes(L):
    out = (ci * 4)()
    shapes = [(256, 256, 8), (6912, 2560, 128), (8640, 3200, 256), (3200, 8640, 256), (4096, 4096, 512),
              (14336, 4096, 512), (4096, 14336, 512)]
    shapes += [(m, k, n) for (m, k) in [(2560, 2560), (640, 2560), (6912, 2560), (2560, 6912)]
               for n in (1, 2, 3, 4, 7, 8, 16, 24, 32, 33, 64, 256, 1024)]
    for (M, K, N) in shapes:
        assert L.vlut_query_plan(M, K, N, out) == 0
        J, R, S, tiles = list(out)
        if J == 0:                                     # the few-token kernel: R = rows per workgroup, a grid per token pair
            pairs = (N + 1) // 2
            assert N <= 32 and R in (32, 64, 128, 256) and S == 1 and tiles % pairs == 0 and (tiles // pairs) * R >= M
            # more than two tokens: one round of workgroups, and cheaper than the general path by the library's estimate
            per_chunk = {32: 0.9, 64: 1.35, 128: 2.0, 256: 3.4}[R]
            c = K / 1024
            assert N <= 2 or (tiles <= 256 and (3.6 + c * per_chunk) * 1.1 < 5.8 + 0.94 * c + 0.41 * M * N / 1e4)
            assert L.vlut_workspace_bytes(M, K, N) == 0 and L.vlut_query_lookup_waves(M, K, N) == 0
            continue
        assert N > 2
        assert J in (1, 2, 4, 8, 16) and 1 <= R <= 16 and 1 <= S <= 16 and tiles >= 1
        n_tile = 128 // J
        tiles_n = -(-N // n_tile)
        assert tiles % (tiles_n * S) == 0
        tiles_m = tiles // (tiles_n * S)
        waves = L.vlut_query_lookup_waves(M, K, N)
        assert waves in (12, 14)
        assert tiles_m * 4 * waves * R >= M                            # every row is covered (lookup waves x 4 rows x R)


def test_g5_host_logic(L):
    """1.60-bit packing: sizes (Sec. 3.3: 5 weights per byte, g | K), layout bijection, argument checks, plan coverage."""
    assert L.vlut_packed_weight_bytes_g5(6912, 2560) == 6912 * 512             # 1.60 bits per weight, no padding needed
    assert L.vlut_packed_weight_bytes_g5(6912, 2560) * 5 == L.vlut_packed_weight_bytes(6912, 2560) * 4
    assert L.vlut_packed_weight_bytes_g5(5, 100) == 2 * 2 * 64                 # rows padded to 4, groups to 16
    assert L.vlut_packed_weight_bytes_g5(8, 64) == 0 and L.vlut_packed_weight_bytes_g5(0, 80) == 0
    M, K = 10, 100
    offs = {L.vlut_packed_offset_g5(M, K, m, kg) for m in range(M) for kg in range(K // 5)}
    assert len(offs) == M * (K // 5) and max(offs) < L.vlut_packed_weight_bytes_g5(M, K)
    assert L.vlut_packed_offset_g5(M, K, M, 0) == 2 ** 64 - 1 and L.vlut_packed_offset_g5(M, K, 0, K // 5) == 2 ** 64 - 1
    d = ctypes.c_void_p(0x1000)                                                # never dereferenced: checks come first
    assert L.vlut_pack_weights_g5(None, 8, 80, d, 1 << 20, None) == -1
    assert L.vlut_pack_weights_g5(d, 8, 64, d, 1 << 20, None) == -2            # 5 does not divide 64
    assert L.vlut_pack_weights_g5(d, 8, 80, d, 63, None) == -3
    assert L.vlut_mpgemm_g5(None, 1.0, d, d, 8, 80, 4, d, 8, None, None, 0, None) == -1
    assert L.vlut_mpgemm_g5(d, 1.0, d, d, 8, 80, 4, None, 8, None, None, 0, None) == -1
    assert L.vlut_mpgemm_g5(d, 1.0, d, d, 8, 82, 4, d, 8, None, None, 0, None) == -2
    assert L.vlut_mpgemm_g5(d, 1.0, d, d, 8, 80, 4, d, 7, None, None, 0, None) == -2
    assert L.vlut_set_plan_g5(3, 0) == -6 and L.vlut_set_plan_g5(0, 17) == -6
    out = (ci * 3)()
    try:
        assert L.vlut_set_plan_g5(2, 4) == 0
        need = L.vlut_workspace_bytes_g5(300, 5120, 40)
        assert need == 4 * 300 * 40 * 4
        assert L.vlut_mpgemm_g5(d, 1.0, d, d, 300, 5120, 40, d, 300, None, None, 0, None) == -1
        assert L.vlut_mpgemm_g5(d, 1.0, d, d, 300, 5120, 40, d, 300, None, d, need - 1, None) == -3
    finally:
        assert L.vlut_set_plan_g5(0, 0) == 0
    for (M, K, N) in [(6912, 2560, 128), (8640, 3200, 256), (3200, 8640, 256), (2560, 2560, 1), (640, 2560, 1024)]:
        assert L.vlut_query_plan_g5(M, K, N, out) == 0
        R, S, tiles = out[0], out[1], out[2]
        assert R in (1, 2, 4, 6, 9, 12, 14) and 1 <= S <= 16 and tiles >= 1
        stages = -(-(K // 5) // 64)
        per_split = -(-stages // S)
        assert per_split * 4 <= 51 or R <= 6                                   # INT16 block bound of Sec. 3.4
        tiles_m = tiles // (S * -(-N // 8))
        assert tiles_m * 48 * R >= M                                           # the tiles cover every row


def test_f32_entry_host_logic(L):
    """vlut_mpgemm_f32: which kernels it picks, what workspace that needs, and argument errors before any device call."""
    out = (ci * 5)()
    # a few tokens: the kernel that sweeps all of K, quantising inside, a copy of the row tiles per token pair; no
    # workspace
    for (M, K, N) in [(6912, 2560, 1), (2560, 6912, 2), (640, 2560, 1), (6912, 2560, 3), (6912, 2560, 8), (640, 2560, 32)]:
        assert L.vlut_query_plan_f32(M, K, N, out) == 0
        assert out[0] == 0 and out[2] == 1 and out[4] == 1
        assert L.vlut_workspace_bytes_f32(M, K, N) == 0
    # more tokens: quantised once, by a kernel of its own ahead of the lookups; the workspace then holds the scales,
    # the INT8 activations and the split-K partial sums of the ordinary path
    for (M, K, N) in [(6912, 2560, 128), (14336, 4096, 512), (4096, 14336, 512), (3200, 8640, 256), (6912, 2560, 24), (2560, 6912, 24), (640, 2560, 33)]:
        assert L.vlut_query_plan_f32(M, K, N, out) == 0
        assert out[4] == 0
        r256 = lambda v: (v + 255) // 256 * 256
        amax = r256(4 * N) if (N * K >= 1 << 22 and N >= 64) else 0      # scratch between the two kernels of the quantiser
        assert L.vlut_workspace_bytes_f32(M, K, N) == r256(4 * N) + amax + r256(L.vlut_act_bytes(K, N)) + L.vlut_workspace_bytes(M, K, N)
    # a forced plan with 16 sub-tables per table row selects the fused kernel when the K range fits next to the
    # tables (34 stages of 256 values), with the scales in front of the split-K partial sums
    try:
        assert L.vlut_set_plan(16, 2, 0, 4) == 0
        assert L.vlut_query_plan_f32(300, 14336, 40, out) == 0 and tuple(out) == (16, 2, 4, 4 * 4 * 5, 1)
        assert L.vlut_workspace_bytes_f32(300, 14336, 40) == 256 + 4 * 300 * 40 * 4
        assert L.vlut_set_plan(16, 2, 0, 1) == 0
        assert L.vlut_query_plan_f32(300, 14336, 40, out) == 0 and out[4] == 0     # 56 stages in one range
        assert L.vlut_set_plan(8, 2, 0, 1) == 0
        assert L.vlut_query_plan_f32(300, 2560, 40, out) == 0 and out[4] == 0      # 16-token tiles
    finally:
        assert L.vlut_set_plan(0, 0, 0, 0) == 0
    d = ctypes.c_void_p(0x1000)                                                # never dereferenced: checks come first
    ok = [d, 1.0, None, d, 2560, 6912, 2560, 1, d, 6912, None, None, None, 0, None]
    def call(**kw):
        names = ["packed", "w_scale", "rows", "x", "ldx", "M", "K", "N", "y", "ldy", "acc", "scales", "ws", "ws_bytes", "stream"]
        a = list(ok)
        for k, v in kw.items():
            a[names.index(k)] = v
        return L.vlut_mpgemm_f32(*a)
    assert call(packed=None) == -1 and call(x=None) == -1 and call(y=None) == -1
    assert call(ldx=2559) == -2 and call(ldy=6911) == -2 and call(K=2562) == -2 and call(N=0) == -2
    assert call(M=14336, K=4096, N=512, ldx=4096, ldy=14336) == -1             # needs a workspace
    need = L.vlut_workspace_bytes_f32(14336, 4096, 512)
    assert call(M=14336, K=4096, N=512, ldx=4096, ldy=14336, ws=d, ws_bytes=need - 1) == -3
    assert call(M=14336, K=4096, N=512, ldx=4096, ldy=14336, ws=ctypes.c_void_p(0x1004), ws_bytes=need) == -6
    assert L.vlut_query_plan_f32(8, 8, 8, None) == -1 and L.vlut_query_plan_f32(8, 6, 8, out) == -2
    assert L.vlut_workspace_bytes_f32(8, 6, 8) == 0


def test_mixed_packing_host_logic(L):
    """Mixed 1.60-bit / 2-bit packing (Sec. 3.3): how K is divided, blob sizes, bits per weight, argument checks."""
    assert [L.vlut_mixed_k5(K) for K in (4, 16, 20, 36, 2560, 4096, 6912, 14336)] == [0, 0, 20, 20, 2560, 4080, 6900, 14320]
    assert L.vlut_mixed_k5(0) == -1 and L.vlut_mixed_k5(18) == -1
    for (M, K) in [(6912, 2560), (14336, 4096), (4096, 14336), (2560, 6912), (8, 16), (8, 36)]:
        K5 = L.vlut_mixed_k5(K)
        want = (L.vlut_packed_weight_bytes_g5(M, K5) if K5 else 0) + (L.vlut_packed_weight_bytes(M, K - K5) if K > K5 else 0)
        assert L.vlut_packed_weight_bytes_mixed(M, K) == want
        if K >= 2560:                                      # "near-1.6-bit" (Sec. 3.3): the 2-bit part is one tile column
            assert 1.6 <= want * 8 / (M * K) < 1.65
            assert want < L.vlut_packed_weight_bytes(M, K) * 0.82
        assert L.vlut_workspace_bytes_mixed(M, K, 8) >= (1 + (K > K5 > 0)) * M * 8 * 4
    assert L.vlut_packed_weight_bytes_mixed(8, 18) == 0 and L.vlut_workspace_bytes_mixed(8, 18, 8) == 0
    d = ctypes.c_void_p(0x1000)                                                # never dereferenced: checks come first
    assert L.vlut_pack_weights_mixed(None, 8, 36, d, 1 << 20, None) == -1
    assert L.vlut_pack_weights_mixed(d, 8, 18, d, 1 << 20, None) == -2
    assert L.vlut_pack_weights_mixed(d, 8, 36, d, 100, None) == -3
    assert L.vlut_mpgemm_mixed(None, 1.0, d, d, 8, 36, 4, d, 8, None, d, 1 << 20, None) == -1
    assert L.vlut_mpgemm_mixed(d, 1.0, d, d, 8, 36, 4, None, 8, None, d, 1 << 20, None) == -1
    assert L.vlut_mpgemm_mixed(d, 1.0, d, d, 8, 38, 4, d, 8, None, d, 1 << 20, None) == -2
    assert L.vlut_mpgemm_mixed(d, 1.0, d, d, 8, 36, 4, d, 7, None, d, 1 << 20, None) == -2
    assert L.vlut_mpgemm_mixed(d, 1.0, d, d, 8, 36, 4, d, 8, None, None, 0, None) == -1        # the workspace is required
    assert L.vlut_mpgemm_mixed(d, 1.0, d, d, 8, 36, 4, d, 8, None, d, 16, None) == -3


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_binding_imports_without_the_private_stream_functions(monkeypatch, missing):
    """A torch without a GPU build has neither of the two functions the stream handle is taken from; the module still
    imports there and its size helpers work."""
    import importlib.util

    import torch
    from paper_2512_06443_amd import binding
    monkeypatch.delattr(torch._C, missing)
    spec = importlib.util.spec_from_file_location("binding_without_gpu_build", binding.__file__)
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    assert mod.packed_weight_bytes(256, 256) == 16384
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: type("S", (), {"cuda_stream": 77})())
    assert mod._stream() == 77


def test_queries_name_the_kernel_that_runs(L):
    """vlut_query_plan_f32 tells one launch from two also where the matrix cores take a few tokens from fp32, and
    vlut_query_kernel names the kernel of every form of the call, with and without an override."""
    L.vlut_query_kernel.argtypes = [ci, i64, i64, i64]
    codes, f32, g5, mixed = range(4)
    lookup, few, matrix, matrix_few = 1, 2, 3, 4
    out = (ci * 5)()
    for (M, K, N, rows) in [(4096, 6552, 10, 16), (4097, 2560, 16, 32), (13824, 2560, 16, 64), (32768, 2560, 16, 128)]:
        assert L.vlut_query_kernel(f32, M, K, N) == matrix_few                 # one launch, 16 to 128 rows per workgroup
        assert L.vlut_query_plan_f32(M, K, N, out) == 0
        assert tuple(out) == (0, rows, 1, -(-M // rows), 1)
    assert L.vlut_query_plan_f32(2560, 6912, 16, out) == 0 and out[4] == 0     # N * K beyond 65536: two launches
    assert L.vlut_query_plan_f32(32769, 2560, 16, out) == 0 and out[4] == 0
    assert L.vlut_query_kernel(f32, 2560, 6912, 16) == L.vlut_query_kernel(codes, 2560, 6912, 16)
    for (M, K, N) in [(14336, 4096, 512), (4096, 14336, 512), (3203, 3116, 77), (6912, 2560, 128)]:
        assert L.vlut_query_kernel(codes, M, K, N) == L.vlut_query_kernel(f32, M, K, N) == matrix
        assert L.vlut_query_kernel(mixed, M, K, N) == matrix
    assert L.vlut_query_kernel(codes, 640, 2560, 4) == few
    assert L.vlut_query_kernel(g5, 640, 2560, 4) == matrix and L.vlut_query_kernel(g5, 640, 2555, 4) == lookup   # 4 does not divide K
    assert L.vlut_query_kernel(mixed, 64, 16, 8) == matrix
    try:
        assert L.vlut_set_plan(16, 2, 0, 1) == 0
        for form in (codes, f32, mixed):
            assert L.vlut_query_kernel(form, 300, 2560, 40) == lookup
        assert L.vlut_query_kernel(g5, 300, 2560, 40) == matrix                # the other packing has an override of its own
        assert L.vlut_set_plan(16, 2, 0, 4) == 0
        assert L.vlut_query_kernel(codes, 300, 256, 40) == -6                  # more K splits than stages
        assert L.vlut_set_plan(0, 0, 0, 0) == 0 and L.vlut_set_plan_g5(2, 1) == 0
        assert L.vlut_query_kernel(g5, 300, 2560, 40) == L.vlut_query_kernel(mixed, 300, 2560, 40) == lookup
        assert L.vlut_query_kernel(codes, 300, 2560, 40) == matrix
    finally:
        assert L.vlut_set_plan(0, 0, 0, 0) == 0 and L.vlut_set_plan_g5(0, 0) == 0
    assert L.vlut_query_kernel(codes, 8, 6, 8) == -2 and L.vlut_query_kernel(g5, 8, 64, 8) == -2
    assert L.vlut_query_kernel(4, 8, 64, 8) == -6


def test_bench_line_is_one_line_that_fits(L):
    """The line of the default run (41 shapes, five layers) is complete within the last 12 kB of the output."""
    import json

    import bench
    f = 0.12345678901234567
    entry = {"workload": "layer2b4_nsweep", "linear": "gateup", "M": 14336, "K": 14336, "N": 1024, "seed": 4,
             "kernel": "matrix_few_tokens", "one_launch_from_fp32": True, "bound": "mfma"}
    entry.update({k: f for k in ("ms", "kernel_ms", "two_call_ms", "mpgemm_ms", "floor_ms", "frac", "kernel_frac", "mfma_ms",
                                 "lut_over_mfma_time", "mfma_frac_of_int8_peak")}, GOPS=123456.78901234567, weight_stream_GBs=1234.5678901234567)
    layer = {"N": 1024, "seed": 4, "launches": 4, "what": "w" * 80, "kernels": ["matrix_few_tokens"] * 4, "ms": f, "gpu_ms": f, "GOPS": 123456.78901234567,
             "weight_stream_GBs": 1234.5678901234567, "bound": "mfma", "floor_ms": f, "frac": f}
    out = {"metric": "m", "value": 723456.78901234567, "config": {"workload": "x" * 600}, "roofline": {"what": "x" * 900},
           "sweep": [dict(entry) for _ in range(41)], "layer": [dict(layer) for _ in range(5)]}
    line = bench.json_line(out)
    assert "\n" not in line and len(line) < 12000
    back = json.loads(line)
    assert back["value"] == 723457.0 and len(back["sweep"]["rows"]) == 41
    row = dict(zip(back["sweep"]["columns"], back["sweep"]["rows"][0]))
    assert row["ms"] == 0.123457 and row["kernel"] == "matrix_few_tokens"
    assert len(out["sweep"]) == 41 and isinstance(out["sweep"][0], dict)       # the caller's table is left alone


def test_long_rows_of_few_outputs_take_the_faster_kernel(L):
    """INT8 codes with a long K: the side of the rule on which the times measured when its line was drawn (us, lookup kernel with
    split-K / matrix cores) put a shape, on both sides of 4096 outputs.  gemm_kernel has become faster since: the comment at the rule
    has both sides as they are now."""
    L.vlut_query_kernel.argtypes = [ci, i64, i64, i64]
    lookup, matrix = 1, 3
    measured = [((16, 65532, 33), 23.8, 45.0), ((64, 16384, 40), 10.8, 14.0), ((64, 16384, 128), 10.85, 14.06), ((200, 16384, 48), 11.94, 14.15),
                ((100, 24000, 72), 13.87, 19.37), ((256, 20480, 40), 12.85, 16.78), ((512, 45000, 72), 28.74, 34.41), ((640, 30000, 64), 20.5, 23.83),
                ((1280, 65532, 64), 42.62, 48.48), ((2048, 36000, 20), 23.14, 27.72), ((2560, 20480, 16), 16.4, 17.4), ((2560, 30000, 16), 20.19, 23.87),
                ((4096, 45000, 16), 30.26, 35.91),
                ((256, 14336, 72), 13.39, 12.79), ((640, 16384, 128), 19.99, 14.83), ((640, 30000, 128), 26.82, 25.57), ((1280, 30000, 64), 28.12, 23.87),
                ((2048, 14336, 16), 15.39, 12.91), ((640, 2560, 40), 8.4, 5.9)]
    for shape, t_lookup, t_matrix in measured:
        assert L.vlut_query_kernel(0, *shape) == (lookup if t_lookup < t_matrix else matrix), shape


def test_one_token_on_many_rows_takes_the_table_kernel(L):
    """From fp32, one token: above 16384 rows the table kernel is the faster one while its one launch covers K."""
    L.vlut_query_kernel.argtypes = [ci, i64, i64, i64]
    few, matrix_few = 2, 4
    for M, K, want in [(16384, 4096, matrix_few), (16385, 4096, few), (32768, 1024, few), (32768, 1020, matrix_few), (20000, 14336, few),
                       (32768, 35840, few), (32768, 35844, matrix_few), (32768, 65536, matrix_few), (32769, 64, few), (13824, 2560, matrix_few)]:
        assert L.vlut_query_kernel(1, M, K, 1) == want, (M, K)
        assert L.vlut_workspace_bytes_f32(M, K, 1) == (0 if K <= 35840 else 256 + (8 * K + 255) // 256 * 256)
    assert L.vlut_query_kernel(1, 32768, 4096, 2) == matrix_few


def test_nine_to_sixteen_tokens_on_few_rows_take_the_faster_kernel(L):
    """From fp32: the side of the rule on which the measured times (us, table kernel / matrix cores in one launch) put a shape.  The
    rule does not weigh two launches: the comment at it has their times."""
    L.vlut_query_kernel.argtypes = [ci, i64, i64, i64]
    few, matrix_few = 2, 4
    measured = [((4, 6552, 9), 10.57, 11.52), ((100, 4680, 14), 9.52, 10.3), ((100, 4096, 16), 8.79, 9.15), ((640, 4680, 14), 9.65, 10.39),
                ((1000, 4680, 14), 9.85, 10.44), ((100, 4096, 12), 8.70, 8.24), ((640, 2560, 16), 7.42, 6.93), ((2560, 2560, 16), 9.59, 7.17)]
    for shape, t_table, t_matrix in measured:
        assert L.vlut_query_kernel(1, *shape) == (few if t_table < t_matrix else matrix_few), shape
    assert L.vlut_query_kernel(1, 4, 8188, 8) == matrix_few                    # up to eight tokens two waves share a row: never


def test_matrix_plan_names_the_workgroups_that_run(L):
    """vlut_query_matrix_plan tells the kernels for a few tokens (up to 16 per workgroup) from the tiled product, which
    vlut_query_kernel and vlut_query_plan do not from INT8 codes, and refuses where a kernel that looks up tables runs."""
    L.vlut_query_kernel.argtypes = [ci, i64, i64, i64]
    L.vlut_query_matrix_plan.argtypes = [ci, i64, i64, i64, ctypes.POINTER(ci)]
    codes, f32, g5, mixed = range(4)
    few, matrix = 2, 3
    out = (ci * 4)()

    def plan(*shape):
        rc = L.vlut_query_matrix_plan(*shape, out)
        if rc == 0:
            rows, tokens, parts, workgroups = out
            assert workgroups == -(-shape[1] // rows) * -(-shape[3] // tokens)
            assert tokens in (32, 64, 128) or (tokens <= 16 and rows * parts == 256)       # sixteen waves: row tiles x parts of K
        return tuple(out)[:3] if rc == 0 else rc

    # one kernel behind two names, and another behind one of them
    assert L.vlut_query_kernel(codes, 640, 2560, 4) == few and plan(codes, 640, 2560, 4) == (16, 8, 16)
    assert L.vlut_query_kernel(codes, 2560, 6912, 16) == matrix and plan(codes, 2560, 6912, 16)[1] <= 16
    assert L.vlut_query_kernel(codes, 13824, 2560, 1024) == matrix and plan(codes, 13824, 2560, 1024) == (256, 128, 1)
    assert plan(f32, 2560, 6912, 16) == plan(codes, 2560, 6912, 16)                        # two launches: the same product
    assert plan(f32, 4097, 2560, 16) == (32, 16, 8) and plan(f32, 16384, 4096, 1) == (64, 1, 4) and plan(f32, 64, 64, 3)[1] == 4
    assert plan(g5, 4096, 4000, 16)[1] <= 16 and plan(mixed, 4096, 4096, 256)[1] >= 32 and plan(mixed, 64, 16, 8)[1] <= 16
    # table kernels: K beyond what decode_codes_kernel holds, more rows than it repeats its copy for, K that four do not divide
    for shape in [(codes, 2560, 30000, 2), (codes, 32769, 64, 2), (g5, 640, 2555, 4), (codes, 64, 16384, 40), (f32, 16385, 4096, 1)]:
        assert plan(*shape) == -6, shape
    assert plan(codes, 32768, 14592, 2)[1] == 8
    try:
        assert L.vlut_set_plan(16, 2, 0, 1) == 0
        assert plan(codes, 300, 2560, 40) == plan(f32, 300, 2560, 40) == plan(mixed, 300, 2560, 40) == -6 and isinstance(plan(g5, 300, 2560, 40), tuple)
        assert plan(f32, 4097, 2560, 16) == -6
    finally:
        assert L.vlut_set_plan(0, 0, 0, 0) == 0
    assert L.vlut_query_matrix_plan(codes, 8, 8, 8, None) == -1
    assert plan(codes, 8, 6, 8) == -2 and plan(g5, 8, 64, 8) == -2 and plan(4, 8, 64, 8) == -6
    from paper_2512_06443_amd import binding
    assert binding.query_matrix_plan("codes", 13824, 2560, 1024) == (256, 128, 1, 54 * 8)
    assert binding.query_matrix_plan("codes", 2560, 30000, 2) is None
    with pytest.raises(binding.VlutError):
        binding.query_matrix_plan("codes", 8, 6, 8)


def test_several_rounds_of_five_weights_per_byte_take_the_faster_kernel(L):
    """1.60-bit packing, more workgroups of the kernel for a few tokens than compute units: one of them fills a unit (registers), so
    the side of the rule on which the measured times (us, tiled product / a few tokens) put a shape is the tiled product's."""
    L.vlut_query_kernel.argtypes = [ci, i64, i64, i64]
    out = (ci * 4)()
    measured = [((3079, 360, 233), 4.85, 6.67), ((8624, 1640, 170), 10.96, 13.86), ((12659, 2020, 98), 11.96, 14.99), ((4391, 1320, 219), 7.11, 8.99),
                ((9743, 900, 92), 6.10, 7.39), ((2943, 340, 216), 4.71, 6.46), ((11837, 340, 97), 6.97, 9.12),
                ((4096, 4000, 16), 6.5, 4.8), ((2560, 6900, 8), 7.7, 4.8)]
    for shape, t_tiles, t_few in measured:
        for form in (2, 3):
            assert L.vlut_query_matrix_plan(form, *shape, out) == 0
            assert (out[1] <= 16) == (t_few < t_tiles), (form, shape)


def test_lean_calls_demand_the_workspace_that_is_used(L):
    """No device call: every refusal comes first.  A workspace that the matrix cores leave alone may be NULL in the lean form and only
    there, one that is handed over has to have its size, and what a shape runs is asked for anew when a plan is forced or released."""
    d = 0x1000
    forms = {"": (0, L.vlut_mpgemm_lean, L.vlut_mpgemm, (None,)), "_g5": (2, L.vlut_mpgemm_g5_lean, L.vlut_mpgemm_g5, ()),
             "_mixed": (3, L.vlut_mpgemm_mixed_lean, L.vlut_mpgemm_mixed, ())}
    for suffix, (form, lean, full, lut) in forms.items():
        used, demanded = getattr(L, "vlut_workspace_used" + suffix), getattr(L, "vlut_workspace_bytes" + suffix)
        used.argtypes, used.restype = [i64, i64, i64], sz
        demanded.argtypes, demanded.restype = [i64, i64, i64], sz
        args = [vp, cf, vp, vp] + ([vp] if lut else []) + [i64, i64, i64, vp, i64, vp, vp, sz, vp]
        for f in (lean, full):
            f.argtypes, f.restype = args, ci
        shape = (640, 2560, 77)
        need = demanded(*shape)
        assert need > 0 and used(*shape) == 0
        call = lambda f, ws, size: f(d, 1.0, d, d, *lut, *shape, d, 640, None, ws, size, None)   # noqa: E731
        assert call(full, None, 0) == -1 and call(full, d, need - 1) == call(lean, d, need - 1) == -3
        force, release = (L.vlut_set_plan_g5, (0, 0)) if form == 2 else (L.vlut_set_plan, (0, 0, 0, 0))
        try:
            assert force(*((2, 3) if form == 2 else (16, 2, 0, 3))) == 0
            assert used(*shape) == demanded(*shape) >= 3 * 640 * 77 * 4            # the lookup kernel, K in three parts
            assert call(lean, None, 0) == call(full, None, 0) == -1
        finally:
            assert force(*release) == 0
        assert used(*shape) == 0 and demanded(*shape) == need
        assert used(8, 6, 8) == demanded(8, 6, 8) == 0
    assert L.vlut_workspace_used(64, 16384, 40) == L.vlut_workspace_bytes(64, 16384, 40) > 0     # the lookup kernel's


def test_shapes_that_take_turns_keep_their_own_routes(L):
    """What a shape runs is kept in a table in which shapes replace each other (those of a decoder layer among them): every one is answered
    as if it had been asked for alone."""
    shapes = [(3840, 2560), (2560, 2560), (13824, 2560), (2560, 6912), (640, 2560), (4096, 4096), (14336, 4096), (4096, 14336), (64, 16384)]
    L.vlut_query_kernel.argtypes = [ci, i64, i64, i64]
    L.vlut_query_matrix_plan.argtypes = [ci, i64, i64, i64, ctypes.POINTER(ci)]
    out = (ci * 4)()

    def answer(form, suffix, M, K, N):
        used, demanded = getattr(L, "vlut_workspace_used" + suffix), getattr(L, "vlut_workspace_bytes" + suffix)
        for f in (used, demanded, L.vlut_workspace_bytes_f32):
            f.argtypes, f.restype = [i64, i64, i64], sz
        rc = L.vlut_query_matrix_plan(form, M, K, N, out)
        return L.vlut_query_kernel(form, M, K, N), rc, tuple(out), used(M, K, N), demanded(M, K, N), L.vlut_workspace_bytes_f32(M, K, N)
    cases = [(form, suffix, M, K // 20 * 20 if form == 2 else K, N) for N in (1, 16, 64, 1024) for M, K in shapes
             for form, suffix in ((0, ""), (2, "_g5"), (3, "_mixed"))]
    alone = {}
    for c in cases:
        assert L.vlut_set_plan(0, 0, 0, 0) == 0              # (empties the table)
        alone[c] = answer(*c)
    assert any(a[3] for a in alone.values()) and len(set(alone.values())) > 20
    for _ in range(3):
        for c in cases:
            assert answer(*c) == alone[c], c
