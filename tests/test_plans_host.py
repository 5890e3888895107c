"""The sizes of the GPU tests against the plans that the library makes for them: each runs the workgroup that it is there for, and the
tests run every workgroup that is built."""
import os
import re

import pytest

from tests.conftest import ROOT

pytest.importorskip("torch")


@pytest.fixture(scope="module")
def B(vlut_lib_path):
    from paper_2512_06443_amd import binding
    binding.lib()
    return binding


def built_tiles():
    """(rows, tokens, parts of K) of every row of kGemmTiles, of those that are built for five weights per byte, and of kGemmTilesLong."""
    text = open(os.path.join(ROOT, "paper_2512_06443_amd", "csrc", "gemm_kernel.hip.h")).read()
    four, five, long_k = set(), set(), set()
    for name, tiles in (("kGemmTiles", four), ("kGemmTilesLong", long_k)):
        table = re.search(name + r"\[\] = \{\n(.*?)\n\};", text, flags=re.S).group(1)
        for line in table.splitlines():
            numbers = [float(v) for v in re.findall(r"[0-9.]+", line.split("//")[0])]
            rt, ct, wm, wk = (int(v) for v in numbers[:4])
            tiles.add((32 * rt * wm, 32 * ct, wk))
            if numbers[-1] > 0.0:
                five.add((32 * rt * wm, 32 * ct, wk))
    return four, five, long_k


def test_gpu_tests_run_every_workgroup(B):
    from tests import test_codes_gpu as G
    from tests import test_gemm_gpu as T
    few = {(16 * mt, 8 * ch, 16 // mt) for mt in (1, 2, 4, 8) for ch in (1, 2)}
    four, five, long_k = built_tiles()
    assert len(four) == 8 and len(five) == 5 and len(long_k) == 3
    for form, M, K, N, workgroup in G.WORKGROUPS:
        assert B.query_matrix_plan(form, M, K, N)[:3] == workgroup, (form, M, K, N)
        assert M % workgroup[0] and N % workgroup[1], (form, M, K, N)
    run = {form: {w for f, _, _, _, w in G.WORKGROUPS if f == form} for form in ("codes", "g5", "mixed")}
    assert run["codes"] == few | four and run["g5"] == few | five and run["mixed"] >= five
    # the tile without parts of K, also at sizes whose outputs are stored past the caches
    assert any(w == (256, 128, 1) and 4 * M * N >= 16 << 20 for _, M, _, N, w in G.WORKGROUPS)
    # the tiles from ten macro steps of 128 on: where they divide nothing, and the last step neither
    for M, K, N, workgroup in T.TILES_LOADED_TO_LDS:
        assert B.query_matrix_plan("codes", M, K, N)[:3] == workgroup, (M, K, N)
    assert long_k == {w for M, K, N, w in T.TILES_LOADED_TO_LDS if K > 9 * 128 and M % w[0] and N % w[1] and K % 128}


def test_gpu_tests_run_two_chunks_up_to_their_largest_k(B):
    from tests import test_codes_gpu as G
    for shapes, form, largest in ((G.FEW_TOKENS, "codes", 7168), (G.FEW_TOKENS_FIVE, "mixed", 7360)):
        plans = {s: B.query_matrix_plan(form, *s) for s in shapes}
        two = [s for s, p in plans.items() if p and p[1] == 16]
        assert largest - 4 <= max(K for _, K, _ in two) <= largest and largest in {K for _, K, _ in two}
        assert any(largest < K <= largest + 4 and N > 8 and plans[M, K, N][1] == 8 for M, K, N in shapes)      # one beyond: one chunk
        assert any(K >= largest - 4 and (N + 7) // 8 % 2 == 0 and N % 8 for _, K, N in two)                    # a partly filled second chunk
        assert any((N + 7) // 8 % 2 == 1 for _, _, N in two)                                                    # an absent one


def test_bench_names_the_kernel_of_a_tile():
    """bench.py against the two conditions that choose the kernel (gemm_ring_built, gemm_private_built) for every tile and K it is considered at."""
    import bench
    csrc = os.path.join(ROOT, "paper_2512_06443_amd", "csrc")
    tables = open(os.path.join(csrc, "gemm_kernel.hip.h")).read()

    def condition(name):
        text = open(os.path.join(csrc, f"gemm_{name}_kernel.hip.h")).read()
        c = re.search(rf"gemm_{name}_built\(.*?\) {{ return (.*?); }}", text).group(1)
        return c.replace("&&", "and").replace("||", "or")
    ring, private = condition("ring"), condition("private")
    for name, first, last in (("kGemmTiles", 4, 14336), ("kGemmTilesLong", 1156, 14336)):
        table = re.search(name + r"\[\] = \{\n(.*?)\n\};", tables, flags=re.S).group(1)
        for line in table.splitlines():
            rt, ct, wm, wk = (int(v) for v in re.findall(r"\d+", line)[:4])
            tile = {"gw": 4, "rt": rt, "ct": ct, "wm": wm, "wk": wk}
            want = "gemm_private_kernel" if eval(private, {}, tile) else "gemm_ring_kernel" if eval(ring, {}, tile) else "gemm_kernel"
            for K in (first, last) if (rt, ct) != (2, 2) else (first, 1152):      # 128 x 64 in four parts: two kernels, by K
                assert bench.tiled_kernel(32 * rt * wm, 32 * ct, wk, K) == want, (rt, ct, wm, wk, K)
