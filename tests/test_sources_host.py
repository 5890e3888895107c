"""What the kernels' sources have to hold that no result shows: stray reads meet zero weights, misstated alignments happen to work."""
import glob
import os
import re
import subprocess

import pytest

from paper_2512_06443_amd.build import HIPCC_FLAGS
from tests.conftest import ROOT

CSRC = os.path.join(ROOT, "paper_2512_06443_amd", "csrc")


def test_loads_behind_a_descriptor_have_no_scalar_offset():
    """The length of a descriptor is what keeps the tails of K inside the tensors.  Whether it is checked against an offset with or without the
    load's scalar offset is described both ways, so none of these loads has one."""
    text = "\n".join(open(f).read() for f in sorted(glob.glob(os.path.join(CSRC, "*"))))
    written_out = re.findall(r'buffer_load\w* %\d, %\d, (\S+) ', text)
    assert written_out and set(written_out) == {"0"}
    by_builtin = re.findall(r"__builtin_amdgcn_raw_buffer_load_\w+\([^;]*?, \(int\)at, (\w+), \w+\)", text)
    assert len(by_builtin) == text.count("__builtin_amdgcn_raw_buffer_load_") > 0 and set(by_builtin) == {"0"}


def test_wide_stores_of_outputs_state_the_alignment_that_callers_owe(tmp_path):
    """y and its rows may start at any float.  The vector stores of a tiled product, as the compiler takes them: aligned to 4 bytes, not to
    the vector's size."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    (tmp_path / "one.hip").write_text("""#include <hip/hip_runtime.h>
#include <cstdint>
#include <type_traits>
#include "common.hip.h"
#include "prepare_kernels.hip.h"
#include "gemm_kernel.hip.h"
#include "gemm_ring_kernel.hip.h"
void* both[] = {(void*)gemm_kernel<5, 2, 4, 4, 2>, (void*)gemm_ring_kernel<2, 2, 2, 4>};
""")
    out = subprocess.run([hipcc, *[f for f in HIPCC_FLAGS if f != "-shared"], "-I", os.path.join(ROOT, "include"), "-I", CSRC, "--offload-device-only", "-S", "-emit-llvm",
                          str(tmp_path / "one.hip"), "-o", str(tmp_path / "one.ll")], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert out.returncode == 0, out.stdout
    stores = re.findall(r"store <([24]) x float> .*, ptr addrspace\(1\) .*, align (\d+)", (tmp_path / "one.ll").read_text())
    assert set(stores) == {("2", "4"), ("4", "4")}
