"""What the kernels' sources have to hold that no result shows: stray reads meet zero weights, misstated alignments happen to work."""
import glob
import os
import re

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
