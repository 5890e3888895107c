"""build.build(): the library needs hipcc alone; the native form of the binding's calls is built where it can be."""
from __future__ import annotations

import os
import stat
import sys
import warnings

import pytest

from paper_2512_06443_amd import build as b

COMPILER = """#!/bin/sh
[ "$1" = --fails ] && echo no such header && exit 1
while [ $# -gt 1 ]; do [ "$1" = -o ] && echo "$CONTENT" > "$2"; shift; done
exit 0
"""


@pytest.fixture
def scratch(monkeypatch, tmp_path):
    """Compilers that only write their output file, and output files in a scratch folder."""
    compiler = tmp_path / "compiler"
    compiler.write_text(COMPILER)
    compiler.chmod(compiler.stat().st_mode | stat.S_IXUSR)
    monkeypatch.setattr(b, "LIB", str(tmp_path / "lib.so"))
    monkeypatch.setattr(b, "TORCH_LIB", str(tmp_path / "torch.so"))
    monkeypatch.setenv("HIPCC", str(compiler))
    monkeypatch.setenv("CXX", str(compiler))
    monkeypatch.setenv("CONTENT", "new")
    return tmp_path


def test_library_is_built_without_what_only_the_native_calls_need(monkeypatch, scratch):
    (scratch / "fails").write_text(COMPILER.replace('"$1" = --fails', "1"))
    (scratch / "fails").chmod(0o755)
    for missing in ("compiler", "header", "torch"):
        (scratch / "torch.so").write_text("of older sources")
        with monkeypatch.context() as m:
            if missing == "compiler":
                m.setenv("CXX", str(scratch / "none"))
            elif missing == "header":
                m.setenv("CXX", str(scratch / "fails"))
            else:
                m.setitem(sys.modules, "torch", None)
            with pytest.warns(RuntimeWarning, match="Python form"):
                assert b.build() == b.LIB
        assert (scratch / "lib.so").exists() and not (scratch / "torch.so").exists(), missing
        os.remove(b.LIB)


def test_a_library_that_does_not_compile_is_an_error(monkeypatch, scratch):
    (scratch / "fails").write_text("#!/bin/sh\nexit 1\n")
    (scratch / "fails").chmod(0o755)
    monkeypatch.setenv("HIPCC", str(scratch / "fails"))
    with pytest.raises(RuntimeError):
        b.build()


def test_only_what_is_missing_or_stale_is_built(scratch):
    torch = pytest.importorskip("torch")
    if torch.version.hip is None:
        pytest.skip("built with a torch for ROCm only")
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        b.build()
        (scratch / "lib.so").write_text("kept")
        os.remove(b.TORCH_LIB)
        b.build(force=False)
        assert (scratch / "lib.so").read_text() == "kept" and (scratch / "torch.so").exists()
        (scratch / "torch.so").write_text("kept, " + b._built_for())
        b.build(force=False)
        assert (scratch / "torch.so").read_text().startswith("kept")
        (scratch / "torch.so").write_text("for another torch")
        b.build(force=False)
    assert (scratch / "torch.so").read_text().strip() == "new" and (scratch / "lib.so").read_text() == "kept"


def test_compiler_may_be_given_with_arguments(monkeypatch, scratch):
    torch = pytest.importorskip("torch")
    if torch.version.hip is None:
        pytest.skip("built with a torch for ROCm only")
    monkeypatch.setenv("CXX", f"env CONTENT=wrapped '{scratch}/compiler'")
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        b.build()
    assert (scratch / "torch.so").read_text().strip() == "wrapped"
