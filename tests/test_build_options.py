"""A source's own compiler options are left out where the compiler does not know them; an error in the
source is still one."""
import os
import shutil

import pytest

from paper_2103_14897_amd import build

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")


def test_unknown_option_is_left_out(tmp_path, monkeypatch):
    (tmp_path / "one.hip").write_text("#include <hip/hip_runtime.h>\n__global__ void k(int* p) { *p = 1; }\n")
    (tmp_path / "two.hip").write_text("int f() { return undeclared; }\n")
    monkeypatch.setattr(build, "CSRC", str(tmp_path))
    monkeypatch.setattr(build, "BUILD", str(tmp_path))
    bad = ["-mllvm", "-no-such-llvm-option=1"]
    monkeypatch.setattr(build, "EXTRA", {"one.hip": bad, "two.hip": bad})
    obj = build._compile("one.hip")
    assert os.path.getsize(obj) > 0
    with pytest.raises(RuntimeError, match="undeclared"):
        build._compile("two.hip")
