"""The host side of the Fokker-Planck doubling tree (stages, matrices in
fragment order, unit records) under AddressSanitizer and
UndefinedBehaviorSanitizer, against the eliminations' matrices (no GPU)."""
import os
import shutil

import pytest

from test_sanitizers import HERE, ROOT, SAN, _run


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_tree_under_sanitizers(tmp_path):
    exe = str(tmp_path / "tree_driver")
    csrc = os.path.join(ROOT, "paper_1907_13013_amd", "csrc")
    out = _run(["g++", "-std=c++17", *SAN, "-I", csrc, "-o", exe, os.path.join(HERE, "sanitize", "tree_driver.cpp"),
                os.path.join(csrc, "setup_math.cpp")], exe, tmp_path)
    assert "tree driver ok" in out
