"""The cut of a batch of trees into groups, tiles and launches
(paper_1812_01329_amd/csrc/tree_cut.hpp, host code) over random batches: whole
trees and pieces of trees, binary, of any arity, caterpillars, stars and
chains, with groups of few and of many nodes."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_cuts_hold_what_the_kernels_assume(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not found")
    out = str(tmp_path / "tree_cut_check")
    r = subprocess.run([cxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                        os.path.join(ROOT, "tests", "sanitize", "tree_cut_check.cpp"), "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([out], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr[-3000:]
    assert int(r.stdout.split()[2]) > 100, r.stdout   # of the cuts were in pieces
