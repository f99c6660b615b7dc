"""The LDS addresses of the sorted conversion's merge search, walked on the CPU:
merge_search_model.cpp runs a wave of the group kernel through the same address
functions (csrc/merge_search.hpp), with strips far past a group's capacity beside
short ones, under AddressSanitizer and UndefinedBehaviorSanitizer."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")
def test_merge_search_stays_in_its_slice(tmp_path):
    exe = str(tmp_path / "merge_model")
    src = [os.path.join(ROOT, "tests", "merge_search_model.cpp"), "-o", exe]
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-Wall", "-I", os.path.join(ROOT, "paper_1203_2946_amd", "csrc")]
    san = ["-fsanitize=address,undefined", "-fno-sanitize-recover=all"]
    b = subprocess.run([*cmd, *san, *src], capture_output=True, text=True)
    if b.returncode != 0 and "sanitize" in b.stderr:
        b = subprocess.run([*cmd, *src], capture_output=True, text=True)
    assert b.returncode == 0, b.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout == "ok\n"
