"""The pool that lends device memory to calls (scratch.hpp), over a runtime that only records what is
asked of it: reuse on one stream, other streams, the bound, blocks never lent twice, failures, memory
given back with the last handle, threads."""
from __future__ import annotations

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_scratch_pool(tmp_path):
    exe = str(tmp_path / "scratch_driver")
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-pthread", "-Wall", "-Werror",
                    "-I", os.path.join(ROOT, "paper_1212_2287_amd", "csrc"),
                    os.path.join(ROOT, "tests", "scratch_driver.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
