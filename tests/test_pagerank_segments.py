"""The gather segments of PageRank's binned edges near 2^32 edges, where a set is too
large for a test: their arithmetic alone, built for the host with sanitizers."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_segments_cover_their_parts(tmp_path):
    exe = tmp_path / "pagerank_segments"
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=undefined",
                        "-I", os.path.join(ROOT, "paper_2305_05055_amd", "csrc"),
                        os.path.join(ROOT, "tests", "pagerank_segments_driver.cpp"), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, (run.stdout + run.stderr)[-2000:]
