"""The kernels' address arithmetic on the CPU: where a logical byte of a flat
buffer or ring window lies (locate) and how a chunk's bytes are described
(chunk_loc), against the piece list of the same descriptor and, for rings too
many to list, against exact integer arithmetic; the work items of a bank
shrink's moves; and the items of Merkle lists, to the most a buffer can have.  The checks live in tests/host/test_geometry.cpp, compiled
with g++ under UndefinedBehaviorSanitizer."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "host", "test_geometry.cpp")


def test_geometry_matches_the_piece_list(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ is not installed")
    exe = str(tmp_path / "geometry")
    r = subprocess.run([cxx, "-std=c++17", "-O1", "-g", "-Wall", "-Wextra", "-Werror", "-fsanitize=undefined",
                        "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "include"), SRC, "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.strip() == "ok"
