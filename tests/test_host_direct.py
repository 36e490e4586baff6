"""The tiles of the direct steps (paper_1101_0265_amd/csrc/direct_tiles.h), checked on the CPU:
snf_purify_dense_noalloc has one for every order up to its maximum on devices of any number of
compute units (a part of a partitioned GPU has 32), in buffers of its size, and on a whole device
the one that snf_purify_dense takes."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_noalloc_tiles(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "direct_check")
    r = subprocess.run([gxx, "-std=c++17", "-O1", os.path.join(HERE, "host", "direct_check.cpp"),
                        "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    ok, other = r.stdout.split()[0], r.stdout.split()[-1]
    assert r.returncode == 0 and ok == "ok", r.stdout
    assert int(other) > 0                       # devices where the two entry points differ
