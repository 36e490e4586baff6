"""The tiles of the direct steps (paper_1101_0265_amd/csrc/direct_tiles.h), checked on the CPU:
snf_purify_dense_noalloc has one for every order up to its maximum on devices of any number of
compute units (a part of a partitioned GPU has 32), in buffers of its size, and on a whole device
the one that snf_purify_dense takes."""
import ctypes
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_workspace_bytes_hold_the_rows_of_the_direct_steps():
    """snf_workspace_bytes covers three FP64 buffers of the longest rows a step takes at n."""
    from paper_1101_0265_amd import build_lib
    if not os.path.exists(build_lib.LIB):
        build_lib.build()
    lib = ctypes.CDLL(build_lib.LIB)
    lib.snf_workspace_bytes.restype = ctypes.c_size_t
    lib.snf_workspace_bytes.argtypes = [ctypes.c_int64, ctypes.c_int32]
    for n in range(1, 2300):
        ld = (n + 127) // 128 * 128
        for t in range(32, 97, 16):
            nt = (n + t - 1) // t
            if nt * (nt + 1) // 2 <= 256:
                ld = max(ld, nt * t if nt * t % 256 else nt * t + 16)
        assert lib.snf_workspace_bytes(n, 0) >= 3 * 8 * ld * ld, n


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
