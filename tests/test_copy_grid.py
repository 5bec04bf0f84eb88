"""Appends and gathers of every size that memory can hold fit one launch: a grid
has fewer than 2^32 threads, and the rows a workgroup takes do not shrink with
the page (on pages of one token, rows of 256 bytes would reach that limit at 4
GiB)."""
import ctypes
import os
import shutil
import subprocess

import pytest

from paper_2606_24506_amd import build


@pytest.mark.skipif(shutil.which("g++") is None, reason="no C++ compiler")
def test_largest_copies_fit_a_launch(tmp_path):
    src = os.path.join(os.path.dirname(os.path.abspath(__file__)), "c", "copy_shim.cpp")
    out = str(tmp_path / "shim.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-I", build.CSRC, src, "-o", out], check=True)
    lib = ctypes.CDLL(out)
    threads = lib.threads_per_block()
    for row_elems in [*range(64, 4096, 8), *(2 * kv * d for kv in range(1, 257) for d in (64, 128, 256, 512))]:
        rows = lib.rows_per_block(row_elems)
        assert rows == 1 or rows * row_elems // 8 <= 5 * threads  # one pass of the workgroup
        assert rows <= threads                                    # a thread for every page that starts in it
        most = (144 << 30) // (2 * row_elems)                     # as many rows again stand in the pages
        assert -(-most // rows) * threads < 1 << 32, row_elems
