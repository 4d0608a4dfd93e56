"""Pieces of j-splits, checked on the host with the library's own functions
(g6mi_device.h, compiled for the host by hipcc; no HIP runtime function is
called): every tile in one piece, and no piece reads a minimum that the launch
before it does not write."""

import os
import subprocess

import pytest

from tests.test_plan_host import ROOT, hipcc

SRC = os.path.join(ROOT, "tests", "host", "piece_check.hip")


def test_pieces_read_only_written_minima(tmp_path):
    cc = hipcc()
    if cc is None:
        pytest.skip("hipcc not found")
    exe = str(tmp_path / "piece_check")
    r = subprocess.run([cc, "--offload-arch=gfx950", "--cuda-host-only", "-O2", "-std=c++17",
                        "-I", os.path.join(ROOT, "include"), SRC, "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-3000:]
    assert "violations 0" in r.stdout
