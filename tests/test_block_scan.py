"""The one-workgroup scan under every late wavefront: its source compiled for
the CPU and run with the wavefronts in adverse orders between barriers."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def scan(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("scan") / "block_scan")
    subprocess.run(["g++", "-std=c++17", "-O1", os.path.join(HERE, "host", "block_scan.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("order", ["up", "down", "1", "2", "3"])
@pytest.mark.parametrize("n", [0, 1, 63, 64, 65, 4095, 4096, 4097, 12289])
def test_sums_do_not_depend_on_the_order_of_wavefronts(scan, order, n):
    r = subprocess.run([scan, order, str(n)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
