"""The packed pair keys up to the largest atom index, their source compiled for
the CPU."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_fields_and_order(tmp_path):
    exe = str(tmp_path / "pair_key")
    subprocess.run(["g++", "-std=c++17", "-O1", os.path.join(HERE, "host", "pair_key.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
