"""Indices of the PCG loop over the chip, replayed on the host for every grid it is
built for (tests/chip_layout.cpp): every access in bounds, the row and column tiles of
one mind about the exchange, every element with one owner."""

import os
import subprocess

import pytest

from paper_2606_06720_amd import build_lib

HERE = os.path.dirname(os.path.abspath(__file__))


def test_indices_of_every_grid(tmp_path):
    try:
        cc = build_lib.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not found")
    exe = str(tmp_path / "chip_layout")
    subprocess.run([cc, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-I", build_lib.INCLUDE, "-I",
                    build_lib.CSRC, os.path.join(HERE, "chip_layout.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    print(out.stdout)
    assert out.returncode == 0, out.stdout
