"""The block orders of the Wilson operator, enumerated on the host (a C++ program
over csrc/schedule.h, the header that the kernels use): in every order each half
site belongs to exactly one block and every row of partial sums to one block, and
where the forms that stage x and y neighbours in LDS can run, each block is whole
x rows of one (z, t) plane."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_orders_cover_every_site_once_and_keep_lds_blocks_in_a_plane(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    exe = str(tmp_path / "block_orders")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2602_14450_amd", "csrc"), "-o", exe,
                    os.path.join(ROOT, "tests", "block_orders.cpp")], check=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout
    assert "0 faults" in run.stdout
