"""Limits shared by the host and the kernels (bc_device.h) and the scratch memory
of the calls (bc_scratch.h), checked on the CPU."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2403_07858_amd", "csrc")


def run_check(name, tmp_path, *args):
    exe = str(tmp_path / name)
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC,
                    "-I", os.path.join(os.path.dirname(HERE), "include"), "-pthread", os.path.join(HERE, name + ".cpp"), "-o", exe], check=True)
    r = subprocess.run([exe, *args], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


def test_every_column_has_a_number_of_its_own(tmp_path):
    run_check("column_limits_check", tmp_path)


@pytest.mark.parametrize("part", ["cap", "devices", "host_full"])
def test_scratch(part, tmp_path):
    run_check("scratch_check", tmp_path, part)


def test_row_pool_serves_its_roots(tmp_path):
    run_check("row_pool_check", tmp_path)
