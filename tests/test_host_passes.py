"""Control flow of the minimizer's passes, played on the CPU: the kernels'
source compiled as C++ with a stand-in for the HIP header that runs
wavefronts and workgroups in an order the test chooses."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("hostsim") / "passes")
    sim = os.path.join(ROOT, "tests", "hostsim")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-pthread", "-I", sim,
                    "-I", os.path.join(ROOT, "paper_1810_03358_amd", "csrc"), "-x", "c++",
                    os.path.join(sim, "passes.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=60).stdout
    return [line.split(maxsplit=1) for line in out.splitlines()]


@pytest.mark.parametrize("name", ["accept_gd", "accept_hb", "accept_fgm"])
def test_workgroups_without_a_product_row_stay_whole(lines, name):
    got = [text for n, text in lines if n == name]
    assert got == ["ok", "ok"], got


@pytest.mark.parametrize("name", ["kick_counts", "resume_counts"])
def test_a_minimization_starts_its_counts_at_zero(lines, name):
    assert [text for n, text in lines if n == name] == ["ok"]
