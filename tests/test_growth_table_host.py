"""Host cost of the collapse-redshift tables (CPU): a call of pin_plan_set_growth is mostly its
quadrature, and what else it does (the polynomials per bucket) must not make it longer than that
quadrature on one thread.  Its parts are evaluated on several threads, which must not show in the
values."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_growth_table_takes_less_than_its_quadrature_on_one_thread(tmp_path):
    csrc = os.path.join(ROOT, "paper_1305_1505_amd", "csrc")
    exe = str(tmp_path / "growth_table")
    subprocess.run(["g++", "-std=c++17", "-O3", "-pthread", "-I", csrc, os.path.join(ROOT, "tests", "native", "growth_table.cpp"),
                    os.path.join(csrc, "host_math.cpp"), "-o", exe], check=True, capture_output=True)
    same, worst, table, quadrature = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split()
    assert same == "1"
    # sums of 32764 panels in the same order, whose nodes and weights may differ in the last bits
    assert float(worst) <= 1e-12
    if len(os.sched_getaffinity(0)) < 2:
        pytest.skip("one CPU: nothing to share the work with")
    assert float(table) < float(quadrature), (table, quadrature)


def test_sigma8_quadrature_takes_less_than_on_one_thread(tmp_path):
    """Nearly all of pin_plan_create on a small grid is the sigma_8 quadrature."""
    csrc = os.path.join(ROOT, "paper_1305_1505_amd", "csrc")
    exe = str(tmp_path / "sigma_table")
    subprocess.run(["g++", "-std=c++17", "-O3", "-pthread", "-I", csrc, os.path.join(ROOT, "tests", "native", "sigma_table.cpp"),
                    os.path.join(csrc, "host_math.cpp"), "-o", exe], check=True, capture_output=True)
    worst, parts, one = (float(x) for x in subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split())
    assert worst <= 1e-9        # the integrand is smooth over 64000 steps, but oscillates beyond k R = 2000
    if len(os.sched_getaffinity(0)) < 2:
        pytest.skip("one CPU: nothing to share the work with")
    assert parts < 0.7 * one, (parts, one)
