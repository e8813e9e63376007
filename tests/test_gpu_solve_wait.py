"""A solve whose workgroups stop waiting for each other: NaN in the rows that were
not solved, MPCHOL_EHIP from the next call that synchronizes, and nothing left
behind (tests/solve_wait_driver.cpp, built with the library)."""
import os
import subprocess

import pytest

pytestmark = pytest.mark.gpu

EXE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2408_04440_amd", "solve_wait_check")


def test_a_wait_that_runs_out_is_reported_once():
    if not os.path.exists(EXE):
        pytest.skip("the driver is not built (python -m paper_2408_04440_amd.build_sanitize)")
    r = subprocess.run([EXE], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), (r.stdout + r.stderr)[-4000:]
