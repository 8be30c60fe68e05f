"""The default plan of red_sum between the one-workgroup sum and the largest
inputs, without a GPU: one ticket kernel up to 32 MiB of any type, two kernels
above, both with nontemporal loads (a ticket with ordinary loads is slower
for inputs that the caches do not hold).  In a process of its own, since plans
that other tests install stay."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHOW = """
import sys
from paper_2004_05371_amd import redsum as R
for a in sys.argv[2:]:
    p = R.red_get_plan(int(sys.argv[1]), R.RED_ACC_COMPENSATED, int(a))
    print(p.variant, p.flags)
"""
ATOMIC, RELAUNCH = 2, 1
LINE = 32 << 20


@pytest.mark.parametrize("dtype,size", [(0, 4), (1, 4), (2, 2), (3, 2)])
def test_ticket_and_two_kernels(dtype, size):
    want = [(1 << 20, ATOMIC), (10_000_000, ATOMIC), (LINE, ATOMIC), (LINE + 4, RELAUNCH), (40 << 20, RELAUNCH),
            (1 << 28, RELAUNCH)]
    r = subprocess.run([sys.executable, "-c", SHOW, str(dtype)] + [str(b // size) for b, _ in want], cwd=ROOT,
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    got = [tuple(int(a) for a in line.split()) for line in r.stdout.splitlines()]
    assert got == [(v, 1) for _, v in want], (dtype, got)
