"""Lane-level CPU emulation of the segmented batch's reduce-by-key walk
(tests/emu/seg_keys_emu.cpp): every global and LDS access bounds-checked,
every segment written once with the exact sum (integer values); planted
mistakes are caught."""
import json
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "emu", "seg_keys_emu.cpp")
CXX = shutil.which("g++")

pytestmark = pytest.mark.skipif(CXX is None, reason="needs g++")


def build(out_dir, mutation=0):
    exe = os.path.join(out_dir, "keys_m%d" % mutation)
    subprocess.run([CXX, "-O2", "-std=c++17", "-Wall", "-Werror", "-DMUTATION=%d" % mutation, "-o", exe, SRC],
                   check=True)
    return exe


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    return build(str(tmp_path_factory.mktemp("keys")))


def run(exe, case):
    p = subprocess.run([exe] + [str(a) for a in case], capture_output=True, text=True, timeout=300)
    lines = p.stdout.strip().splitlines()
    rec = json.loads(lines[-1]) if lines else {"ok": False, "violation": p.stderr[-500:]}
    return dict(rec, rc=p.returncode, case=case)


# E, mean, layout, grid, wg, ipt, shift, seed
CASES = [(0, 5, 3, 8, 256, 4, 0, 1), (1, 1, 0, 8, 256, 4, 3, 1), (63, 1, 1, 3, 64, 1, 1, 2), (257, 300, 0, 2, 64, 4, 1, 1),
         (1000, 7, 1, 1, 64, 2, 2, 3), (100_003, 5, 1, 8, 512, 4, 1, 4), (100_003, 1, 0, 3, 256, 4, 2, 1),
         (100_003, 2, 3, 5, 64, 4, 3, 5), (1_000_003, 16, 1, 8, 256, 4, 0, 6), (1_000_003, 16, 2, 7, 64, 2, 1, 7),
         (1_000_003, 16, 2, 7, 64, 1, 1, 8), (1_000_003, 64, 1, 3, 256, 4, 2, 9), (1_000_003, 700, 1, 5, 512, 4, 3, 10),
         (1_000_003, 5000, 1, 64, 256, 4, 1, 11), (3_000_001, 40, 3, 16, 256, 4, 1, 12), (3_000_001, 4, 3, 1024, 256, 4, 0, 13),
         (500_000, 100_000, 3, 50, 128, 2, 1, 14), (2_000_000, 4, 0, 64, 256, 4, 0, 1), (2_000_000, 8, 0, 1024, 256, 4, 0, 1)]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_geometries(emu, case):
    rec = run(emu, CASES[case])
    assert rec["rc"] == 0 and rec["ok"], rec


def test_every_branch_is_taken(emu):
    recs = [run(emu, c) for c in CASES]
    for key in ("dense_tiles", "scanned", "plain", "late_chunks"):
        assert any(r.get(key, 0) > 0 for r in recs), key


@pytest.mark.parametrize("mutation", range(1, 6))
def test_planted_mistakes_are_caught(tmp_path, mutation):
    exe = build(str(tmp_path), mutation)
    assert any(r["rc"] != 0 and not r["ok"] for r in (run(exe, c) for c in CASES)), mutation
