"""Lane-level CPU emulation of the reduce-by-key form of a segmented batch
over whole launches (tests/emu/seg_slices_emu.cpp): the kernel's own slice
lengths, tile rows and LDS bounds (csrc/seg_rules.h), carry slots, tickets and
the three fix-ups; every access bounds-checked, every segment written once with
the exact sum (integer values); planted mistakes are caught; the emulator
itself under ASan and UBSan."""
import json
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "emu", "seg_slices_emu.cpp")
CXX = shutil.which("g++")

pytestmark = pytest.mark.skipif(CXX is None, reason="needs g++")


def build(out_dir, mutation=0, sanitize=False):
    exe = os.path.join(out_dir, "slices_m%d%s" % (mutation, "_san" if sanitize else ""))
    cmd = [CXX, "-O2", "-std=c++17", "-Wall", "-Werror", "-DMUTATION=%d" % mutation, "-o", exe, SRC]
    if sanitize:
        cmd[1:1] = ["-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-fno-omit-frame-pointer"]
    subprocess.run(cmd, check=True)
    return exe


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    return build(str(tmp_path_factory.mktemp("slices")))


def run(exe, case):
    p = subprocess.run([exe] + [str(a) for a in case], capture_output=True, text=True, timeout=300)
    lines = p.stdout.strip().splitlines()
    rec = json.loads(lines[-1]) if lines else {"ok": False, "violation": p.stderr[-500:]}
    return dict(rec, rc=p.returncode, case=case)


# E, mean, layout, grid, wg, ipt, wide, shift, seed; then the rows of the tiles that it takes
CASES = [
    ((0, 5, 3, 8, 256, 4, 1, 0, 1), 2), ((1, 1, 0, 8, 256, 4, 1, 3, 1), 2), ((63, 1, 1, 3, 64, 1, 0, 1, 2), 2),
    ((257, 300, 0, 2, 64, 4, 0, 1, 1), 2), ((1000, 7, 1, 1, 64, 2, 1, 2, 3), 4), ((100_003, 5, 1, 8, 512, 4, 1, 1, 4), 4),
    ((100_003, 1, 0, 3, 256, 4, 1, 2, 1), 8), ((100_003, 1, 0, 3, 256, 4, 0, 2, 1), 4), ((100_003, 2, 3, 5, 64, 4, 1, 3, 5), 8),
    ((100_003, 1, 0, 1024, 256, 4, 1, 1, 5), 2), ((1_000_003, 16, 1, 8, 256, 4, 1, 0, 6), 8),
    ((1_000_003, 16, 2, 7, 64, 2, 1, 1, 7), 4), ((1_000_003, 16, 2, 7, 64, 2, 0, 1, 7), 2),
    ((1_000_003, 16, 2, 7, 64, 1, 0, 1, 8), 2), ((1_000_003, 64, 1, 3, 256, 4, 0, 2, 9), 4),
    ((1_000_003, 700, 1, 5, 512, 4, 1, 3, 10), 8), ((1_000_003, 5000, 1, 64, 256, 4, 1, 1, 11), 4),
    ((1_000_003, 30_000, 1, 1024, 256, 4, 1, 1, 11), 4), ((3_000_001, 40, 3, 16, 256, 4, 1, 1, 12), 8),
    ((3_000_001, 4, 3, 1024, 256, 4, 1, 0, 13), 4), ((500_000, 100_000, 3, 50, 128, 2, 1, 1, 14), 4),
    ((2_000_000, 4, 0, 64, 256, 4, 1, 0, 1), 8), ((2_000_000, 8, 0, 1024, 256, 4, 1, 0, 1), 2),
    ((2_000_003, 9, 4, 1024, 256, 4, 1, 2, 1), 2), ((300_001, 70_000, 0, 300, 64, 4, 1, 0, 1), 4),
    ((4_000_000, 3, 1, 512, 512, 4, 0, 1, 15), 4), ((8_000_003, 512, 0, 100, 128, 4, 1, 3, 16), 8),
]


@pytest.mark.parametrize("fix", [0, 1, 2])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_launches(emu, case, fix):
    args, rows = CASES[case]
    rec = run(emu, args[:7] + (fix,) + args[7:])
    assert rec["rc"] == 0 and rec["ok"], rec
    assert rec["rows"] == rows, rec


@pytest.mark.parametrize("shift", range(4))
def test_the_shortest_slices_are_one_tile(emu, shift):
    """Also where the values are not aligned to 16 bytes."""
    rec = run(emu, (1_000_003, 300, 1, 1024, 256, 4, 1, 0, shift, 17))
    assert rec["ok"] and rec["rows"] == 2 and rec["max_tiles"] == 1, rec


def test_every_branch_is_taken(emu):
    recs = [run(emu, c[:7] + (0,) + c[7:]) for c, _ in CASES]
    for rows in (2, 4, 8):
        for key in ("halves", "scanned", "plain", "late_chunks", "cut"):
            assert any(r["rows"] == rows and r.get(key, 0) > 0 for r in recs), (rows, key)


@pytest.mark.parametrize("mutation", range(1, 10))
def test_planted_mistakes_are_caught(tmp_path, mutation):
    exe = build(str(tmp_path), mutation)
    assert any(r["rc"] != 0 and not r["ok"] for r in (run(exe, c[:7] + (2,) + c[7:]) for c, _ in CASES)), mutation


def test_emulation_under_sanitizers(tmp_path):
    exe = build(str(tmp_path), sanitize=True)
    for fix in (0, 1, 2):
        for c, _ in CASES:
            if c[0] <= 1_000_003:
                rec = run(exe, c[:7] + (fix,) + c[7:])
                assert rec["rc"] == 0 and rec["ok"], rec
