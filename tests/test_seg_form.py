"""The form that a segmented batch takes by itself, evaluated on the CPU
(csrc/seg_rules.h, which the kernel evaluates too): even and random lengths,
log-uniform ones, one segment that holds all values, empty segments spread or
in stretches."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CXX = shutil.which("g++")

pytestmark = pytest.mark.skipif(CXX is None, reason="needs g++")

WORKGROUP, PIECES, RUNS = 1, 2, 3
THREADS = 1024 * 256  # the default plan on 256 CUs


@pytest.fixture(scope="module")
def form(tmp_path_factory):
    d = tmp_path_factory.mktemp("form")
    exe = str(d / "form")
    subprocess.run([CXX, "-O1", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=undefined",
                    "-o", exe, os.path.join(HERE, "emu", "seg_form_main.cpp")], check=True)

    def of(off):
        path = str(d / "off.bin")
        np.asarray(off, dtype=np.int64).tofile(path)
        p = subprocess.run([exe, path, str(THREADS)], capture_output=True, text=True, timeout=60)
        assert p.returncode == 0, p.stderr[-2000:]
        return int(p.stdout)
    return of


def offsets(layout, total, mean):
    nseg = total // mean
    rng = np.random.default_rng(total + mean)
    k = np.arange(nseg + 1)
    if layout == "equal":
        off = k * total // nseg
    elif layout == "random cuts":
        off = np.concatenate([[0], np.sort(rng.integers(0, total + 1, nseg - 1)), [total]])
    elif layout == "log-uniform":
        w = np.exp(rng.random(nseg) * np.log(1 << 20))
        off = np.concatenate([[0], np.cumsum(w) * (total / w.sum())]).astype(np.int64)
    elif layout == "one, others empty":
        off = np.where(k > nseg // 2, total, 0)
    elif layout == "one, others 100":
        off = np.where(k > nseg // 2, total - 100 * nseg, 0) + 100 * k
    elif layout == "empty at the end":  # two of three
        off = np.minimum(3 * k * total // nseg, total)
    elif layout == "every other one empty":
        off = (k + 1) // 2 * 2 * total // nseg
    else:  # three of four empty, spread
        w = np.where(rng.random(nseg) < 0.75, 0.0, rng.random(nseg))
        off = np.concatenate([[0], np.cumsum(w) * (total / w.sum())]).astype(np.int64)
    off[-1] = total
    return off


# Of each layout: (total, mean) and the form that is the fastest, or as fast as the best.
CASES = [
    ("equal", 60_000_000, 512, RUNS), ("equal", 60_000_000, 2048, PIECES), ("equal", 60_000_000, 20_000, WORKGROUP),
    ("equal", 200_000, 40_000, RUNS), ("random cuts", 10_000_000, 1100, RUNS), ("random cuts", 10_000_000, 4000, PIECES),
    ("log-uniform", 10_000_000, 1100, RUNS), ("log-uniform", 60_000_000, 17_000, RUNS),
    ("log-uniform", 10_000_000, 60_000, RUNS), ("log-uniform", 60_000_000, 100_000, WORKGROUP),
    ("one, others 100", 10_000_000, 60_000, RUNS), ("one, others 100", 100_000_000, 17_000, RUNS),
    ("one, others empty", 10_000_000, 17_000, WORKGROUP), ("one, others empty", 10_000_000, 60_000, WORKGROUP),
    ("one, others empty", 10_000_000, 4000, RUNS), ("one, others empty", 60_000_000, 17_000, RUNS),
    ("one, others empty", 1_000_000, 60_000, RUNS), ("empty at the end", 60_000_000, 17_000, RUNS),
    ("empty at the end", 10_000_000, 17_000, RUNS), ("empty, spread", 10_000_000, 4000, RUNS),
    ("empty, spread", 60_000_000, 4000, PIECES), ("empty, spread", 10_000_000, 60_000, WORKGROUP),
    ("empty, spread", 60_000_000, 1100, PIECES), ("every other one empty", 1_000_000, 60_000, WORKGROUP),
    ("empty, spread", 200_000_000, 17_000, WORKGROUP), ("empty, spread", 1_000_000, 60_000, RUNS),
]


@pytest.mark.parametrize("layout,total,mean,want", CASES)
def test_form_of_a_batch(form, layout, total, mean, want):
    assert form(offsets(layout, total, mean)) == want
