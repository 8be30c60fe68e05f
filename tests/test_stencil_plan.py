"""The shape of the stencil's blocked steps, evaluated on the CPU
(csrc/stencil_plan.h compiled with g++ and UBSan): every shape covers the
array with margins that hold its steps, up to the largest step count the call
takes, and the sizes that the GPU tests use reach every window width."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "emu", "stencil_plan_main.cpp")
CXX = shutil.which("g++")

pytestmark = pytest.mark.skipif(CXX is None, reason="needs g++")

INT_MAX = 2**31 - 1

# Values per lane -> (n, steps) of an array that the planner gives windows of
# that width; the GPU tests run these.
WIDTHS = {2: (1000, 50), 4: (65_536, 131), 6: (100_003, 200), 8: (262_146, 131), 12: (1_000_002, 200),
          16: (1_890_062, 60), 20: (4_194_304, 200), 24: (2_965_823, 75), 28: (5_163_796, 84), 36: (8_684_434, 117)}


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan")
    subprocess.run([CXX, "-O1", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined",
                    "-fno-sanitize-recover=undefined", "-o", exe, SRC], check=True)

    def shapes(cases):
        p = subprocess.run([exe] + [str(a) for c in cases for a in c], capture_output=True, text=True, timeout=60)
        assert p.returncode == 0, p.stderr[-2000:]
        return [tuple(int(a) for a in line.split()) for line in p.stdout.splitlines()]
    return shapes


@pytest.mark.parametrize("n", [1, 2, 127, 128, 511, 512, 513, 1000, 65_534, 299_998, 4_194_302, 23_999_999, 2**31, 2**35])
def test_shapes_cover_the_array(plan, n):
    """n interior values: windows inside the interior, margins of at least
    the steps of one launch, something left between them, enough wavefronts,
    and a grid that one launch takes (fewer than 2^32 threads)."""
    cases = [(n, s) for s in (1, 2, 3, 8, 40, 200, 863, 864, 1000, 12_345, 10**6, INT_MAX - 864, INT_MAX - 863,
                              INT_MAX - 47, INT_MAX)]
    for (_, steps), (v, launches, k, m, waves) in zip(cases, plan(cases)):
        if launches == 0:  # one launch per step
            assert steps <= 2 and n >= 2**21, (n, steps)
            continue
        if launches == 1:
            assert v in (2, 4, 8) and n <= 64 * v, (n, steps, v)
            continue
        assert v in (2, 4, 6, 8, 12, 16, 20, 24, 28, 36) and 64 * v <= n, (n, steps, v)
        assert launches >= 2 and launches % 2 == 0, (n, steps, launches)
        assert k >= -(-steps // launches) and k % 4 == 0, (n, steps, launches, k)
        assert m >= 1 and m == 64 * v - 2 * k, (n, steps, k, m)
        assert waves == -(-n // m), (n, steps, m, waves)
        assert -(-waves // 4) * 256 < 2**32, (n, steps, waves)


def test_one_launch_per_step_where_it_is_faster(plan):
    """One or two steps on 2^21 interior values and more; three steps, or
    fewer values, run on windows."""
    for n, steps, per_step in ((2**21 - 1, 1, False), (2**21, 1, True), (2**21, 2, True), (2**21, 3, False),
                               (10_000_000, 1, True), (24_000_001, 2, True), (24_000_001, 3, False), (4096, 1, False)):
        (_, launches, _, _, _), = plan([(n, steps)])
        assert (launches == 0) == per_step, (n, steps, launches)


def test_every_window_width_has_a_size(plan):
    """The sizes that stand for the widths in the GPU tests take them."""
    got = plan([(n - 2, steps) for n, steps in WIDTHS.values()])
    assert [g[0] for g in got] == list(WIDTHS) and all(g[1] >= 2 for g in got), got
