"""Infinities, NaN and values whose binary32 sum overflows in segmented
batches: what is not finite stays in its own segment, although many segments
share a lane's running sum, a scan across the lanes and one tile; every other
sum stays within the bound."""
import sys

import numpy as np
import pytest

from paper_2004_05371_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

FORMS = {"auto": 0, "workgroup": 32, "pieces": 64, "runs": 128}


def lengths(kind):
    r = np.random.default_rng(700)
    return {"short": r.integers(0, 9, 40_000), "rows": np.full(900, 300), "mixed": r.choice([0, 1, 5, 64, 700, 3000], 900),
            "long": np.array([70_000, 0, 3, 150_000, 40_000, 1])}[kind].astype(np.int64)


@pytest.mark.parametrize("variant", [1, 2])
@pytest.mark.parametrize("form", list(FORMS))
@pytest.mark.parametrize("kind", ["short", "rows", "mixed", "long"])
def test_nonfinite_values_stay_in_their_segment(lib, kind, form, variant):
    off = inputs.offsets_from_lengths(lengths(kind))
    x = inputs.normal_f32(int(off[-1]), sub=85)
    nonempty = np.flatnonzero(np.diff(off))
    r = np.random.default_rng(701)
    hit = r.permutation(nonempty)[:max(4, len(nonempty) // 20)]
    want = np.full(off.size - 1, np.nan)
    for i, s in enumerate(hit):  # +inf, -inf, NaN, both infinities, at the first, last or any value
        a, b = off[s], off[s + 1]
        at = (a, b - 1, r.integers(a, b))[i % 3]
        x[at] = (np.inf, -np.inf, np.nan, np.inf)[i % 4]
        want[s] = x[at]
        if i % 4 == 3 and b - a > 1:
            x[a if at != a else b - 1] = -np.inf
            want[s] = np.nan
    is_hit = np.zeros(off.size - 1, bool)
    is_hit[hit] = True
    xs = torch.from_numpy(x).to("cuda")
    ot = torch.from_numpy(off).to("cuda")
    for grid, wg, ipt in ((0, 256, 4), (7, 128, 2)):
        print("non-finite", kind, form, variant, grid, file=sys.stderr, flush=True)
        out = torch.full((off.size - 1,), -7.0, dtype=torch.float64, device="cuda")
        lib.red_sum_segmented_ex(xs.data_ptr(), ot.data_ptr(), off.size - 1, out.data_ptr(), lib.current_stream(),
                                 lib.make_opts(variant=variant, wg=wg, ipt=ipt, grid=grid, flags=FORMS[form]))
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        assert np.array_equal(got[is_hit], want[is_hit], equal_nan=True), (kind, form, variant, grid)
        clean = np.flatnonzero(~is_hit)
        # 64-bit sums of at most 150,000 values: their own error is below 2e-11 of the sum of magnitudes.
        c = np.concatenate([[0.0], np.cumsum(np.where(np.isfinite(x), x, 0).astype(np.float64))])
        m = np.concatenate([[0.0], np.cumsum(np.abs(np.where(np.isfinite(x), x, 0)).astype(np.float64))])
        ref, mag = c[off[1:]] - c[off[:-1]], m[off[1:]] - m[off[:-1]]
        bad = clean[~(np.abs(got[clean] - ref[clean]) <= 1e-6 * mag[clean] + 2e-11 * m[-1])]
        assert bad.size == 0, (kind, form, variant, grid, bad[:3], got[bad[:3]], ref[bad[:3]])


@pytest.mark.parametrize("grid,wg,ipt", [(0, 256, 4), (7, 128, 2)])
def test_sums_beyond_binary32_in_the_runs_form(lib, grid, wg, ipt):
    """Lane runs are added in binary64: segments of finite values whose sum
    no binary32 holds have it."""
    off = inputs.offsets_from_lengths(np.tile(np.array([3, 0, 17, 1, 40]), 3000).astype(np.int64))
    x = np.full(int(off[-1]), 3.0e38, dtype=np.float32)
    xs, ot = torch.from_numpy(x).to("cuda"), torch.from_numpy(off).to("cuda")
    out = torch.full((off.size - 1,), -7.0, dtype=torch.float64, device="cuda")
    lib.red_sum_segmented_ex(xs.data_ptr(), ot.data_ptr(), off.size - 1, out.data_ptr(), lib.current_stream(),
                             lib.make_opts(variant=2, wg=wg, ipt=ipt, grid=grid, flags=128))
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), np.diff(off) * np.float64(x[0]))
