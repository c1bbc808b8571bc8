"""Harmonic sums of planes with most rows above threshold, where emission is the work.

Spectra short enough for row segments list every segment's rows by themselves;
the emission must not visit all rows for each.  A spectrum four bins longer than
the longest with segments does the same work in one: the shorter one may not
take longer (1.3 x for the segments' own launch shape and the box).  Nor may a false-alarm
probability of 1e-4, whose candidates fit in the default lists, take 1.5 x the time of
the default 1e-6 on a long spectrum.  Lists, counts and order are checked where rows
are full in one segment and empty in another.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import harmonic as oh  # noqa: E402
from paper_1806_01556_amd import fdas  # noqa: E402

MAPS = {"stretch": fdas.HSUM_STRETCH, "fundamental": fdas.HSUM_FUNDAMENTAL, "highest": fdas.HSUM_HIGHEST}


def _time(n, z_max, index, p_fa=0.05):
    with fdas.plan_create(n_max=1 << 21, z_max=z_max, hsum_index=MAPS[index]) as plan:
        g = torch.Generator(device="cuda:0").manual_seed(3)
        fop = torch.empty((plan.rows, fdas.fop_ld(n)), device="cuda:0").exponential_(generator=g)
        thr = fdas.thresholds(8, p_fa).astype(np.float32)
        ta = torch.from_numpy(np.repeat(thr[:, None], plan.rows, 1).copy()).to("cuda:0")
        cands, counts = fdas.alloc_cands(plan, "cuda:0")
        best = 1e9
        for _ in range(6):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(5):
                fdas.harmonic_sum(plan, fop, n, cands, counts, ta=ta)
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1) / 5)
    return best


@pytest.mark.parametrize("index,z_max,n", [("stretch", 42, 1 << 18), ("stretch", 17, 393_216),
                                           ("fundamental", 17, 393_216), ("fundamental", 42, 393_216)])
def test_dense_planes_take_no_longer_in_segments(index, z_max, n):
    with_segments, without = _time(n, z_max, index), _time(n + 4, z_max, index)
    print(f"dense planes: {index} z_max={z_max} n={n}: {1e3 * with_segments:.0f} us, n + 4: {1e3 * without:.0f}", flush=True)
    assert with_segments <= 1.3 * without


@pytest.mark.parametrize("index", ["fundamental", "highest"])
def test_isolated_hits_take_little_of_the_time(index):
    n, z_max = 1 << 21, 42
    many, few = _time(n, z_max, index, 1e-4), _time(n, z_max, index, 1e-6)
    print(f"isolated hits: {index}: {1e3 * many:.0f} us at 1e-4, {1e3 * few:.0f} at 1e-6", flush=True)
    assert many <= 1.5 * few


@pytest.mark.parametrize("index", sorted(MAPS))
@pytest.mark.parametrize("z_max,n", [(42, 3000), (17, 5001), (48, 900), (2, 7000)])
def test_full_and_empty_segments(index, z_max, n):
    n_harm, rows = 8, 2 * z_max + 1
    rng = np.random.default_rng(n)
    plane = rng.exponential(size=(rows, n)).astype(np.float32)
    buf = np.full((rows, fdas.fop_ld(n)), np.nan, dtype=np.float32)
    buf[:, :n] = plane
    ta = np.repeat(oh.threshold_array(n_harm, z_max, 0.2).astype(np.float32)[:, :1], rows, axis=1)
    ta[:, rows // 5:rows // 2] = 1e6  # no cell of these rows
    ta[:, -1] = 0.0                   # every cell of the last
    ref = oh.candidates(plane, n_harm, ta=ta, index=index)
    print(f"dense planes: {index} z_max={z_max} n={n} candidates={ref.size}", flush=True)
    cap = 1 << 18
    with fdas.plan_create(z_max=z_max, n_harm=n_harm, n_max=n, hsum_index=MAPS[index], cand_capacity=cap) as plan:
        fop, ta_t = torch.from_numpy(buf).to("cuda:0"), torch.from_numpy(ta).to("cuda:0")
        cands, counts = fdas.alloc_cands(plan, "cuda:0")
        fdas.harmonic_sum(plan, fop, n, cands, counts, ta=ta_t)
        got, hc = fdas.candidates(plan, cands, counts)
    assert np.array_equal(hc, oh.plane_counts(ref, n_harm))
    for f in ("harm", "z", "r"):
        assert np.array_equal(got[f], ref[f]), f
    assert np.array_equal(got["power"].view(np.int32), ref["power"].astype(np.float32).view(np.int32))
