"""Harmonic sums at the lengths where their row segments begin and end: the 85-row
stretch sum has four segments up to 2^18 bins and one above, whatever the plan's
longest spectrum, the highest-anchored map three, four and one around 2^18 and
2^20.  Hits in the first and last row of every segment and over the whole plane,
bit for bit against the oracle's FP32 twin, through both entry points.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import harmonic as oh  # noqa: E402
from paper_1806_01556_amd import fdas  # noqa: E402


@pytest.mark.parametrize("n,n_max", [(204_800, 204_800), (204_801, 204_801), ((1 << 18) - 1, (1 << 18) - 1),
                                     (1 << 18, 1 << 18), ((1 << 18) + 1, (1 << 18) + 1), (1 << 18, 1 << 21)])
def test_segment_edges(n, n_max):
    z_max, n_harm = 42, 8
    rng = np.random.default_rng(n)
    plane = rng.exponential(size=(85, n)).astype(np.float32)
    for row in (0, 20, 21, 41, 42, 62, 63, 84):  # segments begin at rows 0, 21, 42 and 63
        plane[row, rng.integers(0, n, 12)] += 40.0
    plane[:, n - 1] += 40.0
    buf = np.full((85, fdas.fop_ld(n)), np.nan, dtype=np.float32)
    buf[:, :n] = plane
    ta = oh.threshold_array(n_harm, z_max, 1e-6).astype(np.float32)
    ref = oh.candidates(plane, n_harm, ta=ta)
    fop, ta_t = torch.from_numpy(buf).to("cuda:0"), torch.from_numpy(ta).to("cuda:0")
    print(f"segment edges: n={n} n_max={n_max} candidates={ref.size}", flush=True)
    with fdas.plan_create(z_max=z_max, n_harm=n_harm, n_max=n_max) as plan:
        for call in (fdas.harmonic_sum, fdas.harmonic_sum_noalloc):
            cands, counts = fdas.alloc_cands(plan, "cuda:0")
            call(plan, fop, n, cands, counts, ta=ta_t)
            got, hc = fdas.candidates(plan, cands, counts)
            assert np.array_equal(hc, oh.plane_counts(ref, n_harm)), call
            for f in ("harm", "z", "r"):
                assert np.array_equal(got[f], ref[f]), (call, f)
            assert np.array_equal(got["power"].view(np.int32), ref["power"].astype(np.float32).view(np.int32)), call


@pytest.mark.parametrize("z_max,n", [(3, 1 << 18), (3, (1 << 18) + 1), (5, 1 << 19), (3, 1 << 20), (3, (1 << 20) + 1)])
def test_highest_segment_edges(z_max, n):
    n_harm, rows = 8, 2 * z_max + 1
    rng = np.random.default_rng(n)
    plane = rng.exponential(size=(rows, n)).astype(np.float32)
    for row in range(rows):
        plane[row, rng.integers(0, n, 20)] += 40.0
    plane[:, n - 1] += 40.0
    buf = np.full((rows, fdas.fop_ld(n)), np.nan, dtype=np.float32)
    buf[:, :n] = plane
    ta = oh.threshold_array(n_harm, z_max, 1e-6).astype(np.float32)
    ref = oh.candidates(plane, n_harm, ta=ta, index="highest")
    fop, ta_t = torch.from_numpy(buf).to("cuda:0"), torch.from_numpy(ta).to("cuda:0")
    print(f"highest segment edges: n={n} z_max={z_max} candidates={ref.size}", flush=True)
    with fdas.plan_create(z_max=z_max, n_harm=n_harm, n_max=n, hsum_index=fdas.HSUM_HIGHEST) as plan:
        for call in (fdas.harmonic_sum, fdas.harmonic_sum_noalloc):
            cands, counts = fdas.alloc_cands(plan, "cuda:0")
            call(plan, fop, n, cands, counts, ta=ta_t)
            got, hc = fdas.candidates(plan, cands, counts)
            assert np.array_equal(hc, oh.plane_counts(ref, n_harm)), call
            for f in ("harm", "z", "r"):
                assert np.array_equal(got[f], ref[f]), (call, f)
            assert np.array_equal(got["power"].view(np.int32), ref["power"].astype(np.float32).view(np.int32)), call
