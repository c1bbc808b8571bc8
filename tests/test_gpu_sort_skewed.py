"""Ordering of lists that crowd into few (plane, row) buckets.

A row that interference fills, or a plan of few rows, brings up to 65,536
records to one bucket: more than 4096 are divided among workgroups by rank.
Sizes at the edges of the division, r spread, consecutive, in two clusters and
all alike (positions then decide the division), through the copying, the mapped
and the batch readback, against numpy's sort.  And such a list may take no longer
than in the radix sort of longer lists, which spreads any list over the chip
(1.25 x for the noise of the box; best of 20 calls each, in turn).
"""

import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1806_01556_amd import fdas  # noqa: E402

N = 1 << 22
CAP = 65_536


def _row(c, how, rng):
    if how == "spread":
        return rng.choice(N, size=c, replace=False)
    if how == "run":
        return 3 + rng.permutation(c)
    if how == "ascending":
        return N - c + np.arange(c)
    if how == "clusters":
        return np.concatenate([rng.permutation(c // 2), N - 1 - rng.permutation(c - c // 2)])
    return np.full(c, 77)


def _plane(k, z_max, rows, rng):
    recs = []
    for row, c, how in rows:
        v = np.zeros(c, dtype=fdas.CAND_DTYPE)
        v["harm"], v["z"], v["r"] = k + 1, row - z_max, _row(c, how, rng)
        v["power"] = 20.0 + rng.exponential(size=c)
        recs.append(v)
    return np.concatenate(recs) if recs else np.zeros(0, dtype=fdas.CAND_DTYPE)


def _upload(planes, cap):
    buf = np.zeros((len(planes), cap), dtype=fdas.CAND_DTYPE)
    for k, v in enumerate(planes):
        buf[k, :v.size] = v
    return (torch.from_numpy(buf.reshape(-1).view(np.int32).copy()).to("cuda:0"),
            torch.tensor([v.size for v in planes], dtype=torch.int32, device="cuda:0"))


def _canon(v):
    """(harm, z, r, power) order: equal cells, which no harmonic sum makes, may come in any."""
    return v[np.lexsort((v["power"], v["r"], v["z"], v["harm"]))]


def _check(got, planes):
    got = np.asarray(got)
    key = (got["harm"].astype(np.int64) * 256 + got["z"] + 64) * (1 << 32) + got["r"]
    assert np.all(np.diff(key) >= 0)
    assert np.array_equal(_canon(got), _canon(np.concatenate(planes)))


CASES = {
    "edges": (42, [[(0, 4096, "spread"), (84, 4097, "spread")], [(3, 8191, "run")], [(3, 8192, "run"), (4, 8193, "spread")],
                   [(7, 12_289, "clusters")], []]),
    "full rows": (42, [[(42, CAP, how)] for how in ("spread", "run", "ascending", "clusters")]),
    "alike": (3, [[(0, 5000, "alike"), (1, 5000, "spread")], [(6, CAP, "alike")]]),
    "one row": (0, [[(0, CAP, "spread")]] * 8),
    "early": (1, [[(1, 8192, "spread")]]),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_large_buckets(name):
    z_max, rows = CASES[name]
    rng = np.random.default_rng(len(name))
    planes = [_plane(k, z_max, r, rng) for k, r in enumerate(rows)]
    print(f"skewed lists: {name}", flush=True)
    with fdas.plan_create(n_max=N, z_max=z_max, n_harm=len(rows), cand_capacity=CAP) as plan:
        cands, counts = _upload(planes, CAP)
        for _ in range(2):  # the second round finds the counters as the first left them
            _check(fdas.candidates(plan, cands, counts)[0], planes)
            _check(fdas.candidates(plan, cands, counts, capacity=sum(v.size for v in planes))[0], planes)
        small = [_plane(k, z_max, [(0, 9, "spread")], rng) for k in range(len(rows))]
        sc, sn = _upload(small, CAP)
        trials = fdas.trials_array([(0, N, 0, N, sc, sn), (0, N, 0, N, cands, counts), (0, N, 0, N, sc, sn)])
        for _ in range(2):
            got, _ = fdas.candidates_batch(plan, trials, capacity=sum(v.size for v in planes) + 200)
            _check(got[0], small)
            _check(got[1], planes)
            _check(got[2], small)


@pytest.mark.parametrize("z_max,rows", [(42, [[(42, CAP, "spread")]]), (42, [[(42, CAP, "ascending")]]),
                                        (42, [[(5, 12_000, "spread")]]), (0, [[(0, CAP, "spread")]] * 8)])
def test_skewed_lists_take_no_longer_than_the_radix_sort(z_max, rows):
    rng = np.random.default_rng(3)
    planes = [_plane(k, z_max, r, rng) for k, r in enumerate(rows)]
    best = {}
    plans = {cap: fdas.plan_create(n_max=N, z_max=z_max, n_harm=len(rows), cand_capacity=cap) for cap in (CAP, CAP + 1)}
    try:
        lists = {cap: _upload(planes, cap) for cap in plans}
        for _ in range(20):
            for cap, plan in plans.items():
                torch.cuda.synchronize()
                t = time.perf_counter()
                fdas.candidates(plan, *lists[cap], copy=False)
                best[cap] = min(best.get(cap, 1.0), time.perf_counter() - t)
    finally:
        for plan in plans.values():
            plan.destroy()
    print(f"skewed lists: {[[r[0][1:] for r in rows][:2]]}: buckets {1e6 * best[CAP]:.1f} us, radix {1e6 * best[CAP + 1]:.1f}",
          flush=True)
    assert best[CAP] <= 1.25 * best[CAP + 1]
