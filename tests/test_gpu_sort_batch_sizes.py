"""Ordering of a batch's candidates: bucket sizes around the kernels' limits, and
batches of many trials with few records.

A wave orders up to 512 records of one (plane, row) in a batch, over 64, 128, 256
and 512 keys; a workgroup those above.  The plan is called twice without more
trials, so that the second call finds the counters as the first left them, with
empty trials between full ones.  And 1024 trials of 10 records may not take longer
than in the radix sort of longer lists (1.25 x for the noise of the box; best of
15 calls each, in turn).
"""

import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1806_01556_amd import fdas  # noqa: E402

N = 1 << 20


def _trial(sizes, z_max, nh, cap, seed):
    """(records in order, device lists, device counts) of {(plane, row): records}."""
    rng = np.random.default_rng(seed)
    buf = np.zeros((nh, cap), dtype=fdas.CAND_DTYPE)
    ordered, counts = [], []
    for k in range(nh):
        recs = []
        for (kk, row), c in sorted(sizes.items()):
            if kk == k:
                v = np.zeros(c, dtype=fdas.CAND_DTYPE)
                v["harm"], v["z"] = k + 1, row - z_max
                v["r"] = np.sort(rng.choice(N, size=c, replace=False))
                v["power"] = 20.0 + rng.exponential(size=c)
                recs.append(v)
        v = np.concatenate(recs) if recs else np.zeros(0, dtype=fdas.CAND_DTYPE)
        ordered.append(v)
        counts.append(v.size)
        buf[k, :v.size] = v[rng.permutation(v.size)]
    return (np.concatenate(ordered), torch.from_numpy(buf.reshape(-1).view(np.int32).copy()).to("cuda:0"),
            torch.tensor(counts, dtype=torch.int32, device="cuda:0"))


SIZES = [1, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1023, 1025, 4095, 4096, 4097]


@pytest.mark.parametrize("trials", [1, 2, 7])
def test_bucket_sizes_of_a_batch(trials):
    nh, z_max, cap = 3, 42, 20_000
    print(f"batch buckets: trials={trials}", flush=True)
    with fdas.plan_create(n_max=N, z_max=z_max, n_harm=nh, cand_capacity=cap) as plan:
        for turn in range(2):
            sets = []
            for i in range(trials):
                rows = {} if i % 3 == 1 else {((q + i) % nh, (5 * q + i) % 85): c for q, c in enumerate(SIZES)}
                if i == 6:  # a trial of one record
                    rows = {(2, 84): 1}
                sets.append(_trial(rows, z_max, nh, cap, 10 * i + turn))
            arr = fdas.trials_array([(0, N, 0, N, c, n) for _, c, n in sets])
            got, hc = fdas.candidates_batch(plan, arr, capacity=sum(s[0].size for s in sets) + 1)
            for i, (ref, _, n) in enumerate(sets):
                assert np.array_equal(got[i], ref), (turn, i)
                assert np.array_equal(hc[i], n.cpu().numpy())


@pytest.mark.parametrize("per_plane", [0, 1, 40, 300])
def test_many_trials_of_few_records(per_plane):
    # every trial of the batch reads the same lists: nothing is written to them
    nh, z_max, cap, trials = 8, 42, 65_536, 1024
    rows = {(k, (11 * k + q) % 85): 1 + (per_plane // 85 if q < 84 else 0) for k in range(nh) for q in range(min(per_plane, 85))}
    ref, cands, counts = _trial(rows, z_max, nh, cap, per_plane)
    print(f"many trials: {ref.size} records each", flush=True)
    with fdas.plan_create(n_max=N, z_max=z_max, n_harm=nh, cand_capacity=cap) as plan:
        arr = fdas.trials_array([(0, N, 0, N, cands, counts)] * trials)
        for _ in range(2):
            got, _ = fdas.candidates_batch(plan, arr, capacity=trials * ref.size + 1)
            assert all(np.array_equal(g, ref) for g in got)


def test_many_trials_take_no_longer_than_the_radix_sort():
    nh, z_max, trials = 8, 42, 1024
    plans = {cap: fdas.plan_create(n_max=N, z_max=z_max, n_harm=nh, cand_capacity=cap) for cap in (65_536, 65_537)}
    best, lists = {}, {}
    try:
        for cap in plans:
            ref, cands, counts = _trial({(k, 5 + k): 2 for k in range(5)}, z_max, nh, cap, 1)
            lists[cap] = (cands, counts, fdas.trials_array([(0, N, 0, N, cands, counts)] * trials))
        for _ in range(15):
            for cap, plan in plans.items():
                torch.cuda.synchronize()
                t = time.perf_counter()
                fdas.candidates_batch(plan, lists[cap][2], capacity=trials * ref.size, copy=False)
                best[cap] = min(best.get(cap, 1.0), time.perf_counter() - t)
    finally:
        for plan in plans.values():
            plan.destroy()
    print(f"many trials: buckets {1e6 * best[65_536]:.1f} us, radix {1e6 * best[65_537]:.1f}", flush=True)
    assert best[65_536] <= 1.25 * best[65_537]
