"""Ordering of candidate lists fed directly, against numpy's lexsort.

Lists of up to 65,536 records per plane are ordered by (plane, row) buckets,
longer ones by a radix sort of the whole key: the same lists go through a plan
on either side of the line and through the copying, the mapped and the batch
readback.  Bucket sizes: empty, one record, around the bitonic sizes (64, 128,
256), and 4096 / 4097 / 12,000 records of one row, where a bucket no longer fits
in LDS.  The N_cand selection keeps the highest powers, ties to the lower (z, r).
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1806_01556_amd import fdas  # noqa: E402

N = 20_000


def _lists(nh, z_max, sizes, seed):
    """Per plane: shuffled records; sizes[(plane, row)] of them in that bucket."""
    rng = np.random.default_rng(seed)
    planes = []
    for k in range(nh):
        recs = []
        for (kk, row), c in sizes.items():
            if kk == k:
                v = np.zeros(c, dtype=fdas.CAND_DTYPE)
                v["harm"], v["z"] = k + 1, row - z_max
                v["r"] = rng.choice(N, size=c, replace=False)
                v["power"] = 20.0 + np.round(rng.exponential(size=c) * 8) / 8  # ties
                recs.append(v)
        v = np.concatenate(recs) if recs else np.zeros(0, dtype=fdas.CAND_DTYPE)
        planes.append(v[rng.permutation(v.size)])
    return planes


def _upload(planes, cap):
    buf = np.zeros((len(planes), cap), dtype=fdas.CAND_DTYPE)
    for k, v in enumerate(planes):
        buf[k, :v.size] = v
    return (torch.from_numpy(buf.reshape(-1).view(np.int32).copy()).to("cuda:0"),
            torch.tensor([v.size for v in planes], dtype=torch.int32, device="cuda:0"))


def _ordered(planes, top_k=0):
    out = []
    for v in planes:
        if top_k and v.size > top_k:
            v = v[np.lexsort((v["r"], v["z"], -v["power"]))[:top_k]]
        out.append(v[np.lexsort((v["r"], v["z"]))])
    return np.concatenate(out)


CASES = {
    "empty": (8, 42, {}),
    "single": (1, 0, {(0, 0): 1}),
    "bitonic": (4, 3, {(0, 0): 64, (0, 6): 65, (1, 2): 128, (1, 3): 129, (2, 0): 1, (3, 1): 256, (3, 6): 257}),
    "rows": (8, 64, {(k, r): 3 + (7 * r + k) % 40 for k in range(8) for r in range(129)}),
    "lds": (2, 1, {(0, 1): 4096, (0, 2): 4095, (1, 0): 4097, (1, 1): 2, (1, 2): 12_000}),
}


@pytest.mark.parametrize("top_k", [0, 100])
@pytest.mark.parametrize("cap", [20_000, 65_536, 65_537])
@pytest.mark.parametrize("name", sorted(CASES))
def test_readbacks_match_lexsort(name, cap, top_k):
    nh, z_max, sizes = CASES[name]
    print(f"sort buckets: {name} cap={cap} top_k={top_k}", flush=True)
    with fdas.plan_create(n_max=N, z_max=z_max, n_harm=nh, cand_capacity=cap, top_k=top_k) as plan:
        for seed in (1, 2):  # the second call finds the counters as the first left them
            planes = _lists(nh, z_max, sizes, seed)
            cands, counts = _upload(planes, cap)
            ref = _ordered(planes, top_k)
            got, hc = fdas.candidates(plan, cands, counts)  # mapped
            copied, _ = fdas.candidates(plan, cands, counts, capacity=max(ref.size, 1))
            assert np.array_equal(hc, [v.size for v in planes])
            assert np.array_equal(got, ref) and np.array_equal(copied, ref)


@pytest.mark.parametrize("cap", [20_000, 65_537])
def test_batch_readback_matches_lexsort(cap):
    nh, z_max = 2, 1
    with fdas.plan_create(n_max=N, z_max=z_max, n_harm=nh, cand_capacity=cap) as plan:
        for count in (3, 9):  # the second call grows the trials' counters
            sets = [_lists(nh, z_max, {(0, 0): 5 * i, (0, 2): 40, (1, 1): 4090 + 3 * i} if i % 3 else {}, i)
                    for i in range(count)]
            ups = [_upload(p, cap) for p in sets]
            trials = fdas.trials_array([(0, N, 0, N, c, n) for c, n in ups])
            got, hc = fdas.candidates_batch(plan, trials, capacity=count * 30_000)
            for i in range(count):
                assert np.array_equal(got[i], _ordered(sets[i])), i
                assert np.array_equal(hc[i], [v.size for v in sets[i]])
