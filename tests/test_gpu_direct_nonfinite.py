"""Non-finite and very large bins in the direct correlations.

A cell is a sum over its own template's taps, so a NaN or an infinity in the
spectrum reaches exactly the cells whose support holds that bin: the kernels
multiply tiles of eight |z| over the widest member's distances and add the bins
on both sides of a cell first, and neither the padded zero taps of a narrower
template nor that sum may carry it further.  The bad bins below lie at block
edges and inside; 3e38 is finite, but the sum of two such bins is not.  Other
cells keep the methods' usual bounds against the FP64 oracle.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import fop as ofop  # noqa: E402
from paper_1806_01556_amd import fdas, synth  # noqa: E402

BAD = {0: np.nan, 255: np.inf, 640: -np.inf, 1407: np.nan, 2048: 3e38, 2999: np.inf}


def _supports(n, z_max, bins):
    """[row, column]: the cell's support (offsets -L/2 .. L/2 - 1) holds one of the bins."""
    hit = np.zeros((2 * z_max + 1, n), dtype=bool)
    for i in range(2 * z_max + 1):
        half = fdas.template_taps(i - z_max).size // 2
        for b in bins:
            hit[i, max(0, b - half + 1):min(n, b + half + 1)] = True
    return hit


@pytest.mark.parametrize("prec,tol", [(fdas.PREC_FP32, 1e-4), (fdas.PREC_SPLIT_FP16, 1e-4),
                                      (fdas.PREC_SPLIT_BF16, 4e-3)])
@pytest.mark.parametrize("z_max", [3, 42, 64])
def test_bad_bins_reach_their_own_supports_only(prec, tol, z_max):
    n = 3000
    spec, _ = synth.make_spectrum(n, 77)
    clean = spec.astype(np.complex128)
    bad = spec.astype(np.complex64)
    for b, v in BAD.items():
        clean[b] = 0.0
        bad[b] = np.complex64(complex(v, 0.25))
    print(f"direct non-finite: prec={prec} z_max={z_max}", flush=True)
    with fdas.plan_create(z_max=z_max, n_max=n, method=fdas.CONV_DIRECT_MFMA, precision=prec) as plan:
        out = torch.full((plan.rows, fdas.fop_ld(n)), -1.0, dtype=torch.float32, device="cuda:0")
        fdas.convolve(plan, torch.from_numpy(bad).to("cuda:0"), out, n=n)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
    assert np.all(got[:, n:] == -1.0), "columns >= n must not be written"
    got = got[:, :n]
    touched = _supports(n, z_max, BAD)
    ref = ofop.fop(clean, z_max=z_max)
    ok = np.abs(got - ref) <= tol * np.maximum(ref, 1.0)
    assert np.all(ok[~touched]), f"{np.count_nonzero(~ok & ~touched)} cells without a bad bin in their support"
    nan = _supports(n, z_max, [b for b, v in BAD.items() if np.isnan(v)])
    inf = _supports(n, z_max, [b for b, v in BAD.items() if np.isinf(v)])
    assert np.all(np.isnan(got[nan]))
    assert not np.any(np.isfinite(got[nan | inf]))
    if prec == fdas.PREC_FP32:
        # one infinity times taps with non-zero parts: the power is infinite, above any threshold
        one = sum(_supports(n, z_max, [b]).astype(int) for b, v in BAD.items() if np.isinf(v)) == 1
        alone = one & inf & ~_supports(n, z_max, [b for b, v in BAD.items() if not np.isinf(v)])
        for i in range(2 * z_max + 1):
            h = fdas.template_taps(i - z_max)
            if np.all(h.real.astype(np.float32) != 0) and np.all(h.imag.astype(np.float32) != 0):
                assert np.all(np.isposinf(got[i][alone[i]])), i
