"""Quiet bins beside a strong line in the split-FP16 correlation.

The kernel scales its strip of the spectrum by a power of two and carries every
value as two FP16 halves, so far below the strip's largest value what is left
of a value is a multiple of 2^-24 in scaled units, whatever its size.  Every bin
below lies 2^24 under a line that each strip holds; only cells whose own
support holds no line are looked at.  With the line brought to 2^14 (the widest
scale that keeps the sum of two bins below FP16's 65504) and every bin rounded by
itself, the error of a cell's amplitude has the variance
2 s^2 sum |h|^2 over its taps, s = 2^-24 / sqrt(12) / 2^14; rounding the sum of the
two bins that share a tap halves it.  Half that scale would double the error.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import fop as ofop  # noqa: E402
from paper_1806_01556_amd import fdas  # noqa: E402


@pytest.mark.parametrize("line", [1.0, 1.75, -1.998])
def test_quiet_bins_keep_their_low_half(line):
    n, z_max, step = 20_000, 42, 640  # a strip covers 768 bins
    rng = np.random.default_rng(5)
    x = (rng.standard_normal(n) + 1j * rng.standard_normal(n)) * 2.0 ** -24
    lines = np.arange(0, n, step)
    x[lines] = line
    x = x.astype(np.complex64)
    print(f"split strip: line={line}", flush=True)
    with fdas.plan_create(z_max=z_max, n_max=n, method=fdas.CONV_DIRECT_MFMA, precision=fdas.PREC_SPLIT_FP16) as plan:
        out = torch.zeros((plan.rows, fdas.fop_ld(n)), dtype=torch.float32, device="cuda:0")
        fdas.convolve(plan, torch.from_numpy(x).to("cuda:0"), out, n=n)
        torch.cuda.synchronize()
        got = out.cpu().numpy()[:, :n].astype(np.float64)
    quiet = x.astype(np.complex128)
    quiet[lines] = 0.0  # the cells looked at hold none
    ref = ofop.fop(quiet, z_max=z_max)
    gap = np.abs(np.arange(n)[:, None] - lines[None, :]).min(axis=1)
    s = 2.0 ** -24 / np.sqrt(12) / 2.0 ** 14
    e2 = []
    for i in range(2 * z_max + 1):
        h = fdas.template_taps(i - z_max)
        use = (gap > h.size // 2 + 1) & (np.arange(n) < lines[-1])
        # dP = 2 Re(conj(Y) dY): variance 2 P E|dY|^2
        var = 2 * ref[i, use] * 2 * s * s * np.sum(np.abs(h) ** 2)
        e2.append((got[i, use] - ref[i, use]) ** 2 / var)
    rms = float(np.sqrt(np.mean(np.concatenate(e2))))
    print(f"split strip: line={line}: rms error {rms:.3f} of one rounding per bin", flush=True)
    assert rms <= 1.0
