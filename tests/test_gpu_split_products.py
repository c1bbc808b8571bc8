"""Which products of the halves the split-BF16 correlation forms.

Every folded value and tap is hi + lo, two BF16 numbers; in BF16 the product
lo * lo is as large as the halves' own rounding and belongs to the sum.  The
contraction is formed here in float64 from the same halves with and without it:
the kernel has to lie within a quarter of the difference of the full one (FP32
accumulation leaves a tenth), which bounds the loss of any of the four products.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1806_01556_amd import fdas, synth  # noqa: E402


def _halves(v):
    v = np.asarray(v, dtype=np.float32)
    rnd = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(torch.bfloat16).to(torch.float32).numpy()  # noqa: E731
    hi = rnd(v)
    return hi.astype(np.float64), rnd(v - hi).astype(np.float64)


def _filter(x, taps, low_low):
    """sum over d of x[j + d] taps[d] for one real part x and real taps d = -P .. P - 1, taps[d] = taps[-d]."""
    P, n = taps.size // 2, x.size
    pad = np.concatenate([np.zeros(P, np.float32), x, np.zeros(P, np.float32)])
    at = lambda d: pad[P + d:P + d + n]  # noqa: E731
    out = at(-P).astype(np.float64) * np.float64(np.float32(taps[0]))  # the unpaired tap stays FP32
    for d in range(P):
        fh, fl = _halves(at(d) + at(-d))
        th, tl = _halves(np.float32(taps[P + d] * (0.5 if d == 0 else 1.0)))
        out += fh * th + fh * tl + fl * th + (fl * tl if low_low else 0.0)
    return out


def test_bf16_keeps_the_product_of_the_low_halves():
    n, z_max = 2000, 42
    spec, _ = synth.make_spectrum(n, 31)
    x = spec.astype(np.complex64)
    print("split products: bf16", flush=True)
    with fdas.plan_create(z_max=z_max, n_max=n, method=fdas.CONV_DIRECT_MFMA, precision=fdas.PREC_SPLIT_BF16) as plan:
        out = torch.zeros((plan.rows, fdas.fop_ld(n)), dtype=torch.float32, device="cuda:0")
        fdas.convolve(plan, torch.from_numpy(x).to("cuda:0"), out, n=n)
        torch.cuda.synchronize()
        got = out.cpu().numpy()[:, :n].astype(np.float64)
    for az in (9, 23, 42):  # z = 0's one tap has no low half, so no such product
        h = fdas.template_taps(az)
        power = {}
        for low_low in (True, False):
            ar, ai = (_filter(p, h.real, low_low) for p in (x.real, x.imag))
            br, bi = (_filter(p, h.imag, low_low) for p in (x.real, x.imag))
            power[low_low] = {az: (ar - bi) ** 2 + (ai + br) ** 2, -az: (ar + bi) ** 2 + (ai - br) ** 2}
        for z in (az, -az):
            full, without, mine = power[True][z], power[False][z], got[z + z_max]
            share = np.linalg.norm(full - without)
            print(f"split products: z={z}: off the full sum {np.linalg.norm(mine - full) / share:.3f}, off the sum without "
                  f"lo*lo {np.linalg.norm(mine - without) / share:.3f} of lo*lo's share", flush=True)
            assert np.linalg.norm(mine - full) <= 0.25 * share
