"""Direct methods with narrow banks.

Banks of one tile (z_max <= 7) run in FP32 whatever precision is asked for: the plane
is the FP32 plan's bit for bit, and the call takes no longer (1.15 x for the box).
Banks of two tiles (z_max 8 .. 15) take four parts of 128 bins to a staged strip
from 262,144 bins on: lengths that end in every part, bad bins at the parts'
edges, against the FP64 oracle with the methods' own bounds.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import fop as ofop  # noqa: E402
from paper_1806_01556_amd import fdas, synth  # noqa: E402

SPLITS = [(fdas.PREC_SPLIT_FP16, 1e-4), (fdas.PREC_SPLIT_BF16, 4e-3)]


def _plane(x, z_max, prec):
    n = x.shape[0]
    with fdas.plan_create(z_max=z_max, n_max=n, method=fdas.CONV_DIRECT_MFMA, precision=prec) as plan:
        out = torch.full((plan.rows, fdas.fop_ld(n)), -1.0, dtype=torch.float32, device="cuda:0")
        fdas.convolve(plan, x, out, n=n)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
    assert np.all(got[:, n:] == -1.0), "columns >= n must not be written"
    return got[:, :n]


@pytest.mark.parametrize("prec", [p for p, _ in SPLITS])
@pytest.mark.parametrize("z_max", [0, 3, 7])
def test_one_tile_runs_in_fp32(prec, z_max):
    spec, _ = synth.make_spectrum(70_001, 5)
    x = torch.from_numpy(spec.astype(np.complex64)).to("cuda:0")
    print(f"narrow banks: z_max={z_max} prec={prec}", flush=True)
    assert np.array_equal(_plane(x, z_max, prec), _plane(x, z_max, fdas.PREC_FP32))


@pytest.mark.parametrize("prec,tol", SPLITS)
@pytest.mark.parametrize("z_max,n", [(8, 262_144), (8, 262_145), (15, 262_144 + 129), (12, 262_144 + 383), (9, 270_000)])
def test_two_tiles_in_four_parts(prec, tol, z_max, n):
    spec, _ = synth.make_spectrum(n, 60 + z_max)
    x = spec.astype(np.complex64)
    clean = spec.astype(np.complex128)
    bad = [0, 127, 128, 511, 512, n // 2, n - 1]
    x[bad] = np.nan
    clean[bad] = 0.0
    print(f"narrow banks: z_max={z_max} n={n} prec={prec}", flush=True)
    got = _plane(torch.from_numpy(x).to("cuda:0"), z_max, prec)
    touched = np.zeros(got.shape, dtype=bool)
    for i in range(2 * z_max + 1):
        half = fdas.template_taps(i - z_max).size // 2
        for b in bad:
            touched[i, max(0, b - half + 1):min(n, b + half + 1)] = True
    ref = ofop.fop(clean, z_max=z_max)
    assert np.all((np.abs(got - ref) <= tol * np.maximum(ref, 1.0))[~touched])
    assert np.all(np.isnan(got[touched]))


@pytest.mark.parametrize("prec", [p for p, _ in SPLITS])
@pytest.mark.parametrize("z_max", [0, 3])
def test_split_of_narrow_banks_takes_no_longer_than_fp32(prec, z_max):
    n = 1 << 21
    x = torch.randn(n, 2, device="cuda:0", generator=torch.Generator(device="cuda:0").manual_seed(2))
    best = {}
    for which in (prec, fdas.PREC_FP32):
        with fdas.plan_create(z_max=z_max, n_max=n, method=fdas.CONV_DIRECT_MFMA, precision=which) as plan:
            out = fdas.alloc_fop(plan, n)
            for _ in range(8):
                e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                e0.record()
                for _ in range(10):
                    fdas.convolve(plan, x, out, n=n)
                e1.record()
                torch.cuda.synchronize()
                best[which] = min(best.get(which, 1e9), e0.elapsed_time(e1) / 10)
    print(f"narrow banks: z_max={z_max} split {1e3 * best[prec]:.1f} us, FP32 {1e3 * best[fdas.PREC_FP32]:.1f}", flush=True)
    assert best[prec] <= 1.15 * best[fdas.PREC_FP32]
