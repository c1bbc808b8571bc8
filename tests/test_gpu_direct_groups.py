"""GPU parity of the direct FP32 correlation at the edges of its work split.

The kernel covers 256 bins per workgroup block and runs groups of up to six
8-slot tiles of |z| per launch: the template counts below fill one tile
exactly (z_max = 7), start a second with one slot (8), fill the widest single
group (39: five tiles), and need two launches (48, 64); the lengths end one
bin before, at and after a block, a wave's 64 bins and a 16-bin sub-tile, and
cover more blocks than resident workgroups.  Same bound as the other
correlations: |P - P_ref| <= 1e-4 max(P_ref, 1) against the FP64 oracle.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import fop as ofop  # noqa: E402
from paper_1806_01556_amd import fdas, synth  # noqa: E402

TOL = 1e-4


@pytest.mark.parametrize("z_max,n", [(7, 255), (8, 257), (39, 256), (48, 1023), (64, 65), (42, 15), (3, 150_001)])
def test_direct_fp32_group_and_block_edges(z_max, n):
    spec, _ = synth.make_spectrum(n, 900 + z_max)
    x = torch.from_numpy(spec).to("cuda:0")
    print(f"direct groups: n={n} z_max={z_max}", flush=True)
    with fdas.plan_create(z_max=z_max, n_max=n, method=fdas.CONV_DIRECT_MFMA) as plan:
        out = torch.full((plan.rows, fdas.fop_ld(n)), float("nan"), dtype=torch.float32, device="cuda:0")
        fdas.convolve(plan, x, out, n=n)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
    ref = ofop.fop(spec.astype(np.complex128), z_max=z_max)
    assert np.all(np.abs(got[:, :n] - ref) <= TOL * np.maximum(ref, 1.0))
    assert np.all(np.isnan(got[:, n:])), "columns >= n must not be written"


@pytest.mark.parametrize("prec,tol", [(fdas.PREC_SPLIT_FP16, 1e-4), (fdas.PREC_SPLIT_BF16, 4e-3)])
@pytest.mark.parametrize("z_max,n", [(7, 127), (8, 129), (39, 128), (48, 1023), (64, 33), (42, 15), (3, 150_001)])
def test_direct_split_group_and_block_edges(prec, tol, z_max, n):
    """The split kernels: 128-bin blocks, odd and even step counts of 32 distances,
    groups as above; the bounds are the split precisions' own (FP16 keeps 22
    significand bits, BF16 16)."""
    spec, _ = synth.make_spectrum(n, 950 + z_max)
    x = torch.from_numpy(spec).to("cuda:0")
    print(f"split groups: prec={prec} n={n} z_max={z_max}", flush=True)
    with fdas.plan_create(z_max=z_max, n_max=n, method=fdas.CONV_DIRECT_MFMA, precision=prec) as plan:
        out = torch.full((plan.rows, fdas.fop_ld(n)), float("nan"), dtype=torch.float32, device="cuda:0")
        fdas.convolve(plan, x, out, n=n)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
    ref = ofop.fop(spec.astype(np.complex128), z_max=z_max)
    assert np.all(np.abs(got[:, :n] - ref) <= tol * np.maximum(ref, 1.0))
    assert np.all(np.isnan(got[:, n:])), "columns >= n must not be written"
