"""Training gradient of the pre-screen at the edges of its work split.

The weight-gradient kernel deals 8, 2 and half units per sample of the three
32-channel layers to at most 390, 98 and 24 workgroups, the convolutions run
at most 512 tiles at a time: the batches below hold fewer units than
workgroups, one more than fills them (25, 49 samples), and several rounds of
tiles (129, 257).  A batch repeats five distinct blocks, so the oracle's mean
gradient is their weighted mean; bound as in the other gradient test (5e-3 of
each tensor's norm: max-pool positions and ReLU signs are decided in FP32 on
the GPU and in FP64 in the oracle).  Features start at an odd
float, as a caller's slice may.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import prescreen as ops  # noqa: E402
from paper_1806_01556_amd import fdas  # noqa: E402


def _bf16(a):
    return torch.from_numpy(np.asarray(a, dtype=np.float32)).to(torch.bfloat16).to(torch.float64).numpy()


@pytest.mark.parametrize("nb", [1, 2, 3, 24, 25, 49, 129, 257])
def test_gradient_over_partial_and_full_rounds(nb):
    rng = np.random.default_rng(41)
    P = rng.exponential(size=(5, 4096))
    for b in (0, 2, 3):
        t0 = int(rng.integers(100, 3900))
        P[b, t0:t0 + 20] += rng.uniform(5, 40)
    X = ops.features(P).astype(np.float32)
    y = np.array([1, 0, 1, 1, 0], dtype=np.float32)
    theta = fdas.prescreen_init_params(6)
    theta[-33:-1] *= 4.0
    one = [ops.batch_loss_grad(_bf16(theta), X[i:i + 1].astype(np.float64), y[i:i + 1], 3.0) for i in range(5)]
    pick = np.arange(nb) % 5
    ref_loss = np.mean([one[i][0] for i in pick])
    ref = np.mean([one[i][1] for i in pick], axis=0)
    print(f"gradient units: nb={nb}", flush=True)
    ps = fdas.Prescreen(max_batch=nb)
    try:
        ps.set_params(theta)
        flat = torch.zeros(nb * 4096 + 1, device="cuda:0")
        flat[1:] = torch.from_numpy(X[pick].ravel())
        feats = flat[1:]
        labels = torch.from_numpy(y[pick]).to("cuda:0")
        logits, loss = torch.zeros(nb, device="cuda:0"), torch.full((1,), 9.0, device="cuda:0")
        for _ in range(2):  # the second call finds the first one's partials in its workspace
            grad = torch.full((ps.param_count(),), 7.0, device="cuda:0")
            ps.gradient(feats, labels, nb, 3.0, logits, loss, grad)
        got = grad.cpu().numpy().astype(np.float64)
    finally:
        ps.destroy()
    assert abs(float(loss.item()) - ref_loss) <= 1e-4 * (1.0 + ref_loss)
    offs = np.cumsum([0] + [int(np.prod(s)) for s in ops.param_shapes()])
    for a, b in zip(offs[:-1], offs[1:]):
        assert np.linalg.norm(got[a:b] - ref[a:b]) <= 5e-3 * np.linalg.norm(ref[a:b]) + 1e-12
