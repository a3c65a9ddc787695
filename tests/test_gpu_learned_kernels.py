"""The learned early-stop kernels at the edges of their work split: rows
that do not fill a tile, and both sides of each size at which another
form of a kernel is launched."""
import numpy as np
import pytest

import test_gpu_learned as L

pytestmark = pytest.mark.gpu
P = L.P


@pytest.mark.parametrize("B", [15, 16, 17, 65])
def test_forward_tiles(P, oracle_mod, B):
    """Rows around one tile of 16 and one workgroup of 64."""
    L.test_mlp_forward_matches_oracle(P, B)


@pytest.mark.parametrize("B", [65535, 65536, 65537, 65793, 262145])
def test_forward_large_batches(P, oracle_mod, B):
    """One tile of 16 rows per wave below 65,536 rows, four from there on; more
    than 1,024 workgroups' worth of rows above 262,144.  Every row is the same
    sums in the same order in both forms: the same bits as in batches of the
    size that is held against the oracle.  (Against the oracle itself, among
    65,535 rows of 256 rounded activations some round the other way than in
    FP64, which moves their logits by more than the few-row tolerance.)"""
    import torch
    theta, x, norm, _ = L._net_inputs(B)
    t = lambda a: torch.tensor(a, device="cuda")
    th, nm, xd = t(theta), t(norm), t(x)
    parts = [P.mlp_forward(th, nm, xd[i:i + 4099]) for i in range(0, B, 4099)]
    assert torch.equal(P.mlp_forward(th, nm, xd), torch.cat(parts))


@pytest.mark.parametrize("B", [1, 63, 65, 4097, 8192, 8193])
def test_gradient_splits(P, oracle_mod, B):
    """Columns split over four blocks to 4,096 rows, two to 8,192, one above."""
    L.test_mlp_gradient_elementwise_bound(P, B)


@pytest.mark.parametrize("n", [1, 64, 230])
def test_training_step_is_gradient_and_adam(P, oracle_mod, n):
    """One epoch of one batch: the first moment is a tenth of the gradient of
    the same rows in another order (FP32 sums of n terms: each within
    (n + 2) 2^-24 of the sum of their magnitudes, twice; 2 % more for the BF16
    roundings inside the magnitudes), and the step is Adam's of the moments
    (FP32 moments, FP64 update: 1e-6 of the weight)."""
    import torch
    from oracle import mlp
    theta, x, norm, y = L._net_inputs(n, seed=9)
    w = 2.5
    t = lambda a: torch.tensor(a, device="cuda")
    g, loss = P.mlp_grad(t(theta), t(norm), t(x), t(y), w)
    th, m, v = t(theta), torch.zeros(len(theta), device="cuda"), torch.zeros(len(theta), device="cuda")
    _, losses = P.mlp_train(th, m, v, t(norm), t(x), t(y), w, 1, n, 1e-3, 3)
    f64 = lambda a: a.cpu().numpy().astype(np.float64)
    g, m, v, th = f64(g), f64(m), f64(v), f64(th)
    f = mlp.forward(theta.astype(np.float64), mlp.standardise(x, norm))
    p = mlp.unpack(theta)
    s = 1.0 / (1.0 + np.exp(-f["z3"]))
    m3 = np.abs(s * (w * y + (1 - y)) - w * y) / n
    m2 = np.outer(m3, np.abs(p["w3"]))
    m1 = m2 @ np.abs(p["W2"]).T
    scale = mlp.pack({"b3": np.array([m3.sum()]), "w3": np.abs(f["H2"]).T @ m3,
                      "b2": m2.sum(0), "W2": np.abs(f["H1"]).T @ m2,
                      "b1": m1.sum(0), "W1": np.abs(f["X"]).T @ m1})
    assert np.all(np.abs(10 * m - g) <= 2 * (n + 2) * 2.0 ** -24 * 1.02 * scale + 1e-12)
    want = theta - 1e-3 * (m / 0.1) / (np.sqrt(v / 1e-3) + 1e-8)
    assert np.all(np.abs(th - want) <= 1e-6 * np.abs(want) + 1e-9)
    assert abs(losses[0] - float(loss.cpu()[0])) <= 2 * (n + 2) * 2.0 ** -24 * abs(losses[0])
