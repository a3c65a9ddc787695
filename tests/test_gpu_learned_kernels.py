"""The learned early-stop kernels at the edges of their work split: rows and
particles that do not fill a tile, and both sides of each size at which another
form of a kernel is launched."""
import numpy as np
import pytest

import test_gpu_learned as L
from paper_2310_00317_amd import inputs as I

pytestmark = pytest.mark.gpu
P = L.P


@pytest.mark.parametrize("B", [15, 16, 17, 65])
def test_forward_tiles(P, oracle_mod, B):
    """Rows around one tile of 16 and one workgroup of 64."""
    L.test_mlp_forward_matches_oracle(P, B)


@pytest.mark.parametrize("B", [65535, 65536, 65537, 65793, 131072, 131073, 262145])
def test_forward_large_batches(P, oracle_mod, B):
    """One tile of 16 rows per wave below 65,536 rows, four from there on; more
    than 512 workgroups' worth of rows (a pass's, the next read ahead) above
    131,072.  Every row is the same
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


def _betatron(n, seed=4):
    """Two tunes per plane and window (no tracking needed for an oracle of the
    features): x, px, y, py over 1,024 turns, FP32."""
    rng = np.random.default_rng(seed)
    bx, ax, by, ay = L._twiss()
    t = np.arange(1024)[:, None]
    rec = np.empty((1024, 4, n), np.float32)
    for k, (b, a) in enumerate(((bx, ax), (by, ay))):
        q = 0.1 + 0.35 * rng.random(n) + 2e-4 * (t >= 512) * rng.random(n)
        amp = 1e-4 * (1 + 5 * rng.random(n)) * (1 + 2e-4 * t * rng.random(n))
        ph = 2 * np.pi * (q * t + rng.random(n))
        u, pu = amp * np.cos(ph), -amp * np.sin(ph)
        rec[:, 2 * k] = u * np.sqrt(b)
        rec[:, 2 * k + 1] = (pu - a * u) / np.sqrt(b)
    return rec


@pytest.mark.parametrize("n", [1, 3, 4, 5, 1023, 1024, 1025, 1033])
def test_features_groups(P, oracle_mod, n):
    """Groups of four particles to 1,024 of them, of eight above."""
    import torch
    from oracle import features as F
    rec = _betatron(n)
    fg = P.features(torch.tensor(rec, device="cuda"), L._twiss(), L.EMIT, I.CFG1_APERTURE)
    L.assert_features_close(fg.cpu().numpy().astype(np.float64),
                            F.features(rec, L._twiss(), L.EMIT, I.CFG1_APERTURE))


def test_features_wide_offsets(P, oracle_mod):
    """2^22 particles and more take 64-bit offsets: the same bits as the
    particles' copies in a small set."""
    import torch
    small, n = 1032, (1 << 22) + 5
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs a 69 GB record")
    base = torch.tensor(_betatron(small), device="cuda")
    cols = torch.arange(n, device="cuda") % small
    rec = torch.empty((1024, 4, n), dtype=torch.float32, device="cuda")
    for t in range(1024):
        torch.index_select(base[t], 1, cols, out=rec[t])
    fs = P.features(base, L._twiss(), L.EMIT, I.CFG1_APERTURE)
    fw = P.features(rec, L._twiss(), L.EMIT, I.CFG1_APERTURE)
    del rec
    assert torch.equal(fw, fs[cols])
    torch.cuda.empty_cache()


@pytest.mark.parametrize("n", [1, 255, 256, 257, 2047, 2048, 2049, 4500])
@pytest.mark.parametrize("masked", [False, True])
def test_feature_stats_rows(P, oracle_mod, n, masked):
    """256 rows of the workgroup at a time, eight of a thread in flight."""
    import torch
    rng = np.random.default_rng(n)
    f = (rng.normal(size=(n, 16)) * np.arange(1, 17) + 3).astype(np.float32)
    mask = (rng.random(n) < 0.5).astype(np.int32)
    sel = (f[mask != 0] if masked else f).astype(np.float64)
    g = P.feature_stats(torch.tensor(f, device="cuda"),
                        torch.tensor(mask, device="cuda") if masked else None).cpu().numpy()
    mean = sel.mean(0) if len(sel) else np.zeros(16)
    std = sel.std(0) if len(sel) > 1 else np.ones(16)
    assert np.allclose(g[:16], mean, rtol=1e-6, atol=1e-6)
    assert np.allclose(g[16:], 1 / std, rtol=1e-5)
