"""The training loop against the gradient and Adam entry points, step by step
on the same permutations and bit for bit: several epochs, a last batch that is
not full, moments and a step count from an earlier call."""
import numpy as np
import pytest

import test_gpu_learned as L

pytestmark = pytest.mark.gpu
P = L.P


def _mt19937_64(seed):
    """Matsumoto and Nishimura's 64-bit Mersenne twister (the shuffle's generator)."""
    m64, s = (1 << 64) - 1, [seed & ((1 << 64) - 1)]
    for i in range(1, 312):
        s.append((6364136223846793005 * (s[-1] ^ (s[-1] >> 62)) + i) & m64)
    while True:
        for i in range(312):
            v = (s[i] & 0xFFFFFFFF80000000) | (s[(i + 1) % 312] & 0x7FFFFFFF)
            s[i] = s[(i + 156) % 312] ^ (v >> 1) ^ (0xB5026F5AA96619E9 if v & 1 else 0)
        for v in s:
            v ^= (v >> 29) & 0x5555555555555555
            v ^= (v << 17) & 0x71D67FFFEDA60000
            v ^= (v << 37) & 0xFFF7EEE000000000
            yield v ^ (v >> 43)


@pytest.mark.parametrize("n,batch,epochs", [(230, 64, 3), (230, 230, 2), (5000, 1, 1),
                                            (9000, 4100, 2), (20000, 8200, 2)])
def test_training_is_its_steps(P, n, batch, epochs):
    import torch
    theta, x, norm, y = L._net_inputs(n, seed=3)
    w, lr, seed, step = 2.5, 1e-3, 11, 5
    t = lambda a: torch.tensor(a, device="cuda")
    xd, yd, nd = t(x), t(y), t(norm)
    rng = np.random.default_rng(2)
    m0 = (1e-3 * rng.normal(size=len(theta))).astype(np.float32)
    v0 = (1e-6 * rng.random(len(theta))).astype(np.float32)
    got = [t(theta), t(m0), t(v0)]
    steps, losses = P.mlp_train(*got, nd, xd, yd, w, epochs, batch, lr, seed, step=step)
    want = [t(theta), t(m0), t(v0)]
    draws, k, means = _mt19937_64(seed), step, []
    for _ in range(epochs):
        perm = np.arange(n)
        for i in range(n - 1, 0, -1):
            j = next(draws) % (i + 1)
            perm[i], perm[j] = perm[j], perm[i]
        perm, of_batch = t(perm), []
        for b in range(0, n, batch):
            r = perm[b:b + batch]
            g, loss = P.mlp_grad(want[0], nd, xd[r].contiguous(), yd[r].contiguous(), w)
            k += 1
            P.mlp_adam(*want, g, k, lr)
            of_batch.append(loss)
        of_batch = torch.cat(of_batch).cpu().numpy()
        if len(of_batch) <= 4096:   # (the loop keeps the last 4,096 losses)
            means.append(np.float32(of_batch.astype(np.float64).sum() / len(of_batch)))
    assert steps == k
    for a, b in zip(got, want):
        assert torch.equal(a, b)
    if means:
        assert np.allclose(losses, means, rtol=1e-7, atol=0)
