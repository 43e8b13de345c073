"""Gradient of the limiter's training around the sizes of its kernel, a chunk
of 128 records per block (16 per wave) and a grid of 256 blocks, and on half a
million records, where every wave sweeps 15 or 16 chunks, against float64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _records(rng, m):
    R = np.zeros((m, 40), np.float32)
    R[:, :14] = rng.uniform(-1, 1, (m, 14))
    R[:, 14:18] = rng.normal(size=(m, 4))
    R[:, 36:40] = 0.1 * rng.uniform(-1, 1, (m, 4))
    R[:, 32:36] = R[:, 36:40] * rng.uniform(-0.3, 1.7, (m, 4))
    R[:, 18:22] = 0.5 * (R[:, 32:36] + R[:, 36:40])
    R[:, 22] = rng.uniform(1, 3, m)
    R[:, 23:27] = R[:, 14:18] + 0.05 * rng.normal(size=(m, 4))
    R[:, 27] = 1.0
    return R


def _reference(w, R, wv):
    """Loss and gradient as means over the records, and the mean magnitude of
    what is summed for each, in float64."""
    w, R, wv = (np.asarray(a, np.float64) for a in (w, R, wv))
    W1, b1, W2 = w[:448].reshape(32, 14), w[448:480], w[480:1504].reshape(32, 32)
    b2, W3, b3 = w[1504:1536], w[1536:1568], w[1568]
    x, q, s, d, t, sb, sf = R[:, :14], R[:, 14:18], R[:, 18:22], R[:, 22:23], R[:, 23:27], R[:, 32:36], R[:, 36:40]
    a1 = np.maximum(x @ W1.T + b1, 0)
    a2 = np.maximum(a1 @ W2.T + b2, 0)
    phi = (1 / (1 + np.exp(-(a2 @ W3 + b3))))[:, None]
    same, lim = sb * sf > 0, 2 * np.minimum(abs(sb), abs(sf))
    clip = np.where(same, np.copysign(np.minimum(abs(phi * s), lim), sf), 0)
    res = q + d * clip - t
    pull = np.where(same & (abs(phi * s) < lim), 2 * wv * res * d * np.copysign(abs(s), sf), 0)
    dz = pull.sum(1, keepdims=True) * phi * (1 - phi)
    d2 = np.where(a2 > 0, dz * W3, 0)
    d1 = np.where(a1 > 0, d2 @ W2, 0)
    n = len(R)

    def sums(f):
        return np.concatenate([(f(d1).T @ f(x)).ravel(), f(d1).sum(0), (f(d2).T @ f(a1)).ravel(), f(d2).sum(0),
                               (f(dz) * f(a2)).sum(0), f(dz).sum(0)]) / n
    return (wv * res * res).sum() / n, sums(lambda v: v), sums(np.abs)


@pytest.mark.parametrize("n", [112, 127, 128, 129, 255, 257, 32767, 32768, 32769, 65537, 500000])
def test_gradient_around_the_chunks(n):
    import torch

    from paper_2307_16758_amd import swe
    from paper_2307_16758_amd.limiter_train import WV, init_params
    rng = np.random.default_rng(n)
    w = init_params(3)
    w[448:480] = rng.normal(0, 0.1, 32)
    w[1504:1536] = rng.normal(0, 0.1, 32)
    m = n + 5
    R = _records(rng, m)
    idx = rng.permutation(m)[:n].astype(np.int32)
    idx[7], idx[n - 1] = -1, m                     # absent; the mean counts them
    tr = swe.Trainer(w)
    loss, g = tr.loss_grad(torch.from_numpy(R.ravel()).cuda(), torch.from_numpy(idx).cuda(), WV)
    tr.close()
    V = R[idx[(idx >= 0) & (idx < m)]]
    lo, go, mag = _reference(w, V, WV)
    share = len(V) / n
    # FP32 throughout but for the sum over a block's waves and over the blocks
    # (double).  A term carries the roundings (6e-8) of about 15 + 33 + 33
    # products and sums forward and 34 back, some 1e-5 of its size at worst and
    # of either sign, so far less in their mean; a wave's sum of 16 chunks adds
    # 64 more, 4e-6 of the terms' size at worst.  A switch of ReLU or clip at a
    # tie takes a share of 1e-6 of the records.
    assert abs(loss - lo * share) <= 5e-6 * lo
    assert np.all(np.abs(g - go * share) <= 1.5e-5 * mag + 1e-30)
