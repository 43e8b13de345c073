"""Gradient of the limiter's training at batch sizes around the 16 records of
a wave, the 64 of a block and the 512 blocks of a grid, with absent records
and a record array that is not 16-byte aligned, against the oracle."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 17, 63, 65, 1000, 33000])
@pytest.mark.parametrize("offset", [0, 3])
def test_gradient_at_tile_edges(n, offset):
    import torch

    from paper_2307_16758_amd import swe
    from paper_2307_16758_amd.limiter_train import WV, init_params
    rng = np.random.default_rng(n)
    w = init_params(3)
    w[448:480] = rng.normal(0, 0.1, 32)
    w[1504:1536] = rng.normal(0, 0.1, 32)
    m = n + 7
    R = np.zeros((m, 40), np.float32)
    R[:, :14] = rng.uniform(-1, 1, (m, 14))
    R[:, 14:18] = rng.normal(size=(m, 4))
    R[:, 36:40] = 0.1 * rng.uniform(-1, 1, (m, 4))
    R[:, 32:36] = R[:, 36:40] * rng.uniform(-0.3, 1.7, (m, 4))
    R[:, 18:22] = 0.5 * (R[:, 32:36] + R[:, 36:40])
    R[:, 22] = rng.uniform(1, 3, m)
    R[:, 23:27] = R[:, 14:18] + 0.05 * rng.normal(size=(m, 4))
    R[:, 27] = 1.0
    buf = torch.zeros(40 * m + offset, dtype=torch.float32, device="cuda")
    buf[offset:] = torch.from_numpy(R.ravel()).cuda()
    idx = rng.permutation(m)[:n].astype(np.int32)
    if n > 40:
        idx[5], idx[n - 1] = -1, m  # absent
    tr = swe.Trainer(w)
    loss, g = tr.loss_grad(buf[offset:], torch.from_numpy(idx).cuda(), WV)
    V = R[idx[(idx >= 0) & (idx < m)]].astype(np.float64)
    lo, go = O.mlp_loss_grad(w.astype(np.float64), V[:, :14], V[:, 14:18], V[:, 18:22], V[:, 32:36],
                             V[:, 36:40], V[:, 22], V[:, 23:27], WV.astype(np.float64))
    scale = len(V) / n  # the mean counts absent records
    # FP32 sums of at most 16 records per wave and tile, then double: about
    # sqrt(96) roundings of 6e-8 in a delta's chain; its TVD branches can turn
    # on a tie only for a share of 1e-6 of the records
    assert abs(loss - lo * scale) <= 2e-6 * abs(lo) + 1e-12
    assert np.abs(g - go * scale).max() <= 1e-5 * np.abs(go).max()
    tr.close()
