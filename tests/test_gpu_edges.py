"""Kernel variants chosen by size, at the sizes where a tile, a chunk or a segment ends: against the CPU checker."""
import numpy as np
import pytest
import torch

import oracle
import parity
from paper_2112_05923_amd import inputs, podrollout as pr

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _t(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


# 16-, 32- and 64-env tiles of the advantage scan, one segment of each and one step more, rows that are whole lines
# and rows that are not
@pytest.mark.parametrize("T,N", [(1024, 17), (1025, 40), (512, 4097), (513, 5001), (256, 8193), (257, 8224), (300, 8200)])
def test_gae_tiles(T, N):
    rng = np.random.default_rng(T + N)
    r, v = rng.standard_normal((T, N)).astype(np.float32), rng.standard_normal((T + 1, N)).astype(np.float32)
    done = (rng.random((T, N)) < 0.01).astype(np.uint8)
    adv, ret = pr.compute_gae(_t(r), _t(v), _t(done), 0.99, 0.95)
    torch.cuda.synchronize()
    parity.check_gae(r, v, done, 0.99, 0.95, parity.to_np(adv), parity.to_np(ret))


# envs per workgroup 4 / 8 / 16 / 64 of the evaluator, runs of 15 and 31 stocks, chunks of one point, empty chunks
@pytest.mark.parametrize("T,N,D", [(3, 5, 4), (130, 70, 15), (600, 37, 16), (511, 9, 31), (520, 4100, 3), (127, 33, 32),
                                   (200, 8195, 2), (40, 32770, 1)])
def test_trading_metrics_tiles(T, N, D):
    rng = np.random.default_rng(T * 7 + N)
    w = inputs.WORKLOADS["large"].replace(n_envs=N, n_stocks=D, n_ind=0, steps=T)
    S = w.state_dim
    obs = np.empty((T + 1, N, S), np.float32)
    obs[..., 0] = rng.uniform(1e5, 1e6, (T + 1, N)) * w.obs_scale[0]
    obs[..., 1:1 + D] = np.exp(rng.normal(4.0, 0.3, (T + 1, N, D))) * w.obs_scale[1]
    obs[..., 1 + D:] = rng.integers(0, 300, (T + 1, N, D)) * w.obs_scale[2]
    done = (rng.random((T, N)) < 1.5 / T).astype(np.uint8)
    done[:, 0] = 0
    got, length = pr.trading_metrics(_t(obs), _t(done), D, w.obs_scale, 252.0, 0.01)
    torch.cuda.synchronize()
    got, length = parity.to_np(got), parity.to_np(length)
    for n in np.unique(np.concatenate([[0, 1, N - 1], rng.integers(0, N, 40)])):
        L = int(np.argmax(done[:, n])) if done[:, n].any() else T
        assert length[n] == L
        o = obs[:L + 1, n].astype(np.float64)
        V = o[:, 0] / w.obs_scale[0] + ((o[:, 1:1 + D] / w.obs_scale[1]) * (o[:, 1 + D:1 + 2 * D] / w.obs_scale[2])).sum(1)
        if L == 0:
            assert not got[:, n].any()
            continue
        r = V[1:] / V[:-1] - 1.0
        sd = r.std(ddof=1) if L > 1 else 0.0
        mdd = (1.0 - V / np.maximum.accumulate(V)).max()
        ann = (V[-1] / V[0]) ** (252.0 / L) - 1.0
        want = [(V[-1] - V[0]) / V[0], ann, np.sqrt(252.0) * sd, mdd,
                np.sqrt(252.0) * (r.mean() - 0.01 / 252.0) / sd if sd > 0 else 0.0, ann / mdd if mdd > 0 else 0.0]
        np.testing.assert_allclose(got[:, n], want, rtol=1e-8, atol=1e-11)
