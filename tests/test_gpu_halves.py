"""fp32 networks whose products are formed of two fp16 numbers per operand (the value head over many rows)."""
import numpy as np
import pytest
import torch

import parity
from paper_2112_05923_amd import inputs, podrollout as pr

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


# Inputs and weights far from one size: rows whose first 32 inputs (which their scale is taken from) are zero, a thousandth,
# a millionth or a multiple of those behind them, rows of tiny and of huge numbers, features whose weights are 1e15 apart, one
# without weights, large biases; one k-block, an odd and an even number of them, rows of a last tile that is not full.
# What the fp16 parts lose of an input is 2^-29 of the largest one its scale was taken from, which may be 2^-11 of the row's
# largest: against the row's own sum of |w x| that stays below the rounding of fp32 sums over the row, sqrt(S) 2^-24; three
# layers of them and the output's sum over 256 terms leave less than 4e-6 of the values' size.  (Sums of size 1e4 would be rounded
# to 1e4 x 2^-24 = 6e-4, which shows in a unit near zero; of size 1e9 none of 256 units x 170 rows is near zero.)
@pytest.mark.parametrize("D,K", [(3, 1), (12, 4), (30, 8), (31, 8)])
def test_value_head_of_numbers_of_all_sizes(D, K):
    w = inputs.WORKLOADS["dow30"].replace(n_envs=64, n_agents=1, n_stocks=D, n_ind=K, steps=2)
    d = inputs.make_all(w, horizon=2, n_market=1, steps=2)
    S, rng, rows = w.state_dim, np.random.default_rng(D), 16384 + 77
    X = rng.standard_normal((rows, S)).astype(np.float32)
    for first, sizes in ((1, (0.0, 1.0)), (2, (1e-3, 1.0)), (3, (1e-6, 1.0)), (5, (2e-4, 1.0)), (6, (1.0, 1e-4)), (7, (1e-20, 1e-20)), (8, (1e-30, 1e-24)),
                         (9, (1e9, 1e13)), (11, (0.0, 0.0))):
        X[first::97, :32] *= np.float32(sizes[0])
        X[first::97, 32:] *= np.float32(sizes[1])
    critic = {k: v.copy() for k, v in d["critic"].items()}
    critic["W1"][0][:, 1::9] *= np.float32(1e-15)
    critic["W1"][0][:, 2] = 0.0
    critic["W2"][0][:, 3::7] *= np.float32(1e-9)
    critic["b1"][0][::5] *= np.float32(20.0)
    dev = lambda m: {k: _t(v) for k, v in m.items()}
    ro = pr.Rollout(pr.make_config(w, horizon=2, n_market=1, schedule=pr.PR_SCHED_STEPWISE), _t(d["price"]), _t(d["ind"]), dev(d["actor"]), dev(critic))
    y = parity.to_np(ro.mlp_forward(pr.PR_NET_CRITIC, _t(X)))[:, 0].astype(np.float64)
    n = {k: v[0].astype(np.float64) for k, v in critic.items()}
    want = (np.tanh(np.tanh(X.astype(np.float64) @ n["W1"] + n["b1"]) @ n["W2"] + n["b2"]) @ n["W3"] + n["b3"])[:, 0]
    err = np.abs(y - want) / np.sqrt(np.mean(want * want))
    for first in range(12):
        assert err[first::97].max() <= 4e-6, (first, err[first::97].max())


# The persistent rollout forms the market part of layer 1 over a scale of the row's own: envs whose indicators are 1e12, 1e6 and
# 1e3 times smaller than prices, as large, 1e9 times larger, or all zero; both sizes of a workgroup, blocks of market columns
# that are full and not, one and two blocks of portfolio columns.  Bounds as above: what the scale loses is 2^-39 of the row's
# largest number.
@pytest.mark.parametrize("N,D,K", [(64, 30, 8), (4128, 30, 8), (96, 12, 4), (32, 32, 7), (4160, 32, 7), (32, 1, 4)])
def test_rollout_of_markets_of_all_sizes(N, D, K):
    w = inputs.WORKLOADS["dow30"].replace(n_envs=N, n_agents=1, n_stocks=D, n_ind=K, steps=2)
    d = inputs.make_all(w, horizon=2, steps=2)
    sizes = np.array([1e-12, 1e-6, 1e-3, 1.0, 1e9, 0.0], np.float32)
    d["ind"] = d["ind"] * sizes[np.arange(N) % 6][None, :, None]
    dev = lambda m: {k: _t(v) for k, v in m.items()}
    ro = pr.Rollout(pr.make_config(w, horizon=2, schedule=pr.PR_SCHED_FUSED), _t(d["price"]), _t(d["ind"]), dev(d["actor"]), dev(d["critic"]))
    out = ro.alloc_buffers(2, value=False, logp=False, mu=True, shares=False)
    ro.step_T(2, _t(d["noise"]), out)
    torch.cuda.synchronize()
    X, mu = parity.to_np(out["obs"])[:2].reshape(2 * N, -1).astype(np.float64), parity.to_np(out["mu"]).reshape(2 * N, D)
    n = {k: v[0].astype(np.float64) for k, v in d["actor"].items()}
    want = np.tanh(np.tanh(np.tanh(X @ n["W1"] + n["b1"]) @ n["W2"] + n["b2"]) @ n["W3"] + n["b3"])
    assert np.abs(mu - want).max() / np.sqrt(np.mean(want * want)) <= 4e-6
