"""fp32 networks whose inputs and weights are of very different sizes, up to the scales of observations that are accepted: as close to
64 bits as fp32 sums are."""
import numpy as np
import pytest
import torch

import parity
from paper_2112_05923_amd import inputs, podrollout as pr

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _observations_and_actor(case, N, D, K, T=2):
    """Market, observation scales and the first layer's sizes of a case.  `plain`: the package's recipe.  `unscaled`: observations at scale
    1 (cash of 1e6 next to indicators of 1).  `balanced`: the same, and weights in inverse proportion to the size of their
    column, as training leaves them, so that every column matters alike.  `one price`: the package's scales with weights in that
    proportion, one price of 600000 and indicators near 0.01; `one price, unscaled`: at scale 1 next to indicators near 0.001.  `faint units`: the package's scales, first hidden layers of 1e-8 and
    weights behind them that make up for it."""
    w = inputs.WORKLOADS["dow30"].replace(n_envs=N, n_agents=1, n_stocks=D, n_ind=K, steps=T)
    if case in ("unscaled", "balanced", "one price, unscaled"):
        w = w.replace(obs_scale=(1.0, 1.0, 1.0, 1.0))
    d = inputs.make_all(w, horizon=T, steps=T)
    if case.startswith("one price"):
        d["price"][..., 0] = np.float32(600000.0)
        d["ind"] *= np.float32(0.001 if case.endswith("unscaled") else 0.01)
    s = w.obs_scale
    size = np.concatenate([[1e6 * s[0]], d["price"].mean((0, 1)) * s[1], np.full(D, 300.0 * s[2]), d["ind"].std((0, 1)) * s[3]]).astype(np.float32)
    if case in ("balanced", "one price", "one price, unscaled"):
        for net in ("actor", "critic"):
            d[net]["W1"] = d[net]["W1"] / size[None, :, None]
    if case == "faint units":
        for net in ("actor", "critic"):
            for k, f in (("W1", 1e-8), ("b1", 1e-8), ("W2", 1e8)):
                d[net][k] = d[net][k] * np.float32(f)
    return w, d, size


def _network64(X, net, out_tanh):
    n = {k: v[0].astype(np.float64) for k, v in net.items()}
    y = np.tanh(np.tanh(X.astype(np.float64) @ n["W1"] + n["b1"]) @ n["W2"] + n["b2"]) @ n["W3"] + n["b3"]
    return np.tanh(y) if out_tanh else y


def _network32(X, net, out_tanh):
    """The same with every sum formed in fp32, one input after the other."""
    def layer(x, W, b):
        acc = np.repeat(b[None], len(x), 0)
        for k in range(x.shape[1]):
            acc += x[:, k:k + 1] * W[k][None]
        return acc
    n = {k: v[0] for k, v in net.items()}
    y = layer(np.tanh(layer(np.tanh(layer(X, n["W1"], n["b1"])), n["W2"], n["b2"])), n["W3"], n["b3"])
    return np.tanh(y) if out_tanh else y


def _check(case, X, got, net, out_tanh):
    """The stated tolerance of fp32 networks (parity.TOL_NORM_F32 of the largest entry).  Unscaled, where layer 1 adds numbers of 1e5 to
    numbers of 1 and a unit that ends up near zero has the rounding of the former: twice the error of fp32 sums over the same rows."""
    want = _network64(X, net, out_tanh)
    err = np.abs(got.astype(np.float64) - want)
    if case == "unscaled":
        ref = np.abs(_network32(X, net, out_tanh) - want)
        assert err.max() <= 2.0 * ref.max() and np.linalg.norm(err) <= 2.0 * np.linalg.norm(ref), (err.max(), ref.max())
    else:
        assert err.max() <= parity.TOL_NORM_F32 * np.abs(want).max(), err.max() / np.abs(want).max()


CASES = ["plain", "unscaled", "balanced", "one price", "one price, unscaled", "faint units"]


# means of the persistent rollout: 16 and 32 envs a workgroup, blocks of market columns that are full and not
@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("N,D,K", [(1024, 30, 8), (4160, 30, 8), (1024, 12, 4), (4160, 5, 4)])
def test_rollout_of_observations_of_all_scales(case, N, D, K):
    w, d, _ = _observations_and_actor(case, N, D, K)
    dev = lambda m: {k: _t(v) for k, v in m.items()}
    ro = pr.Rollout(pr.make_config(w, horizon=2, schedule=pr.PR_SCHED_FUSED), _t(d["price"]), _t(d["ind"]), dev(d["actor"]), dev(d["critic"]))
    out = ro.alloc_buffers(2, value=False, logp=False, mu=True, shares=False)
    ro.step_T(2, _t(d["noise"]), out)
    torch.cuda.synchronize()
    _check(case, parity.to_np(out["obs"])[:2].reshape(2 * N, -1), parity.to_np(out["mu"]).reshape(2 * N, D), d["actor"], True)
