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


# Inputs and weights far from one size: rows whose first 32 inputs are zero, a thousandth, a millionth or a multiple of those behind
# them, rows of tiny and of huge numbers, features whose weights are 1e15 apart, one without weights, large biases; one k-block,
# an odd and an even number of them, rows of a last tile that is not full.
# A number's three bf16 parts add up to it, so what is left is the rounding of fp32 sums, sqrt(S) 2^-24 of a row's own sum of
# |w x|: three layers of it and the output's sum over 256 terms leave less than 4e-6 of the values' size.  (Sums of size 1e4 would be
# rounded to 1e4 x 2^-24 = 6e-4, which shows in a unit near zero; of size 1e9 none of 256 units x 170 rows is near zero.)
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


# Persistent rollouts of envs whose indicators are 1e12, 1e6 and 1e3 times smaller than prices, as large, 1e9 times larger, or all
# zero; both sizes of a workgroup, blocks of market columns that are full and not.  Bounds as above.
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
    numbers of 1 and a unit that ends up near zero has the rounding of the former: twice the largest error of fp32 sums over the same rows
    (an accumulator that drops bits instead of rounding is off by up to twice as much at a time).  The stated tolerance is one of
    largest errors too; in the 2-norm the few inputs of 3 stocks, whose dropped bits do not even out, are at 2.3 times fp32's."""
    want = _network64(X, net, out_tanh)
    err = np.abs(got.astype(np.float64) - want)
    if case == "unscaled":
        ref = np.abs(_network32(X, net, out_tanh) - want)
        assert err.max() <= 2.0 * ref.max(), (err.max(), ref.max())
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


# the critic asked about few rows and about many
@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("rows,D,K", [(48, 30, 8), (9000, 30, 8), (16384 + 77, 30, 8), (16384 + 77, 12, 4), (16384 + 77, 3, 1)])
def test_value_head_of_observations_of_all_scales(case, rows, D, K):
    w, d, size = _observations_and_actor(case, 64, D, K)
    rng = np.random.default_rng(D + rows)
    X = rng.standard_normal((rows, w.state_dim)).astype(np.float32) * size
    X[:, 0] = rng.uniform(0.0, 1.0, rows) * size[0]
    X[:, 1:1 + D] = np.exp(0.2 * rng.standard_normal((rows, D))) * size[1:1 + D]
    dev = lambda m: {k: _t(v) for k, v in m.items()}
    ro = pr.Rollout(pr.make_config(w, horizon=2, schedule=pr.PR_SCHED_STEPWISE), _t(d["price"]), _t(d["ind"]), dev(d["actor"]), dev(d["critic"]))
    _check(case, X, parity.to_np(ro.mlp_forward(pr.PR_NET_CRITIC, _t(X))), d["critic"], False)


# An infinite weight behind inputs far below the largest of their row, or zero: the unit saturates, or is NaN, as with fp32 sums
@pytest.mark.parametrize("rows", [48, 9000, 16384 + 77])
def test_infinite_weights_of_small_inputs(rows):
    w = inputs.WORKLOADS["dow30"].replace(n_envs=64, n_agents=1, steps=2)
    d = inputs.make_all(w, horizon=2, n_market=1, steps=2)
    X = np.random.default_rng(rows).standard_normal((rows, w.state_dim)).astype(np.float32)
    X[:, 0] *= np.float32(1e3)
    X[::2, 5] = np.float32(1e-12)
    X[1::4, 5] = np.float32(-3e-20)
    X[7::8, 5] = 0.0
    critic = {k: v.copy() for k, v in d["critic"].items()}
    critic["W1"][0, 5, 9], critic["W1"][0, 5, 200] = np.inf, -np.inf
    dev = lambda m: {k: _t(v) for k, v in m.items()}
    ro = pr.Rollout(pr.make_config(w, horizon=2, n_market=1), _t(d["price"]), _t(d["ind"]), dev(d["actor"]), dev(critic))
    got = parity.to_np(ro.mlp_forward(pr.PR_NET_CRITIC, _t(X)))
    with np.errstate(invalid="ignore"):
        want = _network64(X, critic, False)
    assert np.isnan(want[7::8]).all() and np.isnan(want).sum() == len(want[7::8]) and np.array_equal(np.isnan(got), np.isnan(want))
    assert np.nanmax(np.abs(got - want)) <= 2e-5 * np.nanmax(np.abs(want))
