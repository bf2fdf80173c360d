"""Rollouts of bf16 networks over one shared market table (n_market = 1, 33 to 128 stocks, 512 hidden units): the kernels
of pod_table.hip, which form the market part of layer 1 once per table row or once per env and step."""
import numpy as np
import pytest
import torch

import oracle
import parity
from paper_2112_05923_amd import inputs
from paper_2112_05923_amd import podrollout as pr

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (envs, stocks, indicators, table rows, horizon, steps of a call): both sizes of a workgroup (up to 16 envs, up to 32) with
# full and ragged last ones, every instance of the portfolio blocks at its edges (33, 63 | 64, 95 | 96, 127 | 128 stocks) and
# of the output layer (2, 3, 4 feature tiles), rows that end anywhere in a group of four, episodes that end inside a call.
CASES = [
    (200, 100, 8, 90, 40, 90),      # by table row
    (37, 33, 1, 64, 20, 24),
    (37, 63, 3, 2000, 11, 30),      # by env and step
    (4200, 64, 2, 60, 7, 9),        # two rounds' worth of 16: 17 envs a workgroup
    (8192, 95, 1, 50, 5, 6),
    (5000, 96, 3, 300, 9, 10),
    (9001, 127, 1, 40, 4, 5),       # more than 32 for every compute unit
    (300, 128, 2, 80, 30, 33),
    (16, 101, 5, 33, 32, 40),
    (1, 40, 8, 64, 8, 20),
    (1500, 35, 1, 64000, 64, 90),   # a table longer than the rows kept: in pieces of 42 steps
    (200, 33, 1, 9000, 10, 50),     # and than those kept for few steps' envs: in pieces of 40
]


def _setup(N, D, K, rows, H, T):
    w = inputs.WORKLOADS["large"].replace(n_envs=N, n_stocks=D, n_ind=K, steps=T, hidden=512, cost=2.0e-3)
    d = inputs.make_all(w, horizon=min(rows, 500) - 1, n_market=1, steps=T)
    if rows > 500:  # (a price path that long runs into the smallest numbers: the same 500 rows again and again)
        for k in ("price", "ind"):
            d[k] = np.ascontiguousarray(np.resize(d[k], (rows,) + d[k].shape[1:]))
    rng = np.random.default_rng(N + D)
    start = rng.integers(0, rows - H, N).astype(np.int32)
    start[0], start[N - 1] = 0, rows - 1 - H
    dev = lambda net: {k: torch.from_numpy(v).to(DEV) for k, v in net.items()}
    price, ind = torch.from_numpy(d["price"]).to(DEV), torch.from_numpy(d["ind"]).to(DEV)
    cfg = pr.make_config(w, horizon=H, n_market=1, schedule=pr.PR_SCHED_STEPWISE)
    ro = pr.Rollout(cfg, price[:H + 1], ind[:H + 1], dev(d["actor"]), dev(d["critic"]))
    ro.set_replay(price, ind, torch.from_numpy(start).to(DEV))
    return w, d, start, ro, torch.from_numpy(d["noise"]).to(DEV)


@pytest.mark.parametrize("N,D,K,rows,H,T", CASES)
def test_rollout_over_a_shared_table(N, D, K, rows, H, T):
    """Environment stage of sampled envs bit for bit on the recorded means, networks within the stated tolerance on sampled
    rows, and the same bits when the rollout is cut into calls (whose market sums are formed by env and step)."""
    w, d, start, ro, noise = _setup(N, D, K, rows, H, T)
    out = ro.alloc_buffers(T, value=True, logp=True, mu=True, shares=True)
    ro.step_T(T, noise, out)
    end = ro.get_state()
    S = w.state_dim
    rec = {k: parity.to_np(v) for k, v in out.items()}
    pick = np.unique(np.concatenate([np.arange(min(N, 40)), np.arange(max(0, N - 40), N), np.arange(0, N, max(1, N // 50))]))
    sub = {k: np.ascontiguousarray(v[:, pick]) for k, v in rec.items()}
    ocfg = oracle.cfg_from_workload(w.replace(n_envs=len(pick)), horizon=H)
    ost = oracle.State(ocfg, len(pick), start=start[pick])
    chk, ost = parity.check_env_record(w.replace(n_envs=len(pick)), ocfg, sub, d["price"], d["ind"],
                                       np.ascontiguousarray(d["noise"][:, pick]), sub["mu"], state0=ost)
    assert np.array_equal(parity.to_np(end["cursor"])[pick], ost.tau) and np.array_equal(parity.to_np(end["cash"])[pick], ost.cash)
    assert np.array_equal(parity.to_np(end["holdings"])[pick], ost.h)
    ts = sorted({0, min(H, T) - 1, min(H, T - 1), T - 1})
    few = pick[:: max(1, len(pick) // 24)]
    parity.check_networks(w, d["actor"], d["critic"], rec["obs"][ts][:, few].reshape(-1, S), rec["mu"][ts][:, few].reshape(-1, D),
                          rec["value"][ts][:, few].reshape(-1))
    # every value against the critic asked about the recorded observations
    again = ro.mlp_forward(pr.PR_NET_CRITIC, out["obs"].view(-1, S))
    parity.check_two_tier("value", parity.to_np(out["value"]).reshape(1, -1), parity.to_np(again).reshape(1, -1), True)
    ro.reset()
    cut = ro.alloc_buffers(T, value=False, logp=True, mu=True, shares=True)
    t = 0
    for n in [1, 2, T - 3 - T // 3, T // 3]:
        part = {k: v[t:t + n + (k == "obs")] for k, v in cut.items()}
        ro.step_T(n, noise[t:t + n].contiguous(), part)
        t += n
    assert t == T
    for k, v in cut.items():
        assert torch.equal(v, out[k]), k
    for k, v in ro.get_state().items():
        assert torch.equal(v, end[k]), k


# Calls of one step, whose market sums are formed by smaller workgroups on up to 512 rows, give the bits of longer ones: full and ragged
# ones of 32 rows, the last row count, and inputs that end in each of the four places a chunk of them is requested in.
@pytest.mark.parametrize("N,D,K,T", [(32, 47, 5, 24), (33, 33, 3, 24), (512, 34, 6, 9), (513, 64, 8, 9), (480, 90, 8, 9)])
def test_market_sums_of_few_rows(N, D, K, T):
    test_rollout_over_a_shared_table(N, D, K, 700, 9, T)  # (700 rows for the whole of it)


# Values of calls with few rows, on either side of the lines at which the head over table sums takes over from the kernels for any
# network: 4096 rows over a short table (N (T + 1) = 4096, 4097), 8192 over a longer one, 1024 rows of more than 640 inputs (there
# also over tables longer than the rows).
@pytest.mark.parametrize("N,D,K,rows,T", [(40, 40, 2, 33, 1), (2048, 50, 3, 33, 1), (241, 33, 1, 33, 16), (4096, 40, 2, 260, 1),
                                          (2731, 61, 2, 260, 2), (512, 128, 4, 40, 1), (205, 100, 8, 40, 4),
                                          (513, 128, 4, 3000, 1), (600, 128, 3, 8192, 1), (600, 80, 6, 601, 1)])
def test_values_of_few_rows_over_a_shared_table(N, D, K, rows, T):
    w, d, start, ro, noise = _setup(N, D, K, rows, 20, T)
    out = ro.alloc_buffers(T, value=True, logp=False, mu=True)
    ro.step_T(T, noise, out)
    few = np.unique(np.concatenate([np.arange(min(N, 20)), np.arange(N - 20, N)]))
    obs, mu, value = (parity.to_np(out[k]) for k in ("obs", "mu", "value"))
    parity.check_networks(w, d["actor"], d["critic"], obs[:T][:, few].reshape(-1, w.state_dim), mu[:, few].reshape(-1, D),
                          value[:T][:, few].reshape(-1))
    again = parity.to_np(ro.mlp_forward(pr.PR_NET_CRITIC, out["obs"].view(-1, w.state_dim)))
    parity.check_two_tier("value", value.reshape(1, -1), again.reshape(1, -1), True)
