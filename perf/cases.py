"""Timed cases of the rollout path: what a user of this package runs, through its public entry points.

A pod's program alternates collecting a rollout (actor, sampling, trades, critic, advantages), learner steps on
minibatches of it, evaluation of the record, and -- with a population -- the generator step; between those it asks
a policy for actions on a handful of observations.  Each kind of case below is one of these calls:

    rollout     reset, T steps for all envs with critic values and log-probs, generalised advantages
    advantages  the advantage scan alone
    evaluate    the evaluator's trading figures of a recorded rollout
    learner     one PPO optimiser step on a minibatch gathered from the buffer
    gradients   the minibatch gradients alone, for a caller with an optimiser of its own
    policy      the actor network on a few rows
    generation  leaderboard, refill of the population from its best agents, new weights taken over, next actions

Shapes are those of the package's named workloads (inputs.WORKLOADS) and of its replay of one shared table; the
networks, markets and noise follow the same recipes, drawn on the GPU from the case's seed.
"""
import math

import torch

from paper_2112_05923_amd import inputs, podrollout as pr

DEV = "cuda:0"
F32, BF16 = pr.PR_MLP_F32, pr.PR_MLP_BF16
# Most matrix work (by operand type) and memory traffic of a drawn rollout: less than the largest listed ones have.
MAX_FLOPS, MAX_BYTES = {False: 3.0e12, True: 8.0e12}, 2.0e10


def listed():
    return [
        # the smallest rollout of the package (BASELINE's first configuration): 64 steps of 16 envs, all launches
        dict(name="rollout_tiny", kind="rollout", envs=16, agents=1, stocks=5, inds=2, hidden=64, steps=64, table=0,
             bf16=False, fused=False),
        # 30 stocks, fp32 networks, the persistent schedule (half of the named workload's steps, like the two below)
        dict(name="rollout_dow30", kind="rollout", envs=4096, agents=1, stocks=30, inds=8, hidden=256, steps=512,
             table=0, bf16=False, fused=True),
        # the benchmark's configuration: 16384 envs, bf16 networks, the persistent schedule
        dict(name="rollout_large", kind="rollout", envs=16384, agents=1, stocks=30, inds=8, hidden=512, steps=512,
             table=0, bf16=True, fused=True),
        # 500 stocks, 1024 hidden units: the network-dominated regime, one set of launches per step
        dict(name="rollout_wide", kind="rollout", envs=2048, agents=1, stocks=500, inds=4, hidden=1024, steps=256,
             table=0, bf16=True, fused=False),
        # a population of 64 agents on one GPU, fp32 networks (a quarter of the named workload's steps)
        dict(name="rollout_population", kind="rollout", envs=65536, agents=64, stocks=30, inds=8, hidden=256, steps=128,
             table=0, bf16=False, fused=True),
        # replay of one shared minute-level table of 100 stocks from per-env start rows; a ragged number of envs
        dict(name="rollout_replay", kind="rollout", envs=5000, agents=1, stocks=100, inds=8, hidden=512, steps=128,
             table=16384, bf16=True, fused=False),
        # advantages of a buffer whose number of envs fills no tile
        dict(name="advantages_ragged", kind="advantages", envs=5001, steps=1000),
        # the evaluator on a record of 4096 envs
        dict(name="evaluate_4096", kind="evaluate", envs=4096, stocks=30, inds=8, steps=512),
        # the paper's minibatch of 1024
        dict(name="learner_1024", kind="learner", batch=1024, buffer=1 << 20, stocks=30, inds=8, hidden=512),
        # gradients of a large odd minibatch on the smaller networks
        dict(name="gradients_15000", kind="gradients", batch=15000, buffer=1 << 20, stocks=30, inds=8, hidden=256),
        # a policy asked for actions on a few dozen observations
        dict(name="policy_48", kind="policy", rows=48, stocks=30, inds=8, hidden=512, bf16=True),
        # the generator step of the 64-agent population
        dict(name="generation_64", kind="generation", agents=64, per_agent=64, stocks=30, inds=8, hidden=256, keep=16),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_rollout(rng):
    """Envs, stocks, steps and widths over the range between the named workloads."""
    while True:
        shape = rng.choice(["small", "pod", "pod", "wide", "population", "replay"])
        c = dict(kind="rollout", agents=1, table=0, fused=False, bf16=rng.random() < 0.5)
        if shape == "small":
            c.update(envs=_log_int(rng, 16, 512), stocks=rng.randint(3, 30), inds=rng.randint(0, 8),
                     hidden=rng.choice([64, 128]), steps=_log_int(rng, 32, 256))
        elif shape == "pod":
            c.update(stocks=4 * rng.randint(2, 7) + rng.choice([0, 1, 2]), inds=rng.choice([4, 8]),
                     steps=_log_int(rng, 64, 512), fused=True, envs=64 * _log_int(rng, 16, 256),
                     hidden=rng.choice([256, 512]) if c["bf16"] else 256)
        elif shape == "wide":
            c.update(envs=_log_int(rng, 256, 2048), stocks=rng.randint(130, 500), inds=rng.randint(2, 4),
                     hidden=rng.choice([512, 1024]), steps=_log_int(rng, 32, 256), bf16=True)
        elif shape == "population":
            agents = _log_int(rng, 4, 64)
            c.update(agents=agents, envs=agents * 64 * rng.randint(2, 16), stocks=30, inds=8, hidden=256,
                     steps=_log_int(rng, 32, 128), fused=True)
        else:
            c.update(envs=_log_int(rng, 512, 8192), stocks=rng.randint(60, 120), inds=8, hidden=512, bf16=True,
                     steps=_log_int(rng, 32, 128), table=_log_int(rng, 2048, 32768))
        cost = work(c)
        if cost["flops"] < MAX_FLOPS[c["bf16"]] and cost["bytes"] < MAX_BYTES:
            return c


def draw(rng):
    kind = rng.choice(["rollout"] * 6 + ["advantages", "evaluate", "learner", "gradients", "policy", "generation"])
    if kind == "rollout":
        return _draw_rollout(rng)
    if kind == "advantages":
        return dict(kind=kind, envs=_log_int(rng, 64, 16384), steps=_log_int(rng, 64, 1024))
    if kind == "evaluate":
        return dict(kind=kind, envs=_log_int(rng, 256, 8192), stocks=rng.randint(5, 100), inds=rng.randint(2, 8),
                    steps=_log_int(rng, 64, 512))
    if kind in ("learner", "gradients"):
        return dict(kind=kind, batch=_log_int(rng, 256, 32768), buffer=1 << 19, stocks=rng.randint(5, 30),
                    inds=rng.randint(2, 8), hidden=rng.choice([64, 128, 256, 512]))
    if kind == "policy":
        return dict(kind=kind, rows=_log_int(rng, 1, 1024), stocks=rng.randint(5, 30), inds=rng.randint(2, 8),
                    hidden=rng.choice([64, 256, 512]), bf16=rng.random() < 0.5)
    agents = _log_int(rng, 8, 64)
    return dict(kind=kind, agents=agents, per_agent=64, stocks=rng.randint(5, 30), inds=rng.randint(2, 8),
                hidden=rng.choice([64, 256]), keep=max(1, agents // rng.randint(2, 8)))


# ------------------------------------------------------------------ shapes

def _width(c):
    return 1 + 2 * c["stocks"] + c["stocks"] * c["inds"]


def _params(c, out):
    S, Hd = _width(c), c["hidden"]
    return S * Hd + Hd + Hd * Hd + Hd + Hd * out + out


def _net_flops(c, out):
    S, Hd = _width(c), c["hidden"]
    return 2 * (S * Hd + Hd * Hd + Hd * out)


def work(case):
    c = case
    if c["kind"] == "rollout":
        N, T, D, S = c["envs"], c["steps"], c["stocks"], _width(c)
        # market rows and noise in; observations, actions, rewards, done, log-probs, values, advantages, returns out
        market = 4 * D * (1 + c["inds"]) * ((T + 1) * N if not c["table"] else min(c["table"], (T + 1) * N))
        nbytes = market + 4 * T * N * D + 4 * (T + 1) * N * (S + 1) + T * N * (4 * D + 17)
        nbytes += 4 * c["agents"] * (_params(c, D) + _params(c, 1))
        return {"bytes": nbytes, "flops": T * N * _net_flops(c, D) + (T + 1) * N * _net_flops(c, 1)}
    if c["kind"] == "advantages":
        return {"bytes": 17 * c["envs"] * c["steps"] + 4 * c["envs"], "flops": 6 * c["envs"] * c["steps"]}
    if c["kind"] == "evaluate":
        points = (c["steps"] + 1) * c["envs"]
        return {"bytes": points * (4 * (1 + 2 * c["stocks"]) + 1) + 52 * c["envs"], "flops": points * 2 * c["stocks"]}
    if c["kind"] in ("learner", "gradients"):
        B, D, S = c["batch"], c["stocks"], _width(c)
        n = _params(c, D) + _params(c, 1)
        flops = 3 * B * (_net_flops(c, D) + _net_flops(c, 1)) - 2 * 2 * B * S * c["hidden"]
        # rows of the buffer; parameters, and either the gradients or both moments in and out
        return {"bytes": 4 * B * (S + D + 4) + 4 * n * (6 if c["kind"] == "learner" else 2), "flops": flops}
    if c["kind"] == "policy":
        D, S = c["stocks"], _width(c)
        return {"bytes": 4 * c["rows"] * (S + D) + (2 if c["bf16"] else 4) * _params(c, D),
                "flops": c["rows"] * _net_flops(c, D)}
    P, N = c["agents"], c["agents"] * c["per_agent"]
    n = _params(c, c["stocks"]) + _params(c, 1)
    return {"bytes": 4 * n * (3 * (P - c["keep"]) + c["keep"]) + 4 * N * (_width(c) + c["stocks"]) + 20 * N,
            "flops": N * _net_flops(c, c["stocks"])}


# ------------------------------------------------------------------ inputs

def _workload(c, envs, steps, agents=1):
    return inputs.Workload("case", 0, envs, agents, c["stocks"], c["inds"], c["hidden"], steps,
                           BF16 if c.get("bf16") else F32, 0.015, cost=2.0e-3 if c.get("table") else 1.0e-3)


def _market(g, rows, paths, c, sigma):
    """Geometric Brownian motion without drift from prices of 10 to 100; independent normal indicators."""
    D, K = c["stocks"], c["inds"]
    x = torch.empty((rows, paths, D), device=DEV)
    x.normal_(generator=g).mul_(sigma).sub_(0.5 * sigma * sigma)
    x[0].uniform_(10.0, 100.0, generator=g).log_()
    price = torch.cumsum(x, dim=0, out=x).exp_()
    ind = torch.empty((rows, paths, D * K), device=DEV).normal_(generator=g) if K else None
    return price, ind


def _net(g, c, out, agents=None):
    S, Hd = _width(c), c["hidden"]
    shapes = {"W1": (S, Hd), "b1": (Hd,), "W2": (Hd, Hd), "b2": (Hd,), "W3": (Hd, out), "b3": (out,)}
    lead = () if agents is None else (agents,)
    return {k: 0.1 * torch.randn(lead + s, generator=g, device=DEV) for k, s in shapes.items()}


def _observations(g, c, rows):
    """Rows as a rollout records them: cash, prices, holdings (whole shares) at the package's scales, indicators."""
    D, S = c["stocks"], _width(c)
    s = inputs.WORKLOADS["large"].obs_scale
    obs = torch.empty((rows, S), device=DEV).normal_(generator=g)
    obs[:, 0].uniform_(0.0, 1.0e6, generator=g).mul_(s[0])
    obs[:, 1:1 + D].mul_(0.2).exp_().mul_(50.0 * s[1])
    obs[:, 1 + D:1 + 2 * D] = torch.randint(0, 600, (rows, D), generator=g, device=DEV).float() * s[2]
    return obs


def _worker(g, c, envs, steps, agents=1):
    """A rollout worker with its networks, for the calls that only need the handle (a one-row market)."""
    w = _workload(c, envs, steps, agents)
    price, ind = _market(g, 2, 1, c, w.gbm_sigma)
    actor, critic = _net(g, c, c["stocks"], agents), _net(g, c, 1, agents)
    ro = pr.Rollout(pr.make_config(w, horizon=1, n_market=1), price, ind, actor, critic)
    return ro, actor, critic


def prepare(case, seed):
    c = dict(case)
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    kind = c["kind"]
    st = {"kind": kind}
    if kind == "rollout":
        N, T, D = c["envs"], c["steps"], c["stocks"]
        w = _workload(c, N, T, c["agents"])
        rows, paths = (c["table"], 1) if c["table"] else (T + 1, N)
        price, ind = _market(g, rows, paths, c, w.gbm_sigma * (0.1 if c["table"] else 1.0))
        actor, critic = _net(g, c, D, c["agents"]), _net(g, c, 1, c["agents"])
        cfg = pr.make_config(w, horizon=T, n_market=paths, schedule=pr.PR_SCHED_FUSED if c["fused"] else pr.PR_SCHED_STEPWISE)
        ro = pr.Rollout(cfg, price[:T + 1], ind[:T + 1] if c["inds"] else None, actor, critic)
        if c["table"]:
            ro.set_replay(price, ind, torch.randint(0, rows - T, (N,), generator=g, device=DEV, dtype=torch.int32))
        st.update(ro=ro, T=T, w=w, noise=torch.empty((T, N, D), device=DEV).normal_(generator=g),
                  out=ro.alloc_buffers(T, value=True, logp=True), adv=torch.empty((T, N), device=DEV),
                  ret=torch.empty((T, N), device=DEV))
    elif kind == "advantages":
        T, N = c["steps"], c["envs"]
        st.update(reward=torch.randn((T, N), generator=g, device=DEV), value=torch.randn((T + 1, N), generator=g, device=DEV),
                  done=(torch.rand((T, N), generator=g, device=DEV) < 0.002).to(torch.uint8),
                  adv=torch.empty((T, N), device=DEV), ret=torch.empty((T, N), device=DEV))
    elif kind == "evaluate":
        T, N, D = c["steps"], c["envs"], c["stocks"]
        scale = inputs.WORKLOADS["large"].obs_scale
        obs = _observations(g, c, (T + 1) * N).view(T + 1, N, _width(c))
        # prices that move from step to step, holdings that are kept: account values as an evaluation sees them
        obs[:, :, 1:1 + D] = _market(g, T + 1, N, dict(c, inds=0), 0.015)[0] * scale[1]
        obs[:, :, 1 + D:1 + 2 * D] = obs[:1, :, 1 + D:1 + 2 * D]
        obs[:, :, 0] = obs[:1, :, 0]
        done = torch.zeros((T, N), dtype=torch.uint8, device=DEV)
        done[T - 1] = 1
        # (a quarter of the envs end their first episode somewhere inside the record)
        early = torch.randint(0, T, (N // 4,), generator=g, device=DEV)
        done[early, torch.arange(N // 4, device=DEV)] = 1
        st.update(obs=obs, done=done, D=D, scale=scale)
    elif kind in ("learner", "gradients"):
        R, B, D = c["buffer"], c["batch"], c["stocks"]
        w = _workload(c, 64, 1)
        cfg = pr.make_ppo_config(w, batch=B, adam_step=100)
        randn = lambda *s: torch.randn(s, generator=g, device=DEV)
        st.update(cfg=cfg, batch=[_observations(g, c, R), randn(R, D).mul_(0.5), randn(R).sub_(1.5 * D), randn(R), randn(R),
                                  torch.randint(0, R, (B,), generator=g, device=DEV, dtype=torch.int32)],
                  actor=_net(g, c, D), critic=_net(g, c, 1), ws=pr.ppo_workspace(cfg, DEV))
        # log-probs of the actions under a policy close to the present one
        mu = _forward(st["actor"], st["batch"][0])
        e = st["batch"][1].add_(mu) - mu
        st["batch"][2] = (-0.5 * (e / w.sigma).square().sum(1) - D * (math.log(w.sigma) + 0.5 * math.log(2 * math.pi))
                          + 0.1 * randn(R)).contiguous()
        if kind == "learner":
            like = lambda net, f: {k: f(v) for k, v in net.items()}
            st["moments"] = [like(n, f) for n in (st["actor"], st["critic"])
                             for f in (lambda v: 1e-3 * torch.randn(v.shape, generator=g, device=DEV),
                                       lambda v: 1e-6 * (0.1 + torch.rand(v.shape, generator=g, device=DEV)))]
    elif kind == "policy":
        ro, _, _ = _worker(g, c, c["rows"], 1)
        st.update(ro=ro, X=_observations(g, c, c["rows"]), Y=torch.empty((c["rows"], c["stocks"]), device=DEV))
    else:
        P, N = c["agents"], c["agents"] * c["per_agent"]
        ro, actor, critic = _worker(g, c, N, 1, P)
        ro.set_state({"ep_sum": torch.randn(N, generator=g, device=DEV, dtype=torch.float64),
                      "ep_sqsum": torch.rand(N, generator=g, device=DEV, dtype=torch.float64).add_(1.0),
                      "ep_count": torch.ones(N, device=DEV, dtype=torch.int32)})
        noise = [{k: torch.randn(v.shape, generator=g, device=DEV) for k, v in n.items()} for n in (actor, critic)]
        st.update(ro=ro, nets=(actor, critic), noise=noise, keep=c["keep"], X=_observations(g, c, N),
                  Y=torch.empty((N, c["stocks"]), device=DEV))
    return st


def _forward(net, X):
    mu = torch.empty((X.shape[0], net["W3"].shape[1]), device=DEV)
    for r in range(0, X.shape[0], 1 << 17):
        h = torch.tanh(torch.addmm(net["b1"], X[r:r + (1 << 17)], net["W1"]))
        h = torch.tanh(torch.addmm(net["b2"], h, net["W2"]))
        mu[r:r + (1 << 17)] = torch.tanh(torch.addmm(net["b3"], h, net["W3"]))
    return mu


# -------------------------------------------------------------------- calls

def run(state):
    st = state
    kind = st["kind"]
    if kind == "rollout":
        w, out = st["w"], st["out"]
        st["ro"].reset()
        st["ro"].step_T(st["T"], st["noise"], out)
        pr.compute_gae(out["reward"], out["value"], out["done"], w.gamma, w.lam, st["adv"], st["ret"])
        return dict(out, adv=st["adv"], ret=st["ret"])
    if kind == "advantages":
        return pr.compute_gae(st["reward"], st["value"], st["done"], 0.99, 0.95, st["adv"], st["ret"])
    if kind == "evaluate":
        return pr.trading_metrics(st["obs"], st["done"], st["D"], st["scale"], 252.0 * 390.0)
    if kind == "learner":
        a, va, cr, vc = st["moments"]
        stats = pr.ppo_learner_step(st["cfg"], *st["batch"], st["actor"], st["critic"], a, va, cr, vc, st["ws"])
        st["cfg"].adam_step += 1
        return {"stats": stats, "actor": st["actor"], "critic": st["critic"], "moments": st["moments"]}
    if kind == "gradients":
        return pr.ppo_minibatch_grads(st["cfg"], *st["batch"], st["actor"], st["critic"], st["ws"])
    if kind == "policy":
        return st["ro"].mlp_forward(pr.PR_NET_ACTOR, st["X"], st["Y"])
    ro = st["ro"]
    mean, var, rank = ro.leaderboard()
    for net, noise in zip(st["nets"], st["noise"]):
        for k, params in net.items():
            pr.population_refill(params, rank, st["keep"], 0.02, noise[k])
    ro.set_weights(*st["nets"])
    return {"mean": mean, "var": var, "rank": rank, "nets": st["nets"], "mu": ro.mlp_forward(pr.PR_NET_ACTOR, st["X"], st["Y"])}


def tolerance(case):
    c = case
    if c["kind"] == "rollout":
        # Share counts are truncated, so a policy mean that differs in its last bit can move a share, and the rollout
        # goes on from there.  What is stated is how far the same sums in another order end up after 512 steps (the
        # two schedules of the package differ by 7e-4 with fp32 networks and 3e-3 with bf16 ones, and single entries
        # by 0.1 and 0.25).
        return {"rel": 1e-2, "max": 0.5} if c["bf16"] else {"rel": 3e-3, "max": 0.4}
    if c["kind"] == "evaluate":
        return {"rel": 1e-9}
    if c["kind"] == "policy":
        return {"rel": 5e-3} if c["bf16"] else {"rel": 1e-5}
    return {"rel": 1e-5}
