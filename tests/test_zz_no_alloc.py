"""The entry point for callers that cannot allocate (scratch in a fixed device array inside the library) against
the workspace-taking entry point it is a variant of: same kernels, so the results must agree bit for bit."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2112_05923_amd import inputs, podrollout as pr

DEV = "cuda:0"


def _case(w, B, R, seed):
    rng = np.random.default_rng(seed)
    S, D = w.state_dim, w.n_stocks
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to(DEV)
    nets = {k: {kk: t(vv[0]) for kk, vv in inputs.make_weights(w, critic=(k == "critic")).items()}
            for k in ("actor", "critic")}
    obs = rng.standard_normal((R, S)).astype(np.float32)
    obs[:, 0] *= 0.5
    act = rng.uniform(-1.5, 1.5, (R, D)).astype(np.float32)
    logp_old = rng.normal(-30.0, 3.0, R).astype(np.float32)
    adv = rng.standard_normal(R).astype(np.float32)
    ret = rng.standard_normal(R).astype(np.float32)
    rows = torch.from_numpy(rng.permutation(R)[:B].astype(np.int32)).to(DEV)
    return nets, (t(obs), t(act), t(logp_old), t(adv), t(ret), rows)


def _empty_grads(cfg, fill):
    mk = lambda shapes: {k: torch.full(v, fill, dtype=torch.float32, device=DEV) for k, v in shapes.items()}
    return mk(pr._net_shapes(cfg, cfg.n_stocks)), mk(pr._net_shapes(cfg, 1))


@pytest.mark.gpu
def test_noalloc_minibatch_grads_equal_the_workspace_entry_point_on_two_calls_in_a_row():
    # the paper's minibatch on the headline network shape first, a smaller batch on a smaller network second:
    # the second call finds the first call's contents in the shared scratch
    for name, B, R in (("large", 1024, 1300), ("dow30", 96, 200)):
        w = inputs.WORKLOADS[name]
        cfg = pr.make_ppo_config(w, batch=B)
        nets, batch = _case(w, B, R, seed=B)
        want_a, want_c, want_stats = pr.ppo_minibatch_grads(cfg, *batch, nets["actor"], nets["critic"])
        ga, gc = _empty_grads(cfg, float("nan"))
        stats = torch.full((4,), float("nan"), device=DEV)
        pr.ppo_minibatch_grads_noalloc(cfg, *batch, nets["actor"], nets["critic"], ga, gc, stats)
        torch.cuda.synchronize()
        for k in pr.NET_KEYS:
            assert torch.equal(ga[k], want_a[k]), (name, "actor", k)
            assert torch.equal(gc[k], want_c[k]), (name, "critic", k)
        assert torch.equal(stats, want_stats), name
        assert bool(torch.isfinite(ga["W1"]).all()) and float(ga["W2"].abs().max()) > 0.0


@pytest.mark.gpu
def test_noalloc_refuses_shapes_beyond_its_scratch_and_bad_arguments():
    w = inputs.WORKLOADS["large"]
    cfg = pr.make_ppo_config(w, batch=4096)          # 4x the scratch of the 1024-row minibatch
    n = C.c_size_t(0)
    assert pr.lib().ppo_workspace_bytes(C.byref(cfg), C.byref(n)) == pr.PR_OK and n.value > pr.PR_STATIC_SCRATCH_BYTES
    nets, batch = _case(w, 4096, 4096, seed=1)
    ga, gc = _empty_grads(cfg, 7.0)
    stats = torch.zeros(4, device=DEV)
    with pytest.raises(pr.PodError) as e:
        pr.ppo_minibatch_grads_noalloc(cfg, *batch, nets["actor"], nets["critic"], ga, gc, stats)
    assert e.value.code == pr.PR_ETOOBIG and "scratch" in str(e.value)
    torch.cuda.synchronize()
    assert float(ga["W1"].min()) == 7.0 and float(ga["W1"].max()) == 7.0       # nothing was enqueued
    assert pr.lib().ppo_minibatch_grads_noalloc(None, C.byref(cfg), *([None] * 6), *([None] * 4), None) == pr.PR_EINVAL


# refused before any device work, so no device is needed: shapes just past the stated count of the scratch
@pytest.mark.parametrize("B,D,K,Hd", [(1, 1, 0, 1024), (1500, 1, 0, 512), (2000, 5, 0, 512), (1300, 30, 8, 512), (4096, 30, 8, 256)])
def test_noalloc_serves_no_shape_beyond_its_stated_scratch(B, D, K, Hd):
    S = 1 + 2 * D + D * K
    up = lambda floats: (4 * floats + 255) // 256 * 256
    count = up(B * (S + 3 & ~3)) + 6 * up(B * Hd) + 2 * up(B * D) + 2 * up(B) + up((B + 7) // 8 * 4) + up(8 * Hd * Hd)
    assert count > pr.PR_STATIC_SCRATCH_BYTES
    w = inputs.WORKLOADS["large"].replace(n_stocks=D, n_ind=K, hidden=Hd)
    cfg = pr.make_ppo_config(w, batch=B)
    p = pr.PrNetParams(*([256] * 6))
    rc = pr.lib().ppo_minibatch_grads_noalloc(None, C.byref(cfg), *([256] * 6), *([C.byref(p)] * 4), None)
    assert rc == pr.PR_ETOOBIG


# batches the stated scratch covers only with fewer k splits, with rows close together, or with one network after the other:
# the call with a workspace gives the same bits; the optimiser step, which keeps to no such limit, the same to rounding
@pytest.mark.gpu
@pytest.mark.parametrize("B,D,K,Hd", [(2400, 30, 8, 256), (2800, 30, 8, 256), (3100, 15, 8, 256), (4400, 30, 8, 128), (10500, 15, 8, 64)])
def test_noalloc_near_the_end_of_its_scratch(B, D, K, Hd):
    w = inputs.WORKLOADS["dow30"].replace(n_stocks=D, n_ind=K, hidden=Hd)
    cfg = pr.make_ppo_config(w, batch=B, adam_step=3)
    nets, batch = _case(w, B, B + 50, seed=B)
    want_a, want_c, want_stats = pr.ppo_minibatch_grads(cfg, *batch, nets["actor"], nets["critic"])
    ga, gc = _empty_grads(cfg, float("nan"))
    stats = torch.full((4,), float("nan"), device=DEV)
    pr.ppo_minibatch_grads_noalloc(cfg, *batch, nets["actor"], nets["critic"], ga, gc, stats)
    zeros = lambda net: {k: torch.zeros_like(v) for k, v in net.items()}
    like = lambda net: {k: v.clone() for k, v in net.items()}
    a, c, m = like(nets["actor"]), like(nets["critic"]), [zeros(nets[n]) for n in ("actor", "actor", "critic", "critic")]
    pr.ppo_learner_step(cfg, *batch, a, c, *m, pr.ppo_workspace(cfg, DEV))
    torch.cuda.synchronize()
    assert torch.equal(stats, want_stats)
    for got, want, m1 in ((ga, want_a, m[0]), (gc, want_c, m[2])):
        for k in pr.NET_KEYS:
            assert torch.equal(got[k], want[k]), k
            # the first moment after one step is (1 - beta1) times the gradient
            g = m1[k].double() / (1.0 - cfg.beta1)
            assert float((g - want[k]).norm()) <= 1e-5 * float(want[k].double().norm()), k


# no shape beyond that scratch is held to it: two networks' activations side by side
@pytest.mark.parametrize("B,D,K,Hd", [(1540, 30, 8, 512), (2000, 30, 8, 512), (4000, 30, 8, 256), (7800, 30, 8, 128), (15000, 30, 8, 64)])
def test_workspace_of_larger_batches_holds_both_networks(B, D, K, Hd):
    n, last = C.c_size_t(0), 0
    for b in (B - 64, B, B + 64):
        cfg = pr.make_ppo_config(inputs.WORKLOADS["large"].replace(n_stocks=D, n_ind=K, hidden=Hd), batch=b)
        assert pr.lib().ppo_workspace_bytes(C.byref(cfg), C.byref(n)) == pr.PR_OK
        assert n.value >= max(last, 8 * 4 * b * Hd)
        last = n.value
