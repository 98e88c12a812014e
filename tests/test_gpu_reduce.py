"""The launches around a step's forwards: tile sums by one wave where a slot has
fewer, as many and more tiles than lanes, the coefficients from the loss sums'
own launch (one chunk) against the two launches (one direction at a time), and
the one-block check of the rates of more experts than it has threads."""
import numpy as np
import pytest

from gpu_common import assert_losses_close, require_gpu
from paper_2609_37899_amd import soma, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T", [(1, 2), (63, 65), (64, 66), (65, 80)])   # 1, 63, 65 and 81 tiles of 64 rows
def test_one_launch_is_the_two_launches(oracle_mod, B, T):
    torch = require_gpu()
    N, P = 2, 3
    theta = synth.init_theta(N, 1, 16, 16, init_seed=3, distinct=True)
    data = synth.expert_batches([20 + e for e in range(N)], B, T)
    seeds = synth.expert_seeds(N)
    outs = []
    for pc in (0, 1):
        ctx = soma.Context(soma.Shape(N, 1, 16, 16, B, T, P, 0, pc))
        th = torch.from_numpy(theta.copy()).cuda()
        losses = torch.zeros((N, P, 2), dtype=torch.float32, device="cuda")
        coef = torch.zeros((N, P), dtype=torch.float32, device="cuda")
        print(f"B={B} T={T} directions per pass {pc}", flush=True)
        ctx.spsa_step(th, soma.seeds_tensor(seeds), 1, 1e-3, 1e-3, torch.from_numpy(data).cuda(), losses)
        ctx.coefficients(coef)
        torch.cuda.synchronize()
        outs.append([x.cpu().numpy() for x in (th, losses, coef)])
        ctx.close()
    for a, b in zip(*outs):
        assert np.array_equal(a, b)
    cfg = oracle_mod.make_cfg(N, 1, 16, 16, B, T, P)
    assert_losses_close(outs[0][1], oracle_mod.spsa_step(cfg, theta, seeds, 1, 1e-3, 1e-3, data)["losses"])


@pytest.mark.parametrize("N,bad", [(256, None), (257, None), (257, 256), (300, 299), (300, 0)])
def test_rates_of_more_experts_than_threads(N, bad):
    torch = require_gpu()
    B, T, P = 1, 3, 1
    theta = synth.init_theta(N, 1, 16, 16, init_seed=3, distinct=True)
    data = torch.from_numpy(synth.expert_batches([20 + e for e in range(N)], B, T)).cuda()
    seeds = soma.seeds_tensor(synth.expert_seeds(N))
    eps = np.full(N, 1e-3, np.float32)
    if bad is not None:
        eps[bad] = np.inf
    outs = []
    for sched in (True, False):
        ctx = soma.Context(soma.Shape(N, 1, 16, 16, B, T, P))
        th = torch.from_numpy(theta.copy()).cuda()
        m, v = torch.zeros_like(th), torch.zeros_like(th)
        losses = torch.zeros((N, P, 2), dtype=torch.float32, device="cuda")
        print(f"N={N} bad={bad} schedule={sched}", flush=True)
        if sched:
            a = np.zeros((N, 4), np.int32)
            f = a.view(np.float32)
            f[:, 0], f[:, 1], f[:, 2] = 1e-3, eps, np.inf
            entries = torch.from_numpy(a).cuda()
            ctx.spsa_step_adam_sched(th, m, v, 1, soma.Adam(), seeds, 0, entries, data, losses)
        else:
            ctx.spsa_step_adam(th, m, v, 1, soma.Adam(), seeds, 0, 1e-3, 1e-3, data, losses)
        torch.cuda.synchronize()
        outs.append([x.cpu().numpy() for x in (th, losses)])
        ctx.close()
    if bad is None:
        assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])
    else:
        assert np.isnan(outs[0][1]).all() and np.array_equal(outs[0][0], theta)
        assert np.isfinite(outs[1][1]).all()       # a scalar step after it, in a context of its own
