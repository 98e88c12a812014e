"""The one-launch recurrence of widths that are odd multiples of 16 (up to 144)
against the launch per time step, which forms the same fp32 products and sums in
the same order: the same losses, parameters and evaluation bit for bit, at every
width it takes, batches around its row tiles, one step of recurrence and none,
both block shapes (one and two row tiles), several chunks and a masked group."""
import numpy as np
import pytest

from gpu_common import assert_losses_close, require_gpu
from paper_2609_37899_amd import soma, synth

pytestmark = pytest.mark.gpu


# N, L, E, H, B, T, P, directions a pass, law, mask
CASES = [(1, 1, 16, 16, 1, 2, 1, 0, 0, 0), (2, 2, 48, 16, 17, 9, 40, 0, 1, 0), (2, 2, 32, 48, 16, 3, 3, 2, 2, 0),
         (3, 2, 48, 80, 10, 65, 4, 0, 2, 0), (4, 1, 64, 80, 33, 12, 32, 0, 0, soma.PERTURB_LSTM),
         (1, 3, 112, 112, 31, 17, 5, 0, 1, 0), (4, 2, 16, 112, 70, 8, 30, 0, 0, 0),
         (1, 2, 144, 144, 64, 6, 3, 0, 0, soma.PERTURB_HEAD), (2, 2, 32, 144, 5, 20, 2, 1, 1, 0)]


@pytest.mark.parametrize("N,L,E,H,B,T,P,pc,law,mask", CASES)
def test_one_launch_is_the_launch_per_step(oracle_mod, N, L, E, H, B, T, P, pc, law, mask):
    torch = require_gpu()
    theta = synth.init_theta(N, L, E, H, init_seed=4, distinct=True)
    data = synth.expert_batches([70 + e for e in range(N)], B, T)
    seeds = soma.seeds_tensor(synth.expert_seeds(N))
    outs, launches = [], []
    for flags in (0, soma.FLAG_PER_STEP_RECURRENCE):
        ctx = soma.Context(soma.Shape(N, L, E, H, B, T, P, 0, pc, flags, law, 1, soma.ARCH_LSTM, mask))
        ctx.set_phase_timing(True)
        th, db = torch.from_numpy(theta.copy()).cuda(), torch.from_numpy(data).cuda()
        losses = torch.zeros((N, P, 2), dtype=torch.float32, device="cuda")
        loss = torch.zeros(N, dtype=torch.float32, device="cuda")
        print(f"H={H} B={B} T={T} flags={flags}: evaluation, step", flush=True)
        ctx.eval_loss(th, db, loss)
        ctx.spsa_step(th, seeds, 2, 1e-3, 1e-2, db, losses)
        launches.append(ctx.phase_times()["rec_launches"])
        torch.cuda.synchronize()
        outs.append([x.cpu().numpy() for x in (th, losses, loss)])
        ctx.close()
    chunks = (P + (pc or P) - 1) // (pc or P)
    assert launches == [L * chunks, L * (T - 1) * chunks]
    for a, b in zip(*outs):
        assert np.isfinite(a).all() and np.array_equal(a, b)
    cfg = oracle_mod.make_cfg(N, L, E, H, B, T, P)
    assert_losses_close(outs[0][2], oracle_mod.eval_loss(cfg, theta, data))


# the widths of the resident projection and head; few and many slots (rows of a
# slot cut into runs that end in a ragged tile, or whole), B beyond 16 and below
@pytest.mark.parametrize("N,L,E,H,B,T,P,pc,law,mask",
                         [(1, 1, 16, 16, 3, 9, 1, 0, 0, 0), (8, 2, 16, 16, 40, 30, 32, 0, 0, 0),
                          (2, 2, 32, 32, 17, 40, 64, 0, 1, 0), (4, 2, 48, 48, 65, 9, 40, 7, 2, 0),
                          (2, 2, 48, 80, 10, 65, 40, 0, 0, soma.PERTURB_HEAD), (3, 1, 96, 96, 1, 300, 50, 0, 0, 0),
                          (4, 2, 96, 96, 33, 20, 40, 0, 2, 0), (3, 2, 112, 112, 5, 70, 43, 0, 0, soma.PERTURB_LSTM),
                          (2, 2, 144, 144, 64, 12, 48, 0, 1, 0), (1, 3, 144, 144, 2, 33, 129, 0, 0, 0)])
def test_resident_weights_are_the_tiled_weights(N, L, E, H, B, T, P, pc, law, mask):
    """k_head_narrow, and k_proj_narrow where its slots fill the chip (the test below sees to
    that), against k_head_ce and k_proj: the same bits."""
    torch = require_gpu()
    theta = synth.init_theta(N, L, E, H, init_seed=4, distinct=True)
    data = synth.expert_batches([70 + e for e in range(N)], B, T)
    seeds = soma.seeds_tensor(synth.expert_seeds(N))
    outs = []
    for flags in (0, soma.FLAG_TILED_WEIGHTS):
        ctx = soma.Context(soma.Shape(N, L, E, H, B, T, P, 0, pc, flags, law, 1, soma.ARCH_LSTM, mask))
        th, db = torch.from_numpy(theta.copy()).cuda(), torch.from_numpy(data).cuda()
        losses = torch.zeros((N, P, 2), dtype=torch.float32, device="cuda")
        loss = torch.zeros(N, dtype=torch.float32, device="cuda")
        print(f"H={H} B={B} T={T} flags={flags}: evaluation, step", flush=True)
        ctx.eval_loss(th, db, loss)
        ctx.spsa_step(th, seeds, 2, 1e-3, 1e-2, db, losses)
        torch.cuda.synchronize()
        outs.append([x.cpu().numpy() for x in (th, losses, loss)])
        ctx.close()
    for a, b in zip(*outs):
        assert np.isfinite(a).all() and np.array_equal(a, b)


# Slots and 64-row tiles at which the resident projection runs on 256 compute
# units, at every width it has an instance for: rows of a slot in one, two, three
# and four runs, ragged last tiles, gate tiles dealt evenly over a slot's blocks
# and not (H = 80: 20 over 2 x 4 waves, 112: 28 over 4 x 4, 144: 36 over 3 x 4).
PROJ_CASES = [(1, 2, 16, 16, 64, 9, 64, 0, 0, 0), (4, 3, 32, 32, 5, 20, 64, 0, 1, 0), (2, 2, 48, 48, 18, 31, 40, 0, 2, 0),
              (4, 2, 16, 48, 13, 8, 64, 0, 0, soma.PERTURB_LSTM), (2, 2, 80, 80, 33, 16, 32, 0, 0, 0),
              (4, 3, 32, 80, 17, 10, 64, 32, 2, 0), (1, 2, 48, 96, 7, 72, 32, 0, 1, 0),
              (1, 2, 112, 112, 20, 23, 32, 0, 0, 0), (2, 2, 16, 112, 50, 3, 32, 0, 1, soma.PERTURB_HEAD),
              (2, 2, 144, 144, 31, 17, 32, 0, 0, 0), (4, 2, 32, 144, 21, 22, 32, 0, 2, 0)]


@pytest.mark.parametrize("N,L,E,H,B,T,P,pc,law,mask", PROJ_CASES)
def test_resident_projection_is_the_tiled_one(N, L, E, H, B, T, P, pc, law, mask):
    torch = require_gpu()
    theta = synth.init_theta(N, L, E, H, init_seed=6, distinct=True)
    data = synth.expert_batches([90 + e for e in range(N)], B, T)
    seeds = soma.seeds_tensor(synth.expert_seeds(N))
    outs, launches = [], []
    for flags in (0, soma.FLAG_TILED_WEIGHTS):
        ctx = soma.Context(soma.Shape(N, L, E, H, B, T, P, 0, pc, flags, law, 1, soma.ARCH_LSTM, mask))
        ctx.set_phase_timing(True)
        th, db = torch.from_numpy(theta.copy()).cuda(), torch.from_numpy(data).cuda()
        losses = torch.zeros((N, P, 2), dtype=torch.float32, device="cuda")
        print(f"H={H} B={B} T={T} flags={flags}: step", flush=True)
        ctx.spsa_step(th, seeds, 2, 1e-3, 1e-2, db, losses)
        launches.append((ctx.phase_times()["proj_launches"], ctx.narrow_projections()))
        torch.cuda.synchronize()
        outs.append([x.cpu().numpy() for x in (th, losses)])
        ctx.close()
    n = (L - 1) * ((P + (pc or P) - 1) // (pc or P))
    assert launches == [(n, n), (n, 0)]
    for a, b in zip(*outs):
        assert np.isfinite(a).all() and np.array_equal(a, b)


@pytest.mark.parametrize("H", [32, 48, 80, 96, 112, 144])
def test_resident_projection_of_an_evaluation(H):
    """Many experts: an evaluation's slots fill the chip too, perturbed by a radius of zero
    (no flags) and unperturbed (the kernels of the launch per step)."""
    torch = require_gpu()
    N, L, E, B, T, P = 512, 2, 16, 5, 16, 1
    theta = torch.from_numpy(synth.init_theta(N, L, E, H, init_seed=7)).cuda()
    data = torch.from_numpy(np.repeat(synth.expert_batches([95], B, T), N, axis=0)).cuda()
    seeds = soma.seeds_tensor(synth.expert_seeds(N))
    outs = []
    for flags in (0, soma.FLAG_PER_STEP_RECURRENCE, soma.FLAG_PER_STEP_RECURRENCE | soma.FLAG_TILED_WEIGHTS):
        ctx = soma.Context(soma.Shape(N, L, E, H, B, T, P, flags=flags))
        loss = torch.zeros(N, dtype=torch.float32, device="cuda")
        losses = torch.zeros((N, P, 2), dtype=torch.float32, device="cuda")
        print(f"H={H} flags={flags}: step, evaluation", flush=True)
        ctx.spsa_step(theta.clone(), seeds, 2, 1e-3, 1e-2, data, losses)
        before = ctx.narrow_projections()
        ctx.eval_loss(theta, data, loss)
        assert ctx.narrow_projections() - before == (0 if flags & soma.FLAG_TILED_WEIGHTS else 1)
        torch.cuda.synchronize()
        outs.append(loss.cpu().numpy())
        ctx.close()
    assert np.isfinite(outs[0]).all() and np.all(outs[0] == outs[0][0])
    assert np.array_equal(outs[1], outs[2])
    assert_losses_close(outs[0], outs[1])
