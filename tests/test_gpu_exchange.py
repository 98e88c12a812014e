"""GPU parity of the exchange recurrence over the widths and batches it takes:
every multiple of 64 from 128 to 704, batches from 33 sequences (three row
tiles, one of them nearly empty) over 64 (cut into jobs of 64, the last one
ragged), with and without whole row tiles, in one and two layers (the gate
inputs gathered from the folded table and read from the projection), and on
the wide body's pre-formed weights at its smallest padded width.

The tolerances are those of the other parity tests.  lr = 1e-3: a loss error
of 3e-8 of its value (fp32 sums; L = 5.5) moves a weight by
lr max|z| 1.7e-7 / (2 eps P), which at P = 1 and max|z| = 5.5 (5 million
Gaussian draws) is 4.6e-7, 2e-5 of the smallest rms weight here (0.023 at
H = 640); at lr = 1e-2 it would be twice the bar of 1e-4."""
import numpy as np
import pytest

from gpu_common import assert_losses_close, assert_theta_close, require_gpu
from paper_2609_37899_amd import soma, synth

pytestmark = pytest.mark.gpu

# (N, L, E, H, B, T, P, probe)
CASES = [
    (1, 2, 32, 192, 64, 7, 3, 1),     # H / 64 odd, whole tiles
    (1, 2, 32, 320, 33, 6, 2, 0),     # one row of the third tile
    (2, 1, 16, 128, 65, 5, 2, 2),     # one row of a second job
    (1, 2, 32, 256, 80, 5, 2, 0),     # two jobs, whole tiles, the sequence stored split
    (1, 2, 32, 128, 100, 9, 2, 1),    # two jobs, ragged
    (1, 2, 48, 448, 48, 4, 2, 0),     # three whole tiles
    (1, 2, 32, 576, 49, 4, 1, 2),
    (1, 2, 32, 640, 64, 3, 1, 0),
    (1, 1, 32, 384, 129, 5, 1, 0),    # three jobs, the fewest steps of a batch cut into jobs
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "h%d_b%d_l%d" % (c[3], c[4], c[1]))
def test_exchange_step_matches_oracle(oracle_mod, case):
    torch = require_gpu()
    N, L, E, H, B, T, P, probe = case
    theta = synth.init_theta(N, L, E, H, init_seed=2, distinct=True)
    data = synth.expert_batches([700 + e for e in range(N)], B, T)
    seeds = synth.expert_seeds(N)
    print(f"H={H} B={B}: step", flush=True)
    ctx = soma.Context(soma.Shape(N, L, E, H, B, T, P, probe=probe))
    ctx.set_phase_timing(True)
    th = torch.from_numpy(theta.copy()).cuda()
    losses = torch.zeros((N, P, 2), dtype=torch.float32, device="cuda")
    ctx.spsa_step(th, soma.seeds_tensor(seeds), 7, 1e-3, 1e-3, torch.from_numpy(data).cuda(), losses)
    torch.cuda.synchronize()
    assert ctx.phase_times()["xchg_launches"] == L
    ref = oracle_mod.spsa_step(oracle_mod.make_cfg(N, L, E, H, B, T, P, probe=probe), theta, seeds, 7, 1e-3, 1e-3, data)
    assert_losses_close(losses.cpu().numpy(), ref["losses"])
    assert_theta_close(th.cpu().numpy(), ref["theta"])


@pytest.mark.parametrize("dt,B", [(13, 40), (130, 33)])
def test_wide_exchange_matches_oracle(oracle_mod, dt, B):
    torch = require_gpu()
    N, D, T, P = 2, 2, 6, 2
    theta = synth.init_wide(N, D, dt, 32, init_seed=4, distinct=True)
    head = synth.init_tied_head(32, init_seed=6, n_experts=N)
    data = synth.expert_batches([800 + e for e in range(N)], B, T)
    seeds = synth.expert_seeds(N)
    print(f"d_t={dt} B={B}: step", flush=True)
    ctx = soma.Context(soma.Shape(N, D, 32, dt, B, T, P, probe=1, arch=soma.ARCH_WIDE))
    E = torch.from_numpy(head.copy()).cuda()
    ctx.set_tied_head(E, per_expert=True)
    ctx.set_phase_timing(True)
    th = torch.from_numpy(theta.copy()).cuda()
    losses = torch.zeros((N, P, 2), dtype=torch.float32, device="cuda")
    ctx.spsa_step(th, soma.seeds_tensor(seeds), 3, 1e-3, 1e-3, torch.from_numpy(data).cuda(), losses)
    torch.cuda.synchronize()
    assert ctx.phase_times()["xchg_launches"] == D
    cfg = oracle_mod.make_cfg(N, D, 32, dt, B, T, P, probe=1, arch=oracle_mod.ARCH_WIDE, tied_head=head)
    ref = oracle_mod.spsa_step(cfg, theta, seeds, 3, 1e-3, 1e-3, data)
    assert_losses_close(losses.cpu().numpy(), ref["losses"])
    assert_theta_close(th.cpu().numpy(), ref["theta"])


@pytest.mark.parametrize("case", [(1, 2, 32, 256, 49, 12, 6, 0), (1, 2, 32, 128, 100, 15, 20, 1),
                                  (2, 1, 16, 704, 33, 9, 3, 2), (1, 2, 32, 512, 65, 10, 5, 0)],
                         ids=lambda c: "h%d_b%d_l%d" % (c[3], c[4], c[1]))
def test_exchange_step_is_repeatable(case):
    """Ragged row tiles, jobs of a batch beyond 64, several jobs a group: every repeat has the same bits."""
    torch = require_gpu()
    N, L, E, H, B, T, P, probe = case
    theta = torch.from_numpy(synth.init_theta(N, L, E, H, init_seed=2, distinct=True)).cuda()
    data = torch.from_numpy(synth.expert_batches([700 + e for e in range(N)], B, T)).cuda()
    seeds = soma.seeds_tensor(synth.expert_seeds(N))
    ctx = soma.Context(soma.Shape(N, L, E, H, B, T, P, probe=probe))
    ctx.set_phase_timing(True)
    first = None
    for i in range(12):
        th, losses = theta.clone(), torch.zeros((N, P, 2), dtype=torch.float32, device="cuda")
        ctx.spsa_step(th, seeds, 7, 1e-3, 1e-3, data, losses)
        assert ctx.phase_times()["xchg_launches"] == L
        out = (th.cpu().numpy(), losses.cpu().numpy())
        first = first or out
        assert np.all(np.isfinite(out[1]))
        assert np.array_equal(out[0], first[0]) and np.array_equal(out[1], first[1]), f"repeat {i}"


@pytest.mark.parametrize("dt,B", [(130, 33), (361, 50)])
def test_wide_exchange_step_is_repeatable(dt, B):
    torch = require_gpu()
    N, D, T, P = 2, 2, 10, 4
    theta = torch.from_numpy(synth.init_wide(N, D, dt, 32, init_seed=4, distinct=True)).cuda()
    E = torch.from_numpy(synth.init_tied_head(32, init_seed=6, n_experts=N)).cuda()
    data = torch.from_numpy(synth.expert_batches([800 + e for e in range(N)], B, T)).cuda()
    seeds = soma.seeds_tensor(synth.expert_seeds(N))
    ctx = soma.Context(soma.Shape(N, D, 32, dt, B, T, P, probe=1, arch=soma.ARCH_WIDE))
    ctx.set_tied_head(E, per_expert=True)
    first = None
    for i in range(8):
        th, losses = theta.clone(), torch.zeros((N, P, 2), dtype=torch.float32, device="cuda")
        loss = torch.zeros(N, dtype=torch.float32, device="cuda")
        ctx.spsa_step(th, seeds, 3, 1e-3, 1e-3, data, losses)
        ctx.eval_loss(th, data, loss)                     # one sign a job
        torch.cuda.synchronize()
        out = [x.cpu().numpy() for x in (th, losses, loss)]
        first = first or out
        assert all(np.isfinite(x).all() for x in out)
        assert all(np.array_equal(a, b) for a, b in zip(out, first)), f"repeat {i}"
