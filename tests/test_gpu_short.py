"""The shortest windows of the exchange recurrence, on both sides of the lines that its
launch rule draws by jobs and idle compute units: which recurrence runs (one launch a
layer of the exchange or the staged recurrence, or one a time step), the oracle's
losses and weights from either, the same bits whatever the direction chunk (the rule
must not go by the chunk's jobs), and an evaluation by its own few jobs."""
import numpy as np
import pytest

from gpu_common import assert_losses_close, assert_theta_close, require_gpu
from paper_2609_37899_amd import soma, synth

pytestmark = pytest.mark.gpu

# (L, H, B, T, P, probe), exchange: jobs = 2 P ceil(B / 64) for the one expert
CASES = [((2, 128, 33, 2, 8, 0), True), ((2, 128, 33, 2, 9, 0), False), ((1, 192, 64, 2, 1, 1), False),
         ((1, 192, 64, 3, 1, 1), True), ((2, 320, 40, 3, 9, 2), True), ((2, 320, 40, 2, 16, 1), True), ((2, 320, 40, 2, 17, 1), False),
         ((2, 704, 33, 3, 9, 1), False), ((2, 704, 33, 3, 8, 1), True),
         ((1, 384, 65, 5, 8, 0), True), ((1, 384, 65, 5, 9, 0), False), ((1, 384, 65, 6, 9, 0), True),
         ((1, 576, 70, 5, 4, 0), True), ((1, 576, 70, 5, 5, 0), False), ((1, 576, 70, 6, 5, 0), True),
         ((1, 576, 70, 6, 9, 1), False), ((1, 640, 65, 7, 9, 0), True), ((1, 640, 65, 7, 9, 1), False),
         ((1, 512, 65, 5, 30, 0), True), ((1, 512, 65, 4, 1, 0), False)]


@pytest.mark.parametrize("case,exchange", CASES, ids=lambda c: "h%d_b%d_t%d_p%d" % c[1:5] if isinstance(c, tuple) else None)
def test_short_windows(oracle_mod, case, exchange):
    torch = require_gpu()
    L, H, B, T, P, probe = case
    N, E = 1, 16
    theta = synth.init_theta(N, L, E, H, init_seed=8, distinct=True)
    data = synth.expert_batches([730], B, T)
    seeds = synth.expert_seeds(N)
    outs = []
    for pc in (0, max(1, P // 2)):
        ctx = soma.Context(soma.Shape(N, L, E, H, B, T, P, probe=probe, pair_chunk=pc))
        ctx.set_phase_timing(True)
        th = torch.from_numpy(theta.copy()).cuda()
        losses = torch.zeros((N, P, 2), dtype=torch.float32, device="cuda")
        print(f"L={L} H={H} B={B} T={T} P={P} chunk {pc}: step", flush=True)
        ctx.spsa_step(th, soma.seeds_tensor(seeds), 7, 1e-3, 1e-3, torch.from_numpy(data).cuda(), losses)
        pt = ctx.phase_times()
        torch.cuda.synchronize()
        chunks = (P + (pc or P) - 1) // (pc or P)
        assert pt["xchg_launches"] == (L * chunks if exchange else 0)
        assert pt["rec_launches"] == L * chunks * (1 if exchange or B <= 64 else T - 1)
        before = torch.from_numpy(theta.copy()).cuda()
        loss = torch.zeros(N, dtype=torch.float32, device="cuda")
        ctx.eval_loss(before, torch.from_numpy(data).cuda(), loss)
        least = (3 if L == 1 else 2) if B <= 64 else 5      # two or four jobs
        assert ctx.phase_times()["xchg_launches"] - pt["xchg_launches"] == (L if T >= least else 0)
        outs.append((th.cpu().numpy(), losses.cpu().numpy(), loss.cpu().numpy()))
        ctx.close()
    for a, b in zip(*outs):
        assert np.array_equal(a, b)
    cfg = oracle_mod.make_cfg(N, L, E, H, B, T, P, probe=probe)
    ref = oracle_mod.spsa_step(cfg, theta, seeds, 7, 1e-3, 1e-3, data)
    assert_losses_close(outs[0][1], ref["losses"])
    assert_losses_close(outs[0][2], oracle_mod.eval_loss(cfg, theta, data))
    assert_theta_close(outs[0][0], ref["theta"])
