"""The wide body at widths around the edges of the kernels that form its weights (and
the fragments of E) and normalise its rows: fewer column quads than a block has
threads and more (one row over two blocks), the last groups of eight and of four
partial, one, two and three 64-column groups of LayerNorm (one, two and four rows a
wave); rows below, at and past its 16-row tiles; experts with their own and with one
shared tied matrix.  At the tolerances of the other parity tests."""
import numpy as np
import pytest

from gpu_common import assert_losses_close, assert_theta_close, require_gpu
from paper_2609_37899_amd import soma, synth

pytestmark = pytest.mark.gpu


# N, D, d_t, B, T, P, law, one E for all
@pytest.mark.parametrize("N,D,dt,B,T,P,law,shared", [
    (1, 1, 4, 1, 2, 1, 0, False), (2, 2, 5, 3, 6, 2, 1, False), (3, 1, 8, 16, 2, 2, 2, True), (2, 1, 9, 5, 7, 2, 0, False),
    (2, 2, 16, 17, 3, 2, 1, True), (2, 2, 43, 8, 5, 2, 0, False), (1, 1, 63, 33, 4, 2, 1, False),
    (2, 1, 64, 40, 5, 2, 0, False), (2, 2, 64, 64, 3, 1, 2, False), (3, 1, 65, 7, 5, 1, 1, False),
    (2, 1, 127, 9, 4, 1, 0, False), (2, 1, 128, 34, 3, 1, 1, True), (1, 1, 129, 6, 5, 1, 0, False)])
def test_wide_step_matches_oracle(oracle_mod, N, D, dt, B, T, P, law, shared):
    torch = require_gpu()
    theta = synth.init_wide(N, D, dt, 32, init_seed=12, distinct=True)
    head = synth.init_tied_head(32, init_seed=13, n_experts=0 if shared else N)
    data = synth.expert_batches([970 + e for e in range(N)], B, T)
    seeds = synth.expert_seeds(N)
    print(f"d_t={dt} B={B} T={T}: evaluation, step", flush=True)
    ctx = soma.Context(soma.Shape(N, D, 32, dt, B, T, P, probe=law, arch=soma.ARCH_WIDE))
    E = torch.from_numpy(head.copy()).cuda()
    ctx.set_tied_head(E, per_expert=not shared)
    th, db = torch.from_numpy(theta.copy()).cuda(), torch.from_numpy(data).cuda()
    loss = torch.zeros(N, dtype=torch.float32, device="cuda")
    losses = torch.zeros((N, P, 2), dtype=torch.float32, device="cuda")
    ctx.eval_loss(th, db, loss)
    ctx.spsa_step(th, soma.seeds_tensor(seeds), 3, 1e-3, 1e-3, db, losses)
    torch.cuda.synchronize()
    cfg = oracle_mod.make_cfg(N, D, 32, dt, B, T, P, probe=law, arch=oracle_mod.ARCH_WIDE, tied_head=head)
    ref = oracle_mod.spsa_step(cfg, theta, seeds, 3, 1e-3, 1e-3, data)
    assert_losses_close(loss.cpu().numpy(), oracle_mod.eval_loss(cfg, theta, data))
    assert_losses_close(losses.cpu().numpy(), ref["losses"])
    assert_theta_close(th.cpu().numpy(), ref["theta"])
