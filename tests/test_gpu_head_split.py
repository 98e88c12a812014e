"""The streaming head with a job's rows shared by several blocks: an evaluation
and a step whose slots leave compute units idle (so the rows are cut, into runs
of 64-row tiles that start inside a time step and end in a ragged tile), against
the oracle, at the tolerance of the other parity tests."""
import numpy as np
import pytest

from gpu_common import assert_losses_close, require_gpu
from paper_2609_37899_amd import soma, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,H,B,T", [(1, 192, 29, 60), (2, 256, 40, 30), (1, 320, 100, 21)])
def test_head_rows_shared_by_blocks(oracle_mod, N, H, B, T):
    torch = require_gpu()
    theta = synth.init_theta(N, 1, 32, H, init_seed=9, distinct=True)
    data = synth.expert_batches([1000 + e for e in range(N)], B, T)
    cfg = oracle_mod.make_cfg(N, 1, 32, H, B, T, 1)
    ctx = soma.Context(soma.Shape(N, 1, 32, H, B, T, 1))
    th, db = torch.from_numpy(theta.copy()).cuda(), torch.from_numpy(data).cuda()
    print(f"H={H} B={B} T={T}: evaluation, step", flush=True)
    loss = torch.zeros(N, dtype=torch.float32, device="cuda")
    ctx.eval_loss(th, db, loss)
    losses = torch.zeros((N, 1, 2), dtype=torch.float32, device="cuda")
    seeds = synth.expert_seeds(N)
    ctx.spsa_step(th, soma.seeds_tensor(seeds), 4, 1e-3, 1e-3, db, losses)
    torch.cuda.synchronize()
    assert_losses_close(loss.cpu().numpy(), oracle_mod.eval_loss(cfg, theta, data))
    assert_losses_close(losses.cpu().numpy(), oracle_mod.spsa_step(cfg, theta, seeds, 4, 1e-3, 1e-3, data)["losses"])
