"""GPU parity of the batched products (k_mm) at the edges of their tiles, through
the calls that run them: the projection of the stacked LSTM (N = 4 H, whole
row tiles), and the wide body's four products at padded widths that take each
shape of tile (d_p = 64, 192: 128 x 128 down projections; 256, 512: 256 x 256;
384: 384 x 128), with row counts B (T - 1) below, at and past a tile of 128 and
256 and not a multiple of 16.  Against the oracle, at the tolerances of the
other parity tests; the projection also bit for bit against the streaming one,
which sums in the same order."""
import numpy as np
import pytest

from gpu_common import assert_losses_close, assert_theta_close, require_gpu
from paper_2609_37899_amd import soma, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,B,T", [(128, 33, 2), (192, 64, 5), (320, 48, 7), (256, 100, 4)])
def test_projection_equals_the_streaming_one(H, B, T):
    check_projection(H, B, T, 2)


# More 128 x 128 tiles than the chip holds at once: the large tiles run.
@pytest.mark.parametrize("H,B,T", [(128, 33, 7), (192, 64, 5), (256, 100, 5)])
def test_projection_on_large_tiles_equals_the_streaming_one(H, B, T):
    check_projection(H, B, T, 80)


def check_projection(H, B, T, P):
    torch = require_gpu()
    N, L, E = 1, 3, 32
    theta = torch.from_numpy(synth.init_theta(N, L, E, H, init_seed=5)).cuda()
    data = torch.from_numpy(synth.expert_batches([900], B, T)).cuda()
    seeds = soma.seeds_tensor(synth.expert_seeds(N))
    out = []
    for flags in (0, soma.FLAG_FP32_SEQUENCE):
        ctx = soma.Context(soma.Shape(N, L, E, H, B, T, P, flags=flags))
        th, losses = theta.clone(), torch.zeros((N, P, 2), dtype=torch.float32, device="cuda")
        print(f"H={H} B={B} T={T} flags={flags}: step", flush=True)
        ctx.spsa_step(th, seeds, 1, 1e-3, 1e-3, data, losses)
        torch.cuda.synchronize()
        out.append((th.cpu().numpy(), losses.cpu().numpy()))
        ctx.close()
    assert np.all(np.isfinite(out[0][1]))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("dt,B,T", [(50, 7, 3), (190, 16, 9), (250, 17, 9), (361, 43, 4), (300, 64, 5), (449, 34, 9)])
def test_wide_products_match_oracle(oracle_mod, dt, B, T):
    check_wide(oracle_mod, dt, B, T, 2)


@pytest.mark.parametrize("dt,B,T", [(250, 17, 9), (361, 43, 4), (449, 34, 9)])
def test_wide_products_on_large_tiles_match_oracle(oracle_mod, dt, B, T):
    check_wide(oracle_mod, dt, B, T, 40)


def check_wide(oracle_mod, dt, B, T, P):
    torch = require_gpu()
    N, D = 2, 1
    theta = synth.init_wide(N, D, dt, 32, init_seed=7, distinct=True)
    head = synth.init_tied_head(32, init_seed=8, n_experts=N)
    data = synth.expert_batches([950 + e for e in range(N)], B, T)
    seeds = synth.expert_seeds(N)
    ctx = soma.Context(soma.Shape(N, D, 32, dt, B, T, P, arch=soma.ARCH_WIDE))
    E = torch.from_numpy(head.copy()).cuda()
    ctx.set_tied_head(E, per_expert=True)
    th = torch.from_numpy(theta.copy()).cuda()
    losses = torch.zeros((N, P, 2), dtype=torch.float32, device="cuda")
    print(f"d_t={dt} B={B} T={T}: step", flush=True)
    ctx.spsa_step(th, soma.seeds_tensor(seeds), 2, 1e-3, 1e-3, torch.from_numpy(data).cuda(), losses)
    torch.cuda.synchronize()
    cfg = oracle_mod.make_cfg(N, D, 32, dt, B, T, P, arch=oracle_mod.ARCH_WIDE, tied_head=head)
    ref = oracle_mod.spsa_step(cfg, theta, seeds, 2, 1e-3, 1e-3, data)
    assert_losses_close(losses.cpu().numpy(), ref["losses"])
    assert_theta_close(th.cpu().numpy(), ref["theta"])
