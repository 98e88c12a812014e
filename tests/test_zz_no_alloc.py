"""soma_spsa_step_noalloc (the step for callers that cannot allocate) against
soma_spsa_step through the C ABI: two calls in a row on one GPU, the second
with a smaller input, each bit for bit equal to the workspace entry point's
result at the same direction chunk (the same kernels), and the shape limit
of the static scratch."""
import numpy as np
import pytest

from gpu_common import require_gpu
from paper_2609_37899_amd import soma, synth

pytestmark = pytest.mark.gpu

# (N, L, E, H, B, T, P, eps, lr): the persistent recurrence at H = 128 (its
# group counters and abort flag live in the scratch), then a smaller shape at
# H = 64 (one block per job).
CALLS = [(2, 2, 64, 128, 16, 12, 3, 1e-3, 1e-2), (1, 1, 32, 64, 4, 32, 2, 1e-3, 1e-2)]


def _inputs(N, L, E, H, B, T, seed):
    theta = synth.init_theta(N, L, E, H, init_seed=seed, distinct=True)
    data = synth.expert_batches([300 + 10 * seed + e for e in range(N)], B, T)
    return theta, data, synth.expert_seeds(N, base=0x50A10000 + seed)


def test_noalloc_step_matches_the_workspace_step():
    torch = require_gpu()
    for i, (N, L, E, H, B, T, P, eps, lr) in enumerate(CALLS):
        shape = soma.Shape(N, L, E, H, B, T, P)
        theta, data, seeds = _inputs(N, L, E, H, B, T, i)
        dseeds = soma.seeds_tensor(seeds)
        dbytes = torch.from_numpy(data).cuda()
        results = []
        for noalloc in (True, False):
            th = torch.from_numpy(theta.copy()).cuda()
            losses = torch.full((N, P, 2), -1.0, dtype=torch.float32, device="cuda")
            if noalloc:
                soma.spsa_step_noalloc(shape, th, dseeds, 5, eps, lr, dbytes, losses)
            else:
                ctx = soma.Context(shape)
                ctx.spsa_step(th, dseeds, 5, eps, lr, dbytes, losses)
            torch.cuda.synchronize()
            results.append((th.cpu().numpy(), losses.cpu().numpy()))
            if not noalloc:
                ctx.close()
        (t0, l0), (t1, l1) = results
        print(f"call {i} (N={N} H={H} B={B} T={T} P={P}): losses {l0.mean():.6f}")
        assert np.all(np.isfinite(l0)) and np.all(l0 > 0)
        assert np.array_equal(l0, l1)
        assert np.array_equal(t0, t1)
        assert not np.array_equal(t0, theta)


def test_noalloc_rejects_shapes_beyond_its_scratch():
    torch = require_gpu()
    shape = soma.Shape(2, 2, 512, 512, 64, 256, 32)   # ~600 MB of workspace per direction
    th = torch.zeros((2, soma.param_count(shape)), dtype=torch.float32, device="cuda")
    losses = torch.zeros((2, 32, 2), dtype=torch.float32, device="cuda")
    with pytest.raises(soma.SomaError) as e:
        soma.spsa_step_noalloc(shape, th, soma.seeds_tensor(synth.expert_seeds(2)), 0, 1e-3, 1e-3,
                               torch.zeros((2, 64, 256), dtype=torch.uint8, device="cuda"), losses)
    assert e.value.code == soma.SOMA_ESHAPE
    assert torch.all(th == 0)


# Near the limit of the static scratch, two layers on the exchange recurrence:
# 33 sequences (its gate inputs padded to 48 rows a step, the ring beyond the
# limit), 65 (two jobs a slot, 80 rows), a whole tile count, and the widths and
# batches whose ring once counted against the limit and whose ring did not.  The
# direction chunk is what fits; a step's bits do not depend on it, nor on the
# projection (the workspace entry point's k_mm and, with the fp32 sequence, the
# same streaming one).
@pytest.mark.parametrize("L,H,B,T,P", [(2, 128, 33, 160, 3), (2, 256, 65, 37, 2), (2, 320, 64, 30, 2), (2, 256, 64, 40, 2),
                                       (2, 128, 80, 73, 2), (1, 704, 33, 105, 2)])
def test_noalloc_step_on_the_exchange_recurrence(L, H, B, T, P):
    torch = require_gpu()
    N, E = 1, 32
    theta, data, seeds = _inputs(N, L, E, H, B, T, 7)
    dseeds, dbytes = soma.seeds_tensor(seeds), torch.from_numpy(data).cuda()
    # The least chunk comes close to the 32 MiB it may take.
    one = soma.workspace_size(soma.Shape(N, L, E, H, B, T, P, pair_chunk=1, flags=soma.FLAG_STAGED_RECURRENCE))
    assert 24 * 2**20 < one <= 32 * 2**20
    results = []
    for flags in (None, 0, soma.FLAG_FP32_SEQUENCE):
        th = torch.from_numpy(theta.copy()).cuda()
        losses = torch.full((N, P, 2), -1.0, dtype=torch.float32, device="cuda")
        print(f"L={L} H={H} B={B} T={T} flags={flags}: step", flush=True)
        if flags is None:
            soma.spsa_step_noalloc(soma.Shape(N, L, E, H, B, T, P), th, dseeds, 5, 1e-3, 1e-3, dbytes, losses)
        else:
            ctx = soma.Context(soma.Shape(N, L, E, H, B, T, P, flags=flags))
            ctx.set_phase_timing(True)
            ctx.spsa_step(th, dseeds, 5, 1e-3, 1e-3, dbytes, losses)
            assert ctx.phase_times()["xchg_launches"] == L
        torch.cuda.synchronize()
        results.append((th.cpu().numpy(), losses.cpu().numpy()))
        if flags is not None:
            ctx.close()
    assert np.all(np.isfinite(results[0][1])) and not np.array_equal(results[0][0], theta)
    for t, l in results[1:]:
        assert np.array_equal(results[0][0], t) and np.array_equal(results[0][1], l)
