"""What this framework is timed on: SPSA steps, evaluations and delta-rule
updates through its public entry points (paper_2609_37899_amd.soma), over the
sizes, architectures, probe laws and updates that training runs use.

A case is one call on a shape.  ``draw`` gives further shapes of the same
ranges: the stacked LSTM at hidden widths 16 to 704 (multiples of 16), 1 to 4
layers, 1 to 256 experts, 1 to 128 sequences of 2 to 512 bytes, and the paper's
two bodies at the widths they support.
"""
from __future__ import annotations

import math

import torch

from paper_2609_37899_amd import soma

VOCAB = 256
PROBES = {"gaussian": soma.PROBE_GAUSSIAN, "sparse": soma.PROBE_SPARSE_RADEMACHER, "dense": soma.PROBE_RADEMACHER}
ARCHS = {"lstm": soma.ARCH_LSTM, "body": soma.ARCH_BODY, "wide": soma.ARCH_WIDE}
LOSS = {"independent": soma.LOSS_INDEPENDENT, "summed": soma.LOSS_SUMMED}
EPS, LR, FIRST_STEP, FIRST_UPDATE = 1e-3, 1e-3, 1000, 101   # a run in progress, not its first update
MOST_FLOPS = 2e13        # a drawn case's contraction work: a seventh of the largest listed one


def _case(call, arch, experts, layers, embed, hidden, batch, seq_len, pairs, probe="gaussian", loss="independent",
          accum=1, mask=0, name=None):
    c = {"call": call, "arch": arch, "experts": experts, "layers": layers, "embed": embed, "hidden": hidden,
         "batch": batch, "seq_len": seq_len, "pairs": pairs, "probe": probe, "loss": loss, "accum": accum, "mask": mask}
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest training step (smoke tests, hyperparameter trials on one
        # tiny expert): launches and the serial chain of time steps count.
        _case("step", "lstm", 1, 1, 32, 64, 8, 64, 4, name="step_tiny_h64"),
        # A small trial at sizes nobody rounded: widths that are not multiples
        # of 64, ragged batch rows, the paper's update and probe law.
        _case("adam", "lstm", 3, 2, 48, 80, 10, 65, 8, probe="sparse", name="step_odd_h80"),
        # Deeper narrow experts, embedding and head kept out of the search (as
        # the paper keeps its decoder), two accumulated batches per update.
        _case("adam", "lstm", 2, 3, 128, 128, 33, 100, 16, probe="dense", accum=2, mask=soma.PERTURB_LSTM,
              name="step_deep_h128_accum"),
        # A batch beyond 64 sequences.
        _case("step", "lstm", 1, 2, 256, 256, 100, 128, 16, name="step_batch100_h256"),
        # Many small experts, one GPU's share of a large ensemble.
        _case("step", "lstm", 256, 1, 32, 64, 16, 256, 32, name="step_n256_h64"),
        # The benchmark's default: two mid-size experts.
        _case("step", "lstm", 2, 2, 512, 512, 64, 256, 32, name="step_n2_h512"),
        # Four experts on longer windows, summed loss, the Adam-style update.
        _case("adam", "lstm", 4, 2, 384, 384, 32, 512, 32, loss="summed", name="step_n4_h384"),
        # The monolithic control: one wide stacked LSTM, 256 perturbed forwards.
        _case("step", "lstm", 1, 2, 704, 704, 64, 256, 128, name="step_mono_h704"),
        # The paper's own expert body, eight at once, its probe law and schedule.
        _case("sched", "body", 8, 2, 32, 32, 64, 1024, 64, probe="sparse", name="step_body_d32"),
        # The paper's wide fixed-size control (N = 2), its probe law and update.
        _case("adam", "wide", 2, 2, 32, 361, 64, 1024, 32, probe="sparse", name="step_wide_d361"),
        # Validation loss of the benchmark's experts (between updates).
        _case("eval", "lstm", 2, 2, 512, 512, 64, 256, 32, name="eval_n2_h512"),
        # The decoder's delta rule on the wide control's own heads.
        _case("delta", "wide", 2, 2, 32, 361, 64, 1024, 32, probe="sparse", name="delta_wide_d361"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    while True:
        kind = rng.random()
        seq = _log_int(rng, 2, 512)
        if kind < 0.70:
            call = rng.choice(("step", "step", "adam", "adam", "eval"))
            q = 64 if rng.random() < 0.6 else 16     # most users round widths, some do not
            hidden = max(q, _log_int(rng, 16, 704) // q * q)
            embed = hidden if rng.random() < 0.5 else 16 * _log_int(rng, 1, 32)
            c = _case(call, "lstm", _log_int(rng, 1, 64 if hidden <= 128 else 4), rng.choice((1, 2, 2, 3)), embed,
                      hidden, _log_int(rng, 1, 128), seq, _log_int(rng, 2, 64), probe=rng.choice(sorted(PROBES)),
                      loss=rng.choice(sorted(LOSS)), accum=rng.choice((1, 1, 1, 2)),
                      mask=rng.choice((0, 0, soma.PERTURB_LSTM, soma.PERTURB_LSTM | soma.PERTURB_HEAD)))
        elif kind < 0.82:
            call = rng.choice(("step", "adam", "sched", "eval", "delta"))
            d = rng.choice((16, 32))
            c = _case(call, "body", _log_int(rng, 1, 16), rng.choice((1, 2)), d, d, _log_int(rng, 1, 128),
                      2 * seq, _log_int(rng, 2, 64), probe=rng.choice(sorted(PROBES)))
        else:
            call = rng.choice(("step", "adam", "sched", "eval", "delta"))
            c = _case(call, "wide", _log_int(rng, 1, 8), rng.choice((1, 2)), 32, _log_int(rng, 13, 512),
                      _log_int(rng, 1, 64), seq, _log_int(rng, 2, 32), probe=rng.choice(sorted(PROBES)))
        if work(c)["flops"] <= MOST_FLOPS:
            return c


# --------------------------------------------------------------------------
# Shapes

def _shape(c):
    return soma.Shape(c["experts"], c["layers"], c["embed"], c["hidden"], c["batch"], c["seq_len"], c["pairs"],
                      LOSS[c["loss"]], 0, 0, PROBES[c["probe"]], c["accum"], ARCHS[c["arch"]], c["mask"])


def _params(c):
    """Parameters of one expert."""
    L, E, H = c["layers"], c["embed"], c["hidden"]
    if c["arch"] == "body":
        return L * (16 * H * H + 2 * H) + H
    if c["arch"] == "wide":
        return 16 * L * H * H + (2 * L + 1) * H + 2 * E * H
    return VOCAB * E + sum(4 * H * ((E if l == 0 else H) + H) for l in range(L)) + VOCAB * H


def _directions(c):
    return c["pairs"] * c["accum"]


def _own_heads(c):
    """The width-32 body's recipe freezes one E for all experts; the wide controls, and the delta rule, own theirs."""
    return c["arch"] == "wide" or c["call"] == "delta"


def work(case):
    c = case
    N, L, E, H, B, T = c["experts"], c["layers"], c["embed"], c["hidden"], c["batch"], c["seq_len"]
    rows, d = B * (T - 1), _params(c)
    forwards = N if c["call"] in ("eval", "delta") else N * 2 * _directions(c)
    # One forward's products; the input products of the vocabulary's 256 byte
    # values stand for those of all tokens where there are more tokens.
    first = min(rows, VOCAB)
    if c["arch"] == "lstm":
        one = first * E * 4 * H + rows * (L * 4 * H * H + (L - 1) * 4 * H * H + H * VOCAB)
    elif c["arch"] == "body":
        one = rows * (L * 16 * H * H + H * VOCAB)
    else:
        one = first * E * H + rows * (L * 16 * H * H + H * E + E * VOCAB)
    flops = 2 * one * forwards
    size = N * d * 4 + c["accum"] * N * B * T
    if c["arch"] != "lstm":
        size += (N if _own_heads(c) else 1) * VOCAB * E * 4
    if c["call"] == "eval":
        size += 4 * N
    elif c["call"] == "delta":
        flops += 2 * N * rows * VOCAB * E
        size += N * (2 * VOCAB * E + 1) * 4
    else:
        flops += 2 * N * d * _directions(c)
        size += N * d * 4 * (1 if c["call"] == "step" else 5) + N * _directions(c) * 8
    return {"bytes": float(size), "flops": float(flops)}


# --------------------------------------------------------------------------
# Inputs

def _inputs(c, seed, dev="cuda"):
    """Weights, batches and moments in device memory, from the seed alone."""
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed) & 0x7FFFFFFF)
    N, L, E, H, B, T = c["experts"], c["layers"], c["embed"], c["hidden"], c["batch"], c["seq_len"]
    d = _params(c)
    theta = torch.empty((N, d), device=dev).uniform_(-1.0, 1.0, generator=g)

    def gains(start, count):
        theta[:, start:start + count] = 1.0 + 0.1 * torch.randn((N, count), device=dev, generator=g)

    if c["arch"] == "lstm":          # torch's LSTM initialisation
        theta /= math.sqrt(H)
    elif c["arch"] == "body":
        at = 0
        for _ in range(L):
            for fan, count in ((0, H), (2 * H, 8 * H * H), (0, H), (H, 4 * H * H), (4 * H, 4 * H * H)):
                if fan:
                    theta[:, at:at + count] /= math.sqrt(fan)
                else:
                    gains(at, count)
                at += count
        gains(at, H)
    else:
        at = 0
        for fan, count in [(E, E * H)] + L * [(2 * H, 8 * H * H), (H, 4 * H * H), (4 * H, 4 * H * H)] + [(H, E * H)]:
            theta[:, at:at + count] /= math.sqrt(fan)
            at += count
        gains(at, (2 * L + 1) * H)
    # Byte frequencies of text are about Zipfian; each expert's cluster has its
    # own order of the byte values.
    p = (1.0 / torch.arange(1, VOCAB + 1, device=dev, dtype=torch.float32)).expand(N, VOCAB)
    order = torch.rand((N, VOCAB), device=dev, generator=g).argsort(dim=1)
    A = c["accum"]
    pick = torch.multinomial(p, A * B * T, replacement=True, generator=g)
    data = order.gather(1, pick).to(torch.uint8).view(N, A, B, T).transpose(0, 1).contiguous()
    x = {"theta": theta, "bytes": data,
         "seeds": torch.randint(0, 1 << 62, (N,), device=dev, generator=g, dtype=torch.int64)}
    if c["arch"] != "lstm":
        x["E"] = 0.3 * torch.randn((N if _own_heads(c) else 1, VOCAB, E), device=dev, generator=g)
    if c["call"] in ("adam", "sched"):
        x["m"] = 0.05 * torch.randn((N, d), device=dev, generator=g)
        x["v"] = 0.005 * torch.empty((N, d), device=dev).uniform_(0.5, 1.5, generator=g)
    return x


def prepare(case, seed):
    c = case
    s = _inputs(c, seed)
    s["call"], s["step"], s["t"] = c["call"], FIRST_STEP, FIRST_UPDATE
    s["ctx"] = soma.Context(_shape(c))
    if c["arch"] != "lstm":
        s["ctx"].set_tied_head(s["E"], per_expert=_own_heads(c))
    N = c["experts"]
    if c["call"] in ("eval", "delta"):
        s["loss"] = torch.zeros(N, device="cuda")
        if c["accum"] == 1:
            s["bytes"] = s["bytes"].view(N, c["batch"], c["seq_len"])
        else:                        # an evaluation reads one batch
            s["bytes"] = s["bytes"][0].contiguous()
        if c["call"] == "delta":
            s["grad"] = torch.zeros((N, VOCAB, c["embed"]), device="cuda")
    else:
        s["losses"] = torch.zeros((N, _directions(c), 2), device="cuda")
        s["adam"] = soma.Adam()
        if c["call"] == "sched":
            s["sched"] = soma.schedule_tensor(N)
            soma.schedule_init(s["sched"], LR, EPS)
    return s


def run(state):
    s = state
    ctx, call = s["ctx"], s["call"]
    if call == "eval":
        ctx.eval_loss(s["theta"], s["bytes"], s["loss"])
        return {"loss": s["loss"]}
    if call == "delta":
        ctx.head_delta(s["theta"], s["bytes"], LR, s["grad"], s["loss"])
        return {"loss": s["loss"], "grad": s["grad"], "E": s["E"]}
    if call == "step":
        ctx.spsa_step(s["theta"], s["seeds"], s["step"], EPS, LR, s["bytes"], s["losses"])
        out = {"losses": s["losses"], "theta": s["theta"]}
    else:
        if call == "adam":
            ctx.spsa_step_adam(s["theta"], s["m"], s["v"], s["t"], s["adam"], s["seeds"], s["step"], EPS, LR,
                               s["bytes"], s["losses"])
        else:
            ctx.spsa_step_adam_sched(s["theta"], s["m"], s["v"], s["t"], s["adam"], s["seeds"], s["step"],
                                     s["sched"], s["bytes"], s["losses"])
        out = {"losses": s["losses"], "theta": s["theta"], "m": s["m"], "v": s["v"]}
    s["step"] += 1
    s["t"] += 1
    return out


def tolerance(case):
    # About four times the largest error against ``exact`` over the ranges:
    # losses 3e-8 (their fp32 rounding) to 3e-7 (few tokens, the wide body);
    # the delta rule's gradient 3e-6.  An update divides the losses' errors by
    # 2 eps P: up to 2e-7 of the weights under the plain step, 2e-5 of Adam's
    # first moment.
    if case["call"] == "delta":
        return {"rel": 1.2e-5, "max": 5e-4}
    if case["call"] in ("eval", "step"):
        return {"rel": 1e-6, "max": 4e-5}
    return {"rel": 1e-4, "max": 4e-3}


# --------------------------------------------------------------------------
# The same results in 64 bits, from the definitions

def _philox(c0, c1, c2, c3, k0, k1):
    """Philox4x32-10 on int64 tensors (or ints) holding 32-bit words."""
    mask = 0xFFFFFFFF
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = ((p1 >> 32) & mask) ^ c1 ^ k0, p1 & mask, ((p0 >> 32) & mask) ^ c3 ^ k1, p0 & mask
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return c0, c1, c2, c3


def _probes(c, dev, seed, step, first, count):
    """z of directions first .. first + count - 1, [count, d] float64 (rounded to the fp32 values that define it)."""
    d = _params(c)
    per = 4 if c["probe"] == "gaussian" else 64
    q = torch.arange((d + per - 1) // per, device=dev, dtype=torch.int64).expand(count, -1)
    zero = torch.zeros_like(q)
    j = torch.arange(first, first + count, device=dev, dtype=torch.int64)[:, None]
    w = torch.stack(_philox(q, zero + j, zero + (step & 0xFFFFFFFF), zero, seed & 0xFFFFFFFF,
                            (seed >> 32) ^ (step >> 32)), dim=2)
    if c["probe"] == "gaussian":
        u1 = ((w[..., 0::2] >> 8) + 1).double() * 2.0 ** -24
        u2 = (w[..., 1::2] >> 8).double() * 2.0 ** -24
        r, a = (-2.0 * u1.log()).sqrt(), 2.0 * math.pi * u2
        z = torch.stack((r * a.cos(), r * a.sin()), dim=3).reshape(count, -1)[:, :d]
        return z.float().double()
    f = ((w[..., None] >> torch.arange(0, 32, 2, device=dev)) & 3).reshape(count, -1)[:, :d]
    z = 1.0 - 2.0 * (f & 1).double()
    if c["probe"] == "dense":
        return z
    return torch.where((f >= 2) | _gain_coordinates(c, dev), z, torch.zeros_like(z))


def _gain_coordinates(c, dev):
    """The normalisation gains, whose sparse probes are dense."""
    d, H, L = _params(c), c["hidden"], c["layers"]
    g = torch.zeros(d, dtype=torch.bool, device=dev)
    if c["arch"] == "body":
        blk = 16 * H * H + 2 * H
        for l in range(L):
            g[l * blk:l * blk + H] = True
            g[l * blk + H + 8 * H * H:l * blk + 2 * H + 8 * H * H] = True
        g[L * blk:] = True
    elif c["arch"] == "wide":
        g[d - (2 * L + 1) * H:] = True
    return g


def _perturbed(c, dev):
    """1 where a coordinate belongs to a perturbed group, else 0."""
    on = torch.ones(_params(c), dtype=torch.float64, device=dev)
    if c["mask"]:
        emb, head = VOCAB * c["embed"], VOCAB * c["hidden"]
        for bit, part in ((soma.PERTURB_EMBEDDING, on[:emb]), (soma.PERTURB_LSTM, on[emb:-head]),
                          (soma.PERTURB_HEAD, on[-head:])):
            if not c["mask"] & bit:
                part.zero_()
    return on


def _lstm(gin, wh):
    """h [S, T, B, H] from gate inputs [S, T, B, 4H] and recurrent weights [S, 4H, H] (gates i, f, g, o)."""
    S, T, B, H4 = gin.shape
    H = H4 // 4
    wt = wh.transpose(1, 2).contiguous()
    out = torch.empty((S, T, B, H), dtype=gin.dtype, device=gin.device)
    h = cell = None
    for t in range(T):
        a = gin[:, t] if h is None else torch.baddbmm(gin[:, t], h, wt)
        i, f, o = a[..., :H].sigmoid(), a[..., H:2 * H].sigmoid(), a[..., 3 * H:].sigmoid()
        new = i * a[..., 2 * H:3 * H].tanh()
        cell = new if cell is None else f * cell + new
        h = o * cell.tanh()
        out[:, t] = h
    return out


def _mul(x, w):
    """x [S, T, B, K] times w [S, O, K] transposed."""
    S, T, B, K = x.shape
    return torch.bmm(x.reshape(S, T * B, K), w.transpose(1, 2).contiguous()).view(S, T, B, -1)


def _norm(x, g):
    m = x.mean(-1, keepdim=True)
    v = (x - m).square().mean(-1, keepdim=True)
    return (x - m) / (v + 1e-5).sqrt() * g[:, None, None, :]


def _decoder_inputs(c, w, x, E):
    """(decoder inputs [S, T-1, B, width], decoder [S, 256, width]) of S weight vectors w [S, d] on bytes x [S, B, T]."""
    S, L, H, W = w.shape[0], c["layers"], c["hidden"], c["embed"]
    at = [0]

    def take(*shape):
        n = math.prod(shape)
        at[0] += n
        return w[:, at[0] - n:at[0]].view(S, *shape)

    seq = x[:, :, :-1].transpose(1, 2).long()                       # [S, T-1, B]

    def rows(table):                                                # table[s][byte]
        flat = seq.reshape(S, -1, 1).expand(-1, -1, table.shape[2])
        return table.gather(1, flat).view(*seq.shape, table.shape[2])

    if c["arch"] == "lstm":
        emb = take(VOCAB, W)
        h = None
        for l in range(L):
            k = W if l == 0 else H
            m = take(4 * H, k + H)
            wx, wh = m[:, :, :k], m[:, :, k:]
            gin = rows(torch.bmm(emb, wx.transpose(1, 2).contiguous())) if l == 0 else _mul(h, wx)
            h = _lstm(gin, wh)
        return h, take(VOCAB, H)
    if c["arch"] == "body":
        v = rows(E)
        for l in range(L):
            g1, m, g2, w1, w2 = take(H), take(4 * H, 2 * H), take(H), take(4 * H, H), take(H, 4 * H)
            v = v + _lstm(_mul(_norm(v, g1), m[:, :, :H]), m[:, :, H:])
            v = v + _mul(torch.nn.functional.gelu(_mul(_norm(v, g2), w1)), w2)
        return _norm(v, take(H)), E
    pin = take(H, W)
    mats = [[take(H, 4 * H) for _ in range(4)] for _ in range(L)]
    pout = take(H, W)
    gain = [(take(H), take(H)) for _ in range(L)]
    v = rows(torch.bmm(E, pin.transpose(1, 2).contiguous()))
    for (A, R, U, V), (g1, g2) in zip(mats, gain):
        v = v + _lstm(_mul(_norm(v, g1), A.transpose(1, 2)), R.transpose(1, 2))
        v = v + _mul(torch.nn.functional.gelu(_mul(_norm(v, g2), U.transpose(1, 2))), V)
    return _mul(_norm(v, take(H)), pout.transpose(1, 2)), E


def _mean_losses(c, w, x, E):
    """Mean cross entropy of each of S weight vectors on its batch."""
    f, D = _decoder_inputs(c, w, x, E)
    y = x[:, :, 1:].transpose(1, 2).long()
    total = torch.zeros(w.shape[0], dtype=torch.float64, device=w.device)
    for t in range(0, f.shape[1], 64):
        lg = _mul(f[:, t:t + 64], D)
        total += (lg.logsumexp(-1) - lg.gather(-1, y[:, t:t + 64, :, None])[..., 0]).sum((1, 2))
    return total / (y.shape[1] * y.shape[2])


def exact(case, seed):
    c = case
    x = _inputs(c, seed)
    dev, N, D = x["theta"].device, c["experts"], _directions(c)
    theta = x["theta"].double()
    E = x["E"].double().expand(N, -1, -1) if "E" in x else None
    if c["call"] in ("eval", "delta"):
        data = x["bytes"][0]
        if c["call"] == "eval":
            return {"loss": _mean_losses(c, theta, data, E)}
        loss, grad = torch.zeros(N, dtype=torch.float64, device=dev), torch.zeros_like(E)
        for e in range(N):
            f, Ee = _decoder_inputs(c, theta[e:e + 1], data[e:e + 1], E[e:e + 1])
            y = data[e:e + 1, :, 1:].transpose(1, 2).long()
            lg = _mul(f, Ee)
            lse = lg.logsumexp(-1, keepdim=True)
            loss[e] = (lse - lg.gather(-1, y[..., None])).mean()
            p = (lg - lse).exp()
            p.scatter_add_(-1, y[..., None], torch.full_like(lse, -1.0))
            n = y.numel()
            grad[e] = p.reshape(n, VOCAB).t().contiguous() @ f.reshape(n, -1) / n
        return {"loss": loss, "grad": grad, "E": E - _f32(LR) * grad}

    eps, lr = _f32(EPS), _f32(LR)
    on = _perturbed(c, dev)
    seeds = x["seeds"].tolist()
    pairs = [(e, j) for e in range(N) for j in range(D)]
    rows, H, d = c["batch"] * (c["seq_len"] - 1), c["hidden"], _params(c)
    at_once = max(1, (1 << 25) // d)                                # directions drawn at a time
    chunk = max(1, int(40e9 / (16 * (4 * d + rows * (12 * H + 64)) + 16 * c["batch"] * 64 * 3 * VOCAB)))
    losses = torch.zeros((len(pairs), 2), dtype=torch.float64, device=dev)
    for a in range(0, len(pairs), chunk):
        part = pairs[a:a + chunk]
        w = torch.empty((len(part), 2, d), dtype=torch.float64, device=dev)
        i = 0
        while i < len(part):
            e, j = part[i]
            n = sum(1 for k in range(i, min(len(part), i + at_once)) if part[k][0] == e)
            z = eps * _probes(c, dev, seeds[e], FIRST_STEP, j, n) * on
            # a perturbed weight is one fp32 rounding of theta +- eps z
            w[i:i + n, 0], w[i:i + n, 1] = (theta[e] + z).float(), (theta[e] - z).float()
            i += n
        batch = torch.stack([x["bytes"][j // c["pairs"], e] for e, j in part]).repeat_interleave(2, 0)
        tied = torch.stack([E[e] for e, _ in part]).repeat_interleave(2, 0) if E is not None else None
        losses[a:a + chunk] = _mean_losses(c, w.view(-1, d), batch, tied).view(-1, 2)
    losses = losses.view(N, D, 2)
    diff = losses[:, :, 0] - losses[:, :, 1]
    if c["loss"] == "summed":
        diff = diff.sum(0, keepdim=True).expand(N, D)
    coef = diff / (2.0 * eps * D)
    est = torch.zeros_like(theta)
    for e in range(N):
        for j in range(0, D, at_once):
            n = min(at_once, D - j)
            est[e] += (coef[e, j:j + n, None] * _probes(c, dev, seeds[e], FIRST_STEP, j, n)).sum(0)
    if c["call"] == "step":
        return {"losses": losses, "theta": theta - lr * est * on}
    b1, b2, delta, decay = (_f32(v) for v in (0.9, 0.999, 1e-8, 1e-4))
    g = est + decay * theta
    m0, v0 = x["m"].double(), x["v"].double()
    m, v = b1 * m0 + (1.0 - b1) * g, b2 * v0 + (1.0 - b2) * g * g
    new = theta - lr * (m / (1.0 - b1 ** FIRST_UPDATE)) / ((v / (1.0 - b2 ** FIRST_UPDATE)).sqrt() + delta)
    keep = on > 0
    return {"losses": losses, "theta": torch.where(keep, new, theta), "m": torch.where(keep, m, m0),
            "v": torch.where(keep, v, v0)}


def _f32(v):
    return float(torch.tensor(v, dtype=torch.float32))
