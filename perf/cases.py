"""The work a user of this library has it do, as timed cases.

Three kinds of pass, each through the public entry points of
paper_2609_33385_amd.oled:

 layer   one MoE layer of one denoising iteration: route_block (or
         route_block_gate, the gate GEMM in front), moe_forward_cached,
         apply_misses, score_and_retain; returns the layer's output. The cache
         is as a running program has it: every expert resident, or warmed by
         the iteration before and missing the rest from the pinned host pool.
 block   every layer of a stack over all denoising iterations of one block of
         tokens, under partial residency; returns every layer's output.
 replay  routing and permutation of recorded logits without a context:
         oled_route_batch and the priority sums over many blocks, or
         oled_route_noalloc on one block; returns every array they write.

Inputs follow the statistics of the synthetic workloads of this repository:
router logits 3 z[sequence] + n[token] with a random walk over the iterations,
activations and weights N(0, 0.02^2), confidence by an unmasking schedule.
"""
import concurrent.futures
import math

import numpy as np
import torch

from paper_2609_33385_amd import oled

HOST_BLOCKS = 29   # distinct expert blocks in the pinned pool; experts beyond share them


def _layer(name, **kw):
    c = dict(name=name, kind="layer", dtype="bf16", tokens=32, seq=32, experts=64, top_k=8,
             hidden=2048, inter=1024, capacity=64, gate=False, zipf=0.0, report=False)
    c.update(kw)
    return c


def listed():
    return [
        # one decode-sized block routed without a context (graph capture,
        # serving loops that forbid allocation): the smallest call
        dict(name="route_one_block", kind="replay", batch=0, tokens=32, experts=64, top_k=8),
        # recorded routing of 16 layers of an odd-sized request, replayed for a
        # policy study
        dict(name="replay_16x257", kind="replay", batch=16, tokens=257, experts=64, top_k=8),
        # the same of 32 long traces (the largest block the priority sums
        # allow): 1 GiB of logits
        dict(name="replay_32x65535", kind="replay", batch=32, tokens=65535, experts=128, top_k=8),
        # the small fp32 layer, half its experts cached, with the miss report
        _layer("layer_f32_32", dtype="f32", experts=8, top_k=2, hidden=256, inter=512, capacity=4,
               report=True),
        # a decode-sized block of one request: few rows per expert, every
        # launch short
        _layer("layer_32"),
        # a batch of 8 requests, the gate GEMM in front of the routing
        _layer("layer_gate_256", tokens=256, gate=True),
        # many small experts, few rows each
        _layer("layer_e256_512", tokens=512, experts=256, inter=512, capacity=256),
        # an odd-sized prompt: ragged rows per expert between the decode and
        # the prefill shapes
        _layer("layer_3001", tokens=3001, seq=64),
        # the benchmark's layer, batch 16 x block 64, popular experts, all cached
        _layer("layer_e128_1024", tokens=1024, seq=64, experts=128, hidden=4096, inter=1536,
               capacity=128, zipf=1.1),
        # the same under its 40% cache: misses cross the host link
        _layer("layer_e128_1024_cache40", tokens=1024, seq=64, experts=128, hidden=4096,
               inter=1536, capacity=51, zipf=1.1),
        # prefill: compute-bound
        _layer("prefill_e128_16384", tokens=16384, seq=64, experts=128, hidden=4096, inter=1536,
               capacity=128),
        # one denoising block of one request through the 16-layer stack, 40%
        # of the experts cached
        dict(name="block_16x8_cache40", kind="block", dtype="bf16", tokens=32, seq=32, experts=64,
             top_k=8, hidden=2048, inter=1024, capacity=26, layers=16, iters=8, zipf=0.0,
             policy="priority", adapt=0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    u = rng.random()
    if u < 0.1:
        e = rng.choice([8, 60, 64, 96, 128, 256])
        return dict(kind="replay", batch=0, tokens=_log_int(rng, 1, 8192), experts=e,
                    top_k=min(e, rng.choice([1, 2, 6, 8])))
    if u < 0.35:
        e = rng.choice([32, 60, 64, 96, 128, 160, 256])
        k = rng.choice([2, 4, 6, 8, 8])
        b = _log_int(rng, 2, 48)
        return dict(kind="replay", batch=b, experts=e, top_k=k,
                    tokens=_log_int(rng, 33, min(65535, (1 << 28) // (b * e))))
    if u < 0.45:
        e = rng.choice([32, 64, 128])
        return dict(kind="block", dtype="bf16", tokens=_log_int(rng, 8, 96), seq=32, experts=e,
                    top_k=rng.choice([4, 8]), hidden=128 * rng.randint(4, 16),
                    inter=128 * rng.randint(4, 8), capacity=int(e * rng.uniform(0.2, 0.6)),
                    layers=rng.randint(2, 8), iters=rng.randint(2, 8), zipf=0.0,
                    policy=rng.choice(["priority", "priority", "lru", "lfu"]),
                    adapt=rng.choice([0, 0, 5]))
    f32 = rng.random() < 0.15
    e = rng.choice([8, 16, 32, 60, 64, 64, 128, 128, 160, 256])
    full = rng.random() < 0.85
    hidden = 128 * (rng.randint(2, 8) if f32 else rng.randint(4, 32))
    inter = 128 * (rng.randint(2, 6) if f32 else rng.randint(2, 12))
    tokens = _log_int(rng, 1, 512 if f32 else 12000)
    gate = tokens <= 2048 and rng.random() < 0.4
    return dict(kind="layer", dtype="f32" if f32 else "bf16", tokens=tokens,
                seq=rng.choice([32, 64]), experts=e, top_k=min(e, rng.choice([1, 2, 4, 6, 8, 8, 8])),
                hidden=hidden, inter=inter, capacity=e if full else int(e * rng.uniform(0.3, 0.7)),
                gate=gate, zipf=rng.choice([0.0, 1.1]), report=rng.random() < 0.2)


# ------------------------------------------------------------------ inputs
def _gen(seed, part, device="cuda"):
    g = torch.Generator(device=device)
    g.manual_seed(seed * 1009 + part)
    return g


def _logits(case, g, batch, iters, device="cuda"):
    """[batch][iters][T][E] fp32: 3 z[sequence] + n[token] (+ Zipf popularity),
    each later iteration a N(0, 0.3^2) step from the one before."""
    T, E, seq = case["tokens"], case["experts"], case.get("seq", 64)
    out = torch.empty((batch, iters, T, E), device=device)
    for b in range(batch):
        z = torch.randn((-(-T // seq), E), generator=g, device=device).repeat_interleave(seq, 0)[:T]
        v = 3.0 * z + torch.randn((T, E), generator=g, device=device)
        if case.get("zipf"):
            rank = torch.randperm(E, generator=g, device=device) + 1
            v -= case["zipf"] * torch.log(rank.float())
        for i in range(iters):
            if i:
                v = v + 0.3 * torch.randn((T, E), generator=g, device=device)
            out[b, i] = v
    return out


def _confidence(T, iters, g):
    """[iters][T] fp32 rising to 1 at the iteration a token is unmasked."""
    c0 = 0.5 * torch.rand(T, generator=g, device="cuda")
    u = torch.randint(0, max(1, iters), (T,), generator=g, device="cuda")
    i = torch.arange(iters, device="cuda")[:, None]
    return (c0 + (1 - c0) * ((i + 1) / (u + 1)).clamp(max=1.0)).clamp(0, 1).float()


def _torch_dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _n_blocks(case):
    return min(HOST_BLOCKS, case["experts"] * case.get("layers", 1))


def _weights(case, seed, b):
    """Logical weights of host block b: w13 [2I][H], w2 [H][I], on the GPU."""
    H, I = case["hidden"], case["inter"]
    g = _gen(seed, 100 + b)
    w13 = (0.02 * torch.randn((2 * I, H), generator=g, device="cuda")).to(_torch_dtype(case))
    w2 = (0.02 * torch.randn((H, I), generator=g, device="cuda")).to(_torch_dtype(case))
    return w13, w2


def _host(t):
    t = t.cpu()
    return t.numpy() if t.dtype == torch.float32 else t.view(torch.int16).numpy().view(np.uint16)


def _pool(case, seed):
    H, I = case["hidden"], case["inter"]
    dt = np.float32 if case["dtype"] == "f32" else np.uint16
    pool = oled.PinnedPool(_n_blocks(case), 3 * H * I * np.dtype(dt).itemsize)

    def pack(b, w13, w2):
        oled.oled_pack_expert(case["dtype"], H, I, w13, w2, pool.block(b, dt))

    with concurrent.futures.ThreadPoolExecutor(8) as ex:
        jobs = [ex.submit(pack, b, *map(_host, _weights(case, seed, b)))
                for b in range(pool.n_blocks)]
        for j in jobs:
            j.result()
    return pool


def _context(case, pool, layers=1):
    E = case["experts"]
    return oled.Context(case["hidden"], case["inter"], E, case["top_k"], layers, case["capacity"],
                        case["tokens"], case["dtype"], pool.ptr, pool.n_blocks,
                        np.arange(layers * E, dtype=np.int64) % pool.n_blocks,
                        adapt_period=case.get("adapt", 0), policy=case.get("policy", "priority"))


def _cache_pass(ctx, logits, conf):
    """The routing, transfer and retention of one iteration without the experts."""
    s = torch.cuda.current_stream()
    for l in range(logits.shape[0]):
        ctx.route_block(l, logits[l], logits.shape[1], s)
        ctx.apply_misses(l, report=False)
        ctx.score_and_retain(l, conf, s)


def _layer_inputs(case, seed):
    T, E, H = case["tokens"], case["experts"], case["hidden"]
    g = _gen(seed, 1)
    before, logits = _logits(case, g, 1, 2)[0]
    x = (0.02 * torch.randn((T, H), generator=g, device="cuda")).to(_torch_dtype(case))
    conf = _confidence(T, 4, g)[1]
    w_gate = None
    if case["gate"]:
        w_gate = (150.0 / math.sqrt(H) * torch.randn((E, H), generator=g, device="cuda")).to(x.dtype)
    return before, logits, x, conf, w_gate


def _block_inputs(case, seed):
    L, N, T, H = case["layers"], case["iters"], case["tokens"], case["hidden"]
    g = _gen(seed, 1)
    logits = _logits(case, g, L, N).transpose(0, 1).contiguous()
    x = (0.02 * torch.randn((N, L, T, H), generator=g, device="cuda")).to(_torch_dtype(case))
    return logits, x, _confidence(T, N, g)


def _replay_inputs(case, seed):
    B = max(1, case["batch"])
    g = _gen(seed, 1)
    return _logits(case, g, B, 1)[:, 0], torch.rand((B, case["tokens"]), generator=g, device="cuda")


def prepare(case, seed):
    T, E, k = case["tokens"], case["experts"], case["top_k"]
    if case["kind"] == "replay":
        B = max(1, case["batch"])
        logits, conf = _replay_inputs(case, seed)

        def ints(*shape):
            return torch.empty(shape, dtype=torch.int32, device="cuda")

        out = dict(topk_idx=ints(B, T * k), gates=torch.empty((B, T * k), device="cuda"),
                   counts=ints(B, E), offsets=ints(B, E + 1), perm=ints(B, T * k),
                   inv_perm=ints(B, T * k), nonfinite=ints(B))
        s = dict(case=case, logits=logits, conf=conf, out=out)
        if case["batch"]:
            out["score_q"] = torch.empty((B, E), dtype=torch.int64, device="cuda")
            s["workspace"] = torch.empty(oled.oled_route_batch_workspace(B, T, E),
                                         dtype=torch.uint8, device="cuda")
        return s
    pool = _pool(case, seed)
    if case["kind"] == "block":
        ctx = _context(case, pool, case["layers"])
        logits, x, conf = _block_inputs(case, seed)
        for i in range(case["iters"]):
            _cache_pass(ctx, logits[i], conf[i])
        torch.cuda.synchronize()
        return dict(ctx=ctx, case=case, logits=logits, x=x, conf=conf, y=torch.empty_like(x), pool=pool)
    ctx = _context(case, pool)
    before, logits, x, conf, w_gate = _layer_inputs(case, seed)
    if case["capacity"] >= E:   # every expert resident: dummy requests that touch them all
        n = min(-(-E // k), T)
        want = torch.arange(n, device="cuda")[:, None] * k + torch.arange(k, device="cuda")
        for first in range(0, E, n * k):
            dummy = torch.zeros((n, E), device="cuda").scatter_(1, (first + want) % E, 8.0)
            _cache_pass(ctx, dummy[None], torch.ones(n, device="cuda"))
    elif w_gate is None:        # the iteration before this one
        _cache_pass(ctx, before[None], conf)
    torch.cuda.synchronize()
    return dict(ctx=ctx, case=case, logits=logits, x=x, conf=conf, w_gate=w_gate,
                y=torch.empty_like(x), pool=pool)


# -------------------------------------------------------------------- pass
def _run_layer(ctx, layer, logits, x, w_gate, conf, y, report, s):
    T = x.shape[0]
    if w_gate is None:
        ctx.route_block(layer, logits, T, s)
    else:
        ctx.route_block_gate(layer, x, w_gate, T, s)
    ctx.moe_forward_cached(layer, x, y, s)
    ctx.apply_misses(layer, report=report)
    ctx.score_and_retain(layer, conf, s)


def run(state):
    case = state["case"]
    s = torch.cuda.current_stream()
    if case["kind"] == "layer":
        _run_layer(state["ctx"], 0, state["logits"], state["x"], state["w_gate"], state["conf"],
                   state["y"], case["report"], s)
        return state["y"]
    if case["kind"] == "block":
        ctx, lg, x, y, conf = (state[n] for n in ("ctx", "logits", "x", "y", "conf"))
        for i in range(case["iters"]):
            for l in range(case["layers"]):
                _run_layer(ctx, l, lg[i, l], x[i, l], None, conf[i], y[i, l], False, s)
        return y
    B, T, E, k, o = case["batch"], case["tokens"], case["experts"], case["top_k"], state["out"]
    if B:
        st = oled.oled_route_batch(state["logits"], B, T, E, k, o["topk_idx"], o["gates"],
                                   o["counts"], o["offsets"], o["perm"], o["inv_perm"],
                                   o["nonfinite"], state["workspace"], s)
        st = st or oled.oled_priority_batch(o["topk_idx"], o["gates"], state["conf"], B, T, E, k,
                                            o["score_q"], None, s)
    else:
        st = oled.oled_route_noalloc(state["logits"], T, E, k, o["topk_idx"], o["gates"],
                                     o["counts"], o["offsets"], o["perm"], o["inv_perm"],
                                     o["nonfinite"], s)
    if st:
        raise RuntimeError(f"status {st}: {oled.last_error(None)}")
    return o


# -------------------------------------------------------------- accounting
def _active(case):
    """Experts a pass activates in one layer (a seeded draw of its routing)."""
    T, E, k = case["tokens"], case["experts"], case["top_k"]
    g = _gen(0, 1, "cpu")
    c = dict(case, tokens=min(T, 2048))
    v = torch.randn((c["tokens"], E), generator=g) if case.get("gate") else _logits(c, g, 1, 1, "cpu")[0, 0]
    return int(torch.unique(v.topk(k, dim=1).indices).numel())


def work(case):
    T, E, k = case["tokens"], case["experts"], case["top_k"]
    if case["kind"] == "replay":
        B = max(1, case["batch"])
        n = B * (T * E * 4 + T * k * 16 + (2 * E + 2) * 4)
        if case["batch"]:
            n += B * (T * 4 + E * 8)
        return {"bytes": n, "flops": B * T * k}
    H, I, s = case["hidden"], case["inter"], 4 if case["dtype"] == "f32" else 2
    n = _active(case) * 3 * H * I * s + 2 * T * H * s + T * 4
    f = 6 * T * k * H * I
    if case.get("gate"):
        n, f = n + E * H * s, f + 2 * T * E * H
    else:
        n += T * E * 4
    reps = case["layers"] * case["iters"] if case["kind"] == "block" else 1
    return {"bytes": n * reps, "flops": f * reps}


def tolerance(case):
    if case["kind"] == "replay":   # whole numbers, and gates rounded once from 64 bits
        return {"rel": 1e-7, "max": 1.2e-7, "differ": 0.0}
    # a near tie of two logits of the gate GEMM may rank either way: one
    # token's last expert then differs
    most = 0.5 if case.get("gate") else None
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": most or 4e-5}
    return {"rel": 8e-3, "max": most or 3e-2}


# ------------------------------------------------------------ in 64 bits
def _route64(logits, k):
    """Top-k by (logit desc, id asc) and gates of [..][E] logits, in 64 bits."""
    v, i = torch.sort(logits.double() + 0.0, dim=-1, descending=True, stable=True)
    v, i = v[..., :k], i[..., :k]
    e = torch.exp(v - v[..., :1])
    return i, e / e.sum(-1, keepdim=True)


def _moe64(case, weights, logits, x):
    idx, gates = _route64(logits, case["top_k"])
    y = torch.zeros(x.shape, dtype=torch.float64, device="cuda")
    x = x.double()
    I = case["inter"]
    for e in torch.unique(idx).tolist():
        t, j = torch.nonzero(idx == e, as_tuple=True)
        w13, w2 = weights(e)
        a = x[t] @ w13.double().T
        h = torch.nn.functional.silu(a[:, :I]) * a[:, I:]
        y.index_add_(0, t, gates[t, j][:, None] * (h @ w2.double().T))
    return y


def exact(case, seed):
    T, E, k = case["tokens"], case["experts"], case["top_k"]
    if case["kind"] == "replay":
        logits, conf = _replay_inputs(case, seed)
        out = {n: [] for n in ("topk_idx", "gates", "counts", "offsets", "perm", "inv_perm", "nonfinite")}
        if case["batch"]:
            out["score_q"] = []
        for b in range(logits.shape[0]):
            idx, gates = _route64(logits[b], k)
            idx, gates = idx.reshape(-1), gates.reshape(-1)
            counts = torch.bincount(idx, minlength=E)
            perm = torch.argsort(idx, stable=True)
            inv = torch.empty_like(perm)
            inv[perm] = torch.arange(T * k, device="cuda")
            out["topk_idx"].append(idx)
            out["gates"].append(gates)
            out["counts"].append(counts)
            out["offsets"].append(torch.cat([counts.new_zeros(1), counts.cumsum(0)]))
            out["perm"].append(perm)
            out["inv_perm"].append(inv)
            out["nonfinite"].append(counts.new_zeros(()))
            if case["batch"]:   # of the gates as they are held, in 32 bits
                q = torch.floor(gates.float().double() * conf[b].double().repeat_interleave(k) * 2.0 ** 48)
                out["score_q"].append(torch.zeros(E, dtype=torch.int64, device="cuda")
                                      .index_add_(0, idx, q.to(torch.int64)))
        return {n: torch.stack(v) for n, v in out.items()}
    nb = _n_blocks(case)
    held = [_weights(case, seed, b) for b in range(nb)]
    if case["kind"] == "layer":
        _, logits, x, _, w_gate = _layer_inputs(case, seed)
        if w_gate is not None:
            logits = x.double() @ w_gate.double().T
        return _moe64(case, lambda e: held[e % nb], logits, x)
    logits, x, _ = _block_inputs(case, seed)
    y = torch.empty(x.shape, dtype=torch.float64, device="cuda")
    for i in range(case["iters"]):
        for l in range(case["layers"]):
            y[i, l] = _moe64(case, lambda e: held[(l * E + e) % nb], logits[i, l], x[i, l])
    return y
