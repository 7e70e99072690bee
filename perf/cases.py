"""Performance cases of the token-filter path: what its users call, at the sizes they call it.

A case is one pass through the public entry points of `paper_2512_07090_amd.binding`:

  kind "layer"   tf_filtered_attention: one attention layer over a whole prompt (prefill)
  kind "online"  tf_filtered_attention_online: the same with the feedback threshold
  kind "layers"  tf_filtered_attention_layers: a stack of layers under the tail-focused schedule
  kind "prompt"  tf_decode_prefill over a prompt, then `steps` tokens through tf_decode_step
  kind "decode"  `steps` tokens through tf_decode_step on a cache that already holds `cached` kept
                 tokens per row (0: a new sequence, opened with tf_decode_init)

Inputs follow the recipe of `paper_2512_07090_amd.synth` (prototype plus noise, one token identity
shared by all heads and by Q, K and V), drawn on the GPU because they are drawn many times.
"""
import torch

from paper_2512_07090_amd import binding as B

HEAD_DIM = 128
DEVICE = "cuda:0"
ETA, TAU0 = 0.02, 0.5      # the online threshold's step and start, as in bench.py
MHA_7B, MHA_13B, GQA_8B = (32, 32), (40, 40), (32, 8)   # (query heads, KV heads) of synth.WORKLOADS


def _case(kind, dtype, batch, heads, n, ratio, **more):
    c = {"kind": kind, "dtype": dtype, "batch": batch, "n_q_heads": heads[0], "n_kv_heads": heads[1], "n": n, "ratio": ratio,
         "warmup": 1, "fusion": B.TF_FUSE_EQ2, "gamma": 0.0, "identity": "zipf", "sigma_lo": 0.3, "sigma_hi": 0.3,
         "prototypes": 256, "steps": 0, "cached": 0, "n_layers": 1}
    c.update(more)
    return c


def listed():
    return [
        # a new chat turn: the first tokens of an empty sequence, one at a time (smallest calls)
        dict(_case("decode", "bf16", 1, GQA_8B, 0, 0.5, warmup=8, steps=16), name="decode_gqa_b1_start"),
        # steady decoding of a batch of medium-long sequences
        dict(_case("decode", "bf16", 8, MHA_7B, 0, 0.5, warmup=8, steps=16, cached=2048), name="decode_mha32_b8_c2048"),
        # steady decoding of one long sequence
        dict(_case("decode", "bf16", 1, GQA_8B, 0, 0.5, warmup=8, steps=16, cached=16384, identity="runs", sigma_lo=0.05,
                   sigma_hi=0.05, prototypes=512), name="decode_gqa_b1_c16384"),
        # the fp32 configuration of the benchmark
        dict(_case("layer", "f32", 1, MHA_7B, 512, 0.5, prototypes=64), name="layer_f32_mha32_b1_n512"),
        # one short prompt of no round length
        dict(_case("layer", "bf16", 1, MHA_7B, 333, 0.5), name="layer_mha32_b1_n333"),
        # a small batch of medium prompts, odd sizes, the paper's 25 % and incremental anchor, noisy heads
        dict(_case("layer", "bf16", 2, MHA_13B, 1777, 0.25, gamma=0.9, sigma_lo=0.1, sigma_hi=1.0),
             name="layer_mha40_b2_n1777_ema"),
        # the benchmark's headline workload: a full batch of MHA prompts
        dict(_case("layer", "bf16", 8, MHA_7B, 4096, 0.5), name="layer_mha32_b8_n4096"),
        # grouped-query prompts
        dict(_case("layer", "bf16", 2, GQA_8B, 8192, 0.5, prototypes=512), name="layer_gqa_b2_n8192"),
        # one very long document (the largest case)
        dict(_case("layer", "bf16", 1, GQA_8B, 32768, 0.5, identity="runs", sigma_lo=0.05, sigma_hi=0.05, prototypes=512),
             name="layer_gqa_b1_n32768"),
        # a batch under the feedback threshold: kept counts differ from row to row
        dict(_case("online", "bf16", 8, MHA_7B, 4096, 0.5, warmup=8), name="online_mha32_b8_n4096"),
        # four layers, the last half pruned: dense layers beside filtered ones
        dict(_case("layers", "bf16", 1, GQA_8B, 2048, 0.25, n_layers=4), name="layers_gqa_b1_n2048"),
        # a request: prompt, hand-off to the decoding state, first tokens of the answer
        dict(_case("prompt", "bf16", 1, GQA_8B, 3001, 0.5, warmup=8, steps=8), name="prompt_gqa_b1_n3001"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    kind = rng.choice(("layer", "layer", "layer", "online", "layers", "prompt", "decode", "decode"))
    heads = rng.choice((MHA_7B, MHA_13B, GQA_8B))
    dtype = "f32" if kind in ("layer", "decode") and rng.random() < 0.15 else "bf16"
    noise = rng.choice(((0.3, 0.3), (0.1, 1.0), (0.05, 0.05)))
    more = {"prototypes": rng.choice((64, 256, 512)), "sigma_lo": noise[0], "sigma_hi": noise[1],
            "identity": "runs" if noise[1] == 0.05 else "zipf", "gamma": 0.9 if rng.random() < 0.25 else 0.0,
            "fusion": rng.choice((B.TF_FUSE_EQ2,) * 4 + (B.TF_FUSE_INVVAR, B.TF_FUSE_KEY_ONLY))}
    ratio = rng.choice((0.25, 0.5, round(rng.uniform(0.1, 0.75), 3)))
    limit = max(_cost(c) for c in listed())
    while True:
        batch = rng.choice((1, 1, 2, 3, 4, 8))
        if kind == "decode":
            c = _case(kind, dtype, batch, heads, 0, ratio, warmup=8, steps=16, cached=_log_int(rng, 64, 32768), **more)
            fits = batch * c["cached"] <= 65536
        else:
            n = _log_int(rng, 130, 1500 if dtype == "f32" else 32768 if kind == "layer" else 8192)
            c = _case(kind, dtype, batch, heads, n, ratio, warmup=1 if kind in ("layer", "layers") else 8, **more)
            if kind == "layers":
                c["n_layers"], c["ratio"] = 4, min(ratio, 0.4)
            if kind == "prompt":
                c["steps"] = 8
            fits = batch * n <= (2048 if dtype == "f32" else 65536)
        if fits and _cost(c) <= limit:
            return c


# ------------------------------------------------------------------------------ inputs

def _generator(seed):
    return torch.Generator(device=DEVICE).manual_seed(seed)


def _zipf(shape, p, gen):
    weights = torch.arange(1, p + 1, dtype=torch.float64, device=DEVICE).pow(-1.2)
    cdf = torch.cumsum(weights / weights.sum(), 0)
    return torch.searchsorted(cdf, torch.rand(shape, generator=gen, dtype=torch.float64, device=DEVICE)).clamp_(max=p - 1)


def _identities(case, n, gen):
    """Token identities [batch, n]: independent, or runs of one identity (geometric length, mean 8, at most 64)."""
    b, p = case["batch"], case["prototypes"]
    if case["identity"] == "zipf":
        return _zipf((b, n), p, gen)
    fresh = torch.rand((b, n), generator=gen, device=DEVICE) < 1.0 / 8.0
    fresh[:, ::64] = True
    run = torch.cumsum(fresh.to(torch.int64), 1) - 1
    return torch.gather(_zipf((b, n), p, gen), 1, run)


def _tensor(case, heads, z, gen):
    """[batch, heads, n, 128] in the case's type: prototype of each token's identity plus noise."""
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    protos = torch.randn((heads, case["prototypes"], HEAD_DIM), generator=gen, device=DEVICE)
    sigma = torch.full((heads, 1, 1), case["sigma_lo"], device=DEVICE)
    sigma[heads // 2:] = case["sigma_hi"]
    out = torch.empty((z.shape[0], heads, z.shape[1], HEAD_DIM), dtype=dt, device=DEVICE)
    for b in range(z.shape[0]):
        x = torch.randn((heads, z.shape[1], HEAD_DIM), generator=gen, device=DEVICE)
        out[b] = x.mul_(sigma).add_(protos[:, z[b]]).to(dt)
    return out


def _params(case, q_shape, kv_shape):
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    return B.make_params(q_shape, kv_shape, dt, case["ratio"], case["warmup"], case["fusion"],
                         ema_gamma=case["gamma"] if case["gamma"] > 0 else None)


class _State:
    """What a program holds between calls."""


def _by_step(x):
    """[batch, heads, steps, 128] as one contiguous slice per token."""
    return x.permute(2, 0, 1, 3).contiguous()


def _decode_buffers(p, capacity):
    """DecodeBuffers whose small state (anchors, counters, threshold) is one block, so that a program can roll a
    sequence back to its prompt with one copy."""
    d = B.DecodeBuffers(p, capacity)
    d.k_cache.zero_()
    d.v_cache.zero_()
    names = ("anchor_k", "anchor_v", "seen", "skipped", "tau", "cache_len", "overflow")
    sizes = [(getattr(d, n).numel() * getattr(d, n).element_size() + 255) // 256 * 256 for n in names]
    d.block = torch.zeros(sum(sizes), dtype=torch.uint8, device=DEVICE)
    at = 0
    for n, size in zip(names, sizes):
        old = getattr(d, n)
        new = d.block[at:at + old.numel() * old.element_size()].view(old.dtype).view(old.shape)
        setattr(d, n, new)
        setattr(d.state, n, new.data_ptr())
        at += size
    return d


def _outputs_by_step(case, s):
    b, hq, steps = case["batch"], case["n_q_heads"], case["steps"]
    s.o = torch.zeros((steps, b, hq, HEAD_DIM), dtype=s.qs.dtype, device=DEVICE)
    s.skip = torch.zeros((steps, b), dtype=torch.uint8, device=DEVICE)
    s.step_fused = torch.zeros((steps, b), dtype=torch.float32, device=DEVICE)


def _prepare_decode(case, gen, s):
    """A sequence whose prompt is behind it: anchors over the prompt, the kept rows in the caches, a threshold at which
    the new tokens are skipped about as often as the target asks for."""
    b, steps, cached = case["batch"], case["steps"], case["cached"]
    n0 = int(cached / (1.0 - case["ratio"]))
    z = _identities(case, n0 + steps, gen)
    q = _tensor(case, case["n_q_heads"], z[:, n0:], gen)
    k, v = (_tensor(case, case["n_kv_heads"], z, gen) for _ in range(2))
    s.p = _params(case, tuple(q.shape), (b, case["n_kv_heads"], steps, HEAD_DIM))
    s.d = _decode_buffers(s.p, cached + steps)
    s.qs, s.ks, s.vs = _by_step(q), _by_step(k[:, :, n0:]), _by_step(v[:, :, n0:])
    if cached:
        kept = torch.rand((b, n0), generator=gen, device=DEVICE).argsort(1)[:, :cached].sort(1).values
        sims = []
        for x, anchor, cache in ((k, s.d.anchor_k, s.d.k_cache), (v, s.d.anchor_v, s.d.v_cache)):
            if case["gamma"] > 0:
                last = min(n0, 512)
                w = (1 - case["gamma"]) * case["gamma"] ** torch.arange(last - 1, -1, -1, dtype=torch.float64, device=DEVICE)
                anchor.copy_((x[:, :, n0 - last:n0].double() * w[:, None]).sum(2))
            else:
                for row in range(b):
                    anchor[row] = x[row, :, :n0].double().sum(1)
            for row in range(b):
                cache[row, :, :cached] = x[row][:, kept[row]]
            new = x[:, :, n0:].double()
            sims.append(torch.nn.functional.cosine_similarity(new, anchor[:, :, None], dim=3).mean(1))
        score = sims[0] if case["fusion"] == B.TF_FUSE_KEY_ONLY else (sims[0] + sims[1]) / 2
        s.d.tau.copy_(torch.quantile(score, 1.0 - case["ratio"], dim=1).float())
        s.d.seen.fill_(n0)
        s.d.skipped.fill_(n0 - cached)
        s.d.cache_len.fill_(cached)
        s.start = s.d.block.clone()
    _outputs_by_step(case, s)


def prepare(case, seed):
    """Inputs from the seed, outputs, workspace and handle, as a serving program keeps them."""
    gen = _generator(seed)
    s = _State()
    s.case, s.ctx = case, B.Context(0)
    if case["kind"] == "decode":
        _prepare_decode(case, gen, s)
        return s
    hq, hkv = case["n_q_heads"], case["n_kv_heads"]
    n, steps = case["n"], case["steps"]
    s.layers = []
    for _ in range(case["n_layers"]):
        z = _identities(case, n + steps, gen)
        s.layers.append([_tensor(case, h, z, gen) for h in (hq, hkv, hkv)])
    s.q, s.k, s.v = s.layers[0]
    if case["kind"] == "prompt":
        s.qs, s.ks, s.vs = (_by_step(x[:, :, n:]) for x in (s.q, s.k, s.v))
        s.q, s.k, s.v = (x[:, :, :n].contiguous() for x in (s.q, s.k, s.v))
        s.layers = None
    s.p = _params(case, tuple(s.q.shape), tuple(s.k.shape))
    s.buf = B.Buffers(s.p, DEVICE)
    if case["kind"] in ("online", "prompt"):
        s.kept_idx = torch.empty((case["batch"], n), dtype=torch.int32, device=DEVICE)
        s.count = torch.empty(case["batch"], dtype=torch.int32, device=DEVICE)
    if case["kind"] == "prompt":
        s.d = _decode_buffers(s.p, n + steps)
        _outputs_by_step(case, s)
    if case["kind"] == "layers":
        s.ratios, _ = B.tf_tail_schedule(case["n_layers"], case["ratio"], 0.5)
        s.bufs = []
        for r in s.ratios:
            s.bufs.append(B.Buffers(_params(dict(case, ratio=r), tuple(s.q.shape), tuple(s.k.shape)), DEVICE))
            s.bufs[-1].fused.zero_()          # not written by a layer that filters nothing
        s.q, s.k, s.v = ([layer[i] for layer in s.layers] for i in range(3))
    return s


# ------------------------------------------------------------------------------ one pass

def _steps(s):
    d = s.d
    for t in range(s.case["steps"]):
        s.ctx.tf_decode_step(s.p, ETA, d.state, s.qs[t], s.ks[t], s.vs[t], s.o[t], s.skip[t], s.step_fused[t], d.ws)
    return {"o": s.o, "skip": s.skip, "score": s.step_fused, "anchor_k": d.anchor_k, "anchor_v": d.anchor_v, "seen": d.seen,
            "skipped": d.skipped, "tau": d.tau, "cache_len": d.cache_len, "overflow": d.overflow, "k_cache": d.k_cache,
            "v_cache": d.v_cache}


# The kept positions come back as the mask `keep`: kept_idx lists the mask's ones in ascending order.
def run(s):
    kind, b = s.case["kind"], getattr(s, "buf", None)
    if kind == "layer":
        s.ctx.tf_filtered_attention(s.p, s.q, s.k, s.v, b.keep, b.kept_idx, b.fused, b.tau, b.O, b.ws)
        return {"keep": b.keep, "fused": b.fused, "tau": b.tau, "O": b.O}
    if kind == "online":
        s.ctx.tf_filtered_attention_online(s.p, ETA, TAU0, s.q, s.k, s.v, b.keep, s.kept_idx, s.count, b.fused, b.tau, b.O, b.ws)
        return {"keep": b.keep, "count": s.count, "fused": b.fused, "tau": b.tau, "O": b.O}
    if kind == "layers":
        bs = s.bufs
        s.ctx.tf_filtered_attention_layers(s.p, s.ratios, s.q, s.k, s.v, [x.keep for x in bs], [x.kept_idx for x in bs],
                                           [x.fused for x in bs], [x.tau for x in bs], [x.O for x in bs], b.ws)
        return [{"keep": x.keep, "fused": x.fused, "tau": x.tau, "O": x.O} for x in bs]
    if kind == "prompt":
        s.ctx.tf_decode_prefill(s.p, ETA, TAU0, s.d.state, s.q, s.k, s.v, b.keep, s.kept_idx, s.count, b.fused, b.O, b.ws)
        out = _steps(s)
        out.update({"keep": b.keep, "count": s.count, "fused": b.fused, "O": b.O})
        return out
    if s.case["cached"]:
        s.d.block.copy_(s.start)              # back to the end of the prompt: the next answer to it
    else:
        s.ctx.tf_decode_init(s.p, s.d.state, TAU0)
    return _steps(s)


# ------------------------------------------------------------------------------ what a pass needs

def _layer_work(case, ratio, scored):
    e = 4 if case["dtype"] == "f32" else 2
    b, hq, hkv, n = case["batch"], case["n_q_heads"], case["n_kv_heads"], case["n"]
    m = _kept(n, ratio)
    v_rows = m if case["fusion"] == B.TF_FUSE_KEY_ONLY else n
    row = HEAD_DIM * e
    size = b * (hkv * (n + v_rows) + hq * m + hq * n) * row + b * (n + 4 * m + 4)
    flops = 2.0 * HEAD_DIM * m * (m + 1) * hq * b
    if scored:
        size += 4 * b * n
        flops += 7.0 * b * hkv * n * HEAD_DIM * (1 if case["fusion"] == B.TF_FUSE_KEY_ONLY else 2)
    return size, flops


def _kept(n, ratio):
    """Kept tokens of a row (the online decision keeps about as many)."""
    return n - int(ratio * n + 1e-6)


def _step_work(case, cached, steps):
    e = 4 if case["dtype"] == "f32" else 2
    b, hq, hkv = case["batch"], case["n_q_heads"], case["n_kv_heads"]
    share = 1.0 if case["warmup"] >= steps + cached else 1.0 - case["ratio"]   # tokens that attend
    mean = cached + share * (steps + 1) / 2
    keys = steps * b * share * mean
    size = keys * 2 * hkv * HEAD_DIM * e + steps * b * HEAD_DIM * (2 * hkv * (16 + 2 * e) + 2 * hq * e)
    return size, keys * 4.0 * HEAD_DIM * hq + steps * b * hkv * HEAD_DIM * 14.0


def work(case):
    if case["kind"] == "decode":
        size, flops = _step_work(case, case["cached"], case["steps"])
    elif case["kind"] == "layers":
        tail = case["n_layers"] // 2
        dense, pruned = _layer_work(case, 0.0, False), _layer_work(case, 2 * case["ratio"], True)
        size, flops = (tail * p + (case["n_layers"] - tail) * d for d, p in zip(dense, pruned))
    else:
        size, flops = _layer_work(case, case["ratio"], True)
        if case["kind"] == "prompt":
            kept = _kept(case["n"], case["ratio"])
            e = 4 if case["dtype"] == "f32" else 2
            size += case["batch"] * case["n_kv_heads"] * kept * HEAD_DIM * e * 2     # the caches' rows
            more = _step_work(case, kept, case["steps"])
            size, flops = size + more[0], flops + more[1]
    return {"bytes": float(size), "flops": float(flops)}


def _cost(case):
    w = work(case)
    return max(w["bytes"] / 5e12, w["flops"] / (5e12 if case["dtype"] == "f32" else 5e14))


def tolerance(case):
    # About four times the distance of the attention output from the same attention in 64 bits on the path's own kept set:
    # bf16 (weights and outputs rounded to 8 bits of mantissa) rel 1.8e-3, max 1.9e-2; fp32 rel 2.3e-7, max 5.3e-6.
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 4e-5, "differ": 0.001}
    return {"rel": 8e-3, "max": 8e-2, "differ": 0.001}
