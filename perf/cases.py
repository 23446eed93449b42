"""The workloads this library's speed is measured on.

Each case is one call (prefill attention: two, the cache write and the
attention, as a prefill step makes them) of the Python binding on inputs that
a serving program holds on the GPU: queries and a paged cache, token rows and
weights, packed prompts. ``listed()`` names the fixed cases, ``draw(rng)`` gives
further ones of the same ranges, ragged and odd sizes among them; ``exact``
states the result in float64 with plain torch.

The whole decode layer (``af_layer_step``) is not a case of its own: it routes
on a hidden state that was rounded to bf16 on the way, so a near tie between
two experts can flip with any change of rounding; its parts (attention, the
projection, the MoE block, the two-stream step) are cases.
"""
import math

import numpy as np
import torch

from paper_2608_01891_amd import aflex, synth

DEV = "cuda:0"
# (query heads, KV heads, head size): the tiny layer, Qwen3-32B, Mixtral-8x7B
TINY, QWEN, MIXTRAL = (8, 2, 64), (64, 8, 128), (32, 8, 128)


# ------------------------------------------------------------------ the cases
def _attn(B, heads, median, sigma, lo, hi):
    return {"op": "attn_decode", "B": B, "Hq": heads[0], "Hkv": heads[1], "D": heads[2],
            "median": median, "sigma": sigma, "lo": lo, "hi": hi}


def _swiglu(T, H, I):
    return {"op": "swiglu", "T": T, "H": H, "I": I}


def _moe(op, T, H, I, E, k):
    return {"op": op, "T": T, "H": H, "I": I, "E": E, "k": k}


def listed():
    return [
        # The smallest call: a tiny layer's attention over short contexts; launches and host work are all of it.
        dict(_attn(4, TINY, 80, 0.7, 17, 200), name="attn_tiny"),
        # The ordinary decode step of a dense model: 64 sequences of mixed length.
        dict(_attn(64, QWEN, 1024, 0.8, 64, 8192), name="attn_qwen_b64"),
        # A few users with long conversations: few (sequence, head) pairs, long contexts.
        dict(_attn(3, QWEN, 12000, 0.7, 256, 32768), name="attn_few_long"),
        # The attention output projection of a decode batch.
        {"op": "linear", "T": 64, "K": 8192, "N": 5120, "name": "o_proj_t64"},
        # The dense FFN of a small decode batch (weights streamed) ...
        dict(_swiglu(32, 5120, 25600), name="swiglu_t32"),
        # ... of a large one (between weight streaming and matrix cores) ...
        dict(_swiglu(384, 5120, 25600), name="swiglu_t384"),
        # ... and of a prefill batch (matrix cores).
        dict(_swiglu(4096, 5120, 25600), name="swiglu_t4096"),
        # Many small experts, a handful of tokens: routing and launches weigh most.
        dict(_moe("moe", 24, 2048, 1024, 64, 8), name="moe_e64_t24"),
        # The MoE model's FFN block (norm, router, experts, residual) on a decode batch ...
        dict(_moe("moe_block", 256, 4096, 14336, 8, 2), name="moe_block_t256"),
        # ... and its experts on a prefill chunk.
        dict(_moe("moe", 2048, 4096, 14336, 8, 2), name="moe_t2048"),
        # Prefill of a mixed batch of prompts, ragged lengths: cache write and causal attention.
        {"op": "prefill", "Hq": 64, "Hkv": 8, "D": 128, "lens": "4096,1733,128,611,2950", "name": "prefill_mixed"},
        # One interleaved attention/FFN layer step of the MoE model: 256 sequences, long contexts, four microbatches.
        {"op": "pipeline", "B": 256, "M": 4, "median": 4096, "sigma": 0.7, "lo": 256, "hi": 32768,
         "name": "pipeline_b256_m4"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _dim(rng, lo, hi):
    """A multiple of 64 (what the GEMMs take), over the logarithm of the range."""
    return 64 * _log(rng, lo // 64, hi // 64)


def draw(rng):
    """Another case of the same ranges: every operator, its sizes over their whole range."""
    op = rng.choice(["attn_decode", "attn_decode", "linear", "swiglu", "swiglu", "moe", "moe", "moe_block",
                     "prefill", "pipeline"])
    if op == "attn_decode":
        heads = rng.choice([TINY, QWEN, QWEN, MIXTRAL, (28, 4, 128), (16, 16, 64)])
        B = _log(rng, 1, 256)
        hi = 32768 if B <= 64 else 8192
        median = _log(rng, 48, hi // 4)
        return _attn(B, heads, median, round(rng.uniform(0.0, 0.8), 2), min(17, median), hi)
    if op == "linear":
        K, N = rng.choice([(8192, 5120), (4096, 4096), (5120, 5120), (_dim(rng, 512, 8192), _dim(rng, 512, 8192))])
        return {"op": "linear", "T": _log(rng, 1, 4096), "K": K, "N": N}
    if op == "swiglu":
        H, I = rng.choice([(5120, 25600), (512, 1408), (4096, 14336), (_dim(rng, 512, 5120), _dim(rng, 1408, 25600))])
        return _swiglu(_log(rng, 1, 4096), H, I)
    if op in ("moe", "moe_block"):
        H, I, E, k = rng.choice([(4096, 14336, 8, 2), (2048, 1024, 64, 8), (4096, 14336, 8, 2),
                                 (_dim(rng, 512, 4096), _dim(rng, 512, 4096), rng.randint(2, 64), rng.choice([1, 2, 4]))])
        return _moe(op, _log(rng, 1, 2048), H, I, E, min(k, E))
    if op == "prefill":
        heads = rng.choice([QWEN, MIXTRAL, (24, 8, 128)])
        left, lens = 8192, []
        while left > 0 and len(lens) < 32:
            n = min(left, _log(rng, 16, 4096))
            lens.append(n)
            left -= n
            if rng.random() < 0.15:
                break
        return {"op": "prefill", "Hq": heads[0], "Hkv": heads[1], "D": heads[2], "lens": ",".join(map(str, lens))}
    B = _log(rng, 4, 256)
    return {"op": "pipeline", "B": B, "M": rng.choice([1, 2, 3, 4]), "median": _log(rng, 64, 4096),
            "sigma": round(rng.uniform(0.0, 0.7), 2), "lo": 16, "hi": 32768}


# ----------------------------------------------------------- sizes from a case
def _ctx(case, seed):
    """Context lengths (lognormal, clipped) of a batch that decodes."""
    rng = np.random.default_rng([seed, 1])
    return synth.lognormal_contexts(rng, case["B"], case["median"], case["sigma"], case["lo"], case["hi"])


def _mean_ctx(case):
    """Mean of the clipped lognormal, so that work() needs no seed."""
    u = (np.arange(2000) + 0.5) / 2000
    z = math.sqrt(2) * torch.erfinv(torch.from_numpy(2 * u - 1)).numpy()
    return float(np.clip(case["median"] * np.exp(case["sigma"] * z), case["lo"], case["hi"]).mean())


def _touched(T, E, k):
    """Experts that at least one of T tokens is expected to choose."""
    return E * (1.0 - (1.0 - k / E) ** T)


def _lens(case):
    return [int(n) for n in case["lens"].split(",")]


def _microbatches(case):
    M, B = min(case["M"], case["B"]), case["B"]
    return [B // M + (1 if i < B % M else 0) for i in range(M)]


# --------------------------------------------------------------------- inputs
class _Draws:
    """Seeded normal draws on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed))

    def __call__(self, *shape, scale=1.0, dtype=torch.bfloat16):
        out = torch.empty(*shape, dtype=dtype, device=DEV)
        return out.normal_(0.0, scale, generator=self.g)


def _attn_inputs(case, seed, rnd, heads):
    Hq, Hkv, D = heads
    ctx = _ctx(case, seed)
    max_blocks = -(-case["hi"] // 16)
    table, n = synth.paged_block_table(np.random.default_rng([seed, 2]), ctx, max_blocks)
    return synth.AttnInputs(
        q=rnd(case["B"], Hq, D), k_cache=rnd(n, Hkv, 16, D), v_cache=rnd(n, Hkv, D, 16),
        block_table=torch.from_numpy(table).to(DEV), context_lens=torch.from_numpy(ctx).to(DEV),
        B=case["B"], Hq=Hq, Hkv=Hkv, D=D, block_size=16, max_blocks=max_blocks, num_blocks=n,
        max_context_len=max_blocks * 16)


def _weights(rnd, H, I, E=0):
    lead = (E,) if E else ()
    s = synth.WEIGHT_SIGMA
    return synth.FFNWeights(w_gate=rnd(*lead, I, H, scale=s), w_up=rnd(*lead, I, H, scale=s),
                            w_down=rnd(*lead, H, I, scale=s), H=H, I=I, E=E)


def prepare(case, seed):
    rnd, op = _Draws(seed), case["op"]
    s = {"case": case}
    if op == "attn_decode":
        s["a"] = _attn_inputs(case, seed, rnd, (case["Hq"], case["Hkv"], case["D"]))
        s["out"] = torch.empty(case["B"], case["Hq"], case["D"], dtype=torch.bfloat16, device=DEV)
    elif op == "linear":
        s["x"], s["w"] = rnd(case["T"], case["K"]), rnd(case["N"], case["K"], scale=synth.WEIGHT_SIGMA)
        s["y"] = torch.empty(case["T"], case["N"], dtype=torch.bfloat16, device=DEV)
    elif op in ("swiglu", "moe", "moe_block"):
        T, H = case["T"], case["H"]
        s["x"], s["w"] = rnd(T, H), _weights(rnd, H, case["I"], case.get("E", 0))
        s["y"] = torch.empty(T, H, dtype=torch.bfloat16, device=DEV)
        if op == "moe":
            s["logits"] = rnd(T, case["E"], dtype=torch.float32)
        elif op == "moe_block":
            s["norm"] = (1.0 + rnd(H, scale=0.1, dtype=torch.float32)).to(torch.bfloat16)
            s["router"] = rnd(case["E"], H, scale=synth.WEIGHT_SIGMA)
    elif op == "prefill":
        lens, (Hq, Hkv, D) = _lens(case), (case["Hq"], case["Hkv"], case["D"])
        T = sum(lens)
        cu = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).to(DEV)
        s["p"] = synth.PrefillInputs(q=rnd(T, Hq, D), k=rnd(T, Hkv, D), v=rnd(T, Hkv, D), cu_seqlens=cu, lens=lens,
                                     Hq=Hq, Hkv=Hkv, D=D)
        hi = -(-max(lens) // 16)
        ctx = np.asarray(lens, dtype=np.int32)
        table, n = synth.paged_block_table(np.random.default_rng([seed, 2]), ctx, hi)
        s["cache"] = synth.AttnInputs(
            q=None, k_cache=torch.zeros(n, Hkv, 16, D, dtype=torch.bfloat16, device=DEV),
            v_cache=torch.zeros(n, Hkv, D, 16, dtype=torch.bfloat16, device=DEV),
            block_table=torch.from_numpy(table).to(DEV), context_lens=torch.from_numpy(ctx).to(DEV), B=len(lens),
            Hq=Hq, Hkv=Hkv, D=D, block_size=16, max_blocks=hi, num_blocks=n, max_context_len=hi * 16)
        s["out"] = torch.empty(T, Hq, D, dtype=torch.bfloat16, device=DEV)
    else:
        H, E = MIXTRAL[0] * MIXTRAL[2], 8
        s["a"] = _attn_inputs(case, seed, rnd, MIXTRAL)
        s["w"] = _weights(rnd, H, 14336, E)
        s["logits"] = rnd(case["B"], E, dtype=torch.float32)
        s["y"] = torch.empty(case["B"], H, dtype=torch.bfloat16, device=DEV)
    return s


# ----------------------------------------------------------------------- run
def run(s):
    case = s["case"]
    op = case["op"]
    if op == "attn_decode":
        return aflex.attn_decode(s["a"], out=s["out"])
    if op == "linear":
        return aflex.linear(s["x"], s["w"], y=s["y"])
    if op == "swiglu":
        return aflex.ffn_swiglu(s["x"], s["w"], y=s["y"])
    if op == "moe":
        return aflex.moe_ffn(s["x"], s["w"], s["logits"], case["k"], y=s["y"])
    if op == "moe_block":
        return aflex.moe_block(s["x"], s["w"], s["norm"], s["router"], case["k"], residual=True, y=s["y"])
    if op == "prefill":
        p, cache = s["p"], s["cache"]
        aflex.kv_write(cache, p.k, p.v, p.cu_seqlens, max_seqlen=p.max_seqlen)
        return {"out": aflex.attn_prefill(p, out=s["out"]), "k_cache": cache.k_cache, "v_cache": cache.v_cache}
    return aflex.af_pipeline_step(s["a"], s["w"], s["logits"], 2, _microbatches(case), y=s["y"])


# ----------------------------------------------------------------------- work
def work(case):
    op = case["op"]
    if op == "attn_decode":
        Hq, Hkv, D, n = case["Hq"], case["Hkv"], case["D"], case["B"] * _mean_ctx(case)
        return {"bytes": n * Hkv * D * 4 + 2 * case["B"] * Hq * D * 2 + n / 4, "flops": 4 * n * Hq * D}
    if op == "linear":
        T, K, N = case["T"], case["K"], case["N"]
        return {"bytes": 2 * (T * K + N * K + T * N), "flops": 2 * T * K * N}
    if op == "swiglu":
        T, H, I = case["T"], case["H"], case["I"]
        return {"bytes": 2 * (2 * T * H + 3 * H * I), "flops": 6 * T * H * I}
    if op in ("moe", "moe_block"):
        T, H, I, E, k = case["T"], case["H"], case["I"], case["E"], case["k"]
        more = 2 * H + 2 * E * H if op == "moe_block" else 4 * T * E
        return {"bytes": 2 * (2 * T * H + 3 * H * I * _touched(T, E, k)) + more,
                "flops": 6 * T * k * H * I + (2 * T * E * H if op == "moe_block" else 0)}
    if op == "prefill":
        lens, Hq, Hkv, D = _lens(case), case["Hq"], case["Hkv"], case["D"]
        return {"bytes": 2 * sum(lens) * D * (2 * Hq + 4 * Hkv),
                "flops": sum(2 * n * (n + 1) for n in lens) * Hq * D}
    (Hq, Hkv, D), B, I, E = MIXTRAL, case["B"], 14336, 8
    n, H = B * _mean_ctx(case), MIXTRAL[0] * MIXTRAL[2]
    # each microbatch is a call of the FFN of its own and reads the experts it touches
    experts = sum(_touched(t, E, 2) for t in _microbatches(case))
    return {"bytes": n * Hkv * D * 4 + 2 * B * H * 2 + 2 * 3 * H * I * experts + 4 * B * E + n / 4,
            "flops": 4 * n * Hq * D + 6 * B * 2 * H * I}


def tolerance(case):
    # bf16 results with fp32 sums and bf16 intermediates (softmax weights, the
    # FFN's hidden rows): another correct implementation rounds those elsewhere.
    # Measured against exact(): 0.0017 (one product) to 0.0038 (attention into
    # the experts); the limit is about four times the middle of that.
    return {"rel": 0.01, "max": 0.08}


# ---------------------------------------------------------------------- exact
def _attn64(a, q):
    out = torch.zeros(a.B, a.Hq, a.D, dtype=torch.float64, device=DEV)
    G = a.Hq // a.Hkv
    for b in range(a.B):
        n = int(a.context_lens[b])
        if n == 0:
            continue
        ids = a.block_table[b, : -(-n // 16)].long()
        k = a.k_cache[ids].permute(1, 0, 2, 3).reshape(a.Hkv, -1, a.D)[:, :n].double()
        v = a.v_cache[ids].permute(1, 0, 3, 2).reshape(a.Hkv, -1, a.D)[:, :n].double()
        w = torch.matmul(q[b].double().view(a.Hkv, G, a.D), k.transpose(1, 2).contiguous()) / math.sqrt(a.D)
        out[b] = torch.matmul(torch.softmax(w, -1), v).reshape(a.Hq, a.D)
    return out


def _swiglu64(x, wg, wu, wd):
    out = torch.zeros(x.shape[0], wd.shape[0], dtype=torch.float64, device=DEV)
    for i in range(0, wg.shape[0], 4096):  # the hidden columns in parts: float64 copies of the weights are large
        g, u = x @ wg[i:i + 4096].double().t(), x @ wu[i:i + 4096].double().t()
        out += (g / (1.0 + torch.exp(-g)) * u) @ wd[:, i:i + 4096].double().t()
    return out


def _moe64(x, logits, w, k):
    top, ids = torch.sort(logits.double(), dim=-1, descending=True, stable=True)
    ids, p = ids[:, :k], torch.softmax(top[:, :k], -1)
    out = torch.zeros(x.shape[0], w.H, dtype=torch.float64, device=DEV)
    for e in range(w.E):
        t, j = torch.nonzero(ids == e, as_tuple=True)
        if t.numel():
            out[t] += p[t, j, None] * _swiglu64(x[t].double(), w.w_gate[e], w.w_up[e], w.w_down[e])
    return out


def exact(case, seed):
    s, op = prepare(case, seed), case["op"]
    if op == "attn_decode":
        return _attn64(s["a"], s["a"].q)
    if op == "linear":
        return s["x"].double() @ s["w"].double().t()
    if op == "swiglu":
        return _swiglu64(s["x"].double(), s["w"].w_gate, s["w"].w_up, s["w"].w_down)
    if op == "moe":
        return _moe64(s["x"], s["logits"], s["w"], case["k"])
    if op == "moe_block":
        x = s["x"].double()
        xn = x / torch.sqrt((x * x).mean(-1, keepdim=True) + 1e-5) * s["norm"].double()
        return x + _moe64(xn, xn @ s["router"].double().t(), s["w"], case["k"])
    if op == "prefill":
        p, c = s["p"], s["cache"]
        out, k_cache, v_cache = torch.empty(p.q.shape, dtype=torch.float64, device=DEV), c.k_cache.double(), c.v_cache.double()
        start, G = 0, p.Hq // p.Hkv
        for b, n in enumerate(p.lens):
            pos = torch.arange(n, device=DEV)
            blk = c.block_table[b].long()[pos // 16]
            k, v = p.k[start:start + n].double(), p.v[start:start + n].double()
            k_cache[blk, :, pos % 16] = k
            v_cache[blk, :, :, pos % 16] = v
            mask = torch.ones(n, n, dtype=torch.bool, device=DEV).triu(1)
            for h in range(p.Hq):
                sc = p.q[start:start + n, h].double() @ k[:, h // G].t() / math.sqrt(p.D)
                out[start:start + n, h] = torch.softmax(sc.masked_fill_(mask, -math.inf), -1) @ v[:, h // G]
            start += n
        return {"out": out, "k_cache": k_cache, "v_cache": v_cache}
    a = s["a"]
    return _moe64(_attn64(a, a.q).view(a.B, a.Hq * a.D), s["logits"], s["w"], 2)
