"""Cases for timing libsage on one GPU, through the public entry points of the Python binding.

A case is a dict of plain values; ``kind`` names the entry point a user's program calls:

* ``fwd``     ``sage_attn_fwd`` on contiguous [B, H, N, d] tensors: K/V quantisation and attention in one call;
* ``packed``  ``sage_attn_fwd_strided`` on token-major slices of a packed QKV projection, grouped query heads, with a
              workspace and an output the program keeps;
* ``fwd4``    ``sage_attn_fwd_4bit``, the 4+8 variant, grouped query heads;
* ``cache``   ``sage_attn_fwd_decode`` on a K/V cache that was quantised once: one query row per head (decode), a few
              (speculative decode) or a chunk of a prompt (chunked prefill), with a kept workspace and output;
* ``quant``   ``sage_quant_kv``, what a program runs once per prompt to make such a cache;
* ``staged``  ``sage_quant_qk`` + ``sage_quant_v`` + ``sage_attn_fwd_quantized``, the stages one by one.

Values: Q, K, V ~ N(0, 1) and K with a per-channel offset ~ N(0, 3) shared by all tokens (what the smoothing of K is
for); ``heavy`` cases draw Q from Student's t with three degrees of freedom and scale four K channels per head by 20.
"""
import math

import torch

import paper_2505_21136_amd as sage

DTYPES = {"fp16": torch.float16, "bf16": torch.bfloat16}


def _case(kind, B, Hq, Hkv, Nq, Nk, d, causal, dtype, heavy=False, name=None):
    c = dict(kind=kind, B=B, Hq=Hq, Hkv=Hkv, Nq=Nq, Nk=Nk, d=d, causal=causal, dtype=dtype, heavy=heavy)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one short sequence with two heads: a handful of workgroups, so launches and latency are all there is
        _case("fwd", 1, 2, 2, 1024, 1024, 128, False, "fp16", name="fwd_small"),
        # prompt of a language model, all heads with their own K and V
        _case("fwd", 4, 32, 32, 4096, 4096, 128, True, "fp16", name="fwd_causal"),
        # image or video transformer at head dimension 64
        _case("fwd", 2, 32, 32, 8192, 8192, 64, False, "bf16", name="fwd_d64"),
        # token count of a video diffusion transformer, no multiple of any tile
        _case("fwd", 1, 48, 48, 17776, 17776, 64, False, "bf16", name="fwd_ragged"),
        # long sequence, heavy-tailed queries and outlier channels in K: the largest call
        _case("fwd", 1, 24, 24, 32768, 32768, 128, False, "bf16", heavy=True, name="fwd_long"),
        # prompt of a grouped-query model straight from its QKV projection, ragged length
        _case("packed", 2, 32, 8, 5003, 5003, 128, True, "bf16", name="packed_gqa"),
        # the 4+8 variant on a grouped-query prompt
        _case("fwd4", 2, 32, 8, 3000, 3000, 128, True, "fp16", name="fwd4_gqa"),
        # one token of a batch of long conversations: streams the cache
        _case("cache", 8, 32, 8, 1, 32768, 128, True, "bf16", name="decode_batch"),
        # one token of two short conversations: launch-bound
        _case("cache", 2, 32, 8, 1, 1500, 128, True, "bf16", name="decode_short"),
        # the next 512 tokens of one long prompt
        _case("cache", 1, 32, 8, 512, 32768, 128, True, "bf16", name="chunked_prefill"),
        # the cache of a long prompt, quantised once
        _case("quant", 1, 8, 8, 50000, 50000, 128, False, "bf16", name="quant_long"),
        # many short ragged sequences through the separate stages
        _case("staged", 16, 16, 16, 777, 777, 64, False, "fp16", name="staged_short"),
    ]


def _log(rng, lo, hi):
    """Whole number, spread over the logarithm of [lo, hi]: any residue, so most are odd sizes for a tile."""
    return min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    kind = rng.choice(["fwd", "fwd", "fwd", "packed", "fwd4", "cache", "cache", "cache", "quant", "staged"])
    d, dtype = rng.choice([64, 128]), rng.choice(["fp16", "bf16"])
    causal, heavy = rng.random() < 0.5, rng.random() < 0.2
    grouped = kind in ("packed", "fwd4", "cache")
    group = rng.choice([1, 2, 4, 8]) if grouped else 1
    while True:
        Hkv, B = _log(rng, 1, 16 if grouped else 48), _log(rng, 1, 16)
        if kind == "cache":
            Nk = _log(rng, 256, 131072)
            Nq = rng.choice([1, 1, 1, _log(rng, 2, 16), _log(rng, 65, 1024)])
            Nq = min(Nq, Nk)
        else:
            Nk = Nq = _log(rng, 256, 65536 if kind == "quant" else 32768)
        c = _case(kind, B, Hkv * group, Hkv, Nq, Nk, d, causal and kind != "quant", dtype, heavy)
        w = work(c)
        # (at most a third of the largest listed case's operations and half of its tensors' size)
        if w["flops"] <= 4.4e12 and B * Hkv * (group * Nq + 2 * Nk) * d <= 1.5e8:
            return c


def _inputs(c, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    B, Hq, Hkv, Nq, Nk, d, dt = (c[x] for x in ("B", "Hq", "Hkv", "Nq", "Nk", "d", "dtype"))
    dt = DTYPES[dt]

    def normal(*shape):
        return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32)

    q = normal(B, Hq, Nq, d)
    if c["heavy"]:  # Student's t, 3 degrees of freedom: a normal over the root of a mean of three squared normals
        q /= sum(normal(B, Hq, Nq, d).square_() for _ in range(3)).div_(3).sqrt_()
    k = normal(B, Hkv, Nk, d)
    if c["heavy"]:
        pick = torch.rand(B, Hkv, d, generator=g, device="cuda").argsort(-1) < 4
        k *= torch.where(pick, 20.0, 1.0)[:, :, None, :]
    k += 3.0 * normal(B, Hkv, 1, d)
    v = normal(B, Hkv, Nk, d)
    return q.to(dt), k.to(dt), v.to(dt)


def prepare(case, seed):
    c = case
    B, Hq, Hkv, Nq, Nk, d = (c[x] for x in ("B", "Hq", "Hkv", "Nq", "Nk", "d"))
    q, k, v = _inputs(c, seed)
    s = dict(kind=c["kind"], causal=c["causal"], q=q, k=k, v=v)
    if c["kind"] == "packed":
        # [B, N, (Hq + 2 Hkv) * d] as a projection writes it; q, k, v are views of it
        qkv = torch.cat([t.transpose(1, 2).reshape(B, Nk, -1) for t in (q, k, v)], dim=2)
        heads = qkv.view(B, Nk, Hq + 2 * Hkv, d)
        s.update(q=heads[:, :, :Hq], k=heads[:, :, Hq:Hq + Hkv], v=heads[:, :, Hq + Hkv:])
        s["out"] = torch.empty(B, Nq, Hq, d, dtype=q.dtype, device="cuda")
        s["workspace"] = torch.empty(sage.workspace_bytes_gqa(B, Hq, Hkv, Nq, Nk, d), dtype=torch.uint8, device="cuda")
    elif c["kind"] == "cache":
        k_i8, k_scale, _, v_fp8, v_scale = sage.sage_quant_kv(k, v)
        s.update(k=None, v=None, cache=(k_i8, v_fp8, k_scale, v_scale), out=torch.empty_like(q))
        s["workspace"] = torch.empty(max(256, sage.decode_workspace_bytes(B, Hq, Hkv, Nq, Nk, d)), dtype=torch.uint8,
                                     device="cuda")
    elif c["kind"] == "quant":
        s["q"] = None
    return s


def run(state):
    s = state
    kind, causal, q, k, v = s["kind"], s["causal"], s["q"], s["k"], s["v"]
    if kind == "fwd":
        return sage.sage_attn_fwd(q, k, v, causal=causal)
    if kind == "packed":
        return sage.sage_attn_fwd_strided(q, k, v, causal=causal, layout="bnhd", out=s["out"], workspace=s["workspace"])
    if kind == "fwd4":
        return sage.sage_attn_fwd_4bit(q, k, v, causal=causal)
    if kind == "cache":
        return sage.sage_attn_fwd_decode(q, *s["cache"], causal=causal, out=s["out"], workspace=s["workspace"])
    if kind == "quant":
        return sage.sage_quant_kv(k, v)
    q_i8, k_i8, q_scale, k_scale, k_mean = sage.sage_quant_qk(q, k)
    v_fp8, v_scale = sage.sage_quant_v(v)
    out = sage.sage_attn_fwd_quantized(q_i8, k_i8, v_fp8, q_scale, k_scale, v_scale, causal=causal, sm_scale=0.0,
                                       out_dtype=q.dtype)
    return out, q_i8, k_i8, q_scale, k_scale, k_mean, v_fp8, v_scale


def work(case):
    c = case
    B, Hq, Hkv, Nq, Nk, d = (c[x] for x in ("B", "Hq", "Hkv", "Nq", "Nk", "d"))
    eq, ek = B * Hq * Nq * d, B * Hkv * Nk * d
    # (row r of a causal call sees the keys up to r + Nk - Nq)
    pairs = Nq * Nk - (Nq * (Nq - 1) // 2 if c["causal"] else 0)
    flops = 4 * B * Hq * pairs * d
    if c["kind"] == "quant":
        return dict(bytes=6 * ek, flops=0)
    if c["kind"] == "cache":
        return dict(bytes=4 * eq + 2 * ek, flops=flops)
    if c["kind"] == "staged":
        return dict(bytes=2 * (eq + 2 * ek) + (eq + 2 * ek) + 2 * eq, flops=flops)
    return dict(bytes=4 * eq + 4 * ek, flops=flops)


def tolerance(case):
    """What another correct implementation at the same precision shows, from measurements of the listed cases."""
    if case["kind"] == "quant":
        return "exact"  # codes and scales are defined operation by operation
    if case["kind"] == "cache":
        # the keys are cut into ranges of the library's choosing and the FP8 rounding of the weights follows the range's
        # own maximum: half or twice the range length moves the output by 0.015 .. 0.022 (at most 0.14 in one value)
        return {"rel": 0.03, "max": 0.5}
    # against the same steps in double precision: 0.6 .. 1.2e-4 (fp16) and 1.0 .. 3.7e-4 (bf16), most of it the last bit
    # of the output; a weight at the edge between two FP8 values moves a single value by up to 0.1
    return {"rel": 5e-4 if case["dtype"] == "fp16" else 1.5e-3, "max": 0.4}
