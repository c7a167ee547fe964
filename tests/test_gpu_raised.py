"""Attention above 64 rows with the wavefronts' priority raised around the exponentials, on both sides of every line of its rule: a head's
bits are those of the same head in a call of two heads, which other kernels serve, and key ranges agree with each head's own."""
import pytest
import torch

import paper_2505_21136_amd as sage
from gpu_util import say

pytestmark = pytest.mark.gpu

CASES = [  # heads, rows, keys, d, causal: workgroups of 128 rows
    (32, 1000, 900, 128, False),   # 256
    (33, 1000, 900, 128, False),   # 264
    (64, 1000, 300, 128, False),   # 512
    (65, 1000, 300, 128, False),   # 520
    (33, 1000, 900, 64, False),    # 264
    (97, 1000, 300, 64, False),    # 776
    (129, 1000, 300, 64, False),   # 1032
    (511, 500, 500, 64, True),     # 2044
    (512, 500, 500, 64, True),     # 2048
]


def _cache(H, Nq, Nk, d, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    q, k, v = (torch.randn(1, H, n, d, generator=g, device="cuda").to(torch.bfloat16) for n in (Nq, Nk, Nk))
    k_i8, k_scale, _, v_fp8, v_scale = sage.sage_quant_kv(k, v)
    return q, (k_i8, v_fp8, k_scale, v_scale)


def _last_two(q, cache):
    return q[:, -2:].contiguous(), tuple(t[:, -2:].contiguous() for t in cache)


@pytest.mark.parametrize("H,Nq,Nk,d,causal", CASES)
def test_bits_of_a_head_do_not_depend_on_the_priority(H, Nq, Nk, d, causal):
    say(f"[raised] {H} heads {Nq} x {Nk} d{d} causal={causal}")
    q, cache = _cache(H, Nq, Nk, d, H + Nq)
    out = sage.sage_attn_fwd_kvquantized_gqa(q, *cache, causal=causal, sm_scale=0.0)
    q2, cache2 = _last_two(q, cache)
    few = sage.sage_attn_fwd_kvquantized_gqa(q2, *cache2, causal=causal, sm_scale=0.0)
    assert torch.isfinite(out.float()).all()
    assert torch.equal(out[:, -2:].view(torch.int16), few.view(torch.int16))


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d", [64, 128])
def test_bits_of_key_ranges_do_not_depend_on_the_priority(d, causal):
    H, Nq, Nk, split = 35, 200, 1000, 256     # 35 x 2 tiles x 4 ranges: 280 workgroups; 16 for two heads
    q, cache = _cache(H, Nq, Nk, d, 7)
    out = sage.sage_attn_fwd_decode(q, *cache, causal=causal, split_keys=split)
    q2, cache2 = _last_two(q, cache)
    few = sage.sage_attn_fwd_decode(q2, *cache2, causal=causal, split_keys=split)
    assert torch.isfinite(out.float()).all()
    assert torch.equal(out[:, -2:].view(torch.int16), few.view(torch.int16))
