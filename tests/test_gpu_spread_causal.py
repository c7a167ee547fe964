"""Causal calls on both sides of the lines up to which 32 or 64 query rows per workgroup are taken, with more tiles than CUs: a head's bits
do not depend on how many heads the call has (one head alone takes 32 rows per workgroup, many heads 128), grouped, ragged and rectangular."""
import pytest
import torch

import paper_2505_21136_amd as sage
from gpu_util import say

pytestmark = pytest.mark.gpu

# (heads, query heads per K/V head, Nq, Nk, d): tiles of 32 rows beyond 256 (288, 384, 512), of 64 (320, 384, 512), and just past either line
SHAPES = [(9, 1, 1024, 1024, 128), (12, 4, 1021, 1027, 64), (4, 1, 4096, 4096, 128), (4, 2, 4065, 4100, 64), (20, 2, 1024, 1024, 64),
          (24, 1, 1024, 1024, 128), (12, 3, 2047, 2050, 128), (8, 8, 4096, 4096, 64), (9, 1, 4096, 4096, 128), (18, 1, 512, 1500, 128),
          (5, 1, 2048, 4096, 64), (27, 1, 300, 300, 128)]


@pytest.mark.parametrize("heads,group,nq,nk,d", SHAPES)
def test_a_causal_head_has_the_same_bits_in_calls_of_every_size(heads, group, nq, nk, d):
    say(f"[spread causal] {heads} heads, {group} per K/V head, {nq} x {nk} x {d}")
    g = torch.Generator(device="cuda").manual_seed(heads * nq + nk)
    rnd = lambda h, n: torch.randn(1, h, n, d, generator=g, device="cuda").to(torch.bfloat16)
    q, k, v = rnd(heads, nq), rnd(heads // group, nk), rnd(heads // group, nk)
    out = sage.sage_attn_fwd_gqa(q, k, v, causal=True)
    for h in (0, heads - 1):
        kv = slice(h // group, h // group + 1)
        alone = sage.sage_attn_fwd_gqa(q[:, h:h + 1].contiguous(), k[:, kv].contiguous(), v[:, kv].contiguous(), causal=True)
        assert torch.equal(out[:, h:h + 1].view(torch.int16), alone.view(torch.int16))
    many = -(-520 // heads)  # more than two tiles of 64 rows per CU: 128 rows per workgroup
    big = sage.sage_attn_fwd_gqa(*(x.expand(many, *x.shape[1:]).contiguous() for x in (q, k, v)), causal=True)
    assert torch.equal(big[many - 1].view(torch.int16), out[0].view(torch.int16))
