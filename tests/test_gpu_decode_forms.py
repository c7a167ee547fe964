"""sage_attn_fwd_decode in each of the shapes its launch can take -- the ranges of a K/V head in one workgroup or in workgroups of one
or four wavefronts with a second launch, one or two row tiles per wavefront, one or two wavefronts per range, the last tiles ragged --
against the oracle on the same ranges.  (tests/test_tile_copy_bounds.py has the addresses of its copies.)"""
import numpy as np
import pytest
import torch

import paper_2505_21136_amd as sage
from gpu_util import assert_parity, say
from test_gpu_decode import _gpu, _inputs, _oracle

FORMS = [  # B, Hq, Hkv, Nq, Nk, d, split_keys, heads compared
    (1, 2, 2, 1, 1000, 128, 128, None),       # one workgroup of eight wavefronts (64 KB of LDS and more)
    (1, 4, 4, 4, 1001, 64, 384, None),        # three
    (1, 2, 2, 32, 500, 128, 128, None),       # two row tiles, one workgroup of four
    (1, 2, 2, 32, 640, 128, 128, None),       # five ranges of two row tiles: a second launch
    (1, 1, 1, 40, 300, 64, 128, None),        # three row tiles, two wavefronts per range, a second launch
    (2, 260, 65, 16, 129, 64, 128, {(0, 0), (1, 64)}),    # 130 K/V heads of 64 rows: one workgroup of 2 x 2 wavefronts
    (2, 65, 65, 49, 400, 128, 128, {(0, 0), (1, 64)}),    # 130 of 49 rows, 2 x 4 wavefronts: all of LDS
    (1, 16, 16, 1, 8197, 64, 128, {(0, 0), (0, 15)}),     # 1040 wavefronts of one step, four to a workgroup, 65 ranges
    (1, 8, 8, 64, 4700, 128, 128, {(0, 0), (0, 7)}),      # 592 wavefronts in pairs, four to a workgroup
    (1, 2, 2, 1, 8193, 128, 128, None),       # 65 ranges of a row to combine, ...
    (1, 4, 1, 2, 33000, 64, 128, None),       # ... 258: more than a workgroup's threads
]


@pytest.mark.gpu
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("B,Hq,Hkv,Nq,Nk,d,split,heads", FORMS)
def test_decode_forms_against_the_oracle(B, Hq, Hkv, Nq, Nk, d, split, heads, causal):
    q, k, v, sm = _inputs(5 if d == 128 else 1, B, Hq, Hkv, Nq, Nk, d)
    out, _ = _gpu(q, k, v, causal, sm, split)
    want = _oracle(q, k, v, causal, sm, split, heads=heads)
    got = out.cpu().to(torch.float64).numpy()
    assert np.isfinite(got).all()
    g = Hq // Hkv
    pick = [(b, h) for b in range(B) for h in range(Hq) if heads is None or (b, h // g) in heads]
    w, x = (np.concatenate([t[b, h] for b, h in pick]) for t in (want, got))
    assert_parity(w, x, "bf16" if q.dtype == torch.bfloat16 else "fp16", f"decode B{B} Hq{Hq}/{Hkv} Nq{Nq} Nk{Nk} d{d} {split}",
                  flip_factor=4.0)


# K/V heads, query rows of a K/V head, Nk, d, split_keys, whether one launch does it (pairs on both sides of the lines, which were timed
# with caches that are not in the last-level cache)
ROUTES = [
    (8, 4, 1500, 128, 0, True), (8, 4, 2048, 128, 0, False),                          # bytes per head, few heads
    (96, 4, 2048, 128, 0, True), (128, 4, 4096, 128, 0, False), (128, 4, 4096, 64, 0, True),
    (64, 4, 2048, 128, 1024, True), (64, 4, 8192, 128, 2048, False), (8, 4, 16384, 64, 4096, True),  # copies in flight
    (136, 4, 4096, 128, 0, True), (257, 4, 1000, 128, 0, True), (257, 4, 2048, 128, 0, False), (360, 4, 2048, 128, 0, True),  # rounds
    (8, 32, 256, 128, 0, False), (8, 32, 256, 64, 0, True), (8, 32, 1000, 128, 0, True), (300, 32, 4096, 128, 0, False),  # two row tiles
    (16, 64, 700, 128, 0, False), (150, 64, 700, 128, 0, True),
]


@pytest.mark.gpu
@pytest.mark.parametrize("H,rows,Nk,d,split,one", ROUTES)
def test_one_launch_where_it_pays_and_the_same_bits_either_way(H, rows, Nk, d, split, one):
    """A call whose ranges are combined by the workgroup that holds them writes nothing to its scratch."""
    say(f"[decode route] {H} heads {rows} rows Nk{Nk} d{d} split {split}")
    g = torch.Generator(device="cuda").manual_seed(H + Nk)
    q = torch.randn(1, H, rows, d, generator=g, device="cuda").to(torch.bfloat16)
    k, v = (torch.randn(1, H, Nk, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    k_i8, k_scale, _, v_fp8, v_scale = sage.sage_quant_kv(k, v)
    cache = (k_i8, v_fp8, k_scale, v_scale)
    split = split or sage.decode_split_keys(1, H, H, rows, Nk)
    ws = torch.full((sage.decode_workspace_bytes(1, H, H, rows, Nk, d, split),), 0x5A, dtype=torch.uint8, device="cuda")
    out = sage.sage_attn_fwd_decode(q, *cache, causal=True, split_keys=split, workspace=ws)
    assert bool((ws == 0x5A).all()) == one
    few = sage.sage_attn_fwd_decode(q[:, -2:].contiguous(), *(t[:, -2:].contiguous() for t in cache), causal=True, split_keys=split)
    assert torch.isfinite(out.float()).all()
    assert torch.equal(out[:, -2:].view(torch.int16), few.view(torch.int16))
