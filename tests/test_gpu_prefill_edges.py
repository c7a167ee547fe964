"""The kernel behind calls with more than 64 query rows (32 rows per wavefront, 128 per workgroup, key steps of 128) at the
edges of its tiles, whole outputs against the oracle: wavefronts with one, 31, 32 and no valid rows, key tiles of 32 cut at
every kind of place, one key step and the first and last of several, masks whose diagonal falls anywhere in a tile."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_21136_amd as sage
import workloads as wl
from gpu_util import assert_parity, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [  # idx, B, Hq, Hkv, Nq, Nk, d, causal
    (1, 1, 2, 2, 65, 1, 128, False), (3, 1, 2, 2, 96, 31, 64, False), (5, 1, 2, 1, 97, 33, 128, False),
    (1, 1, 2, 2, 127, 127, 128, True), (3, 1, 2, 2, 128, 128, 64, True), (5, 1, 2, 2, 129, 129, 128, True),
    (2, 1, 2, 1, 128, 129, 128, True), (4, 1, 2, 2, 160, 191, 64, True), (1, 1, 1, 1, 129, 255, 128, True),
    (5, 2, 2, 2, 65, 384, 64, True), (2, 1, 2, 2, 257, 385, 128, True), (3, 1, 1, 1, 320, 320, 64, False),
    (5, 1, 1, 1, 130, 4225, 128, False), (4, 1, 1, 1, 100, 8321, 64, True),   # constants re-made every 32 steps
]


@pytest.mark.parametrize("idx,B,Hq,Hkv,Nq,Nk,d,causal", CASES)
def test_tile_edges_against_the_oracle(idx, B, Hq, Hkv, Nq, Nk, d, causal):
    base = wl.CONFIGS[idx - 1]
    say(f"[prefill edges] cfg{idx}-like B{B} Hq{Hq} Hkv{Hkv} Nq{Nq} Nk{Nk} d{d} {base.dtype} causal={causal}")
    q, _, _ = wl.generate(wl.Workload("q", base.index, B, Hq, Nq, d, False, base.dtype, base.q_dist,
                                      base.k_outlier_channels), seed=31 + Nq)
    _, k, v = wl.generate(wl.Workload("kv", base.index, B, Hkv, Nk, d, False, base.dtype, base.q_dist,
                                      base.k_outlier_channels), seed=37 + Nk)
    sm = np.float32(1.0 / np.sqrt(d))
    out = torch.full(q.shape, float("nan"), dtype=q.dtype, device=DEV)
    sage.sage_attn_fwd_gqa(q.to(DEV), k.to(DEV), v.to(DEV), causal=causal, sm_scale=float(sm), out=out)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy()
    assert np.isfinite(got).all()
    ref = oracle.sage_attention(wl.as_f32(q), wl.as_f32(k), wl.as_f32(v), causal=causal, sm_scale=sm,
                                out_dtype=base.dtype)
    # (the limits of the parity gate, derived there for any evaluation of the exponents in binary32)
    assert_parity(ref, got, base.dtype, f"prefill edges Nq{Nq} Nk{Nk}")
