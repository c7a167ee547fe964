"""The kernels behind calls with more than 64 query rows at the edges of their tiles, whole outputs against the oracle:
wavefronts with one, 31, 32 and no valid rows, key tiles of 32 cut at every kind of place, one key step and the first and last
of several, masks whose diagonal falls anywhere in a tile.  Which kernel runs depends on how many workgroups the query rows
make, so every shape runs with few heads (a key step spread over a workgroup of 32 rows), with more (64 rows, where there are more
than two key steps) and with many (whole steps per wavefront)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_21136_amd as sage
import workloads as wl
from gpu_util import assert_parity, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [  # idx, Hkv, Nq, Nk, d, causal
    (1, 2, 65, 1, 128, False), (3, 2, 96, 31, 64, False), (5, 1, 97, 33, 128, False),
    (1, 2, 127, 127, 128, True), (3, 2, 128, 128, 64, True), (5, 2, 129, 129, 128, True),
    (2, 1, 128, 129, 128, True), (4, 2, 160, 191, 64, True), (1, 1, 129, 255, 128, True),
    (5, 2, 65, 384, 64, True), (2, 2, 257, 385, 128, True), (3, 1, 320, 320, 64, False), (4, 1, 193, 640, 128, True),
]
CASES += [(2, 2, 65, 257, 128, True), (3, 1, 97, 300, 64, False), (5, 1, 129, 383, 128, False)]  # three key steps
LONG = [  # de-quantisation constants are re-made every 32 steps
    (5, 1, 130, 4225, 128, False), (4, 1, 100, 8321, 64, True),
]


def _heads(kernel, Hkv, Nq):
    """Query heads (a multiple of Hkv) for which the shape takes the kernel: tiles of 32 rows <= 256, of 64 rows <= 256, more."""
    t32, t64 = -(-Nq // 32), -(-Nq // 64)
    h = {"32 rows": Hkv, "64 rows": 256 // t32 + 1, "whole steps": 256 // t64 + 1}[kernel]
    h = -(-h // Hkv) * Hkv
    assert {"32 rows": h * t32 <= 256, "64 rows": h * t32 > 256 >= h * t64, "whole steps": h * t64 > 256}[kernel]
    return h


def _run(idx, Hq, Hkv, Nq, Nk, d, causal, what):
    base = wl.CONFIGS[idx - 1]
    say(f"[prefill edges] {what}: cfg{idx}-like Hq{Hq} Hkv{Hkv} Nq{Nq} Nk{Nk} d{d} {base.dtype} causal={causal}")
    q, _, _ = wl.generate(wl.Workload("q", base.index, 1, Hq, Nq, d, False, base.dtype, base.q_dist,
                                      base.k_outlier_channels), seed=31 + Nq)
    _, k, v = wl.generate(wl.Workload("kv", base.index, 1, Hkv, Nk, d, False, base.dtype, base.q_dist,
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
    assert_parity(ref, got, base.dtype, f"prefill edges, {what}, Nq{Nq} Nk{Nk}")


@pytest.mark.parametrize("kernel", ["32 rows", "64 rows", "whole steps"])
@pytest.mark.parametrize("idx,Hkv,Nq,Nk,d,causal", CASES)
def test_tile_edges_against_the_oracle(idx, Hkv, Nq, Nk, d, causal, kernel):
    _run(idx, _heads(kernel, Hkv, Nq), Hkv, Nq, Nk, d, causal, kernel)


@pytest.mark.parametrize("kernel", ["32 rows", "64 rows", "whole steps"])
@pytest.mark.parametrize("idx,Hkv,Nq,Nk,d,causal", LONG)
def test_many_steps_against_the_oracle(idx, Hkv, Nq, Nk, d, causal, kernel):
    _run(idx, _heads(kernel, Hkv, Nq), Hkv, Nq, Nk, d, causal, kernel)
