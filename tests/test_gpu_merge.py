"""The combination of key ranges at the counts where its launch changes form (up to four and up to eight ranges in one
thread, more on a workgroup per row), with row counts that do not fill its workgroups, against the oracle's key-split mode
on the same ranges."""
import pytest
import torch

import workloads as wl
from gpu_util import say
from test_gpu_decode import _gpu, _inputs, _oracle

pytestmark = pytest.mark.gpu


# packed rows and the prefill kernel's ranges (more than 64 rows per K/V head); both head dimensions and types
@pytest.mark.parametrize("n_ranges", [2, 4, 5, 8, 9])
@pytest.mark.parametrize("idx,B,Hq,Hkv,Nq,d,causal", [(2, 1, 6, 2, 1, 128, True), (3, 1, 3, 1, 3, 64, False),
                                                      (5, 1, 1, 1, 131, 128, True), (4, 1, 2, 1, 77, 64, True)])
def test_range_counts(idx, B, Hq, Hkv, Nq, d, causal, n_ranges):
    Nk = 256 * n_ranges - 45
    say(f"[merge] {n_ranges} ranges: cfg{idx} B{B} Hq{Hq} Hkv{Hkv} Nq{Nq} Nk{Nk} d{d} causal={causal}")
    q, k, v, sm = _inputs(idx, B, Hq, Hkv, Nq, Nk, d)
    out, _ = _gpu(q, k, v, causal, sm, 256)
    got = out.cpu().to(torch.float64).numpy()
    want = _oracle(q, k, v, causal, sm, 256)
    # The two norms of the benchmark definition.  (Its element-wise gate wants more rows than these: where GPU and oracle round
    # one FP8 weight to different sides, by 1/16 of it at most, all d elements of the row move.  A range left out or weighted
    # wrongly moves the output by about 1 / n_ranges >= 0.1 of itself.)
    cos, l1 = wl.cos_sim(want, got), wl.rel_l1(want, got)
    say(f"   cos={cos:.7f} relL1={l1:.3e}")
    assert cos >= 0.9999 and l1 <= 1e-3
