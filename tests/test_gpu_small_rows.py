"""The kernel for up to 64 query rows per head at its edges (wavefronts with one, fifteen, sixteen and no rows; one key step, a few,
more than the 32 of one strip of scales; ragged ends), 4+8 variant and key ranges of grouped heads, against the oracle."""
import numpy as np
import pytest
import torch

import workloads as wl
from gpu_util import assert_parity, say
from test_gpu_4bit import _full_check, _inputs as _inputs_4bit
from test_gpu_decode import _gpu, _inputs, _oracle

pytestmark = pytest.mark.gpu

ROWS = [(1, 1), (15, 130), (16, 128), (17, 300), (48, 640), (49, 129), (63, 1000), (64, 64), (64, 4500)]


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("base_idx,d", [(1, 128), (3, 64)])
@pytest.mark.parametrize("Nq,Nk", ROWS)
def test_4bit_few_rows(Nq, Nk, base_idx, d, causal):
    say(f"[small rows] 4+8 Nq{Nq} Nk{Nk} d{d} causal={causal}")
    q, k, v, base = _inputs_4bit(base_idx, 1, 4, 2, Nq, Nk, d, 1.5, Nq + Nk)
    _full_check(q, k, v, base, causal)


# more than 64 rows per K/V head, at most 64 per query head: ranges on workgroups of their own; split_keys that cut the 32-step strips
# of scales and that leave ranges no row sees
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("idx,Hq,Hkv,Nq,Nk,d,split_keys", [
    (2, 8, 1, 9, 700, 128, 128), (3, 8, 1, 16, 1000, 64, 256), (5, 6, 1, 17, 640, 128, 384), (4, 4, 2, 33, 2100, 64, 512),
    (1, 4, 2, 48, 300, 128, 128), (3, 2, 1, 63, 400, 64, 128), (5, 2, 1, 64, 9000, 128, 4224), (4, 3, 1, 64, 129, 64, 128)])
def test_ranges_few_rows(idx, Hq, Hkv, Nq, Nk, d, split_keys, causal):
    say(f"[small rows] ranges of {split_keys}: cfg{idx} Hq{Hq} Hkv{Hkv} Nq{Nq} Nk{Nk} d{d} causal={causal}")
    q, k, v, sm = _inputs(idx, 1, Hq, Hkv, Nq, Nk, d)
    out, _ = _gpu(q, k, v, causal, sm, split_keys)
    got = out.cpu().to(torch.float64).numpy()
    want = _oracle(q, k, v, causal, sm, split_keys)
    assert np.isfinite(got).all()
    # (few rows: the norms and the gate as for the seeded decode shapes)
    assert wl.cos_sim(want, got) >= 0.9999 and wl.rel_l1(want, got) <= 1e-3
    assert_parity(want.reshape(-1, d), got.reshape(-1, d), "bf16" if q.dtype == torch.bfloat16 else "fp16",
                  f"small rows, ranges, Nq{Nq}", flip_factor=4.0)
