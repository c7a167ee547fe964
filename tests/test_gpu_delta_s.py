"""The score correction of the 4+8 variant against 64 bits."""
import math

import pytest
import torch

import paper_2505_21136_amd as sage
from gpu_util import say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
LOG2E = 1.4426950408889634


def _exact(k, k_mean, q_mean, d):
    """[Hq, nQ, Nk] in double precision, from the same binary32 means."""
    kp = k[0].double() - k_mean[0].double()[:, None]
    kp = kp.repeat_interleave(q_mean.shape[1] // kp.shape[0], 0)
    return torch.matmul(q_mean[0].double(), kp.transpose(1, 2).contiguous()) * (1.0 / math.sqrt(d)) * LOG2E


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,Nq,Nk", [(2, 2, 1000, 1000), (8, 2, 3000, 3000), (1, 1, 100, 4000), (4, 1, 128, 2000)])
def test_error_against_64_bits(Hq, Hkv, Nq, Nk, d):
    say(f"[delta_s precision] Hq{Hq} Hkv{Hkv} Nq{Nq} Nk{Nk} d{d}")
    g = torch.Generator(device=DEV)
    g.manual_seed(Nq + d)
    q = torch.randn(1, Hq, Nq, d, generator=g, device=DEV).half()
    k = torch.randn(1, Hkv, Nk, d, generator=g, device=DEV).half()
    k_mean = sage.sage_quant_kv4(k, torch.zeros_like(k))[2]
    q_mean = sage.sage_quant_q4(q, codes=False)[0]
    got = sage.delta_s_to_key_order(sage.sage_delta_s(k, k_mean, q_mean, Nq, causal=False), Nk)[0].double()
    want = _exact(k, k_mean, q_mean, d)
    err = ((got - want).norm() / want.norm()).item()
    # Sums of independent terms in four chains of d / 4: a rounding adds a relative error of at most u = 2^-24 with a mean square of
    # u^2 / 3, a chain's partial sums grow like the square root of their length, so the chains contribute d u^2 / 24 to the mean
    # square relative to the result; the smoothing of K, adding the chains and the scale at most u^2 / 3 each.  (One chain
    # would be d u^2 / 6: measured 1.4e-7 at d = 64 and 2.0e-7 at d = 128.)
    bound = 2.0**-24 * math.sqrt(d / 24 + 1.0)
    say(f"   {err:.3e}, bound {bound:.3e}")
    assert err <= bound


def test_more_column_tiles_than_a_grid_dimension_takes():
    """257 query heads on one K/V head, 2^22 query rows: 263168 tiles of 32 (Q block, head) columns, at most four per workgroup
    by the ordinary rule, and the grid's third dimension ends at 65535."""
    Hq, Nq, Nk, d = 257, 1 << 22, 40, 64
    nQ = Nq // 128
    say(f"[delta_s] Hq{Hq} Nq{Nq} Nk{Nk} d{d}")
    g = torch.Generator(device=DEV)
    g.manual_seed(5)
    k = torch.randn(1, 1, Nk, d, generator=g, device=DEV).half()
    k_mean = k.float().mean(2)
    q_mean = torch.randn(1, Hq, nQ, d, generator=g, device=DEV)
    dsx = sage.sage_delta_s(k, k_mean, q_mean, Nq, causal=False)
    torch.cuda.synchronize()
    for h0 in range(0, Hq, 32):
        got = sage.delta_s_to_key_order(dsx[:, h0:h0 + 32], Nk)[0].double()
        want = _exact(k, k_mean, q_mean[:, h0:h0 + 32], d)
        # (as above; the largest single value within sqrt(d) times the typical error)
        assert ((got - want).norm() / want.norm()).item() <= 2.0**-24 * math.sqrt(d / 24 + 1.0), h0
        assert ((got - want).abs().max() / want.square().mean().sqrt()).item() <= 2.0**-24 * 64, h0
