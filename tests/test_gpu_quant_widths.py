"""The single-read quantiser at the token counts where its launch changes form: a head that fits one workgroup (of 256 or 512
threads: nothing is exchanged), groups of 256-thread workgroups, and from 48 of those on groups of 512 threads; K and V together
and each alone.  Every form writes the bits of the three launches, also where a workgroup does not wait for its partners."""
import pytest
import torch

import paper_2505_21136_amd as sage
from gpu_util import say
from test_gpu_quant_paths import SINGLE_READ, THREE_LAUNCHES, _inputs, _quant, _restore_default_path, _same_bits  # noqa: F401

pytestmark = pytest.mark.gpu


def _alone(k, v, path, wait_ticks=50_000):
    sage.diag_quant_kv_path(path, wait_ticks)
    out = sage.sage_quant_k(k) + sage.sage_quant_v(v, 4.5)
    torch.cuda.synchronize()
    return out


# tokens of a 256-thread workgroup: 256 at d = 128, 512 at d = 64
SHAPES = [(1, (1, 2, 256, 128)), (1, (2, 2, 257, 128)), (2, (1, 2, 512, 128)), (2, (1, 2, 513, 128)), (1, (1, 1, 12288, 128)),
          (5, (1, 2, 12289, 128)), (5, (1, 1, 13001, 128)), (4, (1, 2, 512, 64)), (3, (2, 3, 777, 64)), (3, (1, 2, 1024, 64)),
          (4, (1, 2, 1025, 64)), (4, (1, 1, 24576, 64)), (3, (1, 2, 24577, 64)), (4, (1, 1, 25601, 64)),
          # enough heads for the wide workgroups, K alone too
          (5, (2, 3, 12289, 128)), (3, (1, 6, 24577, 64))]


@pytest.mark.parametrize("wait_ticks", [50_000, -1])
@pytest.mark.parametrize("idx,shape", SHAPES)
def test_every_width_writes_the_bits_of_the_three_launches(idx, shape, wait_ticks):
    say(f"[quant widths] cfg{idx} distributions, shape {shape}, wait {wait_ticks}")
    k, v = _inputs(idx, shape)
    want = _quant(k, v, 4.5, THREE_LAUNCHES)
    _same_bits(want, _quant(k, v, 4.5, SINGLE_READ, wait_ticks), "K and V together")
    _same_bits(want, _alone(k, v, THREE_LAUNCHES), "each alone, three launches")
    _same_bits(want, _alone(k, v, SINGLE_READ, wait_ticks), "each alone, single read")
    _same_bits(want, _quant(k, v, 4.5, 0, wait_ticks), "by shape")


# Many workgroups, on both sides of the lines from which on those of a CU start apart (from two rounds on; 256 threads, heads of one
# chunk never and of seven and eight chunks; 512 threads, a chunk less and more than three quarters full) and from which on V's codes go
# through LDS (by the rounds of V's workgroups: d = 128 2.5; d = 64 one, with 512 threads 1.9 -- there with several workgroups per head, too --
# and a head of up to 256 tokens)
MANY = [(1030, 129, 128), (150, 1700, 128), (128, 2048, 128), (513, 300, 128), (513, 384, 128), (700, 600, 128), (860, 601, 128),
        (513, 767, 64), (513, 1010, 64), (340, 1100, 64), (350, 1100, 64), (7, 256, 64), (7, 257, 64), (1000, 600, 64), (14, 70001, 64)]


@pytest.mark.parametrize("wait_ticks", [50_000, -1])
@pytest.mark.parametrize("H,N,d", MANY)
def test_several_rounds_of_workgroups_write_the_bits_of_the_three_launches(H, N, d, wait_ticks):
    say(f"[quant rounds] {H} heads x {N} x {d}, wait {wait_ticks}")
    g = torch.Generator(device="cuda").manual_seed(H + N)
    k, v = (torch.randn(1, H, N, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    want = _quant(k, v, 4.5, THREE_LAUNCHES)
    _same_bits(want, _quant(k, v, 4.5, 0, wait_ticks), "K and V together")
    _same_bits(want, _alone(k, v, 0, wait_ticks), "each alone")
