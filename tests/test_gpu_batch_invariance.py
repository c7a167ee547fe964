"""A head's result does not depend on how many heads the call has.  Which kernel runs above 64 query rows is chosen by the number
of query tiles of all heads (a key step spread over a workgroup of 32 or of 64 rows, or whole steps per wavefront); the C header
tells callers whose results must not depend on the batch size to pass split_keys of their own, and says that one range gives
the bits of the attention call.  So the three kernels have to make the same additions in the same order."""
import pytest
import torch

import paper_2505_21136_amd as sage
from gpu_util import say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# one key step and a few of them, first and last steps of every parity, ragged ends, more than the 32 steps of one strip of scales
SHAPES = [(65, 65), (128, 100), (96, 129), (129, 255), (200, 384), (160, 500), (300, 640), (127, 1000), (512, 513), (100, 4225),
          (130, 8321)]


def _inputs(Nq, Nk, d, dtype):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000 * Nq + Nk + d)
    q, k, v = (torch.randn(1, 2, n, d, generator=g, device=DEV) for n in (Nq, Nk, Nk))
    k += 3.0 * torch.randn(1, 2, 1, d, generator=g, device=DEV)
    q[:, 1] *= 8.0  # (running maxima that move in late steps too)
    return q.to(dtype), k.to(dtype), v.to(dtype)


def _batches(Nq):
    """Copies of two heads that take each of the three kernels."""
    t32, t64 = -(-Nq // 32), -(-Nq // 64)
    b = [1, 256 // (2 * t32) + 1, 256 // (2 * t64) + 1]
    assert 2 * t32 <= 256 and 2 * b[1] * t32 > 256 >= 2 * b[1] * t64 and 2 * b[2] * t64 > 256
    return b


def _same_for_all(call, copies, what):
    want = None
    for b in copies:
        got = call(b)
        torch.cuda.synchronize()
        assert torch.isfinite(got.float()).all(), what
        want = got[:1].clone() if want is None else want
        same = got.view(torch.int16) == want.view(torch.int16)
        assert bool(same.all()), f"{what}: {b} copies: {int((~same).sum())} of {got.numel()} elements differ from one copy"


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Nq,Nk", SHAPES)
def test_result_of_a_head_does_not_depend_on_the_number_of_heads(Nq, Nk, d, causal):
    if causal and Nk < Nq:
        Nk = Nq
    dtype = torch.float16 if (Nq + Nk) % 2 else torch.bfloat16
    say(f"[batch invariance] Nq{Nq} Nk{Nk} d{d} causal={causal} {dtype}")
    q, k, v = _inputs(Nq, Nk, d, dtype)
    k_i8, k_scale, _, v_fp8, v_scale = sage.sage_quant_kv(k, v)
    q_i8, q_scale = sage.sage_quant_q(q)
    one_range = -(-Nk // 128) * 128

    def rep(t, b):
        return t.repeat(b, *([1] * (t.dim() - 1)))

    def attention(b):
        return sage.sage_attn_fwd_kvquantized_gqa(rep(q, b), rep(k_i8, b), rep(v_fp8, b), rep(k_scale, b), rep(v_scale, b),
                                                  causal=causal, sm_scale=0.0)

    def quantised(b):
        return sage.sage_attn_fwd_quantized_gqa(rep(q_i8, b), rep(k_i8, b), rep(v_fp8, b), rep(q_scale, b), rep(k_scale, b),
                                                rep(v_scale, b), causal=causal, sm_scale=0.0, out_dtype=dtype)

    def one(b):
        return sage.sage_attn_fwd_decode(rep(q, b), rep(k_i8, b), rep(v_fp8, b), rep(k_scale, b), rep(v_scale, b), causal=causal,
                                         split_keys=one_range)

    copies = _batches(Nq)
    _same_for_all(attention, copies, "attention")
    _same_for_all(quantised, copies, "quantised Q")
    _same_for_all(one, copies, "one range")
    assert torch.equal(attention(1), quantised(1)) and torch.equal(attention(1), one(1))
    if Nk > 128:
        _same_for_all(lambda b: sage.sage_attn_fwd_decode(rep(q, b), rep(k_i8, b), rep(v_fp8, b), rep(k_scale, b),
                                                          rep(v_scale, b), causal=causal, split_keys=256), copies, "ranges")
