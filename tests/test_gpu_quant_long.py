"""The single-read quantiser for long heads (groups of 512-thread workgroups, up to 128 of them) and the borders of the rule that
chooses it, bit for bit against the three launches: K and V together, each alone, and K with Q; also where a workgroup does not wait
for its partners, and next to a kernel that holds the CUs."""
import pytest
import torch

import paper_2505_21136_amd as sage
import workloads as wl
from gpu_util import say
from test_gpu_quant_paths import SINGLE_READ, THREE_LAUNCHES, _quant, _restore_default_path, _same_bits  # noqa: F401

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _inputs(B, H, N, d, dtype, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    q, k, v = (torch.randn(B, H, N, d, generator=g, device=DEV) for _ in range(3))
    k += 3.0 * torch.randn(B, H, 1, d, generator=g, device=DEV)
    return q.to(dtype), k.to(dtype), v.to(dtype)


def _alone(k, v, path, wait_ticks=50_000):
    sage.diag_quant_kv_path(path, wait_ticks)
    out = sage.sage_quant_k(k) + sage.sage_quant_v(v, 4.5)
    torch.cuda.synchronize()
    return out


def _qk(q, k, path, wait_ticks=50_000):
    sage.diag_quant_kv_path(path, wait_ticks)
    out = sage.sage_quant_qk(q, k)
    torch.cuda.synchronize()
    return out


def _compare(B, H, N, d, dtype, waits):
    q, k, v = _inputs(B, H, N, d, dtype, N + H)
    want = _quant(k, v, 4.5, THREE_LAUNCHES)
    q_i8, q_scale = sage.sage_quant_q(q)
    want_qk = (q_i8, want[0], q_scale, want[1], want[2])
    forced = N <= (65536 if d == 128 else 131072)
    for path, wait in [(0, w) for w in waits] + ([(SINGLE_READ, w) for w in waits] if forced else []) + [(THREE_LAUNCHES, 0)]:
        what = f"path {path}, wait {wait}"
        _same_bits(want, _quant(k, v, 4.5, path, wait), f"K and V, {what}")
        _same_bits(want, _alone(k, v, path, wait), f"each alone, {what}")
        for a, b in zip(want_qk, _qk(q, k, path, wait)):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), f"Q and K, {what}"


# tokens: last and first of 96 / 97 and 128 / 129 workgroups of 256 threads, ragged ones, the last that 512 threads reach, one more
@pytest.mark.parametrize("H,N,d", [
    (1, 24576, 128), (2, 24577, 128), (1, 32768, 128), (1, 32769, 128), (3, 33000, 128), (1, 50000, 128), (2, 65536, 128),
    (1, 65537, 128), (1, 65536, 64), (2, 65537, 64), (1, 100001, 64), (1, 131072, 64), (1, 131073, 64)])
def test_long_heads(H, N, d):
    say(f"[quant long] H{H} N{N} d{d}")
    _compare(1, H, N, d, torch.bfloat16 if N % 2 else torch.float16, [50_000, -1])


# both sides of what depends on the number of workgroups: 512 resident at once and 1024 (d = 128, N 36001: 71 of 512 threads per head
# and tensor; d = 64, N 65537: 65), and the small calls that three launches serve (K or V alone at d = 64)
@pytest.mark.parametrize("B,H,N,d", [
    (1, 4, 36001, 128), (1, 8, 36001, 128), (1, 7, 65537, 64), (1, 8, 65537, 64),
    (1, 2, 1000, 64), (2, 64, 1000, 64), (1, 127, 1000, 64), (1, 4, 12000, 64), (3, 4, 12000, 64), (1, 1, 30000, 128),
    (1, 31, 777, 64), (1, 32, 777, 64), (2, 5, 500, 128)])
def test_borders_of_the_rule(B, H, N, d):
    say(f"[quant long] rule: B{B} H{H} N{N} d{d}")
    _compare(B, H, N, d, torch.float16 if H % 2 else torch.bfloat16, [50_000])


def test_k_alone_and_with_q_next_to_a_kernel_that_holds_the_cus():
    """K alone, V alone and K with Q meet inside a launch too: with another stream's attention kernel on the CUs they may have to
    go on alone after the wait bound.  Same bits, and every launch ends."""
    cfg = wl.CONFIGS[4].scaled(H=8)                       # B1 H8 N32768 d128: an attention launch of ~2.5 ms
    qa, ka, va = (t.to(DEV) for t in wl.generate(cfg))
    ws_a = torch.empty(sage.workspace_bytes(cfg.B, cfg.H, cfg.N, cfg.d), dtype=torch.uint8, device=DEV)
    out_a = torch.empty_like(qa)
    shapes = [(1, 8, 33000, 128), (4, 16, 4096, 128), (2, 64, 1000, 64)]  # groups of 512 threads, of 256, nobody to meet
    cases = []
    for s in shapes:
        q, k, v = _inputs(*s, torch.bfloat16, s[2])
        q_i8, q_scale = sage.sage_quant_q(q)
        cases.append((q, k, v, _quant(k, v, 4.5, THREE_LAUNCHES), q_i8, q_scale))
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    sage.diag_quant_kv_path(SINGLE_READ, 20_000)          # 0.2 ms: short enough for some waits to run out
    for rep in range(2):
        got = []
        with torch.cuda.stream(side):
            for _ in range(4):
                sage.sage_attn_fwd(qa, ka, va, causal=False, out=out_a, workspace=ws_a)
        for q, k, v, *_ in cases:
            got.append((sage.sage_quant_k(k) + sage.sage_quant_v(v, 4.5), sage.sage_quant_qk(q, k)))
        torch.cuda.synchronize()
        for s, (kv, qk), (_, _, _, want, q_i8, q_scale) in zip(shapes, got, cases):
            _same_bits(want, kv, f"{s} next to attention, repetition {rep}")
            for a, b in zip((q_i8, want[0], q_scale, want[1], want[2]), qk):
                assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), (s, rep)
