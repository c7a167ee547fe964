"""The quantisers' two launches over chunks (small calls), at the edges of chunks, K blocks and V tiles, and V alone up to the largest calls
that take them: K and V together, each alone, K with Q, the INT4 codes and strided inputs write the bits of the three launches, and the codes
of Q those of a launch of its own."""
import pytest
import torch

import paper_2505_21136_amd as sage
from gpu_util import say
from test_gpu_quant_paths import THREE_LAUNCHES, _against_oracle, _inputs, _quant, _restore_default_path, _same_bits  # noqa: F401

pytestmark = pytest.mark.gpu

# a chunk is 256 tokens at d = 128 and 512 at d = 64
SHAPES = [(1, (1, 2, 257, 128)), (2, (1, 3, 512, 128)), (5, (1, 2, 513, 128)), (1, (2, 2, 1024, 128)), (5, (1, 1, 1089, 128)),
          (2, (1, 1, 32768, 128)), (5, (1, 2, 16129, 128)), (2, (1, 128, 769, 128)),
          (4, (1, 2, 200, 64)), (3, (1, 2, 512, 64)), (4, (2, 3, 513, 64)), (3, (1, 2, 1537, 64)), (4, (1, 32, 2048, 64)),
          (3, (1, 64, 300, 64)),
          # K with Q: its own lines
          (2, (1, 48, 1000, 128)), (5, (1, 64, 400, 128)), (4, (1, 24, 4001, 64)), (3, (1, 96, 900, 64))]


@pytest.mark.parametrize("idx,shape", SHAPES)
def test_chunks_write_the_bits_of_the_three_launches(idx, shape):
    say(f"[quant chunks] cfg{idx} distributions, shape {shape}")
    k, v = _inputs(idx, shape)
    want = _quant(k, v, 4.5, THREE_LAUNCHES)
    want4 = sage.sage_quant_kv4(k, v)  # (the three launches still forced)
    got = _quant(k, v, 4.5, 0)
    _same_bits(want, got, "K and V together")
    _same_bits(want4, sage.sage_quant_kv4(k, v), "INT4 codes")
    _same_bits(want, sage.sage_quant_k(k) + sage.sage_quant_v(v, 4.5), "each alone")
    q_i8, k_i8, q_scale, k_scale, k_mean = sage.sage_quant_qk(v, k)
    _same_bits(want[:3] + sage.sage_quant_q(v), (k_i8, k_scale, k_mean, q_i8, q_scale), "K with Q")
    # token-major views, through the call that quantises strided inputs
    out = sage.sage_attn_fwd(v, k, v, causal=False)
    q_t, k_t, v_t = (x.transpose(1, 2).contiguous() for x in (v, k, v))
    out_t = sage.sage_attn_fwd_strided(q_t, k_t, v_t, causal=False, layout="bnhd")
    assert torch.equal(out.view(torch.int16), out_t.transpose(1, 2).view(torch.int16))
    if shape[1] * shape[2] <= 3000:
        _against_oracle(got, k, v, 4.5, shape[2])


# (q heads, kv heads, q rows, kv rows, d): the block means of Q as the last workgroups of two launches over chunks (teams of two blocks)
# and of the single-read kernel at 256 and 512 threads (1 and 2 blocks a workgroup), odd counts and short last blocks
MEANS = [(4, 2, 1, 300, 128), (2, 2, 385, 513, 128), (6, 2, 1029, 4224, 64), (6, 3, 700, 16200, 128), (4, 4, 513, 32768, 128),
         (3, 3, 129, 65536, 64), (16, 16, 641, 8192, 128)]


@pytest.mark.parametrize("hq,hkv,nq,nk,d", MEANS)
@pytest.mark.parametrize("path", [0, 2])
def test_block_means_beside_the_quantiser_equal_those_of_their_own_launch(hq, hkv, nq, nk, d, path):
    say(f"[block means] {hq}/{hkv} heads, {nq} x {nk} x {d}, quantiser path {path}")
    k, v = _inputs(2 if d == 128 else 4, (2, hkv, nk, d))
    q, _ = _inputs(5 if d == 128 else 3, (2, hq, nq, d))
    q = q.to(k.dtype)
    sage.diag_quant_kv_path(THREE_LAUNCHES)
    want = sage.sage_attn_fwd_4bit(q, k, v, causal=False)
    sage.diag_quant_kv_path(path)
    got = sage.sage_attn_fwd_4bit(q, k, v, causal=False)
    assert torch.equal(want.view(torch.int16), got.view(torch.int16))


# V alone, heads x tokens on both sides of the lines: one workgroup per CU, the most partials beyond it, the single read's reach
V_ROUTES = [(2, 32731, 128, True), (2, 32769, 128, False), (4, 24539, 128, True), (4, 24700, 128, False), (2, 65499, 128, False),
            (1, 65499, 128, True), (1, 131035, 128, True), (4, 65499, 64, True), (3, 70000, 64, False), (2, 65500, 64, True),
            (2, 131035, 64, False), (1, 262107, 64, True)]


@pytest.mark.parametrize("H,N,d,chunks", V_ROUTES)
def test_v_alone_takes_chunks_where_they_pay_and_writes_the_same_bits(H, N, d, chunks):
    """A chunk leaves a partial per channel in the scratch; the single read leaves half as many there (its workgroups hold two chunks)."""
    say(f"[quant chunks] V alone {H} heads x {N} x {d}")
    g = torch.Generator(device="cuda").manual_seed(H + N)
    v = torch.randn(1, H, N, d, generator=g, device="cuda").to(torch.float16)
    sage.diag_quant_kv_path(THREE_LAUNCHES)
    want = sage.sage_quant_v(v)
    sage.diag_quant_kv_path(0)
    ws = torch.full((sage.quant_workspace_bytes(1, H, N, d),), 0x5A, dtype=torch.uint8, device="cuda")
    got = sage.sage_quant_v(v, workspace=ws)
    for a, b in zip(want, got):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    partials = -(-N // (256 if d == 128 else 512)) * H * d * 4
    assert (int((ws != 0x5A).sum()) > 0.75 * partials) == chunks


@pytest.mark.parametrize("H,N,chunks", [(8, 64, False), (64, 128, False), (8, 256, False), (8, 257, True), (64, 512, True), (65, 512, False)])
def test_k_of_heads_that_one_workgroup_holds(H, N, chunks):
    """K alone and with Q, d = 64: two launches from five K blocks on, before that one, which writes nothing to its scratch."""
    say(f"[quant chunks] K alone {H} heads x {N} x 64")
    g = torch.Generator(device="cuda").manual_seed(H + N)
    q, k = (torch.randn(1, H, N, 64, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    sage.diag_quant_kv_path(THREE_LAUNCHES)
    want = sage.sage_quant_k(k)
    sage.diag_quant_kv_path(0)
    for with_q in (False, True):
        ws = torch.full((sage.quant_workspace_bytes(1, H, N, 64),), 0x5A, dtype=torch.uint8, device="cuda")
        got = sage.sage_quant_qk(q, k, workspace=ws)[1::2] if with_q else sage.sage_quant_k(k, workspace=ws)
        for a, b in zip((want[0], want[1]), got):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
        assert bool((ws == 0x5A).all()) != chunks
