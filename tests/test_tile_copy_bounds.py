"""The attention kernels' tile copies (csrc/sage_attn.hip: issue_tile_piece, csrc/sage_prefill.hip: copy_piece, csrc/sage_spread.hip:
copy, csrc/sage_decode.hip: copy_half): the kernels' own per-lane offsets, descriptor sizes and places in LDS, compiled for the CPU from
csrc/sage_tile_copy.h, in models of each kernel's loop over pieces and wavefronts.  For every key step, piece, wavefront and lane, the
16-byte chunk a lane fetches must lie inside the head's K^ (V^) buffer of exactly Nk*D (ceil(Nk/128)*D*128) bytes, together the
fetched chunks must cover every byte of the tile's valid rows exactly once, and each must land in LDS where the kernel reads that
chunk (k_off, v_off: row major, the chunks of a row swizzled).  The hardware bounds check compares the per-lane offset with the
descriptor's size; the model applies the same rule to the same arithmetic, so a caller's buffer of exactly
B*H*Nk*d bytes is never overrun.  (The GPU tests show the values are right; this shows the addresses are.)"""
import numpy as np
import pytest

from tile_copy import addresses  # noqa: F401

LANES = np.arange(64)


# Each model yields (descriptor base, descriptor size, per-lane offsets, LDS offset of lane 0 within the tile's buffer).
def small_rows(a, head_bytes, D, j, is_v):
    """attn_kernel: four wavefronts, a descriptor per piece, piece k of wavefront w at 1 KB * (4 k + w)."""
    TILE = 128 * D
    for w in range(4):
        voff = a.source(is_v, D, w * 64 + LANES)
        for k in range(TILE // 4096):
            first = j * TILE + k * 4096
            yield first, a.copy_left(head_bytes, first), voff, (4 * k + w) * 1024


def prefill(a, head_bytes, D, j, is_v):
    """prefill_kernel: four wavefronts; d = 128: one descriptor per tile, the piece in the lane offsets (those of K^ for V^, too);
    d = 64: a descriptor per piece."""
    TILE = 128 * D
    for w in range(4):
        slot = w * 64 + LANES
        for k in range(TILE // 4096):
            if D == 128:
                first, voff = j * TILE, a.source(False, D, slot) + k * 4096
            else:
                first, voff = j * TILE + k * 4096, a.source(is_v, D, slot)
            yield first, a.copy_left(head_bytes, first), voff, w * 1024 + k * 4096


def spread(a, head_bytes, D, j, is_v):
    """spread_kernel: two wavefronts that take every other piece, one lane offset for all pieces."""
    TILE = 128 * D
    voff = a.source(is_v, D, LANES)
    for pw in range(2):
        for k in range(TILE // 2048):
            off = (2 * k + pw) * 1024
            first = j * TILE + off
            yield first, a.copy_left(head_bytes, first), voff, off


def decode(a, head_bytes, D, j, is_v):
    """decode_kernel: one wavefront, two half tiles with a descriptor each, the piece in the lane offsets (d = 128: those of K^)."""
    for part in (0, 1):
        first = a.half_first(D, j, part)
        for p in range(64 * D // 1024):
            yield first, a.copy_left(head_bytes, first), a.source(is_v and D == 64, D, LANES) + p * 1024, part * 64 * D + p * 1024


def fetched_chunks(a, model, head_bytes, D, j, is_v):
    """(source offsets in the head's buffer, LDS offsets in the tile's buffer) of the 16-byte chunks that step j's copy fetches."""
    src, dst = [], []
    for first, records, voff, lds in model(a, head_bytes, D, j, is_v):
        ok = voff + 16 <= records                                  # the hardware's range check
        src.append((first + voff)[ok])
        dst.append((lds + 16 * LANES)[ok])
    return np.concatenate(src).astype(np.int64), np.concatenate(dst).astype(np.int64)


@pytest.mark.parametrize("model", [small_rows, prefill, spread, decode])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Nk", [1, 5, 63, 64, 65, 127, 128, 129, 200, 255, 256, 600, 1000, 17776])
def test_tile_copies_stay_inside_the_buffer_and_cover_it(addresses, Nk, D, model):
    TILE = 128 * D
    nT = -(-Nk // 128)
    for is_v in (False, True):
        head_bytes = nT * TILE if is_v else Nk * D
        row_bytes = 128 if is_v else D
        for j in sorted({0, nT // 2, nT - 1}):
            src, dst = fetched_chunks(addresses, model, head_bytes, D, j, is_v)
            what = (model.__name__, is_v, Nk, D, j)
            assert src.size == 0 or (src.min() >= 0 and src.max() + 16 <= head_bytes), what
            # exactly the chunks of the tile's valid rows, each once
            lo, hi = j * TILE, min((j + 1) * TILE, head_bytes)
            assert np.array_equal(np.sort(src), np.arange(lo, hi, 16, dtype=np.int64)), what
            # where the operands are read from: row major, chunk c of a row at place c ^ swizzle(row)
            row, c = (src - lo) // row_bytes, (src - lo) % row_bytes // 16
            assert np.array_equal(dst, addresses.place(is_v, D, row, c)), what
