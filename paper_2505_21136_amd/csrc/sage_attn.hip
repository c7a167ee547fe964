// Stage 2 of the SageAttention2++ forward on gfx950: which kernel a call runs (launch_attn), and the fused attention kernel for
// up to 64 query rows per head (paper Sec. 2.1 for the tiling / online softmax and the scales, Sec. 3.1 for the bounded
// FP8 range P_r of P~).
//
// Mapping to CDNA4.  A workgroup of 4 wavefronts owns the (at most 64) query rows of one (batch, head) and, with key ranges, one
// range of the key steps; a wavefront owns 16 rows, so that calls with few rows multiply little padding.  Per
// step of 128 keys the K^ tile [128][D] int8 and the V^ tile [D][128] fp8 are
// copied global -> LDS by buffer loads that write LDS directly (no register
// staging; chunks beyond the end of a head's K^ are not fetched and read as zero), double buffered so that the copy of
// step j+1 runs under the arithmetic of step j, one barrier per step.
// 16-byte LDS chunks are XOR-swizzled against bank conflicts.
//   S^T = K^ Q^T   with v_mfma_i32_16x16x64_i8 (keys are MFMA rows, queries are
//                  MFMA columns).  A lane then holds, for ONE query (lane&15),
//                  the scores of keys 16t + 4(lane>>4) + i, t<8, i<4: the row
//                  maximum and sum are in-lane work plus two cross-lane steps.
//   softmax        base 2, FP32; the de-quantisation constant
//                  delta_Q*delta_K*sm_scale*log2(e) is one FMA operand (kept in
//                  a VGPR: FMAs with a scalar operand issue at half rate), the
//                  maximum is taken on the integer scores per 64-key K block;
//                  the INT32 accumulator starts at the bit pattern of 1.5*2^23,
//                  which makes its bits a valid binary32 number (no conversion).
//   P^             v_cvt_pk_fp8_f32 in registers: the 32 bytes a lane produces
//                  are exactly its B operand of v_mfma_f32_16x16x128_f8f6f4.
//   O^T += V^T P^T with that instruction (FP8 E4M3 both sides, FP32 accumulate;
//                  the older 16x16x32 fp8 MFMA runs at half its rate);
//                  V^ is stored transposed and key-permuted by the quantiser so
//                  that the A operand is two 16-byte LDS chunks read in the same
//                  conflict-free pattern as the K^ operand.
// The accumulator is rescaled only in steps where some row maximum moved
// (multiplying by alpha == 1 is the identity, so skipping is exact).
#include "sage_attn_device.h"
#include "sage_internal.h"

#include <limits.h>
#include <math.h>

namespace sage {
namespace {

// The same step for the 4+8 variant (INT4 codes, Q smoothed by its block means): the de-quantised score of a
// key gets the correction term ds = (qbar . K'[n]) * sm_scale * log2(e) added, which differs from key to key,
// so the step maximum is taken on the finished exponents x = c * S + ds (FP32) instead of on the integers:
// per score one conversion, one FMA, half a max3, one addition, one exp2, one addition, half an FP8 pack.
// s holds plain INT32 scores.  ds: this lane's 32 correction terms of the step (LDS), 8 x float4 in the order
// of its scores.
template <bool MASKED>
__device__ __forceinline__ float softmax_step_q4(const v4i (&s)[8], float c0, float c1, float log2_pr, float &m, float &l,
                                                 v8i &pb, int key_base, int lim, int t_lo, int t_hi,
                                                 const float4 *__restrict__ ds) {
    float mx0 = -INFINITY, mx1 = -INFINITY;
    float xf[8][4];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        bool live = true;
        if constexpr (MASKED) live = t < t_hi;
        if (live) {
            const float4 d4 = ds[t];
            const float dd[4] = {d4.x, d4.y, d4.z, d4.w};
            const float cb = t < 4 ? c0 : c1;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int sv = s[t][i];
                float x = __builtin_fmaf((float)sv, cb, dd[i]);
                if constexpr (MASKED) {
                    if (t >= t_lo && key_base + 16 * t + i > lim) x = -INFINITY;
                }
                xf[t][i] = x;
                if (i < 2) mx0 = fmaxf(mx0, x); else mx1 = fmaxf(mx1, x);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) xf[t][i] = -INFINITY;
        }
        // (keeps the compiler from fetching all 32 correction terms up front)
        if (t == 3) __builtin_amdgcn_sched_barrier(0);
    }
    const float mc = rowgroup_max(fmaxf(mx0, mx1));
    const float m_new = fmaxf(m, mc);
    const float alpha = __builtin_amdgcn_exp2f(m - m_new);
    const float mo = log2_pr - m_new;  // P~ * P_r = 2^(x - m' + log2 P_r)
    float lsum0 = -0.0f, lsum1 = -0.0f;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        if constexpr (MASKED) {
            if (t >= t_hi) {
                pb[t] = 0;
                continue;
            }
        }
        float p[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = __builtin_amdgcn_exp2f(xf[t][i] + mo);  // a masked key: 2^(-inf) = 0
        lsum0 += p[0] + p[1];
        lsum1 += p[2] + p[3];
        int w;  // both halves are overwritten below
        asm volatile("" : "=v"(w));
        w = __builtin_amdgcn_cvt_pk_fp8_f32(p[0], p[1], w, false);
        w = __builtin_amdgcn_cvt_pk_fp8_f32(p[2], p[3], w, true);
        pb[t] = w;
    }
    l = l * alpha + (lsum0 + lsum1);
    m = m_new;
    return alpha;
}

#if defined(__HIP_DEVICE_COMPILE__)
// Enqueue piece k of wavefront w's share of the global -> LDS copy of one [128 x D]-byte tile (K^ or V^) of key step j.  A tile is
// copied by the 4 wavefronts of the workgroup; a piece (one buffer load) moves 16 bytes per
// lane straight into LDS at dst + 1024*(4*k + w) + 16*lane; the per-lane source offset carries the
// swizzle.  Every piece gets a buffer descriptor of its own whose base is the piece's first byte and whose
// size is what is left of the head's buffer from there (scalar arithmetic only): the hardware bounds check
// covers the per-lane offset but not a scalar offset, and this way a 16-byte chunk beyond the last byte of
// the buffer (rows >= Nk of the last K^ tile) is never fetched and reads as zero.
template <int D>
__device__ __forceinline__ void issue_tile_piece(uint8_t *dst, const uint8_t *head, int head_bytes, int voff, int w,
                                                 int k, int j) {
    constexpr int TILE = 128 * D;
    // (piece k of a wavefront lies 4 KB after piece 0 on both sides: the swizzles repeat every 8 rows)
    const int first = j * TILE + k * 4096;
    lds_copy16(lds_copy_rsrc(head + first, copy_left(head_bytes, first)), voff, lds_address(dst) + (4 * k + w) * 1024);
}
#endif  // __HIP_DEVICE_COMPILE__

// Wavefronts per SIMD the register budget is set for: LDS holds two workgroups per CU at d = 128, four at d = 64.
template <int D>
constexpr int attn_waves_per_simd() {
    return D == 128 ? 2 : 4;
}

// QRAW: Q arrives unquantised (16-bit, the output's type) and the workgroup, whose rows are the head's whole
// Q quantisation block, quantises it in its prologue (paper Sec. 2.1: per-block INT8,
// delta = max|Q| / 127) with the same binary32 operations as the stand-alone quantiser, so codes
// and scale are the same bits; Q^ and delta_Q then never touch memory.
//
// Q4 (with QRAW): the 4+8 variant.  K^ holds INT4 codes (one per byte, same INT8 MFMA), Q is smoothed by the
// block means `q_mean` before its INT4 quantisation (delta = max|Q - qbar| / 7), and the score correction
// `dsx` (see softmax_step_q4) is added in the softmax part; everything else is shared with the 8+8 kernel.
//
// SPLIT (with QRAW, without Q4): the key steps are cut into `n_splits` ranges of `steps_per_split` steps and the
// grid holds one workgroup per (head, range).  A workgroup runs the recurrence on its range alone, from
// m = -inf, l = 0, acc = 0, and instead of O writes the range's (m, l, acc) of every row to `part_ml` / `part_acc`
// ([head][range][128 rows][2] and [...][D] floats, as prefill_kernel does); merge_kernel (sage_decode.hip)
// combines the ranges.
//
// Why the 4+8 variant and the ranges exist here and not only in prefill_kernel: with at most 64 rows two of that kernel's four
// wavefronts have none and the others make 32 rows each, twice the chain of 16.  Measured, us, here / there: 4+8, 32 / 8 heads,
// 33 rows, 4096 keys 46.6 / 59.1 (d 64: 37.9 / 50.5), 512 heads x 64 rows 64.0 / 95.8 (46.6 / 76.3); ranges and their
// combination, 64 / 8 heads x 16 rows, 32768 keys 48.3 / 55.7 (38.1 / 46.7), 32 / 8 heads x 48 rows 36.5 / 48.8 (28.4 / 42.0).
// What bounds it is that chain (matrix part, then softmax part of one step, in one wavefront) where a SIMD has one wavefront,
// and the vector issue port with more.
template <int D, bool CAUSAL, bool BF16, bool QRAW, bool Q4, bool SPLIT>
__global__ __launch_bounds__(256, (attn_waves_per_simd<D>())) void attn_kernel(
    const void *__restrict__ Qsrc, const int8_t *__restrict__ Kc, const uint8_t *__restrict__ Vt,
    const float *__restrict__ dq, const float *__restrict__ dk, const float *__restrict__ dv,
    uint16_t *__restrict__ out, Strides q_st, Strides o_st, int Nq, int Nk, int nT, int nKblk, int Hq,
    int group, float sm_scale, float log2_pr, const float *__restrict__ q_mean, const float *__restrict__ dsx,
    int n_splits, int steps_per_split, float *__restrict__ part_acc, float *__restrict__ part_ml) {
    static_assert(!Q4 || QRAW, "the 4+8 variant quantises Q in the kernel");
    static_assert(!SPLIT || (QRAW && !Q4), "key ranges: unquantised Q, 8+8");
#if defined(__HIP_DEVICE_COMPILE__)  // the body uses device-only types; the host pass only needs the stub
    constexpr int NWAVE = kSmallRows / 16;
    constexpr int KC = D / 64;           // 64-wide contraction chunks of Q.K^T
    constexpr int CT = D / 16;           // 16-channel tiles of the output
    constexpr int TILE = 128 * D;        // bytes of one K^ (or V^) tile
    constexpr int NP = TILE / 4096;      // 1 KB pieces of a tile that a wavefront copies
    __shared__ __attribute__((aligned(1024))) uint8_t ldsK[2][TILE];
    __shared__ __attribute__((aligned(1024))) uint8_t ldsV[2][TILE];
    __shared__ float q_wave_max[NWAVE];
    // per wavefront: the de-quantisation constants (c, kh, kl, -) of 64 consecutive K blocks (32 key steps)
    __shared__ __attribute__((aligned(16))) float4 cst_lds[NWAVE][64];
    // 4+8 variant: the score-correction terms of a key step (128 floats, lane order), even and odd steps
    __shared__ __attribute__((aligned(16))) float ds_lds[2][Q4 ? 128 : 1];
    __shared__ __attribute__((aligned(16))) float dv_lds[D];  // delta_V of this head, for the epilogue

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lq = lane & 15, g = lane >> 4;
    int bh, split = 0;  // (batch, query head), key range
    if constexpr (SPLIT) {
        // the ranges of a head are adjacent workgroup ids
        split = (int)blockIdx.x % n_splits;
        bh = (int)blockIdx.x / n_splits;
    } else {
        int tile;  // one per head; the query heads of a K/V head stay on one XCD
        map_workgroup<false>((int)blockIdx.x, (int)gridDim.x, 1, bh, tile);
    }
    const int row0 = wave * 16;
    // grouped-query attention: `group` consecutive query heads share one K/V head
    const int bhk = (bh / Hq) * (Hq / group) + (bh % Hq) / group;
    // causal mask aligned to the end of both sequences: key n visible to query r iff n <= r + shift
    const int shift = Nk - Nq;

    // this head's K^ [Nk][D] and V^ [nT][D][128] and their sizes in bytes (the tile copies are bounded to them)
    const uint8_t *Kh = reinterpret_cast<const uint8_t *>(Kc) + (size_t)bhk * Nk * D;
    const uint8_t *Vh = Vt + (size_t)bhk * nT * D * 128;
    const int k_bytes = Nk * D, v_bytes = nT * D * 128;

    // per-lane source offsets of this wavefront's piece 0 (the LDS side is linear in the lane index)
    const int k_voff = k_source<D>(wave * 64 + lane), v_voff = v_source(wave * 64 + lane);

    // key steps [jb, nsteps) of this workgroup (jb = 0 unless SPLIT)
    int nsteps = nT;
    if constexpr (CAUSAL) nsteps = min(nT, (Nq - 1 + shift) / kW + 1);
    const int jb = SPLIT ? split * steps_per_split : 0;
    if constexpr (SPLIT) nsteps = max(jb, min(nsteps, jb + steps_per_split));  // (empty when the range lies above the rows)
    // steps this wavefront takes part in (causal: tiles entirely above its rows are skipped)
    int my_steps = nsteps;
    if constexpr (CAUSAL) my_steps = min(nsteps, (row0 + 15 + shift) / kW + 1);
    if (row0 >= Nq) my_steps = jb;  // a wavefront without a valid row only takes part in the copies and barriers

    const auto copy_k = [&](int j) {
        if (j < nsteps) {
#pragma unroll
            for (int k = 0; k < NP; ++k) issue_tile_piece<D>(ldsK[j & 1], Kh, k_bytes, k_voff, wave, k, j);
        }
    };
    const auto copy_v = [&](int j) {
        if (j < nsteps) {
#pragma unroll
            for (int k = 0; k < NP; ++k) issue_tile_piece<D>(ldsV[j & 1], Vh, v_bytes, v_voff, wave, k, j);
        }
    };
    // 4+8 variant: the correction terms of the head's Q block, [nT][128] floats; the first wavefront copies those of step j
    const auto copy_ds = [&](int j) {
        if constexpr (Q4) {
            if (wave == 0 && j < nsteps) {
                const v4i r = lds_copy_rsrc(dsx + ((size_t)bh * nT + j) * 128, 512);
                lds_copy4(r, lane * 4, lds_address(&ds_lds[j & 1][0]));
                lds_copy4(r, 256 + lane * 4, lds_address(&ds_lds[j & 1][64]));
            }
        }
    };
    copy_k(jb);
    copy_ds(jb);

    // the lane's B operand of S^T = K^ Q^T: 16 consecutive channels (64*ch + 16*g ..) of query row lq
    v4i qreg[KC];
    uint4 qraw[KC][2];  // QRAW: the same 16 channels as 16-bit values
    const int qrow = row0 + lq;
    // 4+8 variant: the Q values minus the block's means (one binary32 subtraction, as the quantiser does)
    const auto q_values = [&](int ch, int h, float (&f)[8]) {
        unpack8<BF16>(qraw[ch][h], f);
        if constexpr (Q4) {
            const float *qm = q_mean + (size_t)bh * D + ch * 64 + g * 16 + h * 8;
            const float4 ma = *reinterpret_cast<const float4 *>(qm), mb = *reinterpret_cast<const float4 *>(qm + 4);
            const float mu[8] = {ma.x, ma.y, ma.z, ma.w, mb.x, mb.y, mb.z, mb.w};
#pragma unroll
            for (int i = 0; i < 8; ++i) f[i] = f[i] - mu[i];
        }
    };
    if constexpr (QRAW) {
        const uint16_t *Qr = static_cast<const uint16_t *>(Qsrc) + (bh / Hq) * q_st.b + (bh % Hq) * q_st.h + qrow * q_st.n;
        float amax = 0.0f;
#pragma unroll
        for (int ch = 0; ch < KC; ++ch)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                qraw[ch][h] = qrow < Nq ? *reinterpret_cast<const uint4 *>(Qr + ch * 64 + g * 16 + h * 8)
                                        : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
        for (int ch = 0; ch < KC; ++ch)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float f[8];
                q_values(ch, h, f);
                if (qrow < Nq) {  // (a missing row would contribute its mean)
#pragma unroll
                    for (int i = 0; i < 8; ++i) amax = fmaxf(amax, fabsf(f[i]));
                }
            }
        amax = wave_max(amax);
        if (lane == 0) q_wave_max[wave] = amax;
    } else {
        const int8_t *Qr = static_cast<const int8_t *>(Qsrc) + (bh / Hq) * q_st.b + (bh % Hq) * q_st.h + qrow * q_st.n;
#pragma unroll
        for (int ch = 0; ch < KC; ++ch) {
            v4i z = {0, 0, 0, 0};
            qreg[ch] = qrow < Nq ? *reinterpret_cast<const v4i *>(Qr + ch * 64 + g * 16) : z;
        }
    }
    // (the 4+8 variant converts its scores explicitly: plain INT32 accumulators)
    constexpr int kInit = Q4 ? 0 : kMagic;
    const v4i cinit = {kInit, kInit, kInit, kInit};

    // the output scales are fetched now and parked in LDS: the epilogue then waits for no global load
    if (tid < D / 4)
        *reinterpret_cast<float4 *>(dv_lds + 4 * tid) = *reinterpret_cast<const float4 *>(dv + (size_t)bhk * D + 4 * tid);
    __syncthreads();

    float delta_q;
    if constexpr (QRAW) {
        const float a = fmaxf(fmaxf(q_wave_max[0], q_wave_max[1]), fmaxf(q_wave_max[2], q_wave_max[3]));
        constexpr float kRange = Q4 ? 7.0f : 127.0f;
        const float rcp = a > 0.0f ? kRange / a : 0.0f;
        delta_q = a / kRange;
#pragma unroll
        for (int ch = 0; ch < KC; ++ch)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float f[8];
                q_values(ch, h, f);
                const uint2 w = int8_codes(f, rcp);
                qreg[ch][2 * h] = (int)w.x;
                qreg[ch][2 * h + 1] = (int)w.y;
            }
    } else {
        delta_q = dq[bh];
    }
    const double cq = (double)delta_q * (double)sm_scale * 1.4426950408889634;

    float m = -INFINITY, l = 0.0f, alpha = 1.0f;
    v4f o[CT];
    v4i s[8];
    v8i pb = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) o[ct] = v4f{0.f, 0.f, 0.f, 0.f};

    // O^T += V^T P^T of step j (FP8 E4M3 x E4M3, FP32 accumulation); O is rescaled only when some running maximum moved
    const auto add_pv = [&](int j) {
        if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) o[ct] *= alpha;
        }
        const uint8_t *Vs = ldsV[j & 1];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            const int row = 16 * ct + lq;
            const v4i lo = *reinterpret_cast<const v4i *>(Vs + v_off(row, g));
            const v4i hi = *reinterpret_cast<const v4i *>(Vs + v_off(row, 4 + g));
            const v8i a = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            o[ct] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, pb, o[ct], 0, 0, 0, 0, 0, 0);
        }
    };
    // S^T = K^ Q^T of step j (INT8, INT32 accumulation onto the float-view bias); contraction chunk outermost: consecutive
    // MFMAs never depend on each other
    const auto make_scores = [&](int j) {
        const uint8_t *Ks = ldsK[j & 1];
#pragma unroll
        for (int ch = 0; ch < KC; ++ch) {
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const v4i a = *reinterpret_cast<const v4i *>(Ks + k_off<D>(16 * t + lq, 4 * ch + g));
                s[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, qreg[ch], ch == 0 ? cinit : s[t], 0, 0, 0);
            }
        }
    };
    const auto softmax = [&](int j) {
        const int key0 = j * kW;
        // de-quantisation constants of the two K blocks of this step: every 32 steps each lane computes the
        // constants of one K block (c, and the exact split -K*c = kh + kl) and parks them in this wavefront's own
        // strip of LDS; a step then fetches its two blocks with two broadcast reads and no vector arithmetic
        if ((j & 31) == 0 || (SPLIT && j == jb)) {
            const int blk = min(64 * (j >> 5) + lane, nKblk - 1);
            const float c = (float)(cq * (double)dk[(size_t)bhk * nKblk + blk]);
            const float kh = -kMagicF * c;
            cst_lds[wave][lane] = make_float4(c, kh, __builtin_fmaf(-kMagicF, c, -kh), 0.0f);
        }
        const float4 k0 = cst_lds[wave][(2 * j) & 63], k1 = cst_lds[wave][(2 * j + 1) & 63];
        const float c0 = k0.x, c1 = k1.x, kh0 = k0.y, kh1 = k1.y, kl0 = k0.z, kl1 = k1.z;
        const float4 *ds = reinterpret_cast<const float4 *>(&ds_lds[j & 1][Q4 ? 32 * g : 0]);
        if ((key0 + kW > Nk) || (CAUSAL && key0 + kW - 1 > row0 + shift)) {
            int lim = Nk - 1;  // last visible key of this lane's query row
            if constexpr (CAUSAL) lim = min(lim, qrow + shift);
            // last visible key of the wavefront's first / last row: 16-key tiles wholly at or below the former
            // need no mask, tiles wholly above the latter are invisible
            const int lim_min = CAUSAL ? min(Nk - 1, row0 + shift) : Nk - 1;
            const int lim_max = CAUSAL ? min(Nk - 1, row0 + 15 + shift) : Nk - 1;
            const int t_lo = min(8, max(0, (lim_min - key0 + 1) >> 4));
            const int t_hi = min(8, max(0, ((lim_max - key0) >> 4) + 1));
            if constexpr (Q4) {
                alpha = softmax_step_q4<true>(s, c0, c1, log2_pr, m, l, pb, key0 + 4 * g, lim, t_lo, t_hi, ds);
            } else {
                const float l_old = l;
                alpha = softmax_step<true>(s, c0, c1, kh0, kh1, kl0, kl1, log2_pr, m, l, pb, key0 + 4 * g, lim, t_lo, t_hi);
                if constexpr (SPLIT) {
                    // a row that has seen no key of this range yet and sees none in this step keeps its empty
                    // state (the step's arithmetic on (-inf) - (-inf) is undefined; its P^ is zero either way);
                    // without ranges every row sees key 0 in its first step
                    if (lim < key0 && m == -INFINITY) {
                        alpha = 1.0f;
                        l = l_old;
                    }
                }
            }
        } else {
            if constexpr (Q4)
                alpha = softmax_step_q4<false>(s, c0, c1, log2_pr, m, l, pb, 0, 0, 8, 8, ds);
            else
                alpha = softmax_step<false>(s, c0, c1, kh0, kh1, kl0, kl1, log2_pr, m, l, pb, 0, 0, 8, 8);
        }
    };

    // Iteration j adds P^V^ of step j-1 and makes scores and P^ of step j.  It starts with a barrier: K^(j) and V^(j-1) have landed
    // for every wavefront, and the buffers of K^(j-1) and V^(j-2) have no reader left, so the copies of K^(j+1) and V^(j) may start.
    for (int j = jb; j <= nsteps; ++j) {
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wavefront's pieces have landed
        __syncthreads();
        copy_k(j + 1);
        copy_ds(j + 1);
        copy_v(j);
        if (j > jb && j <= my_steps) add_pv(j - 1);
        if (j < my_steps) {
            make_scores(j);
            // (ahead of a wavefront of another workgroup that wants the issue port for its matrix part: 512 heads x 33 rows, 4096 keys,
            // d 128, 52.7 -> 48.9 us, d 64 43.0 -> 40.2; with few heads, where nobody else is on the SIMD, 1-2 % slower)
            __builtin_amdgcn_s_setprio(1);
            softmax(j);
            __builtin_amdgcn_s_setprio(0);
        }
    }

    if constexpr (SPLIT) {
        // ---- the range's (m, l, acc) of every valid row; l is the sum over the row's four lanes ----
        const float lsum = rowgroup_sum(l);
        if (qrow < Nq) {
            const size_t prow = ((size_t)bh * n_splits + split) * kBQ + qrow;
            if (g == 0) *reinterpret_cast<float2 *>(part_ml + prow * 2) = make_float2(m, lsum);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
                *reinterpret_cast<float4 *>(part_acc + prow * D + 16 * ct + 4 * g) =
                    make_float4(o[ct][0], o[ct][1], o[ct][2], o[ct][3]);
        }
        return;
    }
    // ---- epilogue: O = acc * delta_V / (P_r * l); l already carries the factor P_r ----
    const float inv = 1.0f / rowgroup_sum(l);
    if (qrow < Nq) {
        uint16_t *orow = out + (bh / Hq) * o_st.b + (bh % Hq) * o_st.h + qrow * o_st.n;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            const int c = 16 * ct + 4 * g;
            const float4 sc = *reinterpret_cast<const float4 *>(dv_lds + c);
            const float y0 = o[ct][0] * (sc.x * inv), y1 = o[ct][1] * (sc.y * inv);
            const float y2 = o[ct][2] * (sc.z * inv), y3 = o[ct][3] * (sc.w * inv);
            *reinterpret_cast<uint2 *>(orow + c) = make_uint2(pack2<BF16>(y0, y1), pack2<BF16>(y2, y3));
        }
    }
#endif  // __HIP_DEVICE_COMPILE__
}

// Up to kSmallRows query rows per head; part_acc != NULL: key ranges on separate workgroups (see attn_kernel).
template <int D>
hipError_t launch_small(const void *q, bool q_raw, Strides q_st, const int8_t *k_i8, const uint8_t *v_fp8, const float *q_scale,
                        const float *k_scale, const float *v_scale, void *out, Strides o_st, int B, int Hq, int Hkv, int Nq,
                        int Nk, bool causal, float sm_scale, float log2_pr, bool bf16, hipStream_t stream, const float *q_mean,
                        const float *dsx, int n_splits, int steps_per_split, float *part_acc, float *part_ml) {
    const dim3 grid(B * Hq * n_splits);
    const int nT = cdiv(Nk, kW), nK = cdiv(Nk, kBK);
    uint16_t *o16 = static_cast<uint16_t *>(out);
    const bool q4 = dsx != nullptr, ranges = part_acc != nullptr;
#define SAGE_LAUNCH(C, BF, QR, F4, SP)                                                                                    \
    attn_kernel<D, C, BF, QR, F4, SP><<<grid, 256, 0, stream>>>(                                                           \
        q, k_i8, v_fp8, q_scale, k_scale, v_scale, o16, q_st, o_st, Nq, Nk, nT, nK, Hq, Hq / Hkv, sm_scale, log2_pr,       \
        q_mean, dsx, n_splits, steps_per_split, part_acc, part_ml)
#define SAGE_LAUNCH_Q(C, BF)                                    \
    do {                                                        \
        if (ranges) SAGE_LAUNCH(C, BF, true, false, true);      \
        else if (q4) SAGE_LAUNCH(C, BF, true, true, false);     \
        else if (q_raw) SAGE_LAUNCH(C, BF, true, false, false); \
        else SAGE_LAUNCH(C, BF, false, false, false);           \
    } while (0)
    if (causal) {
        if (bf16) SAGE_LAUNCH_Q(true, true); else SAGE_LAUNCH_Q(true, false);
    } else {
        if (bf16) SAGE_LAUNCH_Q(false, true); else SAGE_LAUNCH_Q(false, false);
    }
#undef SAGE_LAUNCH_Q
#undef SAGE_LAUNCH
    return hipGetLastError();
}

}  // namespace

hipError_t launch_attn(const void *q, bool q_raw, Strides q_st, const int8_t *k_i8, const uint8_t *v_fp8,
                       const float *q_scale, const float *k_scale, const float *v_scale, void *out, Strides o_st, int B,
                       int Hq, int Hkv, int Nq, int Nk, int d, bool causal, float sm_scale, float p_r, bool bf16,
                       hipStream_t stream, const float *q_mean, const float *dsx, int n_splits, int steps_per_split,
                       float *part_acc, float *part_ml) {
    if (Nq <= kSmallRows) {
        const float log2_pr = (float)log2((double)p_r);
#define SAGE_SMALL(D)                                                                                                           \
    launch_small<D>(q, q_raw, q_st, k_i8, v_fp8, q_scale, k_scale, v_scale, out, o_st, B, Hq, Hkv, Nq, Nk, causal, sm_scale,     \
                    log2_pr, bf16, stream, q_mean, dsx, n_splits, steps_per_split, part_acc, part_ml)
        return d == 128 ? SAGE_SMALL(128) : SAGE_SMALL(64);
#undef SAGE_SMALL
    }
    // Which kernel above kSmallRows rows: by how many workgroups the query rows make.  Up to one workgroup of 32 rows per CU, a key
    // step is spread over a workgroup's wavefronts (sage_spread.hip); then with 64 rows per workgroup, where there are more than two
    // key steps to shorten; beyond one of those per CU the CUs are filled better by whole steps per wavefront and two
    // workgroups of 128 rows each (sage_prefill.hip).  The bits of a row are the same.  Measured, us, spread 32 / spread 64 / prefill,
    // full attention, 1024 x 1024 rows x keys: 256 tiles of 32 rows, d 128 11.9 / 15.2 / 17.5, d 64 9.7 / 12.3 / 14.3; 512 tiles
    // 21.1 / 15.9 / 18.0 and 16.3 / 12.5 / 14.4; 1024 tiles 38.8 / 28.7 / 19.2 and 29.1 / 22.7 / 15.1.  1024 x 8192: 256 tiles
    // 45 / 60 / 92 and 39 / 54 / 79; 512 tiles 85 / 64 / 95 and 72 / 55 / 79; 1024 tiles 162 / 119 / 100 and 138 / 103 / 82.  512 tiles
    // over 128 keys 12.7 / 9.4 / 8.2 and 9.3 / 7.2 / 6.3, 256 keys 13.6 / 10.4 / 9.5 and 10.1 / 7.8 / 7.4, 512 keys 16.3 / 12.3 / 12.2
    // and 12.2 / 9.4 / 9.7.  The 4+8 variant and key ranges exist in the prefill kernel only.
    // Causal: a head's last tiles are its longest and start first, so a second tile of a CU is a short one and the lines move with how
    // short, Nq against Nk, and with what a tile costs besides its keys.  Rows = keys: 32 rows win up to 512 tiles of 32 from 4096 keys
    // on (384 tiles 27.2 / 32.5 / 49.5 and, d 64, 21.6 / 28.7 / 42.8; 512 tiles 29.5 / 32.6 / 49.7), with 2048 up to 450 (384 tiles 17.7 /
    // 20.1 / 28.5, 448 20.6 / 20.6), with 1024 up to 370 (288 tiles 11.4 / 13.9, 384 14.4 / 14.1), with 300 up to 256 (10.3 / 9.8 at 260);
    // 64 rows up to 512 tiles of 64 from 4096 on (320 tiles 41.0 / 34.4 / 50.3, 512 tiles 54.9 / 40.8 / 50.6, 768 tiles 80 / 62 / 54.5; 2 heads x
    // 16384 165 / 125 / 174), with 2048 up to 450 (320 tiles 28.2 / 20.6 / 28.8; 512 37.9 / 27.6 / 29.6), with 1024 up to 340 (320 tiles
    // 20.7 / 17.0 / 18.5, 384 22.7 / 19.4 / 18.8), with 700 not beyond 256 (308 tiles 18.3 / 15.8 / 14.8).  Nk = 4 Nq (1024 x 4096) as
    // full attention: 144 tiles of 64 40.7 / 32.7, 288 61 / 53.6 / 50.4.
    const long heads = (long)B * Hq, t32 = heads * cdiv(Nq, 32), t64 = heads * cdiv(Nq, 64);
    const auto rounds_fit = [&](long tiles, int tile_keys, int thirds) {
        return tiles <= kCUs || (causal && tiles <= 2 * kCUs && 3 * tiles * ((long)Nk + tile_keys) <= (long)thirds * kCUs * Nq);
    };
    const int row_groups = dsx || part_acc ? 0 : rounds_fit(t32, 5 * kW, 7) ? 1 : rounds_fit(t64, 8 * kW, 8) && Nk > 2 * kW ? 2 : 0;
    if (row_groups)
        return launch_spread(q, q_raw, q_st, k_i8, v_fp8, q_scale, k_scale, v_scale, out, o_st, B, Hq, Hkv, Nq, Nk, d,
                             causal, sm_scale, p_r, bf16, stream, row_groups);
    return launch_prefill(q, q_raw, q_st, k_i8, v_fp8, q_scale, k_scale, v_scale, out, o_st, B, Hq, Hkv, Nq, Nk, d, causal,
                          sm_scale, p_r, bf16, stream, q_mean, dsx, n_splits, steps_per_split, part_acc, part_ml);
}

}  // namespace sage
