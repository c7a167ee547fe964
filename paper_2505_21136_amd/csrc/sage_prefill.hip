// The fused attention kernel of the SageAttention2++ forward on gfx950 for calls with many query rows (paper
// Sec. 2.1 for the tiling, the online softmax and the scales, Sec. 3.1 for the bounded FP8 range P_r of P~).
//
// Mapping to CDNA4.  A workgroup of 4 wavefronts owns 128 query rows of one (batch, head) -- one Q quantisation
// block --, a wavefront 32 of them: the columns of the 32x32 MFMAs.  Two workgroups per CU at d = 128 (256 registers
// per thread, two wavefronts per SIMD), three at d = 64.
//   S^T = K^ Q^T   with v_mfma_i32_32x32x32_i8 (keys are MFMA rows): a lane holds, for ONE query (lane & 31), the
//                  scores of keys 32t + 8b + 4h + i (t, b, i < 4; h = lane >> 5), so the row maximum and sum are
//                  in-lane work plus one exchange of the wavefront's halves.
//   softmax        base 2, FP32: the quantities of softmax_step (sage_attn_device.h), but converted scores instead of biased ones, so
//                  that an exponent is one FMA, rounded once, where softmax_step rounds twice: weights differ in their last binary32
//                  bits, single FP8 weights and with them outputs by what one such rounding decides.
//   P^             v_cvt_pk_fp8_f32 in registers: the 32 bytes of 64 keys are the lane's B operand of
//   O^T += V^T P^T v_mfma_f32_32x32x64_f8f6f4 (FP8 E4M3 both sides, FP32 accumulation).
// K^ and V^ tiles of 128 keys are copied global -> LDS by buffer loads that write LDS directly, double buffered,
// 16-byte chunks XOR-swizzled against bank conflicts (with a period of 8 rows, which leaves the 32-row operand reads two-way
// conflicts: 128 of 388 LDS cycles per step; LDS is 17 % busy and hardly waited for).
//
// Schedule.  What bounds the kernel is the issue of vector instructions and, at d = 128, the power the chip may draw (the clock
// floats: 2.07 GHz with d = 128, 2.2 to 2.3 with d = 64, of 2.4).  Per score one conversion, one FMA, one addition, one exponential, half an FP8 pack, half a
// max3; 389 vector instructions per step of 64 scores per lane at d = 128 (1 head x 32768 x 24), 386 at d = 64, causal rows of 4096 keys 477, the
// difference being the rescaling of O.  Measured with single instructions on every SIMD: two wavefronts issue one instruction each per 4
// cycles if one of them is an FP32 add, multiply or FMA (or a move or an integer addition); conversions and maxima take 4 alone or beside one of those; an
// exponential or an FP8 pack takes 8 and nothing issues beside it, nor while the matrix pipe works on an MFMA.  A
// wavefront's matrix work
// therefore runs INSIDE its own vector work, software-pipelined over the key steps: while the scores of step j turn
// into P^, the freed score registers already receive Q K^T of step j+1, and the P^ V^ product of step j-1 runs under
// the maximum and the first exponentials of step j.  The step is cut into slots of about 18 vector instructions with
// one or two MFMAs each (sched_barrier keeps the compiler from moving work between slots): a wavefront that
// issues an MFMA while the matrix pipe is busy waits, and nothing behind it can issue.  One barrier per step.
// RAISE: left alone the wavefronts of a SIMD take turns, one's exponentials against another's additions, and next to nothing is issued
// together (64 scores of two wavefronts: 1657 cycles measured, 1664 if every instruction were issued alone).  With the priority raised around
// the exponentials and packs the rest of the two meets: 1344 cycles, with 16 MFMAs 1484 against 1781 (profiles/vector_issue_microbenchmark.hip).
// In this kernel, d = 64: 1904 -> 1821 cycles per step and SIMD at the same clock with the MFMAs behind the exponentials, and with them first
// thing in the raised part 24 heads x 16384 1282 -> 1233 us, 9 x 8192 171 -> 158; d = 128, 10 x 4480 rows 7 % less, full
// chip 1 % (the clock falls with every cycle saved).  raise_pays has the rule.
// The accumulator is rescaled only in steps after which some row maximum has moved (multiplying by 1 is the identity).
#include "sage_attn_device.h"
#include "sage_internal.h"

#include <limits.h>
#include <math.h>

namespace sage {
namespace {

typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));

// This lane's number, made on the spot: what seldom-run code (constants, masks, epilogue) derives from it then needs no
// register through the key loop.
__device__ __forceinline__ int lane_now() {
    int x;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(x));
    return x;
}

// Wavefronts per SIMD the register budget is set for: at d = 64 the accumulator is half as large and a third wavefront fits
// (B 16, H 16, N 777: 60.7 -> 57.0 us, B 2, H 32, N 8192: 906 -> 885 us with 2 -> 3); the 4+8 variant needs a few registers more.
template <int D, bool Q4>
constexpr int prefill_waves_per_simd() {
    return D == 128 || Q4 ? 2 : 3;
}

// QRAW: Q arrives unquantised and the workgroup quantises its block in the prologue (the stand-alone quantiser's binary32
// steps: same bits); Q^ and delta_Q then never touch memory.
// Q4 (with QRAW): the 4+8 variant.  K^ holds INT4 codes (one per byte), Q is smoothed by its block means `q_mean`, and the
// score correction `dsx` ((qbar . K'[n]) * sm_scale * log2(e), one float per key and Q block) is added to the scores: the
// maximum is taken on the finished exponents x = c * S + ds in FP32.
// RAISE: see above; masked steps and the 4+8 variant without.
// SPLIT (with QRAW, without Q4): the key steps are cut into `n_splits` ranges of `steps_per_split` steps and the grid holds
// one workgroup per (head, query tile, range), which runs the recurrence on its range alone and writes (m, l, acc) per row
// to `part_ml` / `part_acc` ([item][range][128 rows][2] and [...][D] floats); merge_kernel (sage_decode.hip) combines them.
template <int D, bool CAUSAL, bool BF16, bool QRAW, bool Q4, bool SPLIT, bool RAISE>
__global__ __launch_bounds__(256, (prefill_waves_per_simd<D, Q4>())) void prefill_kernel(
    const void *__restrict__ Qsrc, const int8_t *__restrict__ Kc, const uint8_t *__restrict__ Vt,
    const float *__restrict__ dq, const float *__restrict__ dk, const float *__restrict__ dv,
    uint16_t *__restrict__ out, Strides q_st, Strides o_st, int Nq, int Nk, int nT, int nQblk, int nKblk, int Hq,
    int group, float sm_scale, float log2_pr, const float *__restrict__ q_mean, const float *__restrict__ dsx,
    int n_splits, int steps_per_split, float *__restrict__ part_acc, float *__restrict__ part_ml) {
    static_assert(!Q4 || QRAW, "the 4+8 variant quantises Q in the kernel");
    static_assert(!SPLIT || (QRAW && !Q4), "key ranges: unquantised Q, 8+8");
#if defined(__HIP_DEVICE_COMPILE__)  // the body uses device-only types; the host pass only needs the stub
    constexpr int NWAVE = 4, BM = 32 * NWAVE;
    constexpr int KC = D / 32;              // 32-wide contraction chunks of Q.K^T
    constexpr int CT = D / 32;              // 32-channel tiles of the output
    constexpr int TILE = 128 * D;           // bytes of one K^ (or V^) tile
    constexpr int NP = TILE / (1024 * NWAVE);  // 1 KB pieces of a tile that a wavefront copies
    static_assert(BM == kBQ, "a workgroup owns exactly one Q quantisation block");
    // K^ tiles of even and odd steps, then V^ tiles of even and odd steps
    __shared__ __attribute__((aligned(1024))) uint8_t lds[4 * TILE];
    __shared__ float q_wave_max[NWAVE];
    // per wavefront: the de-quantisation constants of 64 consecutive K blocks (32 key steps)
    __shared__ __attribute__((aligned(16))) float cst_lds[NWAVE][64];
    __shared__ __attribute__((aligned(16))) float ds_lds[2][Q4 ? 128 : 1];
    __shared__ __attribute__((aligned(16))) float dv_lds[D];  // delta_V of this head, for the epilogue

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lq = lane & 31, h = lane >> 5;
    int bh, qtile, split = 0;
    if constexpr (SPLIT) {
        // the ranges of an item are adjacent workgroup ids
        split = (int)blockIdx.x % n_splits;
        bh = ((int)blockIdx.x / n_splits) / nQblk;
        qtile = ((int)blockIdx.x / n_splits) % nQblk;
    } else {
        map_workgroup<CAUSAL>((int)blockIdx.x, (int)gridDim.x, nQblk, bh, qtile);
    }
    const int row0 = qtile * BM + wave * 32;
    const int bhk = (bh / Hq) * (Hq / group) + (bh % Hq) / group;  // `group` consecutive query heads share a K/V head
    const int shift = Nk - Nq;  // causal: key n visible to query r iff n <= r + shift

    // this head's K^ [Nk][D] and V^ [nT][D][128] and their sizes in bytes (the tile copies are bounded to them)
    const uint8_t *Kh = reinterpret_cast<const uint8_t *>(Kc) + (size_t)bhk * Nk * D;
    const uint8_t *Vh = Vt + (size_t)bhk * nT * D * 128;
    const int k_bytes = Nk * D, v_bytes = nT * D * 128;

    // Per-lane source offsets within a tile of this wavefront's first piece (the LDS side is linear in the lane index); piece k
    // lies 4 KB after it on both sides, a whole number of swizzle periods.  At D = 128 the rows of both tiles are 128 bytes
    // and their swizzles the same, and each piece's offset has a register; at D = 64 a piece has a descriptor instead.
    constexpr int NVO = D == 128 ? NP : 1;
    int kvoff[NVO], vvoff_ = 0;
    {
        const int slot = wave * 64 + lane;
#pragma unroll
        for (int k = 0; k < NVO; ++k) kvoff[k] = k_source<D>(slot) + k * 4096;
        if constexpr (D != 128) vvoff_ = v_source(slot);
    }

    // key steps [jb, nsteps) of this workgroup (jb = 0 unless SPLIT)
    int nsteps = nT;
    if constexpr (CAUSAL) nsteps = min(Nk - 1, qtile * BM + BM - 1 + shift) / kW + 1;
    const int jb = SPLIT ? split * steps_per_split : 0;
    if constexpr (SPLIT) nsteps = max(jb, min(nsteps, jb + steps_per_split));  // (empty when the range lies above the rows)
    // steps this wavefront takes part in, and those of them before the first that needs a mask
    int my_steps = nsteps;
    if constexpr (CAUSAL) my_steps = min(nsteps, (row0 + 31 + shift) / kW + 1);
    if (row0 >= Nq) my_steps = jb;  // a wavefront without a valid row only takes part in the copies and barriers
    int full_steps = Nk / kW;
    if constexpr (CAUSAL) full_steps = min(full_steps, (row0 + shift + 1) / kW);
    full_steps = min(full_steps, my_steps);

    // Copy piece k of this wavefront of the K^ (V^) tile of step j.  The descriptor's base is the tile's (piece's) first byte
    // and its size what is left of the head's buffer from there, so a chunk beyond the last byte (rows >= Nk of the last K^
    // tile) is never fetched and reads as zero; a step the workgroup does not have gets size 0.
    const int lds_piece = lds_address(lds) + wave * 1024;
    const auto copy_piece = [&](const uint8_t *head, int bytes, int voff, int j, int dst, int k) {
        const int first = j * TILE + (D == 128 ? 0 : k * 4096), left = j < nsteps ? copy_left(bytes, first) : 0;
        lds_copy16(lds_copy_rsrc(head + first, left), voff, lds_piece + dst + k * 4096);
    };
    const auto copy_k = [&](int j, int k) { copy_piece(Kh, k_bytes, kvoff[D == 128 ? k : 0], j, (j & 1) * TILE, k); };
    const auto copy_v = [&](int j, int k) {
        copy_piece(Vh, v_bytes, D == 128 ? kvoff[D == 128 ? k : 0] : vvoff_, j, (2 + (j & 1)) * TILE, k);
    };
    // 4+8 variant: the correction terms of this Q block, [nT][128] floats; the first wavefront copies those of step j
    const auto copy_ds = [&](int j) {
        if constexpr (Q4) {
            if (wave == 0 && j < nsteps) {
                const float *src = dsx + (((size_t)bh * nQblk + qtile) * nT + j) * 128;
                const v4i r = lds_copy_rsrc(src, 512);
                lds_copy4(r, lane * 4, lds_address(&ds_lds[j & 1][0]));
                lds_copy4(r, 256 + lane * 4, lds_address(&ds_lds[j & 1][64]));
            }
        }
    };
    {
#pragma unroll
        for (int k = 0; k < NP; ++k) copy_k(jb, k);
        copy_ds(jb);
    }
    // the lane's B operand of S^T = K^ Q^T: 16 consecutive channels (32*ch + 16*h ..) of query row lq
    v4i qreg[KC];
    uint4 qraw[KC][2];  // QRAW: the same 16 channels as 16-bit values
    const int qrow = row0 + lq;
    if constexpr (QRAW) {
        // The wavefront's 32 rows come as whole rows (a load in the operand's layout, a row per lane, costs the texture path 64 cycles
        // instead of 16) and change lanes in LDS, in the wavefront's own strip of what will be the V^ buffers.  Rows past the end repeat
        // the last one, which is in the block, too.
        const uint16_t *Qh = static_cast<const uint16_t *>(Qsrc) + (bh / Hq) * q_st.b + (bh % Hq) * q_st.h;
        constexpr int RC = D / 8, SW = RC - 1;  // 16-byte chunks per row, and the swizzle's mask
        uint8_t *q_lds = lds + 2 * TILE + wave * (64 * D);
        uint4 rows[RC / 2];
#pragma unroll
        for (int x = 0; x < RC / 2; ++x) {
            const int e = 64 * x + lane;
            rows[x] = *reinterpret_cast<const uint4 *>(Qh + min(row0 + e / RC, Nq - 1) * q_st.n + e % RC * 8);
        }
#pragma unroll
        for (int x = 0; x < RC / 2; ++x) {
            const int e = 64 * x + lane, row = e / RC;
            *reinterpret_cast<uint4 *>(q_lds + row * D * 2 + ((e % RC ^ (row & SW)) << 4)) = rows[x];
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        float amax = 0.0f;
#pragma unroll
        for (int ch = 0; ch < KC; ++ch)
#pragma unroll
            for (int e = 0; e < 2; ++e)
                qraw[ch][e] = *reinterpret_cast<const uint4 *>(q_lds + lq * D * 2 + (((4 * ch + 2 * h + e) ^ (lq & SW)) << 4));
#pragma unroll
        for (int ch = 0; ch < KC; ++ch)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                float f[8];
                unpack8<BF16>(qraw[ch][e], f);
                if constexpr (Q4) {
                    // max |Q - qbar| over the valid rows (a missing row would contribute |qbar|)
                    const float *qm = q_mean + ((size_t)bh * nQblk + qtile) * D + ch * 32 + h * 16 + e * 8;
                    if (qrow < Nq) {
#pragma unroll
                        for (int i = 0; i < 8; ++i) amax = fmaxf(amax, fabsf(f[i] - qm[i]));
                    }
                } else {
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
            qreg[ch] = qrow < Nq ? *reinterpret_cast<const v4i *>(Qr + ch * 32 + h * 16) : z;
        }
    }
    // the output scales are fetched now and parked in LDS: the epilogue then waits for no global load
    if (tid < D / 4)
        *reinterpret_cast<float4 *>(dv_lds + 4 * tid) = *reinterpret_cast<const float4 *>(dv + (size_t)bhk * D + 4 * tid);
    const float *dkh = dk + (size_t)bhk * nKblk;
    const float dk_first = dkh[min(64 * (jb >> 5) + lane, nKblk - 1)];
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): K^(jb) has landed
    __syncthreads();
    // the first step's "P^ V^ of the step before" multiplies zeros: its V^ buffer must hold numbers
#pragma unroll
    for (int k = 0; k < TILE / 4096; ++k)
        *reinterpret_cast<uint4 *>(lds + (2 + ((jb + 1) & 1)) * TILE + k * 4096 + tid * 16) = make_uint4(0u, 0u, 0u, 0u);

    // (not before: the loads above would be waited for behind it)
#pragma unroll
    for (int k = 0; k < NP; ++k) copy_k(jb + 1, k);

    float delta_q;
    if constexpr (QRAW) {
        const float a = fmaxf(fmaxf(q_wave_max[0], q_wave_max[1]), fmaxf(q_wave_max[2], q_wave_max[3]));
        constexpr float kRange = Q4 ? 7.0f : 127.0f;
        const float rcp = a > 0.0f ? kRange / a : 0.0f;
        delta_q = a / kRange;
#pragma unroll
        for (int ch = 0; ch < KC; ++ch)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                float f[8];
                unpack8<BF16>(qraw[ch][e], f);
                if constexpr (Q4) {
                    const float *qm = q_mean + ((size_t)bh * nQblk + qtile) * D + ch * 32 + h * 16 + e * 8;
#pragma unroll
                    for (int i = 0; i < 8; ++i) f[i] = f[i] - qm[i];  // one binary32 subtraction, as the quantiser does
                }
                const uint2 w = int8_codes(f, rcp);
                qreg[ch][2 * e] = (int)w.x;
                qreg[ch][2 * e + 1] = (int)w.y;
            }
    } else {
        delta_q = dq[(size_t)bh * nQblk + qtile];
    }
    delta_q = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, delta_q)));
    // de-quantisation constants delta_Q * delta_K * sm_scale * log2(e): every 32 steps each lane computes that of one K block
    // and parks it in this wavefront's own strip of LDS, from which a step takes its two
    const auto park_constants = [&](int j) {
        // (the product is made each time: kept, it would cost registers of every lane)
        float f, sm;
        asm volatile("v_mov_b32 %0, %2\n\tv_mov_b32 %1, %3" : "=&v"(f), "=v"(sm) : "s"(delta_q), "s"(sm_scale));
        const double cq = (double)f * (double)sm * 1.4426950408889634;
        const int ln = lane_now();
        const int blk = min(64 * (j >> 5) + ln, nKblk - 1);
        cst_lds[wave][ln] = (float)(cq * (double)dkh[blk]);
    };
    cst_lds[wave][lane] = (float)((double)delta_q * (double)sm_scale * 1.4426950408889634 * (double)dk_first);

    // ---- state of the recurrence ----
    // (l is kept per key tile of a step, as the wavefronts of spread_kernel hold it, and every addition here has that kernel's
    // order: a row's bits must not depend on which of the two the number of heads selects)
    float m = -INFINITY, l[4] = {0.0f, 0.0f, 0.0f, 0.0f}, alpha = 1.0f;
    v16f o[CT];
    v16i s[4];
    v8i pb[2];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[ct][i] = 0.0f;
    pb[0] = v8i{0, 0, 0, 0, 0, 0, 0, 0};
    pb[1] = v8i{0, 0, 0, 0, 0, 0, 0, 0};
    const v16i zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};

    // LDS offsets of the operand chunks this lane reads: row lq of a 32-row tile, 16-byte chunk 2x + h, whose swizzled place is
    // that of chunk h xor 32x bytes (K^: x = ch; V^: x = 2*chunk + half).  `par` is the buffer parity of step j+1, which is
    // that of step j-1 too.
    const int kof0 = k_off<D>(lq, h), vof0 = D == 128 ? kof0 : v_off(lq, h);
    int par = ((jb + 1) & 1) * TILE;

    // operands of the n-th Q.K^T MFMA (key tile n / KC, chunk n % KC) of the tiles at `base`, and of the r-th P^V^ MFMA (64-key
    // chunk r / CT, channel tile r % CT)
    const auto read_k = [&](int base, int n) {
        return *reinterpret_cast<const v4i *>(lds + ((kof0 + base) ^ 32 * (n % KC)) + (n / KC) * 32 * D);
    };
    const auto read_v = [&](int base, int r) {
        const uint8_t *p = lds + 2 * TILE + (r % CT) * 32 * 128;
        const v4i lo = *reinterpret_cast<const v4i *>(p + ((vof0 + base) ^ 64 * (r / CT)));
        const v4i hi = *reinterpret_cast<const v4i *>(p + ((vof0 + base) ^ (64 * (r / CT) + 32)));
        return v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    };
    const auto mfma_qk = [&](v4i a, int n) {
        s[n / KC] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, qreg[n % KC], n % KC == 0 ? zero : s[n / KC], 0, 0, 0);
    };
    const auto mfma_pv = [&](v8i a, int r) {
        o[r % CT] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, pb[r / CT], o[r % CT], 0, 0, 0, 0, 0, 0);
    };
    const auto rescale = [&]() {
        if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) o[ct] *= alpha;
        }
    };

    // scores of the first step
    {
        const int base = (jb & 1) * TILE;
#pragma unroll
        for (int n = 0; n < 4 * KC; ++n) mfma_qk(read_k(base, n), n);
    }

    // ---- the arithmetic of a step, in pieces ----
    // Maximum over the scores of key tile t (MASKED: keys beyond this lane's limit count as minus infinity from here on; `lim`
    // is counted from this lane's first key of the step).  im: integer maxima, two chains per K block; fm: the 4+8 variant's,
    // whose scores become finished exponents here (ds: the step's correction terms).
    const auto max_tile = [&](auto masked, int t, int lim, float cb, const float *ds, int (&im)[4], float (&fm)[4])
                              __attribute__((always_inline)) {
        constexpr bool MASKED = decltype(masked)::value;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            if constexpr (Q4) {
                // position 32g' + 4t' + i of a tile is key 16t' + 4g' + i: here t' = 2t + (b >> 1), g' = 2(b & 1) + h
                const float4 d4 = *reinterpret_cast<const float4 *>(ds + 32 * (2 * (b & 1) + h) + 4 * (2 * t + (b >> 1)));
                const float dd[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int sv = s[t][4 * b + i];
                    float x = __builtin_fmaf((float)sv, cb, dd[i]);
                    if constexpr (MASKED) x = 32 * t + 8 * b + i > lim ? -INFINITY : x;
                    fm[2 * (t & 1) + (i & 1)] = fmaxf(fm[2 * (t & 1) + (i & 1)], x);
                    s[t][4 * b + i] = __builtin_bit_cast(int, x);
                }
            } else {
                if constexpr (MASKED) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (32 * t + 8 * b + i > lim) s[t][4 * b + i] = INT_MIN;
                }
                int &a = im[2 * (t >> 1) + (b & 1)];
                if (!(t & 1) && b < 2) {
                    a = imax3(s[t][4 * b], s[t][4 * b + 1], s[t][4 * b + 2]);
                    a = max(a, s[t][4 * b + 3]);
                } else {
                    a = imax3(a, s[t][4 * b], s[t][4 * b + 1]);
                    a = imax3(a, s[t][4 * b + 2], s[t][4 * b + 3]);
                }
            }
        }
    };
    // The row's new running maximum; alpha becomes the factor of this step.
    const auto new_max = [&](auto masked, float c0, float c1, const int (&im)[4], const float (&fm)[4])
                             __attribute__((always_inline)) {
        constexpr bool MASKED = decltype(masked)::value;
        float mc;
        if constexpr (Q4) {
            mc = fmaxf(fmaxf(fm[0], fm[1]), fmaxf(fm[2], fm[3]));
        } else {
            const int im0 = max(im[0], im[1]), im1 = max(im[2], im[3]);
            float mc0 = (float)im0 * c0, mc1 = (float)im1 * c1;
            if constexpr (MASKED) {
                mc0 = im0 == INT_MIN ? -INFINITY : mc0;
                mc1 = im1 == INT_MIN ? -INFINITY : mc1;
            }
            mc = fmaxf(mc0, mc1);
        }
        const float m_new = max_no_nan(m, halves_max(mc));
        alpha = __builtin_amdgcn_exp2f(m - m_new);
        return m_new;
    };
    // P^ of the four keys 32t + 8b + 4h .. + 3, and their share of the key tile's sum.  mo = log2 P_r - m.
    // `matrix` issues what the matrix pipe does meanwhile.
    const auto exp_quad = [&](auto masked, int t, int b, float cb, float mo, float &lsum0, float &lsum1, auto matrix)
                              __attribute__((always_inline)) {
        constexpr bool MASKED = decltype(masked)::value;
        constexpr bool UP = RAISE && !MASKED;
        float p[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int sbits = s[t][4 * b + i];
            p[i] = Q4 ? __builtin_bit_cast(float, sbits) + mo : __builtin_fmaf((float)sbits, cb, mo);
        }
        if constexpr (UP) {
            asm volatile("" : "+v"(p[0]), "+v"(p[1]), "+v"(p[2]), "+v"(p[3]));
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(1);
            matrix();
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            p[i] = __builtin_amdgcn_exp2f(p[i]);
            if constexpr (MASKED && !Q4) p[i] = s[t][4 * b + i] == INT_MIN ? 0.0f : p[i];
        }
        if constexpr (!UP) {
            lsum0 += p[0] + p[1];
            lsum1 += p[2] + p[3];
        }
        int w;  // both halves are overwritten below: an opaque undefined seed saves the v_mov of a zero
        asm volatile("" : "=v"(w));
        w = __builtin_amdgcn_cvt_pk_fp8_f32(p[0], p[1], w, false);
        w = __builtin_amdgcn_cvt_pk_fp8_f32(p[2], p[3], w, true);
        if constexpr (UP) {
            asm volatile("" : "+v"(w));
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(0);
            __builtin_amdgcn_sched_barrier(0);
            lsum0 += p[0] + p[1];
            lsum1 += p[2] + p[3];
        }
        // (pinned to their place: nothing else keeps the arithmetic from sinking to its use a step later)
        asm volatile("" : "+v"(w), "+v"(lsum0), "+v"(lsum1));
        pb[t >> 1][4 * (b & 1) + 2 * (t & 1) + (b >> 1)] = w;
        if constexpr (!UP) matrix();
    };

    // One key step without a mask: P^ of step j from its scores, with P^V^ of step j-1 and Q.K^T of step j+1 in between.
    const auto step = [&](int j) __attribute__((always_inline)) {
        constexpr std::false_type no_mask{};
        constexpr int NQK = 4 * KC, NPV = 2 * CT;
        // operands read ahead: VA P^V^ tiles, KA Q.K^T tiles (d = 64 has half as many of both, and 168 registers)
        constexpr int VA = D == 128 ? 2 : 1, KA = D == 128 ? 4 : 2;
        v8i vf[VA];
        v4i kf[KA];
#pragma unroll
        for (int r = 0; r < VA; ++r) vf[r] = read_v(par, r);
        const float2 cc = *reinterpret_cast<const float2 *>(&cst_lds[wave][(2 * j) & 63]);
        rescale();  // (by the factor of the step before, whose P^V^ follows now)

        // ---- maximum of the step, P^V^ of the first 64 keys of step j-1 in between ----
        int im[4] = {INT_MIN, INT_MIN, INT_MIN, INT_MIN};
        float fm[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            max_tile(no_mask, t, 0, t < 2 ? cc.x : cc.y, ds_lds[j & 1], im, fm);
            if (t < CT) {
                mfma_pv(vf[t % VA], t);
                if (t + VA < NPV) vf[t % VA] = read_v(par, t + VA);
            }
            if (t < NP) copy_v(j, t);
            __builtin_amdgcn_sched_barrier(0);
        }
        const float m_new = new_max(no_mask, cc.x, cc.y, im, fm);
        const float mo = log2_pr - m_new;  // P~ * P_r = 2^(x - m' + log2 P_r)
        float lsum0 = -0.0f, lsum1 = -0.0f;  // x + (-0) is x for every x: the first addition folds away
#pragma unroll
        for (int n = 0; n < KA; ++n) kf[n] = read_k(par, n);
        __builtin_amdgcn_sched_barrier(0);

        // ---- exponentials and FP8 codes, 16 slots of 4 scores; Q.K^T of step j+1 follows one tile behind ----
        constexpr int SPT = 4 / KC;  // slots per Q.K^T MFMA (1 at d = 128, 2 at d = 64)
#pragma unroll
        for (int sl = 0; sl < 16; ++sl) {
            // P^V^ of the last 64 keys of step j-1 in the slots of the first two tiles (their registers are rewritten by the
            // last two)
            constexpr int EVERY = 8 / CT;
            const bool pv = sl < 8 && sl % EVERY == EVERY - 1, qk = sl >= 4 && sl % SPT == 0;
            const int r = CT + sl / EVERY, n = (sl - 4) / SPT;
            exp_quad(no_mask, sl >> 2, sl & 3, sl < 8 ? cc.x : cc.y, mo, lsum0, lsum1, [&]() __attribute__((always_inline)) {
                if (pv) mfma_pv(vf[r % VA], r);
                if (qk) mfma_qk(kf[n % KA], n);
            });
            if ((sl & 3) == 3) {
                l[sl >> 2] = __builtin_fmaf(l[sl >> 2], alpha, lsum0 + lsum1);
                lsum0 = lsum1 = -0.0f;
            }
            if (pv && r + VA < NPV) vf[r % VA] = read_v(par, r + VA);
            if (qk && n + KA < NQK) kf[n % KA] = read_k(par, n + KA);
            if (sl < NP) copy_k(j + 2, sl);
            if (sl == NP) copy_ds(j + 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        // the last tile's Q.K^T
#pragma unroll
        for (int n = NQK - KC; n < NQK; ++n) mfma_qk(kf[n % KA], n);
        static_assert(KA <= KC, "the last tile's operands are all read ahead");
        m = m_new;
        if (((j + 1) & 31) == 0) park_constants(j + 1);
        __builtin_amdgcn_sched_barrier(0);
    };

    // A step with a mask (the causal diagonal, the ragged end: at most the last two of a wavefront), without the fine
    // interleaving.  Key tiles that no row of the wavefront sees (t >= t_hi) cost no arithmetic.
    const auto masked_step = [&](int j) __attribute__((always_inline)) {
        constexpr std::true_type mask{};
        const int key0 = j * kW;
#pragma unroll
        for (int k = 0; k < NP; ++k) copy_v(j, k);
#pragma unroll
        for (int k = 0; k < NP; ++k) copy_k(j + 2, k);
        copy_ds(j + 1);
        const float2 cc = *reinterpret_cast<const float2 *>(&cst_lds[wave][(2 * j) & 63]);
        rescale();
#pragma unroll
        for (int r = 0; r < 2 * CT; ++r) mfma_pv(read_v(par, r), r);
        const int ln = lane_now();
        int lim = Nk - 1;  // last visible key of this lane's row
        if constexpr (CAUSAL) lim = min(lim, row0 + (ln & 31) + shift);
        const bool blind = lim < key0;  // the row sees no key of this step
        lim -= key0 + 4 * (ln >> 5);
        const int lim_max = CAUSAL ? min(Nk - 1, row0 + 31 + shift) : Nk - 1;
        const int t_hi = min(4, ((lim_max - key0) >> 5) + 1);
        int im[4] = {INT_MIN, INT_MIN, INT_MIN, INT_MIN};
        float fm[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (t < t_hi) max_tile(mask, t, lim, t < 2 ? cc.x : cc.y, ds_lds[j & 1], im, fm);
        const float m_new = new_max(mask, cc.x, cc.y, im, fm);
        const float mo = log2_pr - m_new;
        // a row that has seen no key of this range yet and sees none in this step keeps its empty state (the step's arithmetic on
        // (-inf) - (-inf) is undefined; its P^ is zero either way); without ranges every row sees key 0
        if constexpr (SPLIT) alpha = blind && m == -INFINITY ? 1.0f : alpha;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            float lsum0 = -0.0f, lsum1 = -0.0f;
            if (t < t_hi) {
#pragma unroll
                for (int b = 0; b < 4; ++b) exp_quad(mask, t, b, t < 2 ? cc.x : cc.y, mo, lsum0, lsum1, []() {});
            } else {
#pragma unroll
                for (int b = 0; b < 4; ++b) pb[t >> 1][4 * (b & 1) + 2 * (t & 1) + (b >> 1)] = 0;
            }
            l[t] = __builtin_fmaf(l[t], alpha, lsum0 + lsum1);
        }
        if (j + 1 < my_steps) {
#pragma unroll
            for (int n = 0; n < 4 * KC; ++n) mfma_qk(read_k(par, n), n);
        }
        m = m_new;
        if (((j + 1) & 31) == 0) park_constants(j + 1);
    };

    // Step j's iteration starts with a barrier: K^(j+1) and V^(j-1) have landed for every wavefront, and the buffers of K^(j)
    // and V^(j-2) have no reader left, so the copies of K^(j+2) and V^(j) may start.  The iteration after a wavefront's last
    // step adds that step's P^V^.
    // (Three loops one after the other, not one loop with three bodies: that would tie the accumulators of all
    // bodies together at every iteration, which the register allocator does not survive.)
    const auto arrive = [&]() {
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wavefront's pieces have landed
        __syncthreads();
    };
    int j = jb;
    for (; j < full_steps; ++j) {
        arrive();
        step(j);
        par ^= TILE;
    }
    for (; j < my_steps; ++j) {
        arrive();
        masked_step(j);
        par ^= TILE;
    }
    arrive();
    if (my_steps > jb) {
        rescale();
#pragma unroll
        for (int r = 0; r < 2 * CT; ++r) mfma_pv(read_v(par, r), r);
    }
    for (; j < nsteps; ++j) {  // the workgroup's other wavefronts have steps left
#pragma unroll
        for (int k = 0; k < NP; ++k) copy_v(j, k);
#pragma unroll
        for (int k = 0; k < NP; ++k) copy_k(j + 2, k);
        copy_ds(j + 1);
        arrive();
    }

    const float lsum = halves_sum((l[0] + l[1]) + (l[2] + l[3]));
    const int eln = lane_now(), eh = eln >> 5, erow = row0 + (eln & 31);
    if constexpr (SPLIT) {
        // ---- the range's (m, l, acc) of every valid row ----
        if (erow < Nq) {
            const size_t prow = (((size_t)bh * nQblk + qtile) * n_splits + split) * BM + erow - qtile * BM;
            if (eh == 0) *reinterpret_cast<float2 *>(part_ml + prow * 2) = make_float2(m, lsum);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    *reinterpret_cast<float4 *>(part_acc + prow * D + 32 * ct + 8 * b + 4 * eh) =
                        make_float4(o[ct][4 * b], o[ct][4 * b + 1], o[ct][4 * b + 2], o[ct][4 * b + 3]);
        }
        return;
    }
    // ---- epilogue: O = acc * delta_V / (P_r * l); l already carries the factor P_r ----
    {
        const float inv = 1.0f / lsum;
        uint16_t *orow = out + (bh / Hq) * o_st.b + (bh % Hq) * o_st.h + erow * o_st.n;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int b2 = 0; b2 < 2; ++b2) {
                // channels 32ct + 8b + 4h .. + 3 for b = 2*b2 and 2*b2 + 1; after the exchange between the wavefront's halves a
                // lane holds the eight channels of b = 2*b2 + h and stores 16 bytes
                uint32_t w[2][2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int b = 2 * b2 + e;
                    const float4 sc = *reinterpret_cast<const float4 *>(dv_lds + 32 * ct + 8 * b + 4 * eh);
                    const float y0 = o[ct][4 * b] * (sc.x * inv), y1 = o[ct][4 * b + 1] * (sc.y * inv);
                    const float y2 = o[ct][4 * b + 2] * (sc.z * inv), y3 = o[ct][4 * b + 3] * (sc.w * inv);
                    w[e][0] = pack2<BF16>(y0, y1);
                    w[e][1] = pack2<BF16>(y2, y3);
                }
                swap32(w[0][0], w[1][0]);
                swap32(w[0][1], w[1][1]);
                if (erow < Nq)
                    *reinterpret_cast<uint4 *>(orow + 32 * ct + 16 * b2 + 8 * eh) = make_uint4(w[0][0], w[0][1], w[1][0], w[1][1]);
            }
    }
#endif  // __HIP_DEVICE_COMPILE__
}

// Whether the exponentials run at raised priority (RAISE).  That pays while a SIMD has two wavefronts or more and costs a lone one 5 to
// 8 % (32 switches per step), so it depends on the last round of workgroups.  Measured, speed with / without:
//   * up to one workgroup per CU 0.93 (32 heads x 1024, causal 0.93 to 0.95);
//   * d = 128, two workgroups per CU, rounds of 512: the last one more than half full or full 1.08 .. 1.02 (257 .. 512 workgroups), 1.04 (808
//     .. 832), 1.02 (1296 .. 1363), 1.00 (2445 .. 2496, 6144); less than half full 0.94 (544 .. 612), 0.97 (1044 .. 1136), 0.98 (1584 ..
//     1776), 0.99 (2050 .. 2752);
//   * d = 64, three per CU: 1.04 .. 1.10 up to 768, 0.93 .. 1.01 in 776 .. 1024, 1.03 .. 1.05 in 1032 .. 1160, 1.01 .. 1.05 from there on (6144: 1.06);
//   * causal calls end on lone wavefronts: d = 64 0.92 .. 0.96 at 1280 .. 1920 workgroups, 1.00 .. 1.06 from 1980 on, d = 128 0.94 .. 1.006
//     up to 4096.  Key ranges do not (512 workgroups: d = 128 1.02, d = 64 1.06).
bool raise_pays(int wgs, int d, bool causal, bool ranges) {
    if (wgs <= kCUs) return false;
    if (causal && !ranges) return d == 64 && wgs >= 8 * kCUs;
    if (d == 64) return wgs <= 3 * kCUs || wgs > 4 * kCUs;
    const int last = wgs % (2 * kCUs);
    return wgs <= 8 * kCUs && (last == 0 || last > kCUs);
}

template <int D>
hipError_t launch_prefill_d(const void *q, bool q_raw, Strides q_st, const int8_t *k_i8, const uint8_t *v_fp8,
                            const float *q_scale, const float *k_scale, const float *v_scale, void *out, Strides o_st, int B,
                            int Hq, int Hkv, int Nq, int Nk, bool causal, float sm_scale, float log2_pr, bool bf16,
                            hipStream_t stream, const float *q_mean, const float *dsx, int n_splits, int steps_per_split,
                            float *part_acc, float *part_ml) {
    const int nT = cdiv(Nk, kW), nQ = cdiv(Nq, kBQ), nK = cdiv(Nk, kBK);
    const dim3 grid(B * Hq * nQ * n_splits);  // (at most 65535 * 32768 < 2^31 workgroups; ranges only for small calls)
    uint16_t *o16 = static_cast<uint16_t *>(out);
    const bool q4 = dsx != nullptr, ranges = part_acc != nullptr;
    const bool raise = raise_pays((int)grid.x, D, causal, ranges);
#define SAGE_LAUNCH(C, BF, QR, F4, SP, RS)                                                                           \
    prefill_kernel<D, C, BF, QR, F4, SP, RS><<<grid, 256, 0, stream>>>(                                               \
        q, k_i8, v_fp8, q_scale, k_scale, v_scale, o16, q_st, o_st, Nq, Nk, nT, nQ, nK, Hq, Hq / Hkv, sm_scale,      \
        log2_pr, q_mean, dsx, n_splits, steps_per_split, part_acc, part_ml)
#define SAGE_LAUNCH_R(C, BF, QR, SP, CAN)                          \
    do {                                                           \
        if (raise) SAGE_LAUNCH(C, BF, QR, false, SP, CAN);         \
        else SAGE_LAUNCH(C, BF, QR, false, SP, false);             \
    } while (0)
#define SAGE_LAUNCH_Q(C, BF)                                                     \
    do {                                                                         \
        constexpr bool CAN = D == 64 || !C;                                      \
        if (ranges) SAGE_LAUNCH_R(C, BF, true, true, true);                      \
        else if (q4) SAGE_LAUNCH(C, BF, true, true, false, false);               \
        else if (q_raw) SAGE_LAUNCH_R(C, BF, true, false, CAN);                  \
        else SAGE_LAUNCH_R(C, BF, false, false, CAN);                            \
    } while (0)
    if (causal) {
        if (bf16) SAGE_LAUNCH_Q(true, true); else SAGE_LAUNCH_Q(true, false);
    } else {
        if (bf16) SAGE_LAUNCH_Q(false, true); else SAGE_LAUNCH_Q(false, false);
    }
#undef SAGE_LAUNCH_Q
#undef SAGE_LAUNCH_R
#undef SAGE_LAUNCH
    return hipGetLastError();
}

}  // namespace

hipError_t launch_prefill(const void *q, bool q_raw, Strides q_st, const int8_t *k_i8, const uint8_t *v_fp8,
                          const float *q_scale, const float *k_scale, const float *v_scale, void *out, Strides o_st, int B,
                          int Hq, int Hkv, int Nq, int Nk, int d, bool causal, float sm_scale, float p_r, bool bf16,
                          hipStream_t stream, const float *q_mean, const float *dsx, int n_splits, int steps_per_split,
                          float *part_acc, float *part_ml) {
    const float log2_pr = (float)log2((double)p_r);
    if (d == 128)
        return launch_prefill_d<128>(q, q_raw, q_st, k_i8, v_fp8, q_scale, k_scale, v_scale, out, o_st, B, Hq, Hkv, Nq, Nk,
                                     causal, sm_scale, log2_pr, bf16, stream, q_mean, dsx, n_splits, steps_per_split,
                                     part_acc, part_ml);
    return launch_prefill_d<64>(q, q_raw, q_st, k_i8, v_fp8, q_scale, k_scale, v_scale, out, o_st, B, Hq, Hkv, Nq, Nk, causal,
                                sm_scale, log2_pr, bf16, stream, q_mean, dsx, n_splits, steps_per_split, part_acc, part_ml);
}

}  // namespace sage
