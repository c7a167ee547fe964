// Stage 2 of the SageAttention2++ 8+8 forward on gfx950: the fused attention
// kernel (paper Sec. 2.1 for the tiling / online softmax and the scales,
// Sec. 3.1 for the bounded FP8 range P_r of P~).
//
// Mapping to CDNA4.  A workgroup of NWAVE wavefronts owns BM = 16*NQ*NWAVE query
// rows of one (batch, head); a wavefront owns NQ tiles of 16 query rows.  Per
// step of 128 keys the K^ tile [128][D] int8 and the V^ tile [D][128] fp8 are
// copied global -> LDS by buffer loads that write LDS directly (no register
// staging; chunks beyond the end of a head's K^ are not fetched and read as zero), double buffered so that the copy of
// step j+1 runs under the arithmetic of step j (two barriers per step, see "Schedule").
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

#if defined(__HIP_DEVICE_COMPILE__)
// Enqueue piece k of the global -> LDS copy of one [128 x D]-byte tile (K^ or V^) of key step j.  A tile is
// copied by the NW wavefronts of one group, CPG pieces each; a piece (one buffer load) moves 16 bytes per
// lane straight into LDS at dst + 1024*(k*NW + w) + 16*lane; the per-lane source offset carries the
// swizzle.  Every piece gets a buffer descriptor of its own whose base is the piece's first byte and whose
// size is what is left of the head's buffer from there (scalar arithmetic only): the hardware bounds check
// covers the per-lane offset but not a scalar offset, and this way a 16-byte chunk beyond the last byte of
// the buffer (rows >= Nk of the last K^ tile) is never fetched and reads as zero.
template <int D, int NW>
__device__ __forceinline__ void issue_tile_piece(uint8_t *dst, const uint8_t *head, int head_bytes, int voff, int w,
                                                 int k, int j) {
    constexpr int TILE = 128 * D;
    // (piece k of a wavefront lies NW KB after piece 0 on both sides: the swizzles repeat every 8 rows)
    const int first = j * TILE + k * NW * 1024;
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc((void *)(head + first), 0, max(head_bytes - first, 0), 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void *)(dst + (k * NW + w) * 1024), 16, voff, 0, 0, 0);
}
#endif  // __HIP_DEVICE_COMPILE__

// Schedule.  The wavefronts of a workgroup form two groups (first and second half) that run the
// same per-step sequence  M(j) = [PV(j-1), QK(j)]  ->  S(j) = softmax(j)  one slot apart: while
// one group is in its matrix slot (MFMA + LDS reads) the other is in its softmax slot (vector
// ALU), so the two pipes of every SIMD are busy at the same time instead of colliding.  A slot
// ends with a workgroup barrier.  The copy of K^(j+1) is issued by the first group at the start of
// slot 2j, the copy of V^(j) by the second group at the start of slot 2j+1 (each in its own matrix
// slot); both are needed from slot 2j+2 on.
//
// QRAW: Q arrives unquantised (16-bit, the output's type) and the workgroup, whose 128 rows are
// exactly one Q quantisation block, quantises it in its prologue (paper Sec. 2.1: per-block INT8,
// delta = max|Q| / 127) with the same binary32 operations as the stand-alone quantiser, so codes
// and scale are the same bits; Q^ and delta_Q then never touch memory.
//
template <int D, int NQ, int NWAVE, int WPS, bool CAUSAL, bool BF16, bool QRAW>
__global__ __launch_bounds__(NWAVE * 64, WPS) void attn_kernel(
    const void *__restrict__ Qsrc, const int8_t *__restrict__ Kc, const uint8_t *__restrict__ Vt,
    const float *__restrict__ dq, const float *__restrict__ dk, const float *__restrict__ dv,
    uint16_t *__restrict__ out, Strides q_st, Strides o_st, int Nq, int Nk, int nT, int nQblk, int nKblk, int Hq,
    int group, float sm_scale, float log2_pr, int nQtiles) {
#if defined(__HIP_DEVICE_COMPILE__)  // the body uses device-only types; the host pass only needs the stub
    constexpr int BM = 16 * NQ * NWAVE;  // query rows per workgroup
    constexpr int KC = D / 64;           // 64-wide contraction chunks of Q.K^T
    constexpr int CT = D / 16;           // 16-channel tiles of the output
    constexpr int TILE = 128 * D;        // bytes of one K^ (or V^) tile
    constexpr int NTHR = NWAVE * 64;
    constexpr int NWG = NWAVE / 2;                 // wavefronts per group
    constexpr int CPG = TILE / 16 / (NTHR / 2);    // 16-byte chunks a thread copies per tile (one group copies a tile)
    static_assert(TILE / 16 % (NTHR / 2) == 0, "tile chunks must divide over the threads of a group");
    __shared__ __attribute__((aligned(1024))) uint8_t ldsK[2][TILE];
    __shared__ __attribute__((aligned(1024))) uint8_t ldsV[2][TILE];
    __shared__ float q_wave_max[NWAVE];
    // per wavefront: the de-quantisation constants (c, kh, kl, -) of 64 consecutive K blocks (32 key steps)
    __shared__ __attribute__((aligned(16))) float4 cst_lds[NWAVE][64];
    __shared__ __attribute__((aligned(16))) float dv_lds[D];  // delta_V of this head, for the epilogue

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave >= NWAVE / 2 ? 1 : 0;  // second group runs one slot behind
    const int lq = lane & 15, g = lane >> 4;
    int bh, qtile;  // (batch, query head), query tile
    map_workgroup<CAUSAL>((int)blockIdx.x, (int)gridDim.x, nQtiles, bh, qtile);
    const int wg_row0 = qtile * BM;
    const int row0 = wg_row0 + wave * (16 * NQ);
    // grouped-query attention: `group` consecutive query heads share one K/V head
    const int bhk = (bh / Hq) * (Hq / group) + (bh % Hq) / group;
    // causal mask aligned to the end of both sequences: key n visible to query r iff n <= r + shift
    const int shift = Nk - Nq;

    // this head's K^ [Nk][D] and V^ [nT][D][128] and their sizes in bytes (the tile copies are bounded to them)
    const uint8_t *Kh = reinterpret_cast<const uint8_t *>(Kc) + (size_t)bhk * Nk * D;
    const uint8_t *Vh = Vt + (size_t)bhk * nT * D * 128;
    const int k_bytes = Nk * D, v_bytes = nT * D * 128;

    // Tile copies.  The first group copies the K^ tiles, the second the V^ tiles, each at the start of its own
    // matrix slot: the texture path accepts one 1 KB piece per 16 cycles per CU, and a wavefront that cannot
    // issue its piece cannot issue anything else either -- harmless in the matrix slot (it has slack), costly
    // in front of the softmax arithmetic (which is the critical path).
    // Per-lane source offset of this wavefront's piece 0 (the LDS side is linear in the lane index):
    const int wig = wave % NWG;  // wavefront within its group
    int c_voff;
    {
        static_assert(NWG * 64 % (8 * (D / 16)) == 0 && NWG * 8 % 8 == 0, "pieces must be whole swizzle periods apart");
        const int slot = wig * 64 + lane;
        if (grp == 0) {
            constexpr int CPR = D / 16;  // chunks per K row
            const int row = slot / CPR, pc = slot % CPR;
            c_voff = row * D + ((pc ^ k_swz<D>(row)) << 4);
        } else {
            const int row = slot >> 3, pc = slot & 7;
            c_voff = row * 128 + ((pc ^ (row & 7)) << 4);
        }
    }

    int nsteps = nT;
    if constexpr (CAUSAL) nsteps = min(Nk - 1, wg_row0 + BM - 1 + shift) / kW + 1;
    // steps this wavefront takes part in (causal: tiles entirely above its rows are skipped)
    int my_steps = nsteps;
    if constexpr (CAUSAL) my_steps = min(nsteps, (row0 + 16 * NQ - 1 + shift) / kW + 1);
    if (row0 >= Nq) my_steps = 0;  // a wavefront without a valid row only takes part in the copies and barriers
    if (grp == 0) {
#pragma unroll
        for (int k = 0; k < CPG; ++k) issue_tile_piece<D, NWG>(ldsK[0], Kh, k_bytes, c_voff, wig, k, 0);
    }

    // the lane's B operand of S^T = K^ Q^T: 16 consecutive channels (64*ch + 16*g ..) of query row lq
    v4i qreg[NQ][KC];
    uint4 qraw[NQ][KC][2];  // QRAW: the same 16 channels as 16-bit values
    if constexpr (QRAW) {
        static_assert(BM == kBQ, "a workgroup must own exactly one Q quantisation block");
        const uint16_t *Qh = static_cast<const uint16_t *>(Qsrc) + (bh / Hq) * q_st.b + (bh % Hq) * q_st.h;
        float amax = 0.0f;
#pragma unroll
        for (int qt = 0; qt < NQ; ++qt) {
            const int r = row0 + qt * 16 + lq;
#pragma unroll
            for (int ch = 0; ch < KC; ++ch)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    qraw[qt][ch][h] = r < Nq ? *reinterpret_cast<const uint4 *>(Qh + r * q_st.n + ch * 64 + g * 16 + h * 8)
                                             : make_uint4(0u, 0u, 0u, 0u);
                    const uint32_t w[4] = {qraw[qt][ch][h].x, qraw[qt][ch][h].y, qraw[qt][ch][h].z, qraw[qt][ch][h].w};
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        amax = fmaxf(amax, fmaxf(fabsf(to_f32<BF16>(w[i] & 0xffffu)), fabsf(to_f32<BF16>(w[i] >> 16))));
                }
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off));
        if (lane == 0) q_wave_max[wave] = amax;
    } else {
        const int8_t *Qh = static_cast<const int8_t *>(Qsrc) + (bh / Hq) * q_st.b + (bh % Hq) * q_st.h;
#pragma unroll
        for (int qt = 0; qt < NQ; ++qt) {
            const int r = row0 + qt * 16 + lq;
#pragma unroll
            for (int ch = 0; ch < KC; ++ch) {
                v4i z = {0, 0, 0, 0};
                qreg[qt][ch] = r < Nq ? *reinterpret_cast<const v4i *>(Qh + r * q_st.n + ch * 64 + g * 16) : z;
            }
        }
    }
    const v4i cinit = {kMagic, kMagic, kMagic, kMagic};

    // the output scales are fetched now and parked in LDS: the epilogue then waits for no global load
    if (tid < D / 4)
        *reinterpret_cast<float4 *>(dv_lds + 4 * tid) = *reinterpret_cast<const float4 *>(dv + (size_t)bhk * D + 4 * tid);
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): K^(0) has landed
    __syncthreads();

    // de-quantisation constant of this wave's query block (its 16*NQ rows lie inside one Q block)
    float delta_q;
    if constexpr (QRAW) {
        float a = 0.0f;
#pragma unroll
        for (int w = 0; w < NWAVE; ++w) a = fmaxf(a, q_wave_max[w]);
        const float rcp = a > 0.0f ? 127.0f / a : 0.0f;
        delta_q = a / 127.0f;
#pragma unroll
        for (int qt = 0; qt < NQ; ++qt)
#pragma unroll
            for (int ch = 0; ch < KC; ++ch)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    float f[8];
                    unpack8<BF16>(qraw[qt][ch][h], f);
                    const uint2 w = int8_codes(f, rcp);
                    qreg[qt][ch][2 * h] = (int)w.x;
                    qreg[qt][ch][2 * h + 1] = (int)w.y;
                }
    } else {
        delta_q = dq[(size_t)bh * nQblk + min(row0, Nq - 1) / kBQ];
    }
    const double cq = (double)delta_q * (double)sm_scale * 1.4426950408889634;

    // (the accumulators start their life here, after the prologue, whose Q registers they reuse)
    float m[NQ], l[NQ], alpha[NQ];
    v4f o[CT][NQ];
    v4i s[NQ][8];
    v8i pb[NQ];
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
        m[qt] = -INFINITY;
        l[qt] = 0.0f;
        alpha[qt] = 1.0f;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) o[ct][qt] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 8; ++t) s[qt][t] = cinit;
        pb[qt] = v8i{0, 0, 0, 0, 0, 0, 0, 0};
    }


    // piece k of the copy this group makes during its matrix slot M(j): K^(j+1) (first group), V^(j) (second)
    auto copy_k = [&](int j) {
        if (j + 1 < nsteps) {
#pragma unroll
            for (int k = 0; k < CPG; ++k) issue_tile_piece<D, NWG>(ldsK[(j + 1) & 1], Kh, k_bytes, c_voff, wig, k, j + 1);
        }
    };
    auto copy_v = [&](int j) {
        if (j < nsteps) {
#pragma unroll
            for (int k = 0; k < CPG; ++k) issue_tile_piece<D, NWG>(ldsV[j & 1], Vh, v_bytes, c_voff, wig, k, j);
        }
    };
    // matrix slot M(j): PV(j-1), then QK(j)
    auto matrix_slot = [&](int j) {
        if (j > 0 && j <= my_steps) {
            // ---- rescale O only when some running maximum moved ----
            bool moved = false;
#pragma unroll
            for (int qt = 0; qt < NQ; ++qt) moved |= alpha[qt] != 1.0f;
            if (__builtin_amdgcn_ballot_w64(moved) != 0) {
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                    for (int qt = 0; qt < NQ; ++qt) o[ct][qt] *= alpha[qt];
            }
            // ---- O^T += V^T P^T (FP8 E4M3 x E4M3, FP32 accumulation) ----
            const uint8_t *Vs = ldsV[(j - 1) & 1];
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const int row = 16 * ct + lq;
                const v4i lo = *reinterpret_cast<const v4i *>(Vs + v_off(row, g));
                const v4i hi = *reinterpret_cast<const v4i *>(Vs + v_off(row, 4 + g));
                const v8i a = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
#pragma unroll
                for (int qt = 0; qt < NQ; ++qt)
                    o[ct][qt] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, pb[qt], o[ct][qt], 0, 0, 0, 0, 0, 0);
            }
        }
        if (j < my_steps) {
            // ---- S^T = K^ Q^T (INT8, INT32 accumulation onto the float-view bias) ----
            // contraction chunk outermost: consecutive MFMAs never depend on each other
            const uint8_t *Ks = ldsK[j & 1];
#pragma unroll
            for (int ch = 0; ch < KC; ++ch) {
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const v4i a = *reinterpret_cast<const v4i *>(Ks + k_off<D>(16 * t + lq, 4 * ch + g));
#pragma unroll
                    for (int qt = 0; qt < NQ; ++qt)
                        s[qt][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, qreg[qt][ch], ch == 0 ? cinit : s[qt][t], 0, 0, 0);
                }
            }
        }
    };
    // softmax slot S(j)
    auto softmax_slot = [&](int j) {
        if (j >= my_steps) return;
        // the softmax part is the critical path of a slot (the matrix part has slack): its wavefront goes
        // first when both want the vector issue port
        __builtin_amdgcn_s_setprio(1);
        const int key0 = j * kW;
        // de-quantisation constants of the two K blocks of this step: every 32 steps each lane computes the
        // constants of one K block (c, and the exact split -K*c = kh + kl) and parks them in this wavefront's own
        // strip of LDS; a step then fetches its two blocks with two broadcast reads and no vector arithmetic
        if ((j & 31) == 0) {
            const int blk = min(64 * (j >> 5) + lane, nKblk - 1);
            const float c = (float)(cq * (double)dk[(size_t)bhk * nKblk + blk]);
            const float kh = -kMagicF * c;
            cst_lds[wave][lane] = make_float4(c, kh, __builtin_fmaf(-kMagicF, c, -kh), 0.0f);
        }
        const float4 k0 = cst_lds[wave][(2 * j) & 63], k1 = cst_lds[wave][(2 * j + 1) & 63];
        float c0 = k0.x, c1 = k1.x, kh0 = k0.y, kh1 = k1.y, kl0 = k0.z, kl1 = k1.z;
        const bool masked_step = (key0 + kW > Nk) || (CAUSAL && key0 + kW - 1 > row0 + shift);
#pragma unroll
        for (int qt = 0; qt < NQ; ++qt) {
            if (masked_step) {
                int lim = Nk - 1;  // last visible key of this lane's query row
                if constexpr (CAUSAL) lim = min(lim, row0 + qt * 16 + lq + shift);
                // last visible key of the tile's first / last row: tiles wholly at or below the former
                // need no mask, tiles wholly above the latter are invisible
                const int lim_min = CAUSAL ? min(Nk - 1, row0 + qt * 16 + shift) : Nk - 1;
                const int lim_max = CAUSAL ? min(Nk - 1, row0 + qt * 16 + 15 + shift) : Nk - 1;
                const int t_lo = min(8, max(0, (lim_min - key0 + 1) >> 4));
                const int t_hi = min(8, max(0, ((lim_max - key0) >> 4) + 1));
                alpha[qt] = softmax_step<true>(s[qt], c0, c1, kh0, kh1, kl0, kl1, log2_pr, m[qt], l[qt], pb[qt],
                                               key0 + 4 * g, lim, t_lo, t_hi);
            } else {
                alpha[qt] = softmax_step<false>(s[qt], c0, c1, kh0, kh1, kl0, kl1, log2_pr, m[qt], l[qt], pb[qt], 0, 0, 8, 8);
            }
        }
        __builtin_amdgcn_s_setprio(0);
    };

    // 2*nsteps + 2 slots, one barrier each.  K^(j+1) is copied during slot 2j (the first group's M(j)) and
    // V^(j) during slot 2j+1 (the second group's M(j)); both are first read in slot 2j+2 and both target
    // buffers whose last readers finished in slot 2j-1.  Every wavefront waits for its own pieces before the
    // barrier that ends slot 2j+1.
    if (grp == 0) {
        for (int j = 0; j <= nsteps; ++j) {
            copy_k(j);  // slot 2j
            matrix_slot(j);
            __syncthreads();
            softmax_slot(j);  // slot 2j+1
            __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
            __syncthreads();
        }
    } else {
        __syncthreads();  // slot 0: this group idles
        for (int j = 0; j <= nsteps; ++j) {
            copy_v(j);  // slot 2j+1
            matrix_slot(j);
            __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
            __syncthreads();
            if (j < nsteps) {
                softmax_slot(j);  // slot 2j+2
                __syncthreads();
            }
        }
    }

    // ---- epilogue: O = acc * delta_V / (P_r * l); l already carries the factor P_r ----
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
        const float inv = 1.0f / rowgroup_sum(l[qt]);
        const int r = row0 + qt * 16 + lq;
        if (r < Nq) {
            uint16_t *orow = out + (bh / Hq) * o_st.b + (bh % Hq) * o_st.h + r * o_st.n;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const int c = 16 * ct + 4 * g;
                const float4 sc = *reinterpret_cast<const float4 *>(dv_lds + c);
                const float y0 = o[ct][qt][0] * (sc.x * inv), y1 = o[ct][qt][1] * (sc.y * inv);
                const float y2 = o[ct][qt][2] * (sc.z * inv), y3 = o[ct][qt][3] * (sc.w * inv);
                *reinterpret_cast<uint2 *>(orow + c) = make_uint2(pack2<BF16>(y0, y1), pack2<BF16>(y2, y3));
            }
        }
    }
#endif  // __HIP_DEVICE_COMPILE__
}

template <int D, int NQ, int NWAVE, int WPS>
hipError_t launch_d(const void *q, bool q_raw, Strides q_st, const int8_t *k_i8, const uint8_t *v_fp8, const float *q_scale,
                    const float *k_scale, const float *v_scale, void *out, Strides o_st, int B, int Hq, int Hkv, int Nq,
                    int Nk, bool causal, float sm_scale, float log2_pr, bool bf16_out, hipStream_t stream) {
    constexpr int BM = 16 * NQ * NWAVE;
    const int BH = B * Hq;
    const dim3 grid(BH * cdiv(Nq, BM));  // (at most 65535 * 32768 < 2^31 workgroups)
    const int nT = cdiv(Nk, kW), nQ = cdiv(Nq, kBQ), nK = cdiv(Nk, kBK);
    uint16_t *o16 = static_cast<uint16_t *>(out);
#define SAGE_LAUNCH(C, BF, QR)                                                                                   \
    attn_kernel<D, NQ, NWAVE, WPS, C, BF, QR><<<grid, NWAVE * 64, 0, stream>>>(                                    \
        q, k_i8, v_fp8, q_scale, k_scale, v_scale, o16, q_st, o_st, Nq, Nk, nT, nQ, nK, Hq, Hq / Hkv, sm_scale, \
        log2_pr, cdiv(Nq, BM))
#define SAGE_LAUNCH_Q(C, BF)                    \
    if (q_raw) SAGE_LAUNCH(C, BF, true);        \
    else SAGE_LAUNCH(C, BF, false)
    if (causal) {
        if (bf16_out) { SAGE_LAUNCH_Q(true, true); } else { SAGE_LAUNCH_Q(true, false); }
    } else {
        if (bf16_out) { SAGE_LAUNCH_Q(false, true); } else { SAGE_LAUNCH_Q(false, false); }
    }
#undef SAGE_LAUNCH_Q
#undef SAGE_LAUNCH
    return hipGetLastError();
}

}  // namespace

hipError_t launch_attn(const void *q, bool q_raw, Strides q_st, const int8_t *k_i8, const uint8_t *v_fp8,
                       const float *q_scale, const float *k_scale, const float *v_scale, void *out, Strides o_st, int B,
                       int Hq, int Hkv, int Nq, int Nk, int d, bool causal, float sm_scale, float p_r, bool bf16_out,
                       hipStream_t stream, const float *q_mean, const float *dsx) {
    // Which kernel: by how many workgroups the query rows make.  Up to one workgroup of 32 rows per CU, a key step is spread
    // over a workgroup's wavefronts (sage_spread.hip); then with 64 rows per workgroup; beyond one of those per CU the CUs are
    // filled better by whole steps per wavefront and two workgroups of 128 rows each (sage_prefill.hip).  Measured, us, at
    // 1024 x 1024 and 1024 x 16384 (rows x keys, d 128, full), spread 32 / spread 64 / prefill: 128 tiles of 32 rows
    // 10.6 / 13.7 / 16.5 and 76 / 104 / 172; 512 tiles 20.3 / 14.5 / 16.8 and 152 / 111 / 173; 1024 tiles 38.5 / 27.8 / 17.8
    // and 301 / 220 / 181.  Up to kSmallRows rows the kernel of this file remains (16 rows per wavefront: half the padding),
    // and the 4+8 variant exists in the prefill kernel only.
    if (Nq > kSmallRows || dsx) {
        const long heads = (long)B * Hq;
        const int row_groups = dsx ? 0 : heads * cdiv(Nq, 32) <= kCUs ? 1 : heads * cdiv(Nq, 64) <= kCUs ? 2 : 0;
        if (row_groups)
            return launch_spread(q, q_raw, q_st, k_i8, v_fp8, q_scale, k_scale, v_scale, out, o_st, B, Hq, Hkv, Nq, Nk, d,
                                 causal, sm_scale, p_r, bf16_out, stream, row_groups);
        return launch_prefill(q, q_raw, q_st, k_i8, v_fp8, q_scale, k_scale, v_scale, out, o_st, B, Hq, Hkv, Nq, Nk, d, causal,
                              sm_scale, p_r, bf16_out, stream, q_mean, dsx, 1, 0, nullptr, nullptr);
    }
    const float log2_pr = (float)log2((double)p_r);
    if (d == 128)
        return launch_d<128, 1, 8, 4>(q, q_raw, q_st, k_i8, v_fp8, q_scale, k_scale, v_scale, out, o_st, B, Hq, Hkv, Nq, Nk,
                                      causal, sm_scale, log2_pr, bf16_out, stream);
    return launch_d<64, 1, 8, 4>(q, q_raw, q_st, k_i8, v_fp8, q_scale, k_scale, v_scale, out, o_st, B, Hq, Hkv, Nq, Nk, causal,
                                 sm_scale, log2_pr, bf16_out, stream);
}

}  // namespace sage
