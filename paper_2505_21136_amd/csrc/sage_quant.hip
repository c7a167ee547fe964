// Stage 1 of the SageAttention2++ 8+8 forward on gfx950: K smoothing, per-block
// INT8 quantisation of Q and K, per-channel FP8 (E4M3) quantisation of V.
//
// All kernels here are bandwidth bound (read 2 bytes, write 1 byte per element
// and tensor): every global access is a 16-byte load or a 8/16-byte store whose
// lanes cover whole rows, statistics are reduced in registers -> LDS -> a small
// partial buffer in a fixed order (no atomics), so results do not depend on
// scheduling.
//
// This translation unit must be compiled with -ffp-contract=off: each quantiser
// step (x - mean, a / range, range / a, x * r) is one correctly rounded binary32
// operation, which is what makes codes and scales reproducible bit for bit
// (paper Sec. 2.1 for the scales, Sec. 3 for the smoothing).
#include "sage_attn_device.h"
#include "sage_internal.h"

#include <algorithm>
#include <atomic>

namespace sage {
namespace {

// ---------------------------------------------------------------------------
// Partial column statistics over chunks of kStatRows tokens.
//   IS_V = false: sum_n K[n][c] in double (smoothing mean, Sec. 3)
//   IS_V = true : max_n |V[n][c]|        (per-channel FP8 scale, Sec. 2.1)
// One workgroup of 256 threads per (chunk, batch*head); a thread owns 8 adjacent channels.
// Launched per tensor (grid (chunks, B*H)) or for K and V together (grid (chunks, B*H, 2)).
// ---------------------------------------------------------------------------
template <int D>
constexpr int colstats_smem_bytes() {
    return (256 / (D / 8)) * D * (int)sizeof(double);
}

template <bool BF16, int D, bool IS_V>
__device__ __forceinline__ void colstats_body(const uint16_t *__restrict__ X, Strides st, int H, int N, int chunks,
                                              double *__restrict__ sum_part, float *__restrict__ max_part,
                                              void *smem, int bh, int chunk) {
    constexpr int LPR = D / 8;     // lanes per row
    constexpr int RP = 256 / LPR;  // rows per pass
    using acc_t = typename std::conditional<IS_V, float, double>::type;
    acc_t(*sm)[D] = reinterpret_cast<acc_t(*)[D]>(smem);

    const int co = threadIdx.x % LPR, rr = threadIdx.x / LPR;
    const uint16_t *Xh = X + (bh / H) * st.b + (bh % H) * st.h;
    const int r0 = chunk * kStatRows;
    const int r1 = min(r0 + kStatRows, N);

    acc_t acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = 0;
    // four independent 16-byte loads in flight per thread (one per trip leaves the kernel bound by
    // memory latency); rows past the end contribute zeros, which change neither a sum nor a max of |.|
#ifndef SAGE_STAT_UNROLL
#define SAGE_STAT_UNROLL 4
#endif
    constexpr int UNROLL = SAGE_STAT_UNROLL;
    for (int rb = r0 + rr; rb < r1; rb += RP * UNROLL) {
        uint4 u[UNROLL];
#pragma unroll
        for (int k = 0; k < UNROLL; ++k) {
            const int r = rb + k * RP;
            u[k] = r < r1 ? *reinterpret_cast<const uint4 *>(Xh + r * st.n + co * 8) : make_uint4(0u, 0u, 0u, 0u);
        }
#pragma unroll
        for (int k = 0; k < UNROLL; ++k) {
            float f[8];
            unpack8<BF16>(u[k], f);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if constexpr (IS_V) {
                    acc[j] = fmaxf(acc[j], fabsf(f[j]));
                } else {
                    acc[j] += (double)f[j];
                }
            }
        }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) sm[rr][co * 8 + j] = acc[j];
    __syncthreads();
    if (threadIdx.x < D) {
        acc_t a = sm[0][threadIdx.x];
        for (int i = 1; i < RP; ++i) {
            if constexpr (IS_V) {
                a = fmaxf(a, sm[i][threadIdx.x]);
            } else {
                a += sm[i][threadIdx.x];
            }
        }
        const size_t o = ((size_t)bh * chunks + chunk) * D + threadIdx.x;
        if constexpr (IS_V) {
            max_part[o] = a;
        } else {
            sum_part[o] = a;
        }
    }
}

template <bool BF16, int D, bool IS_V>
__global__ __launch_bounds__(256) void colstats_kernel(const uint16_t *__restrict__ X, Strides st, int H, int N,
                                                       int chunks, double *__restrict__ sum_part,
                                                       float *__restrict__ max_part) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[colstats_smem_bytes<D>()];
    colstats_body<BF16, D, IS_V>(X, st, H, N, chunks, sum_part, max_part, smem, blockIdx.y, blockIdx.x);
}

// K sums (blockIdx.z == 0) and V maxima (blockIdx.z == 1) in one launch
template <bool BF16, int D>
__global__ __launch_bounds__(256) void colstats_kv_kernel(const uint16_t *__restrict__ K, Strides k_st,
                                                          const uint16_t *__restrict__ V, Strides v_st, int H, int N,
                                                          int chunks, double *__restrict__ sum_part,
                                                          float *__restrict__ max_part) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[colstats_smem_bytes<D>()];
    if (blockIdx.z == 0)
        colstats_body<BF16, D, false>(K, k_st, H, N, chunks, sum_part, nullptr, smem, blockIdx.y, blockIdx.x);
    else
        colstats_body<BF16, D, true>(V, v_st, H, N, chunks, nullptr, max_part, smem, blockIdx.y, blockIdx.x);
}

// mean[c] = float(sum / N).  1024 threads: 1024/D threads share a channel, each adds every
// (1024/D)-th partial sum in chunk order, the shares are added in a fixed order through LDS
// (the loads of one thread are independent, so the loop is not a chain of memory latencies).
__device__ __forceinline__ void finalize_mean_body(const double *__restrict__ sum_part, int chunks, int N, int D,
                                                   float *__restrict__ mean, double *sm, int bh) {
    const int c = threadIdx.x % D, part = threadIdx.x / D, parts = 1024 / D;
    double s = 0.0;
    for (int i = part; i < chunks; i += parts) s += sum_part[((size_t)bh * chunks + i) * D + c];
    sm[threadIdx.x] = s;
    __syncthreads();
    if (part == 0) {
        for (int k = 1; k < parts; ++k) s += sm[k * D + c];
        mean[(size_t)bh * D + c] = (float)(s / (double)N);
    }
}

// delta_V[c] = a_c / V_r and the multiplier V_r / a_c (0 for an all-zero channel); same thread layout.
__device__ __forceinline__ void finalize_vscale_body(const float *__restrict__ max_part, int chunks, int D, float v_r,
                                                     float *__restrict__ v_scale, float *__restrict__ v_rcp,
                                                     float *sm, int bh) {
    const int c = threadIdx.x % D, part = threadIdx.x / D, parts = 1024 / D;
    float a = 0.0f;
    for (int i = part; i < chunks; i += parts) a = fmaxf(a, max_part[((size_t)bh * chunks + i) * D + c]);
    sm[threadIdx.x] = a;
    __syncthreads();
    if (part == 0) {
        for (int k = 1; k < parts; ++k) a = fmaxf(a, sm[k * D + c]);
        v_scale[(size_t)bh * D + c] = a / v_r;
        v_rcp[(size_t)bh * D + c] = a > 0.0f ? v_r / a : 0.0f;
    }
}

__global__ __launch_bounds__(1024) void finalize_mean_kernel(const double *__restrict__ sum_part, int chunks, int N,
                                                             int D, float *__restrict__ mean) {
    __shared__ double sm[1024];
    finalize_mean_body(sum_part, chunks, N, D, mean, sm, blockIdx.x);
}

__global__ __launch_bounds__(1024) void finalize_vscale_kernel(const float *__restrict__ max_part, int chunks, int D,
                                                               float v_r, float *__restrict__ v_scale,
                                                               float *__restrict__ v_rcp) {
    __shared__ float sm[1024];
    finalize_vscale_body(max_part, chunks, D, v_r, v_scale, v_rcp, sm, blockIdx.x);
}

// the K mean (blockIdx.y == 0) and the V scales (blockIdx.y == 1) in one launch
__global__ __launch_bounds__(1024) void finalize_kv_kernel(const double *__restrict__ sum_part,
                                                           const float *__restrict__ max_part, int chunks, int N, int D,
                                                           float v_r, float *__restrict__ mean,
                                                           float *__restrict__ v_scale, float *__restrict__ v_rcp) {
    __shared__ double sm[1024];
    if (blockIdx.y == 0)
        finalize_mean_body(sum_part, chunks, N, D, mean, sm, blockIdx.x);
    else
        finalize_vscale_body(max_part, chunks, D, v_r, v_scale, v_rcp, reinterpret_cast<float *>(sm), blockIdx.x);
}

// Maximum over the wavefront of a value >= 0 (not NaN), in every lane: within rows of 16 lanes by DPP, then over the four rows, whose
// bit patterns order like integers, in scalar registers.  (wave_max of the attention kernels exchanges the rows in vector registers, which
// with a block's 16 maxima in a row is slower: K and V of 16 heads x 100000, d 64 148.5 / 145.7 us.)
__device__ __forceinline__ float wave_max_abs(float x) {
#define SAGE_DPP(CTRL) \
    x = fmaxf(x, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true)))
    SAGE_DPP(0xb1);   // quad_perm [1,0,3,2]
    SAGE_DPP(0x4e);   // quad_perm [2,3,0,1]
    SAGE_DPP(0x141);  // row_half_mirror
    SAGE_DPP(0x140);  // row_mirror
#undef SAGE_DPP
    const int b = __builtin_bit_cast(int, x);
    const int lo = max(__builtin_amdgcn_readlane(b, 0), __builtin_amdgcn_readlane(b, 16));
    const int hi = max(__builtin_amdgcn_readlane(b, 32), __builtin_amdgcn_readlane(b, 48));
    return __builtin_bit_cast(float, max(lo, hi));
}

// ---------------------------------------------------------------------------
// Per-block integer quantisation (Sec. 2.1): one workgroup per block of BLOCK
// tokens, the block lives in registers between the max pass and the code pass.
// QMAX = 127: INT8 codes; QMAX = 7: the INT4 codes of the 4+8 variant (one per
// byte).  SMOOTH = 0: no mean is subtracted; 1: `mean` holds one vector per
// head (K smoothing, Sec. 3); 2: one vector per head and block (Q smoothing of
// the 4+8 variant).  256 threads, numbered by tid, each workgroup's teams in step; wmax: four floats of LDS per team.
// Bound by memory, or by its latency: a thread's loads are all in flight at once (rows past the end load the last one; with a branch
// around each load, which then waited for itself, and the maximum through LDS: Q of 512 heads x 1024, d 128 40.4 -> 32.2 us, of 64 heads x 777
// 5.7 -> 4.7; beside K's workgroups in one launch, 256 heads x 777, d 64 21.2 -> 18.2, x 1024 23.2 -> 20.3).
// ---------------------------------------------------------------------------
template <bool BF16, int D, int BLOCK, int SMOOTH, int QMAX>
__device__ __forceinline__ void quant_int8_body(const uint16_t *__restrict__ X, Strides st, int H,
                                                const float *__restrict__ mean, int8_t *__restrict__ codes,
                                                float *__restrict__ scale, int N, int nblk, float *wmax, int bh,
                                                int blk, int tid) {
    constexpr int LPR = D / 8;
    constexpr int RP = 256 / LPR;
    constexpr int ITER = BLOCK / RP;
    constexpr float kRange = (float)QMAX;
    static_assert(BLOCK % RP == 0, "block must be a multiple of the rows covered per pass");

    const int co = tid % LPR, rr = tid / LPR;
    const uint16_t *Xh = X + (bh / H) * st.b + (bh % H) * st.h;

    float mu[8];
    const size_t mrow = SMOOTH == 2 ? (size_t)bh * nblk + blk : (size_t)bh;
#pragma unroll
    for (int j = 0; j < 8; ++j) mu[j] = SMOOTH ? mean[mrow * D + co * 8 + j] : 0.0f;

    uint4 raw[ITER];
#pragma unroll
    for (int it = 0; it < ITER; ++it)
        raw[it] = *reinterpret_cast<const uint4 *>(Xh + (int64_t)min(blk * BLOCK + it * RP + rr, N - 1) * st.n + co * 8);
    float x[ITER][8];
    float amax = 0.0f;
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
        unpack8<BF16>(raw[it], x[it]);
        if constexpr (SMOOTH != 0) {
#pragma unroll
            for (int j = 0; j < 8; ++j) x[it][j] = x[it][j] - mu[j];
        }
        if (blk * BLOCK + it * RP + rr < N) {
#pragma unroll
            for (int j = 0; j < 8; ++j) amax = fmaxf(amax, fabsf(x[it][j]));
        }
    }
    amax = wave_max_abs(amax);
    if ((tid & 63) == 0) wmax[tid >> 6] = amax;
    __syncthreads();
    const float a = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
    const float rcp = a > 0.0f ? kRange / a : 0.0f;
    if (tid == 0 && blk < nblk) scale[(size_t)bh * nblk + blk] = a / kRange;

#pragma unroll
    for (int it = 0; it < ITER; ++it) {
        const int r = blk * BLOCK + it * RP + rr;
        if (r < N) {
            uint32_t w[2] = {0u, 0u};
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int c = (int)__builtin_rintf(x[it][j] * rcp);
                w[j >> 2] |= ((uint32_t)c & 0xffu) << (8 * (j & 3));
            }
            *reinterpret_cast<uint2 *>(codes + ((size_t)bh * N + r) * D + co * 8) = make_uint2(w[0], w[1]);
        }
    }
}

// ---------------------------------------------------------------------------
// 4+8 variant: what smoothing of Q subtracts (Sec. 3 names the step; reading: the mean of each Q block,
// per channel, over the block's valid tokens).  mean[bh][blk][c] = float(sum_r Q[r][c] / rows), the sum in
// double (exact for 16-bit inputs, so the order of the additions does not matter).  One workgroup of 256
// threads per Q block; sm: RP x D doubles.
// ---------------------------------------------------------------------------
// Bound by latency, not by bytes (32 KB per block): all of a thread's loads are in flight at once, and with K and V quantised in the
// same call the blocks are the last workgroups of that launch.  The quantiser's workgroups of the 4+8 variant rarely fill the chip
// (B 2, 32 / 8 heads of 3000 x 128: 384 of 256 threads), so the blocks run beside them and a launch with its gap goes: the whole
// call 180.5 -> 174.4 us (B 1, 8 heads of 1024 x 64: two launches over chunks; with them 37.3 -> 29.5 us).  Teams of 256 threads, numbered by tid, a workgroup's teams in step.
template <int D>
constexpr int block_mean_doubles() {
    return 256 / (D / 8) * D;
}
template <bool BF16, int D>
__device__ __forceinline__ void block_mean_body(const uint16_t *__restrict__ Q, Strides st, int H, int N, int nblk,
                                                float *__restrict__ mean, double *sm, int bh, int blk, int tid) {
    constexpr int LPR = D / 8, RP = 256 / LPR, ITER = kBQ / RP;
    const int co = tid % LPR, rr = tid / LPR;
    const uint16_t *Qh = Q + (bh / H) * st.b + (bh % H) * st.h + co * 8;
    const int r0 = blk * kBQ + rr;
    uint4 raw[ITER];
#pragma unroll
    for (int it = 0; it < ITER; ++it) raw[it] = *reinterpret_cast<const uint4 *>(Qh + (int64_t)min(r0 + it * RP, N - 1) * st.n);
    double acc[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
        float f[8];
        unpack8<BF16>(raw[it], f);
        if (r0 + it * RP < N) {
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] += (double)f[j];
        }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) sm[rr * D + co * 8 + j] = acc[j];
    __syncthreads();
    if (tid < D && blk < nblk) {
        double a = sm[tid];
#pragma unroll
        for (int i = 1; i < RP; ++i) a += sm[i * D + tid];
        mean[((size_t)bh * nblk + blk) * D + tid] = (float)(a / (double)(min(kBQ, N - blk * kBQ)));
    }
}

template <bool BF16, int D>
__global__ __launch_bounds__(256) void block_mean_kernel(const uint16_t *__restrict__ Q, Strides st, int H, int N,
                                                         int nblk, float *__restrict__ mean) {
    __shared__ double sm[block_mean_doubles<D>()];
    block_mean_body<BF16, D>(Q, st, H, N, nblk, mean, sm, blockIdx.y, blockIdx.x, threadIdx.x);
}

// ---------------------------------------------------------------------------
// 4+8 variant: the score correction.  With Q' = Q - qbar_i on Q block i, Q K'^T = Q' K'^T + qbar_i K'^T; the
// second term, dS[i][n] = sum_c qbar[i][c] * K'[n][c] with the smoothed UNquantised keys K' = K - mu_K, is
// computed here in FP32 and stored in the units of the softmax exponent (times sm_scale * log2 e), in the key
// order of the attention kernel's correction buffer: [B*Hq][nQ][nT][128] floats, position 32*g + 4*t + i of a tile =
// key 16*t + 4*g + i (t < 8, g < 4, i < 4).  Keys >= Nk hold 0.
//
// A contraction, so it runs on the matrix pipe (v_mfma_f32_32x32x2_f32: FP32 products and sums): keys are the rows, the
// (Q block, query head) pairs of a K/V head's group the columns, 32 of each per wavefront.  A lane keeps half a K' row (its
// key's channels D/2 * h ..) and half a mean row in registers.  A workgroup of 4 wavefronts takes one 128-key tile and
// `tiles` column tiles.  Columns are numbered Q block major, so that what a causal launch does not need (the Q blocks that
// see no key of the tile) is a prefix that is skipped.  With D / 2 MFMAs of 64 cycles per wavefront and tile it is the
// latency in front of them that counts, with few workgroups: keys, means and K mean are fetched together.  The 64 accumulators of
// the four sums leave three wavefronts per SIMD (d = 64: four; one less costs 2 us with few columns, gains 2 us with 32 and more).
// Measured (B 2, 32 / 8 heads, N 3000, d 128, causal / full): 122 us with one key per thread and the means broadcast from LDS (one
// LDS read per four FMAs); 23.8 / 35.7 us with the K mean read behind the mask of the last keys, pair by pair, and the means piece
// by piece; 16.0 / 20.2 us with everything fetched together and one sum; about 1 us more with four.  One key per thread is the
// faster only with one Q block, ungrouped heads and 1000 to 2000 key tiles (B 2, H 32, Nk 4096, d 64: 11.8 / 14.8 us).
// ---------------------------------------------------------------------------
template <bool BF16, int D>
__global__ __launch_bounds__(256, D == 128 ? 3 : 4) void delta_s_kernel(const uint16_t *__restrict__ K, Strides k_st, int Hkv,
                                                      const float *__restrict__ k_mean,
                                                      const float *__restrict__ q_mean, float *__restrict__ dsx,
                                                      int Hq, int Nq, int Nk, int nQ, int nT, float sm_log2e,
                                                      int causal, int tiles) {
#if defined(__HIP_DEVICE_COMPILE__)
    typedef float v16f __attribute__((ext_vector_type(16)));
    constexpr int HALF = D / 2;
    __shared__ __attribute__((aligned(16))) float qm[32][D + 4];
    __shared__ __attribute__((aligned(16))) float km[D];
    const int T = blockIdx.x, bhk = blockIdx.y;
    const int group = Hq / Hkv;
    // causal (mask aligned to the end of both sequences): Q block i sees key n iff n <= i*kBQ + kBQ-1 + Nk - Nq
    const int i_first = causal ? max(0, (T * 128 - (Nk - Nq)) / kBQ) : 0;
    const int col_end = nQ * group;
    int col0 = i_first * group + 32 * tiles * (int)blockIdx.z;
    if (col0 >= col_end) return;  // (workgroup-uniform)
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lq = lane & 31, h = lane >> 5;
    const int n = T * 128 + wave * 32 + lq;  // this lane's key
    // a column: Q block i of query head bhq (columns past the end repeat the last one and are not stored)
    const auto column = [&](int c, int &i, int &bhq) {
        const int col = min(c, col_end - 1);
        i = col / group;
        bhq = (bhk / Hkv) * Hq + (bhk % Hkv) * group + col % group;
    };
    // every load of the first tile is issued before the first is waited for (a branch around a load makes it wait for itself)
    const uint16_t *Kr = K + (bhk / Hkv) * k_st.b + (bhk % Hkv) * k_st.h + min(n, Nk - 1) * k_st.n + h * HALF;
    uint4 raw[HALF / 8];
#pragma unroll
    for (int c8 = 0; c8 < HALF / 8; ++c8) raw[c8] = *reinterpret_cast<const uint4 *>(Kr + c8 * 8);
    // a tile's 32 mean rows: whole rows from memory, once for the four wavefronts
    constexpr int NM = 32 * D / 4 / 256;
    const auto load_mean = [&](int x) {
        const int e = threadIdx.x + 256 * x;
        int i, bhq;
        column(col0 + e / (D / 4), i, bhq);
        return *reinterpret_cast<const float4 *>(q_mean + ((size_t)bhq * nQ + i) * D + 4 * (e % (D / 4)));
    };
    const auto stage_mean = [&](int x, const float4 &v) {
        const int e = threadIdx.x + 256 * x;
        *reinterpret_cast<float4 *>(&qm[e / (D / 4)][4 * (e % (D / 4))]) = v;
    };
    const auto stage_tile = [&]() {
        const float4 a = load_mean(0), b = load_mean(1);
        if constexpr (NM == 4) {
            const float4 c = load_mean(2), d = load_mean(3);
            stage_mean(2, c);
            stage_mean(3, d);
        }
        stage_mean(0, a);
        stage_mean(1, b);
    };
    static_assert(NM == 2 || NM == 4, "head dimension 64 or 128");
    const int kc = 4 * (threadIdx.x % (D / 4));  // (several threads write the same value)
    const float4 kmean4 = *reinterpret_cast<const float4 *>(k_mean + (size_t)bhk * D + kc);
    stage_tile();
    *reinterpret_cast<float4 *>(km + kc) = kmean4;
    __syncthreads();
    float kp[HALF];  // (of the last key where n is beyond it)
#pragma unroll
    for (int c8 = 0; c8 < HALF / 8; ++c8) {
        float f[8];
        unpack8<BF16>(raw[c8], f);
#pragma unroll
        for (int j4 = 0; j4 < 2; ++j4) {
            const float4 mu = *reinterpret_cast<const float4 *>(km + h * HALF + c8 * 8 + 4 * j4);
            kp[c8 * 8 + 4 * j4] = f[4 * j4] - mu.x;
            kp[c8 * 8 + 4 * j4 + 1] = f[4 * j4 + 1] - mu.y;
            kp[c8 * 8 + 4 * j4 + 2] = f[4 * j4 + 2] - mu.z;
            kp[c8 * 8 + 4 * j4 + 3] = f[4 * j4 + 3] - mu.w;
        }
    }
    for (int ct = 0; ct < tiles && col0 < col_end; ++ct, col0 += 32) {
        if (ct > 0) {
            __syncthreads();
            stage_tile();
            __syncthreads();
        }
        int i, bhq;
        column(col0 + lq, i, bhq);
        // four sums over the channels of one residue modulo 4, added at the end: with one chain over all of them the error against
        // 64 bits is 1.8 times as large (2-norm, d = 128: 2.06e-7 of the result against 1.15e-7)
        const v16f zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        v16f part[4] = {zero, zero, zero, zero};
#pragma unroll
        for (int c4 = 0; c4 < HALF / 4; ++c4) {
            const float4 v = *reinterpret_cast<const float4 *>(&qm[lq][h * HALF + 4 * c4]);
            part[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(kp[4 * c4], v.x, part[0], 0, 0, 0);
            part[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(kp[4 * c4 + 1], v.y, part[1], 0, 0, 0);
            part[2] = __builtin_amdgcn_mfma_f32_32x32x2f32(kp[4 * c4 + 2], v.z, part[2], 0, 0, 0);
            part[3] = __builtin_amdgcn_mfma_f32_32x32x2f32(kp[4 * c4 + 3], v.w, part[3], 0, 0, 0);
        }
        v16f acc = (part[0] + part[1]) + (part[2] + part[3]);
        if (T * 128 + 127 >= Nk) {  // (workgroup-uniform) keys beyond the last hold zeros
#pragma unroll
            for (int e = 0; e < 16; ++e)
                if (T * 128 + 32 * wave + 8 * (e >> 2) + 4 * h + (e & 3) >= Nk) acc[e] = 0.0f;
        }
        // acc[4b + r] is key 32*wave + 8b + 4h + r of the tile: 16-key group t = 2*wave + (b >> 1), quad g = 2*(b & 1) + h
        if (col0 + lq < col_end) {
            float *dst = dsx + (((size_t)bhq * nQ + i) * nT + T) * 128;
#pragma unroll
            for (int b = 0; b < 4; ++b)
                *reinterpret_cast<float4 *>(dst + 32 * (2 * (b & 1) + h) + 4 * (2 * wave + (b >> 1))) =
                    make_float4(acc[4 * b] * sm_log2e, acc[4 * b + 1] * sm_log2e, acc[4 * b + 2] * sm_log2e,
                                acc[4 * b + 3] * sm_log2e);
        }
    }
#endif  // __HIP_DEVICE_COMPILE__
}

// ---------------------------------------------------------------------------
// Per-channel FP8 quantisation of V into the transposed, key-permuted tile
// layout the attention kernel consumes: [B*H][tile][D][128] bytes, byte
// 64*(t>>2) + 16*g + 4*(t&3) + i of a row = key 16*t + 4*g + i of the tile.  A thread converts
// 4 consecutive keys x 8 channels, so the four keys of one channel pack into
// one dword; the tile is transposed through LDS and leaves as one contiguous
// D*128-byte burst.  256 threads; tile: D*32 dwords of LDS.
// ---------------------------------------------------------------------------
template <bool BF16, int D>
__device__ __forceinline__ void quant_v_body(const uint16_t *__restrict__ V, Strides st, int H,
                                             const float *__restrict__ v_rcp, uint8_t *__restrict__ Vt, int N, int nT,
                                             uint32_t *tile, int bh, int T) {
    constexpr int LPR = D / 8;
    constexpr int UPT = 32 * LPR / 256;  // (key quad, channel octet) units per thread

    const uint16_t *Vh = V + (bh / H) * st.b + (bh % H) * st.h;
#pragma unroll
    for (int k = 0; k < UPT; ++k) {
        const int u = threadIdx.x + 256 * k;
        const int co = u % LPR, kq = u / LPR;
        const int t = kq >> 2, g = kq & 3;
        float rc[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) rc[j] = v_rcp[(size_t)bh * D + co * 8 + j];
        float y[4][8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = T * 128 + kq * 4 + i;
            if (r < N) {
                const uint4 raw = *reinterpret_cast<const uint4 *>(Vh + r * st.n + co * 8);
                unpack8<BF16>(raw, y[i]);
#pragma unroll
                for (int j = 0; j < 8; ++j) y[i][j] = y[i][j] * rc[j];
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) y[i][j] = 0.0f;
            }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            int w = 0;
            w = __builtin_amdgcn_cvt_pk_fp8_f32(y[0][j], y[1][j], w, false);
            w = __builtin_amdgcn_cvt_pk_fp8_f32(y[2][j], y[3][j], w, true);
            tile[(co * 8 + j) * 32 + (t >> 2) * 16 + g * 4 + (t & 3)] = (uint32_t)w;
        }
    }
    __syncthreads();
    uint4 *dst = reinterpret_cast<uint4 *>(Vt + ((size_t)bh * nT + T) * D * 128);
    const uint4 *src = reinterpret_cast<const uint4 *>(tile);
#pragma unroll
    for (int k = 0; k < D / 32; ++k) dst[threadIdx.x + 256 * k] = src[threadIdx.x + 256 * k];
}

// grid (blocks, B*H)
template <bool BF16, int D, int BLOCK, int SMOOTH, int QMAX>
__global__ __launch_bounds__(256) void quant_int8_kernel(const uint16_t *__restrict__ X, Strides st, int H,
                                                         const float *__restrict__ mean, int8_t *__restrict__ codes,
                                                         float *__restrict__ scale, int N, int nblk) {
    __shared__ float wmax[4];
    quant_int8_body<BF16, D, BLOCK, SMOOTH, QMAX>(X, st, H, mean, codes, scale, N, nblk, wmax, blockIdx.y, blockIdx.x,
                                                threadIdx.x);
}

// grid (tiles, B*H)
template <bool BF16, int D>
__global__ __launch_bounds__(256) void quant_v_kernel(const uint16_t *__restrict__ V, Strides st, int H,
                                                      const float *__restrict__ v_rcp, uint8_t *__restrict__ Vt, int N,
                                                      int nT) {
    __shared__ uint32_t tile[D * 32];
    quant_v_body<BF16, D>(V, st, H, v_rcp, Vt, N, nT, tile, blockIdx.y, blockIdx.x);
}

// K blocks (blockIdx.x < nK) and V tiles (the rest) in one launch: grid (nK + nT, B*H)
template <bool BF16, int D, int QMAX>
__global__ __launch_bounds__(256) void quant_kv_kernel(const uint16_t *__restrict__ K, Strides k_st,
                                                       const float *__restrict__ mean, int8_t *__restrict__ k_codes,
                                                       float *__restrict__ k_scale, int nK,
                                                       const uint16_t *__restrict__ V, Strides v_st,
                                                       const float *__restrict__ v_rcp, uint8_t *__restrict__ Vt, int nT,
                                                       int H, int N) {
    __shared__ uint32_t tile[D * 32];
    const int x = blockIdx.x;  // (workgroup-uniform branch)
    if (x < nK)
        quant_int8_body<BF16, D, kBK, 1, QMAX>(K, k_st, H, mean, k_codes, k_scale, N, nK,
                                               reinterpret_cast<float *>(tile), blockIdx.y, x, threadIdx.x);
    else
        quant_v_body<BF16, D>(V, v_st, H, v_rcp, Vt, N, nT, tile, blockIdx.y, x - nK);
}

// ---------------------------------------------------------------------------
// K and V quantised with ONE read of each tensor (smoothing of Sec. 3, scales of Sec. 2.1; the same binary32
// steps and the same outputs as the three launches above).  The codes of a token need a statistic of its whole
// head (the K mean, the V maxima), so a token must wait somewhere between the statistics and the codes: here it
// waits in registers.  A workgroup of NTHR threads loads NTHR * 128 elements of one (head, tensor) — with 256 threads
// 256 tokens at d = 128, 512 at d = 64 — keeps them as 16 packed uint4 per thread, publishes its partial column statistic,
// and then (unless the head is its own alone, G = 1) waits for the partials of all G = ceil(N / tokens) workgroups of the (head, tensor).  A partial is
// its own "there" flag: the partial buffers are zero at launch (the host enqueues zero_words_kernel in front)
// and a value is stored with a bit pattern that is never all zero (+0.0 goes out as -0.0, which adds and
// compares like it), each with one write-through store that is atomic for its 4 or 8 bytes.  Thread t first
// polls element 0 of partial t, sleeping between polls, for at most `wait_ticks` ticks of the constant 100 MHz
// clock; once those are there every workgroup loads all G x d values (again until none is zero) and adds them
// itself, in index order, so all workgroups of a head see the same statistic (workgroup 0 of the group also
// writes it out: mean, or delta_V).  No workgroup waits for another one to do work on its behalf: the only chain
// is "partial stored -> partial seen".  A workgroup whose wait runs out (its partners not resident: another
// kernel holds the CUs, or a dispatch order other than by index) computes the head's statistic itself from
// global memory and goes on, so every wavefront leaves the kernel whatever the others do.  (The two questions of
// a poll -- is a partial missing, has my time run out -- are two workgroup-wide reductions: __syncthreads_or only
// tells whether any thread's value is non-zero.)
// Workgroup ids are group-major, and the hardware dispatches them in id order, so the G partners are resident
// together as long as G does not exceed the workgroups the chip holds; since every workgroup reads G partials the
// host takes this path only up to kResidentMaxGroup.  Grid: B*H*2*G, group 2*bh is K of head bh, 2*bh + 1 is V; or, for one
// tensor alone, B*H*G.
// ---------------------------------------------------------------------------
// tokens of a workgroup of n threads: 16 uint4 of 8 elements per thread
constexpr int resident_tokens(int threads, int d) { return threads * 128 / d; }
// Q side of a launch that also works on Q (quant_kv_resident_kernel<..., WITH_Q>, chunk_stats_kernel): INT8 codes and scales or, with
// `mean`, the block means of the 4+8 variant.  BH heads (H per batch) of N rows; first = workgroups of the K and V side.
struct QuantQ {
    const uint16_t *x;
    Strides st;
    int8_t *codes;
    float *scale, *mean;
    int BH, H, N, n_blocks, first;
    // workgroups that the blocks take, `teams` each
    int workgroups(int teams) const { return x ? BH * cdiv(n_blocks, teams) : 0; }
};
constexpr int kBothTensors = 0, kOnlyK = 1, kOnlyV = 2;  // what a launch quantises (both: K and V groups in turn)
constexpr int kResidentMaxGroup = 256;  // largest group, in workgroups of 256 threads (thread t polls partner t)
constexpr long long kResidentWaitTicks = 50000;  // 0.5 ms
inline int resident_group_size(int N, int d, int threads) { return cdiv(N, resident_tokens(threads, d)); }

__global__ __launch_bounds__(256) void zero_words_kernel(uint4 *w, int n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) w[i] = make_uint4(0u, 0u, 0u, 0u);
}


// The FP8 codes of channels 2 j2 and 2 j2 + 1 (one packed dword of each key; of the eight with the reciprocals rc) of four keys.
template <bool BF16>
__device__ __forceinline__ uint2 v_pair_codes(const uint4 *keys, const float (&rc)[8], int j2) {
    float y[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint4 &x = keys[i];
        const uint32_t w16 = j2 == 0 ? x.x : j2 == 1 ? x.y : j2 == 2 ? x.z : x.w;
        y[i][0] = to_f32<BF16>(w16 & 0xffffu) * rc[2 * j2];
        y[i][1] = to_f32<BF16>(w16 >> 16) * rc[2 * j2 + 1];
    }
    int c[2] = {0, 0};
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        c[e] = __builtin_amdgcn_cvt_pk_fp8_f32(y[0][e], y[1][e], c[e], false);
        c[e] = __builtin_amdgcn_cvt_pk_fp8_f32(y[2][e], y[3][e], c[e], true);
    }
    return make_uint2((uint32_t)c[0], (uint32_t)c[1]);
}

// The FP8 codes of 8 channels of the keys 16t + 4g + i (raw[4t + i], t, i < 4) of a half tile: for each channel the 16 bytes at
// `dst` + 128 * channel, straight from the thread that has the keys: with the key quads of a thread chosen like this
// no transposition through LDS is needed (dwords written there by lanes of neighbouring channels fall on one bank).
template <bool BF16>
__device__ __forceinline__ void v_codes(const uint4 (&raw)[16], const float (&rc)[8], uint8_t *dst) {
#pragma unroll
    for (int j2 = 0; j2 < 4; ++j2) {
        uint2 w[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) w[t] = v_pair_codes<BF16>(&raw[4 * t], rc, j2);
        *reinterpret_cast<uint4 *>(dst + 2 * j2 * 128) = make_uint4(w[0].x, w[1].x, w[2].x, w[3].x);
        *reinterpret_cast<uint4 *>(dst + (2 * j2 + 1) * 128) = make_uint4(w[0].y, w[1].y, w[2].y, w[3].y);
    }
}

// The packed rows stay packed between the passes over them: without this the compiler keeps the unpacked
// floats of one pass alive for the next (twice the registers of the packed rows).
__device__ __forceinline__ void keep_packed(uint4 (&raw)[16]) {
#pragma unroll
    for (int it = 0; it < 16; ++it) asm volatile("" : "+v"(raw[it].x), "+v"(raw[it].y), "+v"(raw[it].z), "+v"(raw[it].w));
}

// What the workgroups of a group tell each other goes through device-scope relaxed atomic accesses: stores
// that write through to memory and loads that do not take a line another XCD's L2 may hold stale.  No cache is
// written back or invalidated as a whole (a device-scope release fence does that, per wavefront, and with a
// few thousand workgroups writing codes at the same time it costs ten times the kernel's own work).
template <class T>
__device__ __forceinline__ void put_shared(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ T get_shared(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The bit pattern a partial is stored with (never all zero) and read back from.
__device__ __forceinline__ unsigned long long tag_bits(double a) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, a);
    return b ? b : 0x8000000000000000ull;
}
__device__ __forceinline__ unsigned tag_bits(float a) {
    const unsigned b = __builtin_bit_cast(unsigned, a);
    return b ? b : 0x80000000u;
}

// Wait until element 0 of each of the G partials (rows of d words) is there.  True when they are, false when
// the wait ran out (workgroup-uniform).  Contains a barrier in every case.
template <class W>
__device__ __forceinline__ bool resident_wait(const W *rows, int d, int G, long long wait_ticks, long long t0) {
    if (wait_ticks < 0) {
        __syncthreads();
        return false;
    }
    for (;;) {
        const bool missing = (int)threadIdx.x < G && get_shared(&rows[(size_t)threadIdx.x * d]) == 0;  // partner t
        const bool late = wall_clock64() - t0 >= wait_ticks;                                          // my time is up
        // (__syncthreads_or tells WHETHER any thread's value is non-zero, not which bits: one call per question)
        if (!__syncthreads_or(missing)) return true;
        if (__syncthreads_or(late)) return false;
        __builtin_amdgcn_s_sleep(8);
    }
}

// WITH_Q (K alone): workgroups beyond the groups' quantise NTHR / 256 Q blocks each (no smoothing), which need nobody and fill the
// time the others wait (the separate stages at B 16, H 16, N 777, d 64: 89.8 -> 87.9 us against a launch of their own).
template <bool BF16, int D, int QMAX, int NTHR, bool WITH_Q>
__global__ __launch_bounds__(NTHR, 4) void quant_kv_resident_kernel(
    const uint16_t *__restrict__ K, Strides k_st, const uint16_t *__restrict__ V, Strides v_st, int H, int N, int G,
    double *k_sum_part, float *v_max_part, float *k_mean, float *v_scale, float v_r,
    int8_t *__restrict__ k_codes, float *__restrict__ k_scale, int nK, uint8_t *__restrict__ Vt, int nT,
    long long wait_ticks, int stagger, bool v_through_lds, int tensors, QuantQ q) {
    constexpr int NU = 16;                       // uint4 per thread
    constexpr int NW = NTHR / 64;                // wavefronts
    constexpr int LPR = D / 8;                   // lanes per row
    constexpr int RP = NTHR / LPR;               // rows per pass of the workgroup
    constexpr int C = NU * RP;                   // tokens of a workgroup
    static_assert(C == resident_tokens(NTHR, D), "the host counts the same tokens");
    __shared__ __attribute__((aligned(16))) unsigned char smem[NTHR * 64];
    __shared__ float stat[D];           // the head's mean (K) or V_r / max (V)
    __shared__ __attribute__((aligned(16))) float wmax[C / kBK][NW];  // per K block and wavefront: max |K'|

    if constexpr (WITH_Q) {
        if ((int)blockIdx.x >= q.first) {
            constexpr int TEAMS = NTHR / 256;
            const int team = threadIdx.x >> 8, wgs = (q.n_blocks + TEAMS - 1) / TEAMS;
            const int x = blockIdx.x - q.first, bh = x / wgs, blk = x % wgs * TEAMS + team;
            if constexpr (QMAX == 127) {
                quant_int8_body<BF16, D, kBQ, 0, 127>(q.x, q.st, q.H, nullptr, q.codes, q.scale, q.N, q.n_blocks,
                                                      &wmax[0][0] + 4 * team, bh, blk, threadIdx.x & 255);
            } else {
                static_assert(TEAMS * block_mean_doubles<D>() * sizeof(double) <= sizeof(smem), "teams of the block means");
                block_mean_body<BF16, D>(q.x, q.st, q.H, q.N, q.n_blocks, q.mean,
                                         reinterpret_cast<double *>(smem) + team * block_mean_doubles<D>(), bh, blk,
                                         threadIdx.x & 255);
            }
            return;
        }
    }
    // Workgroups of one round load, meet and store together, so that the memory rests while they meet.  In launches of two rounds and more
    // (launch_resident_n has the rule) those that come second, third and fourth to their CU start later, `stagger` ticks of the 100 MHz clock each, and the phases
    // of a CU's workgroups stay apart.  (us without / with: 128 heads x 4096, d 128 87.6 / 83.6; 48 x 17776, d 64 74.5 / 72.2; with 512
    // threads, two to a CU, 24 x 32768 136 / 132.  Half and twice the step are worse.)
    if (stagger && (int)blockIdx.x < kCUs * (1024 / NTHR)) {
        const long long start = wall_clock64() + (long long)(blockIdx.x / kCUs) * stagger;
        while (wall_clock64() < start) __builtin_amdgcn_s_sleep(4);
    }
    const int grp = blockIdx.x / G, part = blockIdx.x % G;
    const int bh = tensors == kBothTensors ? grp >> 1 : grp;
    const bool is_v = tensors == kBothTensors ? grp & 1 : tensors == kOnlyV;  // (workgroup-uniform)
    const int tid = threadIdx.x;
    const int co = tid % LPR, rr = tid / LPR;
    const int row0 = part * C;
    unsigned long long *k_bits = reinterpret_cast<unsigned long long *>(k_sum_part);
    unsigned *v_bits = reinterpret_cast<unsigned *>(v_max_part);
    uint4 raw[NU];

    if (!is_v) {
        // ---- K: thread owns channels co*8.. of rows row0 + it*RP + rr ----
        const uint16_t *Kh = K + (bh / H) * k_st.b + (bh % H) * k_st.h;
        // (all sixteen loads are issued before the first is waited for: rows past the end are loaded from the
        // head's last row and zeroed afterwards — a branch around a load would make each load wait for itself)
        const int nrow = min(max((N - row0 - rr + RP - 1) / RP, 0), NU);  // this thread's rows that exist
        {
            const uint16_t *last = Kh + (int64_t)(N - 1) * k_st.n + co * 8;
            const uint16_t *p = Kh + (int64_t)(row0 + rr) * k_st.n + co * 8;
            const int64_t step = (int64_t)RP * k_st.n;
#pragma unroll
            for (int it = 0; it < NU; ++it) raw[it] = *reinterpret_cast<const uint4 *>(it < nrow ? p + it * step : last);
        }
#pragma unroll
        for (int it = 0; it < NU; ++it)
            if (it >= nrow) raw[it] = make_uint4(0u, 0u, 0u, 0u);
        double(*smd)[D] = reinterpret_cast<double(*)[D]>(smem);
        {
            double acc[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] = 0.0;
#pragma unroll
            for (int it = 0; it < NU; ++it) {
                float f[8];
                unpack8<BF16>(raw[it], f);
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[j] += (double)f[j];
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) smd[rr][co * 8 + j] = acc[j];
        }
        __syncthreads();
        if (tid < D) {
            double a = smd[0][tid];
            for (int i = 1; i < RP; ++i) a += smd[i][tid];
            if (G == 1) {  // the head is this workgroup's alone: nobody to meet
                const float mu = (float)(a / (double)N);
                k_mean[(size_t)bh * D + tid] = mu;
                stat[tid] = mu;
            } else {
                put_shared(&k_bits[((size_t)bh * G + part) * D + tid], tag_bits(a));
            }
        }
        const long long t0 = wall_clock64();
        bool there = G == 1 || resident_wait(k_bits + (size_t)bh * G * D, D, G, wait_ticks, t0);
        if (there && G > 1) {
            // the G partial sums in index order, NTHR / D threads per channel (eight loads in flight: each is a
            // round trip to memory); repeated in the rare case that a word of a partial lags behind its element 0
            const int c = tid % D, share = tid / D;
            constexpr int SHARES = NTHR / D;
            double s;
            for (;;) {
                s = 0.0;
                int v = 0;
                for (int i0 = share; i0 < G; i0 += 8 * SHARES) {
                    unsigned long long t[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        t[u] = get_shared(&k_bits[((size_t)bh * G + min(i0 + u * SHARES, G - 1)) * D + c]);
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        if (t[u] == 0) v = 1;
                        if (i0 + u * SHARES < G) s += __builtin_bit_cast(double, t[u]);
                    }
                }
                const bool late = wall_clock64() - t0 >= wait_ticks;
                if (!__syncthreads_or(v)) break;
                if (__syncthreads_or(late)) {
                    there = false;
                    break;
                }
                __builtin_amdgcn_s_sleep(8);
            }
            if (there) {
                double *sd = reinterpret_cast<double *>(smem);
                sd[tid] = s;
                __syncthreads();
                if (share == 0) {
                    for (int k = 1; k < SHARES; ++k) s += sd[k * D + c];
                    const float mu = (float)(s / (double)N);
                    if (part == 0) k_mean[(size_t)bh * D + c] = mu;
                    stat[c] = mu;
                }
            }
        }
        if (!there) {
            // alone: the column sums of the whole head, from global memory
            double acc[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] = 0.0;
#pragma unroll 1
            for (int r = rr; r < N; r += RP) {
                float f[8];
                unpack8<BF16>(*reinterpret_cast<const uint4 *>(Kh + r * k_st.n + co * 8), f);
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[j] += (double)f[j];
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) smd[rr][co * 8 + j] = acc[j];
            __syncthreads();
            if (tid < D) {
                double a = smd[0][tid];
                for (int i = 1; i < RP; ++i) a += smd[i][tid];
                const float mu = (float)(a / (double)N);
                if (part == 0) k_mean[(size_t)bh * D + tid] = mu;
                stat[tid] = mu;
            }
        }
        __syncthreads();

        // ---- codes: the quantiser of quant_int8_body on the resident rows, one K block after the other, the smoothed values of a block in
        // registers between its maximum and its codes.  With 16 blocks (512 threads, d = 64) the maxima of all of them come first: one
        // barrier instead of 16, the smoothed values are made twice (128 heads x 1024 tokens 19.4 -> 16.5 us; with 4 or 8 blocks
        // up to 1.5 % slower) ----
        constexpr int NB = C / kBK;    // K blocks of the chunk
        constexpr int IPB = kBK / RP;  // passes per block
        constexpr bool ALL_MAXIMA = NB >= 16 && !(WITH_Q && QMAX == 127);
        constexpr float kRange = (float)QMAX;
        float mu[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) mu[j] = stat[co * 8 + j];
        keep_packed(raw);
        float x[IPB][8];
        const auto smooth = [&](int b) {
#pragma unroll
            for (int i = 0; i < IPB; ++i) {
                unpack8<BF16>(raw[b * IPB + i], x[i]);
#pragma unroll
                for (int j = 0; j < 8; ++j) x[i][j] = x[i][j] - mu[j];
            }
        };
        const auto block_max = [&](int b) {  // this wavefront's part of it goes to LDS
            float a = 0.0f;
#pragma unroll
            for (int i = 0; i < IPB; ++i)
                if (b * IPB + i < nrow) {  // rows past the end do not count
#pragma unroll
                    for (int j = 0; j < 8; ++j) a = fmaxf(a, fabsf(x[i][j]));
                }
            a = wave_max_abs(a);
            if ((tid & 63) == 0) wmax[b][tid >> 6] = a;
        };
        if constexpr (ALL_MAXIMA) {
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                smooth(b);
                block_max(b);
            }
            __syncthreads();
            keep_packed(raw);
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int blk = part * NB + b;  // (workgroup-uniform)
            if (blk >= nK) break;
            smooth(b);
            if constexpr (!ALL_MAXIMA) {
                block_max(b);
                __syncthreads();  // (every block has its own row of wmax: one barrier per block)
            }
            float a = wmax[b][0];
#pragma unroll
            for (int w = 1; w < NW; ++w) a = fmaxf(a, wmax[b][w]);
            const float rcp = a > 0.0f ? kRange / a : 0.0f;
            if (tid == 0) k_scale[(size_t)bh * nK + blk] = a / kRange;
#pragma unroll
            for (int i = 0; i < IPB; ++i) {
                const int it = b * IPB + i;
                const int r = row0 + it * RP + rr;
                if (it < nrow) *reinterpret_cast<uint2 *>(k_codes + ((size_t)bh * N + r) * D + co * 8) = int8_codes(x[i], rcp);
            }
        }
    } else {
        // ---- V: a thread owns 8 channels of four key quads.  Straight from registers: the keys 16t + 4g + i (t, i < 4) of a half tile of 64,
        // whose codes are 16 adjacent bytes of each channel's row.  Through LDS: the quads lie 4 RP keys apart, a round transposes
        // TP tiles and stores them in one piece ----
        const uint16_t *Vh = V + (bh / H) * v_st.b + (bh % H) * v_st.h;
        constexpr bool CAN_LDS = D == 64 || NTHR == 256;
        const bool v_lds = CAN_LDS && v_through_lds;
        const int half = rr >> 2, g = rr & 3;
        uint32_t exists = 0u;  // bit q = 4t + i
        {
            const uint16_t *last = Vh + (int64_t)(N - 1) * v_st.n + co * 8;
            const int rbase = row0 + (v_lds ? 4 * rr : 64 * half + 4 * g), apart = v_lds ? 4 * RP : 16;
            const uint16_t *p = Vh + (int64_t)rbase * v_st.n + co * 8;
#pragma unroll
            for (int q = 0; q < NU; ++q) {
                const bool ok = rbase + apart * (q >> 2) + (q & 3) < N;
                exists |= (ok ? 1u : 0u) << q;
                raw[q] = *reinterpret_cast<const uint4 *>(ok ? p + (q >> 2) * (apart * v_st.n) + (q & 3) * v_st.n : last);
            }
        }
#pragma unroll
        for (int q = 0; q < NU; ++q)
            if (!((exists >> q) & 1u)) raw[q] = make_uint4(0u, 0u, 0u, 0u);
        float(*smf)[D] = reinterpret_cast<float(*)[D]>(smem);
        {
            float acc[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] = 0.0f;
#pragma unroll
            for (int it = 0; it < NU; ++it) {
                float f[8];
                unpack8<BF16>(raw[it], f);
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[j] = fmaxf(acc[j], fabsf(f[j]));
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) smf[rr][co * 8 + j] = acc[j];
        }
        __syncthreads();
        if (tid < D) {
            float a = smf[0][tid];
            for (int i = 1; i < RP; ++i) a = fmaxf(a, smf[i][tid]);
            if (G == 1) {
                v_scale[(size_t)bh * D + tid] = a / v_r;
                stat[tid] = a > 0.0f ? v_r / a : 0.0f;
            } else {
                put_shared(&v_bits[((size_t)bh * G + part) * D + tid], tag_bits(a));
            }
        }
        const long long t0 = wall_clock64();
        bool there = G == 1 || resident_wait(v_bits + (size_t)bh * G * D, D, G, wait_ticks, t0);
        if (there && G > 1) {
            const int c = tid % D, share = tid / D;
            constexpr int SHARES = NTHR / D;
            float a;
            for (;;) {
                a = 0.0f;
                int v = 0;
                for (int i0 = share; i0 < G; i0 += 16 * SHARES) {
                    unsigned t[16];
#pragma unroll
                    for (int u = 0; u < 16; ++u)
                        t[u] = get_shared(&v_bits[((size_t)bh * G + min(i0 + u * SHARES, G - 1)) * D + c]);
#pragma unroll
                    for (int u = 0; u < 16; ++u) {
                        if (t[u] == 0u) v = 1;
                        a = fmaxf(a, fabsf(__builtin_bit_cast(float, t[u])));  // (a partial taken twice does not change a maximum)
                    }
                }
                const bool late = wall_clock64() - t0 >= wait_ticks;
                if (!__syncthreads_or(v)) break;
                if (__syncthreads_or(late)) {
                    there = false;
                    break;
                }
                __builtin_amdgcn_s_sleep(8);
            }
            if (there) {
                float *sf = reinterpret_cast<float *>(smem);
                sf[tid] = a;
                __syncthreads();
                if (share == 0) {
                    for (int k = 1; k < SHARES; ++k) a = fmaxf(a, sf[k * D + c]);
                    if (part == 0) v_scale[(size_t)bh * D + c] = a / v_r;
                    stat[c] = a > 0.0f ? v_r / a : 0.0f;
                }
            }
        }
        if (!there) {
            float acc[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] = 0.0f;
#pragma unroll 1
            for (int r = rr; r < N; r += RP) {
                float f[8];
                unpack8<BF16>(*reinterpret_cast<const uint4 *>(Vh + r * v_st.n + co * 8), f);
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[j] = fmaxf(acc[j], fabsf(f[j]));
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) smf[rr][co * 8 + j] = acc[j];
            __syncthreads();
            if (tid < D) {
                float a = smf[0][tid];
                for (int i = 1; i < RP; ++i) a = fmaxf(a, smf[i][tid]);
                if (part == 0) v_scale[(size_t)bh * D + tid] = a / v_r;
                stat[tid] = a > 0.0f ? v_r / a : 0.0f;
            }
        }
        __syncthreads();

        float rc[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) rc[j] = stat[co * 8 + j];
        keep_packed(raw);
        if (v_lds) {
            constexpr int UNITS = 32 * LPR;  // quads of keys x 8 channels of a tile
            constexpr int UPT = UNITS > NTHR ? UNITS / NTHR : 1, TP = UNITS > NTHR ? 1 : NTHR / UNITS, ROUNDS = C / kW / TP;
            static_assert(ROUNDS * UPT * 4 == NU, "a workgroup's chunk is 16 uint4 per thread");
            static_assert(TP * D * 128 <= NTHR * 64, "the tiles fit in LDS");
            uint32_t *tile = reinterpret_cast<uint32_t *>(smem) + tid / UNITS * D * 32;
#pragma unroll
            for (int rd = 0; rd < ROUNDS; ++rd) {
                const int T = (part * ROUNDS + rd) * TP;  // (workgroup-uniform) first tile of the round
                if (T >= nT) break;
#pragma unroll
                for (int k = 0; k < UPT; ++k) {
                    const int kq = (tid + NTHR * k) % UNITS / LPR;
                    uint32_t *dst = tile + co * 8 * 32 + (kq >> 4) * 16 + (kq & 3) * 4 + (kq >> 2 & 3);
#pragma unroll
                    for (int j2 = 0; j2 < 4; ++j2) {
                        const uint2 w = v_pair_codes<BF16>(&raw[(rd * UPT + k) * 4], rc, j2);
                        dst[2 * j2 * 32] = w.x;
                        dst[(2 * j2 + 1) * 32] = w.y;
                    }
                }
                __syncthreads();
                uint4 *dst = reinterpret_cast<uint4 *>(Vt + ((size_t)bh * nT + T) * D * 128);
#pragma unroll
                for (int k = 0; k < TP * D * 8 / NTHR; ++k) {
                    const int e = tid + NTHR * k;
                    if (TP == 1 || T + e / (D * 8) < nT) dst[e] = reinterpret_cast<const uint4 *>(smem)[e];
                }
                __syncthreads();
            }
            return;
        }
        const int T = (row0 + 64 * half) >> 7;
        if (T < nT)
            v_codes<BF16>(raw, rc, Vt + (((size_t)bh * nT + T) * D + co * 8) * 128 + 64 * (half & 1) + 16 * g);
    }
}

// ---------------------------------------------------------------------------
// Two launches for small calls: partial column statistics of the chunks that the single-read kernel's workgroups of 256 threads would
// hold, then codes in workgroups of one K block or V tile that add the head's partials themselves.  Nothing is cleared, nobody
// waits for anybody, and there are many times as many workgroups; the tokens are read a second time (from the caches, in a
// small call) and every workgroup of a head reads its G partials.
// ---------------------------------------------------------------------------
constexpr int kChunkThreads = 512;
template <int D>
constexpr int chunk_tokens() {
    return resident_tokens(256, D);
}

// Grid: B*H*G workgroups per tensor (K and V groups in turn, or one tensor alone), then, WITH_Q, those of Q: two blocks each.  (Calls
// without Q have a kernel without Q's code: it is what they wait for when they start, 2 heads x 1024 x 128 8.04 -> 7.92 us.)
template <bool BF16, int D, bool WITH_Q>
__global__ __launch_bounds__(kChunkThreads) void chunk_stats_kernel(const uint16_t *__restrict__ K, Strides k_st,
                                                                   const uint16_t *__restrict__ V, Strides v_st, int H, int N, int G,
                                                                   double *__restrict__ k_sum_part, float *__restrict__ v_max_part,
                                                                   int tensors, QuantQ q) {
    constexpr int LPR = D / 8, RP = kChunkThreads / LPR, C = chunk_tokens<D>(), NU = C / RP;
    constexpr int SHARES = kChunkThreads / D, RS = RP / SHARES;  // threads that share a channel, rows of partial sums each adds
    __shared__ __attribute__((aligned(16))) double smem[RP * D];
    const int tid = threadIdx.x;
    if constexpr (WITH_Q) {
        if ((int)blockIdx.x >= q.first) {
            const int team = tid >> 8, wgs = (q.n_blocks + 1) / 2, x = blockIdx.x - q.first, bh = x / wgs, blk = x % wgs * 2 + team;
            if (q.mean)
                block_mean_body<BF16, D>(q.x, q.st, q.H, q.N, q.n_blocks, q.mean, smem + team * block_mean_doubles<D>(), bh, blk,
                                         tid & 255);
            else
                quant_int8_body<BF16, D, kBQ, 0, 127>(q.x, q.st, q.H, nullptr, q.codes, q.scale, q.N, q.n_blocks,
                                                      reinterpret_cast<float *>(smem) + 4 * team, bh, blk, tid & 255);
            return;
        }
    }
    const int grp = blockIdx.x / G, part = blockIdx.x % G;
    const int bh = tensors == kBothTensors ? grp >> 1 : grp;
    const bool is_v = tensors == kBothTensors ? grp & 1 : tensors == kOnlyV;  // (workgroup-uniform)
    const int co = tid % LPR, rr = tid / LPR;
    const Strides st = is_v ? v_st : k_st;
    const uint16_t *X = (is_v ? V : K) + (bh / H) * st.b + (bh % H) * st.h + co * 8;
    uint4 raw[NU];
#pragma unroll
    for (int it = 0; it < NU; ++it)
        raw[it] = *reinterpret_cast<const uint4 *>(X + (int64_t)min(part * C + it * RP + rr, N - 1) * st.n);
#pragma unroll
    for (int it = 0; it < NU; ++it)  // (rows past the end change neither a sum nor a maximum of |.|)
        if (part * C + it * RP + rr >= N) raw[it] = make_uint4(0u, 0u, 0u, 0u);
    const int c = tid % D, share = tid / D;
    const size_t o = ((size_t)bh * G + part) * D + c;
    if (!is_v) {
        double acc[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int it = 0; it < NU; ++it) {
            float f[8];
            unpack8<BF16>(raw[it], f);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] += (double)f[j];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) smem[rr * D + co * 8 + j] = acc[j];
        __syncthreads();
        double a = smem[share * RS * D + c];
#pragma unroll
        for (int i = 1; i < RS; ++i) a += smem[(share * RS + i) * D + c];
        __syncthreads();
        smem[tid] = a;
        __syncthreads();
        if (share == 0) {
#pragma unroll
            for (int k = 1; k < SHARES; ++k) a += smem[k * D + c];
            k_sum_part[o] = a;
        }
    } else {
        float *sm = reinterpret_cast<float *>(smem);
        float acc[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int it = 0; it < NU; ++it) {
            float f[8];
            unpack8<BF16>(raw[it], f);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] = fmaxf(acc[j], fabsf(f[j]));
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) sm[rr * D + co * 8 + j] = acc[j];
        __syncthreads();
        float a = sm[share * RS * D + c];
#pragma unroll
        for (int i = 1; i < RS; ++i) a = fmaxf(a, sm[(share * RS + i) * D + c]);
        __syncthreads();
        sm[tid] = a;
        __syncthreads();
        if (share == 0) {
#pragma unroll
            for (int k = 1; k < SHARES; ++k) a = fmaxf(a, sm[k * D + c]);
            v_max_part[o] = a;
        }
    }
}

// Grid (nK + chunks of V, B*H): K blocks, then V chunks (either count may be 0).
template <bool BF16, int D, int QMAX>
__global__ __launch_bounds__(256) void chunk_codes_kernel(const uint16_t *__restrict__ K, Strides k_st,
                                                          const uint16_t *__restrict__ V, Strides v_st, int H, int N, int G,
                                                          const double *__restrict__ k_sum_part,
                                                          const float *__restrict__ v_max_part, float *__restrict__ k_mean,
                                                          float *__restrict__ v_scale, float v_r, int8_t *__restrict__ k_codes,
                                                          float *__restrict__ k_scale, int nK, uint8_t *__restrict__ Vt, int nT) {
    constexpr int LPR = D / 8, RP = 256 / LPR, SHARES = 256 / D;
    __shared__ double part_sum[256];
    __shared__ float stat[D], wmax[4];
    const int tid = threadIdx.x, bh = blockIdx.y, x = blockIdx.x;  // (workgroup-uniform branch)
    const int co = tid % LPR, rr = tid / LPR, c = tid % D, share = tid / D;
    if (x < nK) {
        constexpr int ITER = kBK / RP;
        constexpr float kRange = (float)QMAX;
        const uint16_t *Kh = K + (bh / H) * k_st.b + (bh % H) * k_st.h + co * 8;
        const int row0 = x * kBK + rr;
        uint4 raw[ITER];  // (in flight under the partials)
#pragma unroll
        for (int it = 0; it < ITER; ++it)
            raw[it] = *reinterpret_cast<const uint4 *>(Kh + (int64_t)min(row0 + it * RP, N - 1) * k_st.n);
        double s = 0.0;
        for (int i0 = share; i0 < G; i0 += 8 * SHARES) {
            double t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = k_sum_part[((size_t)bh * G + min(i0 + u * SHARES, G - 1)) * D + c];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (i0 + u * SHARES < G) s += t[u];
        }
        part_sum[tid] = s;
        __syncthreads();
        if (share == 0) {
#pragma unroll
            for (int k = 1; k < SHARES; ++k) s += part_sum[k * D + c];
            const float mu = (float)(s / (double)N);
            if (x == 0) k_mean[(size_t)bh * D + c] = mu;
            stat[c] = mu;
        }
        __syncthreads();
        float y[ITER][8], a = 0.0f;
#pragma unroll
        for (int it = 0; it < ITER; ++it) {
            unpack8<BF16>(raw[it], y[it]);
#pragma unroll
            for (int j = 0; j < 8; ++j) y[it][j] = y[it][j] - stat[co * 8 + j];
            if (row0 + it * RP < N) {
#pragma unroll
                for (int j = 0; j < 8; ++j) a = fmaxf(a, fabsf(y[it][j]));
            }
        }
        a = wave_max_abs(a);
        if ((tid & 63) == 0) wmax[tid >> 6] = a;
        __syncthreads();
        a = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
        const float rcp = a > 0.0f ? kRange / a : 0.0f;
        if (tid == 0) k_scale[(size_t)bh * nK + x] = a / kRange;
#pragma unroll
        for (int it = 0; it < ITER; ++it) {
            const int r = row0 + it * RP;
            if (r < N)
                *reinterpret_cast<uint2 *>(k_codes + ((size_t)bh * N + r) * D + co * 8) = int8_codes(y[it], rcp);
        }
    } else {
        const int row0 = (x - nK) * chunk_tokens<D>(), half = rr >> 2, g = rr & 3;
        const uint16_t *Vh = V + (bh / H) * v_st.b + (bh % H) * v_st.h + co * 8;
        uint4 raw[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int r = row0 + 64 * half + 4 * g + 16 * (q >> 2) + (q & 3);
            raw[q] = *reinterpret_cast<const uint4 *>(Vh + (int64_t)min(r, N - 1) * v_st.n);
        }
#pragma unroll
        for (int q = 0; q < 16; ++q)
            if (row0 + 64 * half + 4 * g + 16 * (q >> 2) + (q & 3) >= N) raw[q] = make_uint4(0u, 0u, 0u, 0u);
        float a = 0.0f;
        for (int i0 = share; i0 < G; i0 += 8 * SHARES) {
            float t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = v_max_part[((size_t)bh * G + min(i0 + u * SHARES, G - 1)) * D + c];
#pragma unroll
            for (int u = 0; u < 8; ++u) a = fmaxf(a, t[u]);  // (a partial taken twice does not change a maximum)
        }
        float *part_max = reinterpret_cast<float *>(part_sum);
        part_max[tid] = a;
        __syncthreads();
        if (share == 0) {
#pragma unroll
            for (int k = 1; k < SHARES; ++k) a = fmaxf(a, part_max[k * D + c]);
            if (x == nK) v_scale[(size_t)bh * D + c] = a / v_r;
            stat[c] = a > 0.0f ? v_r / a : 0.0f;
        }
        __syncthreads();
        float rc[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) rc[j] = stat[co * 8 + j];
        const int T = (row0 + 64 * half) >> 7;
        if (T < nT) v_codes<BF16>(raw, rc, Vt + (((size_t)bh * nT + T) * D + co * 8) * 128 + 64 * (half & 1) + 16 * g);
    }
}

// which path the K/V quantisers take (0: by shape) and how long a workgroup of the single-read kernel waits for its
// partners (ticks of the 100 MHz clock; negative: not at all)
std::atomic<int> g_kv_path{0};
std::atomic<long long> g_kv_wait_ticks{kResidentWaitTicks};

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

template <bool BF16, int D>
hipError_t quant_q_impl(const uint16_t *q, Strides st, int8_t *q_i8, float *q_scale, int BH, int H, int N,
                        hipStream_t stream) {
    const int nQ = cdiv(N, kBQ);
    // (a block that is half empty at least: its loads would repeat the last row; 1467 heads x 4, d 128 4.9 -> 4.05 us, 1000 x 40 5.05 -> 4.4)
    if (N <= kBQ / 2)
        quant_int8_kernel<BF16, D, kBQ / 2, 0, 127><<<dim3(1, BH), 256, 0, stream>>>(q, st, H, nullptr, q_i8, q_scale, N, 1);
    else
        quant_int8_kernel<BF16, D, kBQ, 0, 127><<<dim3(nQ, BH), 256, 0, stream>>>(q, st, H, nullptr, q_i8, q_scale, N, nQ);
    return hipGetLastError();
}

// Threads of the single-read kernel's workgroups; 0: three launches.  (Small calls do not come here: chunks_pay.)  G: workgroups of 256
// threads that a head of one tensor takes (256 tokens each at d = 128, 512 at d = 64); `groups`: heads times tensors.  Every figure:
// three launches / 256 / 512 threads, us.
//   * With few partners two workgroups of 256 are the better neighbours of a CU.  A group of many wants large ones, half as many
//     partials to wait for and read: at d = 128 from about 96 on (K and V, H 8, G 64 34 / 29.6 / 28.9, G 80 39 / 38.6 / 40.6, G 128
//     57 / 56 / 52; H 16, G 128 118 / 120 / 107).  At d = 64 a partial covers twice the tokens and 256 stays ahead up to 128
//     (H 8, G 96 43.5 / 42.6 / 46.5, G 128 55 / 51 / 55; H 3, N 24578 16.8 with 256, 21.5 with 512).
//   * Two workgroups of 256 that become one of 512 have nobody to meet and nothing to clear (d = 128, H 128 15.6 with 512, 20.9 in three
//     launches; d = 64, H 128 20.2 / 17.6 / 16.2).
//   * Beyond 128 workgroups of 256 only those of 512 come into question.  512 of those are resident at once; a second round that is
//     partly empty costs what the second read of the three launches does (d = 128, K and V, H 4, G 160, 640 workgroups
//     39.8 / - / 43.3; H 4, G 256, 1024 57.7 / - / 54.2; H 1, G 160, 160 24.1 / - / 19.2;
//     inputs that are not in the last-level cache: H 4, G 192 50.8 / - / 50.9, H 8, G 192, 1536 102 / - / 90).
//   * K or V alone: three short launches are independent of each other's workgroups, where the single read has a clear and
//     a meeting, 3 to 4 us that fewer workgroups than fill the chip do not win back (d = 128, K, H 1, G 128 16.3 / 17.2 / 17.5).
enum class Quantise { kBoth, kOnlyK, kOnlyV, kKWithQ };
constexpr int wide_above(int d) { return d == 128 ? 96 : 128; }  // the largest G that is better off with 256 threads
inline int resident_threads(Quantise what, int groups, int N, int d) {
    const int path = g_kv_path.load();
    const int G = resident_group_size(N, d, 256);
    const long wgs = (long)groups * G, wgs512 = (long)groups * resident_group_size(N, d, 512);
    if (path == 1) return 0;
    const bool wide = G > wide_above(d);
    if (path == 2) return G == 2 || wide ? 512 : 256;
    if (G == 1) return 256;
    if (G == 2) return 512;
    if (G > kResidentMaxGroup) return 0;
    if (d == 128) {
        if (!wide) return 256;
        if (what == Quantise::kOnlyK && wgs512 < kCUs / 2) return 0;
        return what != Quantise::kKWithQ && G > 128 && wgs512 > 2 * kCUs && wgs512 < 4 * kCUs ? 0 : 512;
    }
    switch (what) {
        case Quantise::kOnlyK: return !wide && (G <= 48 || wgs >= 2 * kCUs) ? 256 : 0;
        case Quantise::kOnlyV: return wide ? 512 : 256;
        case Quantise::kKWithQ: return wide ? 0 : 256;
        default: return !wide ? 256 : wgs512 >= 4 * kCUs ? 512 : 0;
    }
}

// Whether the two launches over chunks are the fastest form.  They are while the workgroups leave CUs idle, where the single read is a
// clear, a meeting and a chain of K blocks; beyond, the second read costs more.  G as above, wgs: workgroups of 256 threads per
// tensor.  Single read (or three launches) / two, us: K and V, d = 128, H 2, G 4 12.1 / 8.2, G 63 15.1 / 13.8, H 8, G 16 14.0 / 10.9, G 32
// (256 workgroups) 18.4 / 20.0; d = 64, H 2, G 4 13.7 / 8.1, H 32, G 4 14.2 / 12.3.  A head that one workgroup holds meets nobody: K and V,
// G 1 7.4 / 7.8.  K alone d = 128, H 8, G 32 14.3 / 12.5, H 32, G 16 (512) 18.7 / 19.0; d = 64, H 2, G 1 8.5 / 6.7, H 128, G 2 13.4 / 12.5.
// V alone G 2 7.0 / 7.5, H 32, G 4 10.7 / 8.2, G 16 (512) 16.4 / 13.9, H 32, G 32 (1024) 24.7 / 29.2.  K with Q, d = 128, H 2, G 4
// 11.3 / 7.6, H 48, G 4 (192) 16.0 / 14.9, H 64, G 4 (256) 17.2 / 17.2, H 8, G 32 18.3 / 18.4, H 64, G 2 12.7 / 11.9, H 100, G 2 13.9 / 15.0 (the single
// read of G 2 meets nobody); d = 64, H 48, G 4 16.9 / 15.5, H 64, G 4 in the last-level cache 15.8 / 16.6, H 96, G 2 15.9 / 15.0, H 2, G 100 19.3 / 20.9,
// H 32, G 1 8.8 / 7.2, but with few K blocks in the one workgroup of a head (one launch / two) K alone H 8 x 64 tokens 5.0 / 6.1, x 256
// 6.2 / 6.5, H 1 x 320 6.4 / 6.3, H 32 x 512 8.0 / 6.8.  Every workgroup of a head reads the G partials: K alone, d = 64, H 2, G 118 16.4 / 17.6; V alone, beyond one
// workgroup per CU and where the single read has 512 threads, d = 128, H 4, G 96 18.3 / 17.3, G 120 17.5 / 19.9, H 2, G 160 16.5 / 17.3, G 256 18.8 /
// 22.0, d = 64, H 2, G 256 18.1 / 19.0; with one per CU H 2, G 128 14.8 / 13.8, H 1, G 200 14.9 / 14.8; beyond the single read's reach three
// launches are no better, H 1, G 320 27.6 / 20.9, G 512 31.2 / 27.2 (tensors that are not in the last-level cache).
inline bool chunks_pay(Quantise what, int heads, int N, int d) {
    if (g_kv_path.load() != 0) return false;
    const int G = resident_group_size(N, d, 256);
    const long wgs = (long)heads * G;
    if (G == 1) return d == 64 && (what == Quantise::kOnlyK || what == Quantise::kKWithQ) && heads <= kCUs / 4 && N > 4 * kBK;
    switch (what) {
        case Quantise::kOnlyK: return wgs <= kCUs / 2 || (wgs <= kCUs && G <= 64);
        case Quantise::kOnlyV: return G > 2 && (wgs <= kCUs || (wgs <= 2 * kCUs && (G <= wide_above(d) || G > kResidentMaxGroup)));
        case Quantise::kKWithQ: return wgs <= kCUs / 2 || (wgs <= 3 * kCUs / 4 && G <= 64 && (G > 2 || d == 64));
        default: return wgs <= (G == 2 ? kCUs / 4 : kCUs / 2);
    }
}

// The outputs in two launches (chunk_stats_kernel, chunk_codes_kernel).
template <bool BF16, int D, int QMAX>
hipError_t launch_chunks(const uint16_t *k, Strides k_st, const uint16_t *v, Strides v_st, int8_t *k_i8, float *k_scale, float *k_mean,
                         uint8_t *v_fp8, float *v_scale, float v_r, int BH, int H, int N, hipStream_t stream, const QuantScratch &ws,
                         int tensors, QuantQ q = QuantQ{}) {
    const int G = resident_group_size(N, D, 256);
    const int nK = tensors == kOnlyV ? 0 : cdiv(N, kBK), nV = tensors == kOnlyK ? 0 : G;
    q.first = (tensors == kBothTensors ? 2 * BH : BH) * G;
    if (q.x)
        chunk_stats_kernel<BF16, D, true><<<q.first + q.workgroups(2), kChunkThreads, 0, stream>>>(
            k, k_st, v, v_st, H, N, G, ws.k_sum_part, ws.v_max_part, tensors, q);
    else
        chunk_stats_kernel<BF16, D, false><<<q.first, kChunkThreads, 0, stream>>>(
            k, k_st, v, v_st, H, N, G, ws.k_sum_part, ws.v_max_part, tensors, q);
    chunk_codes_kernel<BF16, D, QMAX><<<dim3(nK + nV, BH), 256, 0, stream>>>(
        k, k_st, v, v_st, H, N, G, ws.k_sum_part, ws.v_max_part, k_mean, v_scale, v_r, k_i8, k_scale, nK, v_fp8, cdiv(N, kW));
    return hipGetLastError();
}

// The outputs from one read of the tensors (quant_kv_resident_kernel).
template <bool BF16, int D, int QMAX, int NTHR>
hipError_t launch_resident_n(const uint16_t *k, Strides k_st, const uint16_t *v, Strides v_st, int8_t *k_i8, float *k_scale,
                             float *k_mean, uint8_t *v_fp8, float *v_scale, float v_r, int BH, int H, int N,
                             hipStream_t stream, const QuantScratch &ws, int tensors, QuantQ q) {
    const int G = resident_group_size(N, D, NTHR);
    const int nK = cdiv(N, kBK), nT = cdiv(N, kW);
    const long long wait_ticks = g_kv_wait_ticks.load();
    // the partials of K and V together lie back to back, as many as this launch has (the buffers are laid out for groups of 256 threads,
    // twice as many); K alone and V alone keep to their own buffers
    const size_t n = (size_t)BH * G * D;
    float *v_part = tensors == kBothTensors ? reinterpret_cast<float *>(ws.k_sum_part + n) : ws.v_max_part;
    if (G > 1) {
        void *from = tensors == kOnlyV ? (void *)v_part : (void *)ws.k_sum_part;
        const int words = (int)(n * (tensors == kBothTensors ? 12 : tensors == kOnlyK ? 8 : 4) / 16);
        zero_words_kernel<<<cdiv(words, 256), 256, 0, stream>>>(static_cast<uint4 *>(from), words);
    }
    q.first = (tensors == kBothTensors ? 2 * BH : BH) * G;
    // Where it pays to start the workgroups of a CU apart, from two rounds on (time with / without).  Groups that meet: 512 threads 0.96 .. 1.01;
    // 256 threads from 8 chunks on 0.95 .. 1.02, but not if there are exactly two rounds, whose end is only later (128 heads x 4096 K alone,
    // d 128 48.9 / 46.3 us, K and V 64 x 4096 48.2 / 46.0), nor V alone at d 64 below four (2.0 .. 2.3 rounds 1.01 .. 1.07); 3 to 6 chunks
    // 0.97 .. 1.05 below four rounds and 0.96 .. 1.00 from there on.  A
    // head that one workgroup holds meets nobody, and its start is only late: 256 threads, K and V of 1024 heads x 129 x 128 27.9 / 24.9
    // us, x 256 39.1 / 36.2, 2048 x 129 45.4 / 42.5; 512 threads, 512 x 257 30.5 / 27.6, x 300 31.4 / 28.9; only from three quarters of
    // a chunk on, when a CU's two load and store long enough, 512 x 400 36.6 / 36.1, 1024 x 400 66.7 / 67.7, 600 x 512 46.2 / 48.3, d 64 512 x 800
    // 38.7 / 40.1, x 1024 43.6 / 45.2.
    constexpr int kSlots = kCUs * (1024 / NTHR);
    const bool apart = G == 1 ? NTHR == 512 && 4L * N >= 3 * resident_tokens(NTHR, D)
                              : NTHR == 512 || q.first >= 4 * kSlots ||
                                    (q.first > 2 * kSlots && G >= 8 && !(D == 64 && tensors == kOnlyV));
    const int stagger = !apart || q.first < 2 * kSlots ? 0 : NTHR == 256 ? 400 : 700;
    // The codes of V through LDS or straight from registers.  LDS costs a workgroup a barrier and bank conflicts, the registers' 16-byte
    // pieces, 128 bytes apart, cost the memory where it is the limit.  By rounds of V's workgroups (us, LDS / registers): d 128, 256 threads,
    // V alone 300 heads x 1500 (1.8) 42.7 / 40.0, 200 x 3021 (2.3) 54.0 / 53.8, 300 x 2700 (3.2) 67.8 / 70.0, 700 x 3021 (8.2) 151 / 165, K
    // and V 128 x 4096 (2.0) 84.5 / 83.8, 300 x 2700 123.0 / 126.6; 512 threads 48 x 32768 (6) 277 / 254.  d 64, 256 threads, V alone 300 x
    // 1500 (0.9) 25.1 / 24.2, 2048 x 512 (2.0) 34.6 / 36.8, K and V 700 x 6042 (8.2) 292 / 297; a head of up to 256 tokens, whose chunk half
    // of the threads have, 16 x 100 4.4 / 4.9, x 500 6.1 / 5.6; 512 threads, K and V 4 x 131000 (1.0) 51.2 / 51.0, 8 x 130000 (2.0) 104.7 / 106.4,
    // 40 x 100000 (7.7) 342 / 377.
    const long v_wgs = tensors == kOnlyK ? 0 : (long)BH * G;
    const bool v_lds = D == 128 ? NTHR == 256 && 2 * v_wgs >= 5 * kSlots
                                : NTHR == 256 ? v_wgs >= kSlots || (G == 1 && N <= 256) : 8 * v_wgs >= 15 * kSlots;
#define SAGE_RESIDENT(Q, GRID)                                                                                          \
    quant_kv_resident_kernel<BF16, D, QMAX, NTHR, Q><<<GRID, NTHR, 0, stream>>>(                                        \
        k, k_st, v, v_st, H, N, G, ws.k_sum_part, v_part, k_mean, v_scale, v_r, k_i8, k_scale, nK, v_fp8, nT,     \
        wait_ticks, stagger, v_lds, tensors, q)
    if (q.x) SAGE_RESIDENT(true, q.first + q.workgroups(NTHR / 256));
    else SAGE_RESIDENT(false, q.first);
#undef SAGE_RESIDENT
    return hipGetLastError();
}

template <bool BF16, int D, int QMAX>
hipError_t launch_resident(int threads, const uint16_t *k, Strides k_st, const uint16_t *v, Strides v_st, int8_t *k_i8,
                           float *k_scale, float *k_mean, uint8_t *v_fp8, float *v_scale, float v_r, int BH, int H, int N,
                           hipStream_t stream, const QuantScratch &ws, int tensors, const QuantQ &q = QuantQ{}) {
    if (resident_group_size(N, D, 256) > kResidentMaxGroup) return hipErrorInvalidValue;
    if (threads == 512)
        return launch_resident_n<BF16, D, QMAX, 512>(k, k_st, v, v_st, k_i8, k_scale, k_mean, v_fp8, v_scale, v_r, BH, H, N,
                                                     stream, ws, tensors, q);
    return launch_resident_n<BF16, D, QMAX, 256>(k, k_st, v, v_st, k_i8, k_scale, k_mean, v_fp8, v_scale, v_r, BH, H, N, stream,
                                                 ws, tensors, q);
}

// K and, with `q`, Q of the same shape: their codes in K's launch or, where K takes the three launches, in one of their own.
template <bool BF16, int D>
hipError_t quant_k_impl(const uint16_t *k, Strides st, int8_t *k_i8, float *k_scale, float *k_mean, int BH, int H,
                        int N, hipStream_t stream, const QuantScratch &ws, const QuantQ &q) {
    const Quantise what = q.x ? Quantise::kKWithQ : Quantise::kOnlyK;
    if (chunks_pay(what, BH, N, D))
        return launch_chunks<BF16, D, 127>(k, st, nullptr, st, k_i8, k_scale, k_mean, nullptr, nullptr, 1.0f, BH, H, N, stream, ws,
                                           kOnlyK, q);
    const int threads = resident_threads(what, BH, N, D);
    if (threads && resident_group_size(N, D, 256) <= kResidentMaxGroup)
        return launch_resident<BF16, D, 127>(threads, k, st, nullptr, st, k_i8, k_scale, k_mean, nullptr, nullptr, 0.0f, BH, H, N,
                                             stream, ws, kOnlyK, q);
    const int chunks = cdiv(N, kStatRows);
    const int nK = cdiv(N, kBK);
    colstats_kernel<BF16, D, false><<<dim3(chunks, BH), 256, 0, stream>>>(k, st, H, N, chunks, ws.k_sum_part, nullptr);
    finalize_mean_kernel<<<BH, 1024, 0, stream>>>(ws.k_sum_part, chunks, N, D, k_mean);
    // K right after its statistics pass: its second read can still be served by the last-level cache
    quant_int8_kernel<BF16, D, kBK, 1, 127><<<dim3(nK, BH), 256, 0, stream>>>(k, st, H, k_mean, k_i8, k_scale, N, nK);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess || !q.x ? e : quant_q_impl<BF16, D>(q.x, q.st, q.codes, q.scale, BH, H, N, stream);
}

template <bool BF16, int D>
hipError_t quant_v_impl(const uint16_t *v, Strides st, uint8_t *v_fp8, float *v_scale, float v_r, int BH, int H,
                        int N, hipStream_t stream, const QuantScratch &ws) {
    if (chunks_pay(Quantise::kOnlyV, BH, N, D))
        return launch_chunks<BF16, D, 127>(nullptr, st, v, st, nullptr, nullptr, nullptr, v_fp8, v_scale, v_r, BH, H, N, stream, ws,
                                           kOnlyV);
    const int threads = resident_threads(Quantise::kOnlyV, BH, N, D);
    if (threads && resident_group_size(N, D, 256) <= kResidentMaxGroup)
        return launch_resident<BF16, D, 127>(threads, nullptr, st, v, st, nullptr, nullptr, nullptr, v_fp8, v_scale, v_r, BH, H, N,
                                             stream, ws, kOnlyV);
    const int chunks = cdiv(N, kStatRows);
    const int nT = cdiv(N, kW);
    colstats_kernel<BF16, D, true><<<dim3(chunks, BH), 256, 0, stream>>>(v, st, H, N, chunks, nullptr, ws.v_max_part);
    finalize_vscale_kernel<<<BH, 1024, 0, stream>>>(ws.v_max_part, chunks, D, v_r, v_scale, ws.v_rcp);
    quant_v_kernel<BF16, D><<<dim3(nT, BH), 256, 0, stream>>>(v, st, H, ws.v_rcp, v_fp8, N, nT);
    return hipGetLastError();
}

// K and V of one shape in three launches instead of six (same kernels' bodies, same results)
template <bool BF16, int D, int QMAX>
hipError_t quant_kv_impl(const uint16_t *k, Strides k_st, const uint16_t *v, Strides v_st, int8_t *k_i8, float *k_scale,
                         float *k_mean, uint8_t *v_fp8, float *v_scale, float v_r, int BH, int H, int N,
                         hipStream_t stream, const QuantScratch &ws) {
    const int chunks = cdiv(N, kStatRows);
    const int nK = cdiv(N, kBK), nT = cdiv(N, kW);
    colstats_kv_kernel<BF16, D><<<dim3(chunks, BH, 2), 256, 0, stream>>>(k, k_st, v, v_st, H, N, chunks, ws.k_sum_part,
                                                                         ws.v_max_part);
    finalize_kv_kernel<<<dim3(BH, 2), 1024, 0, stream>>>(ws.k_sum_part, ws.v_max_part, chunks, N, D, v_r, k_mean,
                                                         v_scale, ws.v_rcp);
    quant_kv_kernel<BF16, D, QMAX><<<dim3(nK + nT, BH), 256, 0, stream>>>(k, k_st, k_mean, k_i8, k_scale, nK, v, v_st,
                                                                          ws.v_rcp, v_fp8, nT, H, N);
    return hipGetLastError();
}

// 4+8 variant, Q side: block means, and (stand-alone) the INT4 codes of Q minus its block means
template <bool BF16, int D>
hipError_t q4_impl(const uint16_t *q, Strides st, float *q_mean, int8_t *q_i4, float *q_scale, int BH, int H, int N,
                   hipStream_t stream) {
    const int nQ = cdiv(N, kBQ);
    block_mean_kernel<BF16, D><<<dim3(nQ, BH), 256, 0, stream>>>(q, st, H, N, nQ, q_mean);
    if (q_i4)
        quant_int8_kernel<BF16, D, kBQ, 2, 7><<<dim3(nQ, BH), 256, 0, stream>>>(q, st, H, q_mean, q_i4, q_scale, N, nQ);
    return hipGetLastError();
}

}  // namespace

void set_quant_kv_path(int path, long long wait_ticks) {
    g_kv_path.store(path);
    g_kv_wait_ticks.store(wait_ticks);
}

QuantScratch quant_scratch_layout(void *base, int B, int H, int N, int d) {
    const size_t BH = (size_t)B * H;
    // partial statistics: one per kStatRows tokens (three-launch path) or per resident chunk (single-read path)
    const size_t chunks = (size_t)std::max(cdiv(N, kStatRows), resident_group_size(N, d, 256));
    char *p = static_cast<char *>(base);
    QuantScratch ws;
    size_t off = 0;
    ws.k_sum_part = reinterpret_cast<double *>(p + off);
    off += align256(BH * chunks * d * sizeof(double));
    ws.v_max_part = reinterpret_cast<float *>(p + off);
    off += align256(BH * chunks * d * sizeof(float));
    ws.v_rcp = reinterpret_cast<float *>(p + off);
    off += align256(BH * d * sizeof(float));
    ws.bytes = off;
    return ws;
}

hipError_t launch_quant_q(const void *q, Strides st, int8_t *q_i8, float *q_scale, int B, int H, int N, int d,
                          bool bf16, hipStream_t stream) {
    const uint16_t *q16 = static_cast<const uint16_t *>(q);
    const int BH = B * H;
    if (d == 128)
        return bf16 ? quant_q_impl<true, 128>(q16, st, q_i8, q_scale, BH, H, N, stream)
                    : quant_q_impl<false, 128>(q16, st, q_i8, q_scale, BH, H, N, stream);
    return bf16 ? quant_q_impl<true, 64>(q16, st, q_i8, q_scale, BH, H, N, stream)
                : quant_q_impl<false, 64>(q16, st, q_i8, q_scale, BH, H, N, stream);
}

hipError_t launch_quant_k(const void *k, Strides st, int8_t *k_i8, float *k_scale, float *k_mean, int B, int H,
                          int N, int d, bool bf16, hipStream_t stream, const QuantScratch &ws, const void *q, Strides q_st,
                          int8_t *q_i8, float *q_scale) {
    const uint16_t *k16 = static_cast<const uint16_t *>(k);
    const int BH = B * H;
    const QuantQ qq{static_cast<const uint16_t *>(q), q_st, q_i8, q_scale, nullptr, BH, H, N, cdiv(N, kBQ), 0};
    if (d == 128)
        return bf16 ? quant_k_impl<true, 128>(k16, st, k_i8, k_scale, k_mean, BH, H, N, stream, ws, qq)
                    : quant_k_impl<false, 128>(k16, st, k_i8, k_scale, k_mean, BH, H, N, stream, ws, qq);
    return bf16 ? quant_k_impl<true, 64>(k16, st, k_i8, k_scale, k_mean, BH, H, N, stream, ws, qq)
                : quant_k_impl<false, 64>(k16, st, k_i8, k_scale, k_mean, BH, H, N, stream, ws, qq);
}

hipError_t launch_quant_v(const void *v, Strides st, uint8_t *v_fp8, float *v_scale, float v_r, int B, int H, int N,
                          int d, bool bf16, hipStream_t stream, const QuantScratch &ws) {
    const uint16_t *v16 = static_cast<const uint16_t *>(v);
    const int BH = B * H;
    if (d == 128) {
        return bf16 ? quant_v_impl<true, 128>(v16, st, v_fp8, v_scale, v_r, BH, H, N, stream, ws)
                    : quant_v_impl<false, 128>(v16, st, v_fp8, v_scale, v_r, BH, H, N, stream, ws);
    }
    return bf16 ? quant_v_impl<true, 64>(v16, st, v_fp8, v_scale, v_r, BH, H, N, stream, ws)
                : quant_v_impl<false, 64>(v16, st, v_fp8, v_scale, v_r, BH, H, N, stream, ws);
}

hipError_t launch_quant_kv(const void *k, Strides k_st, const void *v, Strides v_st, int8_t *k_i8, float *k_scale,
                           float *k_mean, uint8_t *v_fp8, float *v_scale, float v_r, int B, int H, int N, int d,
                           bool bf16, hipStream_t stream, const QuantScratch &ws, bool int4, const void *q, Strides q_st,
                           float *q_mean, int Hq, int Nq) {
    const uint16_t *k16 = static_cast<const uint16_t *>(k), *v16 = static_cast<const uint16_t *>(v);
    const int BH = B * H;
    const int threads = resident_threads(Quantise::kBoth, 2 * BH, N, d);
    const bool chunks = chunks_pay(Quantise::kBoth, BH, N, d);
    const QuantQ qm{static_cast<const uint16_t *>(q), q_st, nullptr, nullptr, q_mean, B * Hq, Hq, Nq, cdiv(Nq, kBQ), 0};
#define SAGE_KV(BF, DD, QM)                                                                                           \
    (chunks    ? launch_chunks<BF, DD, QM>(k16, k_st, v16, v_st, k_i8, k_scale, k_mean, v_fp8, v_scale, v_r, BH, H, N, \
                                           stream, ws, kBothTensors, qm)                                              \
     : threads ? launch_resident<BF, DD, QM>(threads, k16, k_st, v16, v_st, k_i8, k_scale, k_mean, v_fp8, v_scale, v_r, \
                                             BH, H, N, stream, ws, kBothTensors, qm)                                  \
               : quant_kv_impl<BF, DD, QM>(k16, k_st, v16, v_st, k_i8, k_scale, k_mean, v_fp8, v_scale, v_r, BH, H, N, \
                                           stream, ws))
    if (int4) {
        const hipError_t e = d == 128 ? (bf16 ? SAGE_KV(true, 128, 7) : SAGE_KV(false, 128, 7))
                                      : (bf16 ? SAGE_KV(true, 64, 7) : SAGE_KV(false, 64, 7));
        // (the three launches have no place for the block means of Q)
        return e != hipSuccess || !q || chunks || threads ? e
                                                          : launch_quant_q4(q, q_st, q_mean, nullptr, nullptr, B, Hq, Nq, d, bf16, stream);
    }
    if (d == 128) return bf16 ? SAGE_KV(true, 128, 127) : SAGE_KV(false, 128, 127);
    return bf16 ? SAGE_KV(true, 64, 127) : SAGE_KV(false, 64, 127);
#undef SAGE_KV
}

hipError_t launch_quant_q4(const void *q, Strides st, float *q_mean, int8_t *q_i4, float *q_scale, int B, int H, int N,
                           int d, bool bf16, hipStream_t stream) {
    const uint16_t *q16 = static_cast<const uint16_t *>(q);
    const int BH = B * H;
    if (d == 128)
        return bf16 ? q4_impl<true, 128>(q16, st, q_mean, q_i4, q_scale, BH, H, N, stream)
                    : q4_impl<false, 128>(q16, st, q_mean, q_i4, q_scale, BH, H, N, stream);
    return bf16 ? q4_impl<true, 64>(q16, st, q_mean, q_i4, q_scale, BH, H, N, stream)
                : q4_impl<false, 64>(q16, st, q_mean, q_i4, q_scale, BH, H, N, stream);
}

hipError_t launch_delta_s(const void *k, Strides k_st, const float *k_mean, const float *q_mean, float *dsx, int B,
                          int Hq, int Hkv, int Nq, int Nk, int d, bool causal, float sm_scale, bool bf16,
                          hipStream_t stream) {
    const uint16_t *k16 = static_cast<const uint16_t *>(k);
    const int nQ = cdiv(Nq, kBQ), nT = cdiv(Nk, kW);
    const float sm_log2e = (float)((double)sm_scale * 1.4426950408889634);
    // a workgroup keeps its keys for up to four column tiles when that leaves enough workgroups (about eight per CU)
    const int col_tiles = cdiv(nQ * (Hq / Hkv), 32);
    const long wgs = (long)nT * B * Hkv * col_tiles;
    // -- and for more where the grid's third dimension would exceed its limit of 65535 otherwise
    const int tiles = std::max((int)std::min<long>(4, std::max<long>(1, wgs / 2048)), cdiv(col_tiles, 65535));
    const dim3 grid(nT, B * Hkv, cdiv(col_tiles, tiles));
#define SAGE_DS(BF, DD) \
    delta_s_kernel<BF, DD><<<grid, 256, 0, stream>>>(k16, k_st, Hkv, k_mean, q_mean, dsx, Hq, Nq, Nk, nQ, nT, sm_log2e, \
                                                     causal ? 1 : 0, tiles)
    if (d == 128) {
        if (bf16) SAGE_DS(true, 128); else SAGE_DS(false, 128);
    } else {
        if (bf16) SAGE_DS(true, 64); else SAGE_DS(false, 64);
    }
#undef SAGE_DS
    return hipGetLastError();
}

}  // namespace sage
