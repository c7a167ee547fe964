// Decode-shaped attention on gfx950: a few query rows per head over a long key sequence (not treated in the
// paper; the arithmetic of a key step is the 8+8 path's, Sec. 2.1 / Sec. 3.1, through the same softmax_step).
//
// The kernels for many rows give a workgroup up to 128 query rows of one head and share every K^/V^ tile among its
// wavefronts through LDS.  Here a head has at most a handful of rows, so that shape leaves most wavefronts
// and MFMA columns idle and B*Hq workgroups cannot fill 256 CUs.  Instead:
//   * the R = (Hq/Hkv) * Nq <= 64 query rows of all query heads that share one K/V head are packed into the 16
//     columns of T = ceil(R/16) <= 4 MFMA tiles (exact: every row keeps its own scale, running maximum and sum), so
//     K^ and V^ of a head leave HBM once for all of them;
//   * the keys are cut into ranges of `steps_per_split` key steps and ONE WAVEFRONT owns one (batch, K/V head, range) and one or two
//     row tiles: it runs the step recurrence on its range from m = -inf, l = 0, acc = 0; the ranges are combined as partial softmax
//     sums (m = max m_s, weights 2^(m_s - m)), by the same workgroup through LDS where it holds all of them, otherwise by a second
//     launch over the (m, l, acc) per row that the wavefronts write;
//   * tiles are copied global -> LDS in halves (64 keys of K^, half the channels of V^: contiguous bytes) into two slots of the
//     wavefront's own, each refilled as soon as its operands are in registers; no barrier.  (Operands loaded straight into registers
//     cost the texture path four times as much: neighbouring lanes want neighbouring rows, so a load of 1 KB takes 64 cycles instead
//     of 16, 2048 per key step and wavefront at d = 128, which is what bounded short calls.  Four or eight slots are no faster than
//     two: 64 heads x 32768 keys, d 128, 97.4 with four, 98.4 us with two; 192 x 4096 41.4 / 36.5.)
// What bounds it: with a large cache HBM, K^ + V^ read once (2 * Nk * d bytes per K/V head); with a small one the chain launch -- Q --
// first tiles -- two steps -- combination.  Measured, us per call in a graph, operands in registers and always two launches / now:
// 16 heads x 1500 keys, d 128, one row of 4 query heads 12.5 / 8.6; 8 x 8192 13.8 / 8.4; 64 x 32768 103 / 98; 128 x 2048 15.9 / 13.1;
// 64 rows per head, 256 x 2048 64 / 32.5, 64 x 16384 95 / 71 (d 64: 56 / 38.5).
#include "sage_attn_device.h"
#include "sage_internal.h"

#include <algorithm>

namespace sage {
namespace {

// Epilogue of the prefill kernel on four channels: O = acc * (delta_V / l) (l carries the factor P_r), rounded to the output
// type.
template <int D, bool BF16>
__device__ __forceinline__ void store_quad(const float4 &acc, float l, const float *__restrict__ dv, int bhk,
                                           uint16_t *__restrict__ out, int row, int cq) {
    const float inv = 1.0f / l;
    const float4 sc = *reinterpret_cast<const float4 *>(dv + (size_t)bhk * D + 4 * cq);
    const float y0 = acc.x * (sc.x * inv), y1 = acc.y * (sc.y * inv);
    const float y2 = acc.z * (sc.z * inv), y3 = acc.w * (sc.w * inv);
    *reinterpret_cast<uint2 *>(out + (size_t)row * D + 4 * cq) = make_uint2(pack2<BF16>(y0, y1), pack2<BF16>(y2, y3));
}

// One range's (m, l, acc) of a row on top of the sums l, acc, which are relative to the row's maximum mx over all ranges.  (Each
// product is rounded before it is added.)
__device__ __forceinline__ void add_range(const float2 &ml, const float4 &a, float mx, float &l, float4 &acc) {
    const float wgt = __builtin_amdgcn_exp2f(ml.x - mx);
    l += __builtin_fmaf(wgt, ml.y, 0.0f);
    acc.x += __builtin_fmaf(wgt, a.x, 0.0f);
    acc.y += __builtin_fmaf(wgt, a.y, 0.0f);
    acc.z += __builtin_fmaf(wgt, a.z, 0.0f);
    acc.w += __builtin_fmaf(wgt, a.w, 0.0f);
}

// D: head dimension; causal: end-aligned mask (key n visible to row r iff n <= r + Nk - Nq); BF16: type of Q / O.
// NT: row tiles per wavefront (1: up to 16 rows per K/V head; 2: up to 32 -- the operands of a key step are read once for both).
// TW = ceil(T / NT) wavefronts share a range.  TOGETHER: a workgroup is the TW * S <= 8 wavefronts of a K/V head, which combine their
// ranges and write the output (the additions of merge_few_kernel: same bits).  Otherwise blockDim / 64 wavefronts,
// w = ((b*Hkv + kvh)*S + split)*TW + group.  Dynamic LDS: two half tiles per wavefront; TOGETHER the partial results take their place.
template <int D, bool BF16, int NT, bool TOGETHER>
__global__ __launch_bounds__(TOGETHER ? 512 : 256, 2) void decode_kernel(
    const uint16_t *__restrict__ Q, const int8_t *__restrict__ Kc, const uint8_t *__restrict__ Vt, const float *__restrict__ dk,
    const float *__restrict__ dv, uint16_t *__restrict__ out, float *__restrict__ part_acc, float *__restrict__ part_ml,
    int n_waves, int Hq, int Hkv, int group, int Nq, int Nk, int nT, int nKblk, int S, int T, int steps_per_split, int causal,
    float sm_scale, float log2_pr) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int KC = D / 64;      // 64-wide contraction chunks of Q.K^T
    constexpr int CT = D / 16;      // 16-channel tiles of the output
    constexpr int HALF = 64 * D;    // bytes of half a tile
    constexpr int NL = HALF / 1024; // copies of 1 KB per half tile
    constexpr int ROWS = 16 * NT, LD = D + 4;  // combination: rows and floats per row (4 more: sixteen rows fall on different banks)
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    __shared__ float row_max[TOGETHER ? 8 : 4][64];  // max |Q| of the K/V head's rows
    __shared__ __attribute__((aligned(8))) float2 ml_lds[TOGETHER ? 8 : 1][TOGETHER ? ROWS : 1];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lq = lane & 15, g = lane >> 4;
    const int TW = (T + NT - 1) / NT;
    int rt0, split, bhk;
    if constexpr (TOGETHER) {
        rt0 = wave % TW * NT, split = wave / TW, bhk = blockIdx.x;
    } else {
        const int w = (int)blockIdx.x * ((int)blockDim.x >> 6) + wave;
        if (w >= n_waves) return;  // (whole wavefronts leave; there is no barrier)
        rt0 = (w % TW) * NT, split = (w / TW) % S, bhk = w / (TW * S);
    }
    const int b = bhk / Hkv, kvh = bhk % Hkv;
    const int R = group * Nq;  // rows in use (<= 16 * T)
    const int shift = Nk - Nq;

    const uint8_t *Kh = reinterpret_cast<const uint8_t *>(Kc) + (size_t)bhk * Nk * D;
    const uint8_t *Vh = Vt + (size_t)bhk * nT * D * 128;
    const int k_bytes = Nk * D, v_bytes = nT * D * 128;
    const int j0 = split * steps_per_split, j1 = min(nT, j0 + steps_per_split);

    // ---- Q: row 16*(rt0 + qt) + lq of the K/V head = query row r of query head hq (rows past R repeat row 0 of head 0 and are
    // never stored) ----
    const auto q_row = [&](int ri) {
        const int i = ri < R ? ri : 0;
        return Q + (((size_t)b * Hq + kvh * group + i / Nq) * Nq + i % Nq) * D + g * 16;
    };
    const auto load_q = [&](uint4 (&x)[KC][2], int ri) {
        const uint16_t *p = q_row(ri);
#pragma unroll
        for (int ch = 0; ch < KC; ++ch)
#pragma unroll
            for (int h = 0; h < 2; ++h) x[ch][h] = *reinterpret_cast<const uint4 *>(p + ch * 64 + h * 8);
    };
    const auto max_q = [&](const uint4 (&x)[KC][2]) {
        float amax = 0.0f;
#pragma unroll
        for (int ch = 0; ch < KC; ++ch)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float f[8];
                unpack8<BF16>(x[ch][h], f);
#pragma unroll
                for (int i = 0; i < 8; ++i) amax = fmaxf(amax, fabsf(f[i]));
            }
        return rowgroup_max(amax);
    };
    uint4 qraw[NT][KC][2];
#pragma unroll
    for (int qt = 0; qt < NT; ++qt) load_q(qraw[qt], 16 * (rt0 + qt) + lq);

    // ---- copies global -> LDS: a half tile is 64 * D contiguous bytes of K^ or V^; 16-byte chunks swizzled for the operand reads.
    // Half tile i of the range (i & 3: the two of K^, the two of V^ of a step) goes to slot i & 1.  The descriptor ends with the
    // head's buffer: chunks beyond the last key are not fetched and read as zero.  Q is waited for first: behind the copies it would
    // arrive with the last of them (1024 wavefronts x 2 steps, d 128: 18.5 -> 17.6 us). ----
    int koff[NL], voff_[NL];
    {
#pragma unroll
        for (int p = 0; p < NL; ++p) {
            koff[p] = k_source<D>(lane) + p * 1024;
            voff_[p] = D == 128 ? koff[p] : v_source(lane) + p * 1024;
        }
    }
    const int ring = wave * (2 * HALF), ring_lds = lds_address(lds) + ring;
    const int halves = 4 * (j1 - j0);
    const auto copy_half = [&](int j, auto part_c, int i) {
        constexpr int PART = decltype(part_c)::value;
        if (i < halves) {
            const int first = half_first<D>(j, PART);
            const v4i r = PART < 2 ? lds_copy_rsrc(Kh + first, copy_left(k_bytes, first)) : lds_copy_rsrc(Vh + first, v_bytes - first);
#pragma unroll
            for (int p = 0; p < NL; ++p) lds_copy16(r, PART < 2 ? koff[p] : voff_[p], ring_lds + (PART & 1) * HALF + p * 1024);
        }
    };
    constexpr std::integral_constant<int, 0> P0{};
    constexpr std::integral_constant<int, 1> P1{};
    constexpr std::integral_constant<int, 2> P2{};
    constexpr std::integral_constant<int, 3> P3{};
#pragma unroll
    for (int qt = 0; qt < NT; ++qt)
#pragma unroll
        for (int ch = 0; ch < KC; ++ch)
#pragma unroll
            for (int h = 0; h < 2; ++h) asm volatile("" : "+v"(qraw[qt][ch][h].x), "+v"(qraw[qt][ch][h].y), "+v"(qraw[qt][ch][h].z), "+v"(qraw[qt][ch][h].w));
    copy_half(j0, P0, 0);
    copy_half(j0, P1, 1);
    // half tile i has landed when at most the one behind it is outstanding
    const auto landed = [&](int i) {
        if (i + 1 < halves) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NL) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };
    const auto was_read = []() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };

    // the maximum of every row of the K/V head (a head's rows may sit in another group's tiles), then quantisation per head over its
    // Nq rows (the stand-alone quantiser's binary32 steps on one block of Nq <= 64 rows: a head's rows are one Q quantisation
    // block), straight into the B operand layout of the INT8 MFMA
#pragma unroll
    for (int qt = 0; qt < NT; ++qt)
        if (rt0 + qt < 4) row_max[wave][16 * (rt0 + qt) + lq] = max_q(qraw[qt]);
    if (Nq > 1) {
        for (int t = 0; t < T; ++t) {
            if (t >= rt0 && t < rt0 + NT) continue;
            uint4 x[KC][2];
            load_q(x, 16 * t + lq);
            row_max[wave][16 * t + lq] = max_q(x);
        }
    }
    was_read();  // (a wavefront's own strip: no barrier)
    v4i qreg[NT][KC];
    double cq[NT];
    int lim[NT];
    bool row_ok[NT];
#pragma unroll
    for (int qt = 0; qt < NT; ++qt) {
        const int ri = 16 * (rt0 + qt) + lq, i0 = ri < R ? ri / Nq * Nq : 0;
        row_ok[qt] = ri < R;
        lim[qt] = causal ? min(Nk - 1, (row_ok[qt] ? ri % Nq : 0) + shift) : Nk - 1;  // last visible key of this lane's row
        float a = 0.0f;
        for (int r = 0; r < Nq; ++r) a = fmaxf(a, row_max[wave][i0 + r]);
        if (!row_ok[qt]) a = 0.0f;
        const float rcp = a > 0.0f ? 127.0f / a : 0.0f;
        cq[qt] = (double)(a / 127.0f) * (double)sm_scale * 1.4426950408889634;
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
    }
    const v4i cinit = {kMagic, kMagic, kMagic, kMagic};

    // last visible key of the first row in use (of the last one: Nk - 1)
    const int lim_min = causal ? min(Nk - 1, shift) : Nk - 1;

    float m[NT], l[NT], alpha[NT];
    v4f o[NT][CT];
    v4i s[NT][8];
    v8i pb[NT];
#pragma unroll
    for (int qt = 0; qt < NT; ++qt) {
        m[qt] = -INFINITY;
        l[qt] = 0.0f;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) o[qt][ct] = v4f{0.f, 0.f, 0.f, 0.f};
    }

    // operands: row 16t + lq, 16-byte chunk 4x + g, whose swizzled place is that of chunk g xor 64x bytes
    const int kof = ring + k_off<D>(lq, g), vof = ring + v_off(lq, g);
    const auto scores_of = [&](auto part_c) {  // S^T of 64 keys
        constexpr int PART = decltype(part_c)::value;
        v4i a[KC][4];
#pragma unroll
        for (int ch = 0; ch < KC; ++ch)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                a[ch][t] = *reinterpret_cast<const v4i *>(lds + ((kof ^ 64 * ch) + (PART & 1) * HALF + t * 16 * D));
        was_read();
#pragma unroll
        for (int ch = 0; ch < KC; ++ch)
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int qt = 0; qt < NT; ++qt)
                    s[qt][4 * PART + t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
                        a[ch][t], qreg[qt][ch], ch == 0 ? cinit : s[qt][4 * PART + t], 0, 0, 0);
    };
    const auto output_of = [&](auto part_c) {  // O^T += V^T P^T of half the channels
        constexpr int PART = decltype(part_c)::value;
        v8i a[CT / 2];
#pragma unroll
        for (int c = 0; c < CT / 2; ++c) {
            const uint8_t *p = lds + ((PART & 1) * HALF + c * 16 * 128);
            const v4i lo = *reinterpret_cast<const v4i *>(p + vof), hi = *reinterpret_cast<const v4i *>(p + (vof ^ 64));
            a[c] = v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        }
        was_read();
#pragma unroll
        for (int c = 0; c < CT / 2; ++c)
#pragma unroll
            for (int qt = 0; qt < NT; ++qt) {
                const int ct = (PART & 1) * (CT / 2) + c;
                o[qt][ct] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a[c], pb[qt], o[qt][ct], 0, 0, 0, 0, 0, 0);
            }
    };

    for (int j = j0; j < j1; ++j) {
        const int key0 = j * kW, i = 4 * (j - j0);
        const float dk0 = dk[(size_t)bhk * nKblk + min(2 * j, nKblk - 1)];
        const float dk1 = dk[(size_t)bhk * nKblk + min(2 * j + 1, nKblk - 1)];
        landed(i);
        scores_of(P0);
        copy_half(j, P2, i + 2);
        landed(i + 1);
        scores_of(P1);
        copy_half(j, P3, i + 3);

        // ---- softmax step: every lane has the constants of its own row (its head's delta_Q) ----
        const bool masked_step = (key0 + kW > Nk) || (causal && key0 + kW - 1 > lim_min);
        const int t_lo = min(8, max(0, (lim_min - key0 + 1) >> 4));
        const int t_hi = min(8, max(0, ((Nk - 1 - key0) >> 4) + 1));
#pragma unroll
        for (int qt = 0; qt < NT; ++qt) {
            const float c0 = (float)(cq[qt] * (double)dk0), c1 = (float)(cq[qt] * (double)dk1);
            const float kh0 = -kMagicF * c0, kh1 = -kMagicF * c1;
            const float kl0 = __builtin_fmaf(-kMagicF, c0, -kh0), kl1 = __builtin_fmaf(-kMagicF, c1, -kh1);
            if (masked_step) {
                const float l_old = l[qt];
                alpha[qt] = softmax_step<true>(s[qt], c0, c1, kh0, kh1, kl0, kl1, log2_pr, m[qt], l[qt], pb[qt], key0 + 4 * g,
                                               lim[qt], t_lo, t_hi);
                // a row that has seen no key yet and sees none in this step keeps its empty state (the step's
                // arithmetic on (-inf) - (-inf) is undefined; its P^ is zero either way)
                if (lim[qt] < key0 && m[qt] == -INFINITY) {
                    alpha[qt] = 1.0f;
                    l[qt] = l_old;
                }
            } else {
                alpha[qt] = softmax_step<false>(s[qt], c0, c1, kh0, kh1, kl0, kl1, log2_pr, m[qt], l[qt], pb[qt], 0, 0, 8, 8);
            }
            if (__builtin_amdgcn_ballot_w64(alpha[qt] != 1.0f) != 0) {
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) o[qt][ct] *= alpha[qt];
            }
        }
        landed(i + 2);
        output_of(P2);
        copy_half(j + 1, P0, i + 4);
        landed(i + 3);
        output_of(P3);
        copy_half(j + 1, P1, i + 5);
    }

    if constexpr (TOGETHER) {
        // ---- the ranges' (m, l, acc) meet in LDS, in the place of the tiles ----
        float *acc_lds = reinterpret_cast<float *>(lds);
        __syncthreads();
#pragma unroll
        for (int qt = 0; qt < NT; ++qt) {
            const float lsum = rowgroup_sum(l[qt]);
            if (g == 0) ml_lds[wave][16 * qt + lq] = make_float2(m[qt], lsum);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
                *reinterpret_cast<float4 *>(acc_lds + (wave * ROWS + 16 * qt + lq) * LD + 16 * ct + 4 * g) =
                    make_float4(o[qt][ct][0], o[qt][ct][1], o[qt][ct][2], o[qt][ct][3]);
        }
        __syncthreads();
        for (int e = threadIdx.x; e < R * (D / 4); e += blockDim.x) {
            const int ri = e / (D / 4), quad = e % (D / 4), w0 = ri / ROWS, row = ri % ROWS;  // the row's ranges: wavefronts w0 + TW * p
            float mx = ml_lds[w0][row].x;
            for (int p = 1; p < S; ++p) mx = fmaxf(mx, ml_lds[w0 + TW * p][row].x);
            float lt = 0.0f;
            float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
            for (int p = 0; p < S; ++p) {
                const int w = w0 + TW * p;
                add_range(ml_lds[w][row], *reinterpret_cast<const float4 *>(acc_lds + (w * ROWS + row) * LD + 4 * quad), mx, lt, acc);
            }
            store_quad<D, BF16>(acc, lt, dv, bhk, out, (b * Hq + kvh * group + ri / Nq) * Nq + ri % Nq, quad);
        }
        return;
    }
    // ---- this range's (m, l, acc) of every row in use; l is the sum over the row's four lanes.  Partial rows are
    // indexed (((b*Hkv + kvh)*S + split)*T + row tile)*16 + lq ----
#pragma unroll
    for (int qt = 0; qt < NT; ++qt) {
        const float lsum = rowgroup_sum(l[qt]);
        if (row_ok[qt]) {
            const size_t prow = (((size_t)bhk * S + split) * T + rt0 + qt) * 16 + lq;
            if (g == 0) *reinterpret_cast<float2 *>(part_ml + prow * 2) = make_float2(m[qt], lsum);
            float *pa = part_acc + prow * D;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
                *reinterpret_cast<float4 *>(pa + 16 * ct + 4 * g) =
                    make_float4(o[qt][ct][0], o[qt][ct][1], o[qt][ct][2], o[qt][ct][3]);
        }
    }
#endif  // __HIP_DEVICE_COMPILE__
}

// Where range s of output row `row` = (b*Hq + hq)*Nq + r lies: partial row p0 + s * ps.  T > 0: the partial results come from
// decode_kernel (T row tiles); T = 0: from prefill_kernel<..., SPLIT> (query tiles of 128 rows).
__device__ __forceinline__ void partial_rows(int row, int Hq, int Hkv, int group, int Nq, int S, int T, int &bhk, size_t &p0,
                                             size_t &ps) {
    const int r = row % Nq, bh = row / Nq, hq = bh % Hq, b = bh / Hq;
    bhk = b * Hkv + hq / group;
    if (T > 0) {
        // decode_kernel: row ri of the K/V head sits in row tile ri / 16, column ri % 16 of wavefront
        // ((b*Hkv + kvh)*S + s)*T + tile
        const int ri = (hq % group) * Nq + r;
        p0 = ((size_t)bhk * S * T + ri / 16) * 16 + ri % 16;
        ps = (size_t)T * 16;
    } else {
        // prefill_kernel<..., SPLIT>: row r of the head sits in query tile r / 128, row r % 128 of workgroup
        // ((b*Hq + hq)*tiles + tile)*S + s
        const int tiles = (Nq + kBQ - 1) / kBQ;
        p0 = (((size_t)bh * tiles + r / kBQ) * S) * kBQ + r % kBQ;
        ps = kBQ;
    }
}

// Combine the S <= MAXS ranges of a row: m = max_s m_s, l = sum_s 2^(m_s - m) l_s, acc likewise.  Bound by memory (S * (D + 2)
// floats read per row) or, with few rows, by its latency: a thread owns four channels of a row and fetches all ranges at
// once; no LDS, no barrier, 256 / (D/4) rows per workgroup.  The additions are those of merge_kernel, whose range lanes hold one
// range each at S <= 8: same bits.
template <int D, bool BF16, int MAXS>
__global__ __launch_bounds__(256) void merge_few_kernel(const float *__restrict__ part_acc, const float *__restrict__ part_ml,
                                                        const float *__restrict__ dv, uint16_t *__restrict__ out, int Hq,
                                                        int Hkv, int group, int Nq, int S, int T, int n_rows) {
    constexpr int Q4 = D / 4;  // channel quads
    const int row = (int)blockIdx.x * (256 / Q4) + (int)threadIdx.x / Q4, cq = threadIdx.x % Q4;
    if (row >= n_rows) return;
    int bhk;
    size_t p0, ps;
    partial_rows(row, Hq, Hkv, group, Nq, S, T, bhk, p0, ps);
    float2 ml[MAXS];
    float4 a[MAXS];
#pragma unroll
    for (int s = 0; s < MAXS; ++s) {
        const size_t p = p0 + min(s, S - 1) * ps;
        ml[s] = *reinterpret_cast<const float2 *>(part_ml + p * 2);
        a[s] = *reinterpret_cast<const float4 *>(part_acc + p * D + 4 * cq);
    }
    float mx = ml[0].x;
#pragma unroll
    for (int s = 1; s < MAXS; ++s) mx = fmaxf(mx, ml[s].x);
    float l = 0.0f;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int s = 0; s < MAXS; ++s) {
        if (s < S) add_range(ml[s], a[s], mx, l, acc);
    }
    store_quad<D, BF16>(acc, l, dv, bhk, out, row, cq);
}

// The same for any number of ranges.  One workgroup of 256 threads per row (grid B*Hq*Nq): thread t owns channels
// 4*(t % (D/4)) .. +3 and the ranges t / (D/4), + 256/(D/4), ...; the shares are added in a fixed order through LDS, so the
// result does not depend on timing.  Bound by latency with few rows: one round trip to memory and one barrier up to 32 ranges (d = 64:
// 64); with the maximum found through LDS first, nine barriers and a second round trip, 1.0 us more (8 heads x 4096 keys, 16 ranges).
// With hundreds of ranges a CU's share of memory is what counts, S * (D + 2) floats on one CU, and every extra read of the maxima shows
// (one row of 512 ranges, whole call, each wavefront reading all of them / sharing them: d 64 14.4 / 12.6 us, d 128 19.8 / 18.1).
template <int D, bool BF16>
__global__ __launch_bounds__(256) void merge_kernel(const float *__restrict__ part_acc, const float *__restrict__ part_ml,
                                                    const float *__restrict__ dv, uint16_t *__restrict__ out, int Hq,
                                                    int Hkv, int group, int Nq, int S, int T) {
    constexpr int Q4 = D / 4;      // channel quads
    constexpr int SL = 256 / Q4;   // range lanes
    __shared__ float4 acc_s[SL][Q4];
    __shared__ float l_s[SL], m_s[4];
    const int row = blockIdx.x;  // (b*Hq + hq)*Nq + r
    int bhk;
    size_t p0, ps;
    partial_rows(row, Hq, Hkv, group, Nq, S, T, bhk, p0, ps);
    const int tid = threadIdx.x, cq = tid % Q4, sl = tid / Q4;
    // this thread's first FIRST ranges and, for the row's maximum (up to 64 ranges every wavefront finds it itself), one m per lane: one round trip to
    // memory up to FIRST * SL ranges
    constexpr int FIRST = 4;
    float2 ml[FIRST];
    float4 a[FIRST];
#pragma unroll
    for (int k = 0; k < FIRST; ++k) {
        const size_t p = p0 + min(sl + k * SL, S - 1) * ps;
        ml[k] = *reinterpret_cast<const float2 *>(part_ml + p * 2);
        a[k] = *reinterpret_cast<const float4 *>(part_acc + p * D + 4 * cq);
    }
    // (a maximum's neighbours are 128 bytes apart, so that 64 of them cost the texture path 64 cycles: beyond 64 the workgroup shares them)
    float mx;
    if (S <= 64) {
        mx = wave_max(part_ml[(p0 + min(tid & 63, S - 1) * ps) * 2]);
    } else {
        mx = -INFINITY;
        for (int s = tid; s < S; s += 256) mx = fmaxf(mx, part_ml[(p0 + s * ps) * 2]);
        mx = wave_max(mx);
        if ((tid & 63) == 0) m_s[tid >> 6] = mx;
        __syncthreads();
        mx = fmaxf(fmaxf(m_s[0], m_s[1]), fmaxf(m_s[2], m_s[3]));
    }
    float l = 0.0f;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    // a range in which the row saw no key has m = -inf, l = 0, acc = 0: its weight 2^(-inf) = 0 is exact
    const auto add = [&](const float2 &mls, const float4 &as) {
        const float wgt = __builtin_amdgcn_exp2f(mls.x - mx);
        l = __builtin_fmaf(wgt, mls.y, l);
        acc.x = __builtin_fmaf(wgt, as.x, acc.x);
        acc.y = __builtin_fmaf(wgt, as.y, acc.y);
        acc.z = __builtin_fmaf(wgt, as.z, acc.z);
        acc.w = __builtin_fmaf(wgt, as.w, acc.w);
    };
#pragma unroll
    for (int k = 0; k < FIRST; ++k)
        if (sl + k * SL < S) add(ml[k], a[k]);
#pragma unroll 4
    for (int s = sl + FIRST * SL; s < S; s += SL)
        add(*reinterpret_cast<const float2 *>(part_ml + (p0 + s * ps) * 2),
            *reinterpret_cast<const float4 *>(part_acc + (p0 + s * ps) * D + 4 * cq));
    acc_s[sl][cq] = acc;
    if (cq == 0) l_s[sl] = l;
    __syncthreads();
    if (sl == 0) {
        for (int k = 1; k < SL; ++k) {
            const float4 a = acc_s[k][cq];
            acc.x += a.x, acc.y += a.y, acc.z += a.z, acc.w += a.w;
            l += l_s[k];
        }
        store_quad<D, BF16>(acc, l, dv, bhk, out, row, cq);
    }
}

// (part_acc, part_ml) of S ranges -> out.  Up to eight ranges a thread takes all of them.  Measured (S = 4, 16384 rows, d 128):
// 7.1 us against 21.1 us with a workgroup per row, half of whose range lanes then have nothing to do.
template <int D, bool BF16>
hipError_t launch_merge(const DecodeScratch &ws, const float *v_scale, uint16_t *out, int B, int Hq, int Hkv, int Nq, int T,
                        hipStream_t stream) {
    const int S = ws.n_splits, n_rows = B * Hq * Nq, group = Hq / Hkv;
    const int few = cdiv(n_rows, 256 / (D / 4));
    if (S <= 4)
        merge_few_kernel<D, BF16, 4>
            <<<few, 256, 0, stream>>>(ws.part_acc, ws.part_ml, v_scale, out, Hq, Hkv, group, Nq, S, T, n_rows);
    else if (S <= 8)
        merge_few_kernel<D, BF16, 8>
            <<<few, 256, 0, stream>>>(ws.part_acc, ws.part_ml, v_scale, out, Hq, Hkv, group, Nq, S, T, n_rows);
    else
        merge_kernel<D, BF16><<<n_rows, 256, 0, stream>>>(ws.part_acc, ws.part_ml, v_scale, out, Hq, Hkv, group, Nq, S, T);
    return hipGetLastError();
}

hipError_t launch_merge(const DecodeScratch &ws, const float *v_scale, void *out, int B, int Hq, int Hkv, int Nq, int d, bool bf16,
                        int T, hipStream_t stream) {
    uint16_t *o16 = static_cast<uint16_t *>(out);
    if (d == 128)
        return bf16 ? launch_merge<128, true>(ws, v_scale, o16, B, Hq, Hkv, Nq, T, stream)
                    : launch_merge<128, false>(ws, v_scale, o16, B, Hq, Hkv, Nq, T, stream);
    return bf16 ? launch_merge<64, true>(ws, v_scale, o16, B, Hq, Hkv, Nq, T, stream)
                : launch_merge<64, false>(ws, v_scale, o16, B, Hq, Hkv, Nq, T, stream);
}

}  // namespace

int decode_auto_steps_per_split(int B, int Hkv, int Nk) {
    // about four wavefronts per CU over the whole launch (measured: 1024 wavefronts stream a 0.3-0.5 GB cache 4-8 %
    // faster than 2048 -- fewer partial results to write and combine -- and much faster than 512), at least two key
    // steps per wavefront
    const int nT = cdiv(Nk, kW);
    const long heads = (long)B * Hkv;
    const int want = (int)std::max<long>(1, std::min<long>(nT, (1024 + heads - 1) / heads));
    return std::max(std::min(nT, 2), cdiv(nT, want));
}

DecodeScratch decode_scratch_layout(void *base, int B, int Hkv, int Nk, int d, int steps_per_split, int row_tiles) {
    const int S = cdiv(cdiv(Nk, kW), steps_per_split);
    const size_t waves = (size_t)B * Hkv * S * row_tiles;
    char *p = static_cast<char *>(base);
    DecodeScratch ws;
    ws.n_splits = S;
    ws.part_acc = reinterpret_cast<float *>(p);
    size_t off = (waves * 16 * d * sizeof(float) + 255) & ~(size_t)255;
    ws.part_ml = reinterpret_cast<float *>(p + off);
    off += (waves * 16 * 2 * sizeof(float) + 255) & ~(size_t)255;
    ws.bytes = off;
    return ws;
}

// Whether the ranges of a K/V head are one workgroup's.  Up to eight wavefronts fit a CU's registers and LDS, and the second launch is
// saved, 2 to 3 us; but up to 128 heads leave half of the CUs or more idle, and a CU draws 55 to 90 GB/s.  A program that steps through
// its layers finds the cache of each one cold, so the lines are those of calls that go round caches of 900 MB together (us, one
// workgroup / one wavefront per workgroup and a second launch; behind the semicolon the same cache again and again):
//   * one row tile, bytes of K^ and V^ per head: d 128, 8 heads x 512 keys (128 KB) 6.3 / 8.4, x 1000 8.1 / 9.5, x 1500 (375 KB) 10.9 /
//     9.7; 8.2 / 8.6, x 2048 (512 KB) 12.7 / 9.4; 8.6 / 8.2; 96 x 2048 15.1 / 14.5; 11.6 / 13.4, 128 x 3000 21.4 / 22.6, 128 x 4096
//     30.3 / 28.7; 22.4 / 25.1; d 64, 128 x 4096 (512 KB) 16.1 / 17.7, x 8192 30.4 / 29.0;
//   * with at most 32 KB of copies in flight a CU is not the limit: 2 ranges at d 128, 64 x 2048 17.6 / 19.8, 4 at d 64, 8 x 16384 47 / 48;
//     with 64 KB it is: 4 ranges at d 128, 64 x 8192 45 / 35;
//   * 129 .. 256 heads leave fewer CUs idle than a fifth wavefront on some of them costs: 136 x 1000 10.4 / 13.2, x 32768 206 / 217, 192 x 4096
//     38 / 44, 256 x 8192 99.6 / 95.7, x 32768 363 / 370; beyond, the last round counts: 257 x 2048 33 / 31, 300 x 8192 132 / 117 (d 64
//     71 / 59), 340 x 4096 70.2 / 68.6, 360 x 4096 72.5 / 75.5, 520 x 4096 111 / 107, 1000 x 4096 177 / 185;
//   * the work of two row tiles adds up on a CU (d 128, 32 rows, 8 x 256 keys in one range 14.4 / 12.6, 8 x 1000 in four 13.3 / 13.5, 64 x 8192
//     in four 52.8 / 51.3, 8 x 2048 in eight 18.5 / 13.8), that of two wavefronts per range more so (64 rows, 16 x 700 18.1 / 14.4).
bool decode_together(int groups, int S, int nt, int TW, int Nk, int d) {
    if (TW * S > 8) return false;
    const long kb = 2L * Nk * d / 1024;
    if (groups > kCUs) return S < 4 || 2L * cdiv(groups, kCUs) * kCUs <= 3L * groups || kb < 512 * nt;
    if (groups > kCUs / 2) return true;
    if (nt == 1) return S * d <= 256 || kb <= std::max(384, 6 * groups);
    return TW == 1 && (S > 1 || d == 64) && S <= 4;
}

// Wavefronts of a workgroup where there is a second launch.  One: they start and end independently (64 heads x 32768 keys, d 128: 98 us
// against 104 with four).  Four where two of them read the same tiles and there are many (64 rows, 64 x 16384: 71 / 95; 256
// wavefronts, 16 x 2048: 16.1 / 14.4), and at d = 64 with a chip full of the shortest ranges (64 x 4096, 8 rows: 10.4 / 11.0).
int decode_waves(int n_waves, int TW, int steps_per_split, int d) {
    if (TW == 2) return n_waves > 2 * kCUs ? 4 : 1;
    return d == 64 && steps_per_split <= 2 && n_waves >= 4 * kCUs ? 4 : 1;
}

hipError_t launch_decode(const void *q, const int8_t *k_i8, const uint8_t *v_fp8, const float *k_scale,
                         const float *v_scale, void *out, int B, int Hq, int Hkv, int Nq, int Nk, int d, bool causal,
                         float sm_scale, float p_r, int steps_per_split, bool bf16, hipStream_t stream,
                         const DecodeScratch &ws) {
    const int group = Hq / Hkv;
    const int nT = cdiv(Nk, kW), nK = cdiv(Nk, kBK);
    const int S = ws.n_splits;
    const int T = cdiv(group * Nq, 16);
    const int nt = T >= 2 ? 2 : 1;  // row tiles per wavefront (measured: 0.16 against 0.25 ms at 64 rows per K/V head, B 8, 32768 keys)
    const int n_waves = B * Hkv * S * cdiv(T, nt);
    const float log2_pr = (float)log2((double)p_r);
    const uint16_t *q16 = static_cast<const uint16_t *>(q);
    const int groups = B * Hkv, TW = cdiv(T, nt);
    const bool together = decode_together(groups, S, nt, TW, Nk, d);
    const int waves = together ? TW * S : decode_waves(n_waves, TW, steps_per_split, d);  // of a workgroup
    const int grid = together ? groups : cdiv(n_waves, waves);
    uint16_t *o16 = static_cast<uint16_t *>(out);
    const int tiles = waves * 128 * d;
    const int lds_bytes = together ? std::max(tiles, waves * 16 * nt * (d + 4) * (int)sizeof(float)) : tiles;
#define SAGE_DEC_N(DD, BF, NT, TG)                                                                                             \
    decode_kernel<DD, BF, NT, TG><<<grid, 64 * waves, lds_bytes, stream>>>(                                                    \
        q16, k_i8, v_fp8, k_scale, v_scale, o16, ws.part_acc, ws.part_ml, n_waves, Hq, Hkv, group, Nq, Nk, nT, nK, S, T,         \
        steps_per_split, causal ? 1 : 0, sm_scale, log2_pr)
#define SAGE_DEC_T(DD, BF, NT)                                                                    \
    do {                                                                                           \
        if (together) SAGE_DEC_N(DD, BF, NT, true); else SAGE_DEC_N(DD, BF, NT, false);             \
    } while (0)
#define SAGE_DEC(DD, BF)                                             \
    do {                                                             \
        if (nt == 1) SAGE_DEC_T(DD, BF, 1); else SAGE_DEC_T(DD, BF, 2); \
    } while (0)
    if (d == 128) {
        if (bf16) SAGE_DEC(128, true); else SAGE_DEC(128, false);
    } else {
        if (bf16) SAGE_DEC(64, true); else SAGE_DEC(64, false);
    }
#undef SAGE_DEC
#undef SAGE_DEC_T
#undef SAGE_DEC_N
    const hipError_t e = hipGetLastError();
    return e != hipSuccess || together ? e : launch_merge(ws, v_scale, out, B, Hq, Hkv, Nq, d, bf16, T, stream);
}


// Few workgroups, many keys (more than 64 query rows per K/V head): the prefill kernel with the key steps cut into
// ranges on separate workgroups, then the same combination launch.
hipError_t launch_attn_ranges(const void *q, const int8_t *k_i8, const uint8_t *v_fp8, const float *k_scale,
                              const float *v_scale, void *out, int B, int Hq, int Hkv, int Nq, int Nk, int d, bool causal,
                              float sm_scale, float p_r, int steps_per_split, bool bf16, hipStream_t stream,
                              const DecodeScratch &ws) {
    const int S = ws.n_splits;
    if (S == 1) {
        // one range is the uncut kernel, which writes the output itself
        const Strides st = contiguous_bhnd(Hq, Nq, d);
        return launch_attn(q, true, st, k_i8, v_fp8, nullptr, k_scale, v_scale, out, st, B, Hq, Hkv, Nq, Nk, d, causal,
                           sm_scale, p_r, bf16, stream);
    }
    const Strides st = contiguous_bhnd(Hq, Nq, d);
    hipError_t e = launch_attn(q, true, st, k_i8, v_fp8, nullptr, k_scale, v_scale, nullptr, st, B, Hq, Hkv, Nq, Nk, d, causal,
                               sm_scale, p_r, bf16, stream, nullptr, nullptr, S, steps_per_split, ws.part_acc, ws.part_ml);
    if (e != hipSuccess) return e;
    return launch_merge(ws, v_scale, out, B, Hq, Hkv, Nq, d, bf16, 0, stream);
}

int ranges_auto_steps_per_split(int B, int Hq, int Nq, int Nk) {
    // Measured (B*Hq*tiles = 16 .. 512 workgroups before the cut, 4096 .. 65536 keys): the cut pays up to 128
    // workgroups, and best with about 512 workgroups after it (one for each of the chip's slots); from 256 workgroups
    // on the uncut kernel is faster (every range writes 128 x (d + 2) floats per workgroup that the combination
    // reads back).  At least four key steps per range.
    const int nT = cdiv(Nk, kW);
    const long items = (long)B * Hq * cdiv(Nq, kBQ);
    if (items > 128) return nT;
    const int want = (int)std::max<long>(1, std::min<long>(nT, 512 / items));
    return std::max(std::min(nT, 4), cdiv(nT, want));
}

DecodeScratch ranges_scratch_layout(void *base, int B, int Hq, int Nq, int Nk, int d, int steps_per_split) {
    const int S = cdiv(cdiv(Nk, kW), steps_per_split);
    const size_t rows = (size_t)B * Hq * cdiv(Nq, kBQ) * S * kBQ;
    char *p = static_cast<char *>(base);
    DecodeScratch ws;
    ws.n_splits = S;
    ws.part_acc = reinterpret_cast<float *>(p);
    size_t off = (rows * d * sizeof(float) + 255) & ~(size_t)255;
    ws.part_ml = reinterpret_cast<float *>(p + off);
    off += (rows * 2 * sizeof(float) + 255) & ~(size_t)255;
    ws.bytes = off;
    return ws;
}

}  // namespace sage
