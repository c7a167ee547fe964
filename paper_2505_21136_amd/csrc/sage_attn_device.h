// Device-side building blocks shared by the attention kernels of libsage (gfx950): vector types, the lane
// exchanges over the four 16-lane rows of a wavefront, 16-bit conversions, and the online-softmax step of the
// 8+8 path (paper Sec. 2.1 for the online softmax and the scales, Sec. 3.1 for the bounded FP8 range of P~).
// Included by the attention translation units and, for the conversions and codes, by the quantiser; every function is inlined.
#pragma once
#include <hip/hip_runtime.h>
#include <limits.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "sage_tile_copy.h"

namespace sage {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void;

__device__ __forceinline__ int imax3(int a, int b, int c) { return max(max(a, b), c); }

#if defined(__HIP_DEVICE_COMPILE__)
// A global -> LDS copy: 64 lanes x 16 (or 4) bytes from the buffer at per-lane offset `voff` to LDS at `dst` + 16 (4) * lane.
// Written as asm because of the compiler's wait insertion: it cannot tell the two buffers of a tile apart and makes every LDS
// read behind such a copy wait for it.  The kernel waits itself (vmcnt(0) in front of the barrier that ends a step).
__device__ __forceinline__ v4i lds_copy_rsrc(const void *base, int bytes) {
    const uint64_t a = (uint64_t)base;
    return v4i{(int)(uint32_t)a, (int)((uint32_t)(a >> 32) & 0xffffu), bytes, 0x00020000};
}
__device__ __forceinline__ int lds_address(const void *p) {
    return (int)(uint32_t)(uint64_t)(const __attribute__((address_space(3))) void *)p;
}
__device__ __forceinline__ void lds_copy16(v4i rsrc, int voff, int dst) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds" ::"v"(voff), "s"(rsrc), "s"(dst) : "m0");
}
__device__ __forceinline__ void lds_copy4(v4i rsrc, int voff, int dst) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dword %0, %1, 0 offen lds" ::"v"(voff), "s"(rsrc), "s"(dst) : "m0");
}
#endif  // __HIP_DEVICE_COMPILE__

// Cross-lane exchange over the four 16-lane rows of a wavefront (lanes l, l^16, l^32, l^48).
// v_permlane16_swap exchanges the odd rows of its first register with the even rows of its second,
// v_permlane32_swap the upper half of the first with the lower half of the second: starting from
// two copies of x, the pair (a, b) then holds both partners' values in every lane.  The two copies
// must live in distinct registers.
// (Written as asm so that the two registers stay distinct; the s_nop around each swap cover the
// wait states between vector ALU writes and a lane-permuting read/write of the same registers.)
__device__ __forceinline__ void swap16(float &a, float &b) {
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ void swap32(uint32_t &a, uint32_t &b) {
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ void swap32(float &a, float &b) {
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
}
// max of two numbers that are known not to be NaN: one v_max_f32 (fmaxf would first canonicalise
// both operands, which come out of an asm statement, with two more instructions)
__device__ __forceinline__ float max_no_nan(float a, float b) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float rowgroup_max(float x) {
    float a = x, b = x;
    swap16(a, b);
    a = b = max_no_nan(a, b);
    swap32(a, b);
    return fmaxf(a, b);
}
// x of another lane of the same row of 16 (DPP control word CTRL); the vector ALU reads it directly, LDS is not involved
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
// maximum over all 64 lanes (no NaN)
__device__ __forceinline__ float wave_max(float x) {
    x = fmaxf(x, dpp<0xb1>(x));   // quad_perm [1,0,3,2]
    x = fmaxf(x, dpp<0x4e>(x));   // quad_perm [2,3,0,1]
    x = fmaxf(x, dpp<0x141>(x));  // row_half_mirror
    x = fmaxf(x, dpp<0x140>(x));  // row_mirror
    return rowgroup_max(x);
}
__device__ __forceinline__ float rowgroup_sum(float x) {
    float a = x, b = x;
    swap16(a, b);
    a = b = a + b;
    swap32(a, b);
    return a + b;
}

// max (no NaN) / sum of a value over the two halves of the wavefront (lanes l and l ^ 32)
__device__ __forceinline__ float halves_max(float x) {
    float a = x, b = x;
    swap32(a, b);
    return max_no_nan(a, b);
}
__device__ __forceinline__ float halves_sum(float x) {
    float a = x, b = x;
    swap32(a, b);
    return a + b;
}

// 16-bit input value (bits in the low half of u) -> binary32, exact
template <bool BF16>
__device__ __forceinline__ float to_f32(uint32_t u) {
    if constexpr (BF16) return __builtin_bit_cast(float, u << 16);
    return (float)__builtin_bit_cast(_Float16, (uint16_t)u);
}

// eight packed 16-bit values -> binary32
template <bool BF16>
__device__ __forceinline__ void unpack8(const uint4 &u, float (&f)[8]) {
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[2 * i] = to_f32<BF16>(w[i] & 0xffffu);
        f[2 * i + 1] = to_f32<BF16>(w[i] >> 16);
    }
}

template <bool BF16>
__device__ __forceinline__ uint32_t pack2(float a, float b) {
    if constexpr (BF16) {
        // one v_cvt_pk_bf16_f32 (round to nearest even)
        typedef float f32x2 __attribute__((ext_vector_type(2)));
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        const f32x2 v = {a, b};
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
    } else {
        const uint32_t ua = __builtin_bit_cast(uint16_t, (_Float16)a);
        const uint32_t ub = __builtin_bit_cast(uint16_t, (_Float16)b);
        return ua | (ub << 16);
    }
}

// The INT8 MFMA accumulates onto kMagic = 0x4B400000 instead of 0: the INT32 result MAGIC + S,
// read as binary32, IS the number K + S with K = 1.5*2^23 (exact for |S| < 2^22; |S| <= 127*127*128
// here), so no int->float conversion instruction is needed.  -K*c is split exactly into two
// binary32 numbers kh + kl; then fma(bits, c, kh) = fl(c*S - kl) and adding (kl + offset) restores c*S.
constexpr int kMagic = 0x4B400000;
constexpr float kMagicF = 12582912.0f;

// Eight INT8 codes rne(fl(x * rcp)), one per byte: adding 1.5*2^23 to the (separately rounded) product rounds it to the
// nearest integer, ties to even, and leaves the code's two's-complement byte in the low byte of the sum's bit pattern;
// three byte permutes pack four codes.
__device__ __forceinline__ uint2 int8_codes(const float (&x)[8], float rcp) {
    uint32_t w[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        uint32_t b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float y = x[4 * e + i] * rcp;
            asm volatile("" : "+v"(y));  // keeps the product a rounded binary32 value (no FMA)
            b[i] = __builtin_bit_cast(uint32_t, y + kMagicF);
        }
        const uint32_t lo2 = __builtin_amdgcn_perm(b[1], b[0], 0x0c0c0400u);
        const uint32_t hi2 = __builtin_amdgcn_perm(b[3], b[2], 0x0c0c0400u);
        w[e] = __builtin_amdgcn_perm(hi2, lo2, 0x05040100u);
    }
    return make_uint2(w[0], w[1]);
}

// Workgroup id -> (batch and query head, query tile) of a one-dimensional grid of n_items = heads * n_qt workgroups.
// The hardware deals consecutive workgroup ids round-robin to the 8 XCDs, each with an L2 of its own: workgroup id is
// the `slot`-th of XCD `xcd`.  Co-resident workgroups of an XCD should stream through the same K^/V^ tiles (its L2 then
// serves every fetch after the first), and a causal launch must also end on its short tiles.
template <bool CAUSAL>
__device__ __forceinline__ void map_workgroup(int id, int n_items, int n_qt, int &bh, int &qtile) {
    const int n_bh = n_items / n_qt, xcd = id % 8, slot = id / 8;
    if (!CAUSAL && n_qt >= 128) {
        // a head has 16 or more tiles per XCD anyway: ids in order (query tile fastest), every XCD works
        // on the same one or two heads, and a tile missed by one L2 is likely still in the last-level cache
        bh = id / n_qt;
        qtile = id % n_qt;
    } else if (!CAUSAL) {
        // shorter sequences: head-major items cut into 8 contiguous ranges, one per XCD, walked in order
        // (otherwise an XCD would hold only n_qt/8 tiles of each of many heads at a time)
        const int pos = xcd * (n_items / 8) + min(xcd, n_items % 8) + slot;
        bh = pos / n_qt;
        qtile = pos % n_qt;
    } else if (n_bh % 8 == 0) {
        // an XCD owns n_bh/8 adjacent heads and takes them in windows of G heads -- enough tiles to fill
        // its 64 workgroup slots twice --, inside a window the longest tiles of all heads first
        const int hp = n_bh / 8;
        const int G = max(1, min(hp, (127 + n_qt) / n_qt));
        const int w = slot / (G * n_qt), r = slot - w * G * n_qt;
        const int hw = min(G, hp - w * G);  // heads in this window (the last one may be short)
        bh = xcd * hp + w * G + r % hw;
        qtile = n_qt - 1 - r / hw;
    } else {
        // any other head count: longest tiles first over all heads
        bh = id % n_bh;
        qtile = n_qt - 1 - id / n_bh;
    }
}

// One online-softmax step for one 16-query tile: biased scores s[t] (t<8: 16-key tiles of the
// 128-key step) -> P^ packed as the FP8 MFMA operand; updates m, l; returns alpha.
// c0/c1: de-quantisation constants of the two 64-key K blocks of the step; kh/kl: the exact split of -K*c.
// MASKED (causal diagonal or ragged tail): keys beyond `lim` are excluded.  The wavefront-uniform
// bounds t_lo <= t_hi say which 16-key tiles need no mask (t < t_lo), an element-wise mask
// (t_lo <= t < t_hi) or are invisible to every lane (t >= t_hi: no arithmetic at all, P^ = 0).
template <bool MASKED>
__device__ __forceinline__ float softmax_step(v4i (&s)[8], float c0, float c1, float kh0, float kh1, float kl0, float kl1, float log2_pr,
                                              float &m, float &l, v8i &pb, int key_base, int lim, int t_lo, int t_hi) {
    // step maximum on the integers of each 64-key K block (its scale is positive; the bias keeps order)
    int im0 = INT_MIN, im1 = INT_MIN;
    if constexpr (MASKED) {
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            if (t >= t_hi) continue;
            if (t >= t_lo) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (key_base + 16 * t + i > lim) s[t][i] = INT_MIN;
            }
            int &im = t < 4 ? im0 : im1;
            im = imax3(im, s[t][0], s[t][1]);
            im = imax3(im, s[t][2], s[t][3]);
        }
    } else {
        im0 = imax3(s[0][0], s[0][1], s[0][2]);
        im1 = imax3(s[4][0], s[4][1], s[4][2]);
        im0 = max(im0, s[0][3]);
        im1 = max(im1, s[4][3]);
#pragma unroll
        for (int t = 1; t < 4; ++t) {
            im0 = imax3(im0, s[t][0], s[t][1]);
            im0 = imax3(im0, s[t][2], s[t][3]);
            im1 = imax3(im1, s[t + 4][0], s[t + 4][1]);
            im1 = imax3(im1, s[t + 4][2], s[t + 4][3]);
        }
    }
    float mc0 = __builtin_fmaf(__builtin_bit_cast(float, im0), c0, kh0) + kl0;
    float mc1 = __builtin_fmaf(__builtin_bit_cast(float, im1), c1, kh1) + kl1;
    if constexpr (MASKED) {
        mc0 = im0 == INT_MIN ? -INFINITY : mc0;
        mc1 = im1 == INT_MIN ? -INFINITY : mc1;
    }
    const float mc = rowgroup_max(fmaxf(mc0, mc1));
    const float m_new = fmaxf(m, mc);
    const float alpha = __builtin_amdgcn_exp2f(m - m_new);
    const float mo = log2_pr - m_new;  // P~ * P_r = 2^(x - m' + log2 P_r)
    const float mo0 = mo + kl0, mo1 = mo + kl1;
    float lsum0 = -0.0f, lsum1 = -0.0f;  // x + (-0) is x for every x: the first addition folds away
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        if constexpr (MASKED) {
            if (t >= t_hi) {
                pb[t] = 0;
                continue;
            }
        }
        const float cb = t < 4 ? c0 : c1, khb = t < 4 ? kh0 : kh1, mob = t < 4 ? mo0 : mo1;
        float p[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int sbits = s[t][i];  // (bit_cast needs a scalar object, not a vector element)
            p[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(__builtin_bit_cast(float, sbits), cb, khb) + mob);
        }
        if constexpr (MASKED) {
            if (t >= t_lo) {
#pragma unroll
                for (int i = 0; i < 4; ++i) p[i] = s[t][i] == INT_MIN ? 0.0f : p[i];
            }
        }
        lsum0 += p[0] + p[1];
        lsum1 += p[2] + p[3];
        int w;  // both halves are overwritten below: an opaque undefined seed saves the v_mov of a zero
        asm volatile("" : "=v"(w));
        w = __builtin_amdgcn_cvt_pk_fp8_f32(p[0], p[1], w, false);
        w = __builtin_amdgcn_cvt_pk_fp8_f32(p[2], p[3], w, true);
        pb[t] = w;
    }
    l = l * alpha + (lsum0 + lsum1);
    m = m_new;
    return alpha;
}

}  // namespace
}  // namespace sage
