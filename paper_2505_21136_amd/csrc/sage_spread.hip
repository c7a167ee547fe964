// The fused attention kernel for calls whose query tiles cannot fill the GPU (same arithmetic as sage_prefill.hip, paper
// Sec. 2.1 and 3.1): the work of a key step is spread over the wavefronts of a workgroup instead of its rows.
//
// A workgroup owns 32 * RG query rows.  Of a step's 128 keys wavefront w of a row group scores keys 32w .. 32w + 31 (one
// 32x32 tile of S^T), so the chain that a row's recurrence is -- scores, maximum, exponentials, P^, the same again -- is a
// quarter as long as where a wavefront scores all 128, and there are 4 / RG times as many workgroups.  The wavefronts of a row
// group meet twice per step in what one barrier separates: the tile maxima of step j+1 and the P^ of step j go through LDS
// together.  P^V^ is split by channels: d = 128: wavefront w makes channels 32w .. +31; at d = 64 there are only two such tiles,
// made by two of the four wavefronts.  (Splitting the keys between all four instead, one MFMA each, is 4 % faster with 64 rows and
// 1 % slower with 32, but adds up in another order.)  Every addition has the order of prefill_kernel: the result of a row does not
// depend on which of the two kernels the number of heads selects.
//
// Two more wavefronts do nothing but copy: K^ and V^ tiles global -> LDS (ring of four steps), three steps ahead, so that
// neither the latency of the memory nor the texture path's 16 cycles per 1 KB piece stands in the chain of the others.  (The
// operands cannot be loaded straight into registers instead: neighbouring lanes want neighbouring rows, 64 cache lines per
// load, and the texture path takes one line per cycle: 0.95 us per step against 0.55 us.)
//
// What bounds it is the chain: about 120 vector instructions of one wavefront, matrix results and LDS round trips waited for
// by it, and a barrier per step: 0.57 us per step with 32 rows, 0.79 us with 64 (d = 64: 0.48 and 0.71), where a wavefront of the
// other kernel, alone on its SIMD, takes 1.33 us (1.15).  (Tried: operands loaded straight into registers; scores made one step instead of two ahead of
// their use: 0.64 us.)  The per-step work that does not shrink with the tile weighs more than in the other kernel and LDS
// holds one workgroup per CU (two of 32 rows at d = 64), so with enough query tiles that one is faster; launch_attn has the lines and both sides.
#include "sage_attn_device.h"
#include "sage_internal.h"

#include <limits.h>
#include <math.h>

namespace sage {
namespace {

typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));

// Workgroup barrier that orders LDS accesses only: copies stay in flight across it.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int D, int RG, bool CAUSAL, bool BF16, bool QRAW>
__global__ __launch_bounds__(256 * RG + 128) void spread_kernel(
    const void *__restrict__ Qsrc, const int8_t *__restrict__ Kc, const uint8_t *__restrict__ Vt,
    const float *__restrict__ dq, const float *__restrict__ dk, const float *__restrict__ dv,
    uint16_t *__restrict__ out, Strides q_st, Strides o_st, int Nq, int Nk, int nT, int nQblk, int nKblk, int Hq,
    int group, float sm_scale, float log2_pr, int n_tiles) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int KC = D / 32;             // 32-wide contraction chunks of Q.K^T
    constexpr int NPV = 2;                 // P^V^ MFMAs of a wavefront per step, one per 64 keys
    constexpr int TILE = 128 * D;          // bytes of one K^ (or V^) tile
    constexpr int ROWS = 32 * RG, NC = 4 * RG;  // query rows and scoring wavefronts of a workgroup
    __shared__ __attribute__((aligned(1024))) uint8_t lds[8 * TILE];  // K^ of steps j & 3, then V^
    __shared__ __attribute__((aligned(16))) uint8_t p_lds[2][ROWS * 128];  // P^ of a step: row = query, V^'s byte order
    __shared__ __attribute__((aligned(16))) float max_lds[2][ROWS][4];     // per query and wavefront: maximum of the key tile
    __shared__ float cst_lds[2][64];  // de-quantisation constants of 64 consecutive K blocks (32 steps), even and odd strips
    __shared__ __attribute__((aligned(16))) float q_wave_max[NC];
    __shared__ float l_lds[RG][4][64];
    __shared__ __attribute__((aligned(16))) float dv_lds[D];  // delta_V of this head, for the epilogue

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lq = lane & 31, h = lane >> 5;
    int bh, tile;
    map_workgroup<CAUSAL>((int)blockIdx.x, (int)gridDim.x, n_tiles, bh, tile);
    const int bhk = (bh / Hq) * (Hq / group) + (bh % Hq) / group;
    const int shift = Nk - Nq;
    const int qblk = tile * ROWS / kBQ;
    const float *dkh = dk + (size_t)bhk * nKblk;
    int nsteps = nT;
    if constexpr (CAUSAL) nsteps = min(nT, (min(tile * ROWS + ROWS - 1, Nq - 1) + shift) / kW + 1);

    const auto block_scale = [&](float &rcp) {
        if constexpr (QRAW) {
            float a = 0.0f;
#pragma unroll
            for (int w = 0; w < NC; ++w) a = fmaxf(a, q_wave_max[w]);
            rcp = a > 0.0f ? 127.0f / a : 0.0f;
            return a / 127.0f;
        }
        rcp = 0.0f;
        return dq[(size_t)bh * nQblk + qblk];
    };
    // The barriers every wavefront passes: P0 (K^ of steps 0 .. 2 and the maxima of Q are there), P1 (K^ of steps 0 .. 2 has been
    // read), one in front of every step j < nsteps (K^(j+3), V^(j), the tile maxima of step j and P^ of step j-1 are there) and
    // one in front of the last P^V^.

    if (wave >= NC) {
        // ---- copies: this wavefront moves every other 1 KB piece of a tile ----
        const int pw = wave - NC;
        constexpr int NP = TILE / 2048;  // pieces per tile and wavefront
        const uint8_t *Kh = reinterpret_cast<const uint8_t *>(Kc) + (size_t)bhk * Nk * D;
        const uint8_t *Vh = Vt + (size_t)bhk * nT * D * 128;
        const int k_bytes = Nk * D, v_bytes = nT * D * 128;
        // (both swizzles repeat every 8 rows, i.e. every 1 KB piece or sooner, so one offset serves all pieces)
        const int kvoff = k_source<D>(lane), vvoff = v_source(lane);
        const int dst0 = lds_address(lds);
        const auto copy = [&](const uint8_t *head, int bytes, int voff, int j, int dst) {
            if (j >= nsteps) return;
#pragma unroll
            for (int k = 0; k < NP; ++k) {
                const int off = (2 * k + pw) * 1024, first = j * TILE + off;
                // (bounded to what is left of the head's buffer: rows >= Nk of the last K^ tile read as zero)
                lds_copy16(lds_copy_rsrc(head + first, copy_left(bytes, first)), voff, dst0 + dst + off);
            }
        };
        const auto copy_k = [&](int j) { copy(Kh, k_bytes, kvoff, j, (j & 3) * TILE); };
        const auto copy_v = [&](int j) { copy(Vh, v_bytes, vvoff, j, (4 + (j & 3)) * TILE); };
        // wait until at most n tiles' copies are outstanding (they complete in order)
        const auto wait_tiles = [&](int n) {
            if (n >= 4) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * NP));
            else if (n == 3) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * NP));
            else if (n == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NP));
            else if (n == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(1 * NP));
            else asm volatile("s_waitcnt vmcnt(0)");
        };
        const auto left = [&](int j, int n) { return min(n, max(0, nsteps - j)); };  // how many of steps j .. j+n-1 exist
        copy_k(0), copy_k(1), copy_k(2), copy_k(3);
        copy_v(0), copy_v(1), copy_v(2);
        wait_tiles(left(3, 1) + left(0, 3));
        lds_barrier();  // P0
        float rcp, dkv = 0.0f;
        const float delta_q = block_scale(rcp);
        lds_barrier();  // P1
        copy_k(4), copy_k(5);
        const double cq = (double)delta_q * (double)sm_scale * 1.4426950408889634;
        if (pw == 0) cst_lds[0][lane] = (float)(cq * (double)dkh[min(lane, nKblk - 1)]);
        for (int j = 0; j < nsteps; ++j) {
            if (pw == 0 && (j & 31) == 15) dkv = dkh[min(2 * j + 34 + lane, nKblk - 1)];
            if (pw == 0 && (j & 31) == 30) cst_lds[((j + 2) >> 5) & 1][lane] = (float)(cq * (double)dkv);
            // K^(j+3) and V^(j) have landed when at most the copies of the next two steps are outstanding (V^(2) went first)
            wait_tiles(left(j + 4, 2) + left(j + 1, 2) - (j == 1 && nsteps > 2 ? 1 : 0));
            lds_barrier();
            copy_k(j + 6);
            copy_v(j + 3);
        }
        lds_barrier();
        return;
    }

    const int rg = wave >> 2, w4 = wave & 3;  // row group, key tile
    const int row0 = tile * ROWS + rg * 32, qrow = row0 + lq;

    // ---- Q: the wavefront's operand (those of a row group hold the same 32 rows) and, unquantised, the maximum of the block ----
    v4i qreg[KC];
    const int ct = D == 128 ? w4 : w4 & 1;
    // (d = 64: two wavefronts of a row group make one; the others multiply what is in their registers, which costs less than a
    // branch inside the exponentials, and store nothing.  On different SIMDs for the two row groups, and not those of the copies.)
    const bool pv = D == 128 || (w4 >> 1) != rg;
    if (tid < D / 4)
        *reinterpret_cast<float4 *>(dv_lds + 4 * tid) = *reinterpret_cast<const float4 *>(dv + (size_t)bhk * D + 4 * tid);
    const float dk0 = dkh[min(w4 >> 1, nKblk - 1)], dk1 = dkh[min(2 + (w4 >> 1), nKblk - 1)];
    float delta_q;
    const int kof = k_off<D>(w4 * 32 + lq, h);
    const auto read_k = [&](v4i (&f)[KC], int j) {
#pragma unroll
        for (int ch = 0; ch < KC; ++ch) f[ch] = *reinterpret_cast<const v4i *>(lds + (j & 3) * TILE + (kof ^ (32 * ch)));
    };
    v4i k0[KC], k1[KC], kf[KC];  // kf: K^ of the step whose scores are made next
    const auto first_tiles = [&](auto also) {
        lds_barrier();  // P0
        read_k(k0, 0);
        read_k(k1, 1);
        read_k(kf, 2);
        also();
        lds_barrier();  // P1
    };
    if constexpr (QRAW) {
        // All loads are of whole rows (a lane of the operand's layout wants a row of its own: 64 cycles of the texture path per
        // load instead of 16, 4096 of them for the two groups of loads below at d = 128): the workgroup's own rows, which go to the
        // wavefronts through LDS, and the whole block for its maximum.  2 heads x 1024 x 1024, d = 128 10.5 -> 9.5 us, 64 x 128 x 128 6.8 -> 5.7.
        const uint16_t *Qh = static_cast<const uint16_t *>(Qsrc) + (bh / Hq) * q_st.b + (bh % Hq) * q_st.h;
        constexpr int RC = D / 8, SW = RC - 1;  // 16-byte chunks per row, and the swizzle's mask
        constexpr int OWN = ROWS * RC / (64 * NC), ALL = kBQ * RC / (64 * NC);
        static_assert(ROWS * D * 2 <= (int)sizeof(p_lds), "the rows wait where P^ goes later");
        uint8_t *q_lds = &p_lds[0][0];
        uint4 own[OWN], all[ALL];
#pragma unroll
        for (int x = 0; x < OWN; ++x) {
            const int e = 64 * NC * x + tid;
            own[x] = *reinterpret_cast<const uint4 *>(Qh + min(tile * ROWS + e / RC, Nq - 1) * q_st.n + e % RC * 8);
        }
#pragma unroll
        for (int x = 0; x < ALL; ++x) {
            const int e = 64 * NC * x + tid;
            all[x] = *reinterpret_cast<const uint4 *>(Qh + min(qblk * kBQ + e / RC, Nq - 1) * q_st.n + e % RC * 8);
        }
#pragma unroll
        for (int x = 0; x < OWN; ++x) {
            const int e = 64 * NC * x + tid, row = e / RC, c = e % RC;
            *reinterpret_cast<uint4 *>(q_lds + row * D * 2 + ((c ^ (row & SW)) << 4)) = own[x];
        }
        float amax = 0.0f;
#pragma unroll
        for (int x = 0; x < ALL; ++x) {  // (rows past the end repeat the last one, which the block has, too)
            float f[8];
            unpack8<BF16>(all[x], f);
#pragma unroll
            for (int i = 0; i < 8; ++i) amax = fmaxf(amax, fabsf(f[i]));
        }
        amax = wave_max(amax);
        if (lane == 0) q_wave_max[wave] = amax;
        uint4 qraw[KC][2];
        first_tiles([&]() {
            const int row = rg * 32 + lq;
#pragma unroll
            for (int ch = 0; ch < KC; ++ch)
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    qraw[ch][e] = *reinterpret_cast<const uint4 *>(q_lds + row * D * 2 + (((4 * ch + 2 * h + e) ^ (row & SW)) << 4));
        });
        float rcp;
        delta_q = block_scale(rcp);
#pragma unroll
        for (int ch = 0; ch < KC; ++ch)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                float f[8];
                unpack8<BF16>(qraw[ch][e], f);
                const uint2 w = int8_codes(f, rcp);
                qreg[ch][2 * e] = (int)w.x;
                qreg[ch][2 * e + 1] = (int)w.y;
            }
    } else {
        const int8_t *Qr = static_cast<const int8_t *>(Qsrc) + (bh / Hq) * q_st.b + (bh % Hq) * q_st.h +
                           min(qrow, Nq - 1) * q_st.n;
#pragma unroll
        for (int ch = 0; ch < KC; ++ch) qreg[ch] = *reinterpret_cast<const v4i *>(Qr + ch * 32 + h * 16);
        first_tiles([]() {});
        float rcp;
        delta_q = block_scale(rcp);
    }

    // where this lane's P^ dwords go (key quads b = 0, 2 and b = 1, 3 are adjacent) and where its operands come from: row lq of
    // a 32-row tile, 16-byte chunk 2x + h, whose swizzled place is that of chunk h xor 32x bytes
    int p_wr[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) p_wr[e] = v_off(rg * 32 + lq, 4 * (w4 >> 1) + 2 * e + h) + 8 * (w4 & 1);
    const int vof = 4 * TILE + v_off(32 * ct + lq, h), pof = v_off(rg * 32 + lq, h);
    const auto operand = [&](const uint8_t *base, int off, int u) {
        const v4i lo = *reinterpret_cast<const v4i *>(base + (off ^ (64 * u)));
        const v4i hi = *reinterpret_cast<const v4i *>(base + (off ^ (64 * u + 32)));
        return v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    };
    const v16i zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    const auto scores = [&](const v4i (&f)[KC]) {
        v16i s = zero;
#pragma unroll
        for (int ch = 0; ch < KC; ++ch) s = __builtin_amdgcn_mfma_i32_32x32x32_i8(f[ch], qreg[ch], s, 0, 0, 0);
        return s;
    };
    // Whether the tile of step j reaches beyond the last key or, causal, beyond the row group's first row's last key; the last
    // visible key of this lane's row, counted from this lane's first key of that tile.
    const auto needs_mask = [&](int j) {
        return j * kW + w4 * 32 + 31 > (CAUSAL ? min(Nk - 1, row0 + shift) : Nk - 1);
    };
    const auto limit = [&](int j) { return (CAUSAL ? min(Nk - 1, qrow + shift) : Nk - 1) - (j * kW + w4 * 32 + 4 * h); };
    // The maximum of the tile of step j per row; keys beyond the row's limit count as minus infinity.
    const auto tile_max = [&](const v16i &s, int j, float c) {
        int a = imax3(s[0], s[1], s[2]), b = imax3(s[3], s[4], s[5]);
#pragma unroll
        for (int i = 6; i < 14; i += 4) {
            a = imax3(a, s[i], s[i + 1]);
            b = imax3(b, s[i + 2], s[i + 3]);
        }
        a = max(imax3(a, s[14], s[15]), b);
        float mx = (float)a * c;
        if (needs_mask(j)) {
            const int lim = limit(j);
            a = INT_MIN;
#pragma unroll
            for (int e = 0; e < 16; ++e) a = max(a, 8 * (e >> 2) + (e & 3) > lim ? INT_MIN : s[e]);
            mx = a == INT_MIN ? -INFINITY : (float)a * c;
        }
        return halves_max(mx);
    };

    float m = -INFINITY, l = 0.0f, alpha = 1.0f;
    v16f o = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const double cq = (double)delta_q * (double)sm_scale * 1.4426950408889634;
    float c0 = (float)(cq * (double)dk0), c1 = (float)(cq * (double)dk1);  // constants of even and odd steps
    v16i s0 = scores(k0), s1 = scores(k1);                                 // scores of even and odd steps
    const v8i none = {0, 0, 0, 0, 0, 0, 0, 0};
    v8i vf[NPV] = {none, none}, pf[NPV] = {none, none};  // V^ and P^ of the step before
    {
        const float mx = tile_max(s0, 0, c0);
        if (h == 0) max_lds[0][rg * 32 + lq][w4] = mx;
    }

    // Step j: P^ of its scores s (which then become those of step j+2), the maximum of step j+1's scores, P^V^ of step j-1.
    const auto step = [&](auto parity, int j, v16i &s, float &c, const v16i &s_next, float c_next) __attribute__((always_inline)) {
        constexpr int PAR = decltype(parity)::value;
        lds_barrier();
        const float4 mx = *reinterpret_cast<const float4 *>(max_lds[PAR][rg * 32 + lq]);
        if (pv && j > 0) {
#pragma unroll
            for (int n = 0; n < NPV; ++n) pf[n] = operand(p_lds[PAR ^ 1], pof, n);
        }
        const float c_after = cst_lds[((j + 2) >> 5) & 1][(2 * (j + 2) + (w4 >> 1)) & 63];
        const float mx_next = tile_max(s_next, j + 1, c_next);
        float x[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int sv = s[i];
            x[i] = (float)sv;
        }
        const float m_new = max_no_nan(max_no_nan(max_no_nan(mx.x, mx.y), max_no_nan(mx.z, mx.w)), m);
        const float mo = log2_pr - m_new;  // P~ * P_r = 2^(x - m' + log2 P_r)
        if (j > 0 && __builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) o *= alpha;
        __builtin_amdgcn_sched_barrier(0);
        // exponentials, with the matrix work in between so that its issue does not wait in one place: Q.K^T of step j+2 first, whose
        // operand registers then take K^ of step j+3, then P^V^ of step j-1
#pragma unroll
        for (int b = 0; b < 4; ++b) {
#pragma unroll
            for (int i = 4 * b; i < 4 * b + 4; ++i) x[i] = __builtin_fmaf(x[i], c, mo);
            if (b < 2) {
#pragma unroll
                for (int ch = b * KC / 2; ch < (b + 1) * KC / 2; ++ch)
                    s = __builtin_amdgcn_mfma_i32_32x32x32_i8(kf[ch], qreg[ch], ch == 0 ? zero : s, 0, 0, 0);
            } else if (b - 2 < NPV) {
                if (j > 0) o = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(vf[b - 2], pf[b - 2], o, 0, 0, 0, 0, 0, 0);
            }
#pragma unroll
            for (int i = 4 * b; i < 4 * b + 4; ++i) x[i] = __builtin_amdgcn_exp2f(x[i]);
            asm volatile("" : "+v"(x[4 * b]), "+v"(x[4 * b + 1]), "+v"(x[4 * b + 2]), "+v"(x[4 * b + 3]));
            if (b == 1) read_k(kf, j + 3);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (pv) {
#pragma unroll
            for (int n = 0; n < NPV; ++n) vf[n] = operand(lds + (j & 3) * TILE, vof, n);
        }
        if (needs_mask(j)) {
            const int lim = limit(j);
#pragma unroll
            for (int e = 0; e < 16; ++e) x[e] = 8 * (e >> 2) + (e & 3) > lim ? 0.0f : x[e];
        }
        int w[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            int y;
            asm volatile("" : "=v"(y));
            y = __builtin_amdgcn_cvt_pk_fp8_f32(x[4 * b], x[4 * b + 1], y, false);
            w[b] = __builtin_amdgcn_cvt_pk_fp8_f32(x[4 * b + 2], x[4 * b + 3], y, true);
        }
        *reinterpret_cast<uint2 *>(&p_lds[PAR][p_wr[0]]) = make_uint2((uint32_t)w[0], (uint32_t)w[2]);
        *reinterpret_cast<uint2 *>(&p_lds[PAR][p_wr[1]]) = make_uint2((uint32_t)w[1], (uint32_t)w[3]);
        if (h == 0) max_lds[PAR ^ 1][rg * 32 + lq][w4] = mx_next;
        __builtin_amdgcn_sched_barrier(0);
        alpha = __builtin_amdgcn_exp2f(m - m_new);
        float lsum0 = x[0] + x[1], lsum1 = x[2] + x[3];
#pragma unroll
        for (int b = 1; b < 4; ++b) {
            lsum0 += x[4 * b] + x[4 * b + 1];
            lsum1 += x[4 * b + 2] + x[4 * b + 3];
        }
        l = __builtin_fmaf(l, alpha, lsum0 + lsum1);
        m = m_new;
        c = c_after;
    };
    for (int j = 0; j < nsteps; j += 2) {
        step(std::integral_constant<int, 0>{}, j, s0, c0, s1, c1);
        if (j + 1 < nsteps) step(std::integral_constant<int, 1>{}, j + 1, s1, c1, s0, c0);
    }
    l_lds[rg][w4][lane] = l;
    lds_barrier();  // P^ of the last step and the row sums
    if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) o *= alpha;
#pragma unroll
    for (int n = 0; n < NPV; ++n)
        o = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(vf[n], operand(p_lds[(nsteps - 1) & 1], pof, n), o, 0, 0, 0,
                                                            0, 0, 0);
    const float inv =
        1.0f / halves_sum((l_lds[rg][0][lane] + l_lds[rg][1][lane]) + (l_lds[rg][2][lane] + l_lds[rg][3][lane]));
    if (!pv) return;
    // ---- epilogue: O = acc * delta_V / (P_r * l); l already carries the factor P_r ----
    uint16_t *orow = out + (bh / Hq) * o_st.b + (bh % Hq) * o_st.h + qrow * o_st.n + 32 * ct;
#pragma unroll
    for (int b2 = 0; b2 < 2; ++b2) {
        // after the exchange between the wavefront's halves a lane holds the eight channels 8 * (2*b2 + h) ..
        uint32_t w[2][2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int b = 2 * b2 + e;
            const float4 sc = *reinterpret_cast<const float4 *>(dv_lds + 32 * ct + 8 * b + 4 * h);
            w[e][0] = pack2<BF16>(o[4 * b] * (sc.x * inv), o[4 * b + 1] * (sc.y * inv));
            w[e][1] = pack2<BF16>(o[4 * b + 2] * (sc.z * inv), o[4 * b + 3] * (sc.w * inv));
        }
        swap32(w[0][0], w[1][0]);
        swap32(w[0][1], w[1][1]);
        if (qrow < Nq)
            *reinterpret_cast<uint4 *>(orow + 16 * b2 + 8 * h) = make_uint4(w[0][0], w[0][1], w[1][0], w[1][1]);
    }
#endif  // __HIP_DEVICE_COMPILE__
}

template <int D, int RG>
hipError_t launch_spread_d(const void *q, bool q_raw, Strides q_st, const int8_t *k_i8, const uint8_t *v_fp8,
                           const float *q_scale, const float *k_scale, const float *v_scale, void *out, Strides o_st, int B,
                           int Hq, int Hkv, int Nq, int Nk, bool causal, float sm_scale, float log2_pr, bool bf16,
                           hipStream_t stream) {
    const int n_tiles = cdiv(Nq, 32 * RG);
    const dim3 grid(B * Hq * n_tiles);
    const int nT = cdiv(Nk, kW), nQ = cdiv(Nq, kBQ), nK = cdiv(Nk, kBK);
    uint16_t *o16 = static_cast<uint16_t *>(out);
#define SAGE_LAUNCH(C, BF, QR)                                                                                         \
    spread_kernel<D, RG, C, BF, QR><<<grid, 256 * RG + 128, 0, stream>>>(                                                 \
        q, k_i8, v_fp8, q_scale, k_scale, v_scale, o16, q_st, o_st, Nq, Nk, nT, nQ, nK, Hq, Hq / Hkv, sm_scale, log2_pr,   \
        n_tiles)
#define SAGE_LAUNCH_Q(C, BF)                                            \
    do {                                                                \
        if (q_raw) SAGE_LAUNCH(C, BF, true); else SAGE_LAUNCH(C, BF, false); \
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

hipError_t launch_spread(const void *q, bool q_raw, Strides q_st, const int8_t *k_i8, const uint8_t *v_fp8,
                         const float *q_scale, const float *k_scale, const float *v_scale, void *out, Strides o_st, int B,
                         int Hq, int Hkv, int Nq, int Nk, int d, bool causal, float sm_scale, float p_r, bool bf16,
                         hipStream_t stream, int row_groups) {
    const float log2_pr = (float)log2((double)p_r);
#define SAGE_SPREAD(D, RG)                                                                                                   \
    launch_spread_d<D, RG>(q, q_raw, q_st, k_i8, v_fp8, q_scale, k_scale, v_scale, out, o_st, B, Hq, Hkv, Nq, Nk, causal, sm_scale, \
                           log2_pr, bf16, stream)
    if (d == 128) return row_groups == 1 ? SAGE_SPREAD(128, 1) : SAGE_SPREAD(128, 2);
    return row_groups == 1 ? SAGE_SPREAD(64, 1) : SAGE_SPREAD(64, 2);
#undef SAGE_SPREAD
}

}  // namespace sage
