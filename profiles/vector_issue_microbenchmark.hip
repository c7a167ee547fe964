// How the vector instructions of the wavefronts of a SIMD issue on gfx950: the program behind vector_issue_microbenchmark.md.
//   hipcc --offload-arch=gfx950 -O3 -std=c++17 -Xclang -target-feature -Xclang -packed-fp32-ops \
//       profiles/vector_issue_microbenchmark.hip -o vector_issue && ./vector_issue
// Everything stays in registers: inline-assembly instructions on eight independent ones, in loops of a fixed length.  Cycles are time x 2.4 GHz.
#include <hip/hip_runtime.h>
#include <stdio.h>

#include <algorithm>

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));

enum Op { ADD, FMA, MUL, MOV, IADD, CVT, MAXI, MAX3, EXP, PACK, NOPS };
static const char *const kNames[] = {"add", "fma", "mul", "mov", "int add", "cvt", "max", "max3", "exp", "FP8 pack"};

#define CHECK(x)                                                                                   \
    do {                                                                                           \
        const hipError_t e_ = (x);                                                                 \
        if (e_ != hipSuccess) { fprintf(stderr, "%s: %s\n", #x, hipGetErrorString(e_)); exit(1); } \
    } while (0)

#if defined(__HIP_DEVICE_COMPILE__)
template <int OP>
__device__ __forceinline__ void op(float &a, float b, float c) {
    if constexpr (OP == ADD) asm volatile("v_add_f32 %0, %1, %0" : "+v"(a) : "v"(b));
    if constexpr (OP == FMA) asm volatile("v_fma_f32 %0, %1, %2, %0" : "+v"(a) : "v"(b), "v"(c));
    if constexpr (OP == MUL) asm volatile("v_mul_f32 %0, %1, %0" : "+v"(a) : "v"(b));
    if constexpr (OP == MOV) asm volatile("v_mov_b32 %0, %1" : "+v"(a) : "v"(b));
    if constexpr (OP == IADD) asm volatile("v_add_u32 %0, %1, %0" : "+v"(a) : "v"(b));
    if constexpr (OP == CVT) asm volatile("v_cvt_f32_i32 %0, %1" : "+v"(a) : "v"(b));
    if constexpr (OP == MAXI) asm volatile("v_max_i32 %0, %1, %0" : "+v"(a) : "v"(b));
    if constexpr (OP == MAX3) asm volatile("v_max3_i32 %0, %0, %1, %2" : "+v"(a) : "v"(b), "v"(c));
    if constexpr (OP == EXP) asm volatile("v_exp_f32 %0, %1" : "+v"(a) : "v"(b));
    if constexpr (OP == PACK) asm volatile("v_cvt_pk_fp8_f32 %0, %1, %2" : "+v"(a) : "v"(b), "v"(c));
}
template <int OP1, int OP2>
__device__ __forceinline__ void loop64(int n, float (&a)[8], float b, float c) {
    for (int r = 0; r < n; ++r) {
#pragma unroll
        for (int i = 0; i < 64; i += 2) {
            op<OP1>(a[i & 7], b, c);
            op<OP2>(a[(i + 1) & 7], b, c);
        }
    }
}
#define SAGE_REGS                                      \
    float a[8], b = threadIdx.x * 1e-3f, c = b * 2.0f; \
    for (int i = 0; i < 8; ++i) a[i] = b + i
#define SAGE_KEEP(extra)                                   \
    float s = extra;                                       \
    for (int i = 0; i < 8; ++i) s += a[i];                 \
    if (s == 12345.678f) out[threadIdx.x] = s
#endif

// two instructions in turn, all wavefronts alike
template <int OP1, int OP2>
__global__ __launch_bounds__(256) void alike(float *out, int n) {
#if defined(__HIP_DEVICE_COMPILE__)
    SAGE_REGS;
    loop64<OP1, OP2>(n, a, b, c);
    SAGE_KEEP(0.0f);
#endif
}
// wavefronts 0 to 3 of a workgroup (one per SIMD) run one instruction, 4 to 7 another
template <int OP1, int OP2>
__global__ __launch_bounds__(512) void two(float *out, int n) {
#if defined(__HIP_DEVICE_COMPILE__)
    SAGE_REGS;
    if (__builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8) == 0) loop64<OP1, OP1>(n, a, b, c);
    else loop64<OP2, OP2>(n, a, b, c);
    SAGE_KEEP(0.0f);
#endif
}
// an INT8 MFMA and COUNT instructions in turn, eight times an iteration
template <int OP, int COUNT>
__global__ __launch_bounds__(256) void mfma_and(float *out, int n) {
#if defined(__HIP_DEVICE_COMPILE__)
    SAGE_REGS;
    v16i m[2] = {};
    const v4i x = {1, 2, 3, (int)threadIdx.x}, y = {1, 1, 1, 1};
    for (int r = 0; r < n; ++r) {
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            m[t & 1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(x, y, m[t & 1], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < COUNT; ++i) op<OP>(a[i & 7], b, c);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    SAGE_KEEP((float)(m[0][0] + m[1][0]));
#endif
}
// The arithmetic of 64 scores per lane in runs of RUN: conversions, FMAs, additions and maxima, then exponentials and packs, at raised priority
// or not.  MFMA 1: an INT8 one per run first thing among the exponentials; 2: first thing among the others; 3: an FP8 one per two runs among
// the exponentials.
template <int RUN, bool RAISED, int MFMA>
__global__ __launch_bounds__(256, 2) void runs(float *out, int n) {
#if defined(__HIP_DEVICE_COMPILE__)
    SAGE_REGS;
    v16i m = {};
    v16f f = {};
    const v4i x = {1, 2, 3, (int)threadIdx.x}, y = {1, 1, 1, 1};
    const v8i z = {1, 2, 3, 4, 5, 6, 7, 8}, w = {1, 1, 1, 1, 1, 1, 1, 1};
    for (int r = 0; r < n; ++r) {
#pragma unroll
        for (int t = 0; t < 64 / RUN; ++t) {
            if constexpr (MFMA == 2) m = __builtin_amdgcn_mfma_i32_32x32x32_i8(x, y, m, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < RUN; ++i) {
                op<CVT>(a[(3 * i) & 7], b, c);
                op<FMA>(a[(3 * i + 1) & 7], b, c);
                op<ADD>(a[(3 * i + 2) & 7], b, c);
            }
#pragma unroll
            for (int i = 0; i < RUN / 2; ++i) op<MAX3>(a[(5 + i) & 7], b, c);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (RAISED) __builtin_amdgcn_s_setprio(1);
            if constexpr (MFMA == 1) m = __builtin_amdgcn_mfma_i32_32x32x32_i8(x, y, m, 0, 0, 0);
            if constexpr (MFMA == 3)
                if (t & 1) f = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(z, w, f, 0, 0, 0, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < RUN / 2; ++i) {
                op<EXP>(a[(3 * i) & 7], b, c);
                op<EXP>(a[(3 * i + 1) & 7], b, c);
                op<PACK>(a[(3 * i + 2) & 7], b, c);
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (RAISED) __builtin_amdgcn_s_setprio(0);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    SAGE_KEEP((float)m[0] + f[0]);
#endif
}

static float *g_out;
static const int kN = 2000;

template <class F>
double seconds(F &&launch) {
    hipEvent_t t0, t1;
    CHECK(hipEventCreate(&t0));
    CHECK(hipEventCreate(&t1));
    float best = 1e9f;
    for (int i = 0; i < 6; ++i) {
        CHECK(hipEventRecord(t0));
        launch();
        CHECK(hipGetLastError());
        CHECK(hipEventRecord(t1));
        CHECK(hipEventSynchronize(t1));
        float ms;
        CHECK(hipEventElapsedTime(&ms, t0, t1));
        if (i) best = std::min(best, ms);
    }
    CHECK(hipEventDestroy(t0));
    CHECK(hipEventDestroy(t1));
    return best * 1e-3;
}
// `per` units of work in each of kN iterations, 1 to 4 wavefronts per SIMD
template <class K>
void row(const char *name, K kernel, double per, int most) {
    printf("%-52s", name);
    for (int waves = 1; waves <= most; ++waves)
        printf(" %8.1f", seconds([&] { kernel<<<256 * waves, 256>>>(g_out, kN); }) * 2.4e9 / (kN * per * waves));
    printf("\n");
    fflush(stdout);
}
template <int I = 0>
void singles() {
    if constexpr (I < NOPS) {
        row(kNames[I], alike<I, I>, 64, 4);
        singles<I + 1>();
    }
}
template <int A, int B>
void pair_of() {
    printf("%s + %s: %.1f\n", kNames[A], kNames[B], seconds([&] { two<A, B><<<256, 512>>>(g_out, kN); }) * 2.4e9 / (kN * 64.0));
    fflush(stdout);
}
template <int A>
void pairs() {
    pair_of<A, ADD>();
    pair_of<A, FMA>();
    pair_of<A, EXP>();
    pair_of<A, CVT>();
    pair_of<A, PACK>();
    pair_of<A, MAX3>();
}

int main() {
    CHECK(hipMalloc(&g_out, 4096));
    printf("cycles per instruction, 1 to 4 wavefronts per SIMD with the same program\n");
    singles();
    row("cvt, fma in turn", alike<CVT, FMA>, 64, 4);
    row("max3, fma in turn", alike<MAX3, FMA>, 64, 4);
    row("exp, add in turn", alike<EXP, ADD>, 64, 4);
    row("INT8 MFMA alone", mfma_and<ADD, 0>, 8, 4);
    row("INT8 MFMA and eight adds", mfma_and<ADD, 8>, 8, 4);
    row("INT8 MFMA and eight conversions", mfma_and<CVT, 8>, 8, 4);
    printf("two wavefronts per SIMD, each with its own instruction: cycles per instruction of each\n");
    pairs<ADD>();
    pairs<FMA>();
    pairs<EXP>();
    pairs<CVT>();
    pairs<PACK>();
    pairs<MAX3>();
    printf("64 scores per lane, cycles per wavefront, 1 to 3 wavefronts per SIMD\n");
    row("runs of 4, no priority", runs<4, false, 0>, 1, 3);
    row("runs of 4, raised", runs<4, true, 0>, 1, 3);
    row("runs of 16, no priority", runs<16, false, 0>, 1, 3);
    row("runs of 16, raised", runs<16, true, 0>, 1, 3);
    row("runs of 4, 16 INT8 MFMAs, no priority", runs<4, false, 1>, 1, 3);
    row("runs of 4, 16 INT8 MFMAs among the exponentials, raised", runs<4, true, 1>, 1, 3);
    row("runs of 4, 16 INT8 MFMAs among the others, raised", runs<4, true, 2>, 1, 3);
    row("runs of 4, 8 FP8 MFMAs among the exponentials, raised", runs<4, true, 3>, 1, 3);
    CHECK(hipFree(g_out));
    return 0;
}
