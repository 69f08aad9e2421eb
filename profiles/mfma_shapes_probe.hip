// Bare loops of MFMAs (gfx950): what the two bf16 shapes cost in cycles, in issue slots and, through the clock that the chip
// can hold, in power.  Its figures stand beside it in this folder.  Stands alone, is part of no library:
//     hipcc --offload-arch=gfx950 -O3 -std=c++17 -Xclang -target-feature -Xclang -packed-fp32-ops profiles/mfma_shapes_probe.hip -o probe
//     ./probe
// Every loop runs on 256 workgroups, one per compute unit.  A line gives the cycles that the matrix pipe of a SIMD has per
// 32,768 flop (one MFMA of 32 x 32 x 16 or two of 16 x 16 x 32; 32 cycles is the pipe's own time), the rate, and the clock.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <utility>
#include <vector>

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Operand fragments, 64 lanes x 16 bytes each: 16 of keys or values, 8 of queries, 4 of weights.
constexpr int kA = 16, kQ = 8, kP = 4;

__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }

// Cycles from the first wavefront's start to the last one's end, of workgroup 0 (the clock counts the shader's cycles).
struct Span {
    uint64_t* out;
    uint64_t t0;
    __device__ __forceinline__ Span(uint64_t* o) : out(o) {
        __syncthreads();
        t0 = clock64();
    }
    __device__ __forceinline__ void end() {
        __syncthreads();
        if (threadIdx.x == 0 && blockIdx.x == 0) *out = clock64() - t0;
    }
};

// ---- products alone, on the operands of an attention tile of 32 queries x 64 keys x 128 dims
enum {
    kBoth32,        // scores into two accumulators that start from zero, then P V into four that stay
    kBoth16B,       // the same as 16 x 16 x 32, query / weight operand kept over neighbouring products
    kBoth16A,       // ... key / value operand kept for both query tiles
    kScores32Tile,  // the scores of kBoth32 alone: two accumulators, zeroed for every tile
    kScores32,      // four accumulators that stay, operand B = queries
    kPV32,          // the same instructions, operand B = weights
    kScores32Zero,  // four accumulators that start from zero every 32 products, operand B = queries
    kPV32Zero,      // the same instructions, operand B = weights
    kProducts
};
template <int VAR>
__global__ __launch_bounds__(512) void products(const u32x4* ops, int iters, float* sink, uint64_t* cycles) {
    const int lane = threadIdx.x & 63;
    bf16x8 a[kA], q[kQ], p[kP];
    for (int f = 0; f < kA; ++f) a[f] = __builtin_bit_cast(bf16x8, ops[f * 64 + lane]);
    for (int f = 0; f < kQ; ++f) q[f] = __builtin_bit_cast(bf16x8, ops[(kA + f) * 64 + lane]);
    for (int f = 0; f < kP; ++f) p[f] = __builtin_bit_cast(bf16x8, ops[(kA + kQ + f) * 64 + lane]);
    float res = 0.f;
    Span span(cycles);
    if constexpr (VAR == kBoth32 || VAR == kScores32Tile) {
        f32x16 o[4] = {}, s[2];
        for (int it = 0; it < iters; ++it) {
            for (int m = 0; m < 2; ++m) s[m] = f32x16{};
#pragma unroll
            for (int t = 0; t < 8; ++t)
#pragma unroll
                for (int m = 0; m < 2; ++m) s[m] = mfma(a[2 * t + m], q[t], s[m]);
            if constexpr (VAR == kBoth32)
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int d = 0; d < 4; ++d) o[d] = mfma(a[4 * k + d], p[k], o[d]);
            asm volatile("" ::"v"(s[0]), "v"(s[1]));
        }
        for (int d = 0; d < 4; ++d) for (int r = 0; r < 16; ++r) res += o[d][r];
    } else if constexpr (VAR == kBoth16B || VAR == kBoth16A) {
        // a: 4 k-steps x 4 key tiles, or 2 k-steps x 8 dim tiles; q: 4 k-steps x 2 query tiles; p: 2 x 2
        f32x4 o[8][2] = {}, s[4][2];
        for (int it = 0; it < iters; ++it) {
            for (int m = 0; m < 4; ++m) for (int n = 0; n < 2; ++n) s[m][n] = f32x4{};
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int x = 0; x < 8; ++x) {
                    const int m = VAR == kBoth16B ? x & 3 : x >> 1, n = VAR == kBoth16B ? x >> 2 : (x ^ m) & 1;
                    s[m][n] = mfma(a[4 * t + m], q[2 * t + n], s[m][n]);
                }
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int x = 0; x < 16; ++x) {
                    const int d = VAR == kBoth16B ? x & 7 : x >> 1, n = VAR == kBoth16B ? x >> 3 : (x ^ d) & 1;
                    o[d][n] = mfma(a[8 * k + d], p[2 * k + n], o[d][n]);
                }
            for (int m = 0; m < 4; ++m) for (int n = 0; n < 2; ++n) asm volatile("" ::"v"(s[m][n]));
        }
        for (int d = 0; d < 8; ++d) for (int n = 0; n < 2; ++n) for (int r = 0; r < 4; ++r) res += o[d][n][r];
    } else {
        constexpr bool kWeights = VAR == kPV32 || VAR == kPV32Zero, kZero = VAR == kScores32Zero || VAR == kPV32Zero;
        f32x16 o[4] = {};
        for (int it = 0; it < iters; ++it) {
            if constexpr (kZero) for (int d = 0; d < 4; ++d) o[d] = f32x16{};
#pragma unroll
            for (int k = 0; k < 8; ++k)
#pragma unroll
                for (int d = 0; d < 4; ++d) o[d] = mfma(a[(4 * k + d) & (kA - 1)], kWeights ? p[k & 3] : q[k & 3], o[d]);
            if constexpr (kZero) for (int d = 0; d < 4; ++d) asm volatile("" ::"v"(o[d]));
        }
        for (int d = 0; d < 4; ++d) for (int r = 0; r < 16; ++r) res += o[d][r];
    }
    span.end();
    sink[blockIdx.x * blockDim.x + threadIdx.x] = res;
}

// ---- groups of products and vector instructions: M = MFMA, v = v_fma_f32, e = v_exp_f32, in this order
struct Pattern { int shape; const char* text; };
constexpr Pattern kPatterns[] = {
    {32, "M"}, {32, "Mvvvv"}, {32, "Mvvvvvv"}, {32, "Mvvvvvvvv"}, {32, "Mvvvvvvvvvv"}, {32, "Mvvvvvvvvvvvv"}, {32, "Mvvvvvvvvvvvvvvvv"},
    {32, "Me"}, {32, "Mvvve"}, {32, "Mvvvve"}, {32, "Mvvvvve"}, {32, "Mvvvvvve"}, {32, "Mvvvvvvvve"}, {32, "Mee"}, {32, "Meee"}, {32, "Meeee"}, {32, "Meeeeee"},
    {16, "MM"}, {16, "MvMv"}, {16, "MvvMvv"}, {16, "MvvvMvvv"}, {16, "MvvvvMvvvv"}, {16, "MvvvvvvMvvvvvv"}, {16, "MMvvvv"},
    {16, "MvvMve"}, {16, "MMvvve"}, {16, "MeMe"}, {16, "MeeMee"},
};
constexpr int kNumPatterns = sizeof(kPatterns) / sizeof(kPatterns[0]);
constexpr int length(const char* s) { int n = 0; while (s[n]) ++n; return n; }
constexpr int count(const char* s, char c, int upto) { int n = 0; for (int i = 0; i < upto; ++i) n += s[i] == c; return n; }
constexpr int kGroups = 16;     // per loop iteration

template <int P, int I, typename Acc, int N>
__device__ __forceinline__ void step(const bf16x8 (&a)[4], const bf16x8 (&b)[4], Acc (&c)[N], float (&x)[8], float (&z)[4], float y) {
    constexpr const char* text = kPatterns[P].text;
    constexpr int len = length(text), at = I % len;
    constexpr char what = text[at];
    constexpr int no = count(text, what, len) * (I / len) + count(text, what, at);
    if constexpr (what == 'M' && N == 4) c[no % 4] = mfma(a[no % 4], b[no / 4 % 4], c[no % 4]);
    else if constexpr (what == 'M') c[no % 16] = mfma(a[no / 2 % 4], b[no % 2 + 2 * (no / 16 % 2)], c[no % 16]);
    else if constexpr (what == 'v') asm volatile("v_fma_f32 %0, %0, %1, %1" : "+v"(x[no % 8]) : "v"(y));
    else asm volatile("v_exp_f32 %0, %1" : "=v"(z[no % 4]) : "v"(y));
    __builtin_amdgcn_sched_barrier(0);
}
template <int P, typename Acc, int N, int... I>
__device__ __forceinline__ void steps(std::integer_sequence<int, I...>, const bf16x8 (&a)[4], const bf16x8 (&b)[4], Acc (&c)[N], float (&x)[8], float (&z)[4], float y) {
    (step<P, I>(a, b, c, x, z, y), ...);
}
template <int P>
__global__ __launch_bounds__(512) void groups(const u32x4* ops, int iters, float* sink, uint64_t* cycles) {
    const int lane = threadIdx.x & 63;
    bf16x8 a[4], b[4];
    for (int f = 0; f < 4; ++f) {
        a[f] = __builtin_bit_cast(bf16x8, ops[f * 64 + lane]);
        b[f] = __builtin_bit_cast(bf16x8, ops[(kA + f) * 64 + lane]);
    }
    constexpr int N = kPatterns[P].shape == 32 ? 4 : 16;
    using Acc = std::conditional_t<N == 4, f32x16, f32x4>;
    Acc c[N] = {};
    float x[8] = {}, z[4] = {}, y = lane * 0.001f, res = 0.f;
    Span span(cycles);
    for (int it = 0; it < iters; ++it)
        steps<P>(std::make_integer_sequence<int, kGroups * length(kPatterns[P].text)>{}, a, b, c, x, z, y);
    span.end();
    for (int i = 0; i < N; ++i) for (int r = 0; r < 64 / N; ++r) res += c[i][r];
    for (int i = 0; i < 8; ++i) res += x[i];
    for (int i = 0; i < 4; ++i) res += z[i];
    sink[blockIdx.x * blockDim.x + threadIdx.x] = res;
}

static void check(hipError_t e) {
    if (e == hipSuccess) return;
    std::fprintf(stderr, "%s\n", hipGetErrorString(e));
    std::exit(1);
}
static u32x4* ops;
static float* sink;
static uint64_t* cycles;
static hipEvent_t e0, e1;

using Kernel = void (*)(const u32x4*, int, float*, uint64_t*);
// `units` of 32,768 flop per iteration and wavefront; three launches after a first one, the last one's cycles
static void time_it(const char* name, Kernel kernel, int threads, int iters, int units) {
    kernel<<<256, threads>>>(ops, iters, sink, cycles);
    check(hipEventRecord(e0));
    for (int i = 0; i < 3; ++i) kernel<<<256, threads>>>(ops, iters, sink, cycles);
    check(hipGetLastError());
    check(hipEventRecord(e1));
    check(hipEventSynchronize(e1));
    float ms;
    uint64_t n;
    check(hipEventElapsedTime(&ms, e0, e1));
    check(hipMemcpy(&n, cycles, sizeof n, hipMemcpyDeviceToHost));
    ms /= 3;
    const double per_simd = double(iters) * units * (threads / 256);
    std::printf("%-24s %d wavefronts per SIMD %7.2f cycles %6.0f TFLOP/s %5.2f GHz\n", name, threads / 256, n / per_simd,
                256. * (threads / 64) * iters * units * 32768 / (ms * 1e9), n / (ms * 1e6));
    std::fflush(stdout);
}
template <int... P>
static void all_groups(std::integer_sequence<int, P...>, int threads) {
    (time_it((std::to_string(kPatterns[P].shape) + " " + kPatterns[P].text).c_str(), groups<P>, threads, 8000,
             kGroups * count(kPatterns[P].text, 'M', length(kPatterns[P].text)) * kPatterns[P].shape / 32), ...);
}
int main() {
    std::mt19937 gen(1);
    std::normal_distribution<float> normal;
    std::vector<uint16_t> h((kA + kQ + kP) * 64 * 8);
    for (size_t i = 0; i < h.size(); ++i) {
        float x = normal(gen);
        if (i >= (kA + kQ) * 512) x = std::exp2(1.44f * x - 3.f);      // weights against a lazy reference
        uint32_t u;
        std::memcpy(&u, &x, 4);
        h[i] = (u + 0x7fff + ((u >> 16) & 1)) >> 16;
    }
    check(hipMalloc(&ops, h.size() * 2));
    check(hipMalloc(&sink, 256 * 512 * sizeof(float)));
    check(hipMalloc(&cycles, sizeof(uint64_t)));
    check(hipMemcpy(ops, h.data(), h.size() * 2, hipMemcpyHostToDevice));
    check(hipEventCreate(&e0));
    check(hipEventCreate(&e1));
    for (int rep = 0; rep < 2; ++rep) {
        time_it("both 32", products<kBoth32>, 512, 20000, 32);
        time_it("both 16, B kept", products<kBoth16B>, 512, 20000, 32);
        time_it("both 16, A kept", products<kBoth16A>, 512, 20000, 32);
        time_it("scores 32, as in a tile", products<kScores32Tile>, 512, 20000, 16);
        time_it("scores 32", products<kScores32>, 512, 20000, 32);
        time_it("P V 32", products<kPV32>, 512, 20000, 32);
        time_it("scores 32, from zero", products<kScores32Zero>, 512, 20000, 32);
        time_it("P V 32, from zero", products<kPV32Zero>, 512, 20000, 32);
    }
    for (int threads : {512, 256}) all_groups(std::make_integer_sequence<int, kNumPatterns>{}, threads);
    return 0;
}
