// Per-token symmetric INT8 activation quantization (Section 6.1 of arXiv 2405.04532; Eq. 1 in
// its symmetric form), with the per-token sums the per-channel GEMM epilogue needs
// (Section 5.2.2: sum of the quantized row for the exact zero-point fold of Eq. 6, and the
// sum of the unquantized row, t_X of Eq. 7).  Memory bound: 2 bytes read, 1 byte written per
// element.  One workgroup per token row.  Rows of up to 32768 elements are read once and held in
// registers between the absmax reduction and the rounding pass (all loads of a row are in flight
// together, which is what matters at decode sizes where the call is pure latency); longer rows
// are read twice (the second read hits cache).
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "qoq_internal.h"
#include "qoq_fp16.h"
#include "qoq_half_decide.h"
#include "qoq_act_codes.h"

namespace qoq {
namespace {

constexpr int kThreads = 256;

// ---- reductions over a wave without LDS traffic: four cross-lane (DPP) steps leave every row of 16 lanes with its
// own result, the four row results are read into scalar registers and combined there.
template <int CTRL>
__device__ __forceinline__ int dpp_i32(int v)
{
    return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xF, 0xF, false);
}
constexpr int kQuadSwap1 = 0xB1, kQuadSwap2 = 0x4E, kRowHalfMirror = 0x141, kRowMirror = 0x140;   // lanes ^1, ^2, 7-l, 15-l
__device__ __forceinline__ float wave_max_nonneg(float v)   // v >= 0: the bit patterns order like the values
{
    int b = __float_as_int(v);
    b = max(b, dpp_i32<kQuadSwap1>(b));
    b = max(b, dpp_i32<kQuadSwap2>(b));
    b = max(b, dpp_i32<kRowHalfMirror>(b));
    b = max(b, dpp_i32<kRowMirror>(b));
    const int r = max(max(__builtin_amdgcn_readlane(b, 0), __builtin_amdgcn_readlane(b, 16)),
                      max(__builtin_amdgcn_readlane(b, 32), __builtin_amdgcn_readlane(b, 48)));
    return __int_as_float(r);
}
__device__ __forceinline__ int wave_sum_i32(int v)
{
    v += dpp_i32<kQuadSwap1>(v);
    v += dpp_i32<kQuadSwap2>(v);
    v += dpp_i32<kRowHalfMirror>(v);
    v += dpp_i32<kRowMirror>(v);
    return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) + __builtin_amdgcn_readlane(v, 32) +
           __builtin_amdgcn_readlane(v, 48);
}
__device__ __forceinline__ float wave_sum_f32(float v)
{
    v += __int_as_float(dpp_i32<kQuadSwap1>(__float_as_int(v)));
    v += __int_as_float(dpp_i32<kQuadSwap2>(__float_as_int(v)));
    v += __int_as_float(dpp_i32<kRowHalfMirror>(__float_as_int(v)));
    v += __int_as_float(dpp_i32<kRowMirror>(__float_as_int(v)));
    return (__int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0)) + __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16))) +
           (__int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32)) + __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 48)));
}

__device__ __forceinline__ double row16_sum_f64(double v)     // over a row of 16 lanes; every lane has the sum
{
    auto moved = [](double d, auto ctrl) {
        const long long b = __double_as_longlong(d);
        const int lo = dpp_i32<decltype(ctrl)::value>((int)(b & 0xFFFFFFFFll)), hi = dpp_i32<decltype(ctrl)::value>((int)(b >> 32));
        return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
    };
    v += moved(v, std::integral_constant<int, kQuadSwap1>());
    v += moved(v, std::integral_constant<int, kQuadSwap2>());
    v += moved(v, std::integral_constant<int, kRowHalfMirror>());
    return v + moved(v, std::integral_constant<int, kRowMirror>());
}
__device__ __forceinline__ double wave_sum_f64(double v)
{
    v = row16_sum_f64(v);
    auto lane = [](double d, int l) {
        const long long b = __double_as_longlong(d);
        const int lo = __builtin_amdgcn_readlane((int)(b & 0xFFFFFFFFll), l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
        return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
    };
    return (lane(v, 0) + lane(v, 16)) + (lane(v, 32) + lane(v, 48));
}

__device__ inline float block_reduce_max(float v, float* smem)
{
    v = wave_max_nonneg(v);
    if ((threadIdx.x & 63) == 0) smem[threadIdx.x >> 6] = v;
    __syncthreads();
    float r = smem[0];
    for (int w = 1; w < kThreads / 64; ++w) r = fmaxf(r, smem[w]);
    __syncthreads();
    return r;
}

__global__ __launch_bounds__(kThreads) void act_quant_kernel(const __half* __restrict__ x, int64_t K,
                                                             int8_t* __restrict__ qx, __half* __restrict__ sx,
                                                             int32_t* __restrict__ rowsum, float* __restrict__ tx)
{
    __shared__ float s_f[kThreads / 64];
    __shared__ int s_i[kThreads / 64];
    const int64_t m = blockIdx.x;
    const uint4* row = reinterpret_cast<const uint4*>(x + m * K);  // 8 halves per 16 bytes
    const int64_t chunks = K / 8;

    float amax = 0.f;
    for (int64_t c = threadIdx.x; c < chunks; c += kThreads) {
        const uint4 v = row[c];
        const __half2* h = reinterpret_cast<const __half2*>(&v);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float2 f = __half22float2(h[j]);
            amax = fmaxf(amax, fmaxf(fabsf(f.x), fabsf(f.y)));
        }
    }
    amax = block_reduce_max(amax, s_f);

    const __half sxh = scale_of_row(amax);
    const float s = __half2float(sxh);
    const float inv_s = 1.0f / s;

    int isum = 0;
    float fsum = 0.f;
    uint2* qrow = reinterpret_cast<uint2*>(qx + m * K);
    for (int64_t c = threadIdx.x; c < chunks; c += kThreads) {
        const uint4 v = row[c];
        const __half2* h = reinterpret_cast<const __half2*>(&v);
        uint32_t packed[2] = {0u, 0u};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float2 f = __half22float2(h[j]);
            const int a = quantize_code(f.x, inv_s), b = quantize_code(f.y, inv_s);   // round half away from zero
            isum += a + b;
            fsum += f.x + f.y;
            packed[j >> 1] |= ((uint32_t)(a & 0xFF) << (16 * (j & 1))) | ((uint32_t)(b & 0xFF) << (16 * (j & 1) + 8));
        }
        qrow[c] = make_uint2(packed[0], packed[1]);
    }
    isum = wave_sum_i32(isum);
    fsum = wave_sum_f32(fsum);
    if ((threadIdx.x & 63) == 0) { s_i[threadIdx.x >> 6] = isum; s_f[threadIdx.x >> 6] = fsum; }
    __syncthreads();
    if (threadIdx.x == 0) {
        int it = 0; float ft = 0.f;
        for (int w = 0; w < kThreads / 64; ++w) { it += s_i[w]; ft += s_f[w]; }
        sx[m] = sxh;
        if (rowsum) rowsum[m] = it;
        if (tx) tx[m] = ft;
    }
}

// Single-read variant: up to 1024 threads, up to kCache 16-byte chunks (8 halves each) per thread in registers.
// row_threads() below says how many threads a row gets; the kernels take that number as an argument, which is there when they start
// (blockDim.x would have to be fetched).
constexpr int kWide = 1024;
constexpr int kCache = 4;
constexpr int64_t kMaxCachedK = 32768;

// A row (or one half of a gate/up row) read by 16-byte chunks; a chunk past the end reads as zeros without touching
// memory (the bounds check of the buffer load), so that no load sits under a condition and all of a thread's loads
// are in flight together.  base and bytes are the same for the whole workgroup.
struct RowReader {
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ __forceinline__ RowReader(const void* base, int bytes)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000)) {}
    __device__ __forceinline__ uint4 operator()(int chunk) const
    {
        return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, chunk * 16, 0, 0));
    }
};

// Quantize a token row that the workgroup holds in registers (chunk c = threadIdx.x + i * threads in v[i],
// zeros past the end): absmax, scale, INT8 codes, sums.  Used by the plain quantizer and by the producers the
// quantization is fused into.  These kernels are bound by vector instructions as much as by memory.
template <int CACHE>
__device__ inline void quantize_cached_row(const uint4 (&v)[CACHE], int chunks, int threads, int64_t m, int64_t K,
                                           int8_t* __restrict__ qx, __half* __restrict__ sx,
                                           int32_t* __restrict__ rowsum, float* __restrict__ tx, float* s_f, int* s_i)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = threads >> 6;
    h2 mx = half2_of(0u);
#pragma unroll
    for (int i = 0; i < CACHE; ++i) mx = max_of_chunk(v[i], mx);
    float amax = wave_max_nonneg(fmaxf((float)mx.x, (float)mx.y));
    if (lane == 0) s_f[wave] = amax;
    __syncthreads();
    amax = wave_max_nonneg(lane < waves ? s_f[lane] : 0.f);

    const __half sxh = scale_of_row(amax);
    const float s = __half2float(sxh);
    const float inv_s = 1.0f / s;

    int isum = 0;
    uint2* qrow = reinterpret_cast<uint2*>(qx + m * K);
    if (__builtin_amdgcn_readfirstlane(__float_as_int(s)) >= __float_as_int(0x1p-14f)) {
        const float push = inv_s * (1.0f + 0x1p-20f);
#pragma unroll
        for (int i = 0; i < CACHE; ++i) {
            const int c = (int)threadIdx.x + i * threads;
            if (c < chunks) qrow[c] = codes_of_chunk(v[i], push, isum);
        }
    } else {
#pragma unroll 1
        for (int i = 0; i < CACHE; ++i) {
            const int c = (int)threadIdx.x + i * threads;
            uint4 vi = v[0];
#pragma unroll
            for (int x = 1; x < CACHE; ++x)            // (selects: an indexed register array would go to scratch memory)
                if (i == x) vi = v[x];
            if (c < chunks) qrow[c] = codes_of_chunk_clamped(vi, inv_s, isum);
        }
    }
    if (!rowsum && !tx) {                          // group mode needs neither sum: no second reduction
        if (threadIdx.x == 0) sx[m] = sxh;
        return;
    }
    float fsum = 0.f;
    if (tx) {
#pragma unroll
        for (int i = 0; i < CACHE; ++i) {
            const uint32_t w[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) fsum += (float)half2_of(w[j]).x + (float)half2_of(w[j]).y;
        }
    }
    isum = wave_sum_i32(isum);
    fsum = wave_sum_f32(fsum);
    __syncthreads();                               // s_f holds the maxima until here
    if (lane == 0) { s_i[wave] = isum; s_f[wave] = fsum; }
    __syncthreads();
    if (threadIdx.x == 0) {
        int it = 0; float ft = 0.f;
        for (int w = 0; w < waves; ++w) { it += s_i[w]; ft += s_f[w]; }
        sx[m] = sxh;
        if (rowsum) rowsum[m] = it;
        if (tx) tx[m] = ft;
    }
}

template <int CACHE>
__global__ __launch_bounds__(kWide) void act_quant_cached_kernel(const __half* __restrict__ x, int K, int threads,
                                                                 int8_t* __restrict__ qx, __half* __restrict__ sx,
                                                                 int32_t* __restrict__ rowsum, float* __restrict__ tx)
{
    __shared__ float s_f[kWide / 64];
    __shared__ int s_i[kWide / 64];
    const int64_t m = blockIdx.x;
    const RowReader row(x + m * K, K * 2);
    uint4 v[CACHE];
#pragma unroll
    for (int i = 0; i < CACHE; ++i) v[i] = row((int)threadIdx.x + i * threads);
    quantize_cached_row(v, K / 8, threads, m, K, qx, sx, rowsum, tx, s_f, s_i);
}

// The same with the input channels taken in a new order (activation-aware channel reordering, Section 4.3):
// qx[m, j] = quantize(x[m, perm[j]]).  The row is copied to LDS in whole lines and gathered there (fetched from memory
// two bytes at a time, a gather is a cache request per element); the per-token scale does not depend on the order.
// Indices are clamped to the row.  LDS: the row, then the two arrays of the reduction.
template <int CACHE>
__global__ __launch_bounds__(kWide) void act_quant_reordered_kernel(const __half* __restrict__ x, const int32_t* __restrict__ perm,
                                                                    int K, int threads, int8_t* __restrict__ qx, __half* __restrict__ sx,
                                                                    int32_t* __restrict__ rowsum, float* __restrict__ tx)
{
    extern __shared__ __attribute__((aligned(16))) char s_mem[];
    uint4* s_row = reinterpret_cast<uint4*>(s_mem);
    float* s_f = reinterpret_cast<float*>(s_mem + K * 2);
    int* s_i = reinterpret_cast<int*>(s_f + kWide / 64);
    const int64_t m = blockIdx.x;
    const RowReader row(x + m * K, K * 2), order(perm, K * 4);
    const int chunks = K / 8, last = K - 1;
    uint4 v[CACHE], p[2 * CACHE];
#pragma unroll
    for (int i = 0; i < CACHE; ++i) v[i] = row((int)threadIdx.x + i * threads);
#pragma unroll
    for (int i = 0; i < 2 * CACHE; ++i) p[i] = order(2 * ((int)threadIdx.x + (i >> 1) * threads) + (i & 1));
#pragma unroll
    for (int i = 0; i < CACHE; ++i) {
        const int c = (int)threadIdx.x + i * threads;
        if (c < chunks) s_row[c] = v[i];
    }
    __syncthreads();
    const unsigned short* s_half = reinterpret_cast<const unsigned short*>(s_mem);
#pragma unroll
    for (int i = 0; i < CACHE; ++i) {
        const int c = (int)threadIdx.x + i * threads;
        if (c < chunks) {
            const uint32_t idx[8] = {p[2 * i].x, p[2 * i].y, p[2 * i].z, p[2 * i].w,
                                     p[2 * i + 1].x, p[2 * i + 1].y, p[2 * i + 1].z, p[2 * i + 1].w};
            uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int j = 0; j < 8; ++j)
                w[j >> 1] |= (uint32_t)s_half[min(max((int)idx[j], 0), last)] << (16 * (j & 1));
            v[i] = make_uint4(w[0], w[1], w[2], w[3]);
        }
    }
    quantize_cached_row(v, chunks, threads, m, K, qx, sx, rowsum, tx, s_f, s_i);
}

// ---- producers with the quantization fused in (Section 5.1: the activations are quantized inside the
// normalisation in front of the QKV / first FFN projection and inside the activation function in front of the
// second FFN projection).  The producer is evaluated in FP64 and rounded once to FP16 (the exact bit routine
// below), which defines the tensor an unfused pipeline would hand to the quantizer; the codes are then decided
// from that FP16 value exactly as in the stand-alone kernel.
__device__ inline void unpack8(const uint4& v, double (&f)[8])
{
    const __half* h = reinterpret_cast<const __half*>(&v);
#pragma unroll
    for (int j = 0; j < 8; ++j) f[j] = (double)__half2float(h[j]);
}

// The machine operations behind the FP32 decision routines of qoq_half_decide.h.  keep(): an empty asm on the value,
// which keeps the compiler from merging an FP32 product with a conversion next to it (of an FP16 factor, or of the
// product to FP16) into one mixed-precision multiply-add with a zero addend: that turns a product of -0 into +0.
struct DevF32 {
    static __device__ __forceinline__ uint32_t bits(float x) { return __float_as_uint(x); }
    static __device__ __forceinline__ float from_bits(uint32_t u) { return __uint_as_float(u); }
    static __device__ __forceinline__ uint32_t half_bits(float x) { return (uint32_t)__half_as_ushort(__float2half_rn(x)); }
    static __device__ __forceinline__ uint32_t half2_bits(float a, float b)      // one conversion instruction for both
    {
        typedef float f2 __attribute__((ext_vector_type(2)));
        return __builtin_bit_cast(uint32_t, __builtin_convertvector((f2){a, b}, h2));
    }
    static __device__ __forceinline__ float keep(float x)
    {
        asm volatile("" : "+v"(x));
        return x;
    }
};
__device__ __forceinline__ float opaque(float x) { return DevF32::keep(x); }

// The product of two FP16 numbers (element e of words a and b), exact in FP32 (22 bits), in one mixed-precision
// multiply-add.  Its addend is -0, which leaves a product of -0 as it is, in a register the compiler cannot see through.
__device__ __forceinline__ float exact_product(uint32_t a, uint32_t b, int e, float minus_zero)
{
    return fmaf((float)half2_of(a)[e], (float)half2_of(b)[e], minus_zero);
}

// Element idx (chunk idx / 8, half idx % 8) of the cached chunks := bits.  Written as compile-time indexed selects: a
// register array indexed at run time would be moved to scratch memory.  Chunks that no lane of the wave changes are skipped.
template <int CACHE>
__device__ __forceinline__ void patch_half(uint4 (&v)[CACHE], int idx, uint32_t bits)
{
#pragma unroll
    for (int i = 0; i < CACHE; ++i) {
        if (__builtin_amdgcn_ballot_w64((idx >> 3) == i) == 0) continue;
        uint32_t w[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (idx == i * 8 + j) w[j >> 1] = (w[j >> 1] & ~(0xFFFFu << (16 * (j & 1)))) | (bits << (16 * (j & 1)));
        v[i] = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// gate / (1 + exp(-gate)) in FP64 for the elements FP32 could not decide.  exp by its definition: -gate = n ln2 + r
// with |r| <= ln2 / 2 (ln2 split so that n * ln2_hi is exact for |n| < 2^20), the Taylor series of exp(r) to the
// term r^13 / 13! (the next one is below 2^-55) and a scaling by 2^n that saturates to 0 or infinity.  Within 2^-49
// of the true value, which rounds to the same FP16 number unless the value lies that close to a midpoint.  One
// FP64 instruction occupies the SIMD for 8 cycles whatever the number of active lanes, so the length of this
// routine (about 40 of them, against several hundred in a general-purpose exp and division) is what the rare path costs.
__device__ __forceinline__ double silu_f64(double g)
{
    const double z = fmin(fmax(-g, -1000.0), 1000.0);  // beyond +-745 exp is 0 or infinite anyway; keeps n small for +-inf and NaN
    const double nf = rint(z * 1.4426950408889634074);
    const double r = fma(-nf, 1.9082149292705877e-10, fma(-nf, 6.93147180369123816490e-01, z));
    double e = 1.0 / 6227020800.0;
    e = fma(e, r, 1.0 / 479001600.0);
    e = fma(e, r, 1.0 / 39916800.0);
    e = fma(e, r, 1.0 / 3628800.0);
    e = fma(e, r, 1.0 / 362880.0);
    e = fma(e, r, 1.0 / 40320.0);
    e = fma(e, r, 1.0 / 5040.0);
    e = fma(e, r, 1.0 / 720.0);
    e = fma(e, r, 1.0 / 120.0);
    e = fma(e, r, 1.0 / 24.0);
    e = fma(e, r, 1.0 / 6.0);
    e = fma(e, r, 0.5);
    e = fma(e, r, 1.0);
    e = fma(e, r, 1.0);
    e = ldexp(e, (int)nf);                             // 2^n over- and underflows as exp does
    return g / (1.0 + e);
}

// The two producers are bound by vector issue where there are rows enough (a compute unit issues 64 lanes of one instruction
// per clock), which is why every step of theirs is counted in instructions: exact products in one multiply-add, both bounds
// in one conversion each, two instructions per code.  Before (58 instructions per element, now about half) and now, in us:
// RMSNorm 2048 x 8192 21.4 -> 14.3, 4096 x 11008 60 -> 38, 64 x 4096 4.4 -> 3.4; SiLU.up 2048 x 28672 80 -> 58 (5.0 TB/s, a
// copy 4.9), 4096 x 11008 65 -> 46, 64 x 11008 7.9 -> 5.9, 37 x 28672 15.5 -> 9.8; the plain quantizer 4096 x 11008
// 25.1 -> 23.8 (5.7 TB/s); reordered 4096 x 11008 74 -> 31, 389 x 11008 11.4 -> 6.1.
// y = x * (1 / sqrt(mean(x^2) + eps)) * gamma
template <int CACHE>
__global__ __launch_bounds__(kWide) void rmsnorm_quant_kernel(const __half* __restrict__ x, const __half* __restrict__ gamma,
                                                              int K, int threads, double eps, double inv_K, int8_t* __restrict__ qx,
                                                              __half* __restrict__ sx, __half* __restrict__ y,
                                                              int32_t* __restrict__ rowsum, float* __restrict__ tx)
{
    __shared__ float s_f[kWide / 64];
    __shared__ int s_i[kWide / 64];
    __shared__ double s_d[kWide / 64];
    const int64_t m = blockIdx.x;
    const RowReader row(x + m * K, K * 2), grow(gamma, K * 2);
    const int chunks = K / 8;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = threads >> 6;
    uint4 v[CACHE], gv[CACHE];                         // the weights are fetched with the row, not after the reduction
    double ss = 0.0, ss1 = 0.0;
#pragma unroll
    for (int i = 0; i < CACHE; ++i) v[i] = row((int)threadIdx.x + i * threads);
#pragma unroll
    for (int i = 0; i < CACHE; ++i) gv[i] = grow((int)threadIdx.x + i * threads);
#pragma unroll
    for (int i = 0; i < CACHE; ++i) {
        double f[8];
        unpack8(v[i], f);
#pragma unroll
        for (int j = 0; j < 8; j += 2) { ss = fma(f[j], f[j], ss); ss1 = fma(f[j + 1], f[j + 1], ss1); }
    }
    ss = wave_sum_f64(ss + ss1);
    if (lane == 0) s_d[wave] = ss;
    __syncthreads();
    ss = row16_sum_f64((lane & 15) < waves ? s_d[lane & 15] : 0.0);
    // 1 / sqrt(mean + eps) to 2^-48 (the FP32 reciprocal root and one step of third order): the compensated decision
    // below needs 2^-40.  The definition's own division and root, 80 FP64 instructions per wave, are left to the
    // elements that go to FP64 and to means outside the FP32 range.
    const double ms = fma(ss, inv_K, eps);
    double inv = (double)__builtin_amdgcn_rsqf((float)ms);
    const double off = fma(-ms * inv, inv, 1.0);
    inv = fma(inv * off, fma(off, 0.375, 0.5), inv);
    if (!(ms > 1e-30 && ms < 1e30)) inv = 1.0 / sqrt(ss / (double)K + eps);
    const float inv32 = (float)inv, inv_lo = (float)(inv - (double)inv32);   // inv = inv32 + inv_lo to 2^-48
    const float below = (float)(inv * (1.0 - 1.5 * 0x1p-23)), above = (float)(inv * (1.0 + 1.5 * 0x1p-23));
    const float minus_zero = opaque(-0.0f);
    uint64_t risky = 0;                                // elements to redo in FP64, bit = chunk * 8 + half
#pragma unroll
    for (int i = 0; i < CACHE; ++i) {
        const int c = (int)threadIdx.x + i * threads;
        if (c < chunks) {
            const __half* hx = reinterpret_cast<const __half*>(&v[i]);
            const __half* hg = reinterpret_cast<const __half*>(&gv[i]);
            const uint32_t xw[4] = {v[i].x, v[i].y, v[i].z, v[i].w}, gw[4] = {gv[i].x, gv[i].y, gv[i].z, gv[i].w};
            uint32_t w[4], diff[4];
            // FP32 first: x * gamma is exact (22 bits), the factors and their products with it round once each, so the
            // two products enclose the FP64 value with factors 1 -+ 1.5 * 2^-23 (relative) of the reciprocal root
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float p0 = exact_product(xw[j], gw[j], 0, minus_zero), p1 = exact_product(xw[j], gw[j], 1, minus_zero);
                diff[j] = half2_bits_between<DevF32>(p0 * below, p0 * above, p1 * below, p1 * above, w[j]);
            }
            if (diff[0] | diff[1] | diff[2] | diff[3]) {   // every sixth wave and chunk has such an element
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    if ((diff[j >> 1] >> (16 * (j & 1))) & 0xFFFFu) {
                        // next to a rounding midpoint: the same product with its rounding errors carried along
                        float hi, lo;
                        scaled_product_pair<DevF32>(__half2float(hx[j]), inv32, inv_lo, __half2float(hg[j]), hi, lo);
                        uint32_t b = 0;
                        if (!half_bits_from_pair<DevF32>(hi, lo, b)) risky |= 1ull << (i * 8 + j);
                        w[j >> 1] = (w[j >> 1] & ~(0xFFFFu << (16 * (j & 1)))) | (b << (16 * (j & 1)));
                    }
                }
            }
            v[i] = make_uint4(w[0], w[1], w[2], w[3]);
        }
    }
    // what is left (overflow range, values within 2^-36 of a midpoint): FP64, one at a time
    while (risky) {
        const int idx = __ffsll((unsigned long long)risky) - 1;
        risky &= risky - 1;
        const int64_t k = ((int64_t)threadIdx.x + (int64_t)(idx >> 3) * (int64_t)threads) * 8 + (idx & 7);
        const double fx = (double)__half2float(x[m * K + k]), fg = (double)__half2float(gamma[k]);
        patch_half(v, idx, (uint32_t)double_to_half_rne(fx * (1.0 / sqrt(ss / (double)K + eps)) * fg));
    }
    if (y) {
#pragma unroll
        for (int i = 0; i < CACHE; ++i) {
            const int c = (int)threadIdx.x + i * threads;
            if (c < chunks) reinterpret_cast<uint4*>(y + m * K)[c] = v[i];
        }
    }
    quantize_cached_row(v, chunks, threads, m, K, qx, sx, rowsum, tx, s_f, s_i);
}

// 1 / (1 + exp(-g)) in FP32 from the hardware exponential (base 2) and reciprocal, one unit in the last place each:
// the part of g log2(e) that the rounded product loses enters as a factor (1 + rest ln 2).  Errors in units of 2^-23
// (relative): exponential 1, factor and product 1/2 each, addition 1/2, reciprocal 1: 3.5; the product with the exact
// gate * up adds 1/2, and the caller's bounds of 5 units contain their own rounding.  exp(-g) is 0 above g = 100 (where
// 1 + exp(-g) = 1 long before) and infinite below -89: the result is then 1 or 0, and NaN for g = -infinity as in FP64.
__device__ __forceinline__ float sigmoid_f32(float g)
{
    constexpr float kHi = 1.4426950408889634f, kLo = (float)(1.4426950408889634074 - (double)kHi);
    const float z = fmaxf(-g, -100.0f), t = z * kHi;
    const float rest = fmaf(z, kLo, fmaf(z, kHi, -t));
    return __builtin_amdgcn_rcpf(fmaf(__builtin_amdgcn_exp2f(t), fmaf(rest, 0.69314718055994531f, 1.0f), 1.0f));
}

// gate_up [M, 2K]: y = gate / (1 + exp(-gate)) * up with gate = first K columns, up = last K
template <int CACHE>
__global__ __launch_bounds__(kWide) void silu_mul_quant_kernel(const __half* __restrict__ gate_up, int K, int threads,
                                                               __half* __restrict__ y, int8_t* __restrict__ qx,
                                                               __half* __restrict__ sx, int32_t* __restrict__ rowsum,
                                                               float* __restrict__ tx)
{
    __shared__ float s_f[kWide / 64];
    __shared__ int s_i[kWide / 64];
    const int64_t m = blockIdx.x;
    const RowReader grow(gate_up + m * 2 * K, K * 2), urow(gate_up + m * 2 * K + K, K * 2);
    const int chunks = K / 8, wave_first = __builtin_amdgcn_readfirstlane(threadIdx.x & ~63u);
    constexpr int kAhead = CACHE < 2 ? CACHE : 2;      // chunks in flight
    uint4 v[CACHE], gb[kAhead], ub[kAhead];
    const float minus_zero = opaque(-0.0f);
    uint64_t risky = 0;                                // elements to redo in FP64, bit = chunk * 8 + half
    uint32_t first = 0;                                // gate and up of the first of them
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
        gb[i] = grow((int)threadIdx.x + i * threads);
        ub[i] = urow((int)threadIdx.x + i * threads);
    }
#pragma unroll
    for (int i = 0; i < CACHE; ++i) {
        const uint4 gv = gb[i % kAhead], uv = ub[i % kAhead];
        if (i + kAhead < CACHE) {
            gb[i % kAhead] = grow((int)threadIdx.x + (i + kAhead) * threads);
            ub[i % kAhead] = urow((int)threadIdx.x + (i + kAhead) * threads);
        }
        v[i] = make_uint4(0u, 0u, 0u, 0u);
        if (wave_first + i * threads < chunks) {   // (whole waves past the end of the row have nothing to do)
            const uint32_t g4[4] = {gv.x, gv.y, gv.z, gv.w}, u4[4] = {uv.x, uv.y, uv.z, uv.w};
            uint32_t w[4], diff[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const h2 hg = half2_of(g4[j]);
                const float p0 = exact_product(g4[j], u4[j], 0, minus_zero) * sigmoid_f32((float)hg.x);
                const float p1 = exact_product(g4[j], u4[j], 1, minus_zero) * sigmoid_f32((float)hg.y);
                diff[j] = half2_bits_from_bounds<DevF32>(p0, p1, 1.0f - 5 * 0x1p-23f, 1.0f + 5 * 0x1p-23f, w[j]);
            }
            if (diff[0] | diff[1] | diff[2] | diff[3]) {
#pragma unroll
                for (int j = 7; j >= 0; --j)
                    if ((diff[j >> 1] >> (16 * (j & 1))) & 0xFFFFu) {
                        if ((risky & ((1ull << (i * 8)) - 1)) == 0)
                            first = __builtin_amdgcn_perm(u4[j >> 1], g4[j >> 1], j & 1 ? 0x07060302u : 0x05040100u);
                        risky |= 1ull << (i * 8 + j);
                    }
            }
            v[i] = make_uint4(w[0], w[1], w[2], w[3]);
        }
    }
    // the few elements (about 1 in 700) whose FP32 value is too close to a rounding midpoint: FP64, one at a time; the
    // lane's first one comes from a register, further ones are fetched again
    for (bool again = false; risky; again = true) {
        const int idx = __ffsll((unsigned long long)risky) - 1;
        risky &= risky - 1;
        if (again) {
            const int64_t k = ((int64_t)threadIdx.x + (int64_t)(idx >> 3) * (int64_t)threads) * 8 + (idx & 7);
            const unsigned short* row = reinterpret_cast<const unsigned short*>(gate_up + m * 2 * K);
            first = (uint32_t)row[k] | ((uint32_t)row[K + k] << 16);
        }
        const double dg = (double)(float)half2_of(first).x, du = (double)(float)half2_of(first).y;
        patch_half(v, idx, (uint32_t)double_to_half_rne(silu_f64(dg) * du));
    }
    if (y) {
#pragma unroll
        for (int i = 0; i < CACHE; ++i) {
            const int c = (int)threadIdx.x + i * threads;
            if (c < chunks) reinterpret_cast<uint4*>(y + m * K)[c] = v[i];
        }
    }
    quantize_cached_row(v, chunks, threads, m, K, qx, sx, rowsum, tx, s_f, s_i);
}

}  // namespace

// Threads per token row: at most four cached chunks (16 bytes) each.  With many rows, 256 threads keep more rows in flight
// per compute unit and repeat the per-row work (reductions, scale) in fewer waves (RMSNorm 4096 x 4096: 14.7 us with 256, 21
// with 512; 1024 x 4096: 7.4 and 8.4; quantizer 4096 x 4096 9.9 and 10.5); with few, a row's own time counts and 256 is
// slower (64 x 4096 SiLU.up 4.3 us against 3.7).  few_rows_wide: 1024 threads for long rows where the chip has room for them
// and the work per element is long (SiLU.up 64 x 11008 6.0 us with 1024, 6.5 with 512; the others are no faster).  Rows of up to
// 512 elements are one chunk for each lane of one wave, which then has no other to wait for (quantizer with sums 4096 x 512
// 3.7 us with 64 threads, 6.0 with 256, 4096 x 128 3.6 and 5.9).
static int64_t row_threads(int64_t M, int64_t K, bool few_rows_wide = false)
{
    if (K <= 512) return 64;
    if (M >= 1024 && K <= (int64_t)256 * kCache * 8) return 256;
    if (M <= 512 && K > (int64_t)8192 && few_rows_wide) return kWide;
    return K <= (int64_t)512 * kCache * 8 ? 512 : kWide;
}

// the kernel with as many cached 16-byte chunks per thread as the row needs: short rows spend no registers on empty ones
#define QOQ_BY_CHUNKS(kernel, wide, K)                                                                                  \
    ((K) <= (wide) * 8 ? kernel<1> : (K) <= (wide) * 2 * 8 ? kernel<2> : kernel<kCache>)

hipError_t launch_act_quant(const void* x_fp16, int64_t M, int64_t K, int8_t* qx, void* sx, int32_t* rowsum,
                            float* tx, hipStream_t s)
{
    if (M == 0) return hipSuccess;
    if (K <= kMaxCachedK) {
        const int64_t wide = row_threads(M, K);
        auto* kern = QOQ_BY_CHUNKS(act_quant_cached_kernel, wide, K);
        kern<<<dim3((unsigned)M), (unsigned)wide, 0, s>>>(static_cast<const __half*>(x_fp16), (int)K, (int)wide, qx, static_cast<__half*>(sx), rowsum, tx);
        return hipGetLastError();
    }
    act_quant_kernel<<<dim3((unsigned)M), kThreads, 0, s>>>(static_cast<const __half*>(x_fp16), K, qx,
                                                           static_cast<__half*>(sx), rowsum, tx);
    return hipGetLastError();
}

hipError_t launch_act_quant_reordered(const void* x_fp16, const int32_t* perm, int64_t M, int64_t K, int8_t* qx, void* sx,
                                      int32_t* rowsum, float* tx, hipStream_t s)
{
    if (M == 0) return hipSuccess;
    if (K > kMaxCachedK) return hipErrorInvalidValue;
    const int64_t wide = row_threads(M, K);
    auto* kern = QOQ_BY_CHUNKS(act_quant_reordered_kernel, wide, K);
    const unsigned lds = (unsigned)(K * 2 + (kWide / 64) * (sizeof(float) + sizeof(int)));
    kern<<<dim3((unsigned)M), (unsigned)wide, lds, s>>>(static_cast<const __half*>(x_fp16), perm, (int)K, (int)wide, qx, static_cast<__half*>(sx),
                                                        rowsum, tx);
    return hipGetLastError();
}

int64_t fused_quant_max_k() { return kMaxCachedK; }

hipError_t launch_rmsnorm_quant(const void* x_fp16, const void* gamma_fp16, double eps, int64_t M, int64_t K, void* y_fp16,
                                int8_t* qx, void* sx, int32_t* rowsum, float* tx, hipStream_t s)
{
    if (M == 0) return hipSuccess;
    const int64_t wide = row_threads(M, K);
    auto* kern = QOQ_BY_CHUNKS(rmsnorm_quant_kernel, wide, K);
    kern<<<dim3((unsigned)M), (unsigned)wide, 0, s>>>(static_cast<const __half*>(x_fp16), static_cast<const __half*>(gamma_fp16), (int)K, (int)wide,
                                            eps, 1.0 / (double)K, qx, static_cast<__half*>(sx), static_cast<__half*>(y_fp16), rowsum, tx);
    return hipGetLastError();
}

hipError_t launch_silu_mul_quant(const void* gate_up_fp16, int64_t M, int64_t K, void* y_fp16, int8_t* qx, void* sx,
                                 int32_t* rowsum, float* tx, hipStream_t s)
{
    if (M == 0) return hipSuccess;
    const int64_t wide = row_threads(M, K, true);
    auto* kern = QOQ_BY_CHUNKS(silu_mul_quant_kernel, wide, K);
    kern<<<dim3((unsigned)M), (unsigned)wide, 0, s>>>(static_cast<const __half*>(gate_up_fp16), (int)K, (int)wide, static_cast<__half*>(y_fp16), qx,
                                            static_cast<__half*>(sx), rowsum, tx);
    return hipGetLastError();
}

#undef QOQ_BY_CHUNKS

}  // namespace qoq
