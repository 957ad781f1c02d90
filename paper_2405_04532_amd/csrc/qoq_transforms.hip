// Data-free offline transforms of QoQ for gfx950 (Section 4.3 of arXiv 2405.04532): channel salience and
// channel gather for the activation-aware reordering, scaled-Hadamard rotation of block-input tensors.
// These run when a model is prepared, not in the serving loop (at run time the reordering is the gather fused
// into the activation quantizer, qoq_act.hip, and the rotation is folded into the preceding layer's weights),
// so they are written for exactness first: the rotation sums in FP64, where sums of FP16 numbers are exact for
// these sizes, and rounds once to FP16.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <numeric>
#include <vector>

#include "qoq_fp16.h"
#include "qoq_internal.h"

namespace qoq {
namespace {

constexpr int kRowsPerSlab = 64;

// salience[k] = max_m |x[m, k]| (Section 4.3: the magnitude of the input activations decides a channel's
// salience).  One thread per 8 channels and slab of rows; non-negative floats order like their bit patterns,
// so the slabs meet with an integer atomic maximum on a zero-filled array.
__global__ __launch_bounds__(256) void channel_absmax_kernel(const __half* __restrict__ x, int64_t M, int64_t K, int* __restrict__ out_bits)
{
    const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (c >= K / 8) return;
    const int64_t r0 = (int64_t)blockIdx.y * kRowsPerSlab, r1 = min(M, r0 + kRowsPerSlab);
    float mx[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int64_t r = r0; r < r1; ++r) {
        const uint4 v = reinterpret_cast<const uint4*>(x + r * K)[c];
        const __half* h = reinterpret_cast<const __half*>(&v);
#pragma unroll
        for (int j = 0; j < 8; ++j) mx[j] = fmaxf(mx[j], fabsf(__half2float(h[j])));
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) atomicMax(out_bits + c * 8 + j, __float_as_int(mx[j]));
}

// dst[r, j] = src[r, perm[j]]; one thread per 8 output channels.  Indices are clamped to the row.
__global__ __launch_bounds__(256) void gather_channels_kernel(const __half* __restrict__ src, const int32_t* __restrict__ perm,
                                                              int64_t rows, int64_t K, __half* __restrict__ dst)
{
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t chunks = K / 8;
    if (idx >= rows * chunks) return;
    const int64_t r = idx / chunks, c = idx % chunks;
    const unsigned short* row = reinterpret_cast<const unsigned short*>(src + r * K);
    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int p = min(max(perm[c * 8 + j], 0), (int)K - 1);
        w[j >> 1] |= (uint32_t)row[p] << (16 * (j & 1));
    }
    reinterpret_cast<uint4*>(dst + r * K)[c] = make_uint4(w[0], w[1], w[2], w[3]);
}

// dst[r, b*n .. b*n+n) = src[r, b*n .. b*n+n) H_n * scale, H_n the Sylvester Hadamard matrix (entry (i, j) =
// (-1)^popcount(i & j)), by the in-place butterfly: log2(n) stages of n/2 additions and subtractions.
// FP64 throughout: every partial sum of at most 8192 FP16 numbers is a multiple of 2^-24 below 2^29 and therefore
// exact, so the result is the exact product times `scale`, rounded once, whatever the order of the stages.
constexpr int kMaxHadamard = 8192;

// FP64 -> FP16, round to nearest even, for results that are zero or of at least 2^-126: the fraction bits below
// FP32's last one are folded into it (round to odd), which makes the conversion to FP32 exact and leaves the one to
// FP16 everything it needs to decide as if it saw the FP64 value (FP32 has two bits more than FP16 needs for that).
__device__ __forceinline__ unsigned short half_rne_by_odd(double d)
{
    const unsigned long long u = (unsigned long long)__double_as_longlong(d);
    const uint32_t lo = (uint32_t)u;
    const uint32_t odd = (min(lo & 0x1FFFFFFFu, 1u) << 29) | (lo & 0xE0000000u);
    const double r = __longlong_as_double((long long)((u & 0xFFFFFFFF00000000ull) | odd));
    float f = (float)r;
    asm("" : "+v"(f));                                   // or the compiler merges the two conversions into a long FP64 one
    return __half_as_ushort(__float2half_rn(f));
}

// Blocks of rows * K contiguous elements are cut into segments of 2048 * CH elements, one workgroup of 256 threads each
// (a segment holds whole blocks; CH = 4 only for n = 8192).  A thread keeps 8 * CH elements in registers and takes the
// stages in three layouts, with two exchanges through LDS instead of one per stage:
//     A  16-byte chunks as they are loaded: element bits 0..2, and 11.. (chunks 256 apart)
//     B  element bits 3..6 in registers
//     C  element bits 7..10 in registers
// and the FP16 results go back to chunk order through LDS for 16-byte stores.  A single workgroup with one LDS round
// trip and one barrier per stage (twelve of them at n = 4096) was bound by LDS and barriers: 22016 x 4096 in 863 us,
// 0.42 TB/s; this one takes 111 us, 3.2 TB/s (a copy of the tensor 67 us), bound by vector issue (FP64 additions,
// conversions) together with its LDS traffic of 36 bytes per element.  LDS position of element i: 8 bytes of padding per 8 elements and 64 more per 128, which spreads all
// three access patterns evenly over the 64 banks.
template <int CH>
__global__ __launch_bounds__(256) void hadamard_kernel(const uint4* __restrict__ src, int64_t chunks, int n, double scale,
                                                       uint4* __restrict__ dst)
{
    constexpr int kElems = 2048 * CH;
    auto pos = [](int i) { return i + (i >> 3) + ((i >> 7) << 3); };
    __shared__ double buf[kElems + kElems / 8 + kElems / 16];
    const int t = threadIdx.x;
    const int64_t c0 = (int64_t)blockIdx.x * (256 * CH);
    double v[CH][8];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int64_t at = c0 + c * 256 + t;
        const uint4 raw = at < chunks ? src[at] : make_uint4(0u, 0u, 0u, 0u);
        const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
        for (int e = 0; e < 8; ++e)
            v[c][e] = (double)__half2float(__ushort_as_half((unsigned short)(w[e >> 1] >> (16 * (e & 1)))));
    }
    auto butterfly = [](double& a, double& b) { const double s = a + b; b = a - b; a = s; };
    // ---- A
#pragma unroll
    for (int h = 1; h < 8; h <<= 1)
        if (h < n)
#pragma unroll
            for (int c = 0; c < CH; ++c)
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (!(e & h)) butterfly(v[c][e], v[c][e | h]);
#pragma unroll
    for (int h = 1; h < CH; h <<= 1)
        if (2048 * h < n)
#pragma unroll
            for (int c = 0; c < CH; ++c)
                if (!(c & h))
#pragma unroll
                    for (int e = 0; e < 8; ++e) butterfly(v[c][e], v[c | h][e]);
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
        for (int e = 0; e < 8; ++e) buf[pos((c * 256 + t) * 8 + e)] = v[c][e];
    __syncthreads();
    // ---- B and C: sixteen elements at a time, `step` elements apart, from element `first` on
    auto stages16 = [&](int first, int step) __attribute__((always_inline)) {
        double x[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) x[j] = buf[pos(first + j * step)];
#pragma unroll
        for (int h = 1; h < 16; h <<= 1)
            if (h * step < n)
#pragma unroll
                for (int j = 0; j < 16; ++j)
                    if (!(j & h)) butterfly(x[j], x[j | h]);
#pragma unroll
        for (int j = 0; j < 16; ++j) v[j >> 3][j & 7] = x[j];
    };
#pragma unroll
    for (int s = 0; s < CH / 2; ++s) {
        const int first = (t & 7) + (t >> 3) * 128 + s * 4096;
        stages16(first, 8);
#pragma unroll
        for (int j = 0; j < 16; ++j) buf[pos(first + j * 8)] = v[j >> 3][j & 7];
    }
    __syncthreads();
    unsigned short r[CH / 2][16];
#pragma unroll
    for (int s = 0; s < CH / 2; ++s) {
        stages16((t & 127) + (t >> 7) * 2048 + s * 4096, 128);
#pragma unroll
        for (int j = 0; j < 16; ++j) r[s][j] = half_rne_by_odd(v[j >> 3][j & 7] * scale);
    }
    __syncthreads();                                     // everybody has read: the buffer takes the results
    unsigned short* out = reinterpret_cast<unsigned short*>(buf);
#pragma unroll
    for (int s = 0; s < CH / 2; ++s)
#pragma unroll
        for (int j = 0; j < 16; ++j) out[(t & 127) + (t >> 7) * 2048 + s * 4096 + j * 128] = r[s][j];
    __syncthreads();
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int64_t at = c0 + c * 256 + t;
        if (at < chunks) dst[at] = reinterpret_cast<const uint4*>(buf)[c * 256 + t];
    }
}

// The same for tensors that are no whole number of 16-byte chunks or not aligned to them: one workgroup per (row, block).
__global__ __launch_bounds__(256) void hadamard_unaligned_kernel(const __half* __restrict__ src, int64_t K, int n, double scale,
                                                                 __half* __restrict__ dst)
{
    __shared__ double buf[kMaxHadamard];
    const int64_t base = (int64_t)blockIdx.y * K + (int64_t)blockIdx.x * n;
    for (int i = threadIdx.x; i < n; i += 256) buf[i] = (double)__half2float(src[base + i]);
    __syncthreads();
    for (int h = 1; h < n; h <<= 1) {
        for (int t = threadIdx.x; t < n / 2; t += 256) {
            const int i = (t / h) * 2 * h + (t % h);
            const double a = buf[i], b = buf[i + h];
            buf[i] = a + b;
            buf[i + h] = a - b;
        }
        __syncthreads();
    }
    for (int i = threadIdx.x; i < n; i += 256) dst[base + i] = __ushort_as_half(double_to_half_rne(buf[i] * scale));
}

}  // namespace

hipError_t launch_channel_absmax(const void* x, int64_t M, int64_t K, float* absmax, hipStream_t s)
{
    hipError_t e = launch_zero(absmax, (size_t)K * sizeof(float), s);
    if (e != hipSuccess || M == 0) return e;
    const dim3 grid((unsigned)((K / 8 + 255) / 256), (unsigned)((M + kRowsPerSlab - 1) / kRowsPerSlab));
    channel_absmax_kernel<<<grid, 256, 0, s>>>(static_cast<const __half*>(x), M, K, reinterpret_cast<int*>(absmax));
    return hipGetLastError();
}

hipError_t launch_gather_channels(const void* src, const int32_t* perm, int64_t rows, int64_t K, void* dst, hipStream_t s)
{
    const int64_t n = rows * (K / 8);
    if (n == 0) return hipSuccess;
    gather_channels_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(static_cast<const __half*>(src), perm, rows, K,
                                                                        static_cast<__half*>(dst));
    return hipGetLastError();
}

int hadamard_max_block() { return kMaxHadamard; }

hipError_t launch_hadamard(const void* src, int64_t rows, int64_t K, int64_t block, void* dst, hipStream_t s)
{
    if (rows == 0) return hipSuccess;
    const double scale = 1.0 / std::sqrt((double)block);     // correctly rounded on the host
    if ((rows * K) % 8 == 0 && (reinterpret_cast<uintptr_t>(src) & 15u) == 0 && (reinterpret_cast<uintptr_t>(dst) & 15u) == 0) {
        const int64_t chunks = rows * K / 8;
        const uint4* from = static_cast<const uint4*>(src);
        uint4* to = static_cast<uint4*>(dst);
        if (block <= 4096) hadamard_kernel<2><<<(unsigned)((chunks + 511) / 512), 256, 0, s>>>(from, chunks, (int)block, scale, to);
        else hadamard_kernel<4><<<(unsigned)((chunks + 1023) / 1024), 256, 0, s>>>(from, chunks, (int)block, scale, to);
        return hipGetLastError();
    }
    const dim3 grid((unsigned)(K / block), (unsigned)rows);
    hadamard_unaligned_kernel<<<grid, 256, 0, s>>>(static_cast<const __half*>(src), K, (int)block, scale, static_cast<__half*>(dst));
    return hipGetLastError();
}

// Host side: most salient channel first, ties by channel index.
void channel_order_host(const float* salience, int64_t K, int32_t* perm)
{
    std::vector<int32_t> idx((size_t)K);
    std::iota(idx.begin(), idx.end(), 0);
    std::stable_sort(idx.begin(), idx.end(), [&](int32_t a, int32_t b) { return salience[a] > salience[b]; });
    std::copy(idx.begin(), idx.end(), perm);
}

}  // namespace qoq
