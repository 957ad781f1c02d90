// Data-free offline transforms of QoQ for gfx950 (Section 4.3 of arXiv 2405.04532): channel salience and
// channel gather for the activation-aware reordering, scaled-Hadamard rotation of block-input tensors.
// These run when a model is prepared, not in the serving loop (at run time the reordering is the gather fused
// into the activation quantizer, qoq_act.hip, and the rotation is folded into the preceding layer's weights),
// so they are written for exactness first: the rotation sums in FP64 or in whole numbers, where sums of FP16 numbers are exact for
// these sizes, and rounds once to FP16.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <numeric>
#include <type_traits>
#include <vector>

#include "qoq_fp16.h"
#include "qoq_internal.h"

namespace qoq {
namespace {

// salience[k] = max_m |x[m, k]| (Section 4.3: the magnitude of the input activations decides a channel's
// salience).  A workgroup takes 256 channels x 128 rows: thread (8-channel chunk c, row group q of 8) has the 16 loads of
// its rows in flight together, maxima of FP16 pairs, the eight row groups meet in LDS and one of them goes on;
// non-negative floats order like their bit patterns, so the slabs of rows meet with an integer atomic maximum on a
// zero-filled array; a slab alone stores its maxima, and nothing is filled (1 x 14336: 3.2 us instead of 4.9).  Bound by HBM
// latency and bandwidth: 1025 x 14336 (29 MB) from memory 9.9 us with its fill (one row less by columns, below, 6.9); with one thread per
// 8 channels and 64 rows one after the other, 112 workgroups in all, it was 33 us.
constexpr int kAbsmaxRows = 128;
__global__ __launch_bounds__(256) void channel_absmax_kernel(const uint4* __restrict__ x, int64_t M, int chunks, int* __restrict__ out_bits, bool alone)
{
    __shared__ uint4 s_max[8][32];
    const int cl = threadIdx.x & 31, q = threadIdx.x >> 5;
    const int c = (int)blockIdx.x * 32 + cl;
    const int64_t r0 = (int64_t)blockIdx.y * kAbsmaxRows + q;
    const uint4* col = x + min(c, chunks - 1);
    uint4 v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = col[min(r0 + 8 * j, M - 1) * chunks];   // past the end: the last row once more
    auto pair_max = [](uint32_t a, uint32_t b) {         // of FP16 pairs; a NaN is not taken
        typedef _Float16 hv2 __attribute__((ext_vector_type(2)));
        return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(hv2, a), __builtin_bit_cast(hv2, b & 0x7FFF7FFFu)));
    };
    uint4 mx = make_uint4(0u, 0u, 0u, 0u);
    auto take = [&](const uint4& t) { mx.x = pair_max(mx.x, t.x); mx.y = pair_max(mx.y, t.y); mx.z = pair_max(mx.z, t.z); mx.w = pair_max(mx.w, t.w); };
#pragma unroll
    for (int j = 0; j < 16; ++j) take(v[j]);
    s_max[q][cl] = mx;
    __syncthreads();
    if (q != 0 || c >= chunks) return;
#pragma unroll
    for (int j = 1; j < 8; ++j) take(s_max[j][cl]);
    const uint32_t w[4] = {mx.x, mx.y, mx.z, mx.w};
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int bits = __float_as_int(__half2float(__ushort_as_half((unsigned short)(w[j >> 1] >> (16 * (j & 1))))));
        if (alone) out_bits[(int64_t)c * 8 + j] = bits;
        else atomicMax(out_bits + (int64_t)c * 8 + j, bits);
    }
}

// The same for up to 1024 rows in one pass, without a zero fill before it or atomics: a workgroup takes 64 channels (whole lines of
// 128 bytes) x all rows, thread (8-channel chunk c, row group q of 128) has its up to eight loads in flight together.
// From memory, with the fill where there is one: 1024 x 14336 6.9 us, 9.6 in slabs; 1024 x 28672 13.7 and 16.4; 129 x 4096 3.2 and 5.0.
constexpr int kColumnRows = 1024;
__global__ __launch_bounds__(1024) void channel_absmax_columns_kernel(const uint4* __restrict__ x, int M, int chunks, int* __restrict__ out_bits)
{
    __shared__ uint4 s_max[16][8];
    typedef _Float16 hv2 __attribute__((ext_vector_type(2)));
    auto pair_max = [](uint32_t a, uint32_t b) {         // of FP16 pairs of magnitudes; a NaN is not taken
        return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(hv2, a), __builtin_bit_cast(hv2, b)));
    };
    const int cl = threadIdx.x & 7, q = threadIdx.x >> 3;
    const int c = (int)blockIdx.x * 8 + cl;
    const uint4* col = x + min(c, chunks - 1);
    uint4 v[kColumnRows / 128];
#pragma unroll
    for (int j = 0; j < kColumnRows / 128; ++j)
        if (128 * j < M) v[j] = col[(int64_t)min(q + 128 * j, M - 1) * chunks];   // past the end: the last row once more
        else v[j] = make_uint4(0u, 0u, 0u, 0u);
    uint32_t mx[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < kColumnRows / 128; ++j) {
        const uint32_t w[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
#pragma unroll
        for (int i = 0; i < 4; ++i) mx[i] = pair_max(mx[i], w[i] & 0x7FFF7FFFu);
    }
    // the eight rows of a wave: lanes 8, 16 and 32 apart
#pragma unroll
    for (int h = 8; h < 64; h <<= 1)
#pragma unroll
        for (int i = 0; i < 4; ++i) mx[i] = pair_max(mx[i], (uint32_t)__shfl_xor((int)mx[i], h));
    if ((threadIdx.x & 63) < 8) s_max[threadIdx.x >> 6][cl] = make_uint4(mx[0], mx[1], mx[2], mx[3]);
    __syncthreads();
    if (threadIdx.x >= 64) return;                       // one wave: thread = channel
    const int ch = threadIdx.x, chunk = (int)blockIdx.x * 8 + (ch >> 3);
    if (chunk >= chunks) return;
    uint32_t m = 0;
#pragma unroll
    for (int wv = 0; wv < 16; ++wv) m = max(m, (uint32_t) reinterpret_cast<const unsigned short*>(s_max[wv])[ch]);   // magnitudes order like their bits
    out_bits[(int64_t)blockIdx.x * 64 + ch] = __float_as_int(__half2float(__ushort_as_half((unsigned short)m)));
}

// Sorting by rank: new place of channel k = how many channels come before it (larger salience, or equal and a smaller
// index).  A workgroup settles 64 channels: it sorts them, finds for every channel of the layer by binary search how many of the 64
// it comes before, and counts those numbers; the sums over the counts are the 64 ranks.  Seven steps per channel and workgroup
// where comparing every pair took 64 (14336 channels: 25.5 us; a host sort with its copies 0.7 ms): 10.8 us, 19 if all are equal, which all
// meet in one counter, for K <= kRankMaxK.
// bad[0] = 1 if some salience is not finite (the order is then meaningless), else 0: the first workgroup's work, which it stores past
// the caches, so that it may lie in pinned host memory.
constexpr int kRankMaxK = 32768, kRankThreads = 1024, kRankAhead = 8, kCheckAhead = 16;
__global__ __launch_bounds__(kRankThreads) void channel_order_kernel(const float* __restrict__ salience, int K, int32_t* __restrict__ perm,
                                                                     int32_t* __restrict__ bad)
{
    __shared__ uint32_t s_sorted[64];                    // keys of the workgroup's channels, ascending
    __shared__ uint32_t s_count[64 + 1];                 // channels elsewhere that come before exactly so many of them
    if (blockIdx.x == 0) {
        bool finite = true;
        for (int j0 = 0; j0 < K; j0 += kRankThreads * kCheckAhead) {
            float f[kCheckAhead];
#pragma unroll
            for (int a = 0; a < kCheckAhead; ++a) f[a] = salience[min(j0 + a * kRankThreads + (int)threadIdx.x, K - 1)];
#pragma unroll
            for (int a = 0; a < kCheckAhead; ++a) finite &= fabsf(f[a]) < __builtin_inff();
        }
        const int all = __syncthreads_and(finite);
        if (threadIdx.x == 0) __hip_atomic_store(bad, all ? 0 : 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        return;
    }
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    auto key_of = [](float f) {                          // unsigned integers in the order of the floats, -0 = +0
        const uint32_t b = __float_as_uint(f + 0.0f);
        return b & 0x80000000u ? ~b : b | 0x80000000u;
    };
    const int k0 = ((int)blockIdx.x - 1) * 64, k = k0 + lane;
    uint32_t before = 0;                                 // of the workgroup's own channels, those before this lane's (wave 0)
    if (wave == 0) {
        const uint32_t mine = k < K ? key_of(salience[k]) : 0u;              // past the end: behind every finite one
        for (int e = 0; e < 64; ++e) {
            const uint32_t other = (uint32_t)__builtin_amdgcn_readlane((int)mine, e);
            before += other > mine || (other == mine && e < lane);
        }
        s_sorted[63 - before] = mine;                    // (a permutation of 0 ... 63)
        s_count[lane] = 0;
        if (lane == 0) s_count[64] = 0;
    }
    __syncthreads();
    for (int j0 = 0; j0 < K; j0 += kRankThreads * kRankAhead) {
        float f[kRankAhead];
#pragma unroll
        for (int a = 0; a < kRankAhead; ++a) f[a] = salience[min(j0 + a * kRankThreads + (int)threadIdx.x, K - 1)];
        uint32_t v[kRankAhead], at[kRankAhead];
#pragma unroll
        for (int a = 0; a < kRankAhead; ++a) {
            const int j = j0 + a * kRankThreads + (int)threadIdx.x;
            v[a] = key_of(f[a]) - (j < k0 ? 0u : 1u);    // ties: a channel in front comes before an equal one, one behind does not
            at[a] = 0;
        }
        // how many of the 64 are at most v
#pragma unroll
        for (int h = 32; h >= 1; h >>= 1)
#pragma unroll
            for (int a = 0; a < kRankAhead; ++a) at[a] += s_sorted[at[a] + h - 1] <= v[a] ? h : 0;
#pragma unroll
        for (int a = 0; a < kRankAhead; ++a) {
            const int j = j0 + a * kRankThreads + (int)threadIdx.x;
            at[a] += s_sorted[at[a]] <= v[a];
            if (j < K && (uint32_t)(j - k0) >= 64u) atomicAdd(&s_count[at[a]], 1u);
        }
    }
    __syncthreads();
    if (wave != 0) return;
    // channel at ascending place p: everybody that comes before more than p of the 64
    const int p = 63 - (int)before;
    uint32_t rank = before;
    for (int c = 1; c <= 64; ++c) rank += c > p ? s_count[c] : 0u;
    if (k < K) perm[min((int)rank, K - 1)] = k;          // (the bound only matters for NaNs)
}

// dst[r, j] = src[r, perm[j]].  A workgroup brings ROWS rows into LDS as whole lines and gathers there: thread t makes
// 8 output channels at a time, whose indices it fetches once for all its rows.  Two-byte gathers from memory, the first
// version, took 134 us for 4096 x 14336 (117 MB each way; a copy takes 44 us), this one 49 us.  Indices are clamped to
// the row.  NT: what is read is not wanted again, what is written is (cache_for_output).
// Where the 256 MB memory-side cache holds the result and not the source beside it, the packing that follows finds the result there if the source
// was read past it (22016 x 4096 reordered and packed 110 -> 107 us; see pack_kernel).  Beyond, every byte of the source kept counts (28672 x
// 8192 rotated and packed 541 us, 547 with the source read past it), and smaller sources lie there already more often than not: 1152 x 15360
// reordered and packed again and again 37.6 us, 44.2 past the cache, 4096 x 4096 25.0 and 26.9; 4096 x 8192 from memory 50.9 and 49.4.
bool cache_for_output(int64_t elements) { return 2 * elements > (int64_t)128 << 20 && 2 * elements <= (int64_t)224 << 20; }

constexpr int kGatherThreads = 512;
constexpr int64_t kGatherLds = 64 << 10;
template <int ROWS, bool NT>
__global__ __launch_bounds__(kGatherThreads) void gather_channels_kernel(const uint4* __restrict__ src, const int4* __restrict__ perm,
                                                                         int64_t rows, int K, uint4* __restrict__ dst)
{
    extern __shared__ __attribute__((aligned(16))) unsigned short s_row[];   // ROWS x K
    const int chunks = K / 8;
    const int64_t r0 = (int64_t)blockIdx.x * ROWS;
    const int here = (int)min((int64_t)ROWS, rows - r0);
    for (int c = threadIdx.x; c < here * chunks; c += kGatherThreads) reinterpret_cast<uint4*>(s_row)[c] = NT ? load_nontemporal(src + r0 * chunks + c) : src[r0 * chunks + c];
    __syncthreads();
    for (int c = threadIdx.x; c < chunks; c += kGatherThreads) {
        const int4 p0 = perm[2 * c], p1 = perm[2 * c + 1];
        const int idx[8] = {p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, p1.z, p1.w};
        int at[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) at[j] = min(max(idx[j], 0), K - 1);
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            if (r < here) {
                uint32_t w[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) w[j] = (uint32_t)s_row[r * K + at[2 * j]] | ((uint32_t)s_row[r * K + at[2 * j + 1]] << 16);
                dst[(r0 + r) * chunks + c] = make_uint4(w[0], w[1], w[2], w[3]);
            }
        }
    }
}

// Rows too long for LDS, short ones and few: one thread per 8 output channels, gathers from memory.
__global__ __launch_bounds__(256) void gather_direct_kernel(const __half* __restrict__ src, const int32_t* __restrict__ perm,
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
// Exact sums: every partial sum of at most 8192 FP16 numbers is a multiple of 2^-24 below 2^29, which FP64 holds (and 32-bit
// integers where the sums are small), so the result is the exact product times `scale`, rounded once, whatever the order of the
// stages.
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

// Sum of non-negative numbers over a wave.
__device__ __forceinline__ float wave_sum_of(float v)
{
    auto moved = [](float x, auto ctrl) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xF, 0xF, false));
    };
    v += moved(v, std::integral_constant<int, 0xB1>());      // lanes ^1, ^2, then the mirrored half row and row of 16
    v += moved(v, std::integral_constant<int, 0x4E>());
    v += moved(v, std::integral_constant<int, 0x141>());
    v += moved(v, std::integral_constant<int, 0x140>());
    auto lane = [&](int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); };
    return (lane(0) + lane(16)) + (lane(32) + lane(48));
}

// Blocks of rows * K contiguous elements are cut into segments of 4096 elements (8192 for blocks of 8192), one workgroup of 256 threads
// each; a segment holds whole blocks.  A thread keeps E = 16 (32) elements in registers and takes the stages in three layouts, with
// two exchanges through LDS instead of one per stage:
//     A  16-byte chunks as they are loaded: element bits 0..2, and 11.. (chunks 256 apart)
//     B  element bits 3..6 in registers, and 12
//     C  element bits 7..10 in registers, and 12
// and the FP16 results go back to chunk order through LDS for 16-byte stores.  LDS position of element i: i + i / 8 + 8 (i / 128),
// which spreads all three access patterns evenly over the 64 banks (two lanes to a bank at most); a thread's places are a constant
// distance apart in each layout, so one address serves them all.  The block size is known when the kernel is compiled: with stages
// under conditions the compiler copied every register at each.
struct HadamardPlaces {
    int a, b, c;
    __device__ __forceinline__ HadamardPlaces(int t) : a(9 * t + (t >> 4) * 8), b((t & 7) + (t >> 3) * 152), c((t & 127) + ((t & 127) >> 3) + (t >> 7) * 2432) {}
    // of the thread's j-th register
    __device__ __forceinline__ int in_a(int j) const { return a + (j >> 3) * 2432 + (j & 7); }
    __device__ __forceinline__ int in_b(int j) const { return b + (j >> 4) * 4864 + (j & 15) * 9; }
    __device__ __forceinline__ int in_c(int j) const { return c + (j >> 4) * 4864 + (j & 15) * 152; }
};
// the stages whose element bits FROM + i are register bits AT + i, i < BITS, as far as the block of 2^LOGN goes
template <int LOGN, int E, int AT, int FROM, int BITS, class T>
__device__ __forceinline__ void hadamard_stages(T (&v)[E])
{
#pragma unroll
    for (int i = 0; i < BITS; ++i)
        if (FROM + i < LOGN)
#pragma unroll
            for (int j = 0; j < E; ++j)
                if (!(j & (1 << (AT + i)))) {
                    const T s = v[j] + v[j | (1 << (AT + i))];
                    v[j | (1 << (AT + i))] = v[j] - v[j | (1 << (AT + i))];
                    v[j] = s;
                }
}
// results of a thread, in layout C as pairs of FP16 numbers, to chunk order and to memory
template <int E>
__device__ __forceinline__ void hadamard_store(const uint32_t (&r)[E / 2], unsigned short* out, int64_t c0, int64_t chunks, uint4* __restrict__ dst)
{
    const int t = threadIdx.x;
    __syncthreads();                                     // everybody has read: the buffer takes the results
#pragma unroll
    for (int j = 0; j < E; ++j) out[(t & 127) + (t >> 7) * 2048 + (j >> 4) * 4096 + (j & 15) * 128] = (unsigned short)(r[j >> 1] >> (16 * (j & 1)));
    __syncthreads();
#pragma unroll
    for (int c = 0; c < E / 8; ++c) {
        const int64_t at = c0 + c * 256 + t;
        if (at < chunks) dst[at] = reinterpret_cast<const uint4*>(out)[c * 256 + t];
    }
}

// Whole numbers in units of scale' = scale / 2^-24, the scale already divided.
template <int LOGN>
__device__ __forceinline__ void hadamard_whole(int (&v)[16], int* buf, int64_t c0, int64_t chunks, double scale, uint4* __restrict__ dst)
{
    const HadamardPlaces at((int)threadIdx.x);
    hadamard_stages<LOGN, 16, 0, 0, 3>(v);
    hadamard_stages<LOGN, 16, 3, 11, 1>(v);
#pragma unroll
    for (int j = 0; j < 16; ++j) buf[at.in_a(j)] = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = buf[at.in_b(j)];
    hadamard_stages<LOGN, 16, 0, 3, 4>(v);
#pragma unroll
    for (int j = 0; j < 16; ++j) buf[at.in_b(j)] = v[j];  // (where it has read: no barrier between)
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = buf[at.in_c(j)];
    hadamard_stages<LOGN, 16, 0, 7, 4>(v);
    // x * scale from both sides in FP32: the conversion, the factor and the product are off by 2^-24 each, the factors'
    // distance from the scale is 3.5 to 4.5 times that.  Rounding is monotonic: where both sides give the same FP16
    // number the exact product does, else (1 element in 1000) FP64 decides.
    const float below = (float)(scale * (1.0 - 4 * 0x1p-24)), above = (float)(scale * (1.0 + 4 * 0x1p-24));
    uint32_t r[8], undecided = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        typedef float f2 __attribute__((ext_vector_type(2)));
        typedef _Float16 hv2 __attribute__((ext_vector_type(2)));
        const float f0 = (float)v[2 * j], f1 = (float)v[2 * j + 1];
        r[j] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f2){f0 * below, f1 * below}, hv2));
        const uint32_t hi = __builtin_bit_cast(uint32_t, __builtin_convertvector((f2){f0 * above, f1 * above}, hv2));
        undecided |= r[j] != hi ? 1u << j : 0u;
    }
    if (undecided) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (undecided >> j & 1) r[j] = (uint32_t)half_rne_by_odd((double)v[2 * j] * scale) | ((uint32_t)half_rne_by_odd((double)v[2 * j + 1] * scale) << 16);
    }
    hadamard_store<16>(r, reinterpret_cast<unsigned short*>(buf), c0, chunks, dst);
}

// A thread's FP64 numbers from one layout to the other, the two halves one after the other through space for one.
template <int E, class From, class To>
__device__ __forceinline__ void exchange_halves(double (&v)[E], uint32_t* words, From from, To to)
{
    uint32_t low[E];
#pragma unroll
    for (int j = 0; j < E; ++j) words[from(j)] = (uint32_t)__double2loint(v[j]);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < E; ++j) low[j] = words[to(j)];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < E; ++j) words[from(j)] = (uint32_t)__double2hiint(v[j]);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < E; ++j) v[j] = __hiloint2double((int)words[to(j)], (int)low[j]);
}

template <int LOGN>
__device__ __forceinline__ void hadamard_fp64(double (&v)[16], uint32_t* buf, int64_t c0, int64_t chunks, double scale, uint4* __restrict__ dst)
{
    const HadamardPlaces at((int)threadIdx.x);
    hadamard_stages<LOGN, 16, 0, 0, 3>(v);
    hadamard_stages<LOGN, 16, 3, 11, 1>(v);
    exchange_halves(v, buf, [&](int j) { return at.in_a(j); }, [&](int j) { return at.in_b(j); });
    hadamard_stages<LOGN, 16, 0, 3, 4>(v);
    exchange_halves(v, buf, [&](int j) { return at.in_b(j); }, [&](int j) { return at.in_c(j); });
    hadamard_stages<LOGN, 16, 0, 7, 4>(v);
    uint32_t r[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) r[j] = (uint32_t)half_rne_by_odd(v[2 * j] * scale) | ((uint32_t)half_rne_by_odd(v[2 * j + 1] * scale) << 16);
    hadamard_store<16>(r, reinterpret_cast<unsigned short*>(buf), c0, chunks, dst);
}

__device__ __forceinline__ uint4 hadamard_load(const uint4* __restrict__ src, int64_t at, int64_t chunks, bool nt)
{
    if (at >= chunks) return make_uint4(0u, 0u, 0u, 0u);
    return nt ? load_nontemporal(src + at) : src[at];
}

// An FP16 number is a whole multiple of 2^-24, so where the magnitudes of a segment add up to less than 128 every partial sum
// fits 32-bit integers in that unit and the butterflies are integer additions: a quarter of the issue time of FP64 ones and half of
// the LDS traffic, the same exact sums.  Weight rows are like that (4096 values of standard deviation 0.02 add up to 65);
// other segments, infinities and NaN among them, and blocks of less than eight or of 8192 take FP64, and so do segments with a -0
// in them: whole numbers have one zero, while FP64 sums of FP16 numbers are -0 only where a -0 went in (-0 - (x - x) = -0).
// 22016 x 4096: a single workgroup per block with one LDS round trip and one barrier per stage, bound by LDS and barriers, took 863 us,
// these layouts 108 (a copy of the tensor 69) while they were bound by 40 vector instructions per element, half of them
// addresses and copies of registers, and 90 with LDS for whole FP64 numbers, four workgroups to a compute unit.  Now 72 (in FP64 92), with eight.
template <int LOGN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8))) void hadamard_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, int64_t chunks,
                                                                                                 double scale, bool nt)
{
    constexpr int kElems = 4096;
    __shared__ __attribute__((aligned(16))) uint32_t buf[kElems + kElems / 8 + kElems / 16];
    __shared__ float s_sum[4];
    typedef short s2 __attribute__((ext_vector_type(2)));
    typedef _Float16 hv2 __attribute__((ext_vector_type(2)));
    const int t = threadIdx.x;
    const int64_t c0 = (int64_t)blockIdx.x * 512;
    const uint4 raw[2] = {hadamard_load(src, c0 + t, chunks, nt), hadamard_load(src, c0 + 256 + t, chunks, nt)};
    const uint32_t w[8] = {raw[0].x, raw[0].y, raw[0].z, raw[0].w, raw[1].x, raw[1].y, raw[1].z, raw[1].w};
    if constexpr (LOGN >= 3) {
        float sum = 0.f;
        s2 lowest = {0, 0};                              // of the bits as 16-bit integers, among which those of -0 are the lowest
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            lowest = __builtin_elementwise_min(lowest, __builtin_bit_cast(s2, w[i]));
            sum = __builtin_amdgcn_fdot2(__builtin_bit_cast(hv2, w[i] & 0x7FFF7FFFu), (hv2){(_Float16)1.f, (_Float16)1.f}, sum, false);
        }
        if (min(lowest.x, lowest.y) == -32768) sum = __builtin_inff();
        sum = wave_sum_of(sum);
        if ((t & 63) == 0) s_sum[t >> 6] = sum;
        __syncthreads();
        // the FP32 sum is off by less than 2^-16 of itself, and by the subnormal numbers, 4096 of less than 2^-14, if the
        // instruction takes them for zeros
        if ((s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]) < 127.5f) {
            int whole[16];                               // in units of 2^-24
#pragma unroll
            for (int j = 0; j < 16; ++j) whole[j] = (int)(__half2float(__ushort_as_half((unsigned short)(w[j >> 1] >> (16 * (j & 1))))) * 0x1p24f);
            hadamard_whole<LOGN>(whole, reinterpret_cast<int*>(buf), c0, chunks, scale * 0x1p-24, dst);
            return;
        }
    }
    double v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = (double)__half2float(__ushort_as_half((unsigned short)(w[j >> 1] >> (16 * (j & 1)))));
    hadamard_fp64<LOGN>(v, buf, c0, chunks, scale, dst);
}

// Blocks of 8192 (weights of the usual size then add up to more than 128): the two halves of the FP64 numbers are exchanged one after
// the other, in half the LDS, which makes four workgroups to a compute unit, not two, and they hide each other's barriers and
// loads (8192 x 8192 from memory 119 -> 76 us with the kernel for this one size, 2048 x 8192 33.7 -> 24.5).
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void hadamard_8192_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, int64_t chunks,
                                                                                                      double scale, bool nt)
{
    constexpr int kElems = 8192, E = 32;
    __shared__ __attribute__((aligned(16))) uint32_t words[kElems + kElems / 8 + kElems / 16];
    const HadamardPlaces at((int)threadIdx.x);
    const int64_t c0 = (int64_t)blockIdx.x * 1024;
    double v[E];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const uint4 raw = hadamard_load(src, c0 + c * 256 + (int)threadIdx.x, chunks, nt);
        const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) v[8 * c + e] = (double)__half2float(__ushort_as_half((unsigned short)(w[e >> 1] >> (16 * (e & 1)))));
    }
    hadamard_stages<13, E, 0, 0, 3>(v);
    hadamard_stages<13, E, 3, 11, 2>(v);
    exchange_halves(v, words, [&](int j) { return at.in_a(j); }, [&](int j) { return at.in_b(j); });
    hadamard_stages<13, E, 0, 3, 4>(v);
    exchange_halves(v, words, [&](int j) { return at.in_b(j); }, [&](int j) { return at.in_c(j); });
    hadamard_stages<13, E, 0, 7, 4>(v);
    uint32_t r[E / 2];
#pragma unroll
    for (int j = 0; j < E / 2; ++j) r[j] = (uint32_t)half_rne_by_odd(v[2 * j] * scale) | ((uint32_t)half_rne_by_odd(v[2 * j + 1] * scale) << 16);
    hadamard_store<E>(r, reinterpret_cast<unsigned short*>(words), c0, chunks, dst);
}

// The same for tensors that are no whole number of 16-byte chunks or not aligned to them, and for a few short blocks: one
// workgroup per (row, block).
__global__ __launch_bounds__(256) void hadamard_block_kernel(const __half* __restrict__ src, int64_t K, int n, double scale,
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
    // One slab of rows is stored as it is; up to 1024 rows go in one pass, whose workgroups take longer the more rows there are; beyond, the
    // slabs of rows meet by atomics.
    if (M > kAbsmaxRows && M <= kColumnRows) {
        channel_absmax_columns_kernel<<<(unsigned)((K / 8 + 7) / 8), 1024, 0, s>>>(static_cast<const uint4*>(x), (int)M, (int)(K / 8),
                                                                                  reinterpret_cast<int*>(absmax));
        return hipGetLastError();
    }
    if (M == 0 || M > kAbsmaxRows) {
        const hipError_t e = launch_zero(absmax, (size_t)K * sizeof(float), s);
        if (e != hipSuccess || M == 0) return e;
    }
    const int64_t chunks = K / 8;
    for (int64_t m0 = 0; m0 < M; m0 += (int64_t)65535 * kAbsmaxRows) {       // at most 65535 slabs in a launch
        const int64_t rows = std::min<int64_t>(M - m0, (int64_t)65535 * kAbsmaxRows);
        const dim3 grid((unsigned)((chunks + 31) / 32), (unsigned)((rows + kAbsmaxRows - 1) / kAbsmaxRows));
        channel_absmax_kernel<<<grid, 256, 0, s>>>(static_cast<const uint4*>(x) + m0 * chunks, rows, (int)chunks, reinterpret_cast<int*>(absmax), M <= kAbsmaxRows);
    }
    return hipGetLastError();
}

int channel_order_max_k() { return kRankMaxK; }

hipError_t launch_channel_order(const float* salience, int64_t K, int32_t* perm, int32_t* bad, hipStream_t s)
{
    channel_order_kernel<<<(unsigned)((K + 63) / 64 + 1), kRankThreads, 0, s>>>(salience, (int)K, perm, bad);
    return hipGetLastError();
}

hipError_t launch_gather_channels(const void* src, const int32_t* perm, int64_t rows, int64_t K, void* dst, hipStream_t s)
{
    if (rows == 0) return hipSuccess;
    // Gathers from memory are ahead where a row is a few cache lines (65536 x 128: 8.8 us, through LDS 11.3; x 320 20.2 and 16.6)
    // and where long rows are few, since all of a workgroup's threads first wait for its row (64 x 11008: 3.1 and 3.9 us,
    // 32 x 28672 3.9 and 4.9, 128 x 11008 4.0 and 3.4).
    if (2 * K <= kGatherLds && K > 256 && (K < 8192 || rows * K >= (int64_t)5 << 18)) {
        // as many rows as fit 64 KiB (two workgroups of 512 threads per compute unit), at most four, and no more than leave
        // a workgroup for every compute unit (256 x 4096: 2.6 us with one row each, 3.4 with four)
        const uint4* from = static_cast<const uint4*>(src);
        const int4* p = reinterpret_cast<const int4*>(perm);
        uint4* to = static_cast<uint4*>(dst);
        auto blocks = [&](int per) { return dim3((unsigned)((rows + per - 1) / per)); };
        const bool nt = cache_for_output(rows * K);
        auto launch = [&](auto* kernel, int per) { kernel<<<blocks(per), kGatherThreads, (size_t)K * 2 * per, s>>>(from, p, rows, (int)K, to); };
        if (8 * K <= kGatherLds && rows >= 2048) launch(nt ? gather_channels_kernel<4, true> : gather_channels_kernel<4, false>, 4);
        else if (4 * K <= kGatherLds && rows >= 512) launch(nt ? gather_channels_kernel<2, true> : gather_channels_kernel<2, false>, 2);
        else launch(nt ? gather_channels_kernel<1, true> : gather_channels_kernel<1, false>, 1);
        return hipGetLastError();
    }
    const int64_t n = rows * (K / 8);
    gather_direct_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(static_cast<const __half*>(src), perm, rows, K, static_cast<__half*>(dst));
    return hipGetLastError();
}

int hadamard_max_block() { return kMaxHadamard; }

hipError_t launch_hadamard(const void* src, int64_t rows, int64_t K, int64_t block, void* dst, hipStream_t s)
{
    if (rows == 0) return hipSuccess;
    const double scale = 1.0 / std::sqrt((double)block);     // correctly rounded on the host
    // A short block needs no exchange between layouts, and 512 workgroups of their own run side by side: 1 x 14336 in blocks of
    // 128 3.0 us, 3.7 in segments; 16 x 4096 3.2 and 3.7, 32 x 4096 5.0 and 3.7; blocks of 512 4.0 and 3.8.
    const bool few = block <= 256 && rows * (K / block) <= 512;
    if (!few && (rows * K) % 8 == 0 && (reinterpret_cast<uintptr_t>(src) & 15u) == 0 && (reinterpret_cast<uintptr_t>(dst) & 15u) == 0) {
        const int64_t chunks = rows * K / 8;
        const uint4* from = static_cast<const uint4*>(src);
        uint4* to = static_cast<uint4*>(dst);
        const bool nt = cache_for_output(rows * K);
        auto launch = [&](auto* kernel, int per) { kernel<<<(unsigned)((chunks + per - 1) / per), 256, 0, s>>>(from, to, chunks, scale, nt); };
        switch (block) {
            case 1: launch(hadamard_kernel<0>, 512); break;
            case 2: launch(hadamard_kernel<1>, 512); break;
            case 4: launch(hadamard_kernel<2>, 512); break;
            case 8: launch(hadamard_kernel<3>, 512); break;
            case 16: launch(hadamard_kernel<4>, 512); break;
            case 32: launch(hadamard_kernel<5>, 512); break;
            case 64: launch(hadamard_kernel<6>, 512); break;
            case 128: launch(hadamard_kernel<7>, 512); break;
            case 256: launch(hadamard_kernel<8>, 512); break;
            case 512: launch(hadamard_kernel<9>, 512); break;
            case 1024: launch(hadamard_kernel<10>, 512); break;
            case 2048: launch(hadamard_kernel<11>, 512); break;
            case 4096: launch(hadamard_kernel<12>, 512); break;
            case kMaxHadamard: launch(hadamard_8192_kernel, 1024); break;
            default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    const dim3 grid((unsigned)(K / block), (unsigned)rows);
    hadamard_block_kernel<<<grid, 256, 0, s>>>(static_cast<const __half*>(src), K, (int)block, scale, static_cast<__half*>(dst));
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
