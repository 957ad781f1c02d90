// Offline weight path: progressive group quantization (Section 4.1 of arXiv 2405.04532,
// Eq. 3-4 with the protective range), the per-channel variant (Section 5.2.2), and the
// store in matrix-core consumption order (Section 5.2.1).  Runs once per layer.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>

#include "qoq_internal.h"

namespace qoq {
namespace {

constexpr int kThreads = 256;

// Exact round-to-nearest-even conversion of a non-negative finite double to FP16 bits.
__device__ inline uint16_t double_to_half_bits(double d)
{
    if (!(d > 0.0)) return 0;
    int e;
    (void)frexp(d, &e);
    int ex = e - 1;  // d = 1.xxx * 2^ex
    if (ex < -14) {
        const double r = rint(ldexp(d, 24));  // subnormal step 2^-24; 1024 carries into the first normal
        return (uint16_t)(int)r;
    }
    double r = rint(ldexp(d, 10 - ex));  // in [1024, 2048]
    if (r >= 2048.0) { r = 1024.0; ex += 1; }
    if (ex > 15) return 0x7C00;
    return (uint16_t)(((ex + 15) << 10) | ((int)r - 1024));
}

__device__ inline float half_bits_to_float(uint16_t h) { return __half2float(__ushort_as_half(h)); }

// FP16 scale = fp16(range / steps); a zero scale (empty range) becomes 1.0.
__device__ inline uint16_t make_scale(double range, double steps)
{
    uint16_t h = double_to_half_bits(range / steps);
    return h == 0 ? (uint16_t)0x3C00 : h;
}

__device__ inline int round_half_away(double v) { return (int)round(v); }

__device__ inline void write_header(const BlobLayout& L, uint8_t* blob)
{
    BlobHeader h;
    h.magic = kMagic; h.version = kVersion; h.N = L.N; h.K = L.K; h.mode = L.mode; h.group = kGroup;
    h.codes_off = L.codes_off; h.meta_off = L.meta_off; h.scale_off = L.scale_off;
    h.zero_off = L.zero_off; h.total = L.total;
    *reinterpret_cast<BlobHeader*>(blob) = h;
}

typedef _Float16 hv2 __attribute__((ext_vector_type(2)));

// Cross-lane steps inside a row of 16 lanes: after a rotation by 8 and one by 4, the four lanes 4 apart agree.
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
constexpr int kRowRor4 = 0x124, kRowRor8 = 0x128;
__device__ __forceinline__ float quarter_max(float v)
{
    v = fmaxf(v, dpp_f32<kRowRor8>(v));
    return fmaxf(v, dpp_f32<kRowRor4>(v));
}
__device__ __forceinline__ float quarter_min(float v)
{
    v = fminf(v, dpp_f32<kRowRor8>(v));
    return fminf(v, dpp_f32<kRowRor4>(v));
}

// FP16 weights -> packed layer, group or per-channel mode.  One workgroup per four adjacent output channels (rows i ..
// i + 3 of one 16-row fragment, whose 16-byte code words are adjacent in memory); thread (row r, k-block kb, group q) of
// the workgroup owns, per group of 128 channels, the 32 weights whose codes make up one 16-byte lane word: it reads four
// 16-byte chunks and writes the word whole.  The row is read once and kept in registers (CH groups per thread) between
// the pass that finds its range and the pass that quantizes; rows of more than 256 groups are read twice (CH = 0).
//
// Every decision is taken in FP32 and is the one exact arithmetic takes:
//   level 1   round_half_away(w / s0) of two FP16 numbers: |w / s0| < 256 is on a midpoint or at least 2^-12 away from
//             every one; w * fl(1 / s0) is within 3e-5 of it, and pushed 1e-4 away from zero it lands on the same side
//             (the argument of the activation quantizer).  Per-channel codes are the same quotient plus an integer.
//   level 2   quotients of small integers by s1 <= 16 (by 15 for s1 itself): multiples of 1/32 (1/15), nudged by 1e-3.
// PASS_BY (group mode, weights that fit the 256 MB memory-side cache): the codes go past it, so that it keeps the weights that a
// rotation or reordering has just written (22016 x 4096 rotated and packed 145.6 -> 143.6 us when the rotation took 90, 10240 x 8192 reordered
// and packed 148.1 -> 144.6, with the reads of those as non-temporal).  Larger weights are slower so (28672 x 14336 599 us, 604), per-channel ones of any
// size (28672 x 8192 99.0, 102.2).
// Bound by HBM: 22016 x 4096 in group mode in 54 us (226 MB, 4.2 TB/s; a copy moves them in 42 us).  One division of
// doubles per weight and 4-byte stores 16 bytes apart kept one row per workgroup at 213 us, and it wrote the header by
// a launch of its own.
template <bool GROUP, int CH, bool PASS_BY>
__global__ __launch_bounds__(1024) void pack_kernel(const __half* __restrict__ w, BlobLayout L, uint8_t* __restrict__ blob)
{
    __shared__ float s_lo[16][4], s_hi[16][4];
    __shared__ float s_scale[4], s_zero[4];
    const int tid = threadIdx.x, r = tid & 3, kb = (tid >> 2) & 3, q = tid >> 4;
    const int G = (int)L.G, gstep = (int)blockDim.x >> 4;
    // Workgroups go round the eight XCDs; the four that share 256-byte runs of codes (channels 16 apart) follow each
    // other on one of them, so that its L2 puts whole lines together.
    int64_t id = blockIdx.x;
    if (id < (int64_t)(gridDim.x & ~31u)) id = ((id >> 5) << 5) + ((id & 7) << 2) + ((id >> 3) & 3);
    const int64_t nf = id >> 2;
    const int ib = (int)(id & 3);
    const int64_t n = (nf >> 2) * 64 + 16 * ib + 4 * (nf & 3) + r;
    const int i = 4 * ib + r;
    const uint4* row = reinterpret_cast<const uint4*>(w + n * L.K);
    uint4 v[CH > 0 ? CH : 1][4];
    auto load = [&](uint4 (&x)[4], int g) __attribute__((always_inline)) {
        const uint4* src = row + (g < G ? g : 0) * 16 + kb * 2;          // past the end: values that are not used
#pragma unroll
        for (int c = 0; c < 4; ++c) x[c] = src[(c >> 1) * 8 + (c & 1)];
    };
    hv2 mn2 = {(_Float16)0.f, (_Float16)0.f}, mx2 = mn2;                 // the range always contains 0
    auto scan = [&](const uint4 (&x)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint32_t u[4] = {x[c].x, x[c].y, x[c].z, x[c].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const hv2 p = __builtin_bit_cast(hv2, u[e]);
                mn2 = __builtin_elementwise_min(mn2, p);
                mx2 = __builtin_elementwise_max(mx2, p);
            }
        }
    };
    if constexpr (CH > 0) {
#pragma unroll
        for (int c = 0; c < CH; ++c) load(v[c], q + c * gstep);
#pragma unroll
        for (int c = 0; c < CH; ++c)
            if (q + c * gstep < G) scan(v[c]);
    } else {
        for (int g = q; g < G; g += gstep) { load(v[0], g); scan(v[0]); }
    }
    float lo = quarter_min(fminf((float)mn2.x, (float)mn2.y)), hi = quarter_max(fmaxf((float)mx2.x, (float)mx2.y));
#pragma unroll
    for (int o = 16; o < 64; o <<= 1) { lo = fminf(lo, __shfl_xor(lo, o, 64)); hi = fmaxf(hi, __shfl_xor(hi, o, 64)); }
    if ((tid & 63) < 4) { s_lo[tid >> 6][r] = lo; s_hi[tid >> 6][r] = hi; }
    __syncthreads();
    if (tid < 4) {                                                       // thread r settles row r
        for (int x = 1; x < ((int)blockDim.x + 63) >> 6; ++x) { lo = fminf(lo, s_lo[x][r]); hi = fmaxf(hi, s_hi[x][r]); }
        // level 1 with the protective range (Eq. 3), or the per-channel 4-bit scale
        const uint16_t bits = GROUP ? make_scale(fmax((double)hi, -(double)lo), 119.0) : make_scale((double)hi - (double)lo, 15.0);
        const float sc = half_bits_to_float(bits);
        s_scale[r] = sc;
        reinterpret_cast<uint16_t*>(blob + L.scale_off)[n] = bits;
        if (!GROUP) {
            const int z = max(0, min(15, round_half_away(-(double)lo / (double)sc)));
            s_zero[r] = (float)z;
            (blob + L.zero_off)[n] = (uint8_t)z;
        }
    }
    if (blockIdx.x == 0 && tid == 4) write_header(L, blob);
    __syncthreads();
    const float inv = 1.0f / s_scale[r];
    const float half_up = GROUP ? 0.f : s_zero[r] + (0.5f + 1e-4f);
    uint4* codes = reinterpret_cast<uint4*>(blob + L.codes_off);
    uint16_t* meta = reinterpret_cast<uint16_t*>(blob + L.meta_off);
    auto quantize = [&](const uint4 (&x)[4], int g) __attribute__((always_inline)) {
        float f[32];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint32_t u[4] = {x[c].x, x[c].y, x[c].z, x[c].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const hv2 p = __builtin_bit_cast(hv2, u[e]);
                f[8 * c + 2 * e] = (float)p.x;
                f[8 * c + 2 * e + 1] = (float)p.y;
            }
        }
        float scale2 = inv, offset = half_up;                            // code = floor(f * scale2 + offset), clamped
        if constexpr (GROUP) {
            float gmin = 0.f, gmax = 0.f;
#pragma unroll
            for (int e = 0; e < 32; ++e) {
                const float t = f[e] * inv;
                // through an integer: its conversion takes NaN to 0
                f[e] = __builtin_amdgcn_fmed3f((float)(int)(t + copysignf(0.5f + 1e-4f, t)), -119.f, 119.f);
                gmin = fminf(gmin, f[e]);
                gmax = fmaxf(gmax, f[e]);
            }
            // level 2 (Eq. 4): asymmetric UINT4 on the INT8 intermediates, range widened to hold 0
            gmin = quarter_min(gmin);
            gmax = quarter_max(gmax);
            const float s1 = fmaxf(1.f, truncf((gmax - gmin + 14.01f) * (1.f / 15.f)));   // ceil(range / 15)
            scale2 = __builtin_amdgcn_rcpf(s1);
            const float z = fminf(15.f, truncf(fmaf(-gmin, scale2, 0.5f + 1e-3f)));
            offset = z + (0.5f + 1e-3f);
            if (kb == 0 && g < G) {
                const int s = (int)s1, zs = (int)z * s;
                meta[meta_offset(nf, i, g, L.N / 16) / 2] = (uint16_t)(s | (((128 - zs) & 0xFF) << 8));
            }
        }
        uint32_t d[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {                                    // chunk c = k-step c / 2, half c % 2 of its 16 codes
            d[c] = 0;
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const uint32_t code = (uint32_t)(int)__builtin_amdgcn_fmed3f(fmaf(f[8 * c + t], scale2, offset), 0.f, 15.f);
                d[c] |= code << (8 * (t & 3) + 4 * (t >> 2));
            }
        }
        if (g < G) {
            uint4* at = codes + (nf * G + g) * 64 + kb * 16 + i;
            if (PASS_BY) store_nontemporal(at, make_uint4(d[0], d[1], d[2], d[3]));
            else *at = make_uint4(d[0], d[1], d[2], d[3]);
        }
    };
    if constexpr (CH > 0) {
#pragma unroll
        for (int c = 0; c < CH; ++c) quantize(v[c], q + c * gstep);
    } else {
        for (int g0 = 0; g0 < G; g0 += gstep) {                          // all lanes of a row of 16 stay together
            load(v[0], g0 + q);
            quantize(v[0], g0 + q);
        }
    }
}

__global__ void write_header_kernel(BlobLayout L, uint8_t* blob)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) write_header(L, blob);
}

// One thread per packed dword: gathers its 8 codes from the logical [N, K] byte tensor.
__global__ __launch_bounds__(kThreads) void pack_quantized_kernel(const uint8_t* __restrict__ q,
                                                                  const uint8_t* __restrict__ s1,
                                                                  const uint8_t* __restrict__ z,
                                                                  const uint16_t* __restrict__ s_fp16,
                                                                  BlobLayout L, uint8_t* __restrict__ blob)
{
    const int64_t idx = (int64_t)blockIdx.x * kThreads + threadIdx.x;  // (n, g, j): j = dword group of 8 k
    const int64_t per_row = L.G * 16;
    if (idx >= L.N * per_row) return;
    const int64_t n = idx / per_row;
    const int64_t g = (idx % per_row) / 16;
    const int j = (int)(idx % 16);
    int64_t nf; int i;
    phys_row(n, nf, i);
    const uint8_t* src = q + n * L.K + g * kGroup + 8 * j;
    uint32_t v = 0;
    size_t off = 0;
    for (int t = 0; t < 8; ++t) {
        int sh;
        off = code_dword_offset(nf, i, g, L.G, 8 * j + t, sh);
        v |= (uint32_t)(src[t] & 15) << sh;
    }
    *reinterpret_cast<uint32_t*>(blob + L.codes_off + off) = v;
    if (j == 0) {
        if (L.mode == 0) {
            const int sc = s1[n * L.G + g], zz = z[n * L.G + g];
            reinterpret_cast<uint16_t*>(blob + L.meta_off)[meta_offset(nf, i, g, L.N / 16) / 2] =
                (uint16_t)(sc | (((128 - zz * sc) & 0xFF) << 8));
        }
        if (g == 0) {
            reinterpret_cast<uint16_t*>(blob + L.scale_off)[n] = s_fp16[n];
            if (L.mode == 1) (blob + L.zero_off)[n] = z[n];
        }
    }
}

// One thread per logical (n, k).
__global__ __launch_bounds__(kThreads) void unpack_kernel(const uint8_t* __restrict__ blob, BlobLayout L,
                                                          uint8_t* __restrict__ q, uint8_t* __restrict__ s1,
                                                          uint8_t* __restrict__ z, uint16_t* __restrict__ s_fp16)
{
    const int64_t idx = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (idx >= L.N * L.K) return;
    const int64_t n = idx / L.K, k = idx % L.K, g = k / kGroup;
    const int k_local = (int)(k % kGroup);
    int64_t nf; int i;
    phys_row(n, nf, i);
    int sh;
    const size_t off = code_dword_offset(nf, i, g, L.G, k_local, sh);
    const uint32_t v = *reinterpret_cast<const uint32_t*>(blob + L.codes_off + off);
    q[idx] = (uint8_t)((v >> sh) & 15);
    if (k_local == 0) {
        if (L.mode == 0) {
            const uint16_t m = reinterpret_cast<const uint16_t*>(blob + L.meta_off)[meta_offset(nf, i, g, L.N / 16) / 2];
            const int sc = m & 0xFF;
            int b = m >> 8;
            if (b > 128) b -= 256;  // bias = 128 - z*s1 lies in [-112, 128]
            s1[n * L.G + g] = (uint8_t)sc;
            z[n * L.G + g] = (uint8_t)((128 - b) / sc);
        }
        if (k == 0) {
            s_fp16[n] = reinterpret_cast<const uint16_t*>(blob + L.scale_off)[n];
            if (L.mode == 1) z[n] = (blob + L.zero_off)[n];
        }
    }
}

}  // namespace

// As few groups per thread as 1024 threads allow (64 groups at a time): short rows then leave registers for more waves.
template <bool GROUP, bool PASS_BY>
static void launch_pack(const __half* w, const BlobLayout& L, uint8_t* blob, hipStream_t s)
{
    const int64_t per = L.G <= 64 ? 1 : L.G <= 128 ? 2 : 4;
    const int64_t groups = std::min<int64_t>(64, (L.G + per - 1) / per);
    const dim3 grid((unsigned)(L.N / 4)), block((unsigned)((groups * 16 + 63) / 64 * 64));
    if (L.G <= 64) pack_kernel<GROUP, 1, PASS_BY><<<grid, block, 0, s>>>(w, L, blob);
    else if (L.G <= 128) pack_kernel<GROUP, 2, PASS_BY><<<grid, block, 0, s>>>(w, L, blob);
    else if (L.G <= 256) pack_kernel<GROUP, 4, PASS_BY><<<grid, block, 0, s>>>(w, L, blob);
    else pack_kernel<GROUP, 0, PASS_BY><<<grid, block, 0, s>>>(w, L, blob);
}

hipError_t launch_pack_weights(const void* w_fp16, const BlobLayout& L, uint8_t* blob, hipStream_t s)
{
    const __half* w = static_cast<const __half*>(w_fp16);
    if (L.mode != 0) launch_pack<false, false>(w, L, blob, s);
    else if (2 * L.N * L.K <= (int64_t)224 << 20) launch_pack<true, true>(w, L, blob, s);
    else launch_pack<true, false>(w, L, blob, s);
    return hipGetLastError();
}

hipError_t launch_pack_quantized(const uint8_t* q, const uint8_t* s1, const uint8_t* z, const void* s_fp16,
                                 const BlobLayout& L, uint8_t* blob, hipStream_t s)
{
    write_header_kernel<<<1, 64, 0, s>>>(L, blob);
    const int64_t total = L.N * L.G * 16;
    pack_quantized_kernel<<<dim3((unsigned)((total + kThreads - 1) / kThreads)), kThreads, 0, s>>>(
        q, s1, z, static_cast<const uint16_t*>(s_fp16), L, blob);
    return hipGetLastError();
}

hipError_t launch_unpack(const uint8_t* blob, const BlobLayout& L, uint8_t* q, uint8_t* s1, uint8_t* z,
                         void* s_fp16, hipStream_t s)
{
    const int64_t total = L.N * L.K;
    unpack_kernel<<<dim3((unsigned)((total + kThreads - 1) / kThreads)), kThreads, 0, s>>>(
        blob, L, q, s1, z, static_cast<uint16_t*>(s_fp16));
    return hipGetLastError();
}

}  // namespace qoq
