// Pieces shared by the translation units of the W4A8 GEMM kernels (internal to the library): kernel arguments,
// the register dequantizer (Sections 5.2.2-5.2.3 of arXiv 2405.04532), the epilogue of four channels of one token
// (Section 5.2.2, Eq. 5-7) and the fence-free loads and stores of the cross-workgroup hand-over.
#pragma once
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qoq_tiles.h"

namespace qoq {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef unsigned short us2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kNFrag = 4;  // 16-row fragments per wave = 64 output channels

struct GemmDev {
    const int8_t* qx;
    const uint4* codes;
    const uint16_t* meta;
    const __half* scales;
    const uint8_t* zeros;
    const __half* sx;
    const int32_t* rowsum;
    __half* out16;
    int32_t* out32;
    int* counters;  // split-k: one per output tile, zero on entry and on exit
    int4* parts;    // split-k: [tile][split][value][thread]
    int M, N, K, G, gps, S;  // gps = groups per k-split, S = number of k-splits (tiled kernel)
    int upw;                 // stream kernel: work units per workgroup
    int token_sum;           // per-channel FP16 epilogue in the token-sum form: `rowsum` then holds the FP32 sums t_X
    int nwg;                 // gridDim.x
};

// How a GemmDev reaches a kernel.  The first fourteen dwords of a kernel's arguments, where they are plain values, arrive in
// scalar registers with the wave (build.py asks for it): what the first loads need is there when the kernel starts.  A structure
// does not, and fetching it took every kernel about 0.3 us before its first load went out (the one-token Llama-2-7B decoder
// layer, ten kernels, 59.5 -> 55.5 us; 16 x 256 x 256 in one launch 4.21 -> 4.11); what only the epilogue needs still comes that way, behind the loads.
struct GemmTail {
    const __half* scales;
    const uint8_t* zeros;
    const int32_t* rowsum;
    __half* out16;
    int32_t* out32;
    int* counters;
    int4* parts;
    int token_sum;
};
#define QOQ_GEMM_PARAMS const int8_t *a_qx, const uint4 *a_codes, const uint16_t *a_meta, const __half *a_sx, int a_M, int a_N, int a_K, int a_share, \
                        int a_S, int a_nwg
#define QOQ_GEMM_ARGS a_qx, a_codes, a_meta, a_sx, a_M, a_N, a_K, a_share, a_S, a_nwg
__device__ __forceinline__ GemmDev gemm_dev(QOQ_GEMM_PARAMS, const GemmTail& t)
{
    GemmDev p;
    p.qx = a_qx; p.codes = a_codes; p.meta = a_meta; p.sx = a_sx;
    p.M = a_M; p.N = a_N; p.K = a_K; p.G = a_K / 128; p.gps = p.upw = a_share; p.S = a_S; p.nwg = a_nwg;
    p.scales = t.scales; p.zeros = t.zeros; p.rowsum = t.rowsum; p.out16 = t.out16; p.out32 = t.out32;
    p.counters = t.counters; p.parts = t.parts; p.token_sum = t.token_sum;
    return p;
}
inline bool weights_pass_by(const GemmDev& p, dim3 grid, int64_t least) { return weights_pass_by(p.N, p.K, grid.y, least); }
// `more`: further arguments of the kernel, behind the structure.
template <class Kernel, class... More>
void launch_gemm_kernel(Kernel* kernel, dim3 grid, int threads, hipStream_t s, const GemmDev& p, const More&... more)
{
    const GemmTail tail{p.scales, p.zeros, p.rowsum, p.out16, p.out32, p.counters, p.parts, p.token_sum};
    kernel<<<grid, threads, 0, s>>>(p.qx, p.codes, p.meta, p.sx, p.M, p.N, p.K, p.upw ? p.upw : p.gps, p.S, (int)grid.x, tail, more...);
}

enum { OUT_FP16 = 0, OUT_I32 = 1 };

__device__ inline uint32_t pk_mad_u16(uint32_t a, uint32_t s, uint32_t b)
{
    us2 r = __builtin_bit_cast(us2, a) * __builtin_bit_cast(us2, s) + __builtin_bit_cast(us2, b);
    return __builtin_bit_cast(uint32_t, r);
}

// Two packed dwords (16 codes) -> one 16-byte INT8 MFMA operand.
template <bool GROUP>
__device__ inline v4i dequant(uint32_t x0, uint32_t x1, uint32_t S, uint32_t B)
{
    const uint32_t m = 0x0F0F0F0Fu;
    uint32_t o0 = x0 & m, o1 = (x0 >> 4) & m, o2 = x1 & m, o3 = (x1 >> 4) & m;
    if (GROUP) {
        const uint32_t sign = 0x80808080u;
        o0 = pk_mad_u16(o0, S, B) ^ sign;
        o1 = pk_mad_u16(o1, S, B) ^ sign;
        o2 = pk_mad_u16(o2, S, B) ^ sign;
        o3 = pk_mad_u16(o3, S, B) ^ sign;
    }
    v4i r;
    r.x = (int)o0; r.y = (int)o1; r.z = (int)o2; r.w = (int)o3;
    return r;
}

__device__ inline v4i as_v4i(uint4 t) { return (v4i){(int)t.x, (int)t.y, (int)t.z, (int)t.w}; }

// Direct global -> LDS copy, 16 (or 4) bytes per lane; lane l lands at lds_addr + 16*l (4*l).
// `base` is wave-uniform, `voff` the lane's byte offset.  Opaque to the compiler on purpose.
// M0 (the copy's LDS base) is a reserved register that nothing else in these kernels uses, so
// it is not listed as a clobber.
__device__ __forceinline__ const void* to_sgpr(const void* ptr)   // value is wave-uniform; pin it to scalar registers
{
    const uint64_t v = reinterpret_cast<uint64_t>(ptr);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<const void*>(((uint64_t)hi << 32) | lo);
}
template <bool NT = false>                               // non-temporal
__device__ __forceinline__ void dma16(const void* base, uint32_t voff, uint32_t lds_addr)
{
    if constexpr (NT) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                     :: "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(voff), "s"(to_sgpr(base)) : "memory");
        return;
    }
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(voff), "s"(to_sgpr(base)) : "memory");
}
__device__ __forceinline__ void dma4(const void* base, uint32_t voff, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
                 :: "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(voff), "s"(to_sgpr(base)) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}
// Bank swizzle of activation rows kept in LDS as whole 128-byte lines (eight 16-byte chunks per token row): chunk c
// of row r is stored at chunk position c ^ row_swizzle(r).  The LDS of gfx950 has 64 banks of 4 bytes and serves
// a 16-byte fragment read 16 lanes at a time; those lanes take the same chunk of 16 consecutive rows, i.e. 8 even
// rows (first half of the banks) and 8 odd ones (second half), and (r >> 1) & 7 gives each of the eight a different
// position.  (Measured: swizzles that only use r & 7 leave two-way conflicts on every such read.)
__device__ __forceinline__ int row_swizzle(int r) { return (r >> 1) & 7; }   // r = row % 16

// Write-through store / cache-bypassing load of 16 bytes (device-coherent without fences).
// A store of more than 8 bytes reads its data registers over several cycles after issue; the instruction that
// follows must not write them (a documented wait-state requirement the compiler honours for its own stores but
// cannot for inline assembly, which it does not know to be a store: partial sums whose registers were reused at
// once came out corrupted in a few lanes).  Hence the idle cycles inside the store statements.  The streaming
// kernel goes further and keeps its stores out of the loop altogether: they go out after the last copy,
// together with the wait for their completion, from registers the same statement keeps alive.
__device__ __forceinline__ void store_sc1(int4* ptr, v4i v)
{
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 3" :: "v"(ptr), "v"(v) : "memory");
}
// The loads are the compiler's own, so that it knows their registers to be empty until it has waited: written as inline
// assembly they are outputs it takes as written at once, and may move before the data is there.  Lane offset voff, then
// soff, from a wave-uniform base (a partial tile: at most 256 KiB).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t part_rsrc(const int4* base, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(to_sgpr(base)), 0, bytes, 0x00020000);
}
__device__ __forceinline__ v4i load_sc1(__amdgpu_buffer_rsrc_t rsrc, int voff, int soff)
{
    return __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, soff, 0x10));   // 0x10 = sc1
}

// Four 16-byte loads past the caches, `stride` apart, and the wait for them in the same statement.  For the kernels whose
// main loop takes every register: loads that the compiler places itself (load_sc1) cost it some (256 x 256 tiles, 4096 x 4096 x
// 4096 per channel 70.2 us, 67.9 with these).
__device__ __forceinline__ void load_sc1_and_wait(v4i* v, const int4* ptr, int stride)
{
    asm volatile("global_load_dwordx4 %0, %4, off sc1\n\tglobal_load_dwordx4 %1, %5, off sc1\n\t"
                 "global_load_dwordx4 %2, %6, off sc1\n\tglobal_load_dwordx4 %3, %7, off sc1\n\ts_waitcnt vmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
                 : "v"(ptr), "v"(ptr + stride), "v"(ptr + 2 * stride), "v"(ptr + 3 * stride) : "memory");
}

// Compiler-visible write-through store / cache-bypassing load (two relaxed device-scope 8-byte atomics each): the
// compiler tracks their registers and waits itself.  For code with no copy queue to preserve, and wherever
// control flow lies between a load and its use (the compiler may copy a register it believes already loaded).
__device__ __forceinline__ void store_through(int4* ptr, int a, int b, int c, int d)
{
    unsigned long long* q = reinterpret_cast<unsigned long long*>(ptr);
    __hip_atomic_store(q, (unsigned long long)(uint32_t)a | ((unsigned long long)(uint32_t)b << 32), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(q + 1, (unsigned long long)(uint32_t)c | ((unsigned long long)(uint32_t)d << 32), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ v4i load_through(const int4* ptr)
{
    unsigned long long* q = const_cast<unsigned long long*>(reinterpret_cast<const unsigned long long*>(ptr));
    const unsigned long long lo = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long hi = __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return (v4i){(int)(uint32_t)lo, (int)(uint32_t)(lo >> 32), (int)(uint32_t)hi, (int)(uint32_t)(hi >> 32)};
}
template <bool GROUP, int OUT>
__device__ __forceinline__ void finish4(const GemmDev& p, int m, int n0, v4i v, const float (&sn)[4],
                                        const int (&zn)[4], float sxm, int rs)
{
    int t[4] = {v.x, v.y, v.z, v.w};
    // Per-channel zero point: exact integer fold acc - z * rowsum (Eq. 6), or, in the token-sum form (Eq. 7),
    // acc * sx * s - t_X * (z * s) in FP32 with `rs` carrying the bits of t_X.
    const bool token_sum = !GROUP && OUT == OUT_FP16 && p.token_sum;
    if constexpr (!GROUP) {
        if (!token_sum) {
#pragma unroll
            for (int j = 0; j < 4; ++j) t[j] -= zn[j] * rs;
        }
    }
    if constexpr (OUT == OUT_I32) {
        *reinterpret_cast<int4*>(p.out32 + (size_t)m * p.N + n0) = make_int4(t[0], t[1], t[2], t[3]);
    } else {
        const float txm = __int_as_float(rs);
        uint32_t h[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            float ra = (float)t[2 * j] * (sxm * sn[2 * j]), rb = (float)t[2 * j + 1] * (sxm * sn[2 * j + 1]);
            if (token_sum) {
                ra -= txm * ((float)zn[2 * j] * sn[2 * j]);
                rb -= txm * ((float)zn[2 * j + 1] * sn[2 * j + 1]);
            }
            const __half a = __float2half_rn(ra);
            const __half b = __float2half_rn(rb);
            h[j] = (uint32_t)__half_as_ushort(a) | ((uint32_t)__half_as_ushort(b) << 16);
        }
        *reinterpret_cast<uint2*>(p.out16 + (size_t)m * p.N + n0) = make_uint2(h[0], h[1]);
    }
}


// qoq_gemm_astat.hip: the activation-stationary kernels for token tiles of 16, 32 and 64 (tile_m codes 69, 70, 71).
// `nwg` workgroups per token tile and k-slice share the layer's 16-channel fragments; p.S k-slices of p.gps groups.
hipError_t launch_astat(const GemmDev& p, int tile_m, int nwg, bool group, bool fp16, hipStream_t s);
// Largest number of quantization groups one workgroup of that kernel can keep resident for `tile` tokens.
int astat_max_groups(int tile);
// The same for sixteen waves and sixteen tokens.
int astat_deep_groups();
// The 16-token kernel that quantizes its tokens itself (quantizer and GEMM in one launch), for what astat_linear_takes.
bool astat_linear_takes(int64_t M, int64_t K);
hipError_t launch_astat_linear(const GemmDev& p, const void* x, int8_t* qx, void* sx, int32_t* rowsum, bool group, hipStream_t s);

// qoq_gemm_mma16.hip: the compute-bound kernel with 16x16x64 matrix instructions, tiles of 128 tokens x 256 or 192 channels
// (tile_m code 132, and 131 without k-slices).
hipError_t launch_mma16(const GemmDev& p, int channels, bool group, bool fp16, hipStream_t s);

// qoq_gemm_mma8.h: eight waves on one output tile of 256 or 128 channels and 16 mf tokens (tile_m code 130); one
// translation unit per mode and width, since each compiles seven kernels.
hipError_t launch_mma8_group_256(const GemmDev& p, int mf, hipStream_t s);
hipError_t launch_mma8_group_128(const GemmDev& p, int mf, hipStream_t s);
hipError_t launch_mma8_channel_256(const GemmDev& p, int mf, hipStream_t s);
hipError_t launch_mma8_channel_128(const GemmDev& p, int mf, hipStream_t s);

}  // namespace qoq
