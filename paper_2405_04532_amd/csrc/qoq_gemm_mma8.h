// W4A8 GEMM kernel for gfx950 with eight waves, two per SIMD, on one output tile that they also split along K (tile code 130):
// 16 MF tokens (MF = 3 ... 9) x 64 WC channels, WC = 2, or 4 where tiles of 128 channels would need more than a round of workgroups.  For token counts between the decode and the
// compute-bound kernels, for layers whose 128- or 256-token tiles leave compute units idle, and for ragged token counts:
// the tokens are cut into equal tiles of a multiple of 16 rows, so 130 tokens are multiplied as 144 rows where 64-token
// tiles take 192, 389 as 432 and not 512.
//
// What binds here.  An INT8 operand of 16 channels is dequantized by sixteen vector instructions and meets the MF token fragments
// of its wave; two vector instructions fit beside a 16-cycle v_mfma_i32_16x16x64_i8 (measured: a third costs 4 cycles), so
// a wave wants many token fragments, and no two waves may dequantize the same weights.  Hence all eight waves
// take all token fragments; they split the channels WC ways and the k-steps of 64 WK = 8 / WC ways.  Small output tiles
// then still keep the matrix cores of a compute unit busy: 1024 tokens x 4096 channels are 256 tiles of 128 x 128.  The WK partial
// sums of an output meet in LDS after the loop (about 0.5 us for two, 1.5 us for four).  The copies are bound by what a compute
// unit keeps in flight (about 32 KiB), i.e. by latency: 46 bytes per ns beyond L2.  Per group of a 128 x 128 tile the loop
// takes 0.37 us with a few workgroups on the chip (0.21 at the matrix cores' peak; 0.31 without copies, 0.25 without the
// dequantizer), 0.5 us with 256.
// Measured against the plans before (us, weights from memory): per channel 130 x 4096 x 28672 32.0 -> 25.5, 389 x 11008 x 4096
// 34.9 -> 32.6, 515 x 28672 x 8192 182 -> 120, 1024 x 4096 x 4096 26.2 -> 23.7, 150 x 8704 x 7744 35.6 -> 22.4.
//
// Copies are global->LDS DMA into a ring of R slabs.  Slab b holds bundle b: the activations of stage b (a stage is WK k-steps,
// one or two quantization groups) and the packed weights and metadata of stage b + 1, because operands are dequantized
// ahead of the matrix instructions.  Activation copies move eight tokens x one whole 128-byte line.
// A stage is taken in two halves, two channel fragments each, token fragment by token fragment: a chunk is one matrix
// instruction, its share of the vector instructions that make the other half's operands, at most one or two LDS reads and at most one
// copy, closed by a scheduling barrier.  One barrier per stage, in front of its second half: every wave has waited for its own
// copies of bundle b + 1 and for its reads of slab b, so behind the barrier b + 1 may be read and slab b is refilled with bundle b + R.
// grid = (token tiles * channel tiles, k-slices); k-slices meet in the workspace as in the other compute-bound kernels.
#pragma once
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "qoq_gemm_common.h"
#include "qoq_layout.h"

namespace qoq {
namespace {

constexpr int kM8Threads = 512, kM8Waves = 8;
constexpr int kNF = 4;                              // 16-channel fragments of a wave

// f(integral_constant 0), f(1), ... f(N - 1): a loop that is unrolled whatever its size
template <class F, int... I>
__device__ __forceinline__ void unrolled_over(F&& f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>()), ...); }
template <int N, class F>
__device__ __forceinline__ void unrolled(F&& f) { unrolled_over(f, std::make_integer_sequence<int, N>()); }

template <int MF, int WC>
struct M8Shape {
    static constexpr int WK = kM8Waves / WC;        // waves that share an output, one k-step of a stage each
    static constexpr int SG = WK / 2;               // quantization groups per stage
    static_assert(WK == 2 || WK == 4, "256 or 128 channels");
    static constexpr int TM = 16 * MF, TN = 64 * WC;
    static constexpr int ABytes = SG * TM * 128, WBytes = SG * TN * 64, MBytes = 512, Slab = ABytes + WBytes + MBytes;
    static constexpr int EBytes = 2304;             // epilogue constants: 256 x (sx, s, rowsum, zero)
    static constexpr int R = 4 * Slab + EBytes <= 160 * 1024 ? 4 : 3;       // slabs of the ring
    static constexpr int XBytes = 4 * kNF * MF * 1024;                      // exchange of partial sums: four pairs of waves
    static constexpr int RingBytes = R * Slab > XBytes ? R * Slab : XBytes;
    static_assert(RingBytes + EBytes <= 160 * 1024, "LDS of a compute unit");
};

template <bool GROUP, int MF, int WC>
__global__ __launch_bounds__(kM8Threads) __attribute__((amdgpu_waves_per_eu(2, 2))) void mma8_kernel(QOQ_GEMM_PARAMS, GemmTail tail)
{
    const GemmDev p = gemm_dev(QOQ_GEMM_ARGS, tail);
    using Sh = M8Shape<MF, WC>;
    constexpr int WK = Sh::WK, SG = Sh::SG, TM = Sh::TM, TN = Sh::TN, R = Sh::R;
    constexpr int kUnits = TN / 16;                 // weight units of a group
    static_assert(SG * kUnits == 2 * kM8Waves, "two weight copies per wave and stage");
    __shared__ __attribute__((aligned(16))) char ring[Sh::RingBytes];
    __shared__ __attribute__((aligned(16))) char ering[Sh::EBytes];   // sx[256] fp16 | s[256] fp16 | rowsum[256] | zeros[256]

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kw = wave % WK, wc = wave / WK;
    const int G = p.G;
    const int slice = blockIdx.y;
    const int g_first = slice * p.gps, Gs = min(G - g_first, p.gps), g_last = g_first + Gs - 1;
    const int T = (Gs + SG - 1) / SG;               // stages
    // Workgroup -> tile: consecutive ids land on consecutive XCDs; each XCD walks panels of four token tiles column by column.
    const int n_tiles = (p.N + TN - 1) / TN, m_tiles = (p.M + TM - 1) / TM;
    int tm, tn;
    {
        const int tiles = n_tiles * m_tiles, xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
        const int q = tiles >> 3, r = tiles & 7;
        const int L = xcd * q + min(xcd, r) + slot;      // slot < q + (xcd < r) because blockIdx.x < tiles
        constexpr int kPanel = 4;
        const int per_panel = kPanel * n_tiles;
        const int panel = L / per_panel;
        const int rows = min(kPanel, m_tiles - panel * kPanel);
        const int rem = L - panel * per_panel;
        tn = rem / rows;
        tm = panel * kPanel + (rem - tn * rows);
    }
    const int m_base = tm * TM, n_base = tn * TN;
    const int nf_base = tn * kUnits;                // first 16-row fragment (unit row) of the tile
    const int nf_total = p.N / 16;

    // ---- copy role.  Copy i of a stage's activations = eight token rows of one group; lane 8r+c fetches 16-byte chunk
    // c ^ row_swizzle of row r.  Wave w makes copies w, w + 8, ..., two of the stage's sixteen weight units, and waves 6
    // and 7 half of the metadata each.  The waves that make one copy more than others are never the same for two reasons
    // (kARem <= 6), so a wave's number of copies per stage is kBase or kBase + 1.
    constexpr int kACopies = SG * TM / 8, kAFull = kACopies / kM8Waves, kARem = kACopies % kM8Waves;
    constexpr int kAMost = kAFull + (kARem ? 1 : 0), kBase = kAFull + 2, kCopySlots = kAMost + 3;
    static_assert(kARem <= 6 && (R - 1) * (kBase + 1) < 64, "a wave makes at most one more, vmcnt range");
    static_assert(kCopySlots <= 2 * MF, "a copy per chunk of a half");
    const bool a_more = wave < kARem, m_copy = GROUP && wave >= 6, more = a_more || m_copy;
    uint32_t a_voff[kAMost], a_dst[kAMost];
    int a_sg[kAMost];
    const uint32_t ring0 = (uint32_t)(uintptr_t)&ring[0];
    {
        const int r = lane >> 3, c = lane & 7;
#pragma unroll
        for (int k = 0; k < kAMost; ++k) {
            const int i = min(k * kM8Waves + wave, kACopies - 1);
            const int rb = i % (TM / 8);
            a_sg[k] = i / (TM / 8);
            const int row = min(m_base + rb * 8 + r, p.M - 1);               // rows past M repeat the last one
            a_voff[k] = (uint32_t)row * (uint32_t)p.K + (uint32_t)((c ^ row_swizzle(((rb & 1) << 3) | r)) * 16);
            a_dst[k] = ring0 + (uint32_t)(a_sg[k] * TM * 128 + rb * 1024);
        }
    }
    const uint32_t w_voff = (uint32_t)lane * 16u;
    const char* abase = reinterpret_cast<const char*>(p.qx);
    const char* wrow[2];
    const int w_sg = wave * 2 / kUnits, w_unit = wave * 2 % kUnits;
#pragma unroll
    for (int u = 0; u < 2; ++u)                     // units past N repeat the last one; their results are never stored
        wrow[u] = reinterpret_cast<const char*>(p.codes) + (size_t)min(nf_base + w_unit + u, nf_total - 1) * G * 1024;
    const int m_unit = SG == 2 ? 0 : (wave & 1) * 8, m_sg = SG == 2 ? wave & 1 : 0;     // waves 6 and 7
    const uint32_t m_voff = (uint32_t)min(nf_base + m_unit + (lane >> 3), nf_total - 1) * 32u + (uint32_t)(lane & 7) * 4u;
    const char* mrow = reinterpret_cast<const char*>(p.meta);
    const size_t m_g_stride = (size_t)nf_total * 32;
    int ca = g_first, cw = g_first;                 // first group of the next stage to copy, activations and weights
    auto group_at = [&](int g) { return min(g, g_last); };                   // past the slice: its last group again
    auto copy = [&](int k, uint32_t slab) __attribute__((always_inline)) {   // the k-th copy of a bundle
        if (k < kAMost) {
            if (k < kAFull || a_more) dma16(abase + (size_t)group_at(ca + a_sg[k]) * kGroup, a_voff[k], a_dst[k] + slab);
        } else if (k < kAMost + 2) {
            const int u = k - kAMost;
            dma16(wrow[u] + (size_t)group_at(cw + w_sg) * 1024, w_voff, ring0 + slab + (uint32_t)(Sh::ABytes + (wave * 2 + u) * 1024));
        } else if (m_copy) {
            dma4(mrow + (size_t)group_at(cw + m_sg) * m_g_stride, m_voff, ring0 + slab + (uint32_t)(Sh::ABytes + Sh::WBytes + (wave - 6) * 256));
        }
    };
    // Epilogue constants first, the oldest entries of each wave's copy queue: 256 of each whatever the tile, indices
    // past M / N repeat the last valid dword and are never used.
    {
        const uint32_t e_dst = (uint32_t)(uintptr_t)&ering[0];
        if (p.out16) {
            if (wave < 2)
                dma4(reinterpret_cast<const char*>(p.sx) + (size_t)m_base * 2, (uint32_t)min(wave * 64 + lane, (p.M - m_base - 1) >> 1) * 4u,
                     e_dst + (uint32_t)wave * 256u);
            else if (wave < 4)
                dma4(reinterpret_cast<const char*>(p.scales) + (size_t)n_base * 2,
                     (uint32_t)min((wave - 2) * 64 + lane, ((p.N - n_base) >> 1) - 1) * 4u, e_dst + 512u + (uint32_t)(wave - 2) * 256u);
        }
        if (!GROUP) {
            if (wave >= 4)
                dma4(reinterpret_cast<const char*>(p.rowsum) + (size_t)m_base * 4, (uint32_t)min((wave - 4) * 64 + lane, p.M - m_base - 1) * 4u,
                     e_dst + 1024u + (uint32_t)(wave - 4) * 256u);
            else if (wave == 0)
                dma4(reinterpret_cast<const char*>(p.zeros) + (size_t)n_base, (uint32_t)min(lane, ((p.N - n_base) >> 2) - 1) * 4u,
                     e_dst + 2048u);
        }
    }
    // prologue: the first stage's weights (into the last slab), then all bundles but the last of the ring
#pragma unroll
    for (int k = kAMost; k < kCopySlots; ++k) copy(k, (uint32_t)((R - 1) * Sh::Slab));
    cw += SG;
    auto advance = [&]() __attribute__((always_inline)) { ca += SG; cw += SG; };
#pragma unroll
    for (int st = 0; st < R - 1; ++st)
        if (st < T) {
#pragma unroll
            for (int k = 0; k < kCopySlots; ++k) copy(k, (uint32_t)(st * Sh::Slab));
            advance();
        }
    // wait until at most the copies of `younger` bundles (R - 2 at most) are outstanding
    auto wait_bundles = [&](int younger) __attribute__((always_inline)) {
        if (younger >= R - 2) { if (more) wait_vmcnt<(R - 2) * (kBase + 1)>(); else wait_vmcnt<(R - 2) * kBase>(); }
        else if (R > 3 && younger == 1) { if (more) wait_vmcnt<kBase + 1>(); else wait_vmcnt<kBase>(); }
        else wait_vmcnt<0>();
    };

    // ---- compute role
    const int r16 = lane & 15, kb = lane >> 4;
    v4i acc[kNF][MF];                               // [channel fragment][token fragment]
#pragma unroll
    for (int a = 0; a < kNF; ++a)
#pragma unroll
        for (int b = 0; b < MF; ++b) acc[a][b] = (v4i){0, 0, 0, 0};
    // this wave's k-step: half my_half of group my_sg of every stage; byte offsets of its operands inside a slab
    const int my_sg = kw >> 1, my_half = kw & 1;
    const uint32_t a_rd = (uint32_t)(my_sg * TM * 128 + r16 * 128 + (((4 * my_half + kb) ^ row_swizzle(r16)) * 16));
    const uint32_t w_rd = (uint32_t)(Sh::ABytes + (my_sg * kUnits + wc * kNF) * 1024 + lane * 16 + my_half * 8);
    const uint32_t m_rd = (uint32_t)(Sh::ABytes + Sh::WBytes + my_sg * 256 + wc * kNF * 32 + (r16 >> 1) * 4);
    const uint32_t sel_s = r16 & 1 ? 0x0c020c02u : 0x0c000c00u, sel_b = r16 & 1 ? 0x03030303u : 0x01010101u;   // s1 in both lanes, bias in all bytes
    auto lds_a = [&](uint32_t slab, int tf) __attribute__((always_inline)) {
        return as_v4i(*reinterpret_cast<const uint4*>(ring + slab + a_rd + tf * 2048));
    };
    uint2 rq[kNF];                                  // packed words and metadata of this stage's, later the next one's fragments
    uint32_t mt[kNF];
    auto load_w = [&](uint32_t slab, int f) __attribute__((always_inline)) {
        rq[f] = *reinterpret_cast<const uint2*>(ring + slab + w_rd + f * 1024);
        mt[f] = GROUP ? *reinterpret_cast<const uint32_t*>(ring + slab + m_rd + f * 32) : 0u;
    };
    // A stage whose second group lies past the slice: the waves of that group multiply by zero.
    uint32_t nib = 0x0F0F0F0Fu, sign = 0x80808080u, bias_keep = 0xFFFFFFFFu;
    auto set_live = [&](int st) __attribute__((always_inline)) {
        if constexpr (SG == 2) {
            const bool live = 2 * st + my_sg < Gs;
            nib = live ? 0x0F0F0F0Fu : 0u;
            sign = live ? 0x80808080u : 0u;
            bias_keep = live ? 0xFFFFFFFFu : 0u;
        }
    };
    v4i w_op[2][2], at[MF];                         // operands of each half; token fragments, each replaced behind its last use
    uint32_t dq[4], S = 0, B = 0;
    // One of the sixteen vector instructions (per-channel mode: six of them) that make operand f, in an order in which none
    // feeds the one behind it.  pin: the value exists here; without it the compiler moves the operand to its first use.
    auto pin = [](uint32_t x) __attribute__((always_inline)) { asm volatile("" : "+v"(x)); return x; };
    auto dequant_op = [&](auto o_, int f, v4i& w) __attribute__((always_inline)) {
        constexpr int o = decltype(o_)::value;
        auto mad = [&](int d) __attribute__((always_inline)) { if (GROUP) dq[d] = pin(pk_mad_u16(dq[d], S, B)); };
        auto flip = [&](int d) __attribute__((always_inline)) { return (int)(GROUP ? pin(dq[d] ^ sign) : dq[d]); };
        if constexpr (o == 0) { if (GROUP) S = pin(__builtin_amdgcn_perm(mt[f], mt[f], sel_s)); }
        if constexpr (o == 1) {
            if (GROUP) {
                B = __builtin_amdgcn_perm(mt[f], mt[f], sel_b);
                if (SG == 2) B &= bias_keep;
                B = pin(B);
            }
        }
        if constexpr (o == 2) dq[0] = pin(rq[f].x & nib);
        if constexpr (o == 3) dq[1] = pin(rq[f].x >> 4);
        if constexpr (o == 4) mad(0);
        if constexpr (o == 5) dq[1] = pin(dq[1] & nib);
        if constexpr (o == 6) w.x = flip(0);
        if constexpr (o == 7) mad(1);
        if constexpr (o == 8) dq[2] = pin(rq[f].y & nib);
        if constexpr (o == 9) dq[3] = pin(rq[f].y >> 4);
        if constexpr (o == 10) mad(2);
        if constexpr (o == 11) dq[3] = pin(dq[3] & nib);
        if constexpr (o == 12) w.y = flip(1);
        if constexpr (o == 13) mad(3);
        if constexpr (o == 14) w.z = flip(2);
        if constexpr (o == 15) w.w = flip(3);
    };
    constexpr int kLastWord = 25 * MF / 16 + 1;     // chunk behind the one that takes the last bits of rq[3] in a first half
    static_assert(kLastWord < 2 * MF, "all words are read before the barrier");

    wait_bundles(min(T, R - 1) - 1);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    set_live(0);
#pragma unroll
    for (int tf = 0; tf < MF; ++tf) at[tf] = lds_a(0, tf);
#pragma unroll
    for (int f = 0; f < kNF; ++f) load_w((uint32_t)((R - 1) * Sh::Slab), f);
    unrolled<32>([&](auto i_) __attribute__((always_inline)) {
        constexpr int i = decltype(i_)::value;
        dequant_op(std::integral_constant<int, i % 16>(), i / 16, w_op[0][i / 16]);
    });
    w_op[1][0] = w_op[1][1] = (v4i){0, 0, 0, 0};
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();                   // everybody has read the first weights: their slab takes the ring's last bundle
    asm volatile("" ::: "memory");
    if (R - 1 < T) {
#pragma unroll
        for (int k = 0; k < kCopySlots; ++k) copy(k, (uint32_t)((R - 1) * Sh::Slab));
        advance();
    }

    uint32_t slab = 0;                              // byte offset of this stage's slab
    auto stage = [&](int st, auto steady_) __attribute__((always_inline)) {
        constexpr bool steady = decltype(steady_)::value;          // the ring is refilled without a question
        const uint32_t slab_next = slab + Sh::Slab == R * Sh::Slab ? 0u : slab + (uint32_t)Sh::Slab;
        const bool refill = steady || st + R < T;
        unrolled<2>([&](auto h_) __attribute__((always_inline)) {
            constexpr int h = decltype(h_)::value;
            if constexpr (h == 1) {
                set_live(st + 1);                                  // the operands made from here on are the next stage's
                if (steady) wait_bundles(R - 2); else wait_bundles(T - 2 - st);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
            unrolled<2 * MF>([&](auto c_) __attribute__((always_inline)) {
                constexpr int c = decltype(c_)::value, tf = c >> 1, e = c & 1;
                acc[2 * h + e][tf] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w_op[h][e], at[tf], acc[2 * h + e][tf], 0, 0, 0);
                constexpr int first = (16 * c + MF - 1) / MF, behind = (16 * (c + 1) + MF - 1) / MF;   // this chunk's share of 32
                unrolled<behind - first>([&](auto i_) __attribute__((always_inline)) {
                    constexpr int i = first + decltype(i_)::value;
                    dequant_op(std::integral_constant<int, i % 16>(), 2 * (1 - h) + i / 16, w_op[1 - h][i / 16]);
                });
                if constexpr (h == 0) {                            // the next stage's weights, each word behind the last use of the old one
                    if constexpr (c < 2) load_w(slab, c);
                    if constexpr (c == MF + 1) load_w(slab, 2);
                    if constexpr (c == kLastWord) load_w(slab, 3);
                } else {
                    if constexpr (e == 1) at[tf] = lds_a(slab_next, tf);
                    if constexpr (c < kCopySlots) { if (refill) copy(c, slab); }
                }
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        advance();
        slab = slab_next;
    };
    int st = 0;
    for (; st < T - R; ++st) stage(st, std::true_type());
    for (; st < T; ++st) stage(st, std::false_type());

    // ---- epilogue
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    const int tile_id = tm * n_tiles + tn;
    const __half* e_sx = reinterpret_cast<const __half*>(ering);
    const __half* e_sn = e_sx + 256;
    const int* e_rs = reinterpret_cast<const int*>(ering + 1024);
    const uint8_t* e_zn = reinterpret_cast<const uint8_t*>(ering + 2048);
    int* s_last = reinterpret_cast<int*>(ring);

    auto finish = [&](auto lo_, auto hi_) __attribute__((always_inline)) {   // token fragments lo .. hi - 1 are this wave's
        constexpr int lo = decltype(lo_)::value, hi = decltype(hi_)::value, CNT = hi - lo;
        if (p.S > 1) {
            // k-slices: partial sums written through to memory, a counter per tile elects the last to arrive, which adds
            // the others' (integer sums: exact, order independent) and alone runs the epilogue; the counter is left at zero.
            constexpr int NJ = kNF * ((MF + WK - 1) / WK);     // int4 per thread in a partial tile
            int4* mine = p.parts + ((size_t)(tile_id * p.S + slice) * NJ) * kM8Threads + threadIdx.x;
#pragma unroll
            for (int j = 0; j < kNF * CNT; ++j) store_sc1(mine + (size_t)j * kM8Threads, acc[j % kNF][lo + j / kNF]);
            wait_vmcnt<0>();
            __syncthreads();
            if (threadIdx.x == 0) {
                int* ctr = p.counters + tile_id;
                const int old = __hip_atomic_fetch_add(ctr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                *s_last = old == p.S - 1;
                if (old == p.S - 1) __hip_atomic_store(ctr, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            __syncthreads();
            if (!*s_last) return;
            for (int s2 = 0; s2 < p.S; ++s2) {
                if (s2 == slice) continue;
                const __amdgpu_buffer_rsrc_t theirs =
                    part_rsrc(p.parts + ((size_t)(tile_id * p.S + s2) * NJ) * kM8Threads, NJ * kM8Threads * 16);
#pragma unroll
                for (int j = 0; j < kNF * CNT; ++j) acc[j % kNF][lo + j / kNF] += load_sc1(theirs, (int)threadIdx.x * 16, j * kM8Threads * 16);
            }
        }
        // Lane (token r16, row quad kb) of fragment f holds logical channels 16 kb + 4 f + v of the wave's 64: 16 consecutive
        // channels of a token, one row segment of 32 bytes.
        const int nl = wc * 64 + 16 * kb, n0 = n_base + nl;
        if (n0 >= p.N) return;                       // N % 64 == 0: a segment is all in or all out
        const bool fp16 = p.out16 != nullptr, token_sum = !GROUP && fp16 && p.token_sum;   // Eq. 7 form: rowsum holds the bits of t_X
        float sn[16];
        int zn[16];
#pragma unroll
        for (int x = 0; x < 16; ++x) { sn[x] = __half2float(e_sn[nl + x]); zn[x] = GROUP ? 0 : (int)e_zn[nl + x]; }
#pragma unroll
        for (int tf = lo; tf < hi; ++tf) {
            const int ml = tf * 16 + r16;
            const int m = m_base + ml;
            if (m >= p.M) continue;
            const int rs = GROUP ? 0 : e_rs[ml];
            int t[16];
#pragma unroll
            for (int x = 0; x < 16; ++x) {
                t[x] = acc[x >> 2][tf][x & 3];
                if (!GROUP && !token_sum) t[x] -= zn[x] * rs;
            }
            if (!fp16) {
                int4* dst = reinterpret_cast<int4*>(p.out32 + (size_t)m * p.N + n0);
#pragma unroll
                for (int q = 0; q < 4; ++q) dst[q] = make_int4(t[4 * q], t[4 * q + 1], t[4 * q + 2], t[4 * q + 3]);
                continue;
            }
            const float sxm = __half2float(e_sx[ml]), txm = __int_as_float(rs);
            uint32_t h[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                float ra = (float)t[2 * j] * (sxm * sn[2 * j]), rb = (float)t[2 * j + 1] * (sxm * sn[2 * j + 1]);
                if (token_sum) {
                    ra -= txm * ((float)zn[2 * j] * sn[2 * j]);
                    rb -= txm * ((float)zn[2 * j + 1] * sn[2 * j + 1]);
                }
                h[j] = (uint32_t)__half_as_ushort(__float2half_rn(ra)) | ((uint32_t)__half_as_ushort(__float2half_rn(rb)) << 16);
            }
            uint4* dst = reinterpret_cast<uint4*>(p.out16 + (size_t)m * p.N + n0);
#pragma unroll
            for (int q = 0; q < 2; ++q) dst[q] = make_uint4(h[4 * q], h[4 * q + 1], h[4 * q + 2], h[4 * q + 3]);
        }
    };
    // The waves that share an output meet in LDS: of token fragments lo .. hi - 1 a wave keeps lo .. mid - 1 where `bit` of its
    // number is clear, else mid .. hi - 1, gives the others to the wave `wave ^ bit` and adds what that one gives.  The branches
    // are the same for a whole wave, and every wave passes the same number of barriers whichever it takes.
    int4* xbuf = reinterpret_cast<int4*>(ring);
    auto exchange = [&](auto lo_, auto hi_, int bit, auto&& then) __attribute__((always_inline)) {
        constexpr int lo = decltype(lo_)::value, hi = decltype(hi_)::value, mid = (lo + hi + 1) / 2;
        // a pair's area: what the wave with its bit clear gives (the upper part), then what the other one gives
        constexpr int kUpper = kNF * (hi - mid) * 64;
        const int low = wave & (bit - 1), pair = (((wave >> 1) & ~(bit - 1)) | low) * (kNF * MF * 64);
        __syncthreads();
        auto give = [&](auto a_, auto b_) __attribute__((always_inline)) {
            constexpr int a = decltype(a_)::value, b = decltype(b_)::value;
#pragma unroll
            for (int j = 0; j < kNF * (b - a); ++j) {
                const v4i v = acc[j % kNF][a + j / kNF];
                xbuf[pair + (a == lo ? kUpper : 0) + j * 64 + lane] = make_int4(v.x, v.y, v.z, v.w);
            }
        };
        auto take = [&](auto a_, auto b_) __attribute__((always_inline)) {
            constexpr int a = decltype(a_)::value, b = decltype(b_)::value;
#pragma unroll
            for (int j = 0; j < kNF * (b - a); ++j) {
                const int4 v = xbuf[pair + (a == lo ? kUpper : 0) + j * 64 + lane];
                acc[j % kNF][a + j / kNF] += (v4i){v.x, v.y, v.z, v.w};
            }
        };
        using L = std::integral_constant<int, lo>;
        using M = std::integral_constant<int, mid>;
        using H = std::integral_constant<int, hi>;
        if (!(wave & bit)) give(M(), H()); else give(L(), M());
        __syncthreads();
        if (!(wave & bit)) { take(L(), M()); then(L(), M()); }
        else { take(M(), H()); then(M(), H()); }
    };
    using Zero = std::integral_constant<int, 0>;
    using All = std::integral_constant<int, MF>;
    auto last = [&](auto lo, auto hi) __attribute__((always_inline)) { __syncthreads(); finish(lo, hi); };
    if constexpr (WK == 2) exchange(Zero(), All(), 1, last);
    else exchange(Zero(), All(), 2, [&](auto lo, auto hi) __attribute__((always_inline)) { exchange(lo, hi, 1, last); });
}

template <bool GROUP, int WC>
hipError_t launch_mma8_tile(const GemmDev& p, int mf, hipStream_t s)
{
    const int tm = 16 * mf, tn = 64 * WC;
    const dim3 grid((unsigned)(((p.N + tn - 1) / tn) * ((p.M + tm - 1) / tm)), (unsigned)p.S);
    switch (mf) {
        case 3: launch_gemm_kernel(mma8_kernel<GROUP, 3, WC>, grid, kM8Threads, s, p); break;
        case 4: launch_gemm_kernel(mma8_kernel<GROUP, 4, WC>, grid, kM8Threads, s, p); break;
        case 5: launch_gemm_kernel(mma8_kernel<GROUP, 5, WC>, grid, kM8Threads, s, p); break;
        case 6: launch_gemm_kernel(mma8_kernel<GROUP, 6, WC>, grid, kM8Threads, s, p); break;
        case 7: launch_gemm_kernel(mma8_kernel<GROUP, 7, WC>, grid, kM8Threads, s, p); break;
        case 8: launch_gemm_kernel(mma8_kernel<GROUP, 8, WC>, grid, kM8Threads, s, p); break;
        case 9: launch_gemm_kernel(mma8_kernel<GROUP, 9, WC>, grid, kM8Threads, s, p); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace
}  // namespace qoq
