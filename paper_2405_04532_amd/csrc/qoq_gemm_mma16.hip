// Compute-bound W4A8 GEMM kernel for gfx950 (Section 5.2 of arXiv 2405.04532): tiles of 128 tokens x 256 channels with two
// workgroups per compute unit (tile code 132).
//
// Four waves per workgroup; a wave owns 128 tokens x 64 channels in 4 x 8 accumulator tiles of v_mfma_i32_16x16x64_i8 (128
// registers per lane).  At this occupancy the matrix cores are power limited, and the 16x16x64 instruction costs less
// energy per multiply-add than 32x32x32: with the operand statistics of this GEMM and nothing else going on they sustain
// 4.2 POP/s against 3.6, with the dequantizer and the LDS reads of this loop beside them 3.3 against 2.95.  Measured against
// the same tile on 32x32x32 (qoq_gemm.hip's loop, which this kernel replaced here): Llama-3-70B gate+up at 2048 tokens 734 us
// against 775, O 111 against 118, Llama-2-7B gate+up at 1024 tokens 88 against 92, per-channel 4096 x 4096 x 12288 148 against
// 173 (2.8 POP/s).  With one workgroup per compute unit the 32x32x32 loop is kept: there a chunk of this one (a matrix
// instruction of 16 cycles and its share of everything else, from one wave) takes more issue cycles than the matrix
// instruction hides (300 x 4096 x 12288: 31.0 us against 28.6).
//
// The main loop is software pipelined by hand into "chunks" of one MFMA (16 cycles) plus what fits in its shadow: two
// of the fourteen vector instructions that dequantize the NEXT weight operand (an operand meets all eight token
// fragments of the wave: 1.75 vector instructions per MFMA), at most two LDS reads and at most one copy.  A scheduling
// barrier after every chunk keeps the compiler from regrouping them.
//
// Copies are global->LDS DMA.  Activations, packed weights (the 16-byte lane word covers both halves of a group) and
// metadata live in rings of two group slabs; an activation copy moves eight tokens x 128 k, i.e. whole cache
// lines.  The main loop works in half-group steps (k = 64); every half-stage's activations are read into registers
// during the half-stage before.  There is one barrier per group, early in its second half-stage: a wave
// first waits for its own copies of group g+1, all waves meet (that publishes g+1 and proves group g's slabs are
// no longer read), and the slabs of group g are refilled with group g+2.  While one workgroup waits for its copies or at its
// barrier, the other one's matrix instructions keep the pipe busy.  What is left above the ceiling is the copies: with
// the slabs loaded once and never refilled the loop runs at 3.2 POP/s (a quarter of that difference is L2 misses).
// grid = (m-tiles * n-tiles, k-slices).
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "qoq_internal.h"
#include "qoq_gemm_common.h"

namespace qoq {
namespace {

constexpr int kMmaThreads = 256;
constexpr int kMSlotBytes = 1024;                   // metadata: 256 B per copying wave
constexpr int kTileM = 128;                         // tokens
constexpr int kDepth = 2;                           // slabs of the rings: small enough for two workgroups per compute unit

// f(integral_constant 0), f(1), ... f(N - 1): a loop that is unrolled whatever its size
template <class F, int... I>
__device__ __forceinline__ void unrolled_over(F&& f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>()), ...); }
template <int N, class F>
__device__ __forceinline__ void unrolled(F&& f) { unrolled_over(f, std::make_integer_sequence<int, N>()); }

// kNF: 16-channel fragments of a wave = blocks of eight chunks per half-stage; 4 = tiles of 256 channels, 3 = of 192, which are never cut
// into k-slices
template <bool GROUP, int OUT, int kNF>
__global__ __launch_bounds__(kMmaThreads, 2) void mma16_kernel(QOQ_GEMM_PARAMS, GemmTail tail)
{
    const GemmDev p = gemm_dev(QOQ_GEMM_ARGS, tail);
    constexpr int kASlots = kDepth, kWSlots = kDepth;
    constexpr int TMt = kTileM, TNt = 64 * kNF;     // tile: tokens x channels
    constexpr int kABlocks = TMt / 16;              // 1 KiB blocks (16 tokens x 64 k) per activation slab
    constexpr int kUnits = TNt / 16;                // 1 KiB weight units per slab
    constexpr int kASlotBytes = 2 * kABlocks * 1024, kWSlotBytes = kUnits * 1024;   // a group of a tile: 128 B per token
    constexpr int kACopies = kABlocks / 4, kWCopies = kUnits / 4;     // per wave
    constexpr int NC = 8 * kNF;                     // chunks per half-stage
    constexpr int BAR = 8;                          // chunk in front of which the half-stage's barrier sits
    __shared__ __attribute__((aligned(16))) char aring[kASlots * kASlotBytes];
    __shared__ __attribute__((aligned(16))) char wring[kWSlots * kWSlotBytes];
    __shared__ __attribute__((aligned(16))) char mring[kWSlots * kMSlotBytes];
    __shared__ __attribute__((aligned(16))) char ering[2304];   // sx[256] fp16 | s[256] fp16 | rowsum[256] | zeros[256]

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int G = p.G;
    // split-k: blockIdx.y selects a run of p.gps groups; the slices of a tile meet in the workspace (below)
    const int slice = blockIdx.y;
    const int g_first = slice * p.gps, Gs = min(G - g_first, p.gps);
    // Workgroup -> tile.  Consecutive workgroup ids land on consecutive XCDs (8, each with its own L2), so
    // workgroup i is the (i / 8)-th of XCD i % 8.  Each XCD gets a contiguous run of a tile order that walks
    // panels of four token tiles column by column: the 64 tiles an XCD works on at a time form a 4 x 16 block
    // sharing 4 activation slabs and 16 weight slabs through that XCD's L2 (panels of 2, 8 and 16 measured no better).
    const int n_tiles = (p.N + TNt - 1) / TNt, m_tiles = (p.M + TMt - 1) / TMt;
    int tm, tn;
    {
        const int T = n_tiles * m_tiles, xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
        const int q = T >> 3, r = T & 7;
        const int L = xcd * q + min(xcd, r) + slot;      // slot < q + (xcd < r) because blockIdx.x < T
        constexpr int kPanel = 4;
        const int per_panel = kPanel * n_tiles;
        const int panel = L / per_panel;
        const int rows = min(kPanel, m_tiles - panel * kPanel);
        const int rem = L - panel * per_panel;
        tn = rem / rows;
        tm = panel * kPanel + (rem - tn * rows);
    }
    const int m_base = tm * TMt, n_base = tn * TNt;
    const int nf_base = tn * kUnits;                     // first 16-row fragment (unit row) of the tile
    const int nf_total = p.N / 16;

    // ---- copy role: wave w copies a quarter of the tile's tokens, weight units kWCopies*w.. and their metadata.
    // One activation copy = eight tokens x one whole quantization group: every eight lanes fetch one whole 128-byte
    // line (the vector cache works in whole lines: 16 tokens x 64 bytes per copy, half a line each, was measured to
    // cost it twice the requests for the same bytes).  Lane 8r+c fetches 16-byte chunk c ^ row_swizzle(r) of token
    // row r, which keeps the fragment reads free of bank conflicts.  The
    // copies of a group are issued in two halves, after the barriers of two consecutive half-stages.
    constexpr int kAll = 2 * kACopies + kWCopies + (GROUP ? 1 : 0);   // copies per wave and group
    static_assert(kDepth * kAll < 64, "vmcnt range");
    static_assert(kAll <= NC - BAR, "one copy per chunk after the barrier");
    static_assert(kACopies % 2 == 0, "copy t of either half starts at row 8 * (t & 1) modulo 16");
    uint32_t a_voff[2][kACopies];                      // [half of the group's copies][copy]
    {
        const int r = lane >> 3, c = lane & 7;
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
#pragma unroll
            for (int t = 0; t < kACopies; ++t) {
                const int row = min(m_base + ((wave * 2 + hf) * kACopies + t) * 8 + r, p.M - 1);   // rows past M repeat the last one
                a_voff[hf][t] = (uint32_t)row * (uint32_t)p.K + (uint32_t)((c ^ row_swizzle(((t & 1) << 3) | r)) * 16);   // (a wave's copies start at a multiple of 16 rows)
            }
    }
    const uint32_t w_voff = (uint32_t)lane * 16u;
    // metadata: 32 B per unit; lane l copies dword l % 8 of the wave's unit l / 8 (units past N repeat the last one,
    // lanes past the wave's units repeat its last dword)
    const int m_lane = min(lane, kWCopies * 8 - 1);
    const uint32_t m_voff = (uint32_t)min(nf_base + wave * kWCopies + (m_lane >> 3), nf_total - 1) * 32u + (uint32_t)(m_lane & 7) * 4u;
    const uint32_t a_dst = (uint32_t)(uintptr_t)&aring[0] + (uint32_t)(wave * 2 * kACopies) * 1024u;
    const uint32_t w_dst = (uint32_t)(uintptr_t)&wring[0] + (uint32_t)(wave * kWCopies) * 1024u;
    const uint32_t m_dst = (uint32_t)(uintptr_t)&mring[0] + (uint32_t)wave * 256u;
    const char* abase = reinterpret_cast<const char*>(p.qx);
    const char* wrow[kWCopies];
#pragma unroll
    for (int u = 0; u < kWCopies; ++u)   // units past N repeat the last one; their results are never stored
        wrow[u] = reinterpret_cast<const char*>(p.codes) + (size_t)min(nf_base + wave * kWCopies + u, nf_total - 1) * G * 1024;
    const char* mrow = reinterpret_cast<const char*>(p.meta);
    const size_t m_g_stride = (size_t)nf_total * 32;
    int ca = g_first, cw = g_first;   // next group of activations / weights to copy; past the end of the slice the last one is copied again into a free slab
    const int cw_last = g_first + Gs - 1;
    auto copy_a = [&](int t, int hf, int slot) {
        dma16(abase + (size_t)ca * kGroup, a_voff[hf][t], a_dst + (uint32_t)(slot * kASlotBytes + (hf * kACopies + t) * 1024));
    };
    auto copy_w = [&](int u, int slot) { dma16(wrow[u] + (size_t)cw * 1024, w_voff, w_dst + (uint32_t)(slot * kWSlotBytes + u * 1024)); };
    auto copy_m = [&](int slot) { if (GROUP) dma4(mrow + (size_t)cw * m_g_stride, m_voff, m_dst + (uint32_t)(slot * kMSlotBytes)); };
    auto adv_a = [&]() { ca = min(ca + 1, cw_last); };
    auto adv_w = [&]() { cw = min(cw + 1, cw_last); };
    // k-th copy a wave issues after a group's barrier: the next group but one, into the slabs the barrier has freed
    auto refill = [&](int k, int islot) {
        if (k < 2 * kACopies) copy_a(k % kACopies, k / kACopies, islot);
        else if (k < 2 * kACopies + kWCopies) copy_w(k - 2 * kACopies, islot);
        else if (k == 2 * kACopies + kWCopies) copy_m(islot);
    };

    // Epilogue constants of the tile (token scales, channel scales; per-channel mode: token sums, zero points)
    // are copied into LDS first of all, so they are the oldest entries of each wave's copy queue and cost no
    // separate wait.  256 entries of each are fetched whatever the tile shape; indices past M / N repeat the
    // last valid dword and are never used.
    {
        const uint32_t e_dst = (uint32_t)(uintptr_t)&ering[0];
        const int d = wave * 64 + lane;
        if (OUT == OUT_FP16) {
            if (wave < 2)      // waves 0, 1: 2 x 64 dwords = 256 token scales
                dma4(reinterpret_cast<const char*>(p.sx) + (size_t)m_base * 2, (uint32_t)min(d, (p.M - m_base - 1) >> 1) * 4u,
                     e_dst + (uint32_t)wave * 256u);
            else               // waves 2, 3: 256 channel scales
                dma4(reinterpret_cast<const char*>(p.scales) + (size_t)n_base * 2,
                     (uint32_t)min(d - 128, ((p.N - n_base) >> 1) - 1) * 4u, e_dst + 512u + (uint32_t)(wave - 2) * 256u);
        }
        if (!GROUP) {
            dma4(reinterpret_cast<const char*>(p.rowsum) + (size_t)m_base * 4, (uint32_t)min(d, p.M - m_base - 1) * 4u,
                 e_dst + 1024u + (uint32_t)wave * 256u);
            if (wave == 0)
                dma4(reinterpret_cast<const char*>(p.zeros) + (size_t)n_base, (uint32_t)min(lane, ((p.N - n_base) >> 2) - 1) * 4u,
                     e_dst + 2048u);
        }
    }

    // prologue: the first two groups, each in the order of the steady state
#pragma unroll
    for (int gg = 0; gg < kDepth; ++gg) {
#pragma unroll
        for (int k = 0; k < kAll; ++k) refill(k, gg);
        adv_a();
        adv_w();
    }

    // ---- compute role ---------------------------------------------------------------------------
    const int r16 = lane & 15, kb = lane >> 4;
    v4i acc[kNF][8];                                      // [channel fragment][token fragment]
#pragma unroll
    for (int a = 0; a < kNF; ++a)
#pragma unroll
        for (int b = 0; b < 8; ++b) acc[a][b] = (v4i){0, 0, 0, 0};

    // LDS byte offsets of this lane's operands inside a slab.
    //   activations, token fragment tf (+ tf * 2048), half hf of the group: token tf*16 + r16 -> row of 128
    //   bytes, 16-byte chunk (4hf + kb) ^ row_swizzle(r16)
    //   weights, unit u (1 KiB: lane word `lane`, both halves); metadata of that unit: 32 B in the 256 B of copying
    //   wave u / kWCopies
    uint32_t a_rd[2];
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) a_rd[hf] = (uint32_t)(r16 * 128 + (((4 * hf + kb) ^ row_swizzle(r16)) * 16));
    // A wave's fragments: the four of a 64-channel block, or with 192 channels its place in each of the three blocks.
    auto unit_of = [&](int f) { return kNF == 4 ? wave * 4 + f : f * 4 + wave; };
    const uint32_t w_rd = (uint32_t)(unit_of(0) * 1024 + lane * 16);
    auto lds_a = [&](uint32_t slab, int hf, int tf) {
        return as_v4i(*reinterpret_cast<const uint4*>(aring + slab + a_rd[hf] + tf * 2048));
    };
    auto lds_w = [&](uint32_t slab, int f) {
        return *reinterpret_cast<const uint4*>(wring + slab + w_rd + f * (kNF == 4 ? 1024 : 4096));
    };
    auto lds_m = [&](uint32_t slab, int f) {
        const int u = unit_of(f);
        return (uint32_t)*reinterpret_cast<const uint16_t*>(mring + slab + (u / kWCopies) * 256 + (u % kWCopies) * 32 + r16 * 2);
    };
    const uint32_t nib_mask = 0x0F0F0F0Fu, sign = 0x80808080u;
    auto src_dword = [&](const uint4& r, int half, int d) { return half == 0 ? (d < 2 ? r.x : r.y) : (d < 2 ? r.z : r.w); };

    // first barrier: group 0 has landed everywhere
    wait_vmcnt<(kDepth - 1) * kAll>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    uint32_t S[kNF], B[kNF], mt[kNF];
#pragma unroll
    for (int f = 0; f < kNF; ++f) {
        S[f] = B[f] = mt[f] = 0;
        if (GROUP) {
            mt[f] = lds_m(0, f);
            S[f] = __builtin_amdgcn_perm(mt[f], mt[f], 0x0c000c00u);
            B[f] = __builtin_amdgcn_perm(mt[f], mt[f], 0x01010101u);
        }
    }
    // Register-level pipeline.  rq[f]: lane word (both k-halves) of fragment f of a group; a word of the next group
    // replaces it in the second half-stage, after the barrier and after its last use.  at[s]: activations of
    // half-stage s, read during the half-stage before.  One operand is dequantized while the one before it is
    // multiplied with the eight token fragments.
    uint4 rq[kNF];
#pragma unroll
    for (int f = 0; f < kNF; ++f) rq[f] = lds_w(0, f);
    v4i at[2][8];
#pragma unroll
    for (int tf = 0; tf < 8; ++tf) { at[0][tf] = lds_a(0, 0, tf); at[1][tf] = (v4i){0, 0, 0, 0}; }
    v4i w_cur = dequant<GROUP>(rq[0].x, rq[0].y, S[0], B[0]), w_nxt = {0, 0, 0, 0};
    uint32_t dq[4] = {src_dword(rq[1], 0, 0) & nib_mask, 0, 0, 0};       // block 1 is one step ahead, as in the steady state

    int gs = 0;                                          // g % 2
    for (int g = 0; g < Gs; ++g) {
        const int gp1 = gs ^ 1;
        unrolled<2>([&](auto s_) __attribute__((always_inline)) {            // half-stage h = 2g + s
            constexpr int s = decltype(s_)::value;
            const uint32_t a_nxt = (uint32_t)((s == 0 ? gs : gp1) * kASlotBytes);   // slab of the next half-stage: half 1 - s of this / the next group
            const uint32_t w_next = (uint32_t)(gp1 * kWSlotBytes), m_nxt = (uint32_t)(gp1 * kMSlotBytes);
            unrolled<NC>([&](auto c_) __attribute__((always_inline)) {       // chunk = (block b = channel fragment, token fragment tf)
                constexpr int c = decltype(c_)::value, b = c >> 3, tf = c & 7;
                if constexpr (c == BAR && s == 1) {
                    // One barrier per group, in its second half-stage.  Before it a wave waits for its own copies of
                    // group g+1 and for its outstanding LDS reads; all waves meeting
                    // publishes group g+1 and proves that nobody reads group g's slabs any more (its second k-half
                    // went to registers during the first half-stage): they are refilled with group g+2.
                    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                }
                acc[b][tf] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w_cur, at[s][tf], acc[b][tf], 0, 0, 0);
                {   // one step of the next block's operand (14 vector instructions in eight chunks, ordered so that no
                    // result feeds the next instruction); the last chunk starts on the block after that
                    const int tb = b + 1, f = tb % kNF, half = tb >= kNF ? 1 - s : s;
                    const uint4& r = rq[f];
                    auto mad = [&](uint32_t x) { return GROUP ? pk_mad_u16(x, S[f], B[f]) : x; };
                    auto flip = [&](uint32_t x) { return (int)(GROUP ? x ^ sign : x); };
                    if (tf == 0) { dq[0] = mad(dq[0]); dq[1] = src_dword(r, half, 1) >> 4; }
                    if (tf == 1) { w_nxt.x = flip(dq[0]); dq[1] &= nib_mask; }
                    if (tf == 2) { dq[1] = mad(dq[1]); dq[2] = src_dword(r, half, 2) & nib_mask; }
                    if (tf == 3) { w_nxt.y = flip(dq[1]); dq[2] = mad(dq[2]); }
                    if (tf == 4) { w_nxt.z = flip(dq[2]); dq[3] = src_dword(r, half, 3) >> 4; }
                    if (tf == 5) dq[3] &= nib_mask;
                    if (tf == 6) dq[3] = mad(dq[3]);
                    if (tf == 7) {
                        w_nxt.w = flip(dq[3]);
                        dq[0] = src_dword(rq[(b + 2) % kNF], b + 2 >= kNF ? 1 - s : s, 0) & nib_mask;
                    }
                }
                if constexpr (s == 0) {
                    if constexpr (c >= 2 && c < 18 && !(c & 1)) at[1][(c - 2) >> 1] = lds_a(a_nxt, 1, (c - 2) >> 1);
                } else if constexpr (c >= BAR) {
                    constexpr int L = c - BAR;
                    // lane words of the next group: 0 and 1 are free since the barrier, 2 and 3 once their own block has begun
                    if constexpr (L < 2) rq[L] = lds_w(w_next, L);
                    else if constexpr (tf == 0) rq[b] = lds_w(w_next, b);
                    if constexpr (GROUP && L >= 2 && L < 2 + kNF) mt[L - 2] = lds_m(m_nxt, L - 2);
                    if constexpr (kNF == 4 && L >= 3 && L < 19 && (L & 1)) at[0][(L - 3) >> 1] = lds_a(a_nxt, 0, (L - 3) >> 1);
                    if constexpr (kNF == 3 && L >= 5 && L != 8 && L < 14) at[0][L - (L < 8 ? 5 : 6)] = lds_a(a_nxt, 0, L - (L < 8 ? 5 : 6));
                    // level-2 constants of the next group, each after the last use of the old one (block f - 1, step 6) and
                    // before its own (the last block's steps make the next half-stage's first operand)
                    constexpr int pf = kNF == 4 ? (c == 21 ? 0 : c == 22 ? 1 : c == 23 ? 2 : c == 27 ? 3 : -1) : (c == 15 ? 0 : c == 17 ? 1 : c == 18 ? 2 : -1);
                    if constexpr (GROUP && pf >= 0) {
                        S[pf] = __builtin_amdgcn_perm(mt[pf], mt[pf], 0x0c000c00u);
                        B[pf] = __builtin_amdgcn_perm(mt[pf], mt[pf], 0x01010101u);
                    }
                    refill(L, gs);                       // refill the slabs the barrier has just freed
                }
                if (tf == 7) w_cur = w_nxt;
                __builtin_amdgcn_sched_barrier(0);
            });
            if constexpr (s == 1) { adv_a(); adv_w(); }
        });
        gs = gp1;
    }

    wait_vmcnt<0>();   // the repeated tail copies still target the ring

    // ---- split-k: every slice writes its partial tile through to memory and bumps the tile's counter; the last
    // one to arrive adds the others' (integer sums: exact, order independent) and alone runs the epilogue.
    // Same fence-free hand-over as in the streaming kernels; the counter is left at zero for the next launch.
    if constexpr (kNF == 4)
    if (p.S > 1) {
        constexpr int NJ = kNF * 8;                      // int4 per thread in a partial tile
        const int tile_id = tm * n_tiles + tn;
        int4* mine = p.parts + ((size_t)(tile_id * p.S + slice) * NJ) * kMmaThreads + threadIdx.x;
#pragma unroll
        for (int j = 0; j < NJ; ++j) store_sc1(mine + (size_t)j * kMmaThreads, acc[j >> 3][j & 7]);
        wait_vmcnt<0>();
        __syncthreads();
        __shared__ int s_last;
        if (threadIdx.x == 0) {
            int* ctr = p.counters + tile_id;
            const int old = __hip_atomic_fetch_add(ctr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_last = old == p.S - 1;
            if (s_last) __hip_atomic_store(ctr, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (!s_last) return;
        for (int s2 = 0; s2 < p.S; ++s2) {
            if (s2 == slice) continue;
            const int4* theirs = p.parts + ((size_t)(tile_id * p.S + s2) * NJ) * kMmaThreads + threadIdx.x;
#pragma unroll
            for (int j0 = 0; j0 < NJ; j0 += 8) {           // four loads in flight: no plan cuts this kernel, only a forced one
                v4i t[8];
#pragma unroll
                for (int x = 0; x < 8; x += 4) load_sc1_and_wait(&t[x], theirs + (size_t)(j0 + x) * kMmaThreads, kMmaThreads);
#pragma unroll
                for (int x = 0; x < 8; ++x) acc[j0 >> 3][x] += t[x];
            }
        }
    }

    const __half* e_sx = reinterpret_cast<const __half*>(ering);
    const __half* e_sn = e_sx + 256;
    const int* e_rs = reinterpret_cast<const int*>(ering + 1024);
    const uint8_t* e_zn = reinterpret_cast<const uint8_t*>(ering + 2048);

    if constexpr (kNF == 3) {
        // ---- epilogue, 192 channels: fragment f of a lane (token r16, row quad kb) holds logical channels 16 kb + 4 wave + v of
        // the tile's f-th block of 64.
#pragma unroll
        for (int f = 0; f < kNF; ++f) {
            const int nl = f * 64 + 16 * kb + 4 * wave, n0 = n_base + nl;
            if (n0 >= p.N) break;                        // N % 64 == 0: a block is all in or all out
            float sn[4];
            int zn[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) { sn[x] = OUT == OUT_FP16 ? __half2float(e_sn[nl + x]) : 0.f; zn[x] = GROUP ? 0 : (int)e_zn[nl + x]; }
#pragma unroll
            for (int tf = 0; tf < 8; ++tf) {
                const int ml = tf * 16 + r16, m = m_base + ml;
                if (m >= p.M) continue;
                finish4<GROUP, OUT>(p, m, n0, acc[f][tf], sn, zn, OUT == OUT_FP16 ? __half2float(e_sx[ml]) : 0.f, GROUP ? 0 : e_rs[ml]);
            }
        }
        return;
    }
    // ---- epilogue.  Lane (token r16, row quad kb) of fragment f holds physical rows 4 kb .. 4 kb + 3, i.e. logical
    // channels 16 kb + 4 f + v of the wave's 64: 16 consecutive channels of a token, one row segment of 32 bytes.
    const int nl = wave * 64 + 16 * kb, n0 = n_base + nl;  // first channel inside the tile, and of all
    if (n0 >= p.N) return;                               // N % 64 == 0: a segment is all in or all out
    float sn[16];
    int zn[16];
#pragma unroll
    for (int x = 0; x < 16; ++x) { sn[x] = OUT == OUT_FP16 ? __half2float(e_sn[nl + x]) : 0.f; zn[x] = GROUP ? 0 : (int)e_zn[nl + x]; }
#pragma unroll
    for (int tf = 0; tf < 8; ++tf) {
        const int ml = tf * 16 + r16;
        const int m = m_base + ml;
        if (m >= p.M) continue;
        const float sxm = OUT == OUT_FP16 ? __half2float(e_sx[ml]) : 0.f;
        const int rs = GROUP ? 0 : e_rs[ml];
        const bool token_sum = !GROUP && OUT == OUT_FP16 && p.token_sum;   // Eq. 7 form, rs = bits of t_X
        const float txm = __int_as_float(rs);
        int t[16];
#pragma unroll
        for (int x = 0; x < 16; ++x) {
            t[x] = acc[x >> 2][tf][x & 3];
            if (!GROUP && !token_sum) t[x] -= zn[x] * rs;
        }
        if constexpr (OUT == OUT_I32) {
            int4* dst = reinterpret_cast<int4*>(p.out32 + (size_t)m * p.N + n0);
#pragma unroll
            for (int q = 0; q < 4; ++q) dst[q] = make_int4(t[4 * q], t[4 * q + 1], t[4 * q + 2], t[4 * q + 3]);
        } else {
            uint32_t h[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                float ra = (float)t[2 * j] * (sxm * sn[2 * j]), rb = (float)t[2 * j + 1] * (sxm * sn[2 * j + 1]);
                if (token_sum) {
                    ra -= txm * ((float)zn[2 * j] * sn[2 * j]);
                    rb -= txm * ((float)zn[2 * j + 1] * sn[2 * j + 1]);
                }
                const __half lo = __float2half_rn(ra);
                const __half hi = __float2half_rn(rb);
                h[j] = (uint32_t)__half_as_ushort(lo) | ((uint32_t)__half_as_ushort(hi) << 16);
            }
            uint4* dst = reinterpret_cast<uint4*>(p.out16 + (size_t)m * p.N + n0);
#pragma unroll
            for (int q = 0; q < 2; ++q) dst[q] = make_uint4(h[4 * q], h[4 * q + 1], h[4 * q + 2], h[4 * q + 3]);
        }
    }
}

}  // namespace

hipError_t launch_mma16(const GemmDev& p, int channels, bool group, bool fp16, hipStream_t s)
{
    if (channels != 256 && (channels != 192 || p.S != 1)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(((p.N + channels - 1) / channels) * ((p.M + kTileM - 1) / kTileM)), (unsigned)p.S);
    auto* wide = group ? (fp16 ? mma16_kernel<true, OUT_FP16, 4> : mma16_kernel<true, OUT_I32, 4>)
                       : (fp16 ? mma16_kernel<false, OUT_FP16, 4> : mma16_kernel<false, OUT_I32, 4>);
    auto* narrow = group ? (fp16 ? mma16_kernel<true, OUT_FP16, 3> : mma16_kernel<true, OUT_I32, 3>)
                         : (fp16 ? mma16_kernel<false, OUT_FP16, 3> : mma16_kernel<false, OUT_I32, 3>);
    launch_gemm_kernel(channels == 256 ? wide : narrow, grid, kMmaThreads, s, p);
    return hipGetLastError();
}

}  // namespace qoq
