// Activation-stationary W4A8 GEMM kernels for token tiles of 16, 32 and 64 (decode sizes), gfx950.
//
// The LDS-staged streaming kernels fetch, for every 64-channel block of weights, the whole [tokens, K] slab of INT8
// activations again.  At 64 tokens that is twice the bytes of the weights themselves, all of it through the
// compute unit's vector cache, which returns data in request order and keeps a bounded number of bytes in flight:
// activation lines that hit in L2 queue behind weight lines that come from memory, and the weights get a third of
// what the cache can keep in flight.  Here the activations are loaded ONCE per workgroup and stay in registers for
// the whole kernel, in the layout of the matrix instruction's token operand, so that the main loop requests nothing
// but packed weights (Section 5.2.4 of arXiv 2405.04532 states the goal: at small m the GEMM is bound by weight
// traffic -- the loop should then move weights only).
//
//   * Workgroup = eight waves, two per SIMD, 256 registers per lane each.  Wave w keeps the activations of the
//     quantization groups g_lo + w * J' + j (j = 0 .. J'-1, J' <= J) of the workgroup's k-slice: J * MF * 2 operands
//     of 16 bytes per lane (MF = tokens / 16), at most 128 registers -- together the 256 KiB a [64, 4096] INT8 slab
//     takes; J <= 4 at 64 tokens, <= 8 at 32 and 16 tokens.  For 16 tokens and K of 8320 ... 14336 sixteen waves of 128
//     registers hold all of K, seven groups each (astat_deep_kernel); sixteen groups in each of eight waves lost to two k-slices.
//     (Four waves with twice the registers each were tried first: the compiler then parks part of the activations
//     in accumulation registers and copies them back in front of every matrix instruction.)  Slots past the end
//     of the slice hold zeros, so the loop needs no bounds logic: whatever weights are loaded for such a slot are
//     multiplied by zero.
//   * Work item = one 16-channel fragment of the packed layout (1 KiB per quantization group, contiguous over the
//     groups).  The layer's fragments are dealt in contiguous, equal runs to the workgroups, so a workgroup reads
//     one contiguous stretch of the packed weights, each wave its own J' consecutive KiB of every fragment, each lane exactly the 16 bytes its
//     matrix-instruction operand consists of (Section 5.2.1: stored in consumption order) -- straight into
//     registers, a ring of D units ahead, no LDS staging, no barrier inside a fragment.
//   * Per unit: the register dequantizer of Sections 5.2.2-5.2.3 (3-operation unpack, packed multiply-add, sign
//     flip) and 2 * MF v_mfma_i32_16x16x64_i8.
//   * End of a fragment: the eight waves' sums over their groups meet in LDS (double buffered: one barrier per
//     fragment); thread t then owns four consecutive channels of one token and runs the epilogue (Eq. 5-7).
//   * More tokens than a tile: token tiles on blockIdx.y, run side by side; the tiles of one fragment run share its
//     weights through L2 (the host keeps token tiles x fragment runs x k-slices at one workgroup per compute unit).
//   * K longer than 8 * J groups: k-slices on blockIdx.z.  Every slice writes its fragment sums through to the
//     workspace; after the loop it bumps the fragments' arrival counters, and whoever arrives last at a fragment
//     adds the slices (integer sums: exact and order independent) and runs the epilogue.  Same fence-free
//     hand-over as in the other kernels: write-through stores, a wait, a relaxed device-scope counter,
//     cache-bypassing loads.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "qoq_act_codes.h"
#include "qoq_gemm_common.h"
#include "qoq_layout.h"

namespace qoq {
namespace {

constexpr int kAsThreads = 512;
constexpr int kAsWaves = 8;
constexpr int kAsMaxFrags = 128;     // fragments per workgroup when k-slices meet in the workspace (host-checked)

// Where the codes, scales and sums of FP16 tokens go that the kernel quantizes itself (rowsum may be null); GemmDev::qx then
// is the address of the tokens.
struct TokensIn {
    int8_t* qx;
    __half* sx;
    int32_t* rowsum;
};
constexpr int kTokenLds = 32 * 1024;         // codes of a workgroup's tokens
constexpr int kTokenChunks = 8;              // 16-byte chunks of FP16 that a thread holds at most
constexpr int kFewTokenChunks = 2;           // compiled for as many too: loads and codes of chunks that are not there take time as well
static_assert(kTokenChunks * 8 * kAsThreads == kTokenLds, "one byte of codes per element held");

// For few and short tokens a launch of the quantizer costs more than its work, on the device (2.3 us) and on the host (2.5 us),
// so every workgroup quantizes all of them itself, while its first weights are on their way: 16 x 256 x 256 with one launch 4.9 us,
// with two 7.9 (issued one after the other); 1 x 4096 x 6144 per channel 5.6 and 8.3, 4 x 8192 x 22016 18.3 and 20.4.  512 / rows threads per
// row (rows: p.M rounded up to a power of two); scales and codes as the quantizer decides them (qoq_act_codes.h).
// Workgroup 0 writes them out for the caller.  Leaves the codes in `codes` (token-major, 16-byte chunks XORed with the row
// number inside each 128 bytes), maxima and sums in s_amax, s_sum.
template <int CHUNKS>
__device__ __forceinline__ void quantize_tokens(const GemmDev& p, const TokensIn& in, const uint4 (&v)[CHUNKS], int row, int tr,
                                                int per_row, bool want_sums, char* codes, uint32_t* s_amax, int* s_sum)
{
    auto row16 = [](auto x, auto join) {               // joined over each 16 lanes, which are of one row
        auto moved = [&](auto ctrl) {
            return __builtin_amdgcn_update_dpp(x, x, decltype(ctrl)::value, 0xF, 0xF, false);
        };
        x = join(x, moved(std::integral_constant<int, 0xB1>()));
        x = join(x, moved(std::integral_constant<int, 0x4E>()));
        x = join(x, moved(std::integral_constant<int, 0x141>()));
        return join(x, moved(std::integral_constant<int, 0x140>()));
    };
    const bool on = row < p.M, lead = on && (threadIdx.x & 15) == 0;
    h2 mx = half2_of(0u);
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) mx = max_of_chunk(v[i], mx);
    const int bits = row16(__float_as_int(fmaxf((float)mx.x, (float)mx.y)), [](int a, int b) { return max(a, b); });
    if (lead) atomicMax(&s_amax[row], (uint32_t)bits);   // non-negative: the bits order like the values
    __syncthreads();
    if (on) {
        const float s = __half2float(scale_of_row(__uint_as_float(s_amax[row]))), inv_s = 1.0f / s;
        int isum = 0;
#pragma unroll
        for (int i = 0; i < CHUNKS; ++i) {
            const int c = tr + i * per_row;
            if (c < p.K / 8) {
                const uint2 q = s >= 0x1p-14f ? codes_of_chunk(v[i], inv_s * (1.0f + 0x1p-20f), isum) : codes_of_chunk_clamped(v[i], inv_s, isum);
                *reinterpret_cast<uint2*>(codes + row * p.K + (((c >> 1) ^ (row & 7)) * 16) + (c & 1) * 8) = q;
                if (blockIdx.x == 0) reinterpret_cast<uint2*>(in.qx + (size_t)row * p.K)[c] = q;
            }
        }
        if (want_sums) {
            isum = row16(isum, [](int a, int b) { return a + b; });
            if (lead) atomicAdd(&s_sum[row], isum);
        }
    }
    __syncthreads();
    if (blockIdx.x == 0 && (int)threadIdx.x < p.M) {
        in.sx[threadIdx.x] = scale_of_row(__uint_as_float(s_amax[threadIdx.x]));
        if (in.rowsum) in.rowsum[threadIdx.x] = s_sum[threadIdx.x];
    }
}

// W waves.  ROWS: tokens that the preload of a 16-token tile moves (8: half the staging, for up to eight tokens).  CHUNKS > 0: the
// tokens come as FP16, so many chunks of them per thread.  NT: weights that no cache is worth keeping for (weights_pass_by).
template <int W, int MF, int J, int R, bool GROUP, int OUT, int ROWS, int CHUNKS, bool NT>
__device__ __forceinline__ void astat_run(const GemmDev& p, const TokensIn& in)
{
    constexpr bool FUSED = CHUNKS > 0;
    static_assert(W == 8 || (W == 16 && MF == 1), "wave counts");
    static_assert(!FUSED || (MF == 1 && W == 8), "the kernel quantizes up to sixteen tokens");
    // R = fragments whose units are in flight ahead of the one being multiplied: a ring of R * J units per wave
    static_assert(J * MF <= 16, "128 registers of activations per lane");
    constexpr int D = R * J;
    constexpr int kEl = MF * 64;                       // int4 elements of a fragment tile: mf * 64 + lane
    // LDS: first every wave's private staging area of the activation preload, afterwards, in the same bytes, the
    // double-buffered exchange of the waves' fragment sums.
    constexpr int kWaveStage = 128 * 1024 / W;
    constexpr int kLds = FUSED ? 2 * kTokenLds : W * kWaveStage;
    __shared__ __attribute__((aligned(16))) char lds_raw[kLds];
    static_assert(2 * W * kEl * 16 <= (FUSED ? kTokenLds : kLds), "the exchange buffers fit in the staging areas");
    int4 (*red)[W][kEl] = reinterpret_cast<int4 (*)[W][kEl]>(lds_raw);
    __shared__ int s_last[kAsMaxFrags];
    __shared__ uint32_t s_amax[16];                    // FUSED: the tokens' largest magnitudes and sums of codes
    __shared__ int s_sum[16];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q = lane >> 4, ml = lane & 15;
    const int mt_idx = blockIdx.y;
    const int m0 = mt_idx * (16 * MF);
    const int G = p.G, nf_total = p.N / 16;
    // fragments of this workgroup: contiguous runs whose lengths differ by at most one
    const int nwg = p.nwg, base = nf_total / nwg, rem = nf_total - base * nwg;
    const int wg = blockIdx.x;
    const int f0 = wg * base + min(wg, rem), f1 = f0 + base + (wg < rem ? 1 : 0);
    if (f0 >= f1) return;                              // whole workgroup: nothing to do
    const int slice = blockIdx.z;
    const int g_lo = slice * p.gps, g_hi = min(G, g_lo + p.gps);   // this workgroup's groups
    // Wave w owns the groups g_lo + w * jeff + j, j < jeff: a contiguous stretch, so that at any moment the eight
    // waves of a workgroup (and, the workgroups running in step, all of them) read eight different 128-byte
    // columns of the activation rows spread over the whole row -- with interleaved ownership every wave would be in
    // the same kilobyte of the row at the same time, which a few L2 channels then have to serve to the whole chip.
    const int jeff = (p.gps + W - 1) / W;             // <= J (host-checked)
    auto slot_valid = [&](int j) __attribute__((always_inline)) { return j < jeff && g_lo + wave * jeff + j < g_hi; };
    auto group_of = [&](int j) __attribute__((always_inline)) { return min(g_lo + wave * jeff + min(j, jeff - 1), g_hi - 1); };

    // ---- weights: ring of D units per wave, filled ahead ----------------------------------------
    // Fragments past the run (the refill at its end) and slots past the slice repeat valid addresses: those lines are in a cache.
    // Non-temporal ones need not be, so there the loads are buffer loads, whose bounds check turns such places into no
    // request at all (16 x 8192 x 10240 11.8 -> 11.2 us; as the only form 0.2 us slower where a workgroup has a fragment or two).
    const int nfr = f1 - f0;
    uint4 w[D];
    uint32_t mt[D];
    const __amdgpu_buffer_rsrc_t meta = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.meta), 0, G * nf_total * 32, 0x00020000);
    auto window = [&](int fi) __attribute__((always_inline)) {     // codes of fragments fi ... fi + 2 R - 1 of the run, as far as it goes
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4*>(p.codes) + (size_t)(f0 + fi) * G * 64, 0, min(nfr - fi, 2 * R) * G * 1024, 0x00020000);
    };
    auto load_unit = [&](__amdgpu_buffer_rsrc_t codes, int slot, int j, int fi, int ahead) __attribute__((always_inline)) {   // fragment fi + ahead
        if constexpr (NT) {
            constexpr uint32_t kNowhere = 0x80000000u;   // past the end of either buffer, also with an offset added
            const uint32_t g = (uint32_t)(g_lo + wave * jeff + j);
            const uint32_t at_w = slot_valid(j) ? g * 1024u : kNowhere, at_m = slot_valid(j) ? (g * (uint32_t)nf_total + (uint32_t)f0) * 32u : kNowhere;
            w[slot] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(codes, lane * 16 + (int)(at_w + (uint32_t)(ahead * G * 1024)), 0, 2));
            mt[slot] = GROUP ? (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(meta, ml * 2 + (int)(at_m + (uint32_t)(fi + ahead) * 32u), 0, 0) : 0u;
        } else {
            const int g = group_of(j), nf = f0 + min(fi + ahead, nfr - 1);
            w[slot] = p.codes[((size_t)nf * G + g) * 64 + lane];
            mt[slot] = GROUP ? (uint32_t)p.meta[((size_t)g * nf_total + nf) * 16 + ml] : 0u;
        }
    };

    // ---- activations: loaded once, resident for the whole kernel ---------------------------------
    // lane (ml, q) holds, of every (group, m-fragment, k-step) operand, token row ml and the 16-byte k-chunk q.
    // Loading those words directly costs the vector cache one request per 64-byte half line (16 rows x 64 B per
    // instruction) and was measured three times slower than reading whole lines, so they go through LDS: every
    // wave copies the columns of ITS OWN groups (JP * 128 contiguous bytes of each token row, whole 128-byte lines,
    // 1 KiB per instruction) into a private 16 KiB staging area by global->LDS DMA and reads its operands back --
    // one or two passes, no barrier: the waves do not wait for one another.  Inside a row the 16-byte chunks are
    // stored XORed with the row number (64-bank LDS: the 16 lanes served together read the same chunk of 16
    // consecutive rows), which keeps the operand reads free of bank conflicts.
    const __amdgpu_buffer_rsrc_t first = window(0);
    v4i a[J][MF][2];
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int mf = 0; mf < MF; ++mf) a[j][mf][0] = a[j][mf][1] = (v4i){0, 0, 0, 0};   // slots past the slice stay zero
    if constexpr (FUSED) {
        const int rows_log = p.M <= 1 ? 0 : 32 - __builtin_clz(p.M - 1), per_row = (64 * W) >> rows_log;
        const int row = (int)threadIdx.x >> (9 - rows_log), tr = (int)threadIdx.x & (per_row - 1);
        const bool want_sums = !GROUP || in.rowsum;
        if (threadIdx.x < 16) { s_amax[threadIdx.x] = 0; s_sum[threadIdx.x] = 0; }
        // the tokens first, then the weights, whose way is the longer one; chunks past the end of a row read as zeros
        const __amdgpu_buffer_rsrc_t tokens = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(p.qx), 0, p.M * p.K * 2, 0x00020000);
        uint4 v[CHUNKS];
#pragma unroll
        for (int i = 0; i < CHUNKS; ++i) {
            const int c = tr + i * per_row;
            v[i] = make_uint4(0u, 0u, 0u, 0u);
            if (i * per_row < p.K / 8)                 // workgroup-uniform
                v[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(tokens, row < p.M && c < p.K / 8 ? (row * (p.K / 8) + c) * 16 : p.M * p.K * 2, 0, 0));
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int j = 0; j < J; ++j) load_unit(first, r * J + j, j, 0, r);
        __syncthreads();
        char* codes = lds_raw + kTokenLds;
        quantize_tokens(p, in, v, row, tr, per_row, want_sums, codes, s_amax, s_sum);
        const int mr = min(ml, p.M - 1);               // rows past M repeat the last one
#pragma unroll
        for (int j = 0; j < J; ++j)
            if (slot_valid(j)) {
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
                    a[j][0][ks] = *reinterpret_cast<const v4i*>(codes + mr * p.K + (((group_of(j) * 8 + ks * 4 + q) ^ (mr & 7)) * 16));
            }
    } else {
        static_assert(ROWS == 16 || (ROWS == 8 && MF == 1), "rows of a pass");
        constexpr int JP = (J >= 8 && W == 8) || (J > 4 && ROWS == 8) ? 8 : 4;                                   // groups per pass
        constexpr int RP = ROWS == 8 ? 8 : (128 / JP) < MF * 16 ? (128 / JP) : MF * 16;      // token rows per pass
        constexpr int kRowPasses = ROWS == 8 ? 1 : (MF * 16 + RP - 1) / RP, kJPasses = (J + JP - 1) / JP, kDma = RP * JP / 8;
        static_assert(kDma * 1024 <= kWaveStage && RP % ROWS == 0, "a pass fits the wave's staging area");
        const char* abase = reinterpret_cast<const char*>(p.qx);
        const uint32_t region = (uint32_t)(uintptr_t)&lds_raw[0] + (uint32_t)wave * kWaveStage;
        const char* region_ptr = lds_raw + wave * kWaveStage;
        auto issue_pass = [&](int rp, int jp) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < kDma; ++i) {
                if (ROWS == 16 && rp * RP + i * 8 / JP >= MF * 16) continue;      // 48 tokens: half of the second pass
                const int flat = i * 64 + lane;                              // 16-byte position inside the pass
                const int row_local = flat / (JP * 8), pos = flat % (JP * 8);
                const uint32_t row = (uint32_t)min(m0 + rp * RP + row_local, p.M - 1);   // rows past M repeat the last one
                const uint32_t col = min((uint32_t)(g_lo + wave * jeff + jp * JP) * (uint32_t)kGroup +
                                             (uint32_t)((pos ^ (row_local & 15)) * 16),
                                         (uint32_t)p.K - 16u);                // groups past K re-read the end of the row
                dma16(abase, row * (uint32_t)p.K + col, region + (uint32_t)(i * 1024));
            }
        };
        auto read_pass = [&](int rp, int jp) __attribute__((always_inline)) {
#pragma unroll
            for (int mm = 0; mm < RP / ROWS; ++mm)
#pragma unroll
                for (int jj = 0; jj < JP; ++jj) {
                    const int mf = rp * (RP / ROWS) + mm, j = jp * JP + jj;
                    if (j < J && mf < MF) {
                        if (slot_valid(j)) {                                 // wave-uniform
                            const int row_local = mm * 16 + (ml & (ROWS - 1));
#pragma unroll
                            for (int ks = 0; ks < 2; ++ks)
                                a[j][mf][ks] = *reinterpret_cast<const v4i*>(region_ptr + row_local * (JP * 128) +
                                                                             (((jj * 8 + ks * 4 + q) ^ (row_local & 15)) * 16));
                        }
                    }
                }
        };
        // Order of the requests: the first pass of activations, then the first R fragments of weights (a trip to
        // memory: data returns in request order, so they must not stand in front of the first pass; behind it
        // their latency passes while the pass is unpacked), then the other passes.  The waits count what this wave
        // requested after the pass it waits for: kNW weight loads (build.py checks that the compiler emits
        // exactly that many).
        constexpr int kNW = R * J * (GROUP ? 2 : 1);
        static_assert(kNW < 64, "vmcnt range");
        issue_pass(0, 0);
        asm volatile("; astat weight prologue begin" ::: "memory");
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int j = 0; j < J; ++j) load_unit(first, r * J + j, j, 0, r);
        asm volatile("; astat weight prologue end" ::: "memory");
        wait_vmcnt<kNW>();
        read_pass(0, 0);
#pragma unroll
        for (int pp = 1; pp < kRowPasses * kJPasses; ++pp) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");               // the reads of the pass before are done
            issue_pass(pp / kJPasses, pp % kJPasses);
            wait_vmcnt<0>();
            read_pass(pp / kJPasses, pp % kJPasses);
        }
    }
    if constexpr (!FUSED) __syncthreads();    // the staging areas become the exchange buffers of the fragment sums

    // ---- epilogue role: thread t owns element t of every fragment tile (one token, four consecutive channels) ----
    const int el = threadIdx.x;
    const int e_ln = el & 63;
    const int e_m = m0 + (el >> 6) * 16 + (e_ln & 15);
    const bool e_on = el < kEl;
    float c_sx = 0.f;
    int c_rs = 0;
    if (e_on) {
        const int mc = min(e_m, p.M - 1);
        if constexpr (FUSED) {
            c_sx = __half2float(scale_of_row(__uint_as_float(s_amax[mc])));
            c_rs = GROUP ? 0 : s_sum[mc];
        } else {
            c_sx = OUT == OUT_FP16 ? __half2float(p.sx[mc]) : 0.f;
            c_rs = GROUP ? 0 : p.rowsum[mc];
        }
    }
    auto channel_of = [&](int nf) __attribute__((always_inline)) { return (nf >> 2) * 64 + 16 * (e_ln >> 4) + 4 * (nf & 3); };
    auto epilogue = [&](int nf, v4i sum, uint2 sw, uint32_t zw) __attribute__((always_inline)) {
        const float sn[4] = {__half2float(__ushort_as_half((unsigned short)(sw.x & 0xFFFFu))),
                             __half2float(__ushort_as_half((unsigned short)(sw.x >> 16))),
                             __half2float(__ushort_as_half((unsigned short)(sw.y & 0xFFFFu))),
                             __half2float(__ushort_as_half((unsigned short)(sw.y >> 16)))};
        const int zn[4] = {(int)(zw & 0xFFu), (int)((zw >> 8) & 0xFFu), (int)((zw >> 16) & 0xFFu), (int)(zw >> 24)};
        finish4<GROUP, OUT>(p, e_m, channel_of(nf), sum, sn, zn, c_sx, c_rs);
    };
    const size_t part_stride = (size_t)p.S * kEl;      // int4 elements per fragment in the workspace
    int4* parts_mt = p.parts + (size_t)mt_idx * nf_total * part_stride;

    // ---- main loop over the fragments, R per trip so that every ring slot is a compile-time constant -----------
    int buf = 0;
    for (int fi0 = 0; fi0 < nfr; fi0 += R) {
        const __amdgpu_buffer_rsrc_t codes = window(fi0);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int fi = fi0 + r;
            if (fi >= nfr) break;                          // workgroup-uniform
            const int nf = f0 + fi;
            uint2 c_s = make_uint2(0, 0);
            uint32_t c_z = 0;
            if (e_on && p.S == 1) {                        // epilogue constants: in flight during the fragment
                if (OUT == OUT_FP16) c_s = *reinterpret_cast<const uint2*>(p.scales + channel_of(nf));
                if (!GROUP) c_z = *reinterpret_cast<const uint32_t*>(p.zeros + channel_of(nf));
            }
            v4i acc[MF];
#pragma unroll
            for (int mf = 0; mf < MF; ++mf) acc[mf] = (v4i){0, 0, 0, 0};
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const int slot = r * J + j;
                const uint4 wq = w[slot];
                uint32_t S = 0, B = 0;
                if (GROUP) {
                    S = __builtin_amdgcn_perm(mt[slot], mt[slot], 0x0c000c00u);   // s1 in both 16-bit lanes
                    B = __builtin_amdgcn_perm(mt[slot], mt[slot], 0x01010101u);   // bias in all four bytes
                }
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    const v4i w_op = dequant<GROUP>(ks ? wq.z : wq.x, ks ? wq.w : wq.y, S, B);
#pragma unroll
                    for (int mf = 0; mf < MF; ++mf)
                        acc[mf] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w_op, a[j][mf][ks], acc[mf], 0, 0, 0);
                }
                // the slot's words are consumed: refill it with the same unit of the fragment R places ahead
                load_unit(codes, slot, j, fi0, r + R);
                // keep the units in program order: otherwise the compiler gathers the first touch of every slot at
                // the top of the fragment and with it the waits for loads issued only a few hundred cycles earlier
                __builtin_amdgcn_sched_barrier(0);
            }
            // the waves' sums meet in LDS; the buffers alternate, so one barrier per fragment is enough (a wave
            // writes buffer b again only after the barrier of the fragment in between, which every wave reaches
            // after its reads of b)
#pragma unroll
            for (int mf = 0; mf < MF; ++mf)
                red[buf][wave][mf * 64 + lane] = make_int4(acc[mf].x, acc[mf].y, acc[mf].z, acc[mf].w);
            __syncthreads();
            if (e_on) {
                v4i sum = (v4i){0, 0, 0, 0};
#pragma unroll
                for (int ww = 0; ww < W; ++ww) {
                    const int4 o = red[buf][ww][el];
                    sum += (v4i){o.x, o.y, o.z, o.w};
                }
                if (p.S == 1) {
                    if (e_m < p.M) epilogue(nf, sum, c_s, c_z);
                } else {
                    store_through(parts_mt + (size_t)nf * part_stride + (size_t)slice * kEl + el, sum.x, sum.y, sum.z, sum.w);
                }
            }
            buf ^= 1;
        }
    }
    if (p.S == 1) return;

    // ---- k-slices meet: wait for the partial sums to reach memory, bump every fragment's counter, finish the
    // fragments at which this workgroup arrived last ----------------------------------------------------------
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    for (int i = threadIdx.x; i < nfr; i += (64 * W)) {
        int* ctr = p.counters + mt_idx * nf_total + f0 + i;
        const int old = __hip_atomic_fetch_add(ctr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const bool last = old == p.S - 1;
        if (last) __hip_atomic_store(ctr, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_last[i] = last;
    }
    __syncthreads();
    if (!e_on) return;
    for (int i = 0; i < nfr; ++i) {
        if (!s_last[i]) continue;                      // workgroup-uniform
        const int nf = f0 + i;
        uint2 c_s = make_uint2(0, 0);
        uint32_t c_z = 0;
        if (OUT == OUT_FP16) c_s = *reinterpret_cast<const uint2*>(p.scales + channel_of(nf));
        if (!GROUP) c_z = *reinterpret_cast<const uint32_t*>(p.zeros + channel_of(nf));
        const int4* src = parts_mt + (size_t)nf * part_stride + el;
        v4i sum = (v4i){0, 0, 0, 0};
        int s = 0;
        for (; s + 4 <= p.S; s += 4) {                 // four loads in flight: the sum is pure load latency
            const v4i t0 = load_through(src + (size_t)s * kEl), t1 = load_through(src + (size_t)(s + 1) * kEl);
            const v4i t2 = load_through(src + (size_t)(s + 2) * kEl), t3 = load_through(src + (size_t)(s + 3) * kEl);
            sum += t0 + t1 + t2 + t3;
        }
        for (; s < p.S; ++s) sum += load_through(src + (size_t)s * kEl);
        if (e_m < p.M) epilogue(nf, sum, c_s, c_z);
    }
}

template <int MF, int J, int R, bool GROUP, int OUT, int ROWS, bool NT>
__global__ __launch_bounds__(kAsThreads) void astat_kernel(QOQ_GEMM_PARAMS, GemmTail tail)
{
    const GemmDev p = gemm_dev(QOQ_GEMM_ARGS, tail);
    astat_run<8, MF, J, R, GROUP, OUT, ROWS, 0, NT>(p, TokensIn{});
}

// Sixteen waves of 128 registers, for sixteen tokens and K between what eight waves hold and 14336 (seven groups per wave): one
// workgroup then holds all of K, where two k-slices of eight waves met in memory (stores drained, a counter, loads past the
// caches: about 2 us).  11008 x 4096 at one token 11.6 us -> 8.9, at sixteen 11.1 -> 10.3; 14336 x 4096 per channel 10.5 -> 8.2; 9216 x
// 28672 per channel 35.5 -> 23.5.  Up to eight tokens need half the staging: all groups of a wave in one pass, not two one
// after the other (8.9 and 9.9 us; eight waves, K = 8192 x 10240: 11.2 and 11.6).
template <int J, bool GROUP, int OUT, int ROWS, bool NT>
__global__ __launch_bounds__(1024) void astat_deep_kernel(QOQ_GEMM_PARAMS, GemmTail tail)
{
    const GemmDev p = gemm_dev(QOQ_GEMM_ARGS, tail);
    astat_run<16, 1, J, 1, GROUP, OUT, ROWS, 0, NT>(p, TokensIn{});
}

// Up to sixteen FP16 tokens through the quantizer and the GEMM in one launch.
template <int J, int R, bool GROUP, int CHUNKS, bool NT>
__global__ __launch_bounds__(kAsThreads) void astat_linear_kernel(QOQ_GEMM_PARAMS, GemmTail tail, TokensIn in)
{
    const GemmDev p = gemm_dev(QOQ_GEMM_ARGS, tail);
    astat_run<8, 1, J, R, GROUP, OUT_FP16, 16, CHUNKS, NT>(p, in);
}

template <int MF, int J, int R, bool GROUP, int OUT, int ROWS>
void launch_nt(const GemmDev& p, dim3 grid, hipStream_t s)
{
    if (weights_pass_by(p, grid, p.S == 1 ? kPassByWhole : kPassBy)) launch_gemm_kernel(astat_kernel<MF, J, R, GROUP, OUT, ROWS, true>, grid, kAsThreads, s, p);
    else launch_gemm_kernel(astat_kernel<MF, J, R, GROUP, OUT, ROWS, false>, grid, kAsThreads, s, p);
}
template <int MF, int J, int R, bool GROUP>
void launch_j(const GemmDev& p, dim3 grid, bool fp16, hipStream_t s)
{
    if constexpr (MF == 1) {
        if (p.M <= 8) {
            if (fp16) launch_nt<MF, J, R, GROUP, OUT_FP16, 8>(p, grid, s);
            else launch_gemm_kernel(astat_kernel<MF, J, R, GROUP, OUT_I32, 8, false>, grid, kAsThreads, s, p);
            return;
        }
    }
    if (fp16) launch_nt<MF, J, R, GROUP, OUT_FP16, 16>(p, grid, s);
    else launch_gemm_kernel(astat_kernel<MF, J, R, GROUP, OUT_I32, 16, false>, grid, kAsThreads, s, p);
}

constexpr int kDeepGroups = 7 * 16;
template <bool GROUP, int OUT, int ROWS, bool NT>
void launch_deep_rows(const GemmDev& p, dim3 grid, hipStream_t s)
{
    if (p.gps <= 6 * 16) launch_gemm_kernel(astat_deep_kernel<6, GROUP, OUT, ROWS, NT>, grid, 1024, s, p);
    else launch_gemm_kernel(astat_deep_kernel<7, GROUP, OUT, ROWS, NT>, grid, 1024, s, p);
}
template <bool GROUP, int OUT>
void launch_deep(const GemmDev& p, dim3 grid, hipStream_t s)
{
    if (OUT == OUT_FP16 && weights_pass_by(p, grid, kPassByWhole)) p.M <= 8 ? launch_deep_rows<GROUP, OUT, 8, OUT == OUT_FP16>(p, grid, s) : launch_deep_rows<GROUP, OUT, 16, OUT == OUT_FP16>(p, grid, s);
    else p.M <= 8 ? launch_deep_rows<GROUP, OUT, 8, false>(p, grid, s) : launch_deep_rows<GROUP, OUT, 16, false>(p, grid, s);
}

template <bool GROUP>
hipError_t launch_mode(const GemmDev& p, int tile, dim3 grid, bool fp16, hipStream_t s)
{
    const int need = (p.gps + kAsWaves - 1) / kAsWaves;   // groups per wave
    if (tile == 48) {
        if (need <= 2) launch_j<3, 2, 2, GROUP>(p, grid, fp16, s);
        else if (need <= 3) launch_j<3, 3, 2, GROUP>(p, grid, fp16, s);
        else if (need <= 4) launch_j<3, 4, 2, GROUP>(p, grid, fp16, s);
        else return hipErrorInvalidValue;
    } else if (tile == 64) {
        if (need <= 2) launch_j<4, 2, 2, GROUP>(p, grid, fp16, s);
        else if (need <= 3) launch_j<4, 3, 2, GROUP>(p, grid, fp16, s);
        else if (need <= 4) launch_j<4, 4, 2, GROUP>(p, grid, fp16, s);
        else return hipErrorInvalidValue;
    } else if (tile == 32) {
        if (need <= 4) launch_j<2, 4, 2, GROUP>(p, grid, fp16, s);
        else if (need <= 8) launch_j<2, 8, 1, GROUP>(p, grid, fp16, s);
        else return hipErrorInvalidValue;
    } else if (p.gps > astat_max_groups(16)) {
        if (p.gps > kDeepGroups) return hipErrorInvalidValue;
        if (fp16) launch_deep<GROUP, OUT_FP16>(p, grid, s);
        else launch_deep<GROUP, OUT_I32>(p, grid, s);
    } else {
        if (need <= 4) launch_j<1, 4, 2, GROUP>(p, grid, fp16, s);
        else if (need <= 8) launch_j<1, 8, 1, GROUP>(p, grid, fp16, s);
        else return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <bool GROUP, int CHUNKS, bool NT>
void launch_linear_nt(const GemmDev& p, const TokensIn& in, dim3 grid, hipStream_t s)
{
    if ((p.G + kAsWaves - 1) / kAsWaves <= 4) launch_gemm_kernel(astat_linear_kernel<4, 2, GROUP, CHUNKS, NT>, grid, kAsThreads, s, p, in);
    else launch_gemm_kernel(astat_linear_kernel<8, 1, GROUP, CHUNKS, NT>, grid, kAsThreads, s, p, in);
}
template <bool GROUP, int CHUNKS>
void launch_linear(const GemmDev& p, const TokensIn& in, dim3 grid, hipStream_t s)
{
    weights_pass_by(p, grid, kPassByWhole) ? launch_linear_nt<GROUP, CHUNKS, true>(p, in, grid, s) : launch_linear_nt<GROUP, CHUNKS, false>(p, in, grid, s);
}

// Elements of M tokens of K, M rounded up to a power of two: what the threads of a workgroup share.
int64_t token_elements(int64_t M, int64_t K)
{
    int64_t rows = 1;
    while (rows < M) rows *= 2;
    return rows * K;
}

}  // namespace

bool astat_linear_takes(int64_t M, int64_t K)
{
    if (M < 1 || M > 16 || K / kGroup > astat_max_groups(16)) return false;
    return token_elements(M, K) <= kTokenLds;            // (16 x 4096 x 6144 per channel: 8.3 us in one launch, 7.7 in two)
}

hipError_t launch_astat_linear(const GemmDev& layer, const void* x, int8_t* qx, void* sx, int32_t* rowsum, bool group, hipStream_t s)
{
    if (!astat_linear_takes(layer.M, layer.K)) return hipErrorInvalidValue;
    const TokensIn in{qx, static_cast<__half*>(sx), rowsum};
    GemmDev p = layer;
    p.qx = static_cast<const int8_t*>(x);
    const dim3 grid((unsigned)(p.N / 16 < 256 ? p.N / 16 : 256));
    const bool few = token_elements(p.M, p.K) <= (int64_t)kFewTokenChunks * 8 * kAsThreads;
    if (group) few ? launch_linear<true, kFewTokenChunks>(p, in, grid, s) : launch_linear<true, kTokenChunks>(p, in, grid, s);
    else few ? launch_linear<false, kFewTokenChunks>(p, in, grid, s) : launch_linear<false, kTokenChunks>(p, in, grid, s);
    return hipGetLastError();
}

int astat_deep_groups() { return kDeepGroups; }

int astat_max_groups(int tile) { return kAsWaves * (tile == 64 ? 4 : 8); }

hipError_t launch_astat(const GemmDev& p, int tile_m, int nwg, bool group, bool fp16, hipStream_t s)
{
    const int tile = tile_m == 71 ? 64 : tile_m == 70 ? 32 : 16;
    const int nf_total = p.N / 16;
    if (nwg < 1 || p.S < 1 || p.gps < 1 || p.gps > (tile == 16 ? kDeepGroups : astat_max_groups(tile))) return hipErrorInvalidValue;
    if (p.S > 1 && (nf_total + nwg - 1) / nwg > kAsMaxFrags) return hipErrorInvalidValue;
    const dim3 grid((unsigned)nwg, (unsigned)((p.M + tile - 1) / tile), (unsigned)p.S);
    // As many tiles of 48 tokens as of 64 hold them all (33 ... 48, 65 ... 96, 129 ... 144): a quarter less to load
    // in front of the loop and to multiply in it (4096 x 12288 at 80 tokens 16.5 -> 14.3 us, at 130 20.9 -> 18.9; 22016 at 37 16.5 -> 15.1).
    const int rows = tile == 64 && p.M <= 48 * (int)grid.y ? 48 : tile;
    return group ? launch_mode<true>(p, rows, grid, fp16, s) : launch_mode<false>(p, rows, grid, fp16, s);
}

}  // namespace qoq
