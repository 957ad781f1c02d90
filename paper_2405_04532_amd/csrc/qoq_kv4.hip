// KV4 cache and decode attention for gfx950 (Sections 5.1 "KV Cache Management" and 5.3 of arXiv 2405.04532,
// re-designed for CDNA4).
//
// Cache.  Keys and values are quantized when they are written: per token and KV head, Eq. 1 with 4 bits on the
// range of that head's 128 values widened to contain 0, FP16 scale s and integer zero z (stored as the FP16
// number -(1024 + z), the form the decode kernel consumes).  A
// page holds 64 consecutive tokens of one (sequence, KV head): 4 KiB of key codes, their 64 (s, z) pairs, 4 KiB
// of value codes, their 64 pairs -- the parameters sit directly behind the codes they belong to, in the same
// page.  The pages of a (sequence, head) are contiguous.
//   key codes of a token: 16 dwords; dword w holds elements 8w .. 8w+7, element 8w+2j in bits 4j.. of the low
//   half, element 8w+2j+1 in bits 4j.. of the high half: (x >> 4j) & 0x000F000F is a pair of consecutive
//   elements, and OR 0x64006400 makes it the FP16 pair (1024 + a, 1024 + b) -- the integer-to-FP16 conversion
//   without a conversion instruction that Section 5.3 takes from earlier work.  One packed add of -(1024 + z)
//   then gives the exact integers (code - z) as FP16.  The odd nibbles need no shift: (x & 0x00F000F0) |
//   0x64006400 is (1024 + 16a, 1024 + 16b), and one packed multiply-add, * 1/16 - (64 + z), is exact too.
//   Two vector operations per pair of elements, plus one shift per dword.
//   value codes: stored tile by tile (16 tokens x 128 elements = 1 KiB) in the order the matrix instruction that
//   forms P.V wants its operand: lane l = 16 kb + r of a wave owns the 16 bytes at 16 l; its dword 2u + h holds, for
//   the four elements d = 4 (r + 16 u) + j (nibble j), token 4 kb + 2h in the low half and token 4 kb + 2h + 1 in the
//   high half.  The same unpacking then yields FP16 pairs (token, next token) of one element, and two such pairs are
//   the four k-values of an MFMA operand row.  A token still owns whole 16-bit words (32 of them), so appending a
//   token is 32 plain 2-byte stores.
//
// Decode kernel.  One workgroup of 4 or 8 waves per (sequence, KV head); every wave streams chunks of the sequence,
// two 16-token tiles at a time, and both products run on v_mfma_f32_16x16x32_f16 (FP16 operands, FP32 sums):
//   S[token][head]  = sum_d (code - z_K)[token][d] * q[head][d]     A = unpacked keys, B = the queries of the up
//                                                                    to 16 heads that share the KV head (GQA
//                                                                    costs nothing extra), 4 MFMAs per tile
//   score = S * s_K[token] * log2(e) / sqrt(D); online softmax in base 2
//   O[d][head]     += sum_token (code - z_V)[token][d] * (p * s_V)[token][head]    8 MFMAs for both tiles
// The output layout of the first product (a lane holds 4 tokens of one head) is exactly the operand layout of the
// second, so the softmax runs in place and nothing moves between lanes except the running maximum.  With up to eight
// heads the columns of a matrix instruction hold both tiles side by side (columns 0..7 the first tile, 8..15 the second):
// the queries are repeated in both halves, a lane keeps the scores of its own half's tile, and every column is a
// softmax stream of its own until the end, so the softmax costs one tile's instructions for two tiles.  The paper's
// kernel computes on scalar cores and fights their compute roof (Section 5.3: FP16 instead of FP32 arithmetic,
// two-operation dequantization); here the two-operation dequantization is kept and the multiply-adds go to the
// matrix cores, which leaves the vector pipe with the unpacking and the softmax only.
// Measured against one tile per matrix instruction and 16x16x16 products: Llama-2-7B heads 64 x 1024 58.8 us instead of 63.5
// (4.85 TB/s; the loads alone, with no arithmetic, take 52), Llama-3-8B heads 64 x 1024 17.5 instead of 19.3, 4 x 8192 12.7
// instead of 16.6, Llama-3-70B heads 64 x 1024 18.2 instead of 19.9.  The vector pipe is active half of the time: 150 of the
// 250 vector instructions per chunk unpack codes.  Taking the longest sequences first, or two waves per workgroup, was slower.
// Relative error of the output against FP64 on the same cache (1 to 64 sequences, 64 to 8192 tokens, 1 to 16 heads per KV head):
// 2.0e-4 to 2.5e-4, the FP16 softmax weights' own; 3% less than with one tile per instruction on average, nowhere more.
// The scale/zero words of a chunk are loaded together with its codes, one chunk ahead of the arithmetic (the
// prefetch of the dequantization parameters of Section 5.3).  Partial (max, sum, acc) of the waves meet in LDS.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "qoq_fp16.h"
#include "qoq_internal.h"

namespace qoq {
namespace {

typedef _Float16 h2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ _Float16 half_of(uint32_t v) { return __builtin_bit_cast(_Float16, (unsigned short)v); }

constexpr int kD = 128;                       // head dimension
constexpr int kPageTokens = 64;
constexpr int kCodeBytes = kPageTokens * kD / 2;          // 4096
constexpr int kParamBytes = kPageTokens * 4;              // 256
constexpr int kHalfPage = kCodeBytes + kParamBytes;       // keys (or values) of a page
constexpr int kPageBytes = 2 * kHalfPage;                 // 8704

// byte offset, inside the value codes of a page, of the 16-bit word of token `tin` (0..63) and elements 4 q4 .. 4 q4 + 3
__device__ __forceinline__ int v_word_offset(int tin, int q4)
{
    const int tile = tin >> 4, kb = (tin >> 2) & 3, h = (tin >> 1) & 1, half = tin & 1;
    const int r = q4 & 15, u = q4 >> 4;
    return tile * 1024 + (kb * 16 + r) * 16 + (2 * u + h) * 4 + half * 2;
}

// ------------------------------------------------------------------------------------------
// Append: one wave per (sequence, KV head, aligned quad of token positions); 16 lanes per token, lane w of a token
// holds its elements 8w .. 8w+7 of the key and of the value (two 16-byte loads, both in flight at once).  A quad of tokens is
// 4 x 64 contiguous bytes of key codes and ONE contiguous 256-byte block of value codes (the value layout groups the
// four tokens of an operand k-block), which a complete quad assembles in LDS and writes with 16-byte stores; a
// quad that this call covers only in part (a decode step appends a single token) writes its own 2-byte words.
// Every decision is the one the reference definition takes, from FP32:
//   s = FP16((hi - lo) / 15), the quotient in exact arithmetic rounded once: the FP32 quotient is within 4 * 2^-24 of it, so
//     where both ends of that interval round to the same FP16 number that is it; else (1 in 2000) the FP64 quotient decides
//   codes and z = floor(x / s + 1/2) + integer: |x / s| < 256 is on a half-integer or at least 2^-12 away from every one;
//     x * fl(1 / s) is within 3e-5 of it, and pushed 1e-4 upwards it lands on the side that rounding half up takes.
// A division per element and an FP64 one per token, and the value loaded behind the key's arithmetic, took
// 492 us for 64 x 1024 tokens of 32 heads and 4.7 us for one token each; now 305 us (4.45 TB/s of FP16 in and cache out) and 3.6 us.
// ------------------------------------------------------------------------------------------
// minimum / maximum over a row of 16 lanes (cross-lane moves without LDS)
template <int CTRL>
__device__ __forceinline__ float row_move(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float row_min16(float v)
{
    v = fminf(v, row_move<0x128>(v));                                      // rotations by 8, 4, 2, 1 lanes
    v = fminf(v, row_move<0x124>(v));
    v = fminf(v, row_move<0x122>(v));
    return fminf(v, row_move<0x121>(v));
}
__device__ __forceinline__ float row_max16(float v)
{
    v = fmaxf(v, row_move<0x128>(v));
    v = fmaxf(v, row_move<0x124>(v));
    v = fmaxf(v, row_move<0x122>(v));
    return fmaxf(v, row_move<0x121>(v));
}

__global__ __launch_bounds__(256) void kv4_append_kernel(const __half* __restrict__ k, const __half* __restrict__ v,
                                                         const int32_t* __restrict__ positions, uint8_t* __restrict__ cache,
                                                         int T, int Hkv, int S_max, uint32_t quads, uint32_t items)
{
    __shared__ uint4 s_block[4][16];                                       // per wave: the value codes of its quad
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, w = lane & 15;                                // token of the quad, 16-byte chunk of its row
    const uint32_t item = blockIdx.x * 4 + (uint32_t)wave;                 // (b * Hkv + h) * quads + j
    if (item >= items) return;
    const uint32_t bh = item / quads, b = bh / (uint32_t)Hkv;
    const int64_t j = item - bh * quads, h = bh - b * (uint32_t)Hkv;
    const int64_t p0 = positions[b];
    const int64_t pos = ((p0 >> 2) + j) * 4 + g;                           // floor(p0 / 4) also for negative p0
    const int64_t t = pos - p0;
    const bool valid = t >= 0 && t < T && pos >= 0 && pos < S_max;         // outside the call or the cache: not written
    const bool whole = __builtin_amdgcn_ballot_w64(valid) == ~0ull;
    if (__builtin_amdgcn_ballot_w64(valid) == 0) return;
    const int64_t row = (((int64_t)b * T + (valid ? t : 0)) * Hkv + h) * kD;
    const uint4 raws[2] = {reinterpret_cast<const uint4*>(k + row)[w], reinterpret_cast<const uint4*>(v + row)[w]};
    const int64_t n_pages = (S_max + kPageTokens - 1) / kPageTokens;
    const int64_t pos_c = valid ? pos : 0;
    uint8_t* page = cache + ((int64_t)bh * n_pages + pos_c / kPageTokens) * kPageBytes;
    const int tin = (int)(pos_c % kPageTokens);

#pragma unroll
    for (int which = 0; which < 2; ++which) {
        uint32_t rw[4] = {raws[which].x, raws[which].y, raws[which].z, raws[which].w};
        h2 mn = {(_Float16)0.f, (_Float16)0.f}, mx = mn;                   // the range is widened to contain 0
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            mn = __builtin_elementwise_min(mn, __builtin_bit_cast(h2, rw[e]));
            mx = __builtin_elementwise_max(mx, __builtin_bit_cast(h2, rw[e]));
        }
        const float lo = row_min16(fminf((float)mn.x, (float)mn.y)), hi = row_max16(fmaxf((float)mx.x, (float)mx.y));
        const float quot = (hi - lo) * (1.0f / 15.0f);
        float q_lo = quot * (1.0f - 4 * 0x1p-24f), q_hi = quot * (1.0f + 4 * 0x1p-24f);
        asm("" : "+v"(q_lo), "+v"(q_hi));                                  // no mixed-precision merging of product and conversion
        uint16_t s_bits = __half_as_ushort(__float2half_rn(q_lo));
        if (s_bits != __half_as_ushort(__float2half_rn(q_hi))) s_bits = double_to_half_rne(((double)hi - (double)lo) / 15.0);
        if ((s_bits & 0x7FFFu) == 0) s_bits = 0x3C00u;                     // all-zero vector: s = 1
        const float inv = 1.0f / __half2float(__ushort_as_half(s_bits));
        const float z = __builtin_amdgcn_fmed3f(floorf(fmaf(-lo, inv, 0.5f + 1e-4f)), 0.f, 15.f);
        const float offset = z + (0.5f + 1e-4f);
        // NaN, and infinity over an infinite scale, are quotient 0 (code z); times zero they leave NaN in the sum
        float bad = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) bad = __builtin_amdgcn_fdot2(__builtin_bit_cast(h2, rw[e]), (h2){(_Float16)0.f, (_Float16)0.f}, bad, false);
        if (bad != bad)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if ((~(rw[e >> 1] >> (16 * (e & 1))) & 0x7C00u) == 0) rw[e >> 1] &= 0xFFFFu << (16 * (~e & 1));
        uint32_t c[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float x = (float)half_of(rw[e >> 1] >> (16 * (e & 1)));
            c[e] = (uint32_t)(int)__builtin_amdgcn_fmed3f(fmaf(x, inv, offset), 0.f, 15.f);
        }
        if (which == 0) {
            // keys: dword w = elements 8w .. 8w+7, element 8w+2j in nibble j of the low half, 8w+2j+1 of the high half
            uint32_t word = 0;
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) word |= (c[2 * jj] << (4 * jj)) | (c[2 * jj + 1] << (16 + 4 * jj));
            if (valid) reinterpret_cast<uint32_t*>(page + tin * (kD / 2))[w] = word;
        } else {
            // values: 16-bit words of element quads 2w (elements 8w .. 8w+3) and 2w+1
            const uint32_t h0 = c[0] | (c[1] << 4) | (c[2] << 8) | (c[3] << 12);
            const uint32_t h1 = c[4] | (c[5] << 4) | (c[6] << 8) | (c[7] << 12);
            if (whole) {
                // inside the quad's 256-byte block: chunk r = q4 % 16, dword 2 (q4 / 16) + (g >> 1), half g & 1
                uint16_t* blk = reinterpret_cast<uint16_t*>(&s_block[wave][0]);
                const int q4a = 2 * w, q4b = 2 * w + 1;
                blk[(q4a & 15) * 8 + (2 * (q4a >> 4) + (g >> 1)) * 2 + (g & 1)] = (uint16_t)h0;
                blk[(q4b & 15) * 8 + (2 * (q4b >> 4) + (g >> 1)) * 2 + (g & 1)] = (uint16_t)h1;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");     // the wave's own LDS writes, then its reads
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                if (lane < 16) {
                    const int tin0 = tin & ~3;                             // lanes 0..15 are token 0 of the quad: tin % 4 == 0
                    uint8_t* dst = page + kHalfPage + (tin0 >> 4) * 1024 + (((tin0 >> 2) & 3) * 16 + lane) * 16;
                    *reinterpret_cast<uint4*>(dst) = s_block[wave][lane];
                }
            } else if (valid) {
                *reinterpret_cast<uint16_t*>(page + kHalfPage + v_word_offset(tin, 2 * w)) = (uint16_t)h0;
                *reinterpret_cast<uint16_t*>(page + kHalfPage + v_word_offset(tin, 2 * w + 1)) = (uint16_t)h1;
            }
        }
        if (valid && w == 0) {
            // the zero point is stored as the FP16 number -(1024 + z) (an exact integer), the constant the decode
            // kernel adds to its unpacked codes
            const uint16_t z_bits = __half_as_ushort(__float2half_rn(-1024.0f - z));
            reinterpret_cast<uint32_t*>(page + which * kHalfPage + kCodeBytes)[tin] = (uint32_t)s_bits | ((uint32_t)z_bits << 16);
        }
    }
}

// Inverse of the layout (tests): one thread per (sequence, head, token, key|value, dword).
__global__ __launch_bounds__(256) void kv4_unpack_kernel(const uint8_t* __restrict__ cache, int64_t B, int64_t Hkv, int64_t S_max,
                                                         uint8_t* __restrict__ k_codes, __half* __restrict__ k_s,
                                                         __half* __restrict__ k_z, uint8_t* __restrict__ v_codes,
                                                         __half* __restrict__ v_s, __half* __restrict__ v_z)
{
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;           // (((b * Hkv + h) * S + t) * 2 + which) * 16 + w
    if (idx >= B * Hkv * S_max * 32) return;
    const int w = (int)(idx & 15), which = (int)((idx >> 4) & 1);
    const int64_t bht = idx >> 5, t = bht % S_max, bh = bht / S_max;
    const int64_t n_pages = (S_max + kPageTokens - 1) / kPageTokens;
    const uint8_t* page = cache + (bh * n_pages + t / kPageTokens) * kPageBytes + which * kHalfPage;
    const int tin = (int)(t % kPageTokens);
    uint8_t* dst = (which ? v_codes : k_codes) + bht * kD + 8 * w;
    if (which == 0) {
        const uint32_t word = reinterpret_cast<const uint32_t*>(page + tin * (kD / 2))[w];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            dst[2 * j] = (uint8_t)((word >> (4 * j)) & 0xFu);
            dst[2 * j + 1] = (uint8_t)((word >> (16 + 4 * j)) & 0xFu);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 2; ++i) {                     // elements 8w + 4i .. + 3 sit in one 16-bit word
            const uint32_t half = *reinterpret_cast<const uint16_t*>(page + v_word_offset(tin, 2 * w + i));
#pragma unroll
            for (int j = 0; j < 4; ++j) dst[4 * i + j] = (uint8_t)((half >> (4 * j)) & 0xFu);
        }
    }
    if (w == 0) {
        const uint32_t prm = reinterpret_cast<const uint32_t*>(page + kCodeBytes)[tin];
        (which ? v_s : k_s)[bht] = __ushort_as_half((unsigned short)(prm & 0xFFFFu));
        (which ? v_z : k_z)[bht] = __float2half_rn(-1024.0f - __half2float(__ushort_as_half((unsigned short)(prm >> 16))));
    }
}

// ------------------------------------------------------------------------------------------
// Decode attention.
// ------------------------------------------------------------------------------------------
// the four FP16 pairs of a code dword, minus the zero point: out[j] = (nibble j of the low half, of the high half)
// c = -(1024 + z), c16 = -(64 + z) = c + 960, per half
// (x & mask) | bits in one instruction.  All three sources are vector registers: with the two constants in scalar
// registers the instruction would exceed its one-scalar-operand limit and the compiler splits it in two.
__device__ __forceinline__ h2 and_or(uint32_t x, uint32_t mask, uint32_t bits)
{
    uint32_t r;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(mask), "v"(bits));
    return __builtin_bit_cast(h2, r);
}
__device__ __forceinline__ void unpack4(uint32_t word, h2 c, h2 c16, h2 (&out)[4])
{
    const h2 sixteenth = {(_Float16)0.0625f, (_Float16)0.0625f};
    const uint32_t hi = word >> 8;
    out[0] = and_or(word, 0x000F000Fu, 0x64006400u) + c;
    out[1] = and_or(word, 0x00F000F0u, 0x64006400u) * sixteenth + c16;
    out[2] = and_or(hi, 0x000F000Fu, 0x64006400u) + c;
    out[3] = and_or(hi, 0x00F000F0u, 0x64006400u) * sixteenth + c16;
}

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ h8 join(h2 a, h2 b, h2 c, h2 d)
{
    struct { h2 v[4]; } t = {{a, b, c, d}};
    return __builtin_bit_cast(h8, t);
}
constexpr int kMaxRatio = 16;                            // query heads per KV head: the columns of one MFMA
constexpr int kPartial = kD + 2;                         // floats per (split, head): 128 sums, the maximum, the weight sum
constexpr int kChunk = 32;                               // tokens per chunk: two tiles of 16 (divides the page)
// Chunks up to which four waves attend to a sequence, also in a workgroup of eight: three each.  Four waves more merge four
// (eight) partial results more, 0.7 us, and save a chunk per wave, 0.75 us, for every eight: 32 pairs of 128 tokens in a cache
// for 700 3.6 us (4.3 with eight waves at work), 300 tokens 4.8 (5.5), 512 tokens 5.6 with eight (one tile per
// instruction and four waves 5.8).
constexpr int kFewChunks = 12;

// LDS of a workgroup: per wave and used column 128 sums, the maximum and the weight sum
constexpr int decode_lds_bytes(int waves, int columns) { return waves * columns * kPartial * (int)sizeof(float); }

// NW waves.  PK: tiles side by side in the columns of a matrix instruction (2 with at most eight heads, else 1).  SPLIT:
// the sequence is cut into `ns` contiguous ranges of chunks, one workgroup each, whose (unnormalised sums, maximum,
// weight sum) go to the workspace for kv4_combine_kernel; used when there are too few (sequence, KV head) pairs to fill
// the chip (grouped-query models).  EARLY (whole sequences): every wave's first chunk is known before the length is, so its loads go out
// at once, where they would wait for that word to come from memory (4 x 256 tokens of 8 KV heads 4.42 -> 4.35 us).  Not where
// there are more workgroups than are resident: others then hide that wait, and chunks past the end are read in vain (64 x 128 of
// 32 heads 11.5 us, 11.9 with them).  Nor with NT, where what is read in vain comes from memory each time (192 pairs of 64 tokens in caches
// for 1000 3.5 us, 3.9 with them; longer ones gain 1% at most).
// NT: codes as non-temporal, for caches so large that the 256 MB memory-side cache cannot hold them until the next step (one call after
// 400 MB of other data: 64 x 1024 tokens of 32 heads 99 -> 62 us, of which 400 tokens each are live 47 -> 32, 31 x 2000 of 8 heads 31 -> 21;
// the same cache again and again, where its live part does fit, up to 7% more: 1024 pairs of 1000 tokens 24.5 and 26.2 us).
template <int NW, int PK, bool SPLIT, bool EARLY, bool NT>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(PK == 1 || NW == 8 ? 2 : 3))) void kv4_decode_kernel(
    const __half* __restrict__ q, const uint8_t* __restrict__ cache, const int32_t* __restrict__ seq_lens, __half* __restrict__ out,
    float* __restrict__ ws, int Hkv, int R, int S_max, int ns)
{
    static_assert(!(SPLIT && EARLY), "where a range begins depends on the length");
    extern __shared__ float s_part[];                    // [wave][column][kPartial]
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r16 = lane & 15, kb = lane >> 4;           // operand row (token / element slot / column) and k-block
    const int head = PK == 2 ? r16 & 7 : r16;            // this lane's column: head and, with PK = 2, which tile's scores it keeps
    const bool second = PK == 2 && r16 >= 8;
    const uint32_t bh = blockIdx.x;                      // b * Hkv + hk
    const int n_pages = (S_max + kPageTokens - 1) / kPageTokens;
    const uint8_t* stream = cache + (int64_t)bh * n_pages * kPageBytes;

    struct Chunk {
        uint4 kc[2];        // keys: token r16 of the tile, elements 32 kb ..
        uint4 vc[2];        // values: this lane's 16 bytes of the tile
        uint32_t kz[2];     // (s, z) of token r16 (zero point for unpacking)
        uint4 ks[2 / PK];   // (s, z) of tokens 4 kb .. 4 kb + 3 (scales of the scores this lane keeps)
        uint4 vp[2];        // (s, z) of tokens 4 kb .. 4 kb + 3 of the values
    };
    // Every address is a wave-uniform chunk base plus a lane offset that never changes: the loads of a chunk
    // cost no vector address arithmetic.
    const uint32_t off_kc = (uint32_t)(r16 * (kD / 2) + kb * 16), off_kz = (uint32_t)(kCodeBytes + r16 * 4);
    const uint32_t off_ks = (uint32_t)(kCodeBytes + kb * 16 + (second ? 64 : 0)), off_vc = (uint32_t)(kHalfPage + lane * 16);
    const uint32_t off_vp = (uint32_t)(kHalfPage + kCodeBytes + kb * 16);
    auto code_words = [](const uint8_t* at) __attribute__((always_inline)) {
        const uint4* p = reinterpret_cast<const uint4*>(at);
        return NT ? load_nontemporal(p) : *p;
    };
    auto load_chunk = [&](Chunk& c, int chunk) __attribute__((always_inline)) {
        const int t0 = __builtin_amdgcn_readfirstlane(chunk * kChunk);         // < n_pages * 64: inside the allocation
        const uint8_t* page = stream + (int64_t)(t0 / kPageTokens) * kPageBytes;
        const int tin = t0 % kPageTokens;                // first token of the chunk inside its page (0 or 32)
        const uint8_t* codes = page + tin * (kD / 2);    // key codes of the chunk; its value codes lie 4352 further
        const uint8_t* prm = page + tin * 4;             // (s, z) words of the chunk
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
            c.kc[tt] = code_words(codes + tt * 1024 + off_kc);
            c.kz[tt] = *reinterpret_cast<const uint32_t*>(prm + tt * 64 + off_kz);
            if (tt < 2 / PK) c.ks[tt] = *reinterpret_cast<const uint4*>(prm + tt * 64 + off_ks);
        }
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
            c.vc[tt] = code_words(codes + tt * 1024 + off_vc);
            c.vp[tt] = *reinterpret_cast<const uint4*>(prm + tt * 64 + off_vp);
        }
    };
    Chunk A, Bf;
    if constexpr (EARLY) load_chunk(A, min(wave, 2 * n_pages - 1));   // past the length: whatever is there, masked

    const int L_seq = min(max(seq_lens[bh / (uint32_t)Hkv], 0), S_max);
    __half* out_bh = out + (size_t)bh * R * kD;
    float* ws_bh = SPLIT ? ws + ((size_t)bh * ns + blockIdx.y) * R * kPartial : nullptr;
    // this workgroup's range of chunks [c0, c1) and the length it masks against
    const int chunks_seq = (L_seq + kChunk - 1) / kChunk;
    const int per_split = SPLIT ? (chunks_seq + ns - 1) / ns : chunks_seq;
    const int c0 = SPLIT ? min(chunks_seq, (int)blockIdx.y * per_split) : 0;
    const int c1 = SPLIT ? min(chunks_seq, c0 + per_split) : chunks_seq;
    const int L = min(L_seq, c1 * kChunk);
    if (c0 >= c1) {                                      // nothing to attend to: zero rows / an empty partial result
        for (int x = threadIdx.x; x < R * (SPLIT ? kPartial : kD); x += 64 * NW) {
            if (SPLIT) ws_bh[x] = x % kPartial == kD ? -1e30f : 0.f;
            else out_bh[x] = __float2half_rn(0.f);
        }
        return;
    }
    // Wave w of the nw that attend takes chunks w, w + nw, ... of the range; they all run the same number of iterations (a wave
    // without a chunk in the last one has one past the end, masked).  Two buffers alternate, and every path through the loop
    // issues a fixed number of loads, so the compiler's wait counts are exact: while a chunk is computed the next
    // one stays in flight.  (With loads under a condition it waits for everything outstanding.)
    const int nw = NW > 4 && c1 - c0 <= kFewChunks ? 4 : NW;
    const int n_iter = wave < nw ? (c1 - c0 + nw - 1) / nw : 0;
    auto chunk_of = [&](int it) __attribute__((always_inline)) { return c0 + it * nw + wave; };
    auto fetch = [&](Chunk& c, int it) __attribute__((always_inline)) { load_chunk(c, min(chunk_of(it), c1 - 1)); };
    if constexpr (!EARLY) fetch(A, 0);

    // B operand of S = K q^T: column = head (both halves of the columns with PK = 2; heads >= R: zero), k-block kb =
    // elements 32 kb .. 32 kb + 31
    h2 qv[16];
    {
        const uint4* src = reinterpret_cast<const uint4*>(q + ((size_t)bh * R + min(head, R - 1)) * kD + kb * 32);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint4 t = src[e];
            const uint32_t u[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
            for (int x = 0; x < 4; ++x) qv[4 * e + x] = __builtin_bit_cast(h2, head < R ? u[x] : 0u);
        }
    }

    float m = -1e30f, l = 0.f;                           // of this lane's column, over the tokens it has seen
    f4 acc[8];                                           // acc[4u + j][x]: element d = 16 kb + 4x + 64u + j of the column
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = (f4){0.f, 0.f, 0.f, 0.f};
    const float kScale = 1.4426950408889634f * 0.08838834764831845f;      // log2(e) / sqrt(128)

    const h2 k960 = {(_Float16)960.0f, (_Float16)960.0f};
    // One chunk of arithmetic.  MASKED: the chunk reaches past the end of the sequence (possibly entirely); the
    // parameters of tokens past the end are whatever the cache holds and must not enter the arithmetic.
    auto process_as = [&](const Chunk& cur, int chunk, auto masked_tag) __attribute__((always_inline)) {
        constexpr bool MASKED = decltype(masked_tag)::value;
        constexpr int NS = 2 / PK;                       // score vectors of a lane
        const int own = chunk * kChunk + (second ? 16 : 0) + 4 * kb;       // first token of the lane's (first) score vector
        f4 d[2];
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
            const int t0 = chunk * kChunk + tt * 16;
            uint32_t kz = cur.kz[tt];
            if (MASKED) kz = t0 + r16 < L ? kz : 0xE4000000u;               // -(1024 + 0)
            const h2 c = __builtin_bit_cast(h2, __builtin_amdgcn_perm(kz, kz, 0x07060706u));   // high half in both halves
            const h2 c16 = c + k960;
            const uint32_t kw[4] = {cur.kc[tt].x, cur.kc[tt].y, cur.kc[tt].z, cur.kc[tt].w};
            d[tt] = (f4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                h2 kh[4];
                unpack4(kw[w], c, c16, kh);              // kh[j] = elements 8w + 2j, 8w + 2j + 1 of this lane's 32
                d[tt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(join(kh[0], kh[1], kh[2], kh[3]),
                                                               join(qv[4 * w], qv[4 * w + 1], qv[4 * w + 2], qv[4 * w + 3]), d[tt], 0, 0, 0);
            }
        }
        f4 sc[NS];                                       // [x] = token own + x (+ 16 for the second vector)
        if (PK == 2) {
#pragma unroll
            for (int x = 0; x < 4; ++x) sc[0][x] = second ? d[1][x] : d[0][x];
        } else {
#pragma unroll
            for (int tt = 0; tt < NS; ++tt) sc[tt] = d[tt];
        }
        float m_new = m;
#pragma unroll
        for (int tt = 0; tt < NS; ++tt) {
            const uint32_t sw[4] = {cur.ks[tt].x, cur.ks[tt].y, cur.ks[tt].z, cur.ks[tt].w};
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const float ks = (float)half_of(sw[x]);
                sc[tt][x] *= ks * kScale;
                if (MASKED) sc[tt][x] = own + tt * 16 + x < L ? sc[tt][x] : -1e30f;
                m_new = fmaxf(m_new, sc[tt][x]);
            }
        }
        m_new = fmaxf(m_new, __shfl_xor(m_new, 16, 64));  // the four k-blocks of a column agree on the maximum
        m_new = fmaxf(m_new, __shfl_xor(m_new, 32, 64));
        if (__builtin_amdgcn_ballot_w64(m_new != m) != 0) {                  // rare once a few chunks have been seen
            const float alpha = __builtin_amdgcn_exp2f(m - m_new);
            m = m_new;
            l *= alpha;
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[i] *= alpha;
        }
        uint32_t pw[2][4];                               // (s, z) of the values, tokens 4 kb .. of both tiles
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
            const uint32_t w4[4] = {cur.vp[tt].x, cur.vp[tt].y, cur.vp[tt].z, cur.vp[tt].w};
#pragma unroll
            for (int x = 0; x < 4; ++x) pw[tt][x] = !MASKED || chunk * kChunk + tt * 16 + 4 * kb + x < L ? w4[x] : 0xE4000000u;   // else scale 0, zero point 0
        }
        uint32_t bw[2][2];                               // B operand: softmax weight * value scale, tokens 4 kb .. of both tiles
#pragma unroll
        for (int tt = 0; tt < NS; ++tt) {
            float wf[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                // a masked score is -1e30: its weight underflows to 0 unless nothing valid has been seen yet
                // (then m is -1e30 too), which the zero scale takes care of
                const float pr = __builtin_amdgcn_exp2f(sc[tt][x] - m);
                l += MASKED ? (own + tt * 16 + x < L ? pr : 0.f) : pr;
                wf[x] = pr * (float)half_of(PK == 2 ? (second ? pw[1][x] : pw[0][x]) : pw[tt][x]);
            }
            const uint32_t lo = __builtin_bit_cast(uint32_t, (h2){(_Float16)wf[0], (_Float16)wf[1]});
            const uint32_t hi = __builtin_bit_cast(uint32_t, (h2){(_Float16)wf[2], (_Float16)wf[3]});
            if (PK == 2) {                               // a column takes part with its own tile only
                bw[0][0] = second ? 0u : lo; bw[0][1] = second ? 0u : hi;
                bw[1][0] = second ? lo : 0u; bw[1][1] = second ? hi : 0u;
            } else {
                bw[tt][0] = lo; bw[tt][1] = hi;
            }
        }
        h2 vh[2][2][2][4];                               // [tile][u][h][j]: (token 4 kb + 2h, + 1) of element 4 (r16 + 16 u) + j
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
            const uint32_t vw[4] = {cur.vc[tt].x, cur.vc[tt].y, cur.vc[tt].z, cur.vc[tt].w};
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const h2 c = __builtin_bit_cast(h2, __builtin_amdgcn_perm(pw[tt][2 * h + 1], pw[tt][2 * h], 0x07060302u));
                const h2 c16 = c + k960;
#pragma unroll
                for (int u = 0; u < 2; ++u) unpack4(vw[2 * u + h], c, c16, vh[tt][u][h]);
            }
        }
        const h8 b8 = join(__builtin_bit_cast(h2, bw[0][0]), __builtin_bit_cast(h2, bw[0][1]), __builtin_bit_cast(h2, bw[1][0]),
                           __builtin_bit_cast(h2, bw[1][1]));
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc[4 * u + j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(join(vh[0][u][0][j], vh[0][u][1][j], vh[1][u][0][j], vh[1][u][1][j]),
                                                                        b8, acc[4 * u + j], 0, 0, 0);
    };
    auto process = [&](const Chunk& cur, int chunk) __attribute__((always_inline)) {
        if (chunk * kChunk + kChunk <= L) process_as(cur, chunk, std::false_type{});
        else process_as(cur, chunk, std::true_type{});
    };

    int it = 0;
    // Only a wave's last chunk can reach past the end of the sequence: every earlier one lies before the final chunk.
    for (; it + 2 < n_iter; it += 2) {
        fetch(Bf, it + 1);
        process_as(A, chunk_of(it), std::false_type{});
        fetch(A, it + 2);
        process_as(Bf, chunk_of(it + 1), std::false_type{});
    }
    if (it + 2 == n_iter) {
        fetch(Bf, it + 1);
        process_as(A, chunk_of(it), std::false_type{});
        process(Bf, chunk_of(it + 1));
    } else if (n_iter > 0) {
        process(A, chunk_of(it));
    }

    // ---- the partial results of the nw waves (and of the column halves) meet in LDS --------------
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    const int columns = PK * R;
    if (head < R && n_iter > 0) {
        float* part = s_part + (wave * columns + (second ? R : 0) + head) * kPartial;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int x = 0; x < 4; ++x) part[16 * kb + 4 * x + 64 * u + j] = acc[4 * u + j][x];
        if (kb == 0) { part[kD] = m; part[kD + 1] = l; }
    }
    __syncthreads();
    auto merge = [&](auto n_) __attribute__((always_inline)) {
        constexpr int N = decltype(n_)::value;           // partial results of a head
        for (int x = threadIdx.x; x < R * kD; x += 64 * NW) {
            const int r = x / kD, d = x % kD;
            const float* part = s_part + r * kPartial;
            float mm = -1e30f;
#pragma unroll
            for (int i = 0; i < N; ++i) mm = fmaxf(mm, part[i * R * kPartial + kD]);
            float num = 0.f, den = 0.f;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const float f = __builtin_amdgcn_exp2f(part[i * R * kPartial + kD] - mm);
                num = fmaf(part[i * R * kPartial + d], f, num);
                den = fmaf(part[i * R * kPartial + kD + 1], f, den);
            }
            if (SPLIT) {
                ws_bh[r * kPartial + d] = num;
                if (d == 0) { ws_bh[r * kPartial + kD] = mm; ws_bh[r * kPartial + kD + 1] = den; }
            } else {
                out_bh[r * kD + d] = __float2half_rn(num / den);
            }
        }
    };
    if (NW > 4 && nw == 4) merge(std::integral_constant<int, 4 * PK>());
    else merge(std::integral_constant<int, NW * PK>());
}

// Second pass of the split variant: one workgroup of 128 threads per (sequence, query head), all loads in flight at once.
constexpr int kMaxSplits = 8;
__global__ __launch_bounds__(kD) void kv4_combine_kernel(const float* __restrict__ ws, __half* __restrict__ out, int NS, int R)
{
    const uint32_t bh = blockIdx.x / (uint32_t)R;        // (sequence, KV head)
    const int r = (int)(blockIdx.x - bh * R), d = threadIdx.x;
    const float* part = ws + (size_t)bh * NS * R * kPartial + (size_t)r * kPartial;
    float acc[kMaxSplits], mx[kMaxSplits], den[kMaxSplits];
#pragma unroll
    for (int s = 0; s < kMaxSplits; ++s) {
        const float* p = part + (size_t)min(s, NS - 1) * R * kPartial;
        acc[s] = p[d]; mx[s] = p[kD]; den[s] = p[kD + 1];
    }
    float mm = mx[0];
#pragma unroll
    for (int s = 1; s < kMaxSplits; ++s) mm = fmaxf(mm, mx[s]);
    float num = 0.f, sum = 0.f;
#pragma unroll
    for (int s = 0; s < kMaxSplits; ++s) {
        const float f = s < NS ? __builtin_amdgcn_exp2f(mx[s] - mm) : 0.f;
        num = fmaf(acc[s], f, num);
        sum = fmaf(den[s], f, sum);
    }
    out[(size_t)blockIdx.x * kD + d] = __float2half_rn(sum > 0.f ? num / sum : 0.f);
}

}  // namespace

size_t kv4_cache_bytes(int64_t B, int64_t Hkv, int64_t S_max)
{
    const int64_t n_pages = (S_max + kPageTokens - 1) / kPageTokens;
    return (size_t)(B * Hkv * n_pages) * kPageBytes;
}

hipError_t launch_kv4_append(const void* k, const void* v, const int32_t* positions, int64_t B, int64_t T, int64_t Hkv,
                             int64_t S_max, uint8_t* cache, hipStream_t s)
{
    if (B * T * Hkv == 0) return hipSuccess;
    const int64_t quads = (T + 3) / 4 + 1;        // aligned quads of positions a run of T tokens can touch
    const int64_t items = B * Hkv * quads;
    if (items >= (int64_t)1 << 31) return hipErrorInvalidValue;           // (a cache of 1 TB)
    kv4_append_kernel<<<(unsigned)((items + 3) / 4), 256, 0, s>>>(static_cast<const __half*>(k), static_cast<const __half*>(v), positions,
                                                                   cache, (int)T, (int)Hkv, (int)S_max, (uint32_t)quads, (uint32_t)items);
    return hipGetLastError();
}

hipError_t launch_kv4_unpack(const uint8_t* cache, int64_t B, int64_t Hkv, int64_t S_max, uint8_t* k_codes, void* k_s, void* k_z,
                             uint8_t* v_codes, void* v_s, void* v_z, hipStream_t s)
{
    const int64_t n = B * Hkv * S_max * 32;
    if (n == 0) return hipSuccess;
    kv4_unpack_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(cache, B, Hkv, S_max, k_codes, static_cast<__half*>(k_s),
                                                                   static_cast<__half*>(k_z), v_codes, static_cast<__half*>(v_s),
                                                                   static_cast<__half*>(v_z));
    return hipGetLastError();
}

// Number of sequence ranges the split variant would use for this problem (1 = single pass).  Cutting the sequence pays only
// while the (sequence, KV head) pairs alone leave compute units idle: measured at 8 KV heads, 1 x 8192 tokens goes from 37.3 to
// 10.7 us with 8 ranges and 8 x 2048 from 12.4 to 9.1 us with 4, while at 64 sequences (512 pairs) every cut is slower than none
// (18.6 us whole, 22.2 in 2 ranges, 25.5 in 4): each range repeats the set-up and adds a second launch that merges them, 2.4 us, which
// is all that short sequences see (16 tokens 3.6 and 6.0 us; two ranges of 512 are not ahead either, 1 x 1024 of 32 heads 7.6 and 7.9).
// The host knows what a sequence may grow to, not its length, so a rule by what full caches gain loses on short sequences.  Up to 32
// workgroups from 640 tokens on, four up to 255 pairs, chunks in turn: full caches up to 1.4 times as fast (32 pairs of 1000 tokens 7.9 -> 5.8
// us), but 192 pairs of 128 in caches for 4096 3.9 -> 9.0, 32 pairs of 128 in caches for 1000 3.3 -> 5.4, 8 pairs of 400 in caches for 8192
// 5.9 -> 7.2, and 0.96 of the speed on average over 1674 sets of lengths from 16 tokens to the whole cache.
constexpr int64_t kDecodeFill = 256;
static int kv4_decode_splits(int64_t B, int64_t Hkv, int64_t S_max)
{
    const int64_t pairs = B * Hkv;
    if (pairs <= 0) return 1;
    int64_t ns = kDecodeFill / pairs;                    // about one workgroup per compute unit
    ns = std::min<int64_t>(ns, kMaxSplits);
    ns = std::min<int64_t>(ns, S_max / 512);             // ranges of at least 512 tokens
    return (int)std::max<int64_t>(ns, 1);
}

size_t kv4_decode_workspace_bytes(int64_t B, int64_t H, int64_t Hkv, int64_t S_max)
{
    const int ns = kv4_decode_splits(B, Hkv, S_max);
    return ns <= 1 ? 0 : (size_t)(B * H) * ns * kPartial * sizeof(float);
}

// Waves of a workgroup: eight where there is at most one workgroup per compute unit and a sequence that fills the cache (its
// share of the ranges) has more chunks than four waves are given, else four (32 pairs of 1023 tokens 8.3 us with eight, 9.4
// with four; 512 pairs of 1024 tokens 17.5 us with four, 20.8 with eight, whose registers and partial results allow one
// workgroup per compute unit).  Of the eight, shorter sequences use four.
static int decode_waves(int64_t workgroups, int64_t tokens) { return workgroups <= 256 && tokens > kFewChunks * kChunk ? 8 : 4; }

template <int PK, bool SPLIT, bool NT>
static void launch_decode_as(int waves, dim3 grid, const __half* q, const uint8_t* cache, const int32_t* seq_lens, int64_t Hkv, int R,
                             int64_t S_max, __half* out, float* ws, int ns, hipStream_t s)
{
    const size_t lds = (size_t)decode_lds_bytes(waves, PK * R);
    constexpr bool early = !SPLIT && !NT;
    auto* kernel = waves == 8 ? kv4_decode_kernel<8, PK, SPLIT, early, NT>
                              : grid.x <= 3 * 256 ? kv4_decode_kernel<4, PK, SPLIT, early, NT> : kv4_decode_kernel<4, PK, SPLIT, false, NT>;
    kernel<<<grid, 64 * waves, lds, s>>>(q, cache, seq_lens, out, ws, (int)Hkv, R, (int)S_max, ns);
}

template <int PK, bool SPLIT, class... Args>
static void launch_decode(bool nt, Args... args)
{
    if (nt) launch_decode_as<PK, SPLIT, true>(args...);
    else launch_decode_as<PK, SPLIT, false>(args...);
}

hipError_t launch_kv4_decode(const void* q, const uint8_t* cache, const int32_t* seq_lens, int64_t B, int64_t H, int64_t Hkv,
                             int64_t S_max, void* out, void* workspace, size_t workspace_bytes, hipStream_t s)
{
    if (B == 0) return hipSuccess;
    const __half* qh = static_cast<const __half*>(q);
    __half* oh = static_cast<__half*>(out);
    const int R = (int)(H / Hkv);
    if (R < 1 || R > kMaxRatio) return hipErrorInvalidValue;
    const int64_t pairs = B * Hkv;
    const bool nt = kv4_cache_bytes(B, Hkv, S_max) >= (size_t)24 << 20;
    const int ns = kv4_decode_splits(B, Hkv, S_max);
    if (workspace && ns > 1 && workspace_bytes >= kv4_decode_workspace_bytes(B, H, Hkv, S_max)) {
        float* ws = static_cast<float*>(workspace);
        const dim3 grid((unsigned)pairs, (unsigned)ns);
        const int waves = decode_waves(pairs * ns, S_max / ns);
        if (R <= 8) launch_decode<2, true>(nt, waves, grid, qh, cache, seq_lens, Hkv, R, S_max, oh, ws, ns, s);
        else launch_decode<1, true>(nt, waves, grid, qh, cache, seq_lens, Hkv, R, S_max, oh, ws, ns, s);
        kv4_combine_kernel<<<(unsigned)(B * H), kD, 0, s>>>(ws, oh, ns, R);
        return hipGetLastError();
    }
    const int waves = decode_waves(pairs, S_max);
    if (R <= 8) launch_decode<2, false>(nt, waves, dim3((unsigned)pairs), qh, cache, seq_lens, Hkv, R, S_max, oh, nullptr, 1, s);
    else launch_decode<1, false>(nt, waves, dim3((unsigned)pairs), qh, cache, seq_lens, Hkv, R, S_max, oh, nullptr, 1, s);
    return hipGetLastError();
}

}  // namespace qoq
