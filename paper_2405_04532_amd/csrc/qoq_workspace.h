// The GEMM workspace, where workgroups that share an output meet, and what its size follows from (internal to the library).
//
// [arrival counters: kCounterBytes][partial tiles].  The counters of every call lie in the first kCounterBytes, its partial
// tiles behind them, whatever the shape and the kernel: calls of different shapes take turns in one workspace, each
// relies on its counters being zero and leaves them zero, and none may find an earlier call's sums there.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace qoq {

constexpr size_t kCounterBytes = (size_t)256 << 10;
constexpr int64_t kMaxCounters = (int64_t)(kCounterBytes / sizeof(int));

// Units (64-channel block, group) per workgroup of the streaming kernels when `nwg` workgroups share a token tile of `tile`.
// With more blocks than counters (600000 channels at 400 tokens) a workgroup takes whole blocks, and nothing is exchanged.
inline int64_t stream_units_per_workgroup(int64_t M, int64_t N, int64_t G, int tile, int64_t nwg)
{
    const int64_t blocks = N / 64, upw = (blocks * G + nwg - 1) / nwg;
    if ((M + tile - 1) / tile * blocks <= kMaxCounters) return upw;
    return (upw + G - 1) / G * G;
}

// Workspace for a call that makes one of its own: what its plan exchanges.  0 as well where the plan without eight-wave
// kernels exchanges nothing and is not further behind than zeroing the counters takes; without a workspace a call takes that one.
size_t gemm_fresh_workspace_bytes(int64_t M, int64_t N, int64_t K, int mode);

// 16-token fragments of a token tile of the eight-wave kernels (qoq_gemm_mma8.h): equal tiles of three to nine.
inline int eight_wave_fragments(int64_t M)
{
    const int64_t frags = (M + 15) / 16, tiles = (frags + 8) / 9, mf = (frags + tiles - 1) / tiles;
    return mf < 3 ? 3 : (int)mf;
}

// Channels of a tile of the eight-wave kernels: 128, or 256 where tiles of 128 (times the S k-slices) need more than a round of
// 256 workgroups.
inline int64_t eight_wave_width(int64_t M, int64_t N, int64_t S)
{
    const int64_t tm = 16 * eight_wave_fragments(M);
    return (M + tm - 1) / tm * ((N + 127) / 128) * S <= 256 ? 128 : 256;
}

}  // namespace qoq
