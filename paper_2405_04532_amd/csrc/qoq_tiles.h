// Which kernel a launch plan's code stands for where that depends on the shape (internal to the library; the host check of the
// plans reads the same rules).
#pragma once
#include "qoq_layout.h"

namespace qoq {

// Times of the two-per-CU tiles, 128 tokens x 192 (tile_m 131 without slices) or 256 channels (132), in microseconds: whole rounds of 512
// workgroups, what is left over two per compute unit or alone, each at a pace that grows with the share of the compute units that are
// busy.  Fitted to 18500 times of drawn shapes (129 ... 3000 tokens, K = 1024 ... 14336 and 28672, weights mostly from memory; standard
// deviation 4 to 8%).
inline double two_per_cu_cost(int64_t M, int64_t N, int64_t G, int mode, int64_t channels)
{
    struct Fit { double start, round, pair, alone, share, per_mb, half; };
    static const Fit fits[2][2] = {                          // [channels][mode]
        {{0.41, 7.66, 1.269, 0.740, 0.242, 0.0226, 0.604}, {0.84, 7.15, 1.063, 0.641, 0.255, 0.0347, 0.664}},
        {{1.21, 5.92, 1.574, 0.874, 0.230, 0.0109, 0.638}, {2.41, 6.53, 1.315, 0.758, 0.231, 0.0211, 0.672}}};
    const Fit& t = fits[channels == 256][mode != 0];
    const int64_t tiles = ((M + 127) / 128) * ((N + channels - 1) / channels), full = tiles / 512, rem = tiles - full * 512;
    double c = t.start + (double)full * (t.pair * (double)G + t.round);
    if (rem > 256) c += (t.alone + (t.pair - t.alone) * (t.half + (1.0 - t.half) * (double)(rem - 256) / 256.0)) * (double)G + t.round;
    else if (rem > 0) c += t.alone * (double)G * (1.0 - t.share + t.share * (double)rem / 256.0) + (full == 0 ? t.round : 0.0);
    return c + t.per_mb * (double)N * (double)G * (double)kGroup / 2.0e6;
}

// Tiles of 192 channels without slices (131): per channel two of 128 tokens per compute unit (1.0 to 1.3 of the speed of one of 256
// tokens over 142 shapes from 291 tokens on, 1.17 on average), in groups one of 256 tokens.  There the dequantizer has twice the work per
// weight, which the taller tile spreads over twice the tokens: where the estimates had two of them 6% ahead they took 0.954 of the speed
// over 71 shapes, 60 of them below 0.98 (2221 x 256 x 5248 13.3 and 14.7 us, 1500 x 4096 x 12288 86.9 and 85.9).
inline bool two_per_cu_narrow(int mode) { return mode != 0; }

// Channels of the tiles of a plan that says two per compute unit (132, without slices): 192 where they are estimated 3% ahead.
inline int two_per_cu_channels(int64_t M, int64_t N, int64_t G, int mode)
{
    return two_per_cu_cost(M, N, G, mode, 192) < 0.97 * two_per_cu_cost(M, N, G, mode, 256) ? 192 : 256;
}

// Tokens and channels of the workgroups' tiles that a plan of a compute-bound kernel (128, 129, 131, 132) with S slices runs.
inline void compute_bound_tile(int64_t M, int64_t N, int64_t G, int mode, int tile_m, int64_t S, int64_t& tokens, int64_t& channels)
{
    const bool narrow = tile_m == 131 && S == 1 && two_per_cu_narrow(mode);
    tokens = tile_m == 129 || tile_m == 132 || narrow ? 128 : 256;
    channels = tile_m == 131 ? 192 : tile_m == 132 && S == 1 ? two_per_cu_channels(M, N, G, mode) : 256;
}

}  // namespace qoq
