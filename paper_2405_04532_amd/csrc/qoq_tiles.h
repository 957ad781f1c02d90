// Which kernel a launch plan's code stands for where that depends on the shape, and in which form it loads its weights (internal to the
// library; the host check of the plans reads the same rules).
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
// tokens over 142 shapes from 291 tokens on, 1.18 on average), in groups one of 256 tokens.  There the dequantizer has twice the work per
// weight, which the taller tile spreads over twice the tokens: where the estimates had two of them 6% ahead they took 0.954 of the speed
// over 71 shapes, 60 of them below 0.98 (2221 x 256 x 5248 13.3 and 14.7 us, 1500 x 4096 x 12288 86.9 and 85.9).
inline bool two_per_cu_narrow(int mode) { return mode != 0; }

// Channels of the tiles of a plan that says two per compute unit (132, without slices): 192 where they are estimated 3% ahead, from ten groups
// on (per channel five).  Shorter rows lie outside of what the estimates were fitted to; there the third more workgroups, each with a start
// and an epilogue, cost what the last round saves: at 5 to 9 groups 0.975 of the speed on average over 33 shapes, 20 of them below 0.98 (1586 x 768 x 11200
// 25.9 and 27.5 us), from 10 on 1.08 over 150, 1 below; per channel at two to four 1.0 over 39, 7 below (623 x 256 x 19520 13.0 and 14.3), from
// five on 1.11 over 175, 2 below (328 x 13696 x 27584 150 and 126).
inline int two_per_cu_channels(int64_t M, int64_t N, int64_t G, int mode)
{
    if (G < (mode == 0 ? 10 : 5)) return 256;
    return two_per_cu_cost(M, N, G, mode, 192) < 0.97 * two_per_cu_cost(M, N, G, mode, 256) ? 192 : 256;
}

// Whether a per-channel plan of four-wave tiles with one workgroup per compute unit (128 or 129, no slices, `cost` estimated) is better off with two
// of 128 x 192.  In place of 256 x 256 they are 1.15 to 1.5 times as fast over 55 shapes.  In place of 128 x 256, 1.2 times (160, none
// below 0.98), with two exceptions: rows of five groups or less where they are more than 256 and the wider ones were not, so that the compute units' second workgroup
// comes on top (0.96 of the speed over 31 shapes, 1920 x 384 x 3648 12.4 and 13.1 us), and layers from 28 MB on, whose weights come from
// memory to few token tiles, where more and narrower workgroups do not help (0.963 over 23, 256 x 4736 x 18752 32.1 and 35.8; 1.03 to
// 1.08 over 9 of 20 to 25 MB).
inline bool narrow_instead_of(int tile_m, int64_t M, int64_t N, int64_t G, int mode, double cost)
{
    if (!two_per_cu_narrow(mode) || (tile_m != 128 && tile_m != 129)) return false;
    if (tile_m == 129 && ((G < 6 && ((M + 127) / 128) * ((N + 191) / 192) > 256) || N * G * (kGroup / 2) >= 28000000)) return false;
    return two_per_cu_cost(M, N, G, mode, 192) < 0.97 * cost;
}

// Tokens and channels of the workgroups' tiles that a plan of a compute-bound kernel (128, 129, 131, 132) with S slices runs.
inline void compute_bound_tile(int64_t M, int64_t N, int64_t G, int mode, int tile_m, int64_t S, int64_t& tokens, int64_t& channels)
{
    const bool narrow = tile_m == 131 && S == 1 && two_per_cu_narrow(mode);
    tokens = tile_m == 129 || tile_m == 132 || narrow ? 128 : 256;
    channels = tile_m == 131 ? 192 : tile_m == 132 && S == 1 ? two_per_cu_channels(M, N, G, mode) : 256;
}

// Weights that are read once, by one token tile, and are so many that the memory-side cache (256 MB) does not hold them
// until the model's next step: loaded as non-temporal they leave it alone, which is faster (us from memory, before and after: 16 x 8192 x
// 57344 47.8 -> 40.5, 37 51.8 -> 46, 8 x 28672 x 8192 26.9 -> 25.6).  Where a program's weights do fit, it is slower: the activation-
// stationary kernels without slices by 2 to 5% (16 x 4096 x 22016 10.8 and 11.1; from memory 12.7 and 11.8), which therefore do it
// from 40 MB on (below, 4096 x 12288 gains nothing either way), the others by up to 20%, which do it from 96 MB on (46 x 11136 x
// 18688, 104 MB again and again, 34.4 and 37.8).
constexpr int64_t kPassByWhole = (int64_t)40 << 20, kPassBy = (int64_t)96 << 20;
inline bool weights_pass_by(int64_t N, int64_t K, int64_t token_tiles, int64_t least) { return token_tiles == 1 && N * K / 2 >= least; }

}  // namespace qoq
