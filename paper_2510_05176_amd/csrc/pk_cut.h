// How many tiles of a stream a quantizer's workgroup takes where the pattern table leaves room for one or two workgroups per CU:
// what a launch takes then hangs on how many workgroups every CU gets.  Plain host code.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace pk {

struct Job {
    int n_tiles, n_streams;   // tiles of the longest stream
    int64_t tiles;            // of all streams
    bool ragged;
    float staging;            // what a workgroup's staging of the table takes, in tiles (four of 64 tokens)
};

// Tiles per workgroup, and the modelled time of the launch in tile times of a full CU.
struct Cut {
    int tiles;
    float cost;
};

// The workgroups per CU are counted as they will be (whole chunks of every stream, over 256 CUs), for one workgroup per CU, two, and so
// on.  A round of those that fit a CU side by side takes their tiles and one staging; fewer wavefronts per CU than twelve take longer,
// 1.08 times with eight and 1.54 with four, also in a last round that is not full.  Over 128 shapes (32 to 4096 streams of 64 to 8192
// vectors, 80 to 256 patterns, 96 to 256 channels) the cut so chosen takes 0.6 % longer on average than the best of ten that were
// timed.  One workgroup per CU whatever the number of streams is the best cut for 256 streams only: 288 streams x 8192 vectors at 256
// patterns K 430 us, V 332 so, 319 and 257 in chunks of 24 and of 16 tiles.
// Ragged appends: the tiles that exist in equal shares, one workgroup that ends last, half a workgroup per stream for the remainders, and
// half a staging for every workgroup behind its sequence's end.  Counted by the longest sequence they were cut far too coarsely: one
// prompt of 32k vectors among fifteen of 512, 8 heads, 256 patterns: K 395 us, V 222; 70 and 46 now.
inline Cut cut_streams(const Job &j, int by_lds, int waves, int waves_per_cu, int multiple)
{
    const int beside = std::max(1, std::min(by_lds, waves_per_cu / waves));
    auto slowness = [](int w) { return w >= 12 ? 1.f : w >= 8 ? 1.08f : 1.54f; };
    const int64_t even = std::max(j.tiles / j.n_tiles, (int64_t)1);   // streams, were all as long as the longest
    const int per_step = j.ragged ? 128 : 256;                        // (finer steps where the shares are uneven anyhow)
    const int64_t first = (even + per_step - 1) / per_step;
    Cut best = {0, 0.f};
    for (int64_t q = first; q < first + 32; ++q) {
        const int64_t chunks = per_step * q / even;
        const int t = (int)(((j.n_tiles + chunks - 1) / chunks + multiple - 1) / multiple * multiple);
        const int64_t groups = (int64_t)j.n_streams * ((j.n_tiles + t - 1) / t);
        float cost;
        if (j.ragged) {
            const float busy = (float)j.tiles / t + 0.5f * j.n_streams, empty = std::max(0.f, groups - busy);
            cost = (j.tiles / 256.f + t) * slowness(beside * waves) + j.staging * (std::max(1.f, busy / (256.f * beside)) + empty / (512.f * beside));
        } else {
            const int64_t per_cu = (groups + 255) / 256;
            const int left = (int)(per_cu % beside), taken = std::min(t, j.n_tiles);
            cost = (float)(per_cu / beside) * (beside * taken * slowness(beside * waves) + j.staging);
            if (left > 0) cost += left * taken * slowness(left * waves) + j.staging;
        }
        if (best.tiles == 0 || cost < best.cost) best = {t, cost};
        if (t == multiple) break;
    }
    return best;
}

// V quantizer beside a large table of up to 128 channels: eight waves and two blocks per pass over the table, or four waves and one
// (`plain`), by the modelled time of their cuts.  Two blocks per pass, of which the model knows nothing, are worth a fifteenth.  Few
// blocks lie better in many small workgroups (eight waves and four, 256 patterns: 8 x 2048 vectors 17.7 and 12.1 us, 128 x 256 18.3
// and 17.1; at 136 8 x 1024 12.8 and 9.3), many in large ones (128 x 1024 27.7 and 31.0, 512 x 1024 72.5 and 87.6).  Up to three blocks of
// a stream are four in pairs (1024 x 192 at 144 patterns of 128 channels 13 % slower).  Over 119 timings (8 to 2048 streams of 3
// to 256 blocks, 136 to 256 patterns) the choice is 0.4 % slower on average than the better of the two, eight waves throughout 12 %.
inline bool eight_waves(const Cut &eight, const Cut &plain, int blocks) { return blocks > 3 && eight.cost < 1.07f * plain.cost; }

// V quantizer beside a small table: two blocks per pass over it, four waves per SIMD either way.  Pays from 16 blocks per stream and 2048 in
// all on (256 streams x 8192 vectors: at 113 patterns 177 -> 165 us, 64 176 -> 162, 16 132 -> 129); below, one is faster (1024 x 320 at 64
// patterns 25.2 and 25.9, 4096 x 64 26.5 and 31.2, 8 x 4096 at 128 7.7 and 8.2).  Not with given indices (131 and 134); with
// 4 bits beyond 112 patterns only (256 x 8192 at 120 patterns 203 -> 191, at 64 196 and 203).
inline bool two_blocks_per_pass(int blocks, int n_streams, int P, int bits, bool idx_given)
{
    return !idx_given && blocks >= 16 && (int64_t)blocks * n_streams >= 2048 && (bits == 2 || P > 112);
}

}  // namespace pk
