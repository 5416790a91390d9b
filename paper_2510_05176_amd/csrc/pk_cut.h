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
inline Cut cut_streams(Job j, int by_lds, int waves, int waves_per_cu, int multiple)
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

// V quantizer beside a large table of up to 128 channels: eight waves that take two blocks per pass over the table, or four waves and one
// (`plain`), by the modelled time of their cuts.  Two blocks per pass take some four fifths of the time per block (264 x 8320 vectors at 256
// patterns 0.76 of four waves' time, 128 x 4096 at 136 0.93).  Few blocks lie better in many small workgroups (eight waves and four, 256
// patterns: 8 x 2048 vectors 17.7 and 12.1 us; at 136 8 x 1024 12.8 and 9.3, 96 x 576 1.09 of the time), many in large ones (256
// patterns: 128 x 1024 27.7 and 31.0 us, 512 x 1024 72.5 and 87.6; 320 x 1024 at 136 of 96 channels 36 and 43).  Up to three blocks of a stream
// are four in pairs (1024 x 192 at 144 patterns 13 % slower).  Over 119 timings (8 to 2048 streams of 3 to 256 blocks, 136 to 256
// patterns) the choice is 0.5 % slower on average than the better of the two, eight waves throughout 12 %.
inline Cut cut_pairs(Job j, int by_lds, int waves, int waves_per_cu, int multiple)
{
    constexpr float kTile = 0.8f;
    j.staging /= kTile;
    Cut c = cut_streams(j, by_lds, waves, waves_per_cu, multiple);
    c.cost *= kTile;
    return c;
}
inline bool eight_waves(const Cut &eight, const Cut &plain, int blocks) { return blocks > 3 && eight.cost < plain.cost; }

inline int tiles_per_wg(int n_tiles, int n_streams)
{
    // aim at ~1024 workgroups, each staging the pattern table once for at most 16 tiles; a job of very many
    // tiles (8 or more resident rounds even then) takes 32 or 64 per workgroup: fewer prologues, and the last,
    // partly filled round stays a small share (-4 % on the V kernel of config 3, worse on small jobs)
    const int64_t total = (int64_t)n_tiles * n_streams;
    const int cap = total >= 64 * 768 * 8 ? 64 : total >= 32 * 768 * 8 ? 32 : 16;
    const int t = (int)((total + 1023) / 1024);
    return t < 1 ? 1 : (t > cap ? cap : t);
}

// V quantizer beside a small table: two blocks per pass over it, four waves per SIMD either way.  A wave takes its unit of all of its
// workgroup's blocks, so what counts is how many those are: 1024 streams of 2, 4, 6, 8, 10, 14 and 16 blocks take 1.03, 1.02, 1.01, 0.98,
// 0.98, 0.95 and 0.96 of one block's time at 64 patterns, 1.01, 0.99, 0.97, 0.96, 0.95, 0.95 and 0.94 at 128, 1.03, 1.04, 1.02, 1.00,
// 1.01, 0.98 and 0.99 at 16; of 3 and 5 blocks, the last of which is searched twice, 1.16 and 1.13.  Workgroups get an even number of blocks
// for it, which changes their rounds of 1024: 512 streams of 10 blocks, in five and five or six and four, 1.09; 320 of 16, of which fives make
// more than a round and sixes do not, 0.76.  Not with given indices (256 x 8192 vectors 131 and 134 us); with 4 bits beyond 112
// patterns only (1024 x 1024 vectors 0.93 at 120 patterns, 1.08 at 64).
inline bool two_blocks_per_pass(int blocks, int n_streams, int P, int bits, bool idx_given)
{
    if (idx_given || (bits == 4 && P <= 112)) return false;
    const int t = tiles_per_wg(blocks, n_streams), even = (t + 1) / 2 * 2, own = std::min(t, blocks);
    auto rounds = [&](int tiles) { return ((int64_t)n_streams * ((blocks + tiles - 1) / tiles) + 1023) / 1024; };
    const int64_t one = rounds(t) * own, two = rounds(even) * ((std::min(even, blocks) + 1) / 2 * 2);
    return two < 0.9f * one || (own >= (P > 64 ? 6 : P > 32 ? 8 : 12) && two <= 1.06f * one);
}

}  // namespace pk
