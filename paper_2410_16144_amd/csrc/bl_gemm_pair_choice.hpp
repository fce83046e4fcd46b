// Which form of the paired tile kernel a launch of bl_gemm takes, and how its dies share the tiles: measured times as lines, host arithmetic only.
#pragma once
#include <cstdint>

#include "bl_gemm_ring.hpp"

namespace bl {

constexpr int kPairDies = 8, kPairRows = 64, kPairK = 64, kPairProducts = 4;   // dies; rows and k of a packed tile; products of a launch

// Workgroups of a launch of gx x gy tiles with the padding of tile_of_workgroup: the dies take whole N positions, or (halves) dies 0-3 those of
// the even token tiles and dies 4-7 those of the odd ones.
inline int64_t pair_padded_tiles(int64_t gx, int64_t gy, int halves) {
    const int64_t columns = kPairDies >> halves, rows = 1 << halves;
    return (gx + columns - 1) / columns * columns * ((gy + rows - 1) / rows * rows);
}

constexpr int pair_code(int mb, int h, int wk, int s) { return 10000 * s + 100 * (wk - 1) + 10 * mb + h; }

// A launch as the choice sees it.
struct PairLaunch {
    int64_t M = 0, widest = 0;   // tokens; weight rows of the widest product
    int     KC = 0, count = 0;   // packed tiles along the longest K; products
    int32_t row_blocks[kPairProducts] = {};
    int64_t positions(int bn) const {
        int64_t gx = 0;
        for (int i = 0; i < count; ++i) gx += ((int64_t)row_blocks[i] * kPairRows + bn - 1) / bn;
        return gx;
    }
    int64_t rows() const { return positions(1); }
};

// Measured times of the forms (us, weights cold; relative least squares over 11065 launches, 9 to 6000 tokens, K 64 to 13000, N 64 to
// 60000, every form on each) as lines over KC, the packed tiles along K, and x, the workgroups per compute unit, counted
// with the padding of tile_of_workgroup (a die gets whole positions):
//     x <= 1:  t0 + a KC + e x      x <= 2:  t1 + b KC + (x - 1) (f + c KC)      beyond:  t2 + d KC x + g x + h KC
// Eight in ten estimates lie within 7 % of the measured time (64 x 384 and 64 x 512 beyond two workgroups per unit: 18 %).
// Three stages are not enough with at most one workgroup per unit and more than two tiles along K: there one wave per SIMD waits
// for weights that come from memory, the lines fall short by up to a quarter, and of 8211 further launches they were ahead on one, by 3 %
// (483 x 5888 -> 15168: 64 x 512 47.3 us, estimated 34; 64 x 256 40.7; 1978 x 6080 -> 3392 48.6 and 39.9).  The last two have four
// stages for that case.  Their lines come from 4959 launches (24 to 2600 tokens, K 256 to 13000, N 512 to 30000, every form on each, with
// both die mappings, weights cold), less 3 %: on those launches the other lines fall 6 % short above 10 us (the clock that power left
// that day), and with 3 % off the choice was best.  With the rules below, over 10 156 launches of those ranges it takes 0.988 of the time
// (geometric mean; 0.967 of those above 15 us) that it took without the two forms and the split of the dies, is ahead by more than 3 % on 980 and
// behind by as much on 36; over 3490 with weights in the memory-side cache (150 tokens and 6e9 products up) 0.969, ahead on 952, behind on 63.
// `least`: 64 x 384 with four stages against 64 x 256 and 64 x 128 in one launch, where both apply, by tiles of K: 24 to 48 warm 1.14 of its time,
// cold 0.99; 48 to 80 1.06 and 0.93; 80 to 120 0.98 and 0.88; beyond 0.93 and 0.88.  128 x 256 where the lines take it against the other forms
// there: 32 to 40 warm 1.08, cold 1.04; 40 to 56 1.06 and 0.99; 56 to 80 1.00 and 0.97; 80 to 96 0.99 and 0.91 (1978 x 6080 -> 3392 34.2 us, 64 x 256
// 37.7; 483 x 5888 -> 15168 36.5 and 37.5); beyond 0.97 and 0.92.
struct PairLine {
    int mb, h, wk, s, bm, bn, least;   // least: fewest tiles of K
    float t0, a, e, t1, b, f, c, t2, d, g, h1;
    constexpr int code() const { return pair_code(mb, h, wk, s); }
};
constexpr PairLine kPairLines[] = {
    {2, 2, 1, 4, 64, 256, 0, 4.16f, 0.1469f, 1.55f, 5.27f, 0.2837f, 1.12f, 0.0366f, 3.24f, 0.1351f, 2.36f, 0.1218f},
    {2, 1, 1, 4, 64, 128, 0, 3.33f, 0.1008f, 1.28f, 4.32f, 0.1417f, 0.35f, 0.0446f, 2.51f, 0.0832f, 1.15f, 0.0638f},
    {2, 1, 2, 4, 64, 128, 0, 4.02f, 0.0723f, 1.30f, 7.29f, 0.1634f, 0.16f, 0.0286f, 3.89f, 0.0948f, 2.62f, 0.0420f},
    {1, 2, 1, 4, 32, 256, 0, 3.53f, 0.1173f, 1.12f, 4.37f, 0.1693f, 0.22f, 0.0336f, 2.41f, 0.0864f, 1.12f, 0.0642f},
    {2, 4, 1, 3, 64, 512, 0, 4.92f, 0.2967f, 2.21f, 7.68f, 0.5438f, 1.89f, 0.0375f, -0.88f, 0.1313f, 5.83f, 0.4951f},
    {2, 3, 1, 3, 64, 384, 0, 4.13f, 0.2674f, 2.05f, 6.57f, 0.4074f, 1.16f, 0.0778f, 1.52f, 0.1353f, 3.85f, 0.3415f},
    {2, 3, 1, 4, 64, 384, 80, 4.44f, 0.2053f, 2.52f, 10.01f, 0.4065f, 2.08f, 0.0629f, 6.46f, 0.2355f, 3.96f, 0.0986f},
    {4, 2, 1, 4, 128, 256, 80, 4.68f, 0.2508f, 3.22f, 11.42f, 0.5206f, 2.93f, 0.0887f, 5.18f, 0.2962f, 5.54f, 0.1514f},
};

// Whether a launch may split the dies over the tokens (tile_of_workgroup), and by what its estimate changes then.  A die fetches its
// tokens and its weights once: with all dies on all tokens M K + N K / 32 bytes, with half of them on each half M K / 2 + N K / 16.  It may
//   - where that leaves fewer padded tiles, the positions going by 4 and not by 8 (1024 x 4096 -> 4096, 64 x 128 tiles: 22.6 -> 18.0 us;
//     700 x 5120 -> 5120, 64 x 256: 26.9 -> 18.5);
//   - with as many tiles if the bytes are at most three quarters and the tokens more than a die's L2 holds (4 MB): 2048 x 11008 -> 4096,
//     128 x 256 tiles 66.2 -> 63.8, 64 x 256 71.4 -> 68.0; with the bytes the other way 512 x 4096 -> 24064 went from 41.0 to 41.8.
// With few tiles of K there are few bytes to save, and the outputs' stores, which the lines know least about, are the launch; measured against the
// choice without the split on 10 156 launches (weights cold) and 3490 (warm), those that became more than 6 % slower: 60 and 37.  So below 32 tiles the
// estimate needs 6 % more in its favour, below 16 the forms with three stages keep all dies on all tokens (2153 x 418 -> 10152, 64 x 512: 24.7 -> 31.5),
// and 32 x 256 always does where it is not asked for (877 x 2624 -> 4736 13.3 -> 15.8, 1599 x 2240 -> 3072 12.7 -> 14.6): 14 and 15 are left, and what
// the split gives on average stays (0.988 and 0.969 of the time).
inline bool pair_may_split(int stages, int64_t gx, int64_t gy, int64_t M, int64_t rows, int KC, float& factor) {
    const int64_t all = pair_padded_tiles(gx, gy, 0), halves = pair_padded_tiles(gx, gy, 1);
    const bool less = 5 * rows <= 32 * M;   // M / 2 + N / 16 <= 3 / 4 (M + N / 32)
    factor = less ? 0.97f : 1.03f;          // geometric mean of the launches at kPairLines, and a margin
    if (KC < 32) factor *= 1.06f;
    if (stages < 4 && KC < 16) return false;
    return halves < all || (halves == all && less && M * KC * kPairK > 4000000);
}

struct PairChoice { int code = 0, halves = 0; float us = 0.0f; };

// The form with the smallest estimate on a machine of `cus` compute units.
inline PairChoice pair_choice(const PairLaunch& p, int cus) {
    PairChoice best;
    const int64_t rows = p.rows();
    const float k = (float)p.KC;
    for (const PairLine& l : kPairLines) {
        if (p.KC < l.least || p.widest > pair_max_columns(l.mb)) continue;
        const int64_t gx = p.positions(l.bn), gy = (p.M + l.bm - 1) / l.bm;
        float factor = 1.0f;
        const int splits = l.mb > 1 && pair_may_split(l.s, gx, gy, p.M, rows, p.KC, factor) ? 2 : 1;
        for (int split = 0; split < splits; ++split) {
            const float x = (float)pair_padded_tiles(gx, gy, split) / (float)cus;
            if (x <= 1.0f && l.s < 4 && p.KC > 2) continue;
            const float est = x <= 1.0f ? l.t0 + l.a * k + l.e * x
                            : x <= 2.0f ? l.t1 + l.b * k + (x - 1.0f) * (l.f + l.c * k)
                                        : l.t2 + l.d * k * x + l.g * x + l.h1 * k;
            const float t = split ? est * factor : est;
            if (!best.code || t < best.us) best = {l.code(), split, t};
        }
    }
    return best;
}

// Whether a form that is asked for splits the dies.
inline int pair_forced_halves(const PairLaunch& p, int code) {
    const int stages = code / 10000, bm = code / 10 % 10 * 32, bn = code % 10 * 128;   // four waves along N in every form
    float factor = 1.0f;
    return pair_may_split(stages, p.positions(bn), (p.M + bm - 1) / bm, p.M, p.rows(), p.KC, factor);
}

}  // namespace bl
