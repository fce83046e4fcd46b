// bl_gemm on tiles, from a few dozen tokens up: the tile kernel of bl_gemm.hip with two packed tiles (128 k) per step.
//
// What bounds that kernel at a few hundred tokens is instruction issue and waiting, not the matrix cores: a wave issues one
// instruction in 4.3 to 5 cycles whatever it is, and a 32-cycle product hides five of them (measured: max(32, 8 + 4.8 n) cycles for a
// product and n other instructions of ONE wave; two waves of a SIMD: 8 per product + 4 per vector instruction, summed), and it had
// eight per product, a barrier per 64 k, operand reads of two cycles for one (below) and 4 us of epilogue.  Here, per wave
// and step (64 x 64 tile: 16 products, 85 other instructions):
//   - a pair of tiles needs no lane exchange: lanes 0-31 carry word j of their row's 16 bytes in the pair's first tile, lanes
//     32-63 word j of the second, and the tokens' operand is chosen alike;
//   - weights and tokens both go from global memory straight into LDS (load_to_lds: one M0 for four pieces), several pairs ahead;
//     scalar and 32-bit lane offsets only.  Weights are read by the wave that brought them, tokens by all waves along N;
//   - tokens: a row's 128 bytes as eight 16-byte chunks, chunk c at place c ^ (row % 8) ^ (row / 8 % 2), so that the sixteen
//     lanes of a cycle meet sixteen columns (without the last term every read took two cycles for one: 1.4 of 3.2 million LDS
//     cycles of a launch were conflicts);
//   - the next operands (codes to int8: 7 vector instructions per 16 codes) are expanded under the products of the present
//     ones, tokens are read two blocks of products ahead; every product has its share of all that beside it, held there by a scheduling
//     barrier (reads and requests in runs kept the wave from its next product: 512 x 4096 -> 24064 43.4 -> 41.1 us, 1024 x 4096 -> 11008 41.2 -> 39.6,
//     2048 x 4096 -> 12288 80.3 -> 77.5 with 64 x 384 tiles);
//   - the epilogue reads all scales first and stores through buffer descriptors without a branch (it used to wait for LDS
//     between any two rows: 64 x 128 -> 256 took 7.8 us, now 3.7).
// Waits: every vector memory operation of the loop is one of these requests, kPer per step, and they complete in issue order;
// PairRing (bl_gemm_ring.hpp) has the counts, tests/ring_model/pair_check.cpp replays them.
//
// Measured, what was chosen before -> now (us, weights cold): 512 x 4096 -> 11008 23.9 -> 20.9, -> 4096 13.3 -> 10.6, -> 24064 42.8 -> 39.1,
// 512 x 11008 -> 4096 24.1 -> 21.5, 256 x 4096 -> 11008 18.2 -> 13.5, 128 12.8 -> 9.2, 1024 x 4096 -> 4096 19.3 -> 15.8, 2048 x 4096 -> 11008
// 78.9 -> 75, 2048 x 11008 -> 4096 68.9 -> 66 (since then 128 x 256 tiles, bl_gemm_pair_wide.hip).  From 1024 tokens on the chip's power limit sets
// the clock: 2048 x 11008 -> 4096 70 us at 1.72 GHz, with all tokens zero 53 at 2.28; products alone, in registers, make 4.3 POP/s on such
// tokens and 4.9 on zeros.  With its requests left out
// the loop of 512 x 11008 -> 4096 takes 17.6 of 22.6 us, on cached operands 18.6: the rest waits for the dies' L2s, which all fetch
// all tokens.  Tried and left: 6, 8 and 12 stages (ahead for 64 x 128 tiles with one or two workgroups per unit only), ordinary
// instead of streaming stores (0.5 to 1 us slower), eight waves with 64 x 256 tiles and with 32 x 256 (no launch gained 3 %).
#include "bl_gemm_pair.hpp"

namespace bl {

namespace {

__global__ __launch_bounds__(256, 2) void mixed_pair_gemm_kernel(const GemmMixed b, const int M) {
    int tile_x, tile_y, item = 0, first = 0;
    if ((int)blockIdx.x < b.wgs) {   // uniform
        if (!tile_of_workgroup(blockIdx.x, b.gx, tile_x, tile_y)) return;
#pragma unroll
        for (int i = 0; i + 1 < kMaxGemmBatch; ++i)
            if (tile_x >= b.end[i]) { item = i + 1; first = b.end[i]; }
        pair_tile<2, 2, 4, 1, 4>(b.p[item], M, tile_x - first, tile_y);
    } else {
        if (!tile_of_workgroup(blockIdx.x - b.wgs, b.small_gx, tile_x, tile_y)) return;
#pragma unroll
        for (int i = 0; i + 1 < kMaxGemmBatch; ++i)
            if (tile_x >= b.small_end[i]) { item = i + 1; first = b.small_end[i]; }
        pair_tile<2, 1, 4, 1, 4>(b.p[item], M, tile_x - first + b.small_first[item], tile_y);
    }
}

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
    {2, 1, 1, 6, 64, 128, 0, 3.66f, 0.0901f, 1.42f, 4.59f, 0.1488f, 0.33f, 0.0442f, 3.97f, 0.0902f, 1.26f, 0.0502f},
    {2, 1, 2, 4, 64, 128, 0, 4.02f, 0.0723f, 1.30f, 7.29f, 0.1634f, 0.16f, 0.0286f, 3.89f, 0.0948f, 2.62f, 0.0420f},
    {1, 2, 1, 4, 32, 256, 0, 3.53f, 0.1173f, 1.12f, 4.37f, 0.1693f, 0.22f, 0.0336f, 2.41f, 0.0864f, 1.12f, 0.0642f},
    {2, 4, 1, 3, 64, 512, 0, 4.92f, 0.2967f, 2.21f, 7.68f, 0.5438f, 1.89f, 0.0375f, -0.88f, 0.1313f, 5.83f, 0.4951f},
    {2, 3, 1, 3, 64, 384, 0, 4.13f, 0.2674f, 2.05f, 6.57f, 0.4074f, 1.16f, 0.0778f, 1.52f, 0.1353f, 3.85f, 0.3415f},
    {2, 3, 1, 4, 64, 384, 80, 4.44f, 0.2053f, 2.52f, 10.01f, 0.4065f, 2.08f, 0.0629f, 6.46f, 0.2355f, 3.96f, 0.0986f},
    {4, 2, 1, 4, 128, 256, 80, 4.68f, 0.2508f, 3.22f, 11.42f, 0.5206f, 2.93f, 0.0887f, 5.18f, 0.2962f, 5.54f, 0.1514f},
};

}  // namespace

bool gemm_pair_form_exists(int code) {
#define X(MB, H, WN, WK, S) if (code == pair_code(MB, H, WK, S)) return true;
    BL_PAIR_FORMS(X)
    BL_PAIR_WIDE_FORMS(X)
#undef X
    return false;
}

// Whether a form of 32 mb tokens takes a launch: its matrices are no wider than pair_max_columns.  (A tile's activation rows and a row
// block's tiles are far from 32-bit offsets' ends: K is at most 2^20.)
static_assert((int64_t)BL_MAX_K * 32 * 4 <= (int64_t)1 << 31, "128 activation rows within 2^31 bytes");
bool gemm_pair_takes(const GemmProblem* ps, int count, int mb) {
    for (int i = 0; i < count; ++i)
        if (ps[i].N > pair_max_columns(mb)) return false;
    return true;
}

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
static bool pair_may_split(int stages, int64_t gx, int64_t gy, int64_t M, int64_t rows, int KC, float& factor) {
    const int64_t all = gemm_padded_tiles(gx, gy, 0), halves = gemm_padded_tiles(gx, gy, 1);
    const bool less = 5 * rows <= 32 * M;   // M / 2 + N / 16 <= 3 / 4 (M + N / 32)
    factor = less ? 0.97f : 1.03f;          // geometric mean of the launches at kPairLines, and a margin
    if (KC < 32) factor *= 1.06f;
    if (stages < 4 && KC < 16) return false;
    return halves < all || (halves == all && less && M * KC * kTileK > 4000000);
}

static int64_t pair_positions(const GemmProblem* ps, int count, int bn) {
    int64_t gx = 0;
    for (int i = 0; i < count; ++i) gx += ((int64_t)ps[i].row_blocks * kTileN + bn - 1) / bn;
    return gx;
}

int gemm_pair_best(const GemmProblem* ps, int count, int64_t M, int cus, float& us, int& halves) {
    int best = 0, KC = 0;
    int64_t rows = 0;
    for (int i = 0; i < count; ++i) {
        KC = ps[i].KC > KC ? ps[i].KC : KC;
        rows += (int64_t)ps[i].row_blocks * kTileN;
    }
    const float k = (float)KC;
    for (const PairLine& l : kPairLines) {
        if (KC < l.least || !gemm_pair_takes(ps, count, l.mb)) continue;
        const int64_t gx = pair_positions(ps, count, l.bn), gy = (M + l.bm - 1) / l.bm;
        float factor;
        const int splits = l.mb > 1 && pair_may_split(l.s, gx, gy, M, rows, KC, factor) ? 2 : 1;
        for (int split = 0; split < splits; ++split) {
            const float x = (float)gemm_padded_tiles(gx, gy, split) / (float)cus;
            if (x <= 1.0f && l.s < 4 && KC > 2) continue;
            const float est = x <= 1.0f ? l.t0 + l.a * k + l.e * x
                            : x <= 2.0f ? l.t1 + l.b * k + (x - 1.0f) * (l.f + l.c * k)
                                        : l.t2 + l.d * k * x + l.g * x + l.h1 * k;
            const float t = split ? est * factor : est;
            if (!best || t < us) { best = l.code(); us = t; halves = split; }
        }
    }
    return best;
}

int gemm_pair_halves(const GemmProblem* ps, int count, int64_t M, int code) {
    for (const PairLine& l : kPairLines) {
        if (l.code() != code) continue;
        int64_t rows = 0;
        int KC = 0;
        for (int i = 0; i < count; ++i) {
            KC = ps[i].KC > KC ? ps[i].KC : KC;
            rows += (int64_t)ps[i].row_blocks * kTileN;
        }
        float factor;
        return pair_may_split(l.s, pair_positions(ps, count, l.bn), (M + l.bm - 1) / l.bm, M, rows, KC, factor);
    }
    return 0;
}

hipError_t launch_gemm_pair(const GemmProblem* ps, int count, int64_t M, int code, int halves, hipStream_t s) {
#define X(MB, H, WN, WK, S) if (code == pair_code(MB, H, WK, S)) return launch_pair_form<MB, H, WN, WK, S>(ps, count, M, halves, s);
    BL_PAIR_FORMS(X)
#undef X
    return launch_gemm_pair_wide(ps, count, M, code, halves, s);
}

hipError_t launch_gemm_pair_mixed(const GemmMixed& b, int64_t M, hipStream_t s) {
    using F = PairForm<2, 2, 4, 1, 4>;
    static LdsCeiling ceiling;
    const hipError_t e = ceiling.ensure(reinterpret_cast<const void*>(&mixed_pair_gemm_kernel), F::kLds);
    if (e != hipSuccess) return e;
    const unsigned grid = (unsigned)(b.wgs + (b.small_gx + kXcds - 1) / kXcds * kXcds * ((M + 63) / 64));
    note_kernel("mixed_pair_gemm_kernel", (int)grid);
    mixed_pair_gemm_kernel<<<dim3(grid), dim3(256), F::kLds, s>>>(b, (int)M);
    return hipGetLastError();
}

}  // namespace bl
