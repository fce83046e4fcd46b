// bl_gemm on tiles, from a few dozen tokens up: the tile kernel of bl_gemm.hip with two packed tiles (128 k) per step.
//
// What bounds that kernel at a few hundred tokens is instruction issue and waiting, not the matrix cores: a wave issues one
// instruction in 4.3 to 5 cycles whatever it is, and a 32-cycle product hides five of them (measured: max(32, 8 + 4.8 n) cycles for a
// product and n other instructions of ONE wave; two waves of a SIMD: 8 per product + 4 per vector instruction, summed), and it had
// eight per product, a barrier per 64 k, operand reads of two cycles for one (below) and 4 us of epilogue.  Here, per wave
// and step (64 x 64 tile: 16 products, 87 other instructions):
//   - a pair of tiles needs no lane exchange: lanes 0-31 carry word j of their row's 16 bytes in the pair's first tile, lanes
//     32-63 word j of the second, and the tokens' operand is chosen alike;
//   - weights and tokens both go from global memory straight into LDS (load_to_lds, load_first_to_lds: one M0 for up to four pieces), several pairs ahead;
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
// Measured, what was chosen before -> this kernel's first form (us, weights cold): 512 x 4096 -> 11008 23.9 -> 20.9, -> 4096 13.3 -> 10.6, -> 24064 42.8 -> 39.1,
// 512 x 11008 -> 4096 24.1 -> 21.5, 256 x 4096 -> 11008 18.2 -> 13.5, 128 12.8 -> 9.2, 1024 x 4096 -> 4096 19.3 -> 15.8, 2048 x 4096 -> 11008
// 78.9 -> 75, 2048 x 11008 -> 4096 68.9 -> 66 (since then 128 x 256 tiles, bl_gemm_pair_wide.hip).  From 1024 tokens on the chip's power limit sets
// the clock: 2048 x 11008 -> 4096 70 us at 1.72 GHz, with all tokens zero 53 at 2.28; products alone, in registers, make 4.3 POP/s on such
// tokens and 4.9 on zeros.  With its requests left out
// the loop of 512 x 11008 -> 4096 takes 17.6 of 22.6 us, on cached operands 18.6: the rest waits for the dies' L2s, which all fetch
// all tokens.  Tried and left: 8 and 12 stages, ordinary instead of streaming stores (0.5 to 1 us slower), eight waves with 64 x 256 tiles and with
// 32 x 256 (no launch gained 3 %).  64 x 128 with six stages is there for bl_set_tuning only: 1.06 of the time of its siblings with weights cold,
// 1.08 warm, and the best form by 2 % on 196 of 10 156 and 7 of 3490 launches.
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

namespace {

PairLaunch pair_launch(const GemmProblem* ps, int count, int64_t M) {
    PairLaunch l;
    l.M = M;
    l.count = count;
    for (int i = 0; i < count; ++i) {
        l.row_blocks[i] = ps[i].row_blocks;
        l.KC = ps[i].KC > l.KC ? ps[i].KC : l.KC;
        l.widest = ps[i].N > l.widest ? ps[i].N : l.widest;
    }
    return l;
}
static_assert(kPairDies == kXcds && kPairRows == kTileN && kPairK == kTileK && kPairProducts == kMaxGemmBatch, "the choice's own constants");

}  // namespace

int gemm_pair_best(const GemmProblem* ps, int count, int64_t M, int cus, float& us, int& halves) {
    const PairChoice c = pair_choice(pair_launch(ps, count, M), cus);
    us = c.us;
    halves = c.halves;
    return c.code;
}

int gemm_pair_halves(const GemmProblem* ps, int count, int64_t M, int code) { return pair_forced_halves(pair_launch(ps, count, M), code); }

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
