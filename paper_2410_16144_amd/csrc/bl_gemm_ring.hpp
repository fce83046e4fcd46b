// Ring depths and wait counts of the prefill kernels' operand pipelines (bl_gemm.hip, bl_gemm_narrow.hip), as compile-time
// constants in a header of their own: the kernels take them from here, and so does the host-side model that replays the
// kernels' issue order and checks every wait (tests/ring_model).  Plain C++, no device code.  First the one of bl_gemm.hip.
//
// The pipeline, per thread and K step i (one packed tile per K group):
//   - activations: the tile of step i + kLead is requested (global -> LDS, kRQ loads per thread of a loader wave, written
//     as assembly, so the compiler neither sees, drops nor moves them) into stage (i + kLead) % kStages;
//   - weights: the packed tiles of step i + kWR - 1 are loaded into registers (NT ordinary loads: the compiler sees
//     them and may DROP the ones whose values are never used, which is what happens in the loop's unrolled tail);
//   - the barrier that ends step i publishes the activation tile of step i + 2 (step i + 1 reads its first half during
//     its predecessor's second half).  Vector memory operations complete in issue order and one counter (vmcnt)
//     counts all of them, so "tile i + 2 has landed" is "at most n operations are outstanding", n = the operations
//     this thread has issued since that tile's request.
#pragma once

namespace bl {

template <int MB, int H, int WK, int WN>
struct GemmRing {
    static constexpr int kNT = (H + 1) / 2;            // packed 64-row tiles a wave loads per step
    static constexpr int kStages = WK == 1 ? 8 : 6;    // LDS stages of the activation ring
    // a stage is WK tiles of 32 MB token rows = WK * 2 MB slabs of 1 KiB, one wave-load each, dealt to the WN * WK waves:
    // a loader wave issues kRQ of them per step (the other waves none)
    static constexpr int kRQ = (WK * 2 * MB + WN * WK - 1) / (WN * WK);
    static constexpr int kLead = 4;                    // the tile of step i + kLead is requested during step i
    static constexpr int kWR = kNT == 1 ? 8 : 4;       // register ring of packed weight tiles, steps i .. i + kWR - 1
    static constexpr int kUnroll = 8;                  // steps per trip of the main loop; the rest is the tail
    // Main loop: since the request of tile i + 2 (first thing in step i + 2 - kLead) the thread has issued that step's
    // weight loads and kLead - 2 whole steps: (kLead - 2) * (kRQ + kNT) + kNT operations.  The count below leaves the
    // kNT out, i.e. it also waits for the weight tiles of the requesting step: stricter than needed, never weaker.
    static constexpr int kYounger = (kLead - 2) * (kRQ + kNT);
    // Tail (the steps after the last whole trip): their weight loads feed nothing and the compiler removes them, so only
    // the requests are sure to have been issued: kLead - 2 steps of kRQ each.
    static constexpr int kYoungerTail = (kLead - 2) * kRQ;
    // Prologue: kWR - 1 steps of weight loads, then the requests of tiles 0 .. kLead - 1 back to back.  The wait leaves
    // only the requests of tiles 3 .. kLead - 1 outstanding, so tiles 0, 1 AND 2 have landed: the barrier that ends step 0
    // is meant to publish tile 2, but only kRQ + kNT + kRQ operations follow its request by then, fewer than kYounger.
    static constexpr int kPrologueWait = (kLead - 3) * kRQ;

    static_assert(kLead >= 3, "the prologue waits for all but the last requested tiles");
    static_assert(kStages >= kLead + 1, "a stage is rewritten only after the barrier that ended its last read");
    static_assert(kYounger < 16 && kYoungerTail < 16 && kPrologueWait < 16, "fits the low vmcnt field");
    static_assert(kUnroll % kWR == 0, "register ring slots are compile-time phases of the unrolled loop");
};

// The kernel for few tokens (bl_gemm_narrow.hip): every wave has stages of its own in LDS and waits for nobody.  Step i's
// requests (kPerStep of them per thread, all assembly) go into stage i % D, D steps ahead; when step i is consumed, the steps
// behind it that have been requested are i + 1 .. i + D - 1, all of them as long as that many are left, so kYounger operations may
// be outstanding; towards the end nothing may.  Whatever else a thread has outstanding was issued before its first request.
template <int T, int RH, int D>
struct NarrowRing {
    static constexpr int kPerStep = RH + T / 8;        // 1 KiB each: the weights of 32 RH rows, the activations of T tokens
    static constexpr int kYounger = (D - 1) * kPerStep;
    static constexpr bool steady(int steps, int i) { return D > 1 && steps - i >= D; }   // kYounger may be outstanding at step i, else 0
    static_assert(kYounger < 64, "fits the wait counter");
};

// The tile kernel with paired packed tiles (bl_gemm_pair.hip): weights and activations both global -> LDS, kPer requests per
// thread and step, all assembly.  Step i requests pair i + kLead into stage (i + kLead) % S; the barrier that ends it publishes
// pair i + 2, behind which the pairs i + 3 .. i + kLead have been requested.
template <int MB, int H, int WN, int S>
struct PairRing {
    static constexpr int kA = 4 * MB / WN;             // 1 KiB each: a wave's share of 32 MB tokens x 128 k
    static constexpr int kPer = H + kA;                // ... and its weights, 32 H rows x 128 k
    static constexpr int kLead = S - 1;                // a stage is requested anew in the step behind the one that read it last
    static constexpr int kYounger = (kLead - 2) * kPer;
    static_assert(kA >= 1 && kA <= 4 && kLead >= 2 && kYounger < 64, "every wave brings tokens; fits the wait counter");
};

// The widest matrix that a form of 32 mb tokens takes: its epilogue reaches a tile's rows of the output by 32-bit byte offsets, of which
// those from 2^31 on stand for columns that are not there, so the 32 mb rows have to end by then.  (Beyond 2^23 columns no form is
// taken: the tile kernel of bl_gemm.hip is ahead there.)
constexpr long long pair_max_columns(int mb) { return (1LL << 31) / (4 * 32 * (mb < 2 ? 2 : mb)); }

// The forms that are built, X(MB, H, WN, WK, S): wave tile of 32 MB tokens x 32 H weight rows, WN waves along N, WK along K, S
// stages.
#define BL_PAIR_FORMS(X) \
    X(2, 2, 4, 1, 4) X(2, 1, 4, 1, 4) X(2, 1, 4, 1, 6) X(2, 1, 4, 2, 4) X(1, 2, 4, 1, 4) X(2, 4, 4, 1, 3) X(2, 3, 4, 1, 3)

// ... of bl_gemm_pair_wide.hip, one workgroup per compute unit:
#define BL_PAIR_WIDE_FORMS(X) X(4, 2, 4, 1, 4) X(2, 3, 4, 1, 4)

// The matrix-core decode kernel's one-off copy of the quantized activations into LDS (bl_gemv.hip, QMODE 1): the copy's
// global -> LDS loads are issued first, then one batch of U weight tiles; the wait that precedes the barrier allows
// exactly those U loads to be outstanding.
template <int U>
struct LdsCopyWait {
    static constexpr int kYounger = U;
    static_assert(U >= 0 && U < 16, "fits the low vmcnt field");
};

}  // namespace bl
