// Host-side model of the wait counts of csrc/bl_gemm_pair.hip: no GPU, the constants come from the header that the kernel uses
// (csrc/bl_gemm_ring.hpp), the issue order is restated here from the kernel's text.
//
// One thread is replayed (all run the same sequence).  Vector memory operations complete in issue order; s_waitcnt vmcnt(n)
// returns when at most n are outstanding; a pair is readable behind a barrier that followed the completion of every
// thread's part of it.  Checked for every form and every number of pairs up to kMaxPairs, odd and even numbers of tiles:
//   1. whatever a step reads (its own pair, and the next one's first operands) has been published by a barrier;
//   2. a request overwrites a stage only behind a barrier that followed the stage's last read;
//   3. behind the main loop no more steps are left than the unrolled tail has, and its requests stay clear of the last pair
//      if that is half a pair, and of pairs that do not exist;
//   4. nothing is outstanding at the end, where the partial sums take the stages' place.
// "--slack": every wait leaves one operation more outstanding; the model must then fail.
#include <cstdio>
#include <cstring>
#include <vector>

#include "bl_gemm_ring.hpp"

namespace {

constexpr int kMaxPairs = 60;

template <int MB, int H, int WN, int WK, int S>
bool check(int pairs, int odd, int slack) {
    using R = bl::PairRing<MB, H, WN, S>;
    const int steps = (pairs + WK - 1) / WK;
    std::vector<int> issued;                                 // the pair (of this K group) each operation belongs to
    size_t completed = 0;
    int barriers = 0;
    std::vector<int> landed(steps + S, -1);                  // barrier behind which the pair is readable
    std::vector<int> last_read(steps + S + 1, -1);           // barriers passed when the pair was last read
    std::vector<int> stage(S, -1);                           // the pair in a stage
    bool ok = true;
    auto request = [&](int t) {
        const int old = stage[t % S];
        if (old >= 0 && last_read[old] >= barriers) ok = false;                     // not fenced
        stage[t % S] = t;
        for (int i = 0; i < R::kPer; ++i) issued.push_back(t);
    };
    auto wait = [&](int allowed) {
        const size_t must = issued.size() > (size_t)(allowed + slack) ? issued.size() - (allowed + slack) : 0;
        if (must > completed) completed = must;
    };
    auto barrier = [&]() {
        ++barriers;
        for (int t = 0; t < steps + S; ++t) {
            bool whole = false;
            for (size_t i = 0; i < issued.size(); ++i)
                if (issued[i] == t) whole = i < completed;   // the last operation of the pair decides
            if (whole && landed[t] < 0) landed[t] = barriers;
        }
    };
    auto read = [&](int t) {
        if (t >= steps) return;                              // the step behind the last one: whatever is there, never used
        if (landed[t] < 0 || landed[t] > barriers || stage[t % S] != t) ok = false;
        last_read[t] = barriers;
    };
    for (int i = 0; i < R::kLead; ++i) request(i);
    wait(R::kYounger);
    barrier();
    read(0);
    int i = 0;
    auto step = [&](bool tail) {
        read(i);
        const bool requests = !tail || i + R::kLead < steps;
        if (!tail && (i + R::kLead) * WK + WK - 1 > pairs - 1 - odd) ok = false;
        if (requests) request(i + R::kLead);
        read(i);
        read(i + 1);
        wait(requests ? R::kYounger : 0);
        barrier();
        ++i;
    };
    while ((i + S + R::kLead) * WK <= pairs - odd)
        for (int k = 0; k < S; ++k) step(false);
    if (steps - i > S + R::kLead) ok = false;
    while (i < steps) step(true);
    // requests of the prologue beyond the end are waited for by the first steps; behind the loop everything has completed
    if (completed != issued.size()) ok = false;
    return ok;
}

template <int MB, int H, int WN, int WK, int S>
int run(int slack) {
    int bad = 0;
    for (int pairs = 1; pairs <= kMaxPairs; ++pairs)
        for (int odd = 0; odd < 2; ++odd)
            if (!check<MB, H, WN, WK, S>(pairs, odd, slack)) ++bad;
    printf("<%d, %d, %d, %d, %d>: %d failing\n", MB, H, WN, WK, S, bad);
    return bad;
}

}  // namespace

int main(int argc, char** argv) {
    const int slack = argc > 1 && !strcmp(argv[1], "--slack") ? 1 : 0;
    int bad = 0;
#define X(MB, H, WN, WK, S) bad += run<MB, H, WN, WK, S>(slack);
    BL_PAIR_FORMS(X)
    BL_PAIR_WIDE_FORMS(X)
#undef X
    printf("%d failing cases\n", bad);
    return bad ? 1 : 0;
}
