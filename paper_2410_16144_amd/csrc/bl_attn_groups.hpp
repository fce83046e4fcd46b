// Workgroups per head of bl_attn_decode (and of bl_attn_prefill for head sizes beyond its matrix-core kernels): host arithmetic only.
#pragma once

namespace bl {

constexpr int kAttnUnits = 256;       // compute units
constexpr int kAttnMaxGroups = 64;    // as many deposits as the merge reads in one go
constexpr int kAttnOneRound = 10;     // workgroups per head from which on one per unit is enough
constexpr int kAttnLongChunks = 128;  // a cache of more than 8192 positions: one workgroup per unit streams best
constexpr int kAttnHalfRow = 64;      // head sizes up to this leave half of a cache row's lanes idle

// By heads, head size and the cache's size, not by the position: the same for every call on a cache.  The launch fills the units
// a whole number of times (rounds), never a little more than that -- units with one workgroup more than the others are the launch's
// duration.  Measured in us, caches from memory, heads of 128 unless stated:
//   - one round or two: 16 heads of 96, 3000 positions 9.9 and 10.5, 8000 16.1 and 16.4; 20 heads, 8000 19.1 and 19.7; but 64 heads, 1270
//     12.6 and 12.1, 40 heads 10.4 and 10.0: one round from 10 workgroups per head on.
//   - one round in long caches, whatever the heads, 16 000 positions: 32 heads 45.4 and 47.1, 48 heads 66.3 and 73.0, 64 90.8 and 96.2, 80 107.2 and
//     117.9, 104 137.3 and 156.0, 40 of 80 47.9 and 49.0, 28 of 160 55.1 and 56.8; where it fills 72 % of the units (90 heads, 70 %: 5000 positions
//     44.2 and 42.2) and more than half of a cache row's lanes have elements: 32 heads of 64 36.0 and 27.7, 52 of 64 63.1 and 39.3.
//   - one workgroup per head where that fills as much: 200 heads, 500 / 1270 / 5000 positions 12.8 / 24.8 / 84.2, two (400 workgroups, 144
//     units with two) 15.1 / 28.3 / 96.7; 256 heads 14.7 / 29.3 / 105.1 and 16.2 / 31.8 / 115.9.
//   - else the fewest rounds that are full: 260 heads, 5000 positions 1 / 4 / 6 workgroups per head 156.9 / 127.3 / 123.1, 300 heads 1 / 4 168.5 / 136.7,
//     180 heads 2 / 4 94.0 / 83.6.  Two rounds that are 80 % full are taken (140 heads, 1270 positions 3 / 5: 21.3 / 20.8; 104
//     heads 4 / 7: 16.8 / 16.8), more only at 85 %: 260 heads have 81 % in five rounds.
constexpr int attn_groups_per_head(int n_heads, int head_dim, int chunks) {
    const int one = kAttnUnits / n_heads;
    const bool few = head_dim > kAttnHalfRow && one * n_heads * 100 >= kAttnUnits * 72 && (one == 1 || chunks > kAttnLongChunks);
    int groups = one;
    if (one < kAttnOneRound && !few) {
        for (int rounds = 2;; ++rounds) {
            groups = rounds * kAttnUnits / n_heads;
            if (groups * n_heads * 20 >= rounds * kAttnUnits * (rounds == 2 ? 16 : 17)) break;
        }
    }
    if (groups > kAttnMaxGroups) groups = kAttnMaxGroups;
    return groups < chunks ? groups : chunks;
}

}  // namespace bl
