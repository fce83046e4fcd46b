// Workgroups per head of bl_attn_decode (and of bl_attn_prefill for head sizes beyond its matrix-core kernels): host arithmetic only.
#pragma once

namespace bl {

constexpr int kAttnUnits = 256;       // compute units
constexpr int kAttnMaxGroups = 64;    // as many deposits as the merge reads in one go
constexpr int kAttnOneRound = 10;     // workgroups per head from which on one per unit is enough

// By heads, head size and the cache's size, not by the position: the same for every call on a cache.  The launch fills the units
// a whole number of times (rounds), never a little more than that -- units with one workgroup more than the others are the launch's
// duration.  Measured in us, caches from memory by streaming loads, heads of 128 unless stated; one round and two:
//   - one round where it fills 72 % of the units and a cache row leaves at most three eighths of its lanes idle (16 lanes for head sizes up
//     to 128, 32 beyond): half as many deposits, and a unit's one workgroup keeps as many requests under way as two that wait for each
//     other's.  26 heads 1000 positions 8.20 and 9.04, 4000 13.6 and 14.5; 32 heads 1000 7.88 and 8.30, 7000 22.7 and 23.5, 12 000 34.8 and 36.2; 64 heads
//     500 8.07 and 8.32, 4000 25.1 and 25.8; 80 heads 7000 46.0 and 48.6; 120 heads 39.7 and 43.0 at 4000; 32 of 96 22.8 and 24.1 at 7000; 28 of 160 13.0 and
//     14.7 at 2000; 30 of 256 15.7 and 17.1; 200 heads 65.4 and 73.4 at 4000.  With 80 of 128 even (40 heads 18.4 and 18.2 at 4000, 7.90 and 8.34 at 500);
//     with fewer two: 52 of 72 22.9 and 21.7 at 4000, 32 of 64 12.5 and 11.1, 36 of 132 30.1 and 27.4.  Less full than that two as well: 90 heads (70 %)
//     37.3 and 33.0 at 4000, 140 (55 %) 60.8 and 52.0.  (With ordinary loads two rounds were ahead below 8192 positions.)
//   - one round from 10 workgroups per head on, whatever the lanes: 16 heads of 256 at 2000 positions 11.0 and 12.8.
//   - else the fewest rounds that are full (ordinary loads): 260 heads, 5000 positions 1 / 4 / 6 workgroups per head 156.9 / 127.3 / 123.1, 300 heads
//     1 / 4 168.5 / 136.7, 180 heads 2 / 4 94.0 / 83.6.  Two rounds that are 80 % full are taken (140 heads, 1270 positions 3 / 5: 21.3 / 20.8; 104
//     heads 4 / 7: 16.8 / 16.8), more only at 85 %: 260 heads have 81 % in five rounds.
// A prompt with head sizes above 128 follows (its tokens are bit for bit one-token calls), with ordinary loads and the launch of
// attn_prompt_units; two rounds per token and one: 28 heads of 160 behind 2000, 4 tokens 31.5 and 29.5, 16 tokens 88 and 74; 40 of 160, 9 behind 4000 168
// and 160; 30 of 256, 9 behind 2000 93 and 76; 52 of 192, 3 behind 1000 28.8 and 24.6.
constexpr int attn_groups_per_head(int n_heads, int head_dim, int chunks) {
    const int one = kAttnUnits / n_heads, row = head_dim <= 128 ? 128 : 256;
    const bool few = head_dim * 8 >= row * 5 && one * n_heads * 100 >= kAttnUnits * 72;
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

// A token's launch: `columns` x workgroups per head x (heads / columns), and workgroup (x, y, z) is head attn_head_at's y-th.  Workgroup i of a
// launch runs on die i % 8.  Where a head's part of a cache row is no whole number of 128-byte lines, neighbouring heads share lines, so every
// die takes an eighth of the heads, all workgroups of one behind those of the one before; else, and where the dies cannot have as many
// heads each, the heads go around the dies one by one.  Caches from memory, us, one by one and so: 32 heads of 48 at 1 / 5000 / 16 000 positions 3.90 and 3.42, 16.6
// and 11.9, 42.0 and 28.3; 16 of 96 at 5000 11.5 and 10.5; 32 of 120 22.6 and 19.1; 40 of 72 at 3000 14.8 and 12.8; 24 of 160 at 4000 17.7 and 16.9.  Dies with
// parts of heads, for the other numbers: 52 of 72 at 3000 17.4 and 15.4, but 12 of 100 at 1 position 4.02 and 4.17, for the division.
constexpr unsigned attn_columns(int n_heads, int head_dim) { return head_dim % 64 && n_heads % 8 == 0 ? 8u : (unsigned)n_heads; }
constexpr int attn_head_at(unsigned x, unsigned z, unsigned depth) { return (int)(x * depth + z); }

// A prompt's launch: heads times workgroups per head, padded to whole rounds of the dies (workgroup i of a launch runs on die i % 8), so
// that every query's workgroup on a piece of the cache is on the same die.
constexpr unsigned attn_prompt_units(int n_heads, int groups) { return ((unsigned)n_heads * (unsigned)groups + 7u) / 8u * 8u; }

}  // namespace bl
