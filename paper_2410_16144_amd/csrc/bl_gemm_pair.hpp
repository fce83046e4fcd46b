// The paired-tile kernel of bl_gemm as a template: a workgroup's tile, the launch of one form.  What it does and what bounds it stand in
// bl_gemm_pair.hip, which builds the forms for any number of tokens and chooses; bl_gemm_pair_wide.hip builds those of one workgroup
// per compute unit.
#pragma once
#include <type_traits>

#include "bl_gemm_pair_choice.hpp"
#include "bl_gemm_ring.hpp"
#include "bl_internal.hpp"

namespace bl {

namespace {

typedef int v16i __attribute__((ext_vector_type(16)));

template <int N, int I = 0, typename Fn>
__device__ __forceinline__ void unroll(Fn&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        unroll<N, I + 1>(f);
    }
}

template <int MB, int H, int WN, int WK, int S>
struct PairForm {
    using Ring = PairRing<MB, H, WN, S>;
    static constexpr int kWaves = WN * WK;
    static constexpr int kPortion = Ring::kPer * 1024;             // one wave's part of a stage: its weights, its share of the tokens
    static constexpr int kStage = kWaves * kPortion;
    static constexpr int kRing = S * kStage;
    static constexpr int kShare = MB * H / WK;
    static constexpr int kExchange = WK == 1 ? 0 : WN * (WK - 1) * kShare * 16 * 64 * 4;
    static constexpr int kBase = kRing > kExchange ? kRing : kExchange;
    static constexpr int kLds = kBase + 32 * MB * 8;
    static_assert(WK == 1 || MB * H % WK == 0, "the K groups share out the wave's MFMA tiles for the final sum");
};

template <int MB, int H, int WN, int WK, int S>
__device__ __forceinline__ void pair_tile(const GemmProblem& p, const int M, const int tile_x, const int tile_y) {
    using F = PairForm<MB, H, WN, WK, S>;
    using Ring = typename F::Ring;
    constexpr int BM = 32 * MB, kA = Ring::kA, kLead = Ring::kLead;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    float* s_scale = reinterpret_cast<float*>(lds + F::kBase);
    int* s_qsum = reinterpret_cast<int*>(s_scale + BM);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_n = wave % WN, kg = wave / WN;
    const int KC = p.KC, pairs = (KC + 1) >> 1, odd = KC & 1;
    const int steps = (pairs + WK - 1) / WK;          // step i: pairs WK i .. WK i + WK - 1, one per K group
    const int m0 = tile_y * BM;
    const int row0 = (tile_x * WN + wave_n) * H * 32; // this wave's first row of W
    const int l32 = lane & 31, second = lane >> 5;
    const int64_t qs = (int64_t)KC * kTileK;

    // ---- requests
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)lds;
    const uint32_t mine = lds0 + (uint32_t)(wave * F::kPortion);
    // One M0 (the LDS address) serves up to four requests: the instruction's immediate offset counts on both sides, so it
    // is taken off the source.  Request r of a pair (weights of 32-row block r, then tokens) has offset 1024 (r % 4).
    const uint8_t* wbase[H];
#pragma unroll
    for (int h = 0; h < H; ++h) {
        const int block = row0 / 32 + h;   // row blocks beyond the matrix are clamped to a valid one and dropped in the epilogue
        wbase[h] = uniform_ptr(reinterpret_cast<const uint8_t*>(p.packed) + (int64_t)min(block >> 1, p.row_blocks - 1) * KC * kTileBytes +
                           (block & 1) * 512 - (h % 4) * 1024);
    }
    const uint32_t w_off = (uint32_t)(second * kTileBytes + l32 * 16);   // lanes 0-31: the pair's first tile, 32-63: its second
    constexpr int kBias = 4096;
    const uint8_t* abase = uniform_ptr(reinterpret_cast<const uint8_t*>(p.q) + (int64_t)m0 * qs - kBias);
    uint32_t a_off[kA];
#pragma unroll
    for (int k = 0; k < kA; ++k) {
        const int row = min(m0 + (wave_n * kA + k) * 8 + (lane >> 3), M - 1) - m0;   // clamped rows: never stored
        a_off[k] = (uint32_t)(row * qs) + ((lane & 7) ^ (lane >> 3) ^ ((wave_n * kA + k) & 1)) * 16 + kBias - (H + k) % 4 * 1024;
    }
    const uint32_t a_second = ((lane & 7) ^ (lane >> 3)) & 4 ? kTileK : 0;   // lanes that bring the pair's second tile
    auto request = [&](uint32_t dst, uint32_t woff, const uint8_t* a, uint32_t back) {
        constexpr int kPer = Ring::kPer;
        uint32_t off[kPer];
        const uint8_t* src[kPer];
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            off[r] = r < H ? woff : a_off[r < H ? 0 : r - H] - back;
            src[r] = r < H ? wbase[r < H ? r : 0] : a;
        }
        load_to_lds(dst, off, src);
    };
    // any pair, also the last one and those behind it (a valid pair instead: its codes are taken as 0)
    auto request_any = [&](int i, int stage) {
        const int pair = min(i * WK + kg, pairs - 1);
        const bool half = odd && pair == pairs - 1;   // uniform: the pair is one tile, its second half brings that one again
        request(mine + (uint32_t)(stage * F::kStage), w_off + (uint32_t)pair * (2 * kTileBytes) - (half ? second * kTileBytes : 0),
                abase + (int64_t)pair * (2 * kTileK), half ? a_second : 0);
    };

    // ---- operands
    const int slab = l32 >> 3;
    const uint32_t a_lane = (uint32_t)((kg * WN + slab / kA) * F::kPortion + H * 1024 + (slab % kA) * 1024 + (l32 & 7) * 128);
    uint32_t a_at[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) a_at[j] = a_lane + (uint32_t)(((4 * second + j) ^ (l32 & 7) ^ (slab & 1)) * 16);
    const uint32_t w_at = (uint32_t)(wave * F::kPortion) + (uint32_t)lane * 16;
    struct AOps { v4i v[MB]; };
    struct WWords { uint4 v[H]; };
    struct BOps { v4i v[H]; };
    auto read_token = [&](int stage, int j, int mb) {
        return *reinterpret_cast<const v4i*>(lds + a_at[j] + stage * F::kStage + mb * (4 / kA) * F::kPortion);
    };
    auto read_a = [&](int stage, int j) {
        AOps a;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) a.v[mb] = read_token(stage, j, mb);
        return a;
    };
    auto read_word = [&](int stage, int h) { return *reinterpret_cast<const uint4*>(lds + w_at + stage * F::kStage + h * 1024); };
    auto read_w = [&](int stage) {
        WWords w;
#pragma unroll
        for (int h = 0; h < H; ++h) w.v[h] = read_word(stage, h);
        return w;
    };
    auto mask_w = [&](WWords& w, int i) {   // codes of tiles that are not there: nothing is added
        const int pair = i * WK + kg;
        if (pair >= pairs || (odd && pair == pairs - 1 && second)) {
#pragma unroll
            for (int h = 0; h < H; ++h) w.v[h] = make_uint4(0, 0, 0, 0);
        }
    };

    v16i c[MB][H];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < H; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) c[i][j][r] = 0;

    if (tid < BM) {   // published by the prologue's barrier
        const int m = min(m0 + tid, M - 1);
        s_scale[tid] = p.w_scale * p.a_scale[m];
        s_qsum[tid] = p.q_sum[m];
    }
#pragma unroll
    for (int i = 0; i < kLead; ++i) request_any(i, i);
    wait_vm<Ring::kYounger>();
    __syncthreads();

    // the main loop's sources: pair kLead WK + kg on
    uint32_t w_next = w_off + (uint32_t)(kLead * WK + kg) * (2 * kTileBytes);
    const uint8_t* a_next = abase + (int64_t)(kLead * WK + kg) * (2 * kTileK);

    AOps a[4];
    a[0] = read_a(0, 0);
    a[1] = read_a(0, 1);
    WWords w = read_w(0);
    mask_w(w, 0);
    BOps b;
#pragma unroll
    for (int h = 0; h < H; ++h) b.v[h] = expand_codes(w.v[h].x);

    // One step: four blocks of MB * H products, and beside each product its share of everything else, held there by a scheduling barrier:
    // a token operand of the block after the next, some of the next block's codes, in block 0 a request of pair i + kLead (right
    // behind the barrier: spread over three blocks the forms with three stages had too little of the step left for them).  The last
    // steps, which ask for any pair or for none, do so in one place.  (M0 written anew for every request, a branch around each one in the last
    // steps and a mapping to tiles by two divisions: 307 x 4032 -> 6464 15.2 us, so 14.6; 437 x 3072 -> 4160 11.6 and 11.0; 598 x 768 -> 11008
    // 10.7 and 9.9; 2048 x 11008 -> 4096 66.9 and 65.9.)
    auto step = [&](auto phase, auto tail, int i) {
        constexpr int st = decltype(phase)::value % S, st1 = (st + 1) % S, stq = (st + kLead) % S;
        constexpr bool T = decltype(tail)::value;
        constexpr int kSlots = MB * H, kCodes = 4 / MB, kPer = Ring::kPer, kSpread = H >= 2 ? 2 : 1;   // products of a block; operand words expanded beside each
        static_assert(4 % MB == 0, "a block's products share out the next block's 4 H operand words");
        WWords wn;
        uint32_t m0 = 0;   // the present request's LDS address register
        unroll<4>([&](auto block) {
            constexpr int j = decltype(block)::value;
            BOps bn;
            unroll<kSlots>([&](auto slot) {
                constexpr int t = decltype(slot)::value, h = t / MB;
                constexpr int mb = h & 1 ? MB - 1 - t % MB : t % MB;   // one operand changes from product to product
                c[mb][h] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[j].v[mb], b.v[h], c[mb][h], 0, 0, 0);
                if constexpr (t % kSpread == 0 && t / kSpread < MB) a[(j + 2) % 4].v[t / kSpread] = read_token(j < 2 ? st : st1, (j + 2) % 4, t / kSpread);
                if constexpr (j == 1 && t >= kSlots - H) wn.v[t - (kSlots - H)] = read_word(st1, t - (kSlots - H));
                unroll<kCodes>([&](auto word) {
                    constexpr int e = t * kCodes + decltype(word)::value, eh = e / 4, q = e % 4;
                    const uint4& from = j == 3 ? wn.v[eh] : w.v[eh];
                    const uint32_t codes = j == 0 ? from.y : j == 1 ? from.z : j == 2 ? from.w : from.x;
                    int x = (int)((codes >> 2 * q) & 0x03030303u);
                    asm volatile("" : "+v"(x));   // expanded here, under this product
                    bn.v[eh][q] = x;
                });
                if constexpr (j == 0 && !T) {
                    constexpr int r0 = t * kPer / kSlots, r1 = (t + 1) * kPer / kSlots;
                    unroll<r1 - r0>([&](auto which) {
                        constexpr int r = r0 + decltype(which)::value;
                        const uint32_t off = r < H ? w_next : a_off[r < H ? 0 : r - H];
                        const uint8_t* src = r < H ? wbase[r < H ? r : 0] : a_next;
                        if constexpr (r % 4 == 0) m0 = load_first_to_lds(mine + (uint32_t)(stq * F::kStage + r * 1024), off, src);
                        else load_next_to_lds<r % 4 * 1024>(m0, off, src);
                    });
                }
                if constexpr (j == 0 && T && t == 0)
                    if (i + kLead < steps) request_any(i + kLead, stq);
                __builtin_amdgcn_sched_barrier(0);
            });
            if constexpr (T && j == 2) mask_w(wn, i + 1);
            b = bn;
        });
        if constexpr (!T) {
            w_next += WK * 2 * kTileBytes;
            a_next += WK * 2 * kTileK;
        }
        w = wn;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (T) {
            if (i + kLead < steps) wait_vm<Ring::kYounger>();
            else wait_vm<0>();
        } else {
            wait_vm<Ring::kYounger>();
        }
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    int i = 0;
    for (; (i + S + kLead) * WK <= pairs - odd; i += S)
        unroll<S>([&](auto phase) { step(phase, std::false_type{}, i + decltype(phase)::value); });
    unroll<S + kLead>([&](auto phase) {
        if (i + decltype(phase)::value < steps) step(phase, std::true_type{}, i + decltype(phase)::value);
    });

    if constexpr (WK > 1) {
        // The K groups add up their accumulators through LDS (the ring is free now: nothing is requested beyond the end).  MFMA
        // tile t = mb * H + nb of a wave is finished by group t % WK, one receiving group at a time.
        int* ex = reinterpret_cast<int*>(lds);
        constexpr int kShare = F::kShare;
#pragma unroll
        for (int owner = 0; owner < WK; ++owner) {
            __syncthreads();
            if (kg != owner) {
                const int sender = kg < owner ? kg : kg - 1;   // 0 .. WK-2
#pragma unroll
                for (int t = owner, i = 0; t < MB * H; t += WK, ++i)
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4)
                        *reinterpret_cast<v4i*>(&ex[(((((wave_n * (WK - 1) + sender) * kShare) + i) * 4 + r4) * 64 + lane) * 4]) =
                            v4i{c[t / H][t % H][4 * r4], c[t / H][t % H][4 * r4 + 1], c[t / H][t % H][4 * r4 + 2], c[t / H][t % H][4 * r4 + 3]};
            }
            __syncthreads();
            if (kg == owner) {
#pragma unroll
                for (int sender = 0; sender < WK - 1; ++sender)
#pragma unroll
                    for (int t = owner, i = 0; t < MB * H; t += WK, ++i)
#pragma unroll
                        for (int r4 = 0; r4 < 4; ++r4) {
                            const v4i v = *reinterpret_cast<const v4i*>(&ex[(((((wave_n * (WK - 1) + sender) * kShare) + i) * 4 + r4) * 64 + lane) * 4]);
#pragma unroll
                            for (int r = 0; r < 4; ++r) c[t / H][t % H][4 * r4 + r] += v[r];
                        }
            }
        }
    }

    // epilogue: register r of a 32x32 tile holds row 8*(r/4) + 4*(lane/32) + r%4, column lane%32.  All scales are read before
    // the first store (read row by row between the stores they cost an LDS round trip each).
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    f32x4 sc[MB][4];
    v4i qsum[MB][4];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            sc[mb][r4] = *reinterpret_cast<const f32x4*>(s_scale + mb * 32 + 8 * r4 + 4 * second);
            qsum[mb][r4] = *reinterpret_cast<const v4i*>(s_qsum + mb * 32 + 8 * r4 + 4 * second);
        }
    // Buffer stores: rows beyond M and columns beyond N lie behind the buffer's end (by 2^31 in the columns' case) and are dropped by
    // the hardware's bounds check, so there is no branch per row.  Streaming (nontemporal): tens of MB of output must not push
    // the operands out of L2.  Row by row, a row's 32-column pieces one behind the other: where N is no multiple of 32 they
    // share lines, and with all rows of one piece first such lines went out to memory twice (1921 x 548 -> 28610: 172 us for 101).
    uint32_t at0[H];
#pragma unroll
    for (int nb = 0; nb < H; ++nb) {
        const int n = row0 + nb * 32 + l32;   // n >= N covers padding rows and clamped row blocks
        at0[nb] = n < p.N ? ((uint32_t)(4 * second) * (uint32_t)p.N + (uint32_t)n) * 4u : 0x80000000u;
    }
    auto store = [&](void* to, auto acc) {
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<uint8_t*>(to) + (int64_t)m0 * p.N * 4, 0,
                                                            (int)((uint32_t)min(M - m0, BM) * (uint32_t)p.N * 4u), 0x00027000);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const uint32_t row = (uint32_t)(mb * 32 + 8 * (r >> 2) + (r & 3)) * (uint32_t)p.N * 4u;
#pragma unroll
                for (int nb = 0; nb < H; ++nb) {
                    if (WK > 1 && (mb * H + nb) % WK != kg) continue;   // another K group finishes this tile
                    const int v = c[mb][nb][r] - qsum[mb][r >> 2][r & 3];
                    if constexpr (decltype(acc)::value) __builtin_amdgcn_raw_buffer_store_b32((uint32_t)v, rsrc, at0[nb] + row, 0, 2);
                    else __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint((float)v * sc[mb][r >> 2][r & 3]), rsrc, at0[nb] + row, 0, 2);
                }
            }
    };
    store(p.out, std::false_type{});
    if (p.acc) store(p.acc, std::true_type{});
}

struct PairBatch {
    GemmProblem p[kMaxGemmBatch];
    int32_t     end[kMaxGemmBatch];
};

template <int MB, int H, int WN, int WK, int S>
__global__ __launch_bounds__(64 * WN * WK, WN * WK == 4 ? 2 : 1) void pair_gemm_kernel(const PairBatch b, const int M, const int gx, const int halves) {
    int tile_x, tile_y;
    if (!tile_of_workgroup(blockIdx.x, gx, (M + 32 * MB - 1) / (32 * MB), halves, tile_x, tile_y)) return;   // uniform
    int item = 0, first = 0;
#pragma unroll
    for (int i = 0; i + 1 < kMaxGemmBatch; ++i)
        if (tile_x >= b.end[i]) { item = i + 1; first = b.end[i]; }
    pair_tile<MB, H, WN, WK, S>(b.p[item], M, tile_x - first, tile_y);
}

template <int MB, int H, int WN, int WK, int S>
hipError_t launch_pair_form(const GemmProblem* ps, int count, int64_t M, int halves, hipStream_t s) {
    using F = PairForm<MB, H, WN, WK, S>;
    PairBatch b;
    int64_t gx = 0;
    for (int i = 0; i < kMaxGemmBatch; ++i) {
        b.p[i] = ps[i < count ? i : count - 1];
        if (i < count) gx += ((int64_t)ps[i].row_blocks * kTileN + WN * H * 32 - 1) / (WN * H * 32);
        b.end[i] = i + 1 < count ? (int32_t)gx : INT32_MAX;
    }
    const int64_t wgs = pair_padded_tiles(gx, (M + 32 * MB - 1) / (32 * MB), halves);
    if (wgs > INT32_MAX) return hipErrorInvalidValue;
    static LdsCeiling ceiling;
    const hipError_t e = ceiling.ensure(reinterpret_cast<const void*>(&pair_gemm_kernel<MB, H, WN, WK, S>), F::kLds);
    if (e != hipSuccess) return e;
    note_kernel("pair_gemm_kernel<%d, %d, %d, %d, %d>", (int)wgs, MB, H, WN, WK, S);
    pair_gemm_kernel<MB, H, WN, WK, S><<<dim3((unsigned)wgs), dim3(64 * WN * WK), F::kLds, s>>>(b, (int)M, (int)gx, halves);
    return hipGetLastError();
}

}  // namespace

}  // namespace bl
