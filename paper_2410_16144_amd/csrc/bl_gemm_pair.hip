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
//     ones, tokens are read two blocks of products ahead;
//   - the epilogue reads all scales first and stores through buffer descriptors without a branch (it used to wait for LDS
//     between any two rows: 64 x 128 -> 256 took 7.8 us, now 3.7).
// Waits: every vector memory operation of the loop is one of these requests, kPer per step, and they complete in issue order;
// PairRing (bl_gemm_ring.hpp) has the counts, tests/ring_model/pair_check.cpp replays them.
//
// Measured, what was chosen before -> now (us, weights cold): 512 x 4096 -> 11008 23.9 -> 20.9, -> 4096 13.3 -> 10.6, -> 24064 42.8 -> 39.1,
// 512 x 11008 -> 4096 24.1 -> 21.5, 256 x 4096 -> 11008 18.2 -> 13.5, 128 12.8 -> 9.2, 1024 x 4096 -> 4096 19.3 -> 15.8, 2048 x 4096 -> 11008
// 78.9 -> 75, 2048 x 11008 -> 4096 68.9 -> 66.  (From 1024 tokens on the chip's power limit sets the clock.)  With its requests left out
// the loop of 512 x 11008 -> 4096 takes 17.6 of 22.6 us, on cached operands 18.6: the rest waits for the dies' L2s, which all fetch
// all tokens.  Tried and left: 6, 8 and 12 stages (ahead for 64 x 128 tiles with one or two workgroups per unit only), ordinary
// instead of streaming stores (0.5 to 1 us slower), eight waves with 64 x 256 tiles and with 32 x 256 (no launch gained 3 %).
#include <type_traits>

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
    auto request_any = [&](int i) {
        const int pair = min(i * WK + kg, pairs - 1);
        const bool half = odd && pair == pairs - 1;   // uniform: the pair is one tile, its second half brings that one again
        request(mine + (uint32_t)((i % S) * F::kStage), w_off + (uint32_t)pair * (2 * kTileBytes) - (half ? second * kTileBytes : 0),
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
    auto read_a = [&](int stage, int j) {
        AOps a;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
            a.v[mb] = *reinterpret_cast<const v4i*>(lds + a_at[j] + stage * F::kStage + mb * (4 / kA) * F::kPortion);
        return a;
    };
    auto read_w = [&](int stage) {
        WWords w;
#pragma unroll
        for (int h = 0; h < H; ++h)
            w.v[h] = *reinterpret_cast<const uint4*>(lds + w_at + stage * F::kStage + h * 1024);
        return w;
    };
    auto mask_w = [&](WWords& w, int i) {   // codes of tiles that are not there: nothing is added
        const int pair = i * WK + kg;
        if (pair >= pairs || (odd && pair == pairs - 1 && second)) {
#pragma unroll
            for (int h = 0; h < H; ++h) w.v[h] = make_uint4(0, 0, 0, 0);
        }
    };
    auto expand = [&](const WWords& w, int j) {
        BOps b;
#pragma unroll
        for (int h = 0; h < H; ++h) b.v[h] = expand_codes(j == 0 ? w.v[h].x : j == 1 ? w.v[h].y : j == 2 ? w.v[h].z : w.v[h].w);
        return b;
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
    for (int i = 0; i < kLead; ++i) request_any(i);
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
    BOps b = expand(w, 0);

    auto mfma_block = [&](const AOps& a, const BOps& b) {
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int k = 0; k < MB; ++k) {
                const int mb = h & 1 ? MB - 1 - k : k;   // one operand changes from product to product
                c[mb][h] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a.v[mb], b.v[h], c[mb][h], 0, 0, 0);
            }
    };
    auto interleave = [&]() {
#pragma unroll
        for (int i = 0; i < H * MB; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // LDS read
            __builtin_amdgcn_sched_group_barrier(0x002, (7 * H + H * MB - 1) / (H * MB), 0);   // VALU
            __builtin_amdgcn_sched_group_barrier(0x004, 1, 0);   // SALU
        }
    };
    // the operands expanded under a block's products stay there
    auto pin = [&](BOps& b) {
#pragma unroll
        for (int h = 0; h < H; ++h) asm volatile("" : "+v"(b.v[h]));
    };
    auto step = [&](auto phase, auto tail, int i) {
        constexpr int st = decltype(phase)::value % S, st1 = (st + 1) % S, stq = (st + kLead) % S;
        constexpr bool T = decltype(tail)::value;
        WWords wn;
        BOps bn;
        // block 0
        a[2] = read_a(st, 2);
        bn = expand(w, 1);
        mfma_block(a[0], b);
        interleave();
        pin(bn);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (T) {
            if (i + kLead < steps) request_any(i + kLead);
        } else {
            request(mine + (uint32_t)(stq * F::kStage), w_next, a_next, 0);
            w_next += WK * 2 * kTileBytes;
            a_next += WK * 2 * kTileK;
        }
        __builtin_amdgcn_sched_barrier(0);
        b = bn;
        // block 1
        a[3] = read_a(st, 3);
        wn = read_w(st1);
        bn = expand(w, 2);
        mfma_block(a[1], b);
        interleave();
        __builtin_amdgcn_sched_barrier(0);
        b = bn;
        // block 2
        a[0] = read_a(st1, 0);
        bn = expand(w, 3);
        mfma_block(a[2], b);
        interleave();
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (T) mask_w(wn, i + 1);
        b = bn;
        // block 3
        a[1] = read_a(st1, 1);
        bn = expand(wn, 0);
        mfma_block(a[3], b);
        interleave();
        __builtin_amdgcn_sched_barrier(0);
        b = bn;
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
__global__ __launch_bounds__(64 * WN * WK, WN * WK == 4 ? 2 : 1) void pair_gemm_kernel(const PairBatch b, const int M, const int gx) {
    int tile_x, tile_y;
    if (!tile_of_workgroup(blockIdx.x, gx, tile_x, tile_y)) return;   // uniform
    int item = 0, first = 0;
#pragma unroll
    for (int i = 0; i + 1 < kMaxGemmBatch; ++i)
        if (tile_x >= b.end[i]) { item = i + 1; first = b.end[i]; }
    pair_tile<MB, H, WN, WK, S>(b.p[item], M, tile_x - first, tile_y);
}

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

template <int MB, int H, int WN, int WK, int S>
hipError_t launch_pair_form(const GemmProblem* ps, int count, int64_t M, hipStream_t s) {
    using F = PairForm<MB, H, WN, WK, S>;
    PairBatch b;
    int64_t gx = 0;
    for (int i = 0; i < kMaxGemmBatch; ++i) {
        b.p[i] = ps[i < count ? i : count - 1];
        if (i < count) gx += ((int64_t)ps[i].row_blocks * kTileN + WN * H * 32 - 1) / (WN * H * 32);
        b.end[i] = i + 1 < count ? (int32_t)gx : INT32_MAX;
    }
    const int64_t wgs = (gx + kXcds - 1) / kXcds * kXcds * ((M + 32 * MB - 1) / (32 * MB));
    if (wgs > INT32_MAX) return hipErrorInvalidValue;
    static LdsCeiling ceiling;
    const hipError_t e = ceiling.ensure(reinterpret_cast<const void*>(&pair_gemm_kernel<MB, H, WN, WK, S>), F::kLds);
    if (e != hipSuccess) return e;
    note_kernel("pair_gemm_kernel<%d, %d, %d, %d, %d>", (int)wgs, MB, H, WN, WK, S);
    pair_gemm_kernel<MB, H, WN, WK, S><<<dim3((unsigned)wgs), dim3(64 * WN * WK), F::kLds, s>>>(b, (int)M, (int)gx);
    return hipGetLastError();
}

constexpr int pair_code(int mb, int h, int wk, int s) { return 10000 * s + 100 * (wk - 1) + 10 * mb + h; }

// Measured times of the forms (us, weights cold; relative least squares over 11065 launches, 9 to 6000 tokens, K 64 to 13000, N 64 to
// 60000, every form on each) as lines over KC, the packed tiles along K, and x, the workgroups per compute unit, counted
// with the N positions padded to a multiple of 8 (a die gets whole positions):
//     x <= 1:  t0 + a KC + e x      x <= 2:  t1 + b KC + (x - 1) (f + c KC)      beyond:  t2 + d KC x + g x + h KC
// Eight in ten estimates lie within 7 % of the measured time (64 x 384 and 64 x 512 beyond two workgroups per unit: 18 %).
// 64 x 384 and 64 x 512 are not taken with at most one workgroup per unit and more than two tiles along K: there one wave per SIMD waits
// for weights that come from memory, the lines fall short by up to a quarter, and of 8211 further launches they were ahead on one, by 3 %
// (483 x 5888 -> 15168: 64 x 512 47.3 us, estimated 34; 64 x 256 40.7; 1978 x 6080 -> 3392 48.6 and 39.9).
struct PairLine { int code, bm, bn; float t0, a, e, t1, b, f, c, t2, d, g, h; };
constexpr PairLine kPairLines[] = {
    {pair_code(2, 2, 1, 4), 64, 256, 4.16f, 0.1469f, 1.55f, 5.27f, 0.2837f, 1.12f, 0.0366f, 3.24f, 0.1351f, 2.36f, 0.1218f},
    {pair_code(2, 1, 1, 4), 64, 128, 3.33f, 0.1008f, 1.28f, 4.32f, 0.1417f, 0.35f, 0.0446f, 2.51f, 0.0832f, 1.15f, 0.0638f},
    {pair_code(2, 1, 1, 6), 64, 128, 3.66f, 0.0901f, 1.42f, 4.59f, 0.1488f, 0.33f, 0.0442f, 3.97f, 0.0902f, 1.26f, 0.0502f},
    {pair_code(2, 1, 2, 4), 64, 128, 4.02f, 0.0723f, 1.30f, 7.29f, 0.1634f, 0.16f, 0.0286f, 3.89f, 0.0948f, 2.62f, 0.0420f},
    {pair_code(1, 2, 1, 4), 32, 256, 3.53f, 0.1173f, 1.12f, 4.37f, 0.1693f, 0.22f, 0.0336f, 2.41f, 0.0864f, 1.12f, 0.0642f},
    {pair_code(2, 4, 1, 3), 64, 512, 4.92f, 0.2967f, 2.21f, 7.68f, 0.5438f, 1.89f, 0.0375f, -0.88f, 0.1313f, 5.83f, 0.4951f},
    {pair_code(2, 3, 1, 3), 64, 384, 4.13f, 0.2674f, 2.05f, 6.57f, 0.4074f, 1.16f, 0.0778f, 1.52f, 0.1353f, 3.85f, 0.3415f},
};

}  // namespace

bool gemm_pair_form_exists(int code) {
#define X(MB, H, WN, WK, S) if (code == pair_code(MB, H, WK, S)) return true;
    BL_PAIR_FORMS(X)
#undef X
    return false;
}

// 32-bit offsets: 64 rows of the output within 2^31 bytes.  (64 rows of the activations and a row block's tiles are far from it:
// K is at most 2^20.)
static_assert(BL_MAX_K <= 1 << 25, "64 activation rows within 2^31 bytes");
bool gemm_pair_takes(const GemmProblem* ps, int count) {
    for (int i = 0; i < count; ++i)
        if (ps[i].N > 1 << 23) return false;
    return true;
}

int gemm_pair_best(const GemmProblem* ps, int count, int64_t M, int cus, float& us) {
    int best = 0, KC = 0;
    for (int i = 0; i < count; ++i) KC = ps[i].KC > KC ? ps[i].KC : KC;
    const float k = (float)KC;
    for (const PairLine& l : kPairLines) {
        int64_t gx = 0;
        for (int i = 0; i < count; ++i) gx += ((int64_t)ps[i].row_blocks * kTileN + l.bn - 1) / l.bn;
        const float x = (float)((gx + kXcds - 1) / kXcds * kXcds * ((M + l.bm - 1) / l.bm)) / (float)cus;
        if (x <= 1.0f && l.bn > 256 && KC > 2) continue;
        const float est = x <= 1.0f ? l.t0 + l.a * k + l.e * x
                        : x <= 2.0f ? l.t1 + l.b * k + (x - 1.0f) * (l.f + l.c * k)
                                    : l.t2 + l.d * k * x + l.g * x + l.h * k;
        if (!best || est < us) { best = l.code; us = est; }
    }
    return best;
}

hipError_t launch_gemm_pair(const GemmProblem* ps, int count, int64_t M, int code, hipStream_t s) {
#define X(MB, H, WN, WK, S) if (code == pair_code(MB, H, WK, S)) return launch_pair_form<MB, H, WN, WK, S>(ps, count, M, s);
    BL_PAIR_FORMS(X)
#undef X
    return hipErrorInvalidValue;
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
