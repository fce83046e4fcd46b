// bl_gemm for few tokens: from one token past the decode kernels up to a few hundred.
//
// What bounds this range is neither the matrix cores nor the weight stream but waiting: a few dozen tokens times one
// matrix are 10 MB of weights and 1 us of matrix-core time, and the tile kernel of bl_gemm.hip, whose waves walk K
// together with a barrier per step and share one activation tile, took 14 to 18 us for it whatever the token count.
// So here the waves of a workgroup divide K instead: a workgroup owns a strip of 32*RH weight rows and T tokens, its W
// waves take every W-th PAIR of packed tiles (128 k), each wave stages its own operands in its own piece of LDS
// (global -> LDS, D pairs ahead) and waits for nobody until the W partial sums meet in LDS at the end.
//
// One step of a wave = one pair (tiles 2i, 2i+1): RH KiB of packed weights and T x 128 bytes of activations.  With a pair the
// matrix operands need no lane exchange: in v_mfma_i32_32x32x32_i8 lanes 0-31 carry 16 contraction indices and lanes
// 32-63 the other 16, and here lanes 0-31 read word j of their row's 16 bytes in tile 2i, lanes 32-63 word j of tile 2i+1.
//   weights:     LDS image as loaded (lane-linear); operand read = 16 bytes per lane, two contiguous 512-byte runs;
//   activations: a token's 128 bytes as eight 16-byte chunks, chunk c at position c ^ (row % 8) ^ (row / 8 % 2): a read of
//                one chunk of many rows takes sixteen lanes per cycle (256 bytes), which meet sixteen different columns.
//                (With c ^ (row % 8) alone rows r and r + 8 met in one column: every read took twice its cycles.)
// The operands of a step are all read into registers before its products start, so the step's piece of LDS is free for
// the next request while they run.
//
// Waits.  Every vector memory operation of the loop is one of the requests below, written as assembly (the compiler
// answers loads into LDS that it can see with a wait for everything), kPerStep of them per step, and they complete in
// issue order: when step i is consumed, the steps behind it that have been requested are i+1 .. i+D-1, so at most
// (D-1)*kPerStep operations may be outstanding, none at all once the last steps are reached (NarrowRing).
#include "bl_gemm_ring.hpp"
#include "bl_internal.hpp"

namespace bl {

namespace {

typedef int v16i __attribute__((ext_vector_type(16)));

// Up to four products over the same tokens: their strips side by side, `end[i]` the first strip behind product i
// (INT32_MAX behind the last one in use).
struct NarrowBatch {
    GemmProblem p[kMaxGemmBatch];
    int32_t     end[kMaxGemmBatch];
};

template <int T, int RH, int W, int D>
struct NarrowForm {
    static_assert(T % 16 == 0 && T <= 64 && (RH == 1 || RH == 2 || RH == 4), "tokens in sixteens, half or whole row blocks");
    static constexpr int kMB = (T + 31) / 32;            // 32-token matrix tiles (the last one half empty if T % 32 == 16)
    static constexpr int kStage = RH * 1024 + T * 128;   // bytes of one step: weights, then activations
    using Ring = NarrowRing<T, RH, D>;                   // requests and wait counts: bl_gemm_ring.hpp, checked by a host-side model
    static_assert(kStage == Ring::kPerStep * 1024, "a step's requests fill its stage");
    static constexpr int kQuads = RH * T / 8;            // accumulator register quadruples that hold tokens < T
    static constexpr int kRing = W * D * kStage;
    // the final exchange goes in as many phases as keep it within half of a compute unit's LDS (two workgroups per unit)
    static constexpr int kPhases = (W * kQuads + 63) / 64;
    static constexpr int kPhaseQuads = kQuads / kPhases;
    static constexpr int kExchange = W * kPhaseQuads * 64 * 16;
    static constexpr int kSets = (kPhaseQuads + W - 1) / W;    // quadruples a wave finishes per phase
    static_assert(kQuads % kPhases == 0, "equal phases");
    static constexpr int kLds = kRing > kExchange ? kRing : kExchange;
    static_assert(kLds <= kMaxDecodeLds, "fits the LDS ceiling");
};

template <int T, int RH, int W, int D>
__global__ __launch_bounds__(64 * W) void gemm_narrow_kernel(const NarrowBatch b, const int M, const int gx) {
    using F = NarrowForm<T, RH, W, D>;
    constexpr int MB = F::kMB;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];

    // workgroup -> (strip, token block): the die depends on the strip only, as in tile_of_workgroup
    const int gxh = (gx + kXcds - 1) / kXcds;
    const int rest = blockIdx.x / kXcds;
    int strip = (rest % gxh) * kXcds + blockIdx.x % kXcds;
    const int m0 = rest / gxh * T;
    if (strip >= gx) return;   // uniform: the grid is padded to a multiple of 8 strips
    int item = 0, first = 0;
#pragma unroll
    for (int i = 0; i + 1 < kMaxGemmBatch; ++i)
        if (strip >= b.end[i]) { item = i + 1; first = b.end[i]; }
    const GemmProblem& p = b.p[item];
    strip -= first;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int KC = p.KC;
    const int rb = RH == 1 ? strip >> 1 : strip * (RH / 2);   // (first) packed row block
    const int half0 = RH == 1 ? (strip & 1) : 0;            // RH 1: which half of it
    const int row0 = rb * kTileN + half0 * 32;
    const uint32_t qs = (uint32_t)KC * kTileK;              // activation row stride in bytes (M * qs < 2^31)
    const int pairs = (KC + 1) >> 1;
    const int steps = pairs > wave ? (pairs - wave + W - 1) / W : 0;   // this wave's pairs: wave, wave + W, ...
    const bool odd = KC & 1;                                // the last pair is one tile: its second half is masked

    const uint8_t* wbase = reinterpret_cast<const uint8_t*>(p.packed) + (int64_t)rb * KC * kTileBytes;
    // RH 4: the second row block, clamped to one that exists (its rows lie beyond N and are never stored)
    const int64_t block2 = RH == 4 && rb + 1 < p.row_blocks ? (int64_t)KC * kTileBytes : 0;
    const uint8_t* qbase = reinterpret_cast<const uint8_t*>(p.q);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)lds;
    const uint32_t ring0 = lds0 + (uint32_t)(wave * D * F::kStage);
    // per-lane byte offsets of the requests, and what to take off them in the masked half of an odd last pair
    const int second = lane >> 5;
    const uint32_t w_off = RH >= 2 ? (uint32_t)lane * 16 : (uint32_t)(second * kTileBytes + (half0 * 32 + (lane & 31)) * 16);
    uint32_t a_off[T / 8];
    constexpr int kBias = 4096;
    const int arow = lane >> 3, chunk = (lane & 7) ^ arow;  // 8 rows per request, position lane % 8 of its row
#pragma unroll
    for (int s = 0; s < T / 8; ++s)   // (the last two terms: a piece's place behind one M0, kept positive)
        a_off[s] = (uint32_t)min(m0 + 8 * s + arow, M - 1) * qs + (chunk ^ (s & 1)) * 16 + kBias - (RH + s) % 4 * 1024;
    const uint32_t a_back = chunk >= 4 ? kTileK : 0;

    auto request = [&](int i) {
        const int pair = wave + i * W;
        const bool last = odd && pair == pairs - 1;         // uniform
        const uint8_t* wsrc = wbase + (int64_t)pair * (2 * kTileBytes);
        const uint8_t* qsrc = qbase + (int64_t)pair * (2 * kTileK) - kBias;
        const uint32_t back = last ? a_back : 0;
        uint32_t off[F::Ring::kPerStep];
        const uint8_t* src[F::Ring::kPerStep];
#pragma unroll
        for (int r = 0; r < RH; ++r) {
            if constexpr (RH >= 2) {   // even pieces: the pair's first tile; odd ones: its second
                off[r] = w_off;
                src[r] = (r >= 2 ? wsrc + block2 : wsrc) - r / 2 * 2048;
                if (r & 1) src[r] = last ? src[r] - kTileBytes : src[r];   // a tile that is not there: any valid one, its codes are dropped
            } else {
                off[r] = last && second ? w_off - kTileBytes : w_off;
                src[r] = wsrc;
            }
        }
#pragma unroll
        for (int s = 0; s < T / 8; ++s) {
            off[RH + s] = a_off[s] - back;
            src[RH + s] = qsrc;
        }
        load_to_lds(ring0 + (uint32_t)((D == 1 ? 0 : i % D) * F::kStage), off, src);
    };

    v16i c[MB][RH];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < RH; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) c[i][j][r] = 0;

    const int l32 = lane & 31;
    // What the end needs of the tokens, requested before the loop where the registers allow, else behind it: quadruple q of a
    // phase -> its 32-token tile, 32-row block and place in the tile (whole 32-token tiles come first, RH * 4 quadruples each)
    struct Quad { int m, n; };
    const auto quad_of = [&](int at) {
        const int mb = at / (RH * 4), in = at - mb * RH * 4;
        const int per_h = mb * 32 + 32 <= T ? 4 : 2;
        const int h = in / per_h;
        return Quad{m0 + mb * 32 + 8 * (in - h * per_h) + 4 * second, row0 + h * 32};
    };
    int qsum[F::kPhases][F::kSets][4];
    float ascale[F::kPhases][F::kSets][4];
    const auto load_scales = [&]() {
#pragma unroll
        for (int phase = 0; phase < F::kPhases; ++phase)
#pragma unroll
            for (int j = 0; j < F::kSets; ++j) {
                const int m = quad_of(phase * F::kPhaseQuads + min(wave + j * W, F::kPhaseQuads - 1)).m;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    qsum[phase][j][r] = p.q_sum[min(m + r, M - 1)];
                    ascale[phase][j][r] = p.a_scale[min(m + r, M - 1)];
                }
            }
    };
    constexpr bool kScalesEarly = F::kPhases * F::kSets <= 2;
    if constexpr (kScalesEarly) load_scales();
    // token rows of a 32-token tile that is half empty repeat its first sixteen (their products are never looked at)
    const auto row_of = [&](int mb) { return mb * 32 + (mb * 32 + 32 <= T ? l32 : l32 & 15); };
#pragma unroll
    for (int i = 0; i < D; ++i)
        if (i < steps) request(i);
    for (int i = 0; i < steps; ++i) {
        if (F::Ring::steady(steps, i)) wait_vm<F::Ring::kYounger>();
        else wait_vm<0>();
        const uint8_t* stage = lds + wave * D * F::kStage + (D == 1 ? 0 : i % D) * F::kStage;
        uint4 w[RH];
#pragma unroll
        for (int h = 0; h < RH; ++h)
            w[h] = *reinterpret_cast<const uint4*>(stage + (RH >= 2 ? (h >> 1) * 2048 + second * 1024 + ((h & 1) * 32 + l32) * 16 : lane * 16));
        v4i a[MB][4];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                a[mb][j] = *reinterpret_cast<const v4i*>(stage + RH * 1024 + row_of(mb) * 128 + ((4 * second + j) ^ (l32 & 7) ^ (l32 >> 3 & 1)) * 16);
        // every operand has left the stage before it is requested anew
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (i + D < steps) request(i + D);
        if (odd && wave + i * W == pairs - 1 && second) {   // codes of the tile that is not there: nothing is added
#pragma unroll
            for (int h = 0; h < RH; ++h) w[h] = make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
#pragma unroll
            for (int h = 0; h < RH; ++h) {
                const v4i codes = expand_codes(j == 0 ? w[h].x : j == 1 ? w[h].y : j == 2 ? w[h].z : w[h].w);
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
                    c[mb][h] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[mb][j], codes, c[mb][h], 0, 0, 0);
            }
        }
    }

    // The W partial sums meet in LDS: register quadruple Q of every wave, 16 bytes per lane; quadruple Q is finished by wave
    // Q % W.  Register r of a 32x32 tile holds token 8*(r/4) + 4*(lane/32) + r%4 and weight row lane%32.
    if constexpr (!kScalesEarly) load_scales();
    v4i* ex = reinterpret_cast<v4i*>(lds);
#pragma unroll
    for (int phase = 0; phase < F::kPhases; ++phase) {
        constexpr int PQ = F::kPhaseQuads;
        __syncthreads();   // every wave has read its last stage (nothing is in flight: the last steps waited for all) or phase
        int Q = 0;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int h = 0; h < RH; ++h)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    if (mb * 32 + 8 * r4 >= T) continue;    // no token of this block there
                    if (Q / PQ == phase)
                        ex[(wave * PQ + Q % PQ) * 64 + lane] =
                            v4i{c[mb][h][4 * r4], c[mb][h][4 * r4 + 1], c[mb][h][4 * r4 + 2], c[mb][h][4 * r4 + 3]};
                    ++Q;
                }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < F::kSets; ++j) {
            const int q = wave + j * W;
            if (q >= PQ) break;   // uniform
            v4i v = ex[q * 64 + lane];
#pragma unroll
            for (int w = 1; w < W; ++w) v += ex[(w * PQ + q) * 64 + lane];
            const Quad at = quad_of(phase * PQ + q);
            const int n = at.n + l32;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = at.m + r;
                if (m < M && n < p.N) {
                    const int s = v[r] - qsum[phase][j][r];
                    p.out[(int64_t)m * p.N + n] = (float)s * (p.w_scale * ascale[phase][j][r]);
                    if (p.acc) p.acc[(int64_t)m * p.N + n] = s;
                }
            }
        }
    }
}

template <int T, int RH, int W, int D>
hipError_t launch_narrow_form(const NarrowBatch& b, int M, int gx, hipStream_t s) {
    using F = NarrowForm<T, RH, W, D>;
    static LdsCeiling ceiling;   // per instantiation, i.e. per kernel
    const hipError_t e = ceiling.ensure(reinterpret_cast<const void*>(&gemm_narrow_kernel<T, RH, W, D>), F::kLds);
    if (e != hipSuccess) return e;
    const int64_t wgs = (int64_t)(gx + kXcds - 1) / kXcds * kXcds * ((M + T - 1) / T);
    if (wgs > INT32_MAX) return hipErrorInvalidValue;
    note_kernel("gemm_narrow_kernel<%d, %d, %d, %d>", (int)wgs, T, RH, W, D);
    gemm_narrow_kernel<T, RH, W, D><<<dim3((unsigned)wgs), dim3(64 * W), F::kLds, s>>>(b, M, gx);
    return hipGetLastError();
}

// The forms that are built, X(T, RH, W, D, t0, a, e, s), with the line that their measured times follow (us; relative least
// squares over the 11065 launches described at choose_kernel in bl_gemm.hip, weights cold; eight in ten points within 9 %):
//     t = t0 + a KC + (X - 1) (e + s KC),   X = max(1, (x + ceil x) / 2),   x = workgroups / compute units
// (KC = packed tiles along K; e: what a workgroup costs however short K is -- with it left out, 718 x 64 -> 6976 took 22.9 us here
// where the tile kernel takes 8.5).  The workgroups are counted with the padding of the strips to a multiple of 8: a die
// gets whole strips, and the die with the most is the one that ends last.  16 x 32: X = max(1, 0.35 x + 0.65 ceil x), from 8211 launches with weights
// from memory and from the memory-side cache: with the common X and the line of the others' launches it was taken where a few units have
// two workgroups (12 x 8320 -> 8704 10.2 us, 16 x 64 8.6).
// Measured, tile kernel before -> this one: 3200^2 14.3 -> 4.7 us at 37 tokens, 12.0 -> 5.4 at 128, 12.2 -> 7.6 at 256;
// 4096 -> 11008 16.6 -> 6.4 at 16, 18.9 -> 9.5 at 64, 17.0 -> 13.9 at 128; 11008 -> 4096 32.7 -> 8.1 at 16, 35 -> 10.4 at 64,
// 37.7 -> 15.8 at 256, 38.4 -> 25.1 at 512.  Also tried: four or sixteen waves along K, 48-token blocks, three or four steps in
// flight, and weights straight into registers -- none ahead of the best of these six by more than 5 % anywhere.
#define BL_NARROW_FORMS(X)                           \
    X(16, 1, 8, 2, 2.98f, 0.0223f, 0.500f, 0.0166f)  \
    X(16, 2, 8, 2, 3.30f, 0.0306f, 0.900f, 0.0281f)  \
    X(32, 1, 8, 2, 3.27f, 0.0244f, 0.868f, 0.0238f)  \
    X(32, 2, 8, 1, 3.57f, 0.0296f, 1.128f, 0.0336f)  \
    X(32, 4, 8, 1, 4.69f, 0.0474f, 1.925f, 0.0576f)  \
    X(64, 4, 8, 1, 6.84f, 0.0753f, 5.966f, 0.1181f)

// Strips of one product: 32*RH rows of W each.
int64_t strips_of(const GemmProblem& p, int rh) {
    return rh == 1 ? (p.N + 31) / 32 : rh == 2 ? p.row_blocks : (p.row_blocks + 1) / 2;
}

constexpr int narrow_code(int t, int rh) { return 1000 * rh + t; }

}  // namespace

bool gemm_narrow_form_exists(int code) {
#define X(T, RH, W, D, T0, A, E, S) if (code == narrow_code(T, RH)) return true;
    BL_NARROW_FORMS(X)
#undef X
    return false;
}

bool gemm_narrow_takes(const GemmProblem* ps, int count, int64_t M) {
    for (int i = 0; i < count; ++i)
        if (M * ps[i].KC * kTileK > INT32_MAX) return false;   // 32-bit offsets into the activations
    return true;
}

int gemm_narrow_best(const GemmProblem* ps, int count, int64_t M, int cus, float& us) {
    int best = 0, KC = 0;
    for (int i = 0; i < count; ++i) KC = ps[i].KC > KC ? ps[i].KC : KC;
    const auto consider = [&](int t, int rh, float t0, float a, float each, float slope) {
        int64_t strips = 0;
        for (int i = 0; i < count; ++i) strips += strips_of(ps[i], rh);
        const int64_t wgs = (strips + kXcds - 1) / kXcds * kXcds * ((M + t - 1) / t);
        const float x = (float)wgs / (float)cus, whole = (float)((wgs + cus - 1) / cus);
        const float turns = x + (t == 16 && rh == 1 ? 0.65f : 0.5f) * (whole - x);
        const float est = t0 + a * (float)KC + (turns > 1.0f ? turns - 1.0f : 0.0f) * (each + slope * (float)KC);
        if (!best || est < us) { best = narrow_code(t, rh); us = est; }
    };
#define X(T, RH, W, D, T0, A, E, S) consider(T, RH, T0, A, E, S);
    BL_NARROW_FORMS(X)
#undef X
    return best;
}

hipError_t launch_gemm_narrow(const GemmProblem* ps, int count, int64_t M, int code, hipStream_t s) {
    NarrowBatch b;
    int64_t gx = 0;
    for (int i = 0; i < kMaxGemmBatch; ++i) {
        b.p[i] = ps[i < count ? i : count - 1];
        if (i < count) gx += strips_of(ps[i], code / 1000);
        b.end[i] = i + 1 < count ? (int32_t)gx : INT32_MAX;
    }
    if (gx > INT32_MAX - kXcds) return hipErrorInvalidValue;
#define X(T, RH, W, D, T0, A, E, S) if (code == narrow_code(T, RH)) return launch_narrow_form<T, RH, W, D>(b, (int)M, (int)gx, s);
    BL_NARROW_FORMS(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace bl
