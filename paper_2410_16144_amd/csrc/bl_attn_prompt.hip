// bl_attn_prefill on the matrix cores, head sizes that are a multiple of 8 up to 128: a prompt's tokens against the cache.
//
// One workgroup = 32 consecutive tokens of one head, SETS waves (four or eight) that share out the cache's 32-row chunks (wave s
// takes chunks s, s + SETS, ...) and merge their running maxima, sums and outputs at the end.  A wave brings its own chunks and
// waits for nobody until the merge: two workgroups of four waves fit a compute unit, so that every SIMD has two waves which are
// not in step, one of them in its products while the other is in its softmax.  (The form before this one had 64 tokens per
// workgroup, two waves sharing each chunk, and a barrier per chunk: the waves of a SIMD wanted the matrix core and the vector ALU at
// the same moments, 4800 cycles per two chunks and SIMD for 2560 cycles of products, and one workgroup per unit made the longest
// block the launch's duration.)
//
// Scores are formed TRANSPOSED, S^T = K Q^T, with v_mfma_f32_32x32x16_bf16: a lane then holds 16 of the chunk's 32 weights of
// ONE query (the other 16 are in lane +-32), so maximum and sum are register operations and one lane exchange, and the
// weights are already laid out as the B operand of O^T += V^T P^T -- they never pass through LDS.  The contraction index
// of that product runs over the keys in the order in which the result registers hold them: slots 0..3 of lane half g are
// keys 4g .. 4g+3 of a 16-key block, slots 4..7 keys 8+4g .. 8+4g+3.  V^T comes from V as it lies in the cache by the
// transposing LDS read (ds_read_b64_tr_b16: per 16 lanes a block of 4 keys x 16 elements, column by column).
//
// Keys and values are bf16 in the cache already; the fp32 queries enter as the sum of three bf16 numbers (all 24 bits, since
// a score's error is multiplied by the scores' size) and the weights, which lie in [0, 1], as the sum of two (about 17 bits);
// each part takes one product, everything is accumulated in fp32.  The scores carry log2(e): weights are powers of two.
//
// A chunk (K and V, 32 rows each) goes from the cache straight into LDS, one tile each per wave: the next chunk's K is requested
// when this chunk's scores are formed and travels under softmax and the second product, its V when the values have been
// read.  The waits count: whatever was requested last may be on its way (KS requests).  The LDS image is lane-linear, so bank conflicts
// are avoided by fetching the 16-byte pieces of a row in permuted order: K for reads of one piece of many rows, V for reads of
// 64 bytes of four rows.
//
// Measured, append launch included, kernel before -> this one (us; inputs from memory).  32 heads of 128: 512 tokens from position 0
// 23.6 -> 20.7, behind 512 cached ones 34.5 -> 31.5, 64 tokens behind 1984 41.5 -> 25.8, 37 from 0 10.8 -> 9.3, 256 behind 500 23.2 ->
// 17.1; 12 heads of 64: 512 behind 512 17.9 -> 12.2, 16 behind 1000 16.3 -> 10.9.  Longer prompts stay where they were (2048 tokens from 0 113 ->
// 110, behind 2048 256 -> 256): at 1.1 PFLOP/s of bf16 products they run at what a large matrix product reaches on this card
// (1.22), which is its power limit.
#include <type_traits>

#include "bl_internal.hpp"

namespace bl {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));   // four floats at any float's address

constexpr int kKeys = 32;       // cache rows per chunk
constexpr int kBlockQ = 32;     // queries per workgroup

struct PromptArgs {
    const float*    q_lin;
    const float2*   rope;
    const uint16_t* k_cache;
    const uint16_t* v_cache;
    float*          out;
    int32_t         n_heads, head_dim, pos0, M;
    int32_t         blocks;     // of 32 tokens
    int32_t         paired;     // blocks in the order last, ..., middle, first, ..., middle instead of last ... first
};

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// Two floats rounded to bf16 (nearest even), the first in the low half.
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
}
__device__ __forceinline__ s16x8 as_s16x8(const uint32_t (&v)[4]) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    return __builtin_bit_cast(s16x8, (u32x4{v[0], v[1], v[2], v[3]}));
}

__device__ __forceinline__ f32x16 mfma(const s16x8& a, const s16x8& b, const f32x16& c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Place of a row's 16-byte piece c (of 2 * KS) in the LDS image; both are their own inverse.  Keys: rows of a power of two of
// bytes are permuted, rows of an odd number of 32 bytes (KS = 3, 5, 7) spread over the banks by themselves.  KS = 6 (head
// size 96) is neither: rows of 192 bytes, the fourth next in the same bank; 47 % of the kernel's LDS cycles there are
// conflicts (8 % with KS = 8).
template <int KS>
__device__ __forceinline__ int k_place(int row, int c) {
    return (KS & (KS - 1)) == 0 ? c ^ (row & (2 * KS - 1)) : c;
}
template <int KS>
__device__ __forceinline__ int v_place(int row, int c) {
    return KS == 8 ? c ^ ((row & 3) << 2) : KS == 4 ? c ^ (((row >> 1) & 1) << 2) : c;
}

// KS: head size rounded up to 16, in sixteens.  SETS: waves of a workgroup.
template <int KS, int SETS>
struct PromptLds {
    static constexpr int kRow = 32 * KS;               // bytes of a cache row's head in LDS
    static constexpr int kTile = kKeys * kRow;         // K or V of one chunk
    static constexpr int DT = (KS + 1) / 2;            // 32-element pieces of the output
    static constexpr int kRing = SETS * 2 * kTile;                 // [set][K, V]
    static constexpr int kMerge = SETS * kBlockQ * DT * 32 * 4;    // [set][query][element]
    static constexpr int kBytes = kRing > kMerge ? kRing : kMerge;
    static constexpr int kRows = kBlockQ / SETS;                   // queries that pass through a set's V tile
    static_assert(kBytes <= kMaxDecodeLds, "fits the LDS ceiling");
    static_assert(kRows * 64 * KS <= kTile, "a set's V tile holds its share of the queries");
};

template <int KS, int SETS>
__global__ __launch_bounds__(64 * SETS, SETS == 4 ? 2 : 1) void attn_prompt_kernel(const PromptArgs p) {
    using L = PromptLds<KS, SETS>;
    constexpr int DT = L::DT, kRow = L::kRow, kThreads = 64 * SETS;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int set = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int turn = (int)blockIdx.x / p.n_heads, head = (int)blockIdx.x - turn * p.n_heads;
    // later blocks walk more chunks: launched first
    const int first_half = (p.blocks + 1) >> 1;
    const int block = p.paired && turn >= first_half ? turn - first_half : p.blocks - 1 - turn;
    const int d = p.head_dim, half = d >> 1, hidden = p.n_heads * d;
    const int l32 = lane & 31, g = lane >> 5;
    const int last_pos = p.pos0 + p.M - 1;                                    // the last cached row
    const int m_last = min(block * kBlockQ + kBlockQ - 1, p.M - 1);
    const int chunks = (p.pos0 + m_last) / kKeys + 1;                         // that any query of the block sees
    const int mine = chunks > set ? (chunks - set + SETS - 1) / SETS : 0;     // chunks of this wave: set, set + SETS, ...

    // requests: KS pieces of 1 KiB for K, as many for V; lane l of piece s fills the 16 bytes at 64 s + l of the image
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)lds;
    const int64_t row_bytes = (int64_t)hidden * 2;
    const int pieces = d >> 3;
    // Offsets of a lane's pieces in a chunk.  Where a piece is a whole number of rows the pattern repeats every kPeriod pieces
    // (a few registers instead of one per piece), the rest of the way goes into the scalar base.
    constexpr bool kWholeRows = (KS & (KS - 1)) == 0;
    constexpr int kPeriodK = !kWholeRows ? KS : KS == 8 ? 4 : 1, kPeriodV = !kWholeRows ? KS : 1;
    uint32_t k_off[kPeriodK], v_off[kPeriodV];
    const auto piece = [&](bool value, int s, int limit) {
        const int at = s * 64 + lane, row = at / (2 * KS), place = at % (2 * KS);
        const int c = min(value ? v_place<KS>(row, place) : k_place<KS>(row, place), pieces - 1);   // padding: any piece of the row
        return (uint32_t)min(row, limit) * (uint32_t)row_bytes + (uint32_t)c * 16;
    };
#pragma unroll
    for (int s = 0; s < kPeriodK; ++s) k_off[s] = piece(false, s, kKeys);
#pragma unroll
    for (int s = 0; s < kPeriodV; ++s) v_off[s] = piece(true, s, kKeys);
    const auto request = [&](int i, auto which) {
        constexpr bool value = decltype(which)::value;
        constexpr int kPeriod = value ? kPeriodV : kPeriodK;
        const int j0 = (set + SETS * i) * kKeys;
        const uint8_t* base = uniform_ptr(reinterpret_cast<const uint8_t*>(value ? p.v_cache : p.k_cache) + (int64_t)head * d * 2 +
                                          (int64_t)j0 * row_bytes);
        uint32_t dst = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)((set * 2 + (value ? 1 : 0)) * L::kTile));
        const auto put = [&](uint32_t off, const uint8_t* src) {
            // M0 carries the LDS address of this instruction and of nothing else in this kernel
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(off), "s"(src) : "memory", "m0");
#pragma clang diagnostic pop
            dst += 1024;
        };
        if (j0 + kKeys - 1 <= last_pos) {   // uniform
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                put(value ? v_off[s % kPeriodV] : k_off[s % kPeriodK], base);
                if (s % kPeriod == kPeriod - 1) base += (uint32_t)(kPeriod * 32 / KS) * (uint32_t)row_bytes;
            }
        } else {                            // rows beyond the prompt repeat its last one (nobody looks at them)
#pragma unroll
            for (int s = 0; s < KS; ++s) put(piece(value, s, last_pos - j0), base);
        }
    };
    if (mine) request(0, std::false_type{});

    // The block's queries, rotated and scaled by log2(e) / sqrt(head_dim), go through LDS (in the V tiles, which are requested
    // when the queries have been read): read from memory row by row, four elements and their partners in the other
    // half of the head per thread.  (Each lane fetching its own query's elements from 64 different rows cost 13 us.)
    // Row r lies in set r / kRows's tile; its 16-byte pieces are permuted for reads of one piece of many rows.
    constexpr int kSpread = KS % 2 == 0 ? 7 : 3;
    const auto q_at = [&](int row, int c) {
        return reinterpret_cast<f32x4*>(lds + (row / L::kRows * 2 + 1) * L::kTile + (row % L::kRows) * (64 * KS) + (c ^ (row & kSpread)) * 16);
    };
    {
        const float scale = 1.4426950408889634f / sqrtf((float)d);
        const int quarters = half >> 2;              // head_dim / 2 is a multiple of 4
        for (int at = tid; at < kBlockQ * quarters; at += kThreads) {
            const int row = at / quarters, c = at - row * quarters;
            const int m = min(block * kBlockQ + row, p.M - 1);   // rows beyond the prompt repeat its last token
            const float* q = p.q_lin + (int64_t)m * hidden + head * d + 4 * c;
            const float* cs = reinterpret_cast<const float*>(p.rope + (int64_t)(p.pos0 + m) * half + 4 * c);
            const f32x4 a = *reinterpret_cast<const f32x4_u*>(q), b = *reinterpret_cast<const f32x4_u*>(q + half);
            const f32x4 c0 = *reinterpret_cast<const f32x4_u*>(cs), c1 = *reinterpret_cast<const f32x4_u*>(cs + 4);
            f32x4 lo, hi;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float cx = j < 2 ? c0[2 * j] : c1[2 * j - 4], cy = j < 2 ? c0[2 * j + 1] : c1[2 * j - 3];
                lo[j] = (a[j] * cx - b[j] * cy) * scale;
                hi[j] = (a[j] * cy + b[j] * cx) * scale;
            }
            *q_at(row, c) = lo;
            *q_at(row, c + quarters) = hi;
        }
    }
    __syncthreads();
    // the queries as B operands: column l32, elements 16 ks + 8 g .. + 7
    s16x8 q_hi[KS], q_mid[KS], q_lo[KS];
    const int q_first = p.pos0 + block * kBlockQ;   // position of the block's first query
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        uint32_t parts[3][4];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int c = 4 * ks + 2 * g + h;
            f32x4 x = *q_at(l32, c);
            if (4 * c >= d) x = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                float a = x[2 * j], b = x[2 * j + 1];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const uint32_t v = bf16_pair(a, b);
                    parts[k][2 * h + j] = v;
                    a -= __uint_as_float(v << 16);
                    b -= __uint_as_float(v & 0xffff0000u);
                }
            }
        }
        q_hi[ks] = as_s16x8(parts[0]);
        q_mid[ks] = as_s16x8(parts[1]);
        q_lo[ks] = as_s16x8(parts[2]);
    }
    __syncthreads();   // every wave has its queries: the V tiles may be filled
    if (mine) request(0, std::true_type{});

    f32x16 o[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[t][r] = 0.0f;
    float run_m = -INFINITY, run_l = 0.0f;      // of this lane's query; run_l: over this lane half's keys only
    const int q_pos = q_first + l32;
    const bool odd_pieces = (d & 15) != 0;      // the last 16 elements are half padding
    // lane constants of the transposing reads: key (lane % 16) / 4 of a group of four, elements 32 t + 16 (lane / 16 % 2) + 4 (lane % 4)
    const int v_key = (lane & 15) >> 2;
    const int v_sub = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
    int v_at[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t) {
        int c = 4 * t + v_sub;
        if (c >= 2 * KS) c = 0;                 // an odd KS: the last piece is 16 elements, the rest of it is never stored
        v_at[t] = (4 * g + v_key) * kRow + v_place<KS>(v_key, c) * 16 + (lane & 1) * 8;
    }

    const uint8_t* sk = lds + set * 2 * L::kTile;
    const uint8_t* sv = sk + L::kTile;
    for (int i = 0; i < mine; ++i) {
        const int j0 = (set + SETS * i) * kKeys;
        wait_vm<KS>();   // K has landed; the V requested behind it may be on its way

        // S^T: 32 keys x 32 queries; register r = key 8 (r / 4) + 4 g + r % 4
        f32x16 sc;
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[r] = 0.0f;
        // (four key operands are on their way from LDS at any time: 3 x 3 products cover its latency)
        constexpr int kAhead = KS < 4 ? KS : 4;
        s16x8 k[kAhead];
        const auto read_k = [&](int ks) { return *reinterpret_cast<const s16x8*>(sk + l32 * kRow + k_place<KS>(l32, 2 * ks + g) * 16); };
#pragma unroll
        for (int ks = 0; ks < kAhead; ++ks) k[ks] = read_k(ks);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            s16x8& kk = k[ks % kAhead];
            if (ks == KS - 1 && odd_pieces && g) kk = s16x8{0, 0, 0, 0, 0, 0, 0, 0};
            sc = mfma(kk, q_lo[ks], sc);
            sc = mfma(kk, q_mid[ks], sc);
            sc = mfma(kk, q_hi[ks], sc);
            if (ks + kAhead < KS) kk = read_k(ks + kAhead);
            __builtin_amdgcn_sched_barrier(0);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // every key has left the tile before it is requested anew
        if (i + 1 < mine) {
            request(i + 1, std::false_type{});
            wait_vm<KS>();   // V has landed; the K just requested may be on its way
        } else {
            wait_vm<0>();
        }
        // the first sixteen keys' value operands travel under the softmax
        typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
        const auto read_v = [&](int kb, int t) {
            const uint8_t* at = sv + v_at[t] + kb * 16 * kRow;
            const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)at);
            const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(at + 8 * kRow));
            return s16x8{v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
        };
        s16x8 v[DT];
#pragma unroll
        for (int t = 0; t < DT; ++t) v[t] = read_v(0, t);
        __builtin_amdgcn_sched_barrier(0);
        // a query sees the keys up to its own position (only chunks around the wave's own positions need the test)
        if (j0 + kKeys - 1 > q_first) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (j0 + 8 * (r >> 2) + 4 * g + (r & 3) > q_pos) sc[r] = -INFINITY;
        }
        float mx = sc[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sc[r]);
        {
            const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);   // the two halves' figures
            mx = fmaxf(__uint_as_float(both[0]), __uint_as_float(both[1]));
        }
        const float m_new = fmaxf(run_m, mx);
        if (__any(m_new > run_m)) {   // else every factor is 1
            // a query that has seen no key yet keeps -inf: nothing to rescale, and no weight below
            const float f = run_m == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(run_m - m_new);
#pragma unroll
            for (int t = 0; t < DT; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[t][r] *= f;
            run_l *= f;
            run_m = m_new;
        }
        const float base = m_new == -INFINITY ? 0.0f : m_new;
        s16x8 w_hi[2], w_lo[2];
        float sum = 0.0f;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            uint32_t hi[4], lo[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float a = __builtin_amdgcn_exp2f(sc[8 * kb + 2 * j] - base), b = __builtin_amdgcn_exp2f(sc[8 * kb + 2 * j + 1] - base);
                sum += a;
                sum += b;
                hi[j] = bf16_pair(a, b);
                lo[j] = bf16_pair(a - __uint_as_float(hi[j] << 16), b - __uint_as_float(hi[j] & 0xffff0000u));
            }
            w_hi[kb] = as_s16x8(hi);
            w_lo[kb] = as_s16x8(lo);
        }
        run_l += sum;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
            for (int t = 0; t < DT; ++t) {
                o[t] = mfma(v[t], w_lo[kb], o[t]);
                o[t] = mfma(v[t], w_hi[kb], o[t]);
                if (kb == 0) v[t] = read_v(1, t);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (i + 1 < mine) request(i + 1, std::true_type{});
    }

    // the sets' figures meet: maxima and sums first, then the outputs, each scaled by its own factor
    run_l += __shfl_xor(run_l, 32);
    __syncthreads();
    float2* ml = reinterpret_cast<float2*>(lds);   // [set][query]
    const int q = l32;
    if (g == 0) ml[set * kBlockQ + q] = make_float2(run_m, run_l);
    __syncthreads();
    float m_all = -INFINITY, l_all = 0.0f;
    float2 part[SETS];
#pragma unroll
    for (int s = 0; s < SETS; ++s) {
        part[s] = ml[s * kBlockQ + q];
        m_all = fmaxf(m_all, part[s].x);
    }
#pragma unroll
    for (int s = 0; s < SETS; ++s) l_all += part[s].y * __builtin_amdgcn_exp2f(part[s].x - m_all);   // (a set without keys: 0 * 0)
    const float f = __builtin_amdgcn_exp2f(run_m - m_all) * (1.0f / l_all);
    __syncthreads();
    constexpr int kQuads = DT * 8;                 // groups of four elements per query; group c at place c ^ (q % 8)
    float* merge = reinterpret_cast<float*>(lds);
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const int c = (t * 8 + 2 * r4 + g) ^ (q & 7);
            *reinterpret_cast<f32x4*>(merge + ((set * kBlockQ + q) * kQuads + c) * 4) =
                f32x4{o[t][4 * r4] * f, o[t][4 * r4 + 1] * f, o[t][4 * r4 + 2] * f, o[t][4 * r4 + 3] * f};
        }
    __syncthreads();
    for (int at = tid; at < kBlockQ * kQuads; at += kThreads) {
        const int row = at / kQuads, c = at % kQuads, m = block * kBlockQ + row;
        if (m >= p.M || c * 4 >= d) continue;
        f32x4 v = *reinterpret_cast<const f32x4*>(merge + (row * kQuads + (c ^ (row & 7))) * 4);
#pragma unroll
        for (int s = 1; s < SETS; ++s)
            v += *reinterpret_cast<const f32x4*>(merge + ((s * kBlockQ + row) * kQuads + (c ^ (row & 7))) * 4);
        *reinterpret_cast<f32x4_u*>(p.out + (int64_t)m * hidden + head * d + c * 4) = v;
    }
}

template <int KS, int SETS>
hipError_t launch_form(const PromptArgs& p, hipStream_t s) {
    using L = PromptLds<KS, SETS>;
    static LdsCeiling ceiling;   // per instantiation, i.e. per kernel
    const hipError_t e = ceiling.ensure(reinterpret_cast<const void*>(&attn_prompt_kernel<KS, SETS>), L::kBytes);
    if (e != hipSuccess) return e;
    const int64_t wgs = (int64_t)p.n_heads * p.blocks;
    if (wgs > INT32_MAX) return hipErrorInvalidValue;
    attn_prompt_kernel<KS, SETS><<<dim3((unsigned)wgs), dim3(64 * SETS), L::kBytes, s>>>(p);
    return hipGetLastError();
}

template <int KS>
hipError_t launch_prompt(PromptArgs p, hipStream_t s) {
    const int found = compute_unit_count();
    const int64_t cus = found > 0 ? found : 256, wgs = (int64_t)p.n_heads * p.blocks;
    // more than one workgroup per unit and all of them resident: a unit's second one is as short as its first one is long
    // (512 tokens from position 0 on 32 heads: 21.6 us in falling order, 20.7 in pairs)
    p.paired = wgs > cus && wgs <= 2 * cus;
    // eight waves where every workgroup has a unit to itself and a wave of four would have more than three chunks to go through
    // (12 heads of 64: 16 tokens behind 240 7.6 us with four, 7.9 with eight; behind 500 10.1 and 9.0, behind 1000 12.9 and 10.9)
    if (wgs <= cus && p.pos0 + p.M > 384) return launch_form<KS, 8>(p, s);
    return launch_form<KS, 4>(p, s);
}

}  // namespace

// Head sizes in multiples of 8 (16-byte pieces of a cache row) up to 128, and rows short enough for 32-bit offsets in a chunk.
bool attn_prompt_takes(int n_heads, int head_dim) {
    return head_dim % 8 == 0 && head_dim <= BL_ATTN_BLOCK_MAX_HEAD_DIM && (int64_t)n_heads * head_dim <= (1 << 24);
}

hipError_t launch_attn_prompt(const bl_attn_prefill_args& a, hipStream_t s) {
    PromptArgs p;
    p.q_lin = a.q_lin_dev;
    p.rope = reinterpret_cast<const float2*>(a.rope_table_dev);
    p.k_cache = a.k_cache_dev;
    p.v_cache = a.v_cache_dev;
    p.out = a.out_dev;
    p.n_heads = a.n_heads; p.head_dim = a.head_dim; p.pos0 = a.pos0; p.M = a.M;
    p.blocks = (a.M + kBlockQ - 1) / kBlockQ;
    switch ((a.head_dim + 15) / 16) {
        case 1: return launch_prompt<1>(p, s);
        case 2: return launch_prompt<2>(p, s);
        case 3: return launch_prompt<3>(p, s);
        case 4: return launch_prompt<4>(p, s);
        case 5: return launch_prompt<5>(p, s);
        case 6: return launch_prompt<6>(p, s);
        case 7: return launch_prompt<7>(p, s);
        case 8: return launch_prompt<8>(p, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace bl
