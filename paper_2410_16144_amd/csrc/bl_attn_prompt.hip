// bl_attn_prefill on the matrix cores, head sizes that are a multiple of 8 up to 128: a prompt's tokens against the cache.
//
// One workgroup = 64 consecutive tokens of one head, eight waves: two groups of 32 queries x four SETS that share out the
// cache's 32-row chunks (set s takes chunks s, s + 4, ...) and merge their running maxima, sums and outputs at the end.  So
// even a prompt of 512 tokens on 32 heads, one workgroup per compute unit, keeps two waves on every SIMD, and the longest
// block walks a quarter of its chunks in a row.  (The form before this one gave a wave 16 queries and all chunks: one wave
// per SIMD, 7400 cycles per 64-row chunk of which the products were 1300.)
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
// A set's chunk (K and V, 32 rows each) goes from the cache straight into LDS, one chunk ahead, K by the set's first wave and
// V by its second.  One barrier per chunk.  The LDS image is lane-linear, so bank conflicts are avoided by fetching the
// 16-byte pieces of a row in permuted order: K for reads of one piece of many rows, V for reads of 64 bytes of four rows.
//
// Measured, append launch included, 32 heads of 128, kernel before -> this one (us): 512 tokens from position 0 43.0 -> 24.1,
// behind 512 cached ones 62.1 -> 33.2 (inputs from memory; 60.2 -> 29.7 where a pass finds them in the caches), behind 1536
// 101 -> 51; 2048 tokens from 0 181 -> 115, behind 2048 363 -> 260; 64 tokens behind 1984 97 -> 41.  Of that the append is 6 to
// 7.  By the slope over longer prompts a step (four chunks, 128 rows) takes 1.9 us, about 4200 cycles, for 2560 cycles of
// products (two waves per SIMD, 40 products of 32 cycles each); the rest is the softmax's vector work that does not hide.  Counters
// over the whole launch, 512 tokens behind 512: the matrix cores are busy in 34 % of the cycles of compute units with waves.
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
constexpr int kSets = 4;        // wave pairs that share out the chunks
constexpr int kBlockQ = 64;     // queries per workgroup
constexpr int kThreads = 512;

struct PromptArgs {
    const float*    q_lin;
    const float2*   rope;
    const uint16_t* k_cache;
    const uint16_t* v_cache;
    float*          out;
    int32_t         n_heads, head_dim, pos0, M;
};

__device__ __forceinline__ short bf16_bits(float v) { return __builtin_bit_cast(short, (__bf16)v); }   // nearest even
__device__ __forceinline__ float bf16_value(short b) { return __uint_as_float((uint32_t)(uint16_t)b << 16); }

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

// KS: head size rounded up to 16, in sixteens.
template <int KS>
struct PromptLds {
    static constexpr int kRow = 32 * KS;               // bytes of a cache row's head in LDS
    static constexpr int kTile = kKeys * kRow;         // K or V of one chunk
    static constexpr int DT = (KS + 1) / 2;            // 32-element pieces of the output
    static constexpr int kRing = kSets * 2 * 2 * kTile;            // [set][buffer][K, V]
    static constexpr int kMerge = kSets * kBlockQ * DT * 32 * 4;   // [set][query][element]
    static constexpr int kBytes = kRing > kMerge ? kRing : kMerge;
    static_assert(kBytes <= kMaxDecodeLds, "fits the LDS ceiling");
    static_assert(kSets * 16 == kBlockQ && 16 * 64 * KS <= 2 * kTile, "a set's second buffers hold sixteen queries");
};

template <int KS>
__global__ __launch_bounds__(kThreads) void attn_prompt_kernel(const PromptArgs p) {
    using L = PromptLds<KS>;
    constexpr int DT = L::DT, kRow = L::kRow;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qg = wave & 1, set = wave >> 1;
    const int head = blockIdx.x, block = (int)(gridDim.y - 1 - blockIdx.y);   // later blocks walk more chunks: launched first
    const int d = p.head_dim, half = d >> 1, hidden = p.n_heads * d;
    const int l32 = lane & 31, g = lane >> 5;
    const int last_pos = p.pos0 + p.M - 1;                                    // the last cached row
    const int m_last = min(block * kBlockQ + kBlockQ - 1, p.M - 1);
    const int chunks = (p.pos0 + m_last) / kKeys + 1;                         // that any query of the block sees
    const int steps = (chunks + kSets - 1) / kSets;

    // requests: the set's first wave brings K, its second V, KS pieces of 1 KiB each; lane l of piece s fills the 16 bytes
    // at 64 s + l of the image
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)lds;
    const uint8_t* src0 = reinterpret_cast<const uint8_t*>(qg ? p.v_cache : p.k_cache) + (int64_t)head * d * 2;
    const int64_t row_bytes = (int64_t)hidden * 2;
    const int pieces = d >> 3;
    const auto request = [&](int i) {
        const int chunk = set + kSets * i;
        if (chunk >= chunks) return;   // uniform
        const int j0 = chunk * kKeys;
        const uint8_t* base = src0 + (int64_t)j0 * row_bytes;
        uint32_t dst = lds0 + (uint32_t)(((set * 2 + (i & 1)) * 2 + qg) * L::kTile);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int at = s * 64 + lane, row = at / (2 * KS), place = at % (2 * KS);
            const int c = min(qg ? v_place<KS>(row, place) : k_place<KS>(row, place), pieces - 1);   // padding: any piece of the row
            // rows beyond the prompt repeat its last one (nobody looks at them)
            const uint32_t off = (uint32_t)min(row, last_pos - j0) * (uint32_t)row_bytes + (uint32_t)c * 16;
            // M0 carries the LDS address of this instruction and of nothing else in this kernel
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(off), "s"(base) : "memory", "m0");
#pragma clang diagnostic pop
            dst += 1024;
        }
    };
    request(0);

    // The block's queries, rotated and scaled by log2(e) / sqrt(head_dim), go through LDS (in the second buffers, which the
    // loop requests behind its first barrier): read from memory row by row, four elements and their partners in the other
    // half of the head per thread.  (Each lane fetching its own query's elements from 64 different rows cost 13 us.)
    // Row r lies in set r / 16's buffers; its 16-byte pieces are permuted for reads of one piece of many rows.
    constexpr int kSpread = KS % 2 == 0 ? 7 : 3;
    const auto q_at = [&](int row, int c) {
        return reinterpret_cast<f32x4*>(lds + ((row >> 4) * 4 + 2) * L::kTile + (row & 15) * (64 * KS) + (c ^ (row & kSpread)) * 16);
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
    // the wave's queries as B operands: column l32, elements 16 ks + 8 g .. + 7
    s16x8 q_hi[KS], q_mid[KS], q_lo[KS];
    const int q_wave0 = p.pos0 + block * kBlockQ + qg * 32;   // position of the wave's first query
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int c = 4 * ks + 2 * g + h;
            const f32x4 x = *q_at(qg * 32 + l32, c);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float v = 4 * c < d ? x[j] : 0.0f;
                const short hi = bf16_bits(v);
                const float r1 = v - bf16_value(hi);
                const short mid = bf16_bits(r1);
                q_hi[ks][4 * h + j] = hi; q_mid[ks][4 * h + j] = mid; q_lo[ks][4 * h + j] = bf16_bits(r1 - bf16_value(mid));
            }
        }
    }

    f32x16 o[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[t][r] = 0.0f;
    float run_m = -INFINITY, run_l = 0.0f;      // of this lane's query; run_l: over this lane half's keys only
    const int q_pos = q_wave0 + l32;
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

    for (int i = 0; i < steps; ++i) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's part of the chunk has landed
        __syncthreads();                                    // ... everybody's; and the other buffer has been read
        if (i + 1 < steps) request(i + 1);
        const int chunk = set + kSets * i, j0 = chunk * kKeys;
        if (chunk >= chunks || j0 > q_wave0 + 31) continue; // uniform: nothing that this wave's queries see
        const uint8_t* sk = lds + ((set * 2 + (i & 1)) * 2) * L::kTile;
        const uint8_t* sv = sk + L::kTile;

        // S^T: 32 keys x 32 queries; register r = key 8 (r / 4) + 4 g + r % 4
        f32x16 sc;
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[r] = 0.0f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            s16x8 k = *reinterpret_cast<const s16x8*>(sk + l32 * kRow + k_place<KS>(l32, 2 * ks + g) * 16);
            if (ks == KS - 1 && odd_pieces && g) k = s16x8{0, 0, 0, 0, 0, 0, 0, 0};
            sc = mfma(k, q_lo[ks], sc);
            sc = mfma(k, q_mid[ks], sc);
            sc = mfma(k, q_hi[ks], sc);
        }
        // a query sees the keys up to its own position (only chunks around the wave's own positions need the test)
        if (j0 + kKeys - 1 > q_wave0) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (j0 + 8 * (r >> 2) + 4 * g + (r & 3) > q_pos) sc[r] = -INFINITY;
        }
        float mx = sc[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sc[r]);
        mx = fmaxf(mx, __shfl_xor(mx, 32));
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
        for (int r = 0; r < 16; ++r) {
            const float w = __builtin_amdgcn_exp2f(sc[r] - base);
            sum += w;
            const short hi = bf16_bits(w);
            w_hi[r >> 3][r & 7] = hi;
            w_lo[r >> 3][r & 7] = bf16_bits(w - bf16_value(hi));
        }
        run_l += sum;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
            for (int t = 0; t < DT; ++t) {
                typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
                const uint8_t* at = sv + v_at[t] + kb * 16 * kRow;
                const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)at);
                const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(at + 8 * kRow));
                const s16x8 v = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
                o[t] = mfma(v, w_lo[kb], o[t]);
                o[t] = mfma(v, w_hi[kb], o[t]);
            }
        }
    }

    // the sets' figures meet: maxima and sums first, then the outputs, each scaled by its own factor
    run_l += __shfl_xor(run_l, 32);
    __syncthreads();
    float2* ml = reinterpret_cast<float2*>(lds);   // [set][query]
    const int q = qg * 32 + l32;
    if (g == 0) ml[set * kBlockQ + q] = make_float2(run_m, run_l);
    __syncthreads();
    float m_all = -INFINITY, l_all = 0.0f;
    float2 part[kSets];
#pragma unroll
    for (int s = 0; s < kSets; ++s) {
        part[s] = ml[s * kBlockQ + q];
        m_all = fmaxf(m_all, part[s].x);
    }
#pragma unroll
    for (int s = 0; s < kSets; ++s) l_all += part[s].y * __builtin_amdgcn_exp2f(part[s].x - m_all);   // (a set without keys: 0 * 0)
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
        for (int s = 1; s < kSets; ++s)
            v += *reinterpret_cast<const f32x4*>(merge + ((s * kBlockQ + row) * kQuads + (c ^ (row & 7))) * 4);
        *reinterpret_cast<f32x4_u*>(p.out + (int64_t)m * hidden + head * d + c * 4) = v;
    }
}

template <int KS>
hipError_t launch_prompt(const PromptArgs& p, hipStream_t s) {
    static LdsCeiling ceiling;   // per instantiation, i.e. per kernel
    const hipError_t e = ceiling.ensure(reinterpret_cast<const void*>(&attn_prompt_kernel<KS>), PromptLds<KS>::kBytes);
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)p.n_heads, (unsigned)((p.M + kBlockQ - 1) / kBlockQ));
    attn_prompt_kernel<KS><<<grid, dim3(kThreads), PromptLds<KS>::kBytes, s>>>(p);
    return hipGetLastError();
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
