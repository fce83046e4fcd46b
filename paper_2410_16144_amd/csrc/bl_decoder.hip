// The decoder block around the BitLinear products, one token at a time: what stands between the seven
// ternary projections of a layer so that a token passes through it without leaving the GPU.
//
// arXiv 2410.16144 reports tokens per second of whole models (Section 3) whose shapes Appendix A lists;
// it does not describe these operations.  They are the LLaMA-like block of BitNet b1.58: RMSNorm, rotary
// position embedding, multi-head attention over a key/value cache, SiLU-gated feed-forward, residuals.
//
// Kernels here:
//   norm_quant_kernel   residual add / SiLU gate  ->  RMSNorm  ->  per-token absmax int8 quantizer, one
//                       workgroup per token row, the row held in registers from its only read to the int8
//                       store (the quantizer is the one of bl_quant_act, bit for bit);
//   rope_table_kernel   cos / sin of every (position, frequency), fp64 arithmetic, rounded to fp32;
//   attn_chunk_kernel   one (head, every G-th chunk of 64 cache rows) per workgroup: rotate query and key, append key
//                       and value to the bf16 cache, running maximum, sum and weighted values over its chunks;
//                       the head's workgroup that finishes last merges the others' figures;
//   kv_append_kernel    a prompt's keys and values into the cache;
//   attn_block_kernel   a prompt's attention on the matrix cores, head sizes that are 4 modulo 8 (the others:
//                       bl_attn_prompt.hip);
//   pos_advance_kernel  the token position lives in device memory, so a captured graph replays unchanged.
// All of it but attn_block_kernel is bandwidth- and latency-bound glue next to the weight streams.
#include "bl_attn_groups.hpp"
#include "bl_quant_device.hpp"
#include "bitlinear_decoder.h"

namespace bl {

namespace {

// ---------------------------------------------------------------------------------------------------------------
// RMSNorm + quantizer

constexpr int kNormThreads = 1024;

struct NormArgs {
    const float* a;
    const float* b;
    float*       h;
    const float* gamma;
    int8_t*      q;
    float*       a_scale;
    int32_t*     q_sum;
    float*       y;
    float2*      scratch;   // wide form: per row kWideMaxSlices x (sum of squares, absmax of x * gamma)
    int32_t      pieces;    // pre-multiplied form: pairs in scratch (read only)
    int32_t      K, Kp;
    float        eps;
    float*       h_out;     // residual form: receives the sum (h itself, another buffer or nobody)
    int32_t*     pos;       // residual form: a token position that the launch moves on, or null
    int32_t      pos_set;   // ... to this, or by one if it is negative
};

// 4 consecutive elements from element k; VEC: one 128-bit access (row base 16-byte aligned, K % 4 == 0);
// elements from K on read as zero.
template <bool VEC>
__device__ __forceinline__ void load4(const float* row, int k, int K, float (&v)[4]) {
    if constexpr (VEC) {
        float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
        if (k < K) t = *reinterpret_cast<const float4*>(row + k);
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = k + j < K ? row[k + j] : 0.0f;
    }
}

template <bool VEC>
__device__ __forceinline__ void store4(float* row, int k, int K, const float (&v)[4]) {
    if constexpr (VEC) {
        if (k < K) *reinterpret_cast<float4*>(row + k) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (k + j < K) row[k + j] = v[j];
    }
}

// Thread t holds elements 4 (t + THREADS i) .. + 3, i = 0 .. NV-1.
// The sum of squares is added up in ONE order whatever THREADS is, that of 1024 threads: a thread of a smaller workgroup
// stands for kParts of those, its vectors i, i + kParts, ... being one of them, and keeps their sums apart until the waves'
// figures meet.  So a row's result is the same bits in every batch, however its launch is shaped.
template <int MODE, int NV, bool VEC, int THREADS>
__global__ __launch_bounds__(THREADS) void norm_quant_kernel(const NormArgs p) {
    constexpr int kNormWaves = THREADS / kWave;
    constexpr int kParts = kNormThreads / THREADS;
    constexpr int kSums = NV < kParts ? NV : kParts;   // (the rest of them hold no elements: zeros)
    __shared__ float s_ss[kSums * kNormWaves];
    __shared__ float s_max[kNormWaves];
    __shared__ int s_sum[kNormWaves];
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    const int K = p.K;
    const int64_t row = (int64_t)blockIdx.x * K;
    float x[NV][4];
    // short rows: the norm weights are requested with the row, before the first barrier (one memory round trip
    // instead of two); long rows have no registers to spare for that
    constexpr bool kGammaEarly = NV <= 4;
    float gam[kGammaEarly ? NV : 1][4];
    float ss[kSums];
#pragma unroll
    for (int v = 0; v < kSums; ++v) ss[v] = 0.0f;
    // the gated form's inputs, all requested together (its arithmetic has branches that loads do not cross)
    constexpr bool kGatedEarly = MODE == BL_NORM_GATED && NV <= 4;
    float gate[kGatedEarly ? NV : 1][4], up[kGatedEarly ? NV : 1][4];
    if constexpr (kGatedEarly) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            load4<VEC>(p.a + row, (tid + i * THREADS) * 4, K, gate[i]);
            load4<VEC>(p.b + row, (tid + i * THREADS) * 4, K, up[i]);
        }
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int k = (tid + i * THREADS) * 4;
        if constexpr (kGammaEarly) load4<VEC>(p.gamma, k, K, gam[i]);
        if constexpr (MODE == BL_NORM_PLAIN) {
            load4<VEC>(p.a + row, k, K, x[i]);
        } else if constexpr (MODE == BL_NORM_RESIDUAL) {
            load4<VEC>(p.h + row, k, K, x[i]);
            if (p.a) {
                float d[4];
                load4<VEC>(p.a + row, k, K, d);
#pragma unroll
                for (int j = 0; j < 4; ++j) x[i][j] += d[j];
                if (p.h_out) store4<VEC>(p.h_out + row, k, K, x[i]);
            }
        } else {
            float g[4], u[4];
            if constexpr (kGatedEarly) {
#pragma unroll
                for (int j = 0; j < 4; ++j) { g[j] = gate[i][j]; u[j] = up[i][j]; }
            } else {
                load4<VEC>(p.a + row, k, K, g);
                load4<VEC>(p.b + row, k, K, u);
            }
            if constexpr (NV <= 8) {
                silu4(g, x[i]);
            } else {   // no registers to spare for two ways of computing it
#pragma unroll
                for (int j = 0; j < 4; ++j) x[i][j] = silu(g[j]);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) x[i][j] *= u[j];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) ss[i % kParts] += x[i][j] * x[i][j];
    }
#pragma unroll
    for (int v = 0; v < kSums; ++v) {
        ss[v] = wave_sum_f(ss[v]);
        if (lane == 0) s_ss[v * kNormWaves + wave] = ss[v];
    }
    if constexpr (MODE == BL_NORM_RESIDUAL)
        if (p.pos && blockIdx.x == 0 && tid == 0) {   // nobody reads it in this launch; the sum is performed without waiting for it
            if (p.pos_set < 0) __hip_atomic_fetch_add(p.pos, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else *p.pos = p.pos_set;
        }
    __syncthreads();
    float total = 0.0f;
#pragma unroll
    for (int w = 0; w < kSums * kNormWaves; ++w) total += s_ss[w];
    const float r = 1.0f / sqrtf(total / (float)K + p.eps);

    float amax = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int k = (tid + i * THREADS) * 4;
        float g[4];
        if constexpr (kGammaEarly) {
#pragma unroll
            for (int j = 0; j < 4; ++j) g[j] = gam[i][j];
        } else {
            load4<VEC>(p.gamma, k, K, g);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            x[i][j] = (x[i][j] * g[j]) * r;
            amax = fmaxf(amax, fabsf(x[i][j]));
        }
        if (p.y) store4<VEC>(p.y + row, k, K, x[i]);
    }
    if (!p.q) return;   // uniform: the final norm of a model quantizes nothing
    amax = wave_max(amax);
    if (lane == 0) s_max[wave] = amax;
    __syncthreads();
    amax = s_max[0];
#pragma unroll
    for (int w = 1; w < kNormWaves; ++w) amax = fmaxf(amax, s_max[w]);
    float inv, scale;
    quant_scales(amax, inv, scale);

    int8_t* qrow = p.q + (int64_t)blockIdx.x * p.Kp;
    int sum = 0;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int k = (tid + i * THREADS) * 4;
        const uint32_t word = quantize4(x[i][0], x[i][1], x[i][2], x[i][3], inv, sum);   // elements from K on are zero and quantize to zero
        if (k < K) *reinterpret_cast<uint32_t*>(qrow + k) = word;
    }
    for (int k = (K + 3) / 4 * 4 + tid * 4; k < p.Kp; k += THREADS * 4) *reinterpret_cast<uint32_t*>(qrow + k) = 0;
    sum = wave_sum(sum);
    if (lane == 0) s_sum[wave] = sum;
    __syncthreads();
    if (tid == 0) {
        int t = 0;
#pragma unroll
        for (int w = 0; w < kNormWaves; ++w) t += s_sum[w];
        p.a_scale[blockIdx.x] = scale;
        if (p.q_sum) p.q_sum[blockIdx.x] = t;
    }
}

template <int MODE, int THREADS, int NV>
hipError_t launch_norm_nv(const NormArgs& p, int M, bool vec, hipStream_t s) {
    if (vec) norm_quant_kernel<MODE, NV, true, THREADS><<<dim3((unsigned)M), dim3(THREADS), 0, s>>>(p);
    else norm_quant_kernel<MODE, NV, false, THREADS><<<dim3((unsigned)M), dim3(THREADS), 0, s>>>(p);
    return hipGetLastError();
}

// The smallest instance of MIN_NV up to MAX_NV vectors per thread that holds the row.
template <int MODE, int THREADS, int MIN_NV, int MAX_NV>
hipError_t launch_norm_threads(const NormArgs& p, int M, bool vec, hipStream_t s) {
    const int per_thread = (p.K + THREADS * 4 - 1) / (THREADS * 4);
#define BL_NORM_NV(NV)                       \
    if constexpr (MIN_NV <= NV && NV <= MAX_NV) \
        if (per_thread <= NV) return launch_norm_nv<MODE, THREADS, NV>(p, M, vec, s);
    BL_NORM_NV(1)
    BL_NORM_NV(2)
    BL_NORM_NV(3)
    BL_NORM_NV(4)
    BL_NORM_NV(6)
    BL_NORM_NV(8)
    BL_NORM_NV(12)
#undef BL_NORM_NV
    return hipErrorInvalidValue;
}

// Threads per row: as few as leave a thread two (rows up to 2048) or four (up to 8192) vectors -- a row's three reductions and
// barriers cost by the wave -- and 1024 for longer rows, where one row's loads and arithmetic have to be spread out.  Measured
// with 1024 / 512 / 256 threads, inputs from memory (us): 2048 rows of 768, plain 10.3 / 6.2 / 4.7; 2048 of 2048, plain 11.4 / 7.4 /
// 6.2, gated 13.7 / 9.2 / 9.2; 1 row of 4096, plain 3.0 / 2.7 / 2.9; 2048 of 4096, residual 19.4 / 18.0 / 18.4, gated 18.1 / 15.8 / 15.9; 512
// of 8192, plain 6.4 / 6.1 / 7.3, gated 9.2 / 9.5 / 11.1; 512 of 8704, residual 9.9 / 10.4 / 12.2, gated 10.8 / 11.2 / 15.2; 512 of 12032,
// gated 12.6 / 13.2 / 17.3, and so from 64 rows (5.8 / 6.0) to 2048 (41.2 / 41.8).
template <int MODE>
hipError_t launch_norm_mode(const NormArgs& p, int M, bool vec, hipStream_t s) {
    if (p.K <= 2048) return launch_norm_threads<MODE, 256, 1, 2>(p, M, vec, s);
    if (p.K <= 8192) return launch_norm_threads<MODE, 512, 2, 4>(p, M, vec, s);
    return launch_norm_threads<MODE, kNormThreads, 3, 12>(p, M, vec, s);
}
static_assert(BL_NORM_MAX_K == 12 * kNormThreads * 4, "the longest row fills 12 vectors per thread");

// Long rows (K >= kWideMinK, with scratch memory from the caller): one workgroup is bound by its compute unit's ALU on
// such a row (45568 gated elements: 20 us), so the row is cut into slices of 2048 elements, one workgroup each, and the
// work into two launches with the grid-wide reductions between them:
//   1. x (residual add stored, or the gate), z = x * gamma; per slice sum(x^2) and max|z| to scratch; sum(q) zeroed;
//   2. every workgroup adds up the slices' figures in the same order (so all get the same bits): r, and max|y| =
//      max|z| * r -- rounding is monotone and r > 0, so the largest |z| gives the largest |z * r|, which is why y is
//      defined as (x * gamma) * r in that order; then y and the codes of its slice; sum(q) by integer atomics.
constexpr int kWideThreads = 256;
constexpr int kWideSlice = kWideThreads * 8;
constexpr int kWideMinK = 16384;
constexpr int kWideMaxSlices = BL_NORM_MAX_K / kWideSlice;
static_assert(kWideMaxSlices * sizeof(float2) <= BL_NORM_SCRATCH_BYTES, "a row's partial figures fit its scratch");

template <int MODE, bool VEC>
__device__ __forceinline__ void wide_inputs(const NormArgs& p, int64_t row, int k, int K, bool second_pass, float (&x)[4]) {
    if constexpr (MODE == BL_NORM_PLAIN || MODE == BL_NORM_PREMULTIPLIED) {
        load4<VEC>(p.a + row, k, K, x);
    } else if constexpr (MODE == BL_NORM_RESIDUAL) {
        load4<VEC>(p.h + row, k, K, x);
        if (p.a && !second_pass) {     // the first launch adds and stores; the second finds the sum in h
            float d[4];
            load4<VEC>(p.a + row, k, K, d);
#pragma unroll
            for (int j = 0; j < 4; ++j) x[j] += d[j];
            store4<VEC>(p.h + row, k, K, x);   // (h_out is h in this form)
        }
    } else {
        float g[4], u[4];
        load4<VEC>(p.a + row, k, K, g);
        load4<VEC>(p.b + row, k, K, u);
        silu4(g, x);
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] *= u[j];
    }
}

template <int MODE, bool VEC>
__global__ __launch_bounds__(kWideThreads) void norm_wide_stats_kernel(const NormArgs p) {
    __shared__ float s_ss[kWideThreads / kWave], s_max[kWideThreads / kWave];
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    const int K = p.K, slice = blockIdx.x;
    const int64_t row = (int64_t)blockIdx.y * K;
    float ss = 0.0f, amax = 0.0f;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int k = slice * kWideSlice + (tid + i * kWideThreads) * 4;
        float x[4], g[4];
        load4<VEC>(p.gamma, k, K, g);
        wide_inputs<MODE, VEC>(p, row, k, K, false, x);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            ss += x[j] * x[j];
            amax = fmaxf(amax, fabsf(x[j] * g[j]));
        }
    }
    ss = wave_sum_f(ss);
    amax = wave_max(amax);
    if (lane == 0) { s_ss[wave] = ss; s_max[wave] = amax; }
    __syncthreads();
    if (tid == 0) {
        static_assert(kWideThreads / kWave == 4, "four partial figures");
        p.scratch[(int64_t)blockIdx.y * kWideMaxSlices + slice] =
            make_float2((s_ss[0] + s_ss[1]) + (s_ss[2] + s_ss[3]), fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3])));
        if (slice == 0 && p.q_sum) p.q_sum[blockIdx.y] = 0;
    }
}

template <int MODE, bool VEC>
__global__ __launch_bounds__(kWideThreads) void norm_wide_quant_kernel(const NormArgs p) {
    __shared__ int s_sum[kWideThreads / kWave];
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    const int K = p.K, slice = blockIdx.x, slices = gridDim.x;
    const int64_t row = (int64_t)blockIdx.y * K;
    float total = 0.0f, amax_z = 0.0f;
    if constexpr (MODE == BL_NORM_PREMULTIPLIED) {
        // the pieces of a gated launch, hundreds of them: every workgroup adds them up the same way (thread t takes
        // pieces t, t + 256, ...; lanes, then waves) and so arrives at the same bits
        __shared__ float s_tot[kWideThreads / kWave], s_amax[kWideThreads / kWave];
        for (int i = tid; i < p.pieces; i += kWideThreads) {
            const float2 f = p.scratch[i];
            total += f.x;
            amax_z = fmaxf(amax_z, f.y);
        }
        total = wave_sum_f(total);
        amax_z = wave_max(amax_z);
        if (lane == 0) { s_tot[wave] = total; s_amax[wave] = amax_z; }
        __syncthreads();
        total = (s_tot[0] + s_tot[1]) + (s_tot[2] + s_tot[3]);
        amax_z = fmaxf(fmaxf(s_amax[0], s_amax[1]), fmaxf(s_amax[2], s_amax[3]));
    } else {
        const float2* part = p.scratch + (int64_t)blockIdx.y * kWideMaxSlices;
        for (int g = 0; g < slices; ++g) {      // the same order in every workgroup
            const float2 f = part[g];
            total += f.x;
            amax_z = fmaxf(amax_z, f.y);
        }
    }
    const float r = 1.0f / sqrtf(total / (float)K + p.eps);
    float inv, scale;
    quant_scales(amax_z * r, inv, scale);
    int8_t* qrow = p.q ? p.q + (int64_t)blockIdx.y * p.Kp : nullptr;
    int sum = 0;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int k = slice * kWideSlice + (tid + i * kWideThreads) * 4;
        float x[4], g[4] = {1.0f, 1.0f, 1.0f, 1.0f};
        if constexpr (MODE != BL_NORM_PREMULTIPLIED) load4<VEC>(p.gamma, k, K, g);
        wide_inputs<MODE, VEC>(p, row, k, K, true, x);
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = MODE == BL_NORM_PREMULTIPLIED ? x[j] * r : (x[j] * g[j]) * r;
        const uint32_t word = quantize4(x[0], x[1], x[2], x[3], inv, sum);
        if (p.y) store4<VEC>(p.y + row, k, K, x);
        if (qrow && k < K) *reinterpret_cast<uint32_t*>(qrow + k) = word;
    }
    if (!qrow) return;   // uniform
    if (slice == slices - 1)
        for (int k = (K + 3) / 4 * 4 + tid * 4; k < p.Kp; k += kWideThreads * 4) *reinterpret_cast<uint32_t*>(qrow + k) = 0;
    sum = wave_sum(sum);
    if (lane == 0) s_sum[wave] = sum;
    __syncthreads();
    if (tid == 0) {
        const int part = (s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]);
        if constexpr (MODE == BL_NORM_PREMULTIPLIED) {
            // no earlier launch of this call could zero sum(q), so the slices meet in one 64-bit word behind the
            // pieces: slice count in the high bits, signed sum in the low 40; the slice that completes the count
            // writes the total and puts the word back to zero (it is zero before the first call)
            if (p.q_sum) {
                unsigned long long* word = reinterpret_cast<unsigned long long*>(p.scratch + p.pieces);
                const unsigned long long add = (1ull << 40) + (unsigned long long)(long long)part;
                const unsigned long long now =
                    __hip_atomic_fetch_add(word, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + add;
                const long long sum = (long long)(now << 24) >> 24;
                if ((long long)((now - (unsigned long long)sum) >> 40) == slices) {
                    p.q_sum[0] = (int)sum;
                    __hip_atomic_store(word, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        } else if (p.q_sum) {
            atomicAdd(p.q_sum + blockIdx.y, part);
        }
        if (slice == 0) p.a_scale[blockIdx.y] = scale;
    }
}

// The pre-multiplied form: the figures of the first launch are there already (a gated product's epilogue left them).
hipError_t launch_norm_premultiplied(const NormArgs& p, bool vec, hipStream_t s) {
    const dim3 grid((unsigned)((p.K + kWideSlice - 1) / kWideSlice), 1u), block(kWideThreads);
    if (vec) norm_wide_quant_kernel<BL_NORM_PREMULTIPLIED, true><<<grid, block, 0, s>>>(p);
    else norm_wide_quant_kernel<BL_NORM_PREMULTIPLIED, false><<<grid, block, 0, s>>>(p);
    return hipGetLastError();
}

template <int MODE>
hipError_t launch_norm_wide(const NormArgs& p, int M, bool vec, hipStream_t s) {
    const dim3 grid((unsigned)((p.K + kWideSlice - 1) / kWideSlice), (unsigned)M), block(kWideThreads);
    if (vec) norm_wide_stats_kernel<MODE, true><<<grid, block, 0, s>>>(p);
    else norm_wide_stats_kernel<MODE, false><<<grid, block, 0, s>>>(p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (vec) norm_wide_quant_kernel<MODE, true><<<grid, block, 0, s>>>(p);
    else norm_wide_quant_kernel<MODE, false><<<grid, block, 0, s>>>(p);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------------------
// Rotary table

__global__ __launch_bounds__(256) void rope_table_kernel(float2* table, int half, int64_t entries, double theta) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= entries) return;
    const int64_t pos = idx / half;
    const int i = (int)(idx - pos * half);
    const double angle = (double)pos * pow(theta, -(double)i / (double)half);   // theta^(-2 i / head_dim)
    table[idx] = make_float2((float)cos(angle), (float)sin(angle));
}

// ---------------------------------------------------------------------------------------------------------------
// Attention over the cache

constexpr int kAttnThreads = 256;
constexpr int kAttnWaves = kAttnThreads / kWave;
constexpr int kChunk = BL_ATTN_CHUNK;
static_assert(kChunk == kWave, "the chunk's softmax runs in one wavefront");

struct AttnArgs {
    const float*   q_lin;
    const float*   k_lin;
    const float*   v_lin;
    const int32_t* pos;
    const float2*  rope;
    uint16_t*      k_cache;
    uint16_t*      v_cache;
    float*         out;
    float*         scratch;     // per query [n_heads][chunks][head_dim + 2] (weighted values, maximum, sum), then n_heads counters
    int32_t        counters_apart;   // the ticket counters are the first words of the heads' last pieces, which nobody deposits in
    int32_t        n_heads, head_dim, max_pos, chunks;
    // several consecutive tokens (a prompt): pos is null, query z has position pos0 + z, its own row of q_lin and out
    // and its own part of scratch; keys and values are in the cache already (kv_append_kernel)
    int32_t        pos0;
    int32_t        groups;           // workgroups per head (the one-token launch's are its grid's)
    int64_t        scratch_stride;   // floats per query
};

__device__ __forceinline__ uint16_t f32_to_bf16(float f) {   // nearest, ties to even; finite inputs
    const uint32_t u = __float_as_uint(f);
    return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

// W bf16 values as one register vector: 128 bits for W = 8, 64 bits for W = 4.
template <int W> struct CacheVec;
template <> struct CacheVec<8> { typedef uint32_t type __attribute__((ext_vector_type(4))); };
template <> struct CacheVec<4> { typedef uint32_t type __attribute__((ext_vector_type(2))); };

template <int W>
__device__ __forceinline__ void unpack_bf16(const typename CacheVec<W>::type& u, float (&f)[W]) {
    const uint32_t* w = reinterpret_cast<const uint32_t*>(&u);
#pragma unroll
    for (int i = 0; i < W / 2; ++i) {
        f[2 * i] = bf16_to_f32(w[i] & 0xffffu);
        f[2 * i + 1] = bf16_to_f32(w[i] >> 16);
    }
}

// Sum or maximum over groups of L neighbouring lanes (16, 32 or 64), on the vector ALU's lane moves instead of a trip through LDS per
// step (ds_bpermute): lane ^ 1 and ^ 2 by quad permutation, the other half of eight and of sixteen lanes by their mirror images -- whose
// lanes all hold their quad's or half's result by then -- and the 16- and 32-lane blocks by the swaps of two registers.  Every step
// adds the two halves' figures (in either order the same bits), so every lane gets the same result.
#define BL_LANES(v, ctrl) __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), (ctrl), 0xf, 0xf, false))
template <int OFF, typename Op>
__device__ __forceinline__ float over_blocks(float v, Op op) {   // lane and lane ^ OFF
    static_assert(OFF == 16 || OFF == 32, "the two swaps");
    const uint32_t u = __float_as_uint(v);
    if constexpr (OFF == 16) {
        const auto s = __builtin_amdgcn_permlane16_swap(u, u, false, false);
        return op(__uint_as_float(s[0]), __uint_as_float(s[1]));
    } else {
        const auto s = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        return op(__uint_as_float(s[0]), __uint_as_float(s[1]));
    }
}
template <int L, typename Op>
__device__ __forceinline__ float over_lanes(float v, Op op) {
    static_assert(L == 16 || L == 32 || L == 64, "whole rows of sixteen lanes");
    v = op(v, BL_LANES(v, 0xb1));    // quad_perm [1, 0, 3, 2]
    v = op(v, BL_LANES(v, 0x4e));    // quad_perm [2, 3, 0, 1]
    v = op(v, BL_LANES(v, 0x141));   // row_half_mirror
    v = op(v, BL_LANES(v, 0x140));   // row_mirror
    if constexpr (L >= 32) v = over_blocks<16>(v, op);
    if constexpr (L >= 64) v = over_blocks<32>(v, op);
    return v;
}
#undef BL_LANES
struct AddOp { __device__ __forceinline__ float operator()(float a, float b) const { return a + b; } };
struct MaxOp { __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); } };

// One head's chunks merged by one workgroup: out = sum_c f_c o_c / sum_c f_c l_c with f_c = exp(m_c - max m) over the
// chunks that hold rows 0 .. pos.  The chunks' maxima and sums are read one per thread; the factors go through LDS.
// A value another workgroup of this launch has published (see publish below): read where it was deposited, by a
// device-scope atomic load (it does not take its value from this die's cache).
__device__ __forceinline__ float read_published(float* at) {
    return __uint_as_float(__hip_atomic_load(reinterpret_cast<unsigned int*>(at), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// Up to kMergeTogether workgroups' figures (all that bl_attn_decode launches by itself): every value is requested at once -- a
// read of this kind is a round trip to memory (32 heads of 128, 32 workgroups per head, four values at a time: 17.6 us, this: 16.0).  The threads of a workgroup are kAttnThreads / MAXD teams of
// MAXD, each taking every so-manieth deposit.  s_f: kMergeTogether floats, s_red: kAttnWaves, s_o: [teams][MAXD].
constexpr int kMergeTogether = 64;   // one wave reads all maxima and sums
static_assert(kMergeTogether <= kWave, "one lane per deposit");
template <int MAXD, int N>   // N: deposits it can take
__device__ __forceinline__ void attn_merge_together(const AttnArgs& p, float* scratch, float* out, int head, int used, float* s_f,
                                                    float* s_red, float* s_o) {
    constexpr int kTeams = kAttnThreads / MAXD, kMine = N / kTeams;
    const int tid = threadIdx.x, d = p.head_dim;
    const int team = tid / MAXD, el = tid % MAXD;
    float* base = scratch + (int64_t)head * p.chunks * (d + 2);
    float part[kMine];
#pragma unroll
    for (int j = 0; j < kMine; ++j) part[j] = read_published(base + min(team + j * kTeams, used - 1) * (d + 2) + min(el, d - 1));
    if (tid < kWave) {
        const int c = min(tid, used - 1);
        const float m_c = read_published(base + c * (d + 2) + d), l_c = read_published(base + c * (d + 2) + d + 1);
        const float m = over_lanes<kWave>(m_c, MaxOp());
        const float f = tid < used ? expf(m_c - m) : 0.0f;
        if (tid < N) s_f[tid] = f;
        const float l = wave_sum_f(f * l_c);
        if (tid == 0) s_red[0] = l;
    }
    __syncthreads();
    float o = 0.0f;
#pragma unroll
    for (int j = 0; j < kMine; ++j)   // beyond the last deposit: the factor is zero, the value finite or that deposit's own
        o = team + j * kTeams < used ? __builtin_fmaf(s_f[team + j * kTeams], part[j], o) : o;
    if constexpr (kTeams > 1) {
        s_o[tid] = o;
        __syncthreads();
        if (tid < MAXD) {
#pragma unroll
            for (int t = 1; t < kTeams; ++t) o += s_o[t * MAXD + tid];
        }
    }
    if (tid < d) out[head * d + tid] = o / s_red[0];
}

// Any number of them.
__device__ __forceinline__ void attn_merge(const AttnArgs& p, float* scratch, float* out, int head, int used, float* s_f,
                                           float* s_red) {
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    const int d = p.head_dim;
    float* base = scratch + (int64_t)head * p.chunks * (d + 2);
    const auto src = [&](int i) { return read_published(base + i); };
    float m = -INFINITY;
    for (int c = tid; c < used; c += kAttnThreads) m = fmaxf(m, src(c * (d + 2) + d));
    m = over_lanes<kWave>(m, MaxOp());
    if (lane == 0) s_red[wave] = m;
    __syncthreads();
    m = fmaxf(fmaxf(s_red[0], s_red[1]), fmaxf(s_red[2], s_red[3]));
    static_assert(kAttnWaves == 4, "four partial maxima");
    float l = 0.0f, o = 0.0f;
    for (int c0 = 0; c0 < used; c0 += kAttnThreads) {   // one pass unless the context exceeds 256 chunks
        __syncthreads();                                // s_f and s_red of the previous pass have been read
        const int c = c0 + tid;
        float f = 0.0f, fl = 0.0f;
        if (c < used) {
            f = expf(src(c * (d + 2) + d) - m);
            fl = f * src(c * (d + 2) + d + 1);
        }
        s_f[tid] = f;
        fl = wave_sum_f(fl);
        if (lane == 0) s_red[wave] = fl;
        __syncthreads();
        l += (s_red[0] + s_red[1]) + (s_red[2] + s_red[3]);
        const int n = min(kAttnThreads, used - c0);
        if (tid < d) {
#pragma unroll 4
            for (int i = 0; i < n; ++i) o += s_f[i] * src((c0 + i) * (d + 2) + tid);
        }
    }
    if (tid < d) out[head * d + tid] = o / l;
}

// A chunk is 64 cache rows.  Its keys and values (64 x head_dim bf16 each) are requested as W values per thread and
// request, MAXD / W consecutive lanes on one row; while they travel the query is rotated (and, in the chunk that
// holds the token's own row, key and value are rotated, rounded and appended).  The lanes of a row keep a running maximum, sum
// and weighted values of THEIR rows over all chunks of the workgroup: the dot product's exchanges are the only ones in the
// loop, and there is no barrier in it, so no wave's requests wait for another wave's rows.  The groups of lanes are merged by
// lane exchanges, the four waves in LDS, once behind the loop.  Bound by HBM in long contexts: 32 heads of 128 at 8000 positions
// 36.3 -> 30 -> 26.9 -> 23.0 us (131 MB: 5.7 TB/s), 16 000 positions 47.8 -> 41.7 (every 8000 positions more 18.2: 7.2 TB/s);
// by the chain of memory round trips in short ones (caches from memory): one position 4.8 -> 3.4, 500 positions 10.2 -> 7.4, 3000 18.0 -> 13.7.
// Before lane sums on the vector ALU, the next chunk's requests without a condition and fewer workgroups per head -> since; the last
// change kept the requests where they are written and put the angle's load ahead of them: 16 heads of 100 at 8000 positions
// 21.2 -> 17.8, 12 of 44 at 16 000 24.2 -> 19.0, 20 of 160 at 500 / 3000 / 8000 8.9 -> 8.0, 16.2 -> 13.3, 31.6 -> 24.4, 30 of 256 10.7 -> 9.4, 25.6 -> 22.4,
// 55.4 -> 48.1, 32 of 128 at 500 8.1 -> 7.4.
// A token's cache rows are read once, by streaming loads: caches from memory, ordinary -> streaming, 32 heads of 128 at 500 positions 7.9 -> 7.6,
// 2000 11.1 -> 10.5, 8000 27.7 -> 25.2, 16 000 47.8 -> 42.0, 64 heads at 4000 28.5 -> 25.9; caches that the memory-side cache holds stay there
// and are as fast (8000: 24.3 and 24.0), and so do a model's weights: 700M shape 810 -> 740 us per token at 3000 positions, 715 -> 694 at 500.
// Heads that share lines of the cache are on one die (attn_columns), so that its L2 hands a line that came for one of them to the other; without
// that, streaming loads brought it from memory twice (32 heads of 48, 5000 positions, ordinary / streaming / so: 16.0 / 16.6 / 11.9).  Whole
// tokens of that shape (1.5B) 967 / 905 / 887 us at 1500, 1142 / 1092 / 987 at 4500, 1722 / 1713 / 1315 at 14 000.
// Below 100 positions a token's rows come from the L2 if the loads are ordinary: there streaming costs a model 0.5 % (7B shape 1075 -> 1081 us at 10,
// 1147 -> 1150 at 100, then 1190 -> 1164 at 450).  Both kinds in one kernel, by the position, cost more than that (1088, 1158, 1183).
// With them one workgroup per unit is enough at any length (bl_attn_groups.hpp: 25.2 -> 23.0 at 8000).
// MAXD: the largest head size of this instance (128 or 256) -- registers and LDS are sized by it, and the smaller one
// lets twice as many workgroups share a compute unit.
// Waves per SIMD: 5 (head sizes up to 128) and 4 (beyond), held for the compiler; every instance fits without spilling: 85, 77,
// 124 and 126 registers.  (Five spilled registers of <8, 256>, reloaded behind the next keys' requests, made every chunk wait for
// those: 40 heads of 160 at 16 000 positions 92.8 us, without spills 79.7.)
// PROMPT: several tokens whose keys and values are cached already, one per grid z.  Its grid's x counts heads and workgroups together,
// padded to whole rounds of the dies, so that one die's L2 serves a piece of the cache to all queries (28 heads of 160, nine workgroups each,
// behind 2000 positions, unpadded and padded: 4 tokens 35.3 and 29.5 us, 16 tokens 107 and 74; 12 of 160, 9 behind 3000 42.2 and 33.3).
template <int W, int MAXD, bool PROMPT>
__device__ __forceinline__ void attn_walk(const AttnArgs& p) {
    typedef typename CacheVec<W>::type vec_t;
    constexpr int kMaxLanesPerRow = MAXD / W;
    constexpr int kVecs = kChunk * kMaxLanesPerRow / kAttnThreads;            // requests per thread at most
    __shared__ __attribute__((aligned(16))) float s_q[MAXD];                  // rotated query / sqrt(head_dim)
    __shared__ __attribute__((aligned(16))) uint16_t s_newk[MAXD];            // the token's own key and value as cached
    __shared__ __attribute__((aligned(16))) uint16_t s_newv[MAXD];
    __shared__ float s_ow[kAttnWaves][MAXD];            // per wave: weighted values of its rows
    __shared__ float s_mw[kAttnWaves], s_lw[kAttnWaves];   // per wave: maximum and sum
    __shared__ float s_w[kChunk];                       // the merge's partial results
    __shared__ float s_o[kAttnThreads];                 // the merge's factors
    const int tid = threadIdx.x;
    const int head = PROMPT ? (int)(blockIdx.x % (unsigned)p.n_heads) : attn_head_at(blockIdx.x, blockIdx.z, gridDim.z);
    const int chunk = PROMPT ? (int)(blockIdx.x / (unsigned)p.n_heads) : (int)blockIdx.y;
    const int groups = PROMPT ? p.groups : (int)gridDim.y;   // workgroups per head
    if (PROMPT && chunk >= groups) return;              // uniform: the grid's padding
    const int d = p.head_dim, half = d / 2;
    const int hidden = p.n_heads * d;
    const int query = PROMPT ? (int)blockIdx.z : 0;     // 0 unless a prompt's tokens are processed together
    const float* q_lin = p.q_lin + (int64_t)query * hidden;
    float* out = p.out + (int64_t)query * hidden;
    float* scratch = p.scratch + (int64_t)query * p.scratch_stride;
    // the token's projections do not depend on the position: requested before the position is waited for
    float qa = 0.0f, qb = 0.0f, ka = 0.0f, kb = 0.0f, va = 0.0f, vb = 0.0f;
    if (tid < half) {
        qa = q_lin[head * d + tid]; qb = q_lin[head * d + tid + half];
        if (!PROMPT) {
            ka = p.k_lin[head * d + tid]; kb = p.k_lin[head * d + tid + half];
            va = p.v_lin[head * d + tid]; vb = p.v_lin[head * d + tid + half];
        }
    }
    const int pos = __builtin_amdgcn_readfirstlane(PROMPT ? p.pos0 + query : *p.pos);
    if (pos < 0 || pos >= p.max_pos) return;            // uniform
    // Workgroup y of a head takes the chunks y, y + G, y + 2G, ... (G = `groups`) that hold
    // rows up to the token's: one chunk each while the context is short, several once it outgrows the launch -- then
    // a workgroup folds its chunks into ONE running maximum, sum and weighted values before it deposits anything.
    const int last_chunk = pos / kChunk;
    if (chunk > last_chunk) return;                     // uniform: nothing cached this far yet
    const bool owner = !PROMPT && last_chunk % groups == chunk;   // uniform: one of this workgroup's chunks holds the row this launch appends
    constexpr int L = kMaxLanesPerRow;                  // lanes per cache row: a power of two; those beyond head_dim / W idle
    constexpr int kRowsPerStep = kAttnThreads / L;      // rows the workgroup takes per request
    const int lane = tid % kWave, wave = tid / kWave;
    const int grp = tid / L, cc = tid % L;
    const bool active = cc * W < d;

    // rows beyond the token's are read as the token's row (always inside the cache) and never used; the token's own
    // row may be read while this workgroup writes it and is replaced by the values kept in LDS
    vec_t kv[kVecs], vv[kVecs];
    const uint32_t row_bytes = 2u * (uint32_t)hidden;   // a chunk's rows: below 2^32 bytes (heads and head size are bounded)
    const auto request = [&](int c, bool keys) {
        // scalar base, 32-bit lane offsets, and neither kept from one request to the next (the registers are needed)
        typedef const __attribute__((address_space(1))) uint8_t* global_t;
        global_t base = (global_t)(uintptr_t)((keys ? p.k_cache : p.v_cache) + (int64_t)c * kChunk * hidden + head * d);
        int rest = pos - c * kChunk;
        asm volatile("" : "+s"(base), "+s"(rest));
        // Requests stay where they are: the compiler moves loads down to their first use if it finds registers short, behind
        // the waits that they were to travel under.
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < kVecs; ++i) {
            // (idle lanes read their row's first piece: a branch around the requests would hide from the compiler how many there are)
            const uint32_t at = (uint32_t)min(grp + i * kRowsPerStep, rest) * row_bytes + (active ? cc * W * 2u : 0u);
            typedef const __attribute__((address_space(1))) vec_t* global_vec;
            vec_t& to = keys ? kv[i] : vv[i];
            // streaming (nontemporal) loads; a prompt's queries read the same rows (16 heads of 164, 9 behind 4000: streaming 87 us, 74)
            if constexpr (!PROMPT) to = __builtin_nontemporal_load((global_vec)(base + at));
            else to = *(global_vec)(base + at);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // (the angle first: what it is needed for goes on under the requests behind it)
    const float2 cs = p.rope[(int64_t)pos * half + min(tid, half - 1)];
    request(chunk, true);
    request(chunk, false);

    const float scale = 1.0f / sqrtf((float)d);
    if (tid < half) {
        s_q[tid] = (qa * cs.x - qb * cs.y) * scale;
        s_q[tid + half] = (qa * cs.y + qb * cs.x) * scale;
        if (owner) {
            const uint16_t k0 = f32_to_bf16(ka * cs.x - kb * cs.y), k1 = f32_to_bf16(ka * cs.y + kb * cs.x);
            const uint16_t v0 = f32_to_bf16(va), v1 = f32_to_bf16(vb);
            uint16_t* krow = p.k_cache + (int64_t)pos * hidden + head * d;
            uint16_t* vrow = p.v_cache + (int64_t)pos * hidden + head * d;
            krow[tid] = k0; krow[tid + half] = k1;
            vrow[tid] = v0; vrow[tid + half] = v1;
            s_newk[tid] = k0; s_newk[tid + half] = k1;
            s_newv[tid] = v0; s_newv[tid + half] = v1;
        }
    }

    // Every group of L lanes keeps ITS rows' running maximum, sum and weighted values over all chunks of the workgroup: no
    // barrier and no exchange beyond the dot products' inside the loop, so a wave's next requests never wait for another
    // wave's rows.  The groups, then the waves, are merged once, behind the loop.
    __syncthreads();                                    // s_q and the token's own row are there
    float q[W];
#pragma unroll
    for (int x = 0; x < W; ++x) q[x] = active ? s_q[cc * W + x] : 0.0f;
    float m_g = -INFINITY, l_g = 0.0f, o_g[W];
#pragma unroll
    for (int x = 0; x < W; ++x) o_g[x] = 0.0f;
    const int wave_row = __builtin_amdgcn_readfirstlane(wave) * (kWave / L);   // the wave's first row of a step
    static_assert(L <= kWave, "a row's lanes are one wave's");
    // One chunk.  While more follow, its successor's keys are requested when the dot products are done and its values when the
    // weighted ones are, without a condition: with one the compiler has to count on the requests not being there, and waited for the
    // next keys before it used this chunk's values.  kVecs requests are on their way at any time (tests/test_wait_counts.py looks at
    // the compiled loop).  Only the last chunk can hold the token's own row or rows beyond it.
    const auto pass = [&](int c, auto last) {
        constexpr bool kLast = decltype(last)::value;
        const int j0 = c * kChunk;
        const int rows = kLast ? min(kChunk, pos + 1 - j0) : kChunk;
        const bool holds_token = kLast && owner && c == last_chunk;   // uniform
        float score[kVecs];
#pragma unroll
        for (int i = 0; i < kVecs; ++i) {
            float k[W], acc = 0.0f;
            vec_t x16 = kv[i];
            if (holds_token && j0 + grp + i * kRowsPerStep == pos)   // this launch appends that row: its values are in LDS
                x16 = *reinterpret_cast<const vec_t*>(&s_newk[active ? cc * W : 0]);
            unpack_bf16<W>(x16, k);
#pragma unroll
            for (int x = 0; x < W; ++x) acc = __builtin_fmaf(q[x], k[x], acc);
            score[i] = active ? acc : 0.0f;
        }
        if constexpr (!kLast) request(c + groups, true);   // the next chunk travels while this one is worked on
#pragma unroll
        for (int i = 0; i < kVecs; ++i) {
            const float acc = over_lanes<L>(score[i], AddOp());
            score[i] = grp + i * kRowsPerStep < rows ? acc : -INFINITY;
        }
        float m_new = m_g;
#pragma unroll
        for (int i = 0; i < kVecs; ++i) m_new = fmaxf(m_new, score[i]);
        const float base = m_new == -INFINITY ? 0.0f : m_new;   // a group without rows so far adds nothing
        const float f = expf(m_g - base);
        m_g = m_new;
        // the chunk's figures by themselves first: a walk's sums then grow by chunks and not by rows (fewer roundings in a row)
        float l_c = 0.0f, o_c[W];
#pragma unroll
        for (int i = 0; i < kVecs; ++i) {
            // the first tokens of a context: the wave has no row in this step (uniform; 8 heads of 128 at 2 positions 5.5 -> 4.9 us)
            if (kLast && i > 0 && wave_row + i * kRowsPerStep >= rows) continue;
            const float w = expf(score[i] - base);
            l_c += w;
            float v[W];
            vec_t x16 = vv[i];
            if (kLast) {
                if (holds_token && j0 + grp + i * kRowsPerStep == pos) x16 = *reinterpret_cast<const vec_t*>(&s_newv[active ? cc * W : 0]);
                // rows beyond the token's are selected out, not multiplied out: their registers hold whatever the cache
                // held before (row `pos` is requested before this launch writes it; a caller's cache need not be finite)
                if (grp + i * kRowsPerStep >= rows) x16 = vec_t{};
            }
            unpack_bf16<W>(x16, v);
#pragma unroll
            for (int x = 0; x < W; ++x) o_c[x] = i == 0 ? w * v[x] : __builtin_fmaf(w, v[x], o_c[x]);   // (idle lanes': never looked at)
        }
        l_g = __builtin_fmaf(l_g, f, l_c);
#pragma unroll
        for (int x = 0; x < W; ++x) o_g[x] = __builtin_fmaf(o_g[x], f, o_c[x]);
        if constexpr (!kLast) request(c + groups, false);
    };
    // The chunks before the last one in blocks of four, whose figures go to sums of their own when a block is through: a long walk's sums
    // then have a quarter of the roundings in a row.  Error against 64 bits, one running sum and this: 32 heads of 128 at 8000 positions 1.99e-7 and
    // 1.94e-7, 64 heads 2.09e-7 and 1.95e-7, 52 heads at 10 000 2.16e-7 and 1.99e-7 (1.65e-7 at 1000 positions); as fast.  A compensated
    // running sum: 1.86e-7, 1.85e-7, 1.85e-7, but 1 to 4 % of the time.  The blocks' figures are written only if there is a chunk before the last one: set
    // to zero by all, they took a short cache's call 2 % (32 heads of 128, warm, at 30 / 63 positions 3.58 / 3.83 us, so 3.50 / 3.71).
    float m_b, l_b, o_b[W];
    const auto with_blocks = [&](float& l, float (&o)[W]) {   // the present figures with the blocks' before them
        const float f = expf(m_b - (m_g == -INFINITY ? 0.0f : m_g));
        l = __builtin_fmaf(l_b, f, l_g);
#pragma unroll
        for (int x = 0; x < W; ++x) o[x] = __builtin_fmaf(o_b[x], f, o_g[x]);
    };
    int c = chunk;
    const int end = last_chunk - groups + 1;
    if (c < end) {   // uniform
        m_b = -INFINITY;
        l_b = 0.0f;
#pragma unroll
        for (int x = 0; x < W; ++x) o_b[x] = 0.0f;
        do {
            const int block = min(c + 4 * groups, end);
            do {
                pass(c, std::false_type{});
                c += groups;
            } while (c < block);
            with_blocks(l_b, o_b);
            m_b = m_g;
            l_g = 0.0f;
#pragma unroll
            for (int x = 0; x < W; ++x) o_g[x] = 0.0f;
        } while (c < end);
    }
    pass(c, std::true_type{});
    if (chunk < end) with_blocks(l_g, o_g);
    // the wave's groups into the wave's figures
    float m_w = m_g;
    if constexpr (L <= 16) m_w = over_blocks<16>(m_w, MaxOp());
    if constexpr (L <= 32) m_w = over_blocks<32>(m_w, MaxOp());
    const float f_g = m_g == -INFINITY ? 0.0f : expf(m_g - m_w);
    l_g *= f_g;
#pragma unroll
    for (int x = 0; x < W; ++x) o_g[x] *= f_g;
    if constexpr (L <= 16) {
        l_g = over_blocks<16>(l_g, AddOp());
#pragma unroll
        for (int x = 0; x < W; ++x) o_g[x] = over_blocks<16>(o_g[x], AddOp());
    }
    if constexpr (L <= 32) {
        l_g = over_blocks<32>(l_g, AddOp());
#pragma unroll
        for (int x = 0; x < W; ++x) o_g[x] = over_blocks<32>(o_g[x], AddOp());
    }
    if (lane < L && active) {
#pragma unroll
        for (int x = 0; x < W; ++x) s_ow[wave][cc * W + x] = o_g[x];
    }
    if (lane == 0) { s_mw[wave] = m_w; s_lw[wave] = l_g; }
    __syncthreads();
    // the four waves' figures into the workgroup's (run_o: element tid, tid < d)
    static_assert(kAttnWaves == 4, "four waves' figures");
    const float run_m = fmaxf(fmaxf(s_mw[0], s_mw[1]), fmaxf(s_mw[2], s_mw[3]));   // finite: the workgroup has a row
    float f_w[kAttnWaves], run_l = 0.0f, run_o = 0.0f;
#pragma unroll
    for (int w = 0; w < kAttnWaves; ++w) {
        f_w[w] = s_mw[w] == -INFINITY ? 0.0f : expf(s_mw[w] - run_m);
        run_l += f_w[w] * s_lw[w];
    }
    if (tid < d) {
#pragma unroll
        for (int w = 0; w < kAttnWaves; ++w) run_o += f_w[w] * s_ow[w][tid];
    }

    // The head's workgroups are merged by whichever of them finishes last.  Nobody waits for anybody: every
    // workgroup DEPOSITS its figures with device-scope atomic exchanges (performed where every compute unit's atomics
    // meet, not in a cache of this die), then draws a ticket from the head's counter the same way; the one that draws
    // the last ticket reads all deposits with device-scope loads, merges, and puts the counter back to zero for the
    // next launch.  Data that crosses workgroups inside this launch travels through these operations only -- no cache
    // write-back or invalidation is involved (a device-wide fence here cost 8-35 us per layer).
    // What orders a deposit before the ticket: the exchange RETURNS a value, so it is counted as outstanding until
    // it has been performed; EVERY publishing wave waits for its own outstanding memory operations (vmcnt(0), below)
    // before the barrier, and the ticket is drawn after the barrier.  A workgroup barrier alone does not wait for
    // memory operations in flight, so the wait is explicit, and it is in every wave, not only in the one that draws.
    const int used = min(groups, last_chunk + 1);       // workgroups of this head that get this far
    const bool alone = used == 1;                       // uniform
    float* dst = scratch + ((int64_t)head * p.chunks + chunk) * (d + 2);
    unsigned int sink = 0;
    const auto publish = [&](float* at, float v) {
        sink ^= __hip_atomic_exchange(reinterpret_cast<unsigned int*>(at), __float_as_uint(v), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
    };
    if (alone) {
        if (tid < d) out[head * d + tid] = run_o / run_l;   // the only workgroup: nothing is deposited
    } else {
        if (tid < d) publish(dst + tid, run_o);
        if (tid == 0) {
            publish(dst + d, run_m);
            publish(dst + d + 1, run_l);
        }
    }
    if (alone) return;                                  // uniform
    __shared__ unsigned int s_ticket;
    // every lane consumes what its exchanges returned (so they stay returning atomics) and waits until none of this
    // wave's memory operations is outstanding
    asm volatile("s_waitcnt vmcnt(0)" ::"v"(sink) : "memory");
    __syncthreads();                                    // all deposits of this workgroup have been performed (and s_o, s_w read)
    // every workgroup of a launch draws a ticket: with the counters of all heads side by side in one or two memory lines those
    // updates queue up behind each other (32 heads of 128 at 2000 positions: 16.0 us, with the counters apart 14.0)
    unsigned int* counter = reinterpret_cast<unsigned int*>(
        p.counters_apart ? scratch + ((int64_t)head * p.chunks + p.chunks - 1) * (d + 2) : scratch + (int64_t)p.n_heads * p.chunks * (d + 2) + head);
    if (tid == 0) s_ticket = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (s_ticket != (unsigned)(used - 1)) return;       // uniform
    static_assert(sizeof(s_ow) >= kAttnThreads * sizeof(float), "the teams' sums go where the waves' figures were");
    if (used <= 16) attn_merge_together<MAXD, 16>(p, scratch, out, head, used, s_w, s_mw, &s_ow[0][0]);   // uniform
    else if (used <= kMergeTogether) attn_merge_together<MAXD, kMergeTogether>(p, scratch, out, head, used, s_w, s_mw, &s_ow[0][0]);
    else attn_merge(p, scratch, out, head, used, s_o, s_w);
    if (tid == 0) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int W, int MAXD>
__global__ __launch_bounds__(kAttnThreads, MAXD <= 128 ? 5 : 4) void attn_chunk_kernel(const AttnArgs p) {
    attn_walk<W, MAXD, false>(p);
}

// A kernel of its own: both kinds of loads in one, behind a uniform branch, cost a token's first positions 0.15 of 3.5 us.
template <int W>
__global__ __launch_bounds__(kAttnThreads, 4) void attn_chunk_prompt_kernel(const AttnArgs p) {
    attn_walk<W, BL_ATTN_MAX_HEAD_DIM, true>(p);
}

// A prompt's keys and values into the cache, ahead of its attention: one token per workgroup, the rotation and
// rounding of attn_chunk_kernel's own append.  A thread takes two neighbouring elements of a head's lower half and
// their partners in the upper half (head_dim is a multiple of 4), so that it loads 8 bytes and stores 4 at a time.
__global__ __launch_bounds__(256) void kv_append_kernel(const AttnArgs p) {
    const int token = blockIdx.x;
    const int d = p.head_dim, half = d / 2, quarter = half / 2, hidden = p.n_heads * d;
    const int pos = p.pos0 + token;
    if (pos < 0 || pos >= p.max_pos) return;
    const float* k_lin = p.k_lin + (int64_t)token * hidden;
    const float* v_lin = p.v_lin + (int64_t)token * hidden;
    uint32_t* krow = reinterpret_cast<uint32_t*>(p.k_cache + (int64_t)pos * hidden);
    uint32_t* vrow = reinterpret_cast<uint32_t*>(p.v_cache + (int64_t)pos * hidden);
    const float2* cs_row = p.rope + (int64_t)pos * half;
    const auto pack = [](float lo, float hi) { return (uint32_t)f32_to_bf16(lo) | ((uint32_t)f32_to_bf16(hi) << 16); };
    for (int i = threadIdx.x; i < p.n_heads * quarter; i += 256) {
        const int head = i / quarter, t = 2 * (i - head * quarter);
        const int lo = head * d + t, hi = lo + half;                    // even element indices
        const float2 ka = *reinterpret_cast<const float2*>(k_lin + lo), kb = *reinterpret_cast<const float2*>(k_lin + hi);
        const float2 va = *reinterpret_cast<const float2*>(v_lin + lo), vb = *reinterpret_cast<const float2*>(v_lin + hi);
        const float2 c0 = cs_row[t], c1 = cs_row[t + 1];
        krow[lo / 2] = pack(ka.x * c0.x - kb.x * c0.y, ka.y * c1.x - kb.y * c1.y);
        krow[hi / 2] = pack(ka.x * c0.y + kb.x * c0.x, ka.y * c1.y + kb.y * c1.x);
        vrow[lo / 2] = pack(va.x, va.y);
        vrow[hi / 2] = pack(vb.x, vb.y);
    }
}

// The same for head sizes that are a multiple of 8, sixteen bytes at a time and keys and values in workgroups of their own
// (blockIdx.y), so that a thread's loads are on their way together.  Bound by memory round trips: with the attention behind it, 32 heads of
// 128, before -> now (us): 512 tokens behind 512 31.5 -> 31.2, 2048 behind 2048 256 -> 250, 37 from 0 9.3 -> 8.8, 96 behind 100 11.4 -> 10.9.  Rows
// of fewer than kAppendWide elements do not fill two workgroups (12 heads of 64, 100 tokens behind 150 7.8 -> 8.1).
constexpr int kAppendWide = 1536;
__global__ __launch_bounds__(256) void kv_append_wide_kernel(const AttnArgs p) {
    typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));
    typedef uint32_t u32x2_u __attribute__((ext_vector_type(2), aligned(4)));
    typedef uint32_t u32x4_u __attribute__((ext_vector_type(4), aligned(4)));
    const int token = blockIdx.x;
    const int d = p.head_dim, half = d / 2, hidden = p.n_heads * d;
    const int pos = p.pos0 + token;
    if (pos < 0 || pos >= p.max_pos) return;
    const auto pack = [](float lo, float hi) { return (uint32_t)f32_to_bf16(lo) | ((uint32_t)f32_to_bf16(hi) << 16); };
    if (blockIdx.y == 0) {
        const float* k_lin = p.k_lin + (int64_t)token * hidden;
        uint16_t* krow = p.k_cache + (int64_t)pos * hidden;
        const float* cs_row = reinterpret_cast<const float*>(p.rope + (int64_t)pos * half);
        const int per_head = half / 4;
#pragma unroll 4
        for (int i = threadIdx.x; i < p.n_heads * per_head; i += 256) {
            const int head = i / per_head, t = 4 * (i - head * per_head);
            const int lo = head * d + t, hi = lo + half;
            const f32x4_u a = *reinterpret_cast<const f32x4_u*>(k_lin + lo), b = *reinterpret_cast<const f32x4_u*>(k_lin + hi);
            const f32x4_u c0 = *reinterpret_cast<const f32x4_u*>(cs_row + 2 * t), c1 = *reinterpret_cast<const f32x4_u*>(cs_row + 2 * t + 4);
            const float cx[4] = {c0[0], c0[2], c1[0], c1[2]}, cy[4] = {c0[1], c0[3], c1[1], c1[3]};
            float x[4], y[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                x[j] = a[j] * cx[j] - b[j] * cy[j];
                y[j] = a[j] * cy[j] + b[j] * cx[j];
            }
            *reinterpret_cast<u32x2_u*>(krow + lo) = u32x2_u{pack(x[0], x[1]), pack(x[2], x[3])};
            *reinterpret_cast<u32x2_u*>(krow + hi) = u32x2_u{pack(y[0], y[1]), pack(y[2], y[3])};
        }
    } else {
        const float* v_lin = p.v_lin + (int64_t)token * hidden;
        uint16_t* vrow = p.v_cache + (int64_t)pos * hidden;
#pragma unroll 4
        for (int i = threadIdx.x * 8; i < hidden; i += 256 * 8) {
            const f32x4_u a = *reinterpret_cast<const f32x4_u*>(v_lin + i), b = *reinterpret_cast<const f32x4_u*>(v_lin + i + 4);
            *reinterpret_cast<u32x4_u*>(vrow + i) = u32x4_u{pack(a[0], a[1]), pack(a[2], a[3]), pack(b[0], b[1]), pack(b[2], b[3])};
        }
    }
}

// A prompt's attention on the matrix cores for head sizes that are 4 more than a multiple of 8 (the others, up to 128, take
// the kernel of bl_attn_prompt.hip, whose 16-byte requests they do not fit): one workgroup per (head, block of 64 consecutive prompt tokens), 16 queries
// per wave.  The block walks the cache's 64-row chunks up to its last token's; per chunk a wave forms its 16 x 64
// scores S = Q K^T and then O += P V with 16x16x32 bf16 products, keeping the running maximum, sum and output of
// every query in registers (the usual rescaling by 2^(old maximum - new maximum); the scores carry log2(e), so the
// weights are plain powers of two).  Keys and values are bf16 in the cache already; the fp32 queries enter as the
// sum of three bf16 numbers (the value rounded, then the remainder, then its remainder: all 24 bits, since a score's
// error is multiplied by the scores' size) and the weights, which lie in [0, 1], as the sum of two (about 17 bits);
// each part takes one product, and everything is accumulated in fp32.  Operand layouts of the product, per lane: A
// holds row lane%16 and eight consecutive contraction indices chosen by lane/16, B holds column lane%16 and the same
// eight indices, the result holds rows 4*(lane/16) .. +3 of column lane%16.  The contraction index has to be the
// register-contiguous one on both sides: K rows serve as they are, V is transposed on its way into LDS, and the
// weights pass through LDS (each wave its own part) to turn from the result layout into the A layout.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kBlockQ = 64;          // queries per workgroup
constexpr int kBlockThreads = 256;   // four waves of 16 queries

// nearest-even bf16 of a finite float, by the hardware's conversion
__device__ __forceinline__ short bf16_bits(float v) { return __builtin_bit_cast(short, (__bf16)v); }
__device__ __forceinline__ float bf16_value(short b) { return __uint_as_float((uint32_t)(uint16_t)b << 16); }

__device__ __forceinline__ f32x4 mfma_bf16(const s16x8& a, const s16x8& b, const f32x4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// max / sum over the 16 lanes of a row of the wave, on the vector ALU's lane rotations; every lane gets the result
#define BL_ROW_ROR(x, n) __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, (x)), 0x120 + (n), 0xf, 0xf, false))
__device__ __forceinline__ float row16_max(float v) {
    v = fmaxf(v, BL_ROW_ROR(v, 8));
    v = fmaxf(v, BL_ROW_ROR(v, 4));
    v = fmaxf(v, BL_ROW_ROR(v, 2));
    return fmaxf(v, BL_ROW_ROR(v, 1));
}
__device__ __forceinline__ float row16_sum(float v) {
    v += BL_ROW_ROR(v, 8);
    v += BL_ROW_ROR(v, 4);
    v += BL_ROW_ROR(v, 2);
    return v + BL_ROW_ROR(v, 1);
}

template <int D16>   // head_dim rounded up to 16, in sixteens; the columns beyond head_dim are zero
__global__ __launch_bounds__(kBlockThreads) void attn_block_kernel(const AttnArgs p, const int M) {
    constexpr int D32 = (D16 + 1) / 2;   // steps of the scores' contraction over the head's elements
    constexpr int kKS = 32 * D32 + 8;    // bf16 elements per key row in LDS: 16 bytes of padding spread the rows over the banks
    constexpr int kVS = kChunk + 8;      // the same for a row of the transposed values
    constexpr int kPS = kChunk + 4;      // floats per row of weights
    __shared__ __align__(16) uint16_t s_k[kChunk * kKS];
    __shared__ __align__(16) uint16_t s_vt[16 * D16 * kVS];
    __shared__ __align__(16) float s_p[kBlockThreads / kWave][16][kPS];
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    // a later block walks more chunks: those are launched first
    const int head = blockIdx.x, block = (int)(gridDim.y - 1 - blockIdx.y);
    const int d = p.head_dim, half = d / 2, hidden = p.n_heads * d;
    const int l16 = lane % 16, g = lane / 16;
    const int m_last = min(block * kBlockQ + kBlockQ - 1, M - 1);      // the block's last token
    const int last_pos = p.pos0 + M - 1;                               // the last cached row

    // the padding beyond head_dim (key columns up to a multiple of 32, value rows up to a multiple of 16) must read as zero
    if (d != 32 * D32)
        for (int i = tid; i < kChunk * kKS / 2; i += kBlockThreads) reinterpret_cast<uint32_t*>(s_k)[i] = 0;
    if (d != 16 * D16)
        for (int i = tid; i < 16 * D16 * kVS / 2; i += kBlockThreads) reinterpret_cast<uint32_t*>(s_vt)[i] = 0;

    // the wave's queries, rotated, scaled by log2(e) / sqrt(head_dim), as A operands: row l16, elements 32 ks + 8 g .. + 7
    s16x8 q_hi[D32], q_mid[D32], q_lo[D32];
    {
        const int m = min(block * kBlockQ + wave * 16 + l16, M - 1);   // rows beyond the prompt repeat its last one
        const float* q = p.q_lin + (int64_t)m * hidden + head * d;
        const float2* cs_row = p.rope + (int64_t)(p.pos0 + m) * half;
        const float scale = 1.4426950408889634f / sqrtf((float)d);
#pragma unroll
        for (int ks = 0; ks < D32; ++ks) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                // element e of the rotated query: pairs (e, e + half); no branches, so that all loads go out together
                const int e = 32 * ks + 8 * g + j;
                const bool low = e < half, valid = e < d;
                const int ea = valid ? (low ? e : e - half) : 0;
                const float a = q[ea], b = q[ea + half];
                const float2 cs = cs_row[ea];
                float v = low ? a * cs.x - b * cs.y : a * cs.y + b * cs.x;
                v = valid ? v * scale : 0.0f;
                const short hi = bf16_bits(v);
                const float r1 = v - bf16_value(hi);
                const short mid = bf16_bits(r1);
                q_hi[ks][j] = hi; q_mid[ks][j] = mid; q_lo[ks][j] = bf16_bits(r1 - bf16_value(mid));
            }
        }
    }

    f32x4 o[D16];
#pragma unroll
    for (int t = 0; t < D16; ++t) o[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    float run_m[4], run_l[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) { run_m[i] = -INFINITY; run_l[i] = 0.0f; }
    const int q_wave0 = p.pos0 + block * kBlockQ + wave * 16;          // position of the wave's first query
    const int q_pos0 = q_wave0 + 4 * g;                                // position of result row 0 of this lane

    // A chunk's keys and values travel cache -> registers -> LDS in pieces of 4 rows x 4 elements (head_dim is a
    // multiple of 4), 8 x 8 pieces per wave and step: the values are transposed inside the piece, so that either matrix
    // is written as 8-byte words, two lanes to a bank at worst.  The next chunk's pieces are requested before this
    // one's products start, so that their way from memory is covered by the arithmetic.
    constexpr int kSteps = (2 * ((D16 + 1) / 2) + 3) / 4;   // wave steps: 2 row halves x ceil(elements / 32), over 4 waves
    const int c_count = d / 4, c_blocks = (c_count + 7) / 8;
    const int c_last = (p.pos0 + m_last) / kChunk;
    uint2 kreg[kSteps][4], vreg[kSteps][4];
    const auto piece = [&](int i, int& c, int& rg) {       // false: nothing to do in this step
        const int wt = wave + 4 * i;
        const int cb = wt % c_blocks, rb = wt / c_blocks;
        c = cb * 8 + lane % 8;
        rg = rb * 8 + lane / 8;
        return rb < 2 && c < c_count;
    };
    const auto request = [&](int chunk) {
        const int j0 = chunk * kChunk;
#pragma unroll
        for (int i = 0; i < kSteps; ++i) {
            int c, rg;
            if (piece(i, c, rg)) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int64_t at = (int64_t)min(j0 + 4 * rg + j, last_pos) * hidden + head * d + c * 4;
                    kreg[i][j] = *reinterpret_cast<const uint2*>(p.k_cache + at);
                    vreg[i][j] = *reinterpret_cast<const uint2*>(p.v_cache + at);
                }
            }
        }
    };
    request(0);
    for (int chunk = 0; chunk <= c_last; ++chunk) {
        const int j0 = chunk * kChunk;
        __syncthreads();                               // the previous chunk's tiles have been used (and the zero fill is done)
#pragma unroll
        for (int i = 0; i < kSteps; ++i) {
            int c, rg;
            if (piece(i, c, rg)) {
#pragma unroll
                for (int j = 0; j < 4; ++j) *reinterpret_cast<uint2*>(s_k + (4 * rg + j) * kKS + c * 4) = kreg[i][j];
                const uint2* v = vreg[i];
                uint2 t[4];
                t[0] = make_uint2((v[0].x & 0xffffu) | (v[1].x << 16), (v[2].x & 0xffffu) | (v[3].x << 16));
                t[1] = make_uint2((v[0].x >> 16) | (v[1].x & 0xffff0000u), (v[2].x >> 16) | (v[3].x & 0xffff0000u));
                t[2] = make_uint2((v[0].y & 0xffffu) | (v[1].y << 16), (v[2].y & 0xffffu) | (v[3].y << 16));
                t[3] = make_uint2((v[0].y >> 16) | (v[1].y & 0xffff0000u), (v[2].y >> 16) | (v[3].y & 0xffff0000u));
#pragma unroll
                for (int e = 0; e < 4; ++e) *reinterpret_cast<uint2*>(s_vt + (c * 4 + e) * kVS + 4 * rg) = t[e];
            }
        }
        if (chunk < c_last) request(chunk + 1);
        __syncthreads();

        // a wave whose queries all lie before this chunk has nothing to add (the block's last chunks; uniform per wave)
        if (j0 > q_wave0 + 15) continue;
        // scores of the wave's 16 queries against the chunk's 64 keys: four 16 x 16 tiles; consecutive products go to
        // different tiles, so that none waits for the one before it
        f32x4 sc[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) sc[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int ks = 0; ks < D32; ++ks) {
            s16x8 b[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) b[t] = *reinterpret_cast<const s16x8*>(s_k + (16 * t + l16) * kKS + 32 * ks + 8 * g);
#pragma unroll
            for (int t = 0; t < 4; ++t) sc[t] = mfma_bf16(q_lo[ks], b[t], sc[t]);
#pragma unroll
            for (int t = 0; t < 4; ++t) sc[t] = mfma_bf16(q_mid[ks], b[t], sc[t]);
#pragma unroll
            for (int t = 0; t < 4; ++t) sc[t] = mfma_bf16(q_hi[ks], b[t], sc[t]);
        }
        // a query sees the keys up to its own position (only the chunks around the wave's own positions need the
        // test); chunk 0 holds key 0, which every query sees, so the running maximum is finite from there on
        if (j0 + kChunk - 1 > q_wave0) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (j0 + 16 * t + l16 > q_pos0 + i) sc[t][i] = -INFINITY;
        }
        float f[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float mx = fmaxf(fmaxf(sc[0][i], sc[1][i]), fmaxf(sc[2][i], sc[3][i]));
            const float m_new = fmaxf(run_m[i], row16_max(mx));
            f[i] = __builtin_amdgcn_exp2f(run_m[i] - m_new);
            float sum = 0.0f;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float w = __builtin_amdgcn_exp2f(sc[t][i] - m_new);
                sum += w;
                s_p[wave][4 * g + i][16 * t + l16] = w;
            }
            run_l[i] = run_l[i] * f[i] + row16_sum(sum);
            run_m[i] = m_new;
        }
#pragma unroll
        for (int t = 0; t < D16; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) o[t][i] *= f[i];
        // the weights are read back by this wave only: LDS serves a wave's requests in their order
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const float4 w0 = *reinterpret_cast<const float4*>(&s_p[wave][l16][32 * ks + 8 * g]);
            const float4 w1 = *reinterpret_cast<const float4*>(&s_p[wave][l16][32 * ks + 8 * g + 4]);
            const float w[8] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w};
            s16x8 w_hi, w_lo;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                w_hi[j] = bf16_bits(w[j]);
                w_lo[j] = bf16_bits(w[j] - bf16_value(w_hi[j]));
            }
            s16x8 b[D16];
#pragma unroll
            for (int t = 0; t < D16; ++t) b[t] = *reinterpret_cast<const s16x8*>(s_vt + (16 * t + l16) * kVS + 32 * ks + 8 * g);
#pragma unroll
            for (int t = 0; t < D16; ++t) o[t] = mfma_bf16(w_lo, b[t], o[t]);
#pragma unroll
            for (int t = 0; t < D16; ++t) o[t] = mfma_bf16(w_hi, b[t], o[t]);
        }
    }

#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int m = block * kBlockQ + wave * 16 + 4 * g + i;
        if (m >= M) continue;
        float* out = p.out + (int64_t)m * hidden + head * d;
        const float inv = 1.0f / run_l[i];
#pragma unroll
        for (int t = 0; t < D16; ++t)
            if (16 * t + l16 < d) out[16 * t + l16] = o[t][i] * inv;
    }
}

template <int D16>
hipError_t launch_attn_block(const AttnArgs& p, int M, hipStream_t s) {
    const dim3 grid((unsigned)p.n_heads, (unsigned)((M + kBlockQ - 1) / kBlockQ));
    attn_block_kernel<D16><<<grid, dim3(kBlockThreads), 0, s>>>(p, M);
    return hipGetLastError();
}

__global__ void pos_advance_kernel(int32_t* pos) {
    if (threadIdx.x == 0) *pos = *pos + 1;
}

}  // namespace

int g_attn_groups = 0;                        // forced workgroups per head (0: automatic)

hipError_t launch_norm_quant(const bl_norm_quant_args& a, hipStream_t s) {
    NormArgs p;
    p.a = a.a_dev; p.b = a.b_dev; p.h = a.h_dev; p.gamma = a.gamma_dev;
    p.q = a.q_dev; p.a_scale = a.a_scale_dev; p.q_sum = a.q_sum_dev; p.y = a.y_dev;
    p.K = (int32_t)a.K; p.Kp = (int32_t)a.Kp; p.eps = a.eps;
    p.scratch = static_cast<float2*>(a.scratch_dev);
    p.h_out = a.h_dev; p.pos = nullptr; p.pos_set = 0;
    auto ok16 = [](const void* ptr) { return (reinterpret_cast<uintptr_t>(ptr) & 15) == 0; };
    const bool vec = a.K % 4 == 0 && ok16(a.a_dev) && ok16(a.b_dev) && ok16(a.h_dev) && ok16(a.gamma_dev) && ok16(a.y_dev);
    p.pieces = a.pieces;
    if (a.mode == BL_NORM_PREMULTIPLIED) return launch_norm_premultiplied(p, vec, s);
    if (a.scratch_dev && a.K >= kWideMinK && a.M <= 65535) {
        switch (a.mode) {
            case BL_NORM_PLAIN: return launch_norm_wide<BL_NORM_PLAIN>(p, a.M, vec, s);
            case BL_NORM_RESIDUAL: return launch_norm_wide<BL_NORM_RESIDUAL>(p, a.M, vec, s);
            case BL_NORM_GATED: return launch_norm_wide<BL_NORM_GATED>(p, a.M, vec, s);
        }
    }
    switch (a.mode) {
        case BL_NORM_PLAIN: return launch_norm_mode<BL_NORM_PLAIN>(p, a.M, vec, s);
        case BL_NORM_RESIDUAL: return launch_norm_mode<BL_NORM_RESIDUAL>(p, a.M, vec, s);
        case BL_NORM_GATED: return launch_norm_mode<BL_NORM_GATED>(p, a.M, vec, s);
    }
    return hipErrorInvalidValue;
}

// A token's last norm and the position's step in one launch: the position's own launch carried four bytes and took 0.8 us of a token's
// graph (7B shape, two layers: 88.7 -> 87.9 us), the host's fill of it behind a prompt 4 us.
hipError_t launch_final_norm(const bl_final_norm_args& a, hipStream_t s) {
    NormArgs p{};
    p.a = a.delta_dev; p.h = const_cast<float*>(a.h_dev); p.h_out = a.h_out_dev; p.gamma = a.gamma_dev; p.y = a.y_dev;
    p.K = (int32_t)a.K; p.eps = a.eps;
    p.pos = a.pos_dev; p.pos_set = a.pos_set;
    auto ok16 = [](const void* ptr) { return (reinterpret_cast<uintptr_t>(ptr) & 15) == 0; };
    const bool vec = a.K % 4 == 0 && ok16(a.h_dev) && ok16(a.delta_dev) && ok16(a.h_out_dev) && ok16(a.gamma_dev) && ok16(a.y_dev);
    return launch_norm_mode<BL_NORM_RESIDUAL>(p, a.M, vec, s);
}

hipError_t launch_rope_table(float* table, int head_dim, int max_pos, double theta, hipStream_t s) {
    const int half = head_dim / 2;
    const int64_t entries = (int64_t)max_pos * half;
    const int64_t blocks = (entries + 255) / 256;
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    rope_table_kernel<<<dim3((unsigned)blocks), dim3(256), 0, s>>>(reinterpret_cast<float2*>(table), half, entries, theta);
    return hipGetLastError();
}

int attn_chunks(int max_pos) { return (max_pos + kChunk - 1) / kChunk; }

static void launch_attn_chunks(const AttnArgs& p, const dim3& grid, hipStream_t s) {
    const dim3 block(kAttnThreads);
    if (p.head_dim % 8 == 0) {
        if (p.head_dim <= 128) attn_chunk_kernel<8, 128><<<grid, block, 0, s>>>(p);
        else attn_chunk_kernel<8, BL_ATTN_MAX_HEAD_DIM><<<grid, block, 0, s>>>(p);
    } else {
        if (p.head_dim <= 128) attn_chunk_kernel<4, 128><<<grid, block, 0, s>>>(p);
        else attn_chunk_kernel<4, BL_ATTN_MAX_HEAD_DIM><<<grid, block, 0, s>>>(p);
    }
}

// Workgroups per head of a call on a cache of so many chunks.  A cache of more chunks than that has pieces of scratch memory to
// spare: the last one of each head takes its counter, and no launch, however its workgroups are forced, deposits there.  (By the
// cache's size only: the same for every call on it.)
static int attn_groups(int n_heads, int head_dim, int chunks, int32_t& counters_apart) {
    const int most = attn_groups_per_head(n_heads, head_dim, chunks);
    counters_apart = chunks > most;
    return min(g_attn_groups > 0 ? g_attn_groups : most, counters_apart ? chunks - 1 : chunks);
}

hipError_t launch_attn_decode(const bl_attn_args& a, hipStream_t s) {
    AttnArgs p;
    p.q_lin = a.q_lin_dev; p.k_lin = a.k_lin_dev; p.v_lin = a.v_lin_dev; p.pos = a.pos_dev;
    p.rope = reinterpret_cast<const float2*>(a.rope_table_dev);
    p.k_cache = a.k_cache_dev; p.v_cache = a.v_cache_dev; p.out = a.out_dev;
    p.scratch = static_cast<float*>(a.scratch_dev);
    p.n_heads = a.n_heads; p.head_dim = a.head_dim; p.max_pos = a.max_pos; p.chunks = attn_chunks(a.max_pos);
    p.pos0 = 0; p.groups = 0; p.scratch_stride = 0;
    const int groups = attn_groups(a.n_heads, a.head_dim, p.chunks, p.counters_apart);
    const unsigned columns = attn_columns(a.n_heads, a.head_dim);
    const dim3 grid(columns, (unsigned)groups, (unsigned)a.n_heads / columns);
    launch_attn_chunks(p, grid, s);
    return hipGetLastError();
}

void set_attn_groups(int groups) { g_attn_groups = groups; }

int64_t attn_scratch_floats(int n_heads, int head_dim, int max_pos) {   // per query
    return (int64_t)n_heads * attn_chunks(max_pos) * (head_dim + 2) + n_heads;
}

hipError_t launch_attn_prefill(const bl_attn_prefill_args& a, hipStream_t s) {
    AttnArgs p;
    p.q_lin = a.q_lin_dev; p.k_lin = a.k_lin_dev; p.v_lin = a.v_lin_dev; p.pos = nullptr;
    p.rope = reinterpret_cast<const float2*>(a.rope_table_dev);
    p.k_cache = a.k_cache_dev; p.v_cache = a.v_cache_dev; p.out = a.out_dev;
    p.scratch = static_cast<float*>(a.scratch_dev);
    p.n_heads = a.n_heads; p.head_dim = a.head_dim; p.max_pos = a.max_pos;
    p.pos0 = a.pos0; p.groups = 0;
    // a prompt's queries never look beyond its last token: chunks up to that one only
    p.chunks = attn_chunks(a.pos0 + a.M);
    p.scratch_stride = attn_scratch_floats(a.n_heads, a.head_dim, a.pos0 + a.M);
    if (a.head_dim % 8 == 0 && a.n_heads * a.head_dim >= kAppendWide) kv_append_wide_kernel<<<dim3((unsigned)a.M, 2), dim3(256), 0, s>>>(p);
    else kv_append_kernel<<<dim3((unsigned)a.M), dim3(256), 0, s>>>(p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // head sizes up to 128 take a matrix-core kernel: the one of bl_attn_prompt.hip (32 tokens per workgroup) where a cache row's
    // head is whole 16-byte pieces, else the one of this file (64 tokens); larger ones go token by token
    if (attn_prompt_takes(a.n_heads, a.head_dim)) return launch_attn_prompt(a, s);
    static_assert(BL_ATTN_BLOCK_MAX_HEAD_DIM == 128, "the dispatch below covers head sizes up to 8 sixteens");
    switch ((a.head_dim + 15) / 16) {
        case 1: return launch_attn_block<1>(p, a.M, s);
        case 2: return launch_attn_block<2>(p, a.M, s);
        case 3: return launch_attn_block<3>(p, a.M, s);
        case 4: return launch_attn_block<4>(p, a.M, s);
        case 5: return launch_attn_block<5>(p, a.M, s);
        case 6: return launch_attn_block<6>(p, a.M, s);
        case 7: return launch_attn_block<7>(p, a.M, s);
        case 8: return launch_attn_block<8>(p, a.M, s);
        default: break;
    }
    // the workgroups that bl_attn_decode takes on this cache: the same sums in the same order, token by token.  They may use every
    // piece of a token's scratch memory (its chunks end at pos0 + M, not at max_pos), so the counters lie behind the pieces.
    p.groups = min(attn_groups(a.n_heads, a.head_dim, attn_chunks(a.max_pos), p.counters_apart), p.chunks);
    p.counters_apart = 0;
    const dim3 grid(attn_prompt_units(a.n_heads, p.groups), 1, (unsigned)a.M);
    if (p.head_dim % 8 == 0) attn_chunk_prompt_kernel<8><<<grid, dim3(kAttnThreads), 0, s>>>(p);   // (head sizes above 128)
    else attn_chunk_prompt_kernel<4><<<grid, dim3(kAttnThreads), 0, s>>>(p);
    return hipGetLastError();
}

hipError_t launch_pos_advance(int32_t* pos, hipStream_t s) {
    pos_advance_kernel<<<dim3(1), dim3(64), 0, s>>>(pos);
    return hipGetLastError();
}

}  // namespace bl
