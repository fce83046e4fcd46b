// bl_quant_act: per-token absmax quantization of activations to int8 (the BitNet b1.58
// activation quantizer that the ternary kernels of arXiv 2410.16144 consume).
//
// One workgroup per token row; one launch takes up to 8 activation matrices (bl_quant_act_batch).
// Pass 1 reduces max|x| over the row (lane moves, then LDS across waves); pass 2 multiplies by
// inv = 127/amax, rounds to nearest-even, clips, stores int8 and reduces sum(q).  The int8 result
// must be bit-identical to the plain definition, so every fp32 operation is a single IEEE
// operation.
#include "bl_quant_device.hpp"

namespace bl {

namespace {

constexpr int kQuantThreads = 256;

// A launch whose rows are all no longer than this and no whole aligned vectors goes element by element, in a kernel instance of
// its own: in vectors most threads would idle and one fetch its tail apart, and that code beside the other, not even
// executed, costs (by elements alone / in vectors, us: 7167 bf16 rows of 6 7.6 / 10.3, 16 rows of 100 2.6 / 3.0, 349 of 464 3.2 / 3.2,
// 434 of 976 3.6 / 3.2; 7702 fp32 rows of 320 by elements in the one kernel 9.9, in its own 9.3).
constexpr int kElementRow = 512;

constexpr int kRegVectors = 6;   // 8-element vectors a thread keeps in registers: rows up to 256 * 8 * 6 = 12288 elements

// The row's inv and scale from the threads' maxima.
__device__ __forceinline__ void row_scales(float amax, float* s_max, float& inv, float& scale) {
    const int tid = threadIdx.x;
    amax = wave_max(amax);
    if ((tid & (kWave - 1)) == 0) s_max[tid / kWave] = amax;
    __syncthreads();
    amax = s_max[0];
#pragma unroll
    for (int w = 1; w < kQuantThreads / kWave; ++w) amax = fmaxf(amax, s_max[w]);

    quant_scales(amax, inv, scale);
}

// The row's figures from the threads' sums.
__device__ __forceinline__ void finish_row(int sum, float scale, float* a_scale, int32_t* q_sum, int* s_sum) {
    const int tid = threadIdx.x;
    sum = wave_sum(sum);
    if ((tid & (kWave - 1)) == 0) s_sum[tid / kWave] = sum;
    __syncthreads();
    if (tid == 0) {
        int total = 0;
#pragma unroll
        for (int w = 0; w < kQuantThreads / kWave; ++w) total += s_sum[w];
        *a_scale = scale;
        if (q_sum) *q_sum = total;
    }
}

// A short row that is not whole aligned vectors.
template <bool BF16>
__device__ __forceinline__ void quant_row_by_element(const void* row, int K, int Kp, int8_t* qrow, float* a_scale, int32_t* q_sum,
                                                     float* s_max, int* s_sum) {
    float inv, scale;
    row_scales(element_absmax<BF16>(row, K, threadIdx.x, kQuantThreads), s_max, inv, scale);
    finish_row(element_quantize<BF16>(row, K, Kp, inv, qrow, threadIdx.x, kQuantThreads), scale, a_scale, q_sum, s_sum);
}

// One token row by one workgroup.  Rows of up to 12288 elements are read ONCE: all of a thread's loads are issued together and
// the raw values stay in registers between the absmax pass and the rounding pass.  Longer rows are read twice (the second
// read hits L2).  VEC: the row is 16-byte aligned and a multiple of 8 long; otherwise the same vectors are loaded at any address
// and one thread picks up the last few elements (512 rows of 12036 fp32 read element by element: 27 us).
// NV: vectors a thread keeps (a short row asked to load six per thread, five of them nothing but its first elements again,
// took 8.7 us instead of 5.4 for 2048 unaligned bf16 rows of 771).
template <bool BF16, bool VEC, int NV>
__device__ __forceinline__ void quant_row(const void* row, int K, int Kp, int8_t* qrow, float* a_scale, int32_t* q_sum,
                                          float* s_max, int* s_sum) {
    const int tid = threadIdx.x;
    const bool in_regs = K >= 8 && K <= kQuantThreads * 8 * NV;   // uniform
    Raw8<BF16> raw[NV];
    float amax = 0.0f;
    if (in_regs) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int k = (tid + i * kQuantThreads) * 8, at = k + 8 <= K ? k : 0;
            raw[i] = VEC ? load_raw8<BF16>(row, at) : load_raw8_any<BF16>(row, at);
        }
        if constexpr (!VEC) {
            const int k = K & ~7;   // the last few elements, if any: one thread's, in one of its vectors
            if (k < K && tid == (k / 8) % kQuantThreads) {
                const Raw8<BF16> tail = load_raw8_tail<BF16>(row, k, K);
#pragma unroll
                for (int i = 0; i < NV; ++i)
                    if (i == (k / 8) / kQuantThreads) raw[i] = tail;
            }
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            float v[8];
            unpack_raw8<BF16>(raw[i], v);
            if ((tid + i * kQuantThreads) * 8 < K) amax = fmaxf(amax, absmax8(v));
        }
    } else {
        amax = thread_absmax<BF16, VEC>(row, K, tid, kQuantThreads);
    }
    float inv, scale;
    row_scales(amax, s_max, inv, scale);

    int sum = 0;
    if (in_regs) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int k = (tid + i * kQuantThreads) * 8;
            float v[8];
            unpack_raw8<BF16>(raw[i], v);
            if (k < K) sum += quantize8(v, inv, qrow + k);
        }
        for (int k = (K + 7) / 8 * 8 + tid * 8; k < Kp; k += kQuantThreads * 8) *reinterpret_cast<uint2*>(qrow + k) = make_uint2(0, 0);   // layout padding
    } else {
        sum = thread_quantize<BF16, VEC>(row, K, Kp, inv, qrow, tid, kQuantThreads);
    }
    finish_row(sum, scale, a_scale, q_sum, s_sum);
}

// The instance by the row's length: a branch inside the one kernel, all of whose rows run with the registers of the longest.
template <bool BF16, bool VEC>
__device__ __forceinline__ void quant_row(const void* row, int K, int Kp, int8_t* qrow, float* a_scale, int32_t* q_sum,
                                          float* s_max, int* s_sum) {
    if (K <= kQuantThreads * 8) quant_row<BF16, VEC, 1>(row, K, Kp, qrow, a_scale, q_sum, s_max, s_sum);             // uniform
    else if (K <= 2 * kQuantThreads * 8) quant_row<BF16, VEC, 2>(row, K, Kp, qrow, a_scale, q_sum, s_max, s_sum);
    else quant_row<BF16, VEC, kRegVectors>(row, K, Kp, qrow, a_scale, q_sum, s_max, s_sum);
}

// Up to BL_MAX_BATCH activation matrices in one launch: workgroup = one token row of one of them.
template <bool BY_ELEMENT>
__global__ __launch_bounds__(kQuantThreads) void quant_kernel(BL_FIRST_WG_PARAMS, const QuantBatch b) {
    __shared__ float s_max[kQuantThreads / kWave];
    __shared__ int s_sum[kQuantThreads / kWave];
    const int blk = blockIdx.x;
    const QuantProblem& p = b.p[BL_PROBLEM_OF(blk)];
    const int64_t m = blk - p.first_row;
    const bool bf16 = p.flags & 1, vec = p.flags & 2;   // uniform
    const void* row = static_cast<const char*>(p.x) + m * p.ldx * (bf16 ? 2 : 4);
    int8_t* qrow = p.q + m * p.Kp;
    float* a_scale = p.a_scale + m;
    int32_t* q_sum = p.q_sum ? p.q_sum + m : nullptr;
    if constexpr (BY_ELEMENT) {
        if (bf16) quant_row_by_element<true>(row, p.K, p.Kp, qrow, a_scale, q_sum, s_max, s_sum);
        else quant_row_by_element<false>(row, p.K, p.Kp, qrow, a_scale, q_sum, s_max, s_sum);
    } else if (bf16) {
        if (vec) quant_row<true, true>(row, p.K, p.Kp, qrow, a_scale, q_sum, s_max, s_sum);
        else quant_row<true, false>(row, p.K, p.Kp, qrow, a_scale, q_sum, s_max, s_sum);
    } else {
        if (vec) quant_row<false, true>(row, p.K, p.Kp, qrow, a_scale, q_sum, s_max, s_sum);
        else quant_row<false, false>(row, p.K, p.Kp, qrow, a_scale, q_sum, s_max, s_sum);
    }
}

}  // namespace

hipError_t launch_quant(const QuantBatch& batch, hipStream_t s) {
    QuantBatch b = batch;
    int64_t rows = 0;
    bool by_element = true;
    for (int i = 0; i < b.count; ++i) {
        b.p[i].first_row = (int32_t)rows;
        rows += b.p[i].M;
        by_element = by_element && !(b.p[i].flags & 2) && b.p[i].K <= kElementRow;
    }
    if (rows > INT32_MAX) return hipErrorInvalidValue;
    struct { int v[BL_MAX_BATCH]; } first;
    for (int i = 0; i < BL_MAX_BATCH; ++i) first.v[i] = i < b.count ? b.p[i].first_row : INT32_MAX;
    if (by_element) quant_kernel<true><<<dim3((unsigned)rows), dim3(kQuantThreads), 0, s>>>(BL_FIRST_WG_ARGS(first), b);
    else quant_kernel<false><<<dim3((unsigned)rows), dim3(kQuantThreads), 0, s>>>(BL_FIRST_WG_ARGS(first), b);
    return hipGetLastError();
}

}  // namespace bl
