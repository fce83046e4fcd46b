// Device-side pieces of the per-token absmax int8 quantizer, shared by the stand-alone
// bl_quant_act kernel and by the fused decode kernel.  Every fp32 operation here is a single
// IEEE round-to-nearest operation (translation units are compiled with -ffp-contract=off).
#pragma once
#include "bl_internal.hpp"

namespace bl {

__device__ __forceinline__ float bf16_to_f32(uint32_t h) { return __uint_as_float(h << 16); }

// Wave-wide reductions on the vector ALU's data-parallel-primitive lane moves (no LDS round trips):
// four steps reduce each row of 16 lanes, four v_readlane pick up the rows.  The result is uniform.
#define BL_DPP(x, ctrl) __builtin_amdgcn_update_dpp(0, (x), (ctrl), 0xf, 0xf, false)
__device__ __forceinline__ float wave_max(float v) {   // v >= 0: compare the bit patterns as integers
    int x = __float_as_int(v);
    x = max(x, BL_DPP(x, 0xB1));    // quad_perm [1,0,3,2]
    x = max(x, BL_DPP(x, 0x4E));    // quad_perm [2,3,0,1]
    x = max(x, BL_DPP(x, 0x141));   // row_half_mirror
    x = max(x, BL_DPP(x, 0x140));   // row_mirror
    const int a = __builtin_amdgcn_readlane(x, 0), b = __builtin_amdgcn_readlane(x, 16);
    const int c = __builtin_amdgcn_readlane(x, 32), d = __builtin_amdgcn_readlane(x, 48);
    return __int_as_float(max(max(a, b), max(c, d)));
}

__device__ __forceinline__ int wave_sum(int x) {
    x += BL_DPP(x, 0xB1);
    x += BL_DPP(x, 0x4E);
    x += BL_DPP(x, 0x141);
    x += BL_DPP(x, 0x140);
    return __builtin_amdgcn_readlane(x, 0) + __builtin_amdgcn_readlane(x, 16) + __builtin_amdgcn_readlane(x, 32) +
           __builtin_amdgcn_readlane(x, 48);
}

__device__ __forceinline__ float wave_sum_f(float v) {   // a fixed tree: the same bits on every run
#define BL_DPP_F(x, ctrl) __int_as_float(BL_DPP(__float_as_int(x), (ctrl)))
    v += BL_DPP_F(v, 0xB1);
    v += BL_DPP_F(v, 0x4E);
    v += BL_DPP_F(v, 0x141);
    v += BL_DPP_F(v, 0x140);
#undef BL_DPP_F
    const int x = __float_as_int(v);
    return (__int_as_float(__builtin_amdgcn_readlane(x, 0)) + __int_as_float(__builtin_amdgcn_readlane(x, 16))) +
           (__int_as_float(__builtin_amdgcn_readlane(x, 32)) + __int_as_float(__builtin_amdgcn_readlane(x, 48)));
}
#undef BL_DPP

__device__ __forceinline__ float silu(float t) { return t / (1.0f + expf(-t)); }

// silu of four values.  Where all of the wave's are below 80 in size nothing overflows or leaves the normal range, and the
// exponential and the quotient need no special cases: exp(-t) = 2^n 2^((h - n) + l) by Cody and Waite's reduction in two
// terms (h + l = -t log2(e) to twice the precision, n = h rounded), the quotient by the reciprocal and one correction step.
// 14 instructions instead of about 26.  Against silu(): the same bits on 33 million normal values of deviation 0.1 to 15, 3 of
// 8.4 million uniform ones in +-80 differ; the error against 64 bits is the same in all of these sets
// (rms 2.9e-8 to 4.3e-8, at most 2.7 last places).  Any other wave takes silu().
__device__ __forceinline__ void silu4(const float (&t)[4], float (&y)[4]) {
    const float size = fmaxf(fmaxf(fabsf(t[0]), fabsf(t[1])), fmaxf(fabsf(t[2]), fabsf(t[3])));
    if (__any(!(size < 80.0f))) {   // uniform
#pragma unroll
        for (int j = 0; j < 4; ++j) y[j] = silu(t[j]);
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            constexpr float kLog2e = 0x1.715476p+0f, kLog2eRest = 0x1.4ae0cp-26f;
            const float h = -t[j] * kLog2e;
            const float l = __builtin_fmaf(-t[j], kLog2eRest, __builtin_fmaf(-t[j], kLog2e, -h)), n = rintf(h);
            const float d = 1.0f + __builtin_amdgcn_ldexpf(__builtin_amdgcn_exp2f((h - n) + l), (int)n);
            const float r = __builtin_amdgcn_rcpf(d), q = t[j] * r;
            y[j] = __builtin_fmaf(__builtin_fmaf(-d, q, t[j]), r, q);
        }
    }
}

// inv = 127/amax and scale = amax/127 (one IEEE division each); a row whose inv is not finite
// (amax zero or tiny) is an all-zero token: inv = 0 makes every product +-0, scale = 0.
__device__ __forceinline__ void quant_scales(float amax, float& inv, float& scale) {
    inv = 127.0f / amax;
    const bool zero_row = !(fabsf(inv) <= 3.402823466e+38f);
    if (zero_row) inv = 0.0f;
    scale = zero_row ? 0.0f : amax / 127.0f;
}

// 8 consecutive elements starting at element k (k % 8 == 0, row base 16-byte aligned).
template <bool BF16>
__device__ __forceinline__ void load8(const void* row, int k, float (&v)[8]) {
    if constexpr (BF16) {
        uint4 u = *reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(row) + k);
        uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[2 * i] = bf16_to_f32(w[i] & 0xffffu);
            v[2 * i + 1] = bf16_to_f32(w[i] >> 16);
        }
    } else {
        const float4* p = reinterpret_cast<const float4*>(static_cast<const float*>(row) + k);
        float4 a = p[0], b = p[1];
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    }
}

// The same 8 elements as raw bits (kept in registers between the absmax and the quantize pass).
template <bool BF16>
struct Raw8 {
    uint4 a, b;   // bf16: a only; fp32: a, b
};

template <bool BF16>
__device__ __forceinline__ Raw8<BF16> load_raw8(const void* row, int k) {
    Raw8<BF16> r;
    if constexpr (BF16) {
        r.a = *reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(row) + k);
        r.b = r.a;
    } else {
        const uint4* p = reinterpret_cast<const uint4*>(static_cast<const float*>(row) + k);
        r.a = p[0];
        r.b = p[1];
    }
    return r;
}

// The same from any element's address (the memory system takes vectors at any alignment; only their lines may be two).
template <bool BF16>
__device__ __forceinline__ Raw8<BF16> load_raw8_any(const void* row, int k) {
    typedef uint32_t u32x4_2 __attribute__((ext_vector_type(4), aligned(2)));
    typedef uint32_t u32x4_4 __attribute__((ext_vector_type(4), aligned(4)));
    Raw8<BF16> r;
    if constexpr (BF16) {
        const u32x4_2 t = *reinterpret_cast<const u32x4_2*>(static_cast<const uint16_t*>(row) + k);
        r.a = make_uint4(t[0], t[1], t[2], t[3]);
        r.b = r.a;
    } else {
        const u32x4_4* p = reinterpret_cast<const u32x4_4*>(static_cast<const float*>(row) + k);
        const u32x4_4 t = p[0], u = p[1];
        r.a = make_uint4(t[0], t[1], t[2], t[3]);
        r.b = make_uint4(u[0], u[1], u[2], u[3]);
    }
    return r;
}

// The last K - k < 8 elements of a row, zeros behind them.
template <bool BF16>
__device__ __forceinline__ Raw8<BF16> load_raw8_tail(const void* row, int k, int K) {
    uint32_t e[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {   // no branches: the loads go out together
        const int at = min(k + j, K - 1);
        if constexpr (BF16) e[j] = static_cast<const uint16_t*>(row)[at];
        else e[j] = static_cast<const uint32_t*>(row)[at];
    }
    uint32_t w[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const uint32_t v = k + j < K ? e[j] : 0;
        if constexpr (BF16) w[j / 2] |= v << (16 * (j & 1));
        else w[j] = v;
    }
    Raw8<BF16> r;
    r.a = make_uint4(w[0], w[1], w[2], w[3]);
    r.b = BF16 ? r.a : make_uint4(w[4], w[5], w[6], w[7]);
    return r;
}

template <bool BF16>
__device__ __forceinline__ void unpack_raw8(const Raw8<BF16>& r, float (&v)[8]) {
    if constexpr (BF16) {
        const uint32_t w[4] = {r.a.x, r.a.y, r.a.z, r.a.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[2 * i] = bf16_to_f32(w[i] & 0xffffu);
            v[2 * i + 1] = bf16_to_f32(w[i] >> 16);
        }
    } else {
        const uint32_t w[8] = {r.a.x, r.a.y, r.a.z, r.a.w, r.b.x, r.b.y, r.b.z, r.b.w};
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = __uint_as_float(w[i]);
    }
}

__device__ __forceinline__ float absmax8(const float (&v)[8]) {
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) m = fmaxf(m, fabsf(v[i]));
    return m;
}

// Four codes q = clip(round_half_even(v * inv), -128, 127) as the bytes of a word, v0's lowest; their sum is added to `sum`.
// The product is clipped before it is rounded (the limits are whole numbers, so the order does not matter), and adding
// 1.5 * 2^23 rounds to nearest, ties to even, leaving the integer in the low bits.  4 vector instructions per code instead of
// the 9 of rounding, clipping and packing one by one -- the quantizer's second pass is bound by the vector ALU.
__device__ __forceinline__ uint32_t code_bits(float v, float inv) {   // the code is the lowest byte
    return __float_as_uint(__builtin_amdgcn_fmed3f(v * inv, -128.0f, 127.0f) + 12582912.0f);
}
__device__ __forceinline__ uint32_t quantize4(float v0, float v1, float v2, float v3, float inv, int& sum) {
    const uint32_t low = __builtin_amdgcn_perm(code_bits(v1, inv), code_bits(v0, inv), 0x0c0c0400u);    // bytes 0 and 1
    const uint32_t high = __builtin_amdgcn_perm(code_bits(v3, inv), code_bits(v2, inv), 0x04000c0cu);   // bytes 2 and 3
    const uint32_t word = low | high;
    sum = __builtin_amdgcn_sdot4((int)word, 0x01010101, sum, false);
    return word;
}

// Quantize 8 values to 8 bytes; returns their sum.
__device__ __forceinline__ int quantize8_packed(const float (&v)[8], float inv, uint32_t& lo, uint32_t& hi) {
    int sum = 0;
    lo = quantize4(v[0], v[1], v[2], v[3], inv, sum);
    hi = quantize4(v[4], v[5], v[6], v[7], inv, sum);
    return sum;
}

// The same, stored at q8.
__device__ __forceinline__ int quantize8(const float (&v)[8], float inv, int8_t* q8) {
    uint32_t lo, hi;
    const int sum = quantize8_packed(v, inv, lo, hi);
    *reinterpret_cast<uint2*>(q8) = make_uint2(lo, hi);
    return sum;
}

// VEC: the row is 16-byte aligned and a multiple of 8 long; otherwise vectors at any address and a tail of up to 7 elements,
// which falls to the thread whose turn it is.
template <bool BF16, bool VEC, typename Fn>
__device__ __forceinline__ void for_thread_vectors(const void* row, int K, int tid, int nthreads, Fn fn) {
    const int full = VEC ? K : K & ~7;
    for (int k = tid * 8; k < full; k += nthreads * 8) {
        float v[8];
        unpack_raw8<BF16>(VEC ? load_raw8<BF16>(row, k) : load_raw8_any<BF16>(row, k), v);
        fn(k, v);
    }
    if (!VEC && full < K && tid == (full / 8) % nthreads) {
        float v[8];
        unpack_raw8<BF16>(load_raw8_tail<BF16>(row, full, K), v);
        fn(full, v);
    }
}

// max |x| over this thread's share of a row (threads stride the row).  K <= BL_MAX_K: 32-bit indices.
template <bool BF16, bool VEC>
__device__ __forceinline__ float thread_absmax(const void* row, int K, int tid, int nthreads) {
    float amax = 0.0f;
    for_thread_vectors<BF16, VEC>(row, K, tid, nthreads, [&](int, const float (&v)[8]) { amax = fmaxf(amax, absmax8(v)); });
    return amax;
}

// Quantize this thread's share of a row into qrow (global or LDS, 8-byte aligned, Kp a multiple of 64); returns the
// thread's sum(q).
template <bool BF16, bool VEC>
__device__ __forceinline__ int thread_quantize(const void* row, int K, int Kp, float inv, int8_t* qrow,
                                               int tid, int nthreads) {
    int sum = 0;
    for_thread_vectors<BF16, VEC>(row, K, tid, nthreads, [&](int k, const float (&v)[8]) { sum += quantize8(v, inv, qrow + k); });
    for (int k = (K + 7) / 8 * 8 + tid * 8; k < Kp; k += nthreads * 8) *reinterpret_cast<uint2*>(qrow + k) = make_uint2(0, 0);  // layout padding
    return sum;
}

// The same two, element by element: short rows of bl_quant_act, and rows of the fused decode kernels that are no whole aligned
// vectors -- there the vector form's code alone, executed or not, cost every such launch a tenth (1 token, K = 28: 3.6 -> 4.0 us;
// 8 tokens, K = 2147: 12.0 -> 14.8).
template <bool BF16>
__device__ __forceinline__ float load1(const void* row, int k) {
    if constexpr (BF16) return bf16_to_f32(static_cast<const uint16_t*>(row)[k]);
    else return static_cast<const float*>(row)[k];
}
template <bool BF16>
__device__ __forceinline__ float element_absmax(const void* row, int K, int tid, int nthreads) {
    float amax = 0.0f;
    for (int k = tid; k < K; k += nthreads) amax = fmaxf(amax, fabsf(load1<BF16>(row, k)));
    return amax;
}
template <bool BF16>
__device__ __forceinline__ int element_quantize(const void* row, int K, int Kp, float inv, int8_t* qrow, int tid, int nthreads) {
    int sum = 0;
    for (int k = tid; k < K; k += nthreads) {
        const int8_t code = (int8_t)code_bits(load1<BF16>(row, k), inv);
        sum += code;
        qrow[k] = code;
    }
    for (int k = K + tid; k < Kp; k += nthreads) qrow[k] = 0;   // layout padding
    return sum;
}

}  // namespace bl
