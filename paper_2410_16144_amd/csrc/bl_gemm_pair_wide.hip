// The paired-tile kernel's forms for launches of one workgroup per compute unit (the template and its account: bl_gemm_pair.hpp,
// bl_gemm_pair.hip): 64 tokens x 384 weight rows and 128 x 256, four waves, one per SIMD, four stages.
//
// Nothing but the wave itself covers its waits there: a request has two steps until its pair is published (with three stages one,
// less than a weight from memory takes under load), a step is 24 or 32 products per wave, and everything else stands between them.  A
// token operand read serves two or three products and, with 128 tokens, a weight operand four: half the expansions per product of the
// 64-token tiles, which counts because the chip's power sets the clock (2048 x 11008 -> 4096: matrix cores busy in 75 to 85 % of the cycles
// at 1.75 to 1.9 GHz; all tokens zero 2.35 GHz and 50 us).
//
// Measured, what was taken before -> these (us, weights cold): 2048 x 11008 -> 4096 70.2 (64 x 256) -> 63.9; 512 x 4096 -> 11008 24.6 (64 x 256 and
// 64 x 128 tiles in one launch) -> 22.4, but 21.2 -> 22.2 with warm weights: the choice takes them where they are ahead either way.  Tried and left: 128 x 256 with three stages and two workgroups per
// unit (within 1 % of the forms there are), with five stages (68.5), 64 x 384 with five (1 to 3 % behind four); and v_mfma_i32_16x16x64_i8 with
// the weights as its first operand, which takes less power for the same products (register-only loop 4.76 POP/s against 4.30 of
// v_mfma_i32_32x32x32_i8) but is 16 cycles long, so that what stands between the products no longer fits under them: 2048 x 11008 -> 4096 65.0
// where this kernel takes 63.9, with all tokens zero 61 and 50.
#include "bl_gemm_pair.hpp"

namespace bl {

hipError_t launch_gemm_pair_wide(const GemmProblem* ps, int count, int64_t M, int code, int halves, hipStream_t s) {
#define X(MB, H, WN, WK, S) if (code == pair_code(MB, H, WK, S)) return launch_pair_form<MB, H, WN, WK, S>(ps, count, M, halves, s);
    BL_PAIR_WIDE_FORMS(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace bl
