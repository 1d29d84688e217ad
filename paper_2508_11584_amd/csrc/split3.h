// fp32 products on the bf16 matrix instructions (GEMMs and attention of fp32 engines).
#pragma once
#include "common.h"

namespace vpe {

// A value is the sum of three bf16 terms, each the rounded rest of the
// one before (8 + 8 + 8 significant bits; the rests are exact), and six of the nine products of the terms are taken: the
// three left out are at most 2^-27 of the product.  The instruction multiplies exactly and accumulates in fp32, so what
// remains is the rounding of the accumulation, once per 16 k elements and product where v_mfma_f32_32x32x2_f32 rounds
// once per 2.  Six bf16 instructions take 192 clocks for a 32 x 32 x 16 block, eight of the fp32 ones 512.
// An infinite operand, or a finite one above 3.396e38 (it rounds to infinity in bf16), has NaN among its terms and makes every
// sum that it enters NaN: users look for infinite and NaN sums and compute those again on the fp32 instructions.  Terms
// below 1e-38 may be lost, so operands smaller than about 1e-33 keep fewer bits (the absolute error stays below 1e-38).
struct Split3 { bf16x8 t[3]; };
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ Split3 split3(const f32x4& lo, const f32x4& hi) {
    // the rest x - term of the lower / upper element of a pair in one instruction, v_dot2c_f32_bf16: (term0, term1) . (-1, 0) + x
    // (the constants are kept in registers: as an inline constant -1.0 stands for the upper element)
    uint32_t c0 = 0x0000BF80u, c1 = 0xBF800000u;
    asm("" : "+s"(c0), "+s"(c1));
    const bf16x2 m0 = __builtin_bit_cast(bf16x2, c0), m1 = __builtin_bit_cast(bf16x2, c1);
    Split3 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float x0 = e < 2 ? lo[2 * e] : hi[2 * e - 4], x1 = e < 2 ? lo[2 * e + 1] : hi[2 * e - 3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const bf16x2 p = {(bf16)x0, (bf16)x1};
            r.t[k][2 * e] = p[0];
            r.t[k][2 * e + 1] = p[1];
            if (k < 2) {
                x0 = __builtin_amdgcn_fdot2_f32_bf16(p, m0, x0, false);
                x1 = __builtin_amdgcn_fdot2_f32_bf16(p, m1, x1, false);
            }
        }
    }
    return r;
}
// Product t of six (small ones first) of two split operands.
__device__ __forceinline__ f32x16 split_mma(int t, const Split3& a, const Split3& b, f32x16 c) {
    const int ia = t == 0 ? 2 : t == 1 ? 0 : t == 2 ? 1 : t == 3 ? 1 : 0, ib = t == 0 ? 0 : t == 1 ? 2 : t == 2 ? 1 : t == 3 ? 0 : t == 4 ? 1 : 0;
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.t[ia], b.t[ib], c, 0, 0, 0);
}

}  // namespace vpe
