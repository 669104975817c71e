// fp32 values as exact sums of three bf16 values: what the kernels on bf16 pieces share (sconv_piece.hip says what the pieces are for).
#pragma once
#include <hip/hip_runtime.h>

namespace sconv {
namespace {

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef unsigned u4 __attribute__((ext_vector_type(4)));

constexpr float kUp = 0x1p24f, kDown = 0x1p-48f;   // scale of an operand before it is cut; of a sum, afterwards

// Two fp32 values times up as three bf16 pieces each: v = p0 + p1 + p2 exactly (24 bits = 3 x 8, every remainder is exact) for all
// values below 2^104 at up = 2^24.
// DOT: a remainder is one dot product with (-1, 0) or (0, -1) where taking the piece apart and subtracting are two instructions, 9 for a pair of
// values instead of 13; the same bits.  Where the compiler places the cuts and three wavefronts a SIMD fill the waits of its two-address form, that is
// ahead (filters as stored: 896 channels in 7 groups @14x14 at batch 32 89.8 -> 87.8 us); between fenced matrix instructions it is not (128 @56x56
// stride 2 48.8 -> 50.3, 5x5 48 -> 128 @7x7 12.55 -> 12.74), nor at two wavefronts a SIMD (92 -> 100).  A piece that is Inf makes the other value's
// remainders NaN as well: their sums, over the same windows or the same filter, are NaN as they are, and are summed again.  The constants
// come from registers: as an inline operand -1.0 stands in the upper half whatever was written.
template <bool DOT = false>
__device__ __forceinline__ void split2(float a, float b, float up_a, float up_b, int i, u4 (&out)[3])
{
    unsigned of_lo = 0x0000bf80u, of_hi = 0xbf800000u;
    if (DOT) asm("" : "+s"(of_lo), "+s"(of_hi));
    auto rest_a = [&](bf2 piece, float v) {
        return DOT ? __builtin_amdgcn_fdot2_f32_bf16(piece, __builtin_bit_cast(bf2, of_lo), v, false)
                   : v - __builtin_bit_cast(float, __builtin_bit_cast(unsigned, piece) << 16);
    };
    auto rest_b = [&](bf2 piece, float v) {
        return DOT ? __builtin_amdgcn_fdot2_f32_bf16(piece, __builtin_bit_cast(bf2, of_hi), v, false)
                   : v - __builtin_bit_cast(float, __builtin_bit_cast(unsigned, piece) & 0xffff0000u);
    };
    a *= up_a;
    b *= up_b;
    const bf2 h = __builtin_convertvector((f2){a, b}, bf2);
    const float ra = rest_a(h, a), rb = rest_b(h, b);
    const bf2 m = __builtin_convertvector((f2){ra, rb}, bf2);
    out[0][i] = __builtin_bit_cast(unsigned, h);
    out[1][i] = __builtin_bit_cast(unsigned, m);
    out[2][i] = __builtin_bit_cast(unsigned, __builtin_convertvector((f2){rest_a(m, ra), rest_b(m, rb)}, bf2));
}

template <bool DOT = false>
__device__ __forceinline__ void split8(const float (&v)[8], u4 (&out)[3])
{
#pragma unroll
    for (int i = 0; i < 4; ++i) split2<DOT>(v[2 * i], v[2 * i + 1], kUp, kUp, i, out);
}

}  // namespace
}  // namespace sconv
