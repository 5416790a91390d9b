// Bit planes to matrix-core operands, shared by the decode kernels: two bit planes are merged into 2-bit fields, and a field
// masked in place inside the mantissa of an fp16 with exponent field 0 is the subnormal number code * 2^(pos - 24).
#pragma once
#include "pk_internal.h"

namespace pk {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float float2v __attribute__((ext_vector_type(2)));

// (a & m) | (b & ~m), in the three-input logic operation: it issues at twice the rate of the bit-field insert
__device__ __forceinline__ uint32_t bfi(uint32_t m, uint32_t a, uint32_t b) { return __builtin_amdgcn_bitop3_b32(m, a, b, 0xca); }

// base + SCALE * byte i of w.  (A byte dot product with one weight would be one operation instead of two; it measured 1 to 5 % of a
// decode slower.)
template <uint32_t SCALE>
__device__ __forceinline__ uint32_t byte_address(uint32_t w, int i, uint32_t base)
{
    return ((w >> (8 * i)) & 255u) * SCALE + base;
}

__device__ __forceinline__ floatx4 mfma16(const uint32_t *a, const uint32_t *b, floatx4 c)
{
    union { uint32_t u[4]; half8 h; } A, B;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        A.u[i] = a[i];
        B.u[i] = b[i];
    }
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(A.h, B.h, c, 0, 0, 0);
}

__device__ __forceinline__ uint32_t pack2(_Float16 lo, _Float16 hi)
{
    half2v v = {lo, hi};
    return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ uint32_t pk_mul(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2v, a) * __builtin_bit_cast(half2v, b));
}
__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c)
{
    return __builtin_amdgcn_fdot2(__builtin_bit_cast(half2v, a), __builtin_bit_cast(half2v, b), c, false);
}
__device__ __forceinline__ uint32_t cvt2(float lo, float hi)
{
    float2v f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, half2v));
}

// Sixteen 2-bit fields at the even bit positions of X -> eight operand registers.  Register v
// holds, in its low half, the field of X-bit e_lo(v) and, in its high half, the field of X-bit
// e_lo(v) + 16, both at mantissa position pos(v):
//   v = 0..4: e_lo = 2v, pos = 2v ;  v = 5..7: e_lo = 10 + 2(v-5), pos = 2(v-5).
__device__ __forceinline__ void fields_to_operand(uint32_t X, uint32_t *out)
{
    out[0] = X & 0x00030003u;
    out[1] = X & 0x000C000Cu;
    out[2] = X & 0x00300030u;
    out[3] = X & 0x00C000C0u;
    out[4] = X & 0x03000300u;
    const uint32_t Y = X >> 10;
    out[5] = Y & 0x00030003u;
    out[6] = Y & 0x000C000Cu;
    out[7] = Y & 0x00300030u;
}
__host__ __device__ constexpr int e_lo(int v) { return v < 5 ? 2 * v : 10 + 2 * (v - 5); }
__host__ __device__ constexpr int fpos(int v) { return v < 5 ? 2 * v : 2 * (v - 5); }

}  // namespace
}  // namespace pk
