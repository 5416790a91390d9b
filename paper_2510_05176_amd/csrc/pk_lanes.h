// Exchange between the four 16-lane rows of a wave (lane = 16 * kb + n, kb the row) by row swaps of the vector registers.  In place
// of permutes through LDS (__shfl_xor compiles to those) the values neither queue behind the wave's other LDS accesses nor wait
// for them, and two or four values that are reduced over the rows share the swaps (512 streams x 32640 vectors, 128 patterns, K and V
// quantizers 3001 -> 2825 us, branches in the directed fp16 roundings taken out with them; mining 13.5 -> 13.2 ms).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pk {

typedef uint32_t rows2 __attribute__((ext_vector_type(2)));

// [0]: rows 0 and 2 of a in rows 0 and 2, rows 0 and 2 of b in rows 1 and 3;  [1]: rows 1 and 3 of both, likewise
__device__ __forceinline__ rows2 swap16(uint32_t a, uint32_t b) { return __builtin_amdgcn_permlane16_swap(a, b, false, false); }
// [0]: rows 0 and 1 of a in rows 0 and 1, rows 0 and 1 of b in rows 2 and 3;  [1]: rows 2 and 3 of both, likewise
__device__ __forceinline__ rows2 swap32(uint32_t a, uint32_t b) { return __builtin_amdgcn_permlane32_swap(a, b, false, false); }

__device__ __forceinline__ uint32_t bits_of(float v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ uint32_t bits_of(uint32_t v) { return v; }

// Operations the compiler knows: it keeps two wait states between a vector operation's result and the lane swap that reads it, and
// does not count what inline assembly writes.  (fminf and fmaxf quieten signalling NaN first, an operation more per operand that
// comes from another lane: K and V quantizers of 512 streams x 32640 vectors 2656 us with the bare instructions, 2665 with these.)
struct MinF {
    __device__ __forceinline__ float operator()(float a, float b) const { return fminf(a, b); }
};
struct MaxF {
    __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); }
};
struct AddF {
    __device__ __forceinline__ float operator()(float a, float b) const { return a + b; }
};

template <class OP>
__device__ __forceinline__ float op_rows(rows2 v, OP op)
{
    const uint32_t first = v[0], second = v[1];   // (a bit cast of the element itself takes the first one both times)
    return op(__builtin_bit_cast(float, first), __builtin_bit_cast(float, second));
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t x)   // the value of another lane of the row (data-parallel-primitive control word)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, true);
}
// Sum over the 16 lanes of a row, in every lane: lanes n ^ 1, n ^ 2, then half rows and rows mirrored, which are n ^ 4 and n ^ 8 by then
__device__ __forceinline__ float row_sum(float v)
{
    v += __builtin_bit_cast(float, dpp<0xb1>(bits_of(v)));
    v += __builtin_bit_cast(float, dpp<0x4e>(bits_of(v)));
    v += __builtin_bit_cast(float, dpp<0x141>(bits_of(v)));
    v += __builtin_bit_cast(float, dpp<0x140>(bits_of(v)));
    return v;
}
__device__ __forceinline__ float row_max(float v)
{
    const MaxF op;
    v = op(v, __builtin_bit_cast(float, dpp<0xb1>(bits_of(v))));
    v = op(v, __builtin_bit_cast(float, dpp<0x4e>(bits_of(v))));
    v = op(v, __builtin_bit_cast(float, dpp<0x141>(bits_of(v))));
    return op(v, __builtin_bit_cast(float, dpp<0x140>(bits_of(v))));
}

// Reduction of N values (1, 2 or 4) over the four rows: row kb gets the total of value kb % N.  Rows are combined as neighbours first.
template <int N, class OP>
__device__ __forceinline__ float fold_rows(const float (&x)[N], OP op)
{
    static_assert(N == 1 || N == 2 || N == 4, "one value per row, or the same one in several");
    if constexpr (N == 4) {
        const float a = op_rows(swap16(bits_of(x[0]), bits_of(x[1])), op), b = op_rows(swap16(bits_of(x[2]), bits_of(x[3])), op);
        return op_rows(swap32(bits_of(a), bits_of(b)), op);
    } else {
        const float a = op_rows(swap16(bits_of(x[0]), bits_of(x[N - 1])), op);
        return op_rows(swap32(bits_of(a), bits_of(a)), op);
    }
}
// The inverse: every lane gets what rows 0 .. N-1 hold for its column.
template <int N>
__device__ __forceinline__ void spread_rows(uint32_t v, uint32_t (&out)[N])
{
    if constexpr (N == 1) {
        out[0] = v;
    } else if constexpr (N == 2) {
        const rows2 p = swap16(v, v);
        out[0] = p[0];
        out[1] = p[1];
    } else {
        const rows2 h = swap32(v, v), p = swap16(h[0], h[0]), q = swap16(h[1], h[1]);
        out[0] = p[0];
        out[1] = p[1];
        out[2] = q[0];
        out[3] = q[1];
    }
}
template <int N>
__device__ __forceinline__ void spread_rows(float v, float (&out)[N])
{
    uint32_t u[N];
    spread_rows<N>(bits_of(v), u);
#pragma unroll
    for (int i = 0; i < N; ++i) out[i] = __builtin_bit_cast(float, u[i]);
}

}  // namespace pk
