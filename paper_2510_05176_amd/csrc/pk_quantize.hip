// Quantize-append kernels: pattern selection (Sec. 3.2 Eq. 6), residual, group
// min/max -> stored (s, z), asymmetric n-bit quantization (Sec. 2.1 Eq. 1), bit-plane
// packing.  K is quantized per channel over groups of G tokens, V per token over
// groups of Gc channels (Sec. 4.1 "Quantization Settings").
//
// The arithmetic that decides a code is a fixed sequence of binary32 operations
// (subtract, one division per group for s, one for 1/s, subtract, multiply, round
// half to even, clamp); contraction into FMAs is switched off for this file so
// that the sequence is exactly what is written.
//
// Kernels, in file order: assign_minmax_kernel (the min-max selection rule of Sec. 3.2 as a search of its own, at every
// head dimension: it writes the indices and the quantizers below then take them as given); quantize_k_group_kernel (groups of 128 tokens,
// a workgroup of eight waves per group) and quantize_k_wave_kernel (groups of 32 / 64 tokens, a wave per group); quantize_v_kernel
// (a wave per 16-token unit); tail_copy_kernel (the fp16 ring); seq_table_kernel (per-sequence launch parameters
// of a ragged append).  Under the Euclidean rule the quantizers search on the matrix cores (pk_assign_mfma.h).
#pragma clang fp contract(off)

#include "pk_assign_mfma.h"
#include "pk_quant_arith.h"
#include "pk_cut.h"
#include "pk_internal.h"

namespace pk {

namespace {

// ---------------------------------------------------------------------------
// Min-max metric (Sec. 3.2): d_mm(x, m) = max_c (x_c - m_c) - min_c (x_c - m_c), argmin over the patterns, lowest
// index on ties.  Every operation of the definition is exact in binary32 apart from one correctly rounded subtraction per
// channel (fp16 values widened exactly) and the last one, so the result is the definition's, bit for bit; it is not a
// contraction and runs on the vector ALUs.  A wave takes 64 vectors, lane <-> vector, the vector's channels in
// registers as loaded.  The indices go to the cache's index array; the quantizers then skip their own search.
//
// Every pattern is ranked in packed fp16, two channels per operation: a subtraction (the pattern row wave-uniform, a
// scalar operand), and half of a three-operand maximum and minimum each.  fp16 rounding is monotone, so the maximum and
// minimum found are the roundings of the true ones, and the distance lies within 2^-11 (|max| + |min|) of their
// difference; with twice that, c = 2^-10, difference - c (|max| + |min|) is a lower bound and the same + 2 c (|max| +
// |min|) an upper one.  The three smallest lower bounds are tracked; where the second does not exceed the upper bound of the
// first, the lane evaluates these two patterns in binary32; where the third does not exceed it either, the wave evaluates
// the vector against all patterns, lane <-> pattern.  Where that is so for many vectors of a tile - repeated patterns, vectors
// so far from the table that all distances lie within the bounds of each other - the tile and the wave's further ones are
// searched in binary32 throughout (minmax_nearest; already after a quarter of the table if it is so by then): 128 streams x 4096
// vectors, every one of 64 patterns four times 2714 -> 637 us for the append (binary32 ranking 640), of 200 8847 -> 1656
// (1658), vectors of spread 0.05 at a distance of 3 1317 -> 705 (591) and 4910 -> 1723 (1646).
// 1.1 vector operations per channel and pattern instead of the 2.1 of ranking in binary32 (a mixed-precision subtraction and
// half of a three-operand maximum and minimum), bound by their issue: 256 streams x 8192 vectors, 64 patterns 998 -> 565 us
// per search alone, 600 to 612 in an append (485 at the issue rate of the packed operations), at 128 patterns a whole append 4.16 -> 2.53 ms, 128 streams
// of 256 channels 3.32 -> 2.33 ms.  (Scalar loads of 32 channels per wait instead of 64: 650 us, and no gain at 256 channels,
// whose two waves per SIMD did not cover their latency.)
// Ruling patterns out by the range over a few channels first (the widest over the table) and evaluating the rest in full
// measured 437 us on keys and 716 us on values in the same job, 1.4 times the binary32 scan's time on unclustered vectors,
// and more than it at 250 patterns: candidates differ from vector to vector, so a wave runs as long as its worst one.
// ---------------------------------------------------------------------------
typedef _Float16 mm_half2 __attribute__((ext_vector_type(2)));

// Sixteen consecutive dwords through the scalar data path (read only: the constant address space; address wave-uniform, 4-byte
// aligned).  arrived(): a use of the values, so that the compiler waits for them here and not behind the next request.
typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));
typedef u32x16 u32x16_dword_aligned __attribute__((aligned(4)));
__device__ __forceinline__ u32x16 sload16(const uint32_t *p)
{
    return *(const __attribute__((address_space(4))) u32x16_dword_aligned *)(uintptr_t)p;
}
__device__ __forceinline__ void arrived(u32x16 (&r)[1]) { asm volatile("" : "+s"(r[0])); }
__device__ __forceinline__ void arrived(u32x16 (&r)[2]) { asm volatile("" : "+s"(r[0]), "+s"(r[1])); }

// x - half(m.lo), x - half(m.hi) of two fp16 numbers, m a scalar operand
__device__ __forceinline__ float sub_s_lo(uint32_t x, uint32_t m)
{
    float r;
    asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[0,0,0] op_sel_hi:[1,0,1]" : "=v"(r) : "v"(x), "s"(m));
    return r;
}
__device__ __forceinline__ float sub_s_hi(uint32_t x, uint32_t m)
{
    float r;
    asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[1,0,1] op_sel_hi:[1,0,1]" : "=v"(r) : "v"(x), "s"(m));
    return r;
}

// Which run of tiles of its stream (blockIdx.y) a workgroup takes.  Workgroups go to the chip's eight XCDs in turn
// by their linear index, y * gridDim.x + x; with the run taken as x itself an XCD would get the runs x = k, k + 8, ...
// of EVERY stream, and when streams have different numbers of runs (a ragged append: the grid is sized for the
// longest sequence and the runs past a sequence's end return at once) the XCDs of low k get up to 55 % more
// work than the last one (measured: 16 prompts of 2 k to 32 k tokens ran 1.55x slower than the same bytes in
// equal lengths).  Rotating the run by the stream index gives every XCD every residue class in turn.
__device__ __forceinline__ int chunk_of_workgroup()
{
    return (int)((blockIdx.x + blockIdx.y) % gridDim.x);
}

// Range of the differences of the vector x from the pattern m, in binary32: the definition.  Both rows are read from
// memory (few lanes do this; the vector held in registers across it spills), kStep pieces of each in flight.
template <int NC>
__device__ __forceinline__ float minmax_distance(const __half *x, const __half *m)
{
    constexpr int kStep = 4;
    // two running maxima and minima, so that consecutive operations do not wait for each other
    float mxa = -INFINITY, mxb = -INFINITY, mna = INFINITY, mnb = INFINITY;
    uint4 xv[kStep], mv[kStep];
#pragma unroll
    for (int i = 0; i < kStep; ++i) {
        xv[i] = *reinterpret_cast<const uint4 *>(x + 8 * i);
        mv[i] = *reinterpret_cast<const uint4 *>(m + 8 * i);
    }
#pragma unroll
    for (int c0 = 0; c0 < NC; c0 += kStep) {
        uint4 xw[kStep], mw[kStep];
        if (c0 + kStep < NC) {
#pragma unroll
            for (int i = 0; i < kStep; ++i) {
                xw[i] = *reinterpret_cast<const uint4 *>(x + 8 * (c0 + kStep + i));
                mw[i] = *reinterpret_cast<const uint4 *>(m + 8 * (c0 + kStep + i));
            }
        }
#pragma unroll
        for (int i = 0; i < kStep; ++i) {
            const uint4 u = xv[i], v = mv[i];
            const float d0 = sub_lo(u.x, v.x), d1 = sub_hi(u.x, v.x), d2 = sub_lo(u.y, v.y), d3 = sub_hi(u.y, v.y);
            const float d4 = sub_lo(u.z, v.z), d5 = sub_hi(u.z, v.z), d6 = sub_lo(u.w, v.w), d7 = sub_hi(u.w, v.w);
            mxa = fmaxf(fmaxf(mxa, d0), d1);
            mna = fminf(fminf(mna, d0), d1);
            mxb = fmaxf(fmaxf(mxb, d2), d3);
            mnb = fminf(fminf(mnb, d2), d3);
            mxa = fmaxf(fmaxf(mxa, d4), d5);
            mna = fminf(fminf(mna, d4), d5);
            mxb = fmaxf(fmaxf(mxb, d6), d7);
            mnb = fminf(fminf(mnb, d6), d7);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < kStep; ++i) {
            xv[i] = xw[i];
            mv[i] = mw[i];
        }
    }
    float dist = fmaxf(mxa, mxb) - fminf(mna, mnb);
    asm volatile("" : "+v"(dist));   // formed here: moved behind a condition, the maxima leave every difference waiting in a register
    return dist;
}

// A wave evaluates one vector against all patterns in the time in which a scan takes 5 of its 64 vectors: beyond this many open
// vectors of a tile the scan is the faster one.
constexpr int kOpen = 12;

// The table's rows through the scalar path.  Scalar loads return in any order, so a wait covers all that are outstanding: the next
// step's channels are requested right after the wait for the current ones and arrive under their 64 (96 channels: 32) vector
// operations.
template <int D>
struct RowSteps {
    static constexpr int W = D % 64 == 0 ? 2 : 1, NS = D / (32 * W);   // scalar loads (32 channels each) per step, steps
    const uint32_t *M;
    int P;
    u32x16 buf[2][W];
    __device__ __forceinline__ void request(const uint32_t *at, u32x16 (&to)[W])
    {
#pragma unroll
        for (int w = 0; w < W; ++w) to[w] = sload16(at + 16 * w);
    }
    // step(32 channels, which) over pattern p's row; at: which buffer holds (will hold) its first step
    template <class STEP>
    __device__ __forceinline__ void row(int p, int at, STEP step)
    {
        const uint32_t *mrow = M + (size_t)p * (D / 2), *mnext = M + (size_t)min(p + 1, P - 1) * (D / 2);   // (past the last row: that row again; unused)
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            arrived(buf[(s + at) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            request(s + 1 < NS ? mrow + 16 * W * (s + 1) : mnext, buf[(s + at + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);   // (the scheduler would issue the request behind most of the scan)
#pragma unroll
            for (int w = 0; w < W; ++w) step(buf[(s + at) & 1][w], s * W + w);
        }
    }
    // pattern(p, at) over the table; given up in front of pattern `probe` (even; 0: never) if give_up() says so
    template <class PATTERN, class GIVE_UP>
    __device__ __forceinline__ void all(PATTERN pattern, int probe, GIVE_UP give_up)
    {
        request(M, buf[0]);
        int p = 0;
        for (int end = probe;; end = P) {
            for (; p + 1 < end; p += 2) {
                pattern(p, 0);
                pattern(p + 1, NS % 2);
            }
            if (end == P) break;
            if (probe > 0 && give_up()) return;
        }
        if (p < P) pattern(p, 0);
    }
};

// The lane's vector, two channels per register
template <int D>
__device__ __forceinline__ void load_vector(const __half *row, uint32_t (&x)[D / 2])
{
#pragma unroll
    for (int ch = 0; ch < D / 8; ++ch) {
        const uint4 v = *reinterpret_cast<const uint4 *>(row + 8 * ch);
        x[4 * ch] = v.x;
        x[4 * ch + 1] = v.y;
        x[4 * ch + 2] = v.z;
        x[4 * ch + 3] = v.w;
    }
}

// Nearest pattern of the lane's vector, all of them in binary32: the definition, 2.1 vector operations per channel and pattern.
template <int D>
__device__ __forceinline__ int minmax_nearest(const __half *xrow, const uint32_t *M, int P)
{
    uint32_t x[D / 2];
    load_vector<D>(xrow, x);
    RowSteps<D> rows;
    rows.M = M;
    rows.P = P;
    float bd = INFINITY;
    int bi = 0;
    rows.all([&](int p, int at) {
        float pa = -INFINITY, pb = -INFINITY, na = INFINITY, nb = INFINITY;   // two chains, as below
        rows.row(p, at, [&](const u32x16 &m, int s) {
#pragma unroll
            for (int k = 0; k < 16; k += 2) {
                const uint32_t m0 = m[k], m1 = m[k + 1];
                const float d0 = sub_s_lo(x[16 * s + k], m0), d1 = sub_s_hi(x[16 * s + k], m0);
                const float d2 = sub_s_lo(x[16 * s + k + 1], m1), d3 = sub_s_hi(x[16 * s + k + 1], m1);
                pa = fmaxf(fmaxf(pa, d0), d1);
                na = fminf(fminf(na, d0), d1);
                pb = fmaxf(fmaxf(pb, d2), d3);
                nb = fminf(fminf(nb, d2), d3);
            }
        });
        const float dist = fmaxf(pa, pb) - fminf(na, nb);
        bi = dist < bd ? p : bi;   // patterns in increasing order
        bd = fminf(dist, bd);
    }, 0, []() { return false; });
    return bi;
}

template <int D>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 256 ? 2 : 4))) void assign_minmax_kernel(QuantKernelArgs a, int tiles_per_wg)
{
    constexpr int NC = D / 8;   // 16-byte pieces of a vector
    const int tid = threadIdx.x, lane = tid & 63, ns = blockIdx.y, P = a.P;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const __half *Mh = a.patterns + (int64_t)a.sets.set_of(ns) * a.P * D;
    const uint32_t *Mg = reinterpret_cast<const uint32_t *>(Mh);
    take_sequence_entry(a, ns);
    const StreamMap map = a.map.of(ns);
    const int n_tiles = a.nq / 64;
    const int tile0 = chunk_of_workgroup() * tiles_per_wg, tile1 = min(n_tiles, tile0 + tiles_per_wg);
    bool undecided = false;   // the bounds left many vectors of a tile open: this tile and the wave's further ones without them
    for (int tile = tile0 + wave; tile < tile1; tile += 4) {
        int best;
        if (!undecided) {
            uint32_t x[D / 2];
            load_vector<D>(a.src.row_d(ns, tile * 64 + lane, D), x);
            constexpr float c = 9.765625e-4f;
            uint32_t k1 = 0xffffffffu, k2 = 0xffffffffu, k3 = 0xffffffffu;   // the three smallest bounds, the pattern in the low byte
            float t1 = 0.f;                                 // |max| + |min| of the first
            mm_half2 mxa, mxb, mna, mnb;                    // two chains, so that consecutive operations do not wait for each other
            auto scan = [&](const u32x16 &m, int s) {
#pragma unroll
                for (int k = 0; k < 16; k += 4) {
                    const uint32_t m0 = m[k], m1 = m[k + 1], m2 = m[k + 2], m3 = m[k + 3];
                    const mm_half2 r0 = __builtin_bit_cast(mm_half2, x[16 * s + k]) - __builtin_bit_cast(mm_half2, m0);
                    const mm_half2 r1 = __builtin_bit_cast(mm_half2, x[16 * s + k + 1]) - __builtin_bit_cast(mm_half2, m1);
                    const mm_half2 r2 = __builtin_bit_cast(mm_half2, x[16 * s + k + 2]) - __builtin_bit_cast(mm_half2, m2);
                    const mm_half2 r3 = __builtin_bit_cast(mm_half2, x[16 * s + k + 3]) - __builtin_bit_cast(mm_half2, m3);
                    if (s == 0 && k == 0) {
                        mxa = __builtin_elementwise_maximum(r0, r1);
                        mna = __builtin_elementwise_minimum(r0, r1);
                        mxb = __builtin_elementwise_maximum(r2, r3);
                        mnb = __builtin_elementwise_minimum(r2, r3);
                    } else {
                        mxa = __builtin_elementwise_maximum(__builtin_elementwise_maximum(mxa, r0), r1);
                        mna = __builtin_elementwise_minimum(__builtin_elementwise_minimum(mna, r0), r1);
                        mxb = __builtin_elementwise_maximum(__builtin_elementwise_maximum(mxb, r2), r3);
                        mnb = __builtin_elementwise_minimum(__builtin_elementwise_minimum(mnb, r2), r3);
                    }
                }
            };
            // whether the lower bound of a key does not exceed the first one's upper bound (first's own low bits, 2^-15 of it, belong to that)
            auto reaches = [&](uint32_t k) {
                const float first = __uint_as_float(k1 & 0xffffff00u);
                return !(__uint_as_float(k & 0xffffff00u) > fmaf(first, 6.103515625e-05f, fmaf(t1, 2.f * c, first)));
            };
            RowSteps<D> rows;
            rows.M = Mg;
            rows.P = P;
            rows.all([&](int p, int at) {
                rows.row(p, at, scan);
                const mm_half2 mx = __builtin_elementwise_maximum(mxa, mxb), mn = __builtin_elementwise_minimum(mna, mnb);
                const float hi = (float)__builtin_elementwise_maximum(mx[0], mx[1]), lo = (float)__builtin_elementwise_minimum(mn[0], mn[1]);
                const float t = fabsf(hi) + fabsf(lo);
                // (not a number - a difference that overflowed fp16 - gives the bound 0 and leads to the exact evaluation)
                const uint32_t key = (__float_as_uint(fmaxf(fmaf(t, -c, hi - lo), 0.f)) & 0xffffff00u) | (uint32_t)p;
                t1 = key < k1 ? t : t1;
                k3 = max(min(k2, k3), min(max(k2, k3), key));   // medians of three
                k2 = max(min(k1, k2), min(max(k1, k2), key));
                k1 = min(k1, key);
            }, P >= 16 ? P / 4 & ~1 : 0, [&]() {   // (as open as that after a quarter of the table, the rest of it seldom decides)
                undecided = __popcll(__ballot(reaches(k3))) > kOpen;
                return undecided;
            });
            best = (int)(k1 & 0xffu);
            const bool two = P > 1 && reaches(k2), more = P > 2 && two && reaches(k3);
            if (two && !more && !undecided) {
                const __half *row = a.src.row_d(ns, tile * 64 + lane, D);
                float bd = INFINITY;
                int bi = 0;
#pragma unroll 1
                for (uint32_t i = 0, q = k1; i < 2; ++i, q = k2) {
                    const int cand = (int)(q & 0xffu);
                    const float dist = minmax_distance<NC>(row, Mh + (int64_t)cand * D);
                    const bool nearer = dist < bd || (dist == bd && cand < bi);
                    bd = nearer ? dist : bd;
                    bi = nearer ? cand : bi;
                }
                best = bi;
            }
            unsigned long long todo = __ballot(more);
            undecided = undecided || __popcll(todo) > kOpen;
            while (!undecided && todo) {
                const int col = __ffsll((long long)todo) - 1;
                todo &= todo - 1;
                const __half *row = a.src.row_d(ns, tile * 64 + col, D);
                float bd = INFINITY;
                int bi = 0;
                for (int q = lane; q < P; q += 64) {
                    const float dist = minmax_distance<NC>(row, Mh + (int64_t)q * D);
                    if (dist < bd) {   // the lane's patterns in increasing order
                        bd = dist;
                        bi = q;
                    }
                }
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const float od = __shfl_xor(bd, off);
                    const int oi = __shfl_xor(bi, off);
                    if (od < bd || (od == bd && oi < bi)) {
                        bd = od;
                        bi = oi;
                    }
                }
                if (lane == col) best = bi;
            }
        }
        if (undecided) best = minmax_nearest<D>(a.src.row_d(ns, tile * 64 + lane, D), Mg, P);
        a.idx[map.pos(a.t0 + tile * 64) + lane] = (uint8_t)best;
    }
}

// ===========================================================================
// Euclidean metric: nearest pattern on the matrix cores (pk_assign_mfma.h).  A wave owns 16-token
// tiles; lane 16*kb + n holds, of token n, the D/4 channels 32*k + 8*kb + j (k < D/32, j < 8) - the MFMA
// B-operand layout - and forms the residuals of those channels in registers.
//
// K: the per-channel minimum / maximum over the group's tokens goes through a small LDS tile of the wave, 32 channels at a
//    time; the parameters come back through LDS; every lane then forms one byte of each plane word (8 channels).
// V: everything per token stays inside the wave: group minimum / maximum by two cross-lane steps,
//    16 codes per plane packed per lane, and a 16x16 bit transpose across the 16 token lanes turns
//    them into the words of 16 tokens per channel.
// The kernels are templates on the head dimension D: 128, and 96 and 256 (the other two head sizes that Sec. 3.3 names),
// which had a search kernel and thread <-> channel quantizers of their own that read the vectors three times: 256 streams x
// 4096 vectors of 96 channels in 32-token groups 583 -> 154 us, of 256 channels in 64-token groups (whole append) 1150 ->
// 350 us.
// ===========================================================================

// (sub_lo / sub_hi, the fp16 differences with one rounding, live in pk_internal.h: the exact search uses them too)
__device__ __forceinline__ float subz_lo(float x, uint32_t z)   // x - half(z.lo)
{
    float r;
    asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[0,0,0] op_sel_hi:[0,0,1]" : "=v"(r) : "v"(x), "v"(z));
    return r;
}
__device__ __forceinline__ float subz_hi(float x, uint32_t z)   // x - half(z.hi)
{
    float r;
    asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[0,0,1] op_sel_hi:[0,0,1]" : "=v"(r) : "v"(x), "v"(z));
    return r;
}

// Codes.  d = r - z >= 0 and d * (1/s) lies in [0, 2^b - 1] up to rounding because z <= min and
// s >= (max - z)/(2^b - 1), so the clamp of the definition never acts.  v_cvt_pk_u8_f32 rounds half to
// even like rintf (and saturates at 0 and 255) and drops the code into one byte of a word: four codes per
// word.  packed <- packed with code(d * inv) in byte `slot`.
__device__ __forceinline__ uint32_t put_code(float d, float inv, int slot, uint32_t packed)
{
    return __builtin_amdgcn_cvt_pk_u8_f32(d * inv, (uint32_t)slot, packed);
}

// Bits p of the 8 codes held in the bytes of (lo, hi), gathered into bits p .. p+7 of the result:
// two masked byte dot products with weights 1, 2, 4, .. 128.
__device__ __forceinline__ uint32_t plane_byte_shifted(uint32_t lo, uint32_t hi, int p)
{
    const uint32_t m = 0x01010101u << p;
    uint32_t acc = __builtin_amdgcn_udot4(lo & m, 0x08040201u, 0u, false);
    return __builtin_amdgcn_udot4(hi & m, 0x80402010u, acc, false);
}

// Sum of the 8 codes held in the bytes of (lo, hi), code i times 2^i.
__device__ __forceinline__ uint32_t byte_sum(uint32_t lo, uint32_t hi)
{
    return __builtin_amdgcn_udot4(hi, 0x80402010u, __builtin_amdgcn_udot4(lo, 0x08040201u, 0u, false), false);
}

// The pattern table at the start of the dynamic LDS of every quantizer: rows, -|m|^2 / 2, one maximum per wave.
struct TableLds {
    __half *tab;      // [pad16(P)][kTabStrideOf<D>]
    float *nh;        // [pad16(P)]
    float *red;       // [16]
};
template <int D>
__host__ __device__ constexpr size_t table_lds_bytes(int P)
{
    return (size_t)pad16(P) * kTabStrideOf<D> * 2 + (size_t)pad16(P) * 4 + 64;
}
template <int D>
__device__ __forceinline__ TableLds table_lds(unsigned char *smem, int P)
{
    TableLds t;
    t.tab = reinterpret_cast<__half *>(smem);
    t.nh = reinterpret_cast<float *>(smem + (size_t)pad16(P) * kTabStrideOf<D> * 2);
    t.red = t.nh + pad16(P);
    return t;
}

template <int NW>
__device__ __forceinline__ PatternTable make_table(const TableLds &sh, int P)
{
    PatternTable tb;
    tb.lds_rows = sh.tab;
    tb.nh = sh.nh;
    tb.norm2_max = sh.red[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) tb.norm2_max = fmaxf(tb.norm2_max, sh.red[w]);
    tb.P = P;
    return tb;
}

// B operand of one 16-token tile: vectors i0 .. i0+15 of stream ns (i0 wave-uniform).  A tile without vectors of the ring - nearly
// all of a long append - takes one scalar address and fixed lane offsets.
template <int KS>
__device__ __forceinline__ void load_tile(const QuantKernelArgs &a, int ns, int i0, uint4 (&xb)[KS])
{
    constexpr int D = 32 * KS;
    const int lane = threadIdx.x & 63, n = lane & 15, kb = lane >> 4;
    if (i0 >= a.src.n_ring) {
        const __half *tile = a.src.fresh + (int64_t)ns * a.src.fresh_stride + (int64_t)(i0 - a.src.n_ring) * D;
        const uint32_t at = n * D + 8 * kb;
#pragma unroll
        for (int k = 0; k < KS; ++k) xb[k] = *reinterpret_cast<const uint4 *>(tile + at + 32 * k);
    } else {
        const __half *row = a.src.row_d(ns, i0 + n, D);
#pragma unroll
        for (int k = 0; k < KS; ++k) xb[k] = *reinterpret_cast<const uint4 *>(row + 32 * k + 8 * kb);
    }
}

// Residuals r[j] of channel 32k + 8kb + j: eight channels of a vector minus those of a pattern.
__device__ __forceinline__ void residuals8(const uint4 xv, const uint4 mv, float *r)   // (mv by value: one 16-byte LDS read)
{
    r[0] = sub_lo(xv.x, mv.x);
    r[1] = sub_hi(xv.x, mv.x);
    r[2] = sub_lo(xv.y, mv.y);
    r[3] = sub_hi(xv.y, mv.y);
    r[4] = sub_lo(xv.z, mv.z);
    r[5] = sub_hi(xv.z, mv.z);
    r[6] = sub_lo(xv.w, mv.w);
    r[7] = sub_hi(xv.w, mv.w);
}

// Residuals r[8k + j] of channel 32k + 8kb + j of the lane's token against pattern bi.
template <int KS>
__device__ __forceinline__ void residuals(const TableLds &sh, const uint4 (&xb)[KS], int bi, float (&r)[8 * KS])
{
    const int kb = (threadIdx.x & 63) >> 4;
    const __half *mrow = sh.tab + bi * kTabStrideOf<32 * KS> + 8 * kb;
#pragma unroll
    for (int k = 0; k < KS; ++k) residuals8(xb[k], *reinterpret_cast<const uint4 *>(mrow + 32 * k), r + 8 * k);
}

// Nearest pattern of the tile's tokens (exact).  Tokens that are not finite take the lowest index: their residuals are read from
// the table by it.
template <int KS>
__device__ __forceinline__ int assign_index(const PatternTable &tb, const uint4 (&xb)[KS], __half *xrow)
{
    const int lane = threadIdx.x & 63;
    int bi;
    float bv, x2, bd;
    bool flag;
    assign_tile_mfma(xb, tb, lane, bi, bv, x2, flag);
    resolve_flagged(xb, flag, xrow, tb, lane, 0, bi, bd);
    return bi;
}

// All LDS writes of the wave so far are visible to its own later reads.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Contiguous store of BYTES bytes from LDS by a wave, in 8- or 16-byte lane pieces.
template <int BYTES>
__device__ __forceinline__ void wave_store(uint8_t *dst, const uint8_t *src)
{
    const int lane = threadIdx.x & 63;
    if (BYTES == 512) {
        reinterpret_cast<uint2 *>(dst)[lane] = reinterpret_cast<const uint2 *>(src)[lane];
    } else {
        static_assert(BYTES == 512 || BYTES % 16 == 0, "whole pieces");
#pragma unroll
        for (int i = 0; i < BYTES / 16; i += 64)
            if (BYTES / 16 - i >= 64 || i + lane < BYTES / 16)
                reinterpret_cast<uint4 *>(dst)[i + lane] = reinterpret_cast<const uint4 *>(src)[i + lane];
    }
}

// ---- K ------------------------------------------------------------------------------------------------------------
// LDS of a wave: the 32-channel residual tile of 16 tokens (also the row under exact evaluation and the output staging:
// code words in memory order, then the indices).  Parameters of a group: zero points and scales (fp16 bits), 1/s.
constexpr int kWkStride = 32 + 4;                     // floats per row of the residual tile
constexpr int kWkTile = 16 * kWkStride * 4;           // bytes: 16 tokens x 32 channels
template <int D>
constexpr int kKParams = D * 2 * 2 + D * 4;           // bytes of one group's parameters

// Running minimum / maximum per channel over a 16-token tile: the residuals of 32 channels (operand step k) at a time
// pass through the wave's LDS tile; lane <-> (channel 32k + lane%32, token half lane/32).  A step's values are used behind the next
// step's stores (the LDS takes a wave's accesses in order): between its own stores and its use a step's loads would be waited for (1483 -> 1453 us).
struct ChannelScan {
    float v[8];
    float *mn, *mx;   // of the step that v belongs to; null: none
    __device__ __forceinline__ void use()
    {
#pragma unroll
        for (int t = 0; t < 8; t += 2) {
            *mn = fminf(fminf(*mn, v[t]), v[t + 1]);
            *mx = fmaxf(fmaxf(*mx, v[t]), v[t + 1]);
        }
    }
    __device__ __forceinline__ void step(const float *r, float *rt, float &low, float &high)
    {
        const int lane = threadIdx.x & 63, n = lane & 15, kb = lane >> 4, sc = lane & 31, sth = lane >> 5;
        float4 *dst = reinterpret_cast<float4 *>(rt + n * kWkStride + 8 * kb);
        dst[0] = make_float4(r[0], r[1], r[2], r[3]);
        dst[1] = make_float4(r[4], r[5], r[6], r[7]);
        if (mn) use();
        wave_lds_sync();
#pragma unroll
        for (int t = 0; t < 8; ++t) v[t] = rt[(8 * sth + t) * kWkStride + sc];
        wave_lds_sync();
        mn = &low;
        mx = &high;
    }
};

// The stored parameters of channel c
__device__ __forceinline__ void put_params(float mn, float mx, int bits, int c, int D, uint16_t *pz, float *pinv)
{
    const GroupParams gp = group_params(mn, mx, bits);
    pz[c] = gp.z16;
    pz[D + c] = gp.s16;
    pinv[c] = gp.inv;
}

// Stored parameters of a group, 16-byte pieces by one wave: zero points, then scales
template <int D>
__device__ __forceinline__ void store_params(const QuantKernelArgs &a, int64_t group, const uint16_t *pz)
{
    const int lane = threadIdx.x & 63;
    if (D == 256 || lane < D / 4) {
        const int arr = lane / (D / 8), piece = lane % (D / 8);
        const uint4 v = *reinterpret_cast<const uint4 *>(pz + arr * D + piece * 8);
        *reinterpret_cast<uint4 *>((arr ? a.scale : a.zero) + group * D + piece * 8) = v;
    }
}

// Codes of eight channels of one token (operand step k) against the group's parameters in LDS (zero points as fp16
// bits, 1/s as binary32, indexed by channel): one byte of each plane word, written to the token's row of the staging
// area stg ([16 tokens][D/32 words][BITS planes] words, memory order).
template <int D, int BITS>
__device__ __forceinline__ void k_codes8(const float *r, int k, const uint16_t *pz, const float *pinv, uint8_t *stg)
{
    const int lane = threadIdx.x & 63, n = lane & 15, kb = lane >> 4;
    const uint4 zq = *reinterpret_cast<const uint4 *>(pz + 32 * k + 8 * kb);
    const float4 i0 = *reinterpret_cast<const float4 *>(pinv + 32 * k + 8 * kb);
    const float4 i1 = *reinterpret_cast<const float4 *>(pinv + 32 * k + 8 * kb + 4);
    uint32_t lo = 0u, hi = 0u;
    lo = put_code(subz_lo(r[0], zq.x), i0.x, 0, lo);
    lo = put_code(subz_hi(r[1], zq.x), i0.y, 1, lo);
    lo = put_code(subz_lo(r[2], zq.y), i0.z, 2, lo);
    lo = put_code(subz_hi(r[3], zq.y), i0.w, 3, lo);
    hi = put_code(subz_lo(r[4], zq.z), i1.x, 0, hi);
    hi = put_code(subz_hi(r[5], zq.z), i1.y, 1, hi);
    hi = put_code(subz_lo(r[6], zq.w), i1.z, 2, hi);
    hi = put_code(subz_hi(r[7], zq.w), i1.w, 3, hi);
    uint8_t *mine = stg + n * (D / 8) * BITS + kb;
#pragma unroll
    for (int p = 0; p < BITS; ++p) mine[(k * BITS + p) * 4] = (uint8_t)(plane_byte_shifted(lo, hi, p) >> p);
}

// Staging area -> global: the 16 tokens' code words as one contiguous run, then their 16 indices.
template <int D, int BITS>
__device__ __forceinline__ void k_store_staging(const QuantKernelArgs &a, int64_t tok0, const uint8_t *stg)
{
    constexpr int kBytes = 16 * D * BITS / 8;
    static_assert(kBytes + 16 <= kWkTile, "output staging fits the residual tile");
    wave_store<kBytes>(reinterpret_cast<uint8_t *>(a.codes_k) + tok0 * (D * BITS / 8), stg);
    if ((threadIdx.x & 63) == 0) *reinterpret_cast<uint4 *>(a.idx + tok0) = *reinterpret_cast<const uint4 *>(stg + kBytes);
}

// K, groups of 128 tokens: 8 / NT waves take one group at a time, NT 16-token tiles each.  Every wave reduces its own tokens
// per channel (ChannelScan) and leaves the minima and maxima in its LDS tile; between two barriers a thread per channel
// combines them and forms the parameters.  A workgroup holds GR groups side by side.  Beyond 128 patterns of up to 128
// channels the table leaves room for one workgroup per CU only: sixteen waves cover the barriers' latency, in four groups
// with two tiles per pass over the table where a workgroup has that many groups to take, else in two.  At 256 channels a workgroup has
// two groups from 65 to 128 patterns where that cut is modelled to take less, else one (beyond 128 there is no room for two).
// (A residual tile of the whole group in LDS, scanned by columns, took 68 KB at 128 channels beside the table: one workgroup
// per CU from 128 patterns on, and no room at all at 256 channels.  Appends, K and V: 256 streams x 8192 at 64 patterns 374
// -> 349 us; 64 streams, 4 bits, 128 patterns 174 -> 150; 4 streams x 131072 at 256 patterns, with the first decode, 220 ->
// 210 - one group of eight waves there measured 235, two groups with a tile per pass 221.)
template <int D, int NT>
constexpr int kGroupLds = 8 / NT * kWkTile + kKParams<D>;   // bytes of LDS per group

template <int D, int BITS, int GR, int NT>
__global__ __launch_bounds__(512 / NT * GR) __attribute__((amdgpu_waves_per_eu(D == 256 ? 2 : 4))) void quantize_k_group_kernel(QuantKernelArgs a, int tiles_per_wg)
{
    constexpr int KS = D / 32, TT = 128, NW = 8 / NT, NTH = 64 * NW;   // waves and threads of a group
    static_assert(2 * D * 4 <= kWkTile, "a wave's minima and maxima fit its tile");
    extern __shared__ __align__(16) unsigned char smem[];
    const TableLds sh = table_lds<D>(smem, a.P);
    const int gr = GR == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / NTH);
    const int tid = threadIdx.x % NTH, ns = blockIdx.y;          // thread inside the group
    const int lane = tid & 63, n = lane & 15, kb = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    unsigned char *work = smem + table_lds_bytes<D>(a.P) + gr * kGroupLds<D, NT>;
    float *rt = reinterpret_cast<float *>(work + wave * kWkTile);
    uint16_t *pz = reinterpret_cast<uint16_t *>(work + NW * kWkTile);   // [D] zero points, then [D] scales
    float *pinv = reinterpret_cast<float *>(pz + 2 * D);
    const __half *Mg = a.patterns + (int64_t)a.sets.set_of(ns) * a.P * D;
    take_sequence_entry(a, ns);
    const StreamMap map = a.map.of(ns);
    const int n_tiles = a.nq / TT;
    const int tile0 = chunk_of_workgroup() * tiles_per_wg, tile1 = min(n_tiles, tile0 + tiles_per_wg);
    if (tile0 >= n_tiles) return;   // a ragged append: this sequence has fewer tiles than the launch was sized for
    uint4 xb[NT][KS];
#pragma unroll
    for (int j = 0; j < NT; ++j) load_tile(a, ns, min(tile0 + gr, tile1 - 1) * TT + (wave * NT + j) * 16, xb[j]);   // in flight while the table is staged
    stage_patterns<D>(Mg, a.P, sh.tab, sh.nh, sh.red, NTH * GR);
    const PatternTable tb = make_table<NW * GR>(sh, a.P);

    for (int tile_base = tile0; tile_base < tile1; tile_base += GR) {
        // (a group past the range repeats the last one, up to the barriers, and stores nothing)
        const bool live = GR == 1 || tile_base + gr < tile1;
        const int tile = live ? tile_base + gr : tile1 - 1;
        const int64_t pq0 = map.pos(a.t0 + tile * TT);   // where the group's first token is stored
        int bi[NT];
        if (a.idx_given) {   // searched beforehand (min-max metric)
#pragma unroll
            for (int j = 0; j < NT; ++j) bi[j] = a.idx[pq0 + (wave * NT + j) * 16 + n];
        } else {
            float bv[NT], x2[NT];
            bool flag[NT];
            assign_tiles_mfma<NT, KS>(xb, tb, lane, bi, bv, x2, flag);
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                float bd;
                resolve_flagged(xb[j], flag[j], reinterpret_cast<__half *>(rt), tb, lane, 0, bi[j], bd);
            }
        }
        float mn[KS], mx[KS];
        ChannelScan scan = {};
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            mn[k] = INFINITY;
            mx[k] = -INFINITY;
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                float r[8];
                residuals8(xb[j][k], *reinterpret_cast<const uint4 *>(sh.tab + bi[j] * kTabStrideOf<D> + 8 * kb + 32 * k), r);
                scan.step(r, rt, mn[k], mx[k]);
            }
        }
        scan.use();
#pragma unroll
        for (int k = 0; k < KS; ++k) {   // the two token halves: minima in the lower half of the lanes, maxima in the upper one
            const rows2 v = swap32(bits_of(mn[k]), bits_of(mx[k]));
            const float lo = op_rows(v, MinF()), hi = op_rows(v, MaxF());
            rt[(lane < 32 ? 0 : D) + 32 * k + (lane & 31)] = lane < 32 ? lo : hi;
        }
        __syncthreads();
        for (int c = tid; c < D; c += NTH) {
            const float *all = reinterpret_cast<const float *>(work) + c;
            float lo = all[0], hi = all[D];
#pragma unroll
            for (int w = 1; w < NW; ++w) {
                lo = fminf(lo, all[w * (kWkTile / 4)]);
                hi = fmaxf(hi, all[w * (kWkTile / 4) + D]);
            }
            put_params(lo, hi, BITS, c, D, pz, pinv);
        }
        __syncthreads();
        if (!live) continue;   // (the last round: no barrier follows)
        if (wave == NW - 1) store_params<D>(a, pq0 / TT, pz);
        // codes; a tile's 16 tokens are put together in the wave's own LDS tile (read by nobody else any more)
        uint8_t *stg = reinterpret_cast<uint8_t *>(rt);
#pragma unroll
        for (int j = 0; j < NT; ++j) {
#pragma unroll
            for (int k = 0; k < KS; ++k) {
                float r[8];
                residuals8(xb[j][k], *reinterpret_cast<const uint4 *>(sh.tab + bi[j] * kTabStrideOf<D> + 8 * kb + 32 * k), r);
                k_codes8<D, BITS>(r, k, pz, pinv, stg);
            }
            if (kb == 0) stg[16 * D * BITS / 8 + n] = (uint8_t)bi[j];
            wave_lds_sync();
            if (tile_base + GR < tile1) load_tile(a, ns, min(tile + GR, tile1 - 1) * TT + (wave * NT + j) * 16, xb[j]);
            k_store_staging<D, BITS>(a, pq0 + (wave * NT + j) * 16, stg);
            wave_lds_sync();
        }
        // (the parameters are rewritten only behind the next group's first barrier, which every wave has to reach)
    }
}

// K, groups of 32 or 64 tokens: a wave owns whole groups, so nothing but the pattern table is shared in
// the workgroup and no workgroup barrier is needed after it is staged.  The group's NTG = G/16 tiles stay
// in registers as loaded (fp16); pass A assigns every tile and feeds its residuals, 32 channels at a time,
// through a small LDS tile to a per-channel running minimum / maximum, pass B forms the residuals again,
// quantizes and stores.  A tile's registers are refilled with the wave's next group as soon as pass B
// has used them.
template <int D>
constexpr int kWkWave = kWkTile + kKParams<D>;   // bytes of LDS per wave

template <int D, int G, int BITS, int NTA, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(D == 256 && G == 64 ? 2 : 3))) void quantize_k_wave_kernel(QuantKernelArgs a, int tiles_per_wg)
{
    constexpr int NTG = G / 16, KS = D / 32;
    static_assert(G == 32 || G == 64, "a wave holds the group's tiles in registers");
    extern __shared__ __align__(16) unsigned char smem[];
    const TableLds sh = table_lds<D>(smem, a.P);
    const int tid = threadIdx.x, ns = blockIdx.y;
    const int lane = tid & 63, n = lane & 15, kb = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    unsigned char *mine = smem + table_lds_bytes<D>(a.P) + (size_t)wave * kWkWave<D>;
    float *rt = reinterpret_cast<float *>(mine);
    uint16_t *pz = reinterpret_cast<uint16_t *>(mine + kWkTile);   // [D] zero points, then [D] scales
    float *pinv = reinterpret_cast<float *>(mine + kWkTile + D * 2 * 2);

    const __half *Mg = a.patterns + (int64_t)a.sets.set_of(ns) * a.P * D;
    take_sequence_entry(a, ns);
    const StreamMap map = a.map.of(ns);
    const int n_tiles = a.nq / 64;
    const int tile0 = chunk_of_workgroup() * tiles_per_wg, tile1 = min(n_tiles, tile0 + tiles_per_wg);
    if (tile0 >= n_tiles) return;   // a ragged append: this sequence has fewer tiles than the launch was sized for
    const int g_end = tile1 * (64 / G);
    int g = tile0 * (64 / G) + wave;
    uint4 xb[NTG][KS];
    if (g < g_end) {
#pragma unroll
        for (int j = 0; j < NTG; ++j) load_tile(a, ns, g * G + j * 16, xb[j]);   // in flight while the table is staged
    }
    stage_patterns<D>(Mg, a.P, sh.tab, sh.nh, sh.red, 64 * NW);
    const PatternTable tb = make_table<NW>(sh, a.P);

    for (; g < g_end; g += NW) {
        const int64_t tq0 = (int64_t)a.t0 + (int64_t)g * G;   // logical position of the group's first token
        const int64_t pq0 = map.pos((int)tq0);            // where it is stored
        // ---- pass A: indices; running minimum / maximum per channel
        float mn[KS], mx[KS];
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            mn[k] = INFINITY;
            mx[k] = -INFINITY;
        }
        int bi[NTG];
        ChannelScan scan = {};
        if (a.idx_given) {   // searched beforehand (min-max metric)
#pragma unroll
            for (int j = 0; j < NTG; ++j) bi[j] = a.idx[pq0 + j * 16 + n];
        } else if (NTA > 1) {   // NTA tiles of the group per pass over the pattern table
#pragma unroll
            for (int j0 = 0; j0 < NTG; j0 += NTA) {
                float bv[NTA], x2[NTA];
                bool flag[NTA];
                int bj[NTA];
                assign_tiles_mfma<NTA, KS>(reinterpret_cast<const uint4 (&)[NTA][KS]>(xb[j0]), tb, lane, bj, bv, x2, flag);
#pragma unroll
                for (int j = 0; j < NTA; ++j) {
                    float bd;
                    resolve_flagged(xb[j0 + j], flag[j], reinterpret_cast<__half *>(rt), tb, lane, 0, bj[j], bd);
                    bi[j0 + j] = bj[j];
                }
            }
        }
#pragma unroll
        for (int j = 0; j < NTG; ++j) {
            if (NTA == 1 && !a.idx_given) bi[j] = assign_index(tb, xb[j], reinterpret_cast<__half *>(rt));
            if constexpr (KS <= 4) {
                float r[8 * KS];
                residuals(sh, xb[j], bi[j], r);
#pragma unroll
                for (int k = 0; k < KS; ++k) scan.step(r + 8 * k, rt, mn[k], mx[k]);
            } else {   // 256 channels: the tiles alone take half of the registers
#pragma unroll
                for (int k = 0; k < KS; ++k) {
                    float r[8];
                    residuals8(xb[j][k], *reinterpret_cast<const uint4 *>(sh.tab + bi[j] * kTabStrideOf<D> + 8 * kb + 32 * k), r);
                    scan.step(r, rt, mn[k], mx[k]);
                }
            }
        }
        scan.use();
        // ---- parameters of the group: the two token halves are combined, lane (c, half) gets the channels
        //      32(2h + half) + c
        const int sc = lane & 31, sth = lane >> 5;
#pragma unroll
        for (int h = 0; h < (KS + 1) / 2; ++h) {
            constexpr int last = KS - 1;
            const int k1 = 2 * h + 1 < KS ? 2 * h + 1 : last;
            const float lo = op_rows(swap32(bits_of(mn[2 * h]), bits_of(mn[k1])), MinF());
            const float hi = op_rows(swap32(bits_of(mx[2 * h]), bits_of(mx[k1])), MaxF());
            if (KS % 2 == 0 || 2 * h + 1 < KS || sth == 0) put_params(lo, hi, BITS, 32 * (2 * h + sth) + sc, D, pz, pinv);
        }
        wave_lds_sync();
        store_params<D>(a, pq0 / G, pz);
        // ---- pass B: residuals again, codes, planes; the tile's registers then take the next group
        uint8_t *stg = reinterpret_cast<uint8_t *>(rt);
#pragma unroll
        for (int j = 0; j < NTG; ++j) {
            if constexpr (KS <= 4) {
                float r[8 * KS];
                residuals(sh, xb[j], bi[j], r);
                if (g + NW < g_end) load_tile(a, ns, (g + NW) * G + j * 16, xb[j]);
#pragma unroll
                for (int k = 0; k < KS; ++k) k_codes8<D, BITS>(r + 8 * k, k, pz, pinv, stg);
            } else {
#pragma unroll
                for (int k = 0; k < KS; ++k) {
                    float r[8];
                    residuals8(xb[j][k], *reinterpret_cast<const uint4 *>(sh.tab + bi[j] * kTabStrideOf<D> + 8 * kb + 32 * k), r);
                    k_codes8<D, BITS>(r, k, pz, pinv, stg);
                }
                if (g + NW < g_end) load_tile(a, ns, (g + NW) * G + j * 16, xb[j]);
            }
            if (kb == 0) stg[16 * D * BITS / 8 + n] = (uint8_t)bi[j];
            wave_lds_sync();
            k_store_staging<D, BITS>(a, pq0 + j * 16, stg);
            wave_lds_sync();   // the staging area is rewritten by the next tile
        }
    }
}

// ---- V ------------------------------------------------------------------------------------------------------------
// Per-wave output staging: the pieces a wave produces for its 16 tokens are put together in LDS so that
// every global store is one contiguous run of 8- or 16-byte lane pieces.
// The vector under exact re-evaluation takes the codes' place (the finished unit that waits there is stored first: one token in several
// hundred is re-evaluated), so that four workgroups fit a CU beside tables of up to 128 patterns of 128 channels: 512 streams x 32640
// vectors 1410 -> 1280 us (3.4 -> 3.9 TB/s), 256 x 8192 at 64 patterns 187 -> 170.
template <int D, int BITS, int NG>
struct VStaging {
    static constexpr int kCodes = 0;                   // the unit's code words in memory order; D halves: one vector for the exact re-evaluation
    static constexpr int kIdx = 2 * D * BITS;          // 16 B: pattern indices
    static constexpr int kScale = kIdx + 16;           // scales [group][16]
    static constexpr int kZero = kScale + 32 * NG;     // zero points [group][16]
    static constexpr int kBytes = kZero + 32 * NG;
};

// 16x16 bit transpose across the 16 lanes of a row, on both 16-bit halves of x at once:
// on return bit t of a half in lane i is what bit i of that half was in lane t.  The partner's word comes by lane permutations inside
// the row, folded into the mask operation (permutes through LDS left a wave waiting for four of them in turn: 512 streams x 32640 vectors
// 1465 -> 1406 us, 4-bit codes over 32-channel groups 217 -> 201).
struct TransposeConst {
    uint32_t sh[4], keep[4];   // stage d = 8, 4, 2, 1: rotation of the partner's bits; bits kept of the own word, which are also the places
                               // of those that the partner's word gives, before the rotation
};
__device__ __forceinline__ TransposeConst transpose_const(int n)
{
    TransposeConst c;
    const uint32_t m0[4] = {0x00ff00ffu, 0x0f0f0f0fu, 0x33333333u, 0x55555555u};   // positions with bit d clear
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int d = 8 >> s;
        const bool lo = (n & d) == 0;
        c.sh[s] = lo ? 32 - d : d;        // lo lanes take the partner's bits d places up, hi lanes d places down
        c.keep[s] = lo ? m0[s] : ~m0[s];
    }
    return c;
}
__device__ __forceinline__ uint32_t transpose16(uint32_t x, const TransposeConst &c)
{
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        // lane n ^ 8: a rotation of the row; n ^ 4: n ^ 7 (mirrored half row), then ^ 3; n ^ 2, n ^ 1: inside quads
        const uint32_t partner = s == 0 ? dpp<0x128>(x) : s == 1 ? dpp<0x1b>(dpp<0x141>(x)) : s == 2 ? dpp<0x4e>(x) : dpp<0xb1>(x);
        const uint32_t t = partner & c.keep[s];
        x = __builtin_amdgcn_bitop3_b32(x, c.keep[s], __builtin_amdgcn_alignbit(t, t, c.sh[s]), 0xea);   // (x & keep) | rotated: the fast three-input form
    }
    return x;
}

// V: workgroup = NW waves (4, 8 or 12), blocks of 64 tokens of one stream; wave w owns the 16-token unit w % 4 of its blocks, and
// waves 4i .. 4i + 3 take the i-th NT blocks of a round of NW / 4 * NT.  NG = channel groups per token (D / Gc).  NT = blocks taken
// together: the wave assigns its units of NT consecutive blocks in one pass over the pattern table (every table tile read
// from LDS serves all of them), then quantizes them one after the other.
template <int D, int BITS, int NG, int NT, int NW>
__global__ __launch_bounds__(64 * NW) void quantize_v_kernel(QuantKernelArgs a, int tiles_per_wg)
{
    using St = VStaging<D, BITS, NG>;
    constexpr int TT = 64, WPU = BITS / 2, KS = D / 32, BPG = KS / NG;   // BPG = 32-channel blocks per group
    static_assert(KS % NG == 0, "groups of whole 32-channel blocks");
    constexpr int GL = (NG + 3) / 4;   // groups whose parameters a lane works out
    extern __shared__ __align__(16) unsigned char smem[];
    const TableLds sh = table_lds<D>(smem, a.P);
    const int tid = threadIdx.x, ns = blockIdx.y;
    const int lane = tid & 63, n = lane & 15, kb = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const __half *Mg = a.patterns + (int64_t)a.sets.set_of(ns) * a.P * D;
    take_sequence_entry(a, ns);
    const StreamMap map = a.map.of(ns);
    const int n_tiles = a.nq / TT;
    const int tile0 = chunk_of_workgroup() * tiles_per_wg, tile1 = min(n_tiles, tile0 + tiles_per_wg);
    if (tile0 >= n_tiles) return;   // a ragged append: this sequence has fewer tiles than the launch was sized for
    const int unit = wave % 4 * 16, first = tile0 + wave / 4 * NT;   // the wave's unit of its blocks, its first block
    constexpr int kRound = NW / 4 * NT;                              // blocks that the workgroup takes at a time
    uint4 xbs[NT][KS];
#pragma unroll
    for (int j = 0; j < NT; ++j)   // a block past the workgroup's range repeats the last one; its result is not used
        load_tile(a, ns, min(first + j, tile1 - 1) * TT + unit, xbs[j]);

    stage_patterns<D>(Mg, a.P, sh.tab, sh.nh, sh.red, 64 * NW);
    const PatternTable tb = make_table<NW>(sh, a.P);
    const TransposeConst tc = transpose_const(n);
    unsigned char *wsc = smem + table_lds_bytes<D>(a.P) + wave * St::kBytes;

    // Contiguous stores of a finished unit (code words, parameters, indices) out of the wave's staging area.
    // They are issued at the start of the NEXT unit, after that unit's vectors have arrived and before the
    // loads for the one after are issued: the wait for those loads at the top of a round would otherwise also
    // wait for stores issued just before it (loads and stores retire through one in-order counter).
    int64_t pend_tok0 = -1;
    auto store_pending = [&]() {
        if (pend_tok0 < 0) return;
        const int64_t tok0 = pend_tok0;
        wave_store<16 * D * BITS / 8>(a.codes_v + tok0 * (D * BITS / 8), wsc + St::kCodes);
        if (lane < 4 * NG) {   // NG*32 bytes per array = 2*NG pieces of 16 bytes; scales first, then zero points
            const int arr = lane / (2 * NG), piece = lane % (2 * NG);
            const uint4 v = *reinterpret_cast<const uint4 *>(wsc + (arr ? St::kZero : St::kScale) + piece * 16);
            *reinterpret_cast<uint4 *>((arr ? a.zero : a.scale) + tok0 * NG + piece * 8) = v;
        }
        if (lane == 63) *reinterpret_cast<uint4 *>(a.idx + tok0) = *reinterpret_cast<const uint4 *>(wsc + St::kIdx);
        wave_lds_sync();   // the staging area is rewritten by the unit that follows
        pend_tok0 = -1;
    };

    for (int tile_base = first; tile_base < tile1; tile_base += kRound) {
        int bis[NT];
        if (a.idx_given) {   // searched beforehand (min-max metric); a block past the range repeats the last one
#pragma unroll
            for (int j = 0; j < NT; ++j)
                bis[j] = a.idx[map.pos(a.t0 + min(tile_base + j, tile1 - 1) * TT) + unit + n];
        } else {
            float bv[NT], x2[NT];
            bool flag[NT];
            assign_tiles_mfma<NT, KS>(xbs, tb, lane, bis, bv, x2, flag);
            bool any = flag[0];
#pragma unroll
            for (int j = 1; j < NT; ++j) any = any || flag[j];
            if (__ballot(any) != 0ull) {
                store_pending();   // the vector under re-evaluation takes the codes' place
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    float bd;
                    resolve_flagged(xbs[j], flag[j], reinterpret_cast<__half *>(wsc + St::kCodes), tb, lane, 0, bis[j], bd);
                }
            }
        }
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        const int tile = tile_base + j;
        if (tile >= tile1) break;
        uint4 (&xb)[KS] = xbs[j];
        float r[8 * KS];
        int bi = bis[j];
        store_pending();
        residuals(sh, xb, bi, r);
        if (a.v_rho > 0.f) {
            // adaptive threshold (Sec. 3.3): keep the pattern iff R_flat <= rho * R_raw, ranges over all d
            // channels of the token: lane-local over its channels, then over the token's 4 lanes
            float rmn = fminf(r[0], r[1]), rmx = fmaxf(r[0], r[1]);
            half2_t xmn = __builtin_bit_cast(half2_t, xb[0].x), xmx = xmn;
#pragma unroll
            for (int e = 2; e < 8 * KS; e += 2) {
                rmn = fminf(fminf(rmn, r[e]), r[e + 1]);
                rmx = fmaxf(fmaxf(rmx, r[e]), r[e + 1]);
            }
#pragma unroll
            for (int k = 0; k < KS; ++k) {
                const uint32_t w[4] = {xb[k].x, xb[k].y, xb[k].z, xb[k].w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    xmn = __builtin_elementwise_min(xmn, __builtin_bit_cast(half2_t, w[i]));
                    xmx = __builtin_elementwise_max(xmx, __builtin_bit_cast(half2_t, w[i]));
                }
            }
            float x_lo = fminf((float)xmn[0], (float)xmn[1]), x_hi = fmaxf((float)xmx[0], (float)xmx[1]);
            // (even rows: of the residual, odd rows: of the vector)
            const float lows[2] = {rmn, x_lo}, highs[2] = {rmx, x_hi};
            float range[2];
            spread_rows<2>(fold_rows<2>(highs, MaxF()) - fold_rows<2>(lows, MinF()), range);
            const bool keep = range[0] <= a.v_rho * range[1];
            if (!keep) {   // quantize the vector itself
                bi = PK_NO_PATTERN;
#pragma unroll
                for (int k = 0; k < KS; ++k) {
                    const uint32_t w[4] = {xb[k].x, xb[k].y, xb[k].z, xb[k].w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const half2_t h = __builtin_bit_cast(half2_t, w[i]);
                        r[8 * k + 2 * i] = (float)h[0];
                        r[8 * k + 2 * i + 1] = (float)h[1];
                    }
                }
            }
        }
        if (tile + kRound < tile1) load_tile(a, ns, (tile + kRound) * TT + unit, xb);   // else the registers keep this block

        // minimum / maximum per channel group: lane-local over its channels here, then over the 4 lanes of the token
        float mn[NG], mx[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            mn[g] = INFINITY;
            mx[g] = -INFINITY;
#pragma unroll
            for (int e = 8 * BPG * g; e < 8 * BPG * (g + 1); e += 2) {
                mn[g] = fminf(fminf(mn[g], r[e]), r[e + 1]);
                mx[g] = fmaxf(fmaxf(mx[g], r[e]), r[e + 1]);
            }
        }
        // row kb works out the parameters of group kb % NG (eight groups: of kb and kb + 4) and stores them; the others
        // fetch them
        float z[NG], inv[NG];
#pragma unroll
        for (int l = 0; l < GL; ++l) {
            constexpr int NF = NG == 3 || NG > 4 ? 4 : NG;   // groups folded together (three: the first one twice)
            float lows[NF], highs[NF], zs[NF], invs[NF];
#pragma unroll
            for (int i = 0; i < NF; ++i) {
                lows[i] = mn[4 * l + i < NG ? 4 * l + i : 0];
                highs[i] = mx[4 * l + i < NG ? 4 * l + i : 0];
            }
            const GroupParams gp = group_params(fold_rows<NF>(lows, MinF()), fold_rows<NF>(highs, MaxF()), BITS);
            if (kb + 4 * l < NG) {
                reinterpret_cast<uint16_t *>(wsc + St::kScale)[(kb + 4 * l) * 16 + n] = gp.s16;
                reinterpret_cast<uint16_t *>(wsc + St::kZero)[(kb + 4 * l) * 16 + n] = gp.z16;
            }
            spread_rows<NF>(gp.z, zs);
            spread_rows<NF>(gp.inv, invs);
#pragma unroll
            for (int i = 0; i < NF; ++i) {
                if (4 * l + i < NG) {
                    z[4 * l + i] = zs[i];
                    inv[4 * l + i] = invs[i];
                }
            }
        }
        if (kb == 0) wsc[St::kIdx + n] = (uint8_t)bi;

        // block b = channels 32*(2b + i/8) + 8*kb + i%8, i < 16: codes -> planes -> transpose -> words, put in
        // memory order in the wave's staging area.  (96 channels: the last block has eight channels per lane.)
        uint32_t *stg = reinterpret_cast<uint32_t *>(wsc + St::kCodes);
#pragma unroll
        for (int b = 0; b < (KS + 1) / 2; ++b) {
            constexpr int kAll = 8 * KS;
            uint32_t cw[4] = {0u, 0u, 0u, 0u};   // codes of elements 4q .. 4q+3 in the bytes of cw[q]
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int e = 16 * b + i < kAll ? 16 * b + i : kAll - 1, g = (e / 8) / BPG;
                if (16 * b + i < kAll) cw[i >> 2] = put_code(r[e] - z[g], inv[g], i & 3, cw[i >> 2]);
            }
            // channel of this lane after the transpose: i = n
            const int c = 32 * (2 * b + (n >> 3)) + 8 * kb + (n & 7);
            uint32_t *dst = stg + ((c & 15) * (D / 16) + (c >> 4)) * WPU;
            if constexpr (BITS == 2) {
                // sums of code << i and of (code & 2) << i over the sixteen codes, twice plane 1; their difference is plane 0
                const uint32_t all = (byte_sum(cw[2], cw[3]) << 8) + byte_sum(cw[0], cw[1]);
                const uint32_t hi2 = (plane_byte_shifted(cw[2], cw[3], 1) << 8) + plane_byte_shifted(cw[0], cw[1], 1);
                const uint32_t word = transpose16(__umul24(hi2, 32767u) + all, tc);   // all - hi2 + (hi2 / 2 << 16)
                if (16 * b + 16 <= kAll || n < 8) dst[0] = word;
            } else {
#pragma unroll
                for (int w = 0; w < WPU; ++w) {
                    // t_p = (bits p of the 16 codes) << p; low half of x = plane 2w, high half = plane 2w+1
                    const uint32_t t0 = (plane_byte_shifted(cw[2], cw[3], 2 * w) << 8) | plane_byte_shifted(cw[0], cw[1], 2 * w);
                    const uint32_t t1 = (plane_byte_shifted(cw[2], cw[3], 2 * w + 1) << 8) | plane_byte_shifted(cw[0], cw[1], 2 * w + 1);
                    const uint32_t x = (t0 >> (2 * w)) | (t1 << (15 - 2 * w));
                    const uint32_t word = transpose16(x, tc);
                    if (16 * b + 16 <= kAll || n < 8) dst[w] = word;
                }
            }
        }
        wave_lds_sync();
        pend_tok0 = map.pos(a.t0 + tile * TT) + unit;   // stored at the start of the next unit
      }
    }
    store_pending();
}

// ---------------------------------------------------------------------------
// Tail ring: place logical vectors [i0, i1) of an append into their ring slots.
// ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void tail_copy_kernel(TailCopyArgs a)
{
    constexpr int kPieces = D / 8;   // 16-byte pieces of a vector
    const int n = blockIdx.y, side = blockIdx.z;
    if (a.seq_table) {   // a ragged append: the ring state and the range of the stream's own sequence
        const int32_t *e = a.seq_table + (int64_t)(n / a.n_kv_heads) * kSeqEntry;
        a.ring_start = e[kSeqRingStart];
        a.n_ring = e[kSeqNRing];
        a.i0 = e[kSeqI0];
        a.i1 = e[kSeqI1];
    }
    int i, ch;   // (the pieces of a ring may be more than 32 bits count, its vectors are not)
    if constexpr (256 % kPieces == 0) {
        i = a.i0 + (int)(blockIdx.x * (256 / kPieces) + threadIdx.x / kPieces);
        ch = threadIdx.x % kPieces;
    } else {
        const uint64_t w = (uint64_t)blockIdx.x * 256 + threadIdx.x;
        i = a.i0 + (int)(w / kPieces);
        ch = (int)(w % kPieces);
    }
    if (i >= a.i1) return;
    const __half *fresh = side == 0 ? a.fresh_k : a.fresh_v;
    __half *ring = side == 0 ? a.ring_k : a.ring_v;
    const uint4 v = *reinterpret_cast<const uint4 *>(fresh + (int64_t)n * a.fresh_stride +
                                                     (int64_t)(i - a.n_ring) * D + ch * 8);
    const int slot = (int)(((int64_t)a.ring_start + i) % a.ring_len);
    *reinterpret_cast<uint4 *>(ring + ((int64_t)n * a.ring_len + slot) * D + ch * 8) = v;
}

__global__ __launch_bounds__(kSeqChunk * kSeqEntry) void seq_table_kernel(SeqTableArgs a)
{
    const int i = threadIdx.x / kSeqEntry, f = threadIdx.x % kSeqEntry;
    if (i >= a.count) return;
    a.table[(int64_t)(a.first + i) * kSeqEntry + f] = a.entry[i][f];
    if (a.states_out && f < 4) a.states_out[(int64_t)(a.first + i) * 4 + f] = f < 3 ? a.state[i][f] : 0;
}

}  // namespace

hipError_t launch_seq_table(const SeqTableArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(seq_table_kernel, dim3(1), dim3(kSeqChunk * kSeqEntry), 0, s, a);
    return hipGetLastError();
}

// Workgroups of at most `tiles` tiles of one stream each.  max_lds: the most that the instantiation is launched with.
template <auto KERNEL, int THREADS = 256>
static hipError_t launch_tiled(const QuantArgs &a, int TT, size_t lds, size_t max_lds, hipStream_t s, int tiles)
{
    static LdsOptIn opt_in;
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(KERNEL), opt_in, max_lds);
    if (e != hipSuccess) return e;
    const int chunks = (a.nq / TT + tiles - 1) / tiles;
    hipLaunchKernelGGL(KERNEL, dim3(chunks, a.n_streams), dim3(THREADS), lds, s, a, tiles);
    return hipGetLastError();
}

// Min-max metric: the search kernel fills the index array, the quantizers then take the indices from there.
template <int D>
static hipError_t launch_minmax(const QuantArgs &a, hipStream_t s)
{
    const int n_tiles = a.nq / 64;
    int tpw = tiles_per_wg(n_tiles, a.n_streams);
    if (tpw < 4) tpw = 4;   // four waves, a 64-vector tile each per round
    hipLaunchKernelGGL(assign_minmax_kernel<D>, dim3((n_tiles + tpw - 1) / tpw, a.n_streams), dim3(256), 0, s, a, tpw);
    return hipGetLastError();
}

static hipError_t launch_assign_minmax(const QuantArgs &a, hipStream_t s)
{
    return a.d == kD ? launch_minmax<kD>(a, s) : a.d == 96 ? launch_minmax<96>(a, s) : launch_minmax<256>(a, s);
}

// Tiles per pass over the pattern table and launch sizes follow the table: every table tile read from LDS serves all the
// 16-token tiles of a pass.  A large table (beyond 128 patterns, or 64 of 256 channels) leaves room for one or two
// workgroups per CU, each of which stages up to 128 KB: what a launch takes then hangs on how many workgroups every CU gets.
template <int D>
static bool large_table(int P)
{
    return P > (D == 256 ? 64 : 128);
}

// multiple: tiles that the workgroup takes side by side; waves_per_cu: what registers allow
static Cut cut_job(const QuantArgs &a, int TT, size_t lds, int waves, int waves_per_cu, int multiple, bool pairs = false)
{
    const Job j = {a.nq / TT, a.n_streams, a.n_vectors / TT, a.seq_table != nullptr, 256.f / TT};
    return (pairs ? cut_pairs : cut_streams)(j, (int)(163840 / lds), waves, waves_per_cu, multiple);
}

template <int D, int G, int BITS, int NTA, int NW>
struct KWaves {
    static constexpr int kMultiple = NW * G / 64 > 0 ? NW * G / 64 : 1;   // a wave owns whole groups: one group per wave at a time
    static size_t lds(int P) { return table_lds_bytes<D>(P) + NW * (size_t)kWkWave<D>; }
    static Cut cut(const QuantArgs &a) { return cut_job(a, 64, lds(a.P), NW, D == 256 && G == 64 ? 8 : 12, kMultiple); }
    static hipError_t launch(const QuantArgs &a, hipStream_t s, int tiles)
    {
        return launch_tiled<quantize_k_wave_kernel<D, G, BITS, NTA, NW>, 64 * NW>(a, 64, lds(a.P), lds(D == 256 && NW > 4 ? 128 : 256), s, tiles);
    }
    static hipError_t launch(const QuantArgs &a, hipStream_t s)   // small tables
    {
        const int t = max(tiles_per_wg(a.nq / 64, a.n_streams), kMultiple);
        return launch(a, s, (t + kMultiple - 1) / kMultiple * kMultiple);
    }
};

// Large tables: four waves per workgroup, or as many as registers allow per CU, whichever cut is modelled to take less.  Twelve (eight
// with 64-token groups of 256 channels) pay where the table leaves room for one workgroup only, which with four has one wave per SIMD
// (288 streams x 64 vectors at 256 patterns 25.7 us with twelve, 27.3 with four; x 4096: 169 and 234), not where two of four fit (at
// 200 patterns 22 and 14, 154 and 152) unless twelve make a whole round (256 streams x 4096: 112 and 119), and not in small jobs, whose
// workgroups are then too few (8 x 4096 at 256 patterns 26 and 16).
// (The V quantizer's of 256 channels likewise.)
template <class MANY, class FOUR>
static hipError_t launch_cheaper(const QuantArgs &a, hipStream_t s)
{
    const Cut many = MANY::cut(a), four = FOUR::cut(a);
    return many.cost < four.cost ? MANY::launch(a, s, many.tiles) : FOUR::launch(a, s, four.tiles);
}

template <int D, int G, int BITS>
static hipError_t launch_k_wave(const QuantArgs &a, hipStream_t s)
{
    if constexpr (D == 256) {      // (64-token groups: the tiles of a group take 128 registers, so pairs at most)
        using Four = KWaves<D, G, BITS, 2, 4>;
        if (a.P > 128) return Four::launch(a, s, Four::cut(a).tiles);   // (more waves don't fit beside the table)
        if (large_table<D>(a.P)) return launch_cheaper<KWaves<D, G, BITS, 2, 8>, Four>(a, s);
        return Four::launch(a, s);
    } else if constexpr (G == 64) {   // the whole group per table pass (256 x 8192 at 64 patterns 220 -> 187 us); pairs up to 32 patterns
        if (large_table<D>(a.P)) return launch_cheaper<KWaves<D, G, BITS, 4, 12>, KWaves<D, G, BITS, 4, 4>>(a, s);
        return a.P > 32 ? KWaves<D, G, BITS, 4, 4>::launch(a, s) : KWaves<D, G, BITS, 2, 4>::launch(a, s);
    } else {                          // 32-token groups gain from pairs only once the table is large
        if (large_table<D>(a.P)) return launch_cheaper<KWaves<D, G, BITS, 2, 12>, KWaves<D, G, BITS, 2, 4>>(a, s);
        return a.P >= 128 ? KWaves<D, G, BITS, 2, 4>::launch(a, s) : KWaves<D, G, BITS, 1, 4>::launch(a, s);
    }
}

template <int D, int BITS, int GR, int NT>
struct KGroups {   // GR groups of 128 tokens side by side
    static size_t lds(int P) { return table_lds_bytes<D>(P) + GR * (size_t)kGroupLds<D, NT>; }
    static Cut cut(const QuantArgs &a) { return cut_job(a, 128, lds(a.P), 8 / NT * GR, 16, GR); }
    static hipError_t launch(const QuantArgs &a, hipStream_t s, int tiles)
    {
        return launch_tiled<quantize_k_group_kernel<D, BITS, GR, NT>, 512 / NT * GR>(a, 128, lds(a.P), lds(D == 256 && GR > 1 ? 128 : 256), s, tiles);
    }
};

template <int D, int BITS>
static hipError_t launch_k_bits(const QuantArgs &a, hipStream_t s)
{
    if (a.G == 32) return launch_k_wave<D, 32, BITS>(a, s);
    if constexpr (D != 96) {   // (64 does not divide 96 channels)
        if (a.G == 64) return launch_k_wave<D, 64, BITS>(a, s);
    }
    using One = KGroups<D, BITS, 1, 1>;
    if (!large_table<D>(a.P)) return One::launch(a, s, tiles_per_wg(a.nq / 128, a.n_streams));
    if constexpr (D == 256) {
        const Cut one = One::cut(a);
        if (a.P <= 128 && a.nq >= 256) {
            using Two = KGroups<D, BITS, 2, 1>;
            const Cut two = Two::cut(a);
            if (two.cost < one.cost) return Two::launch(a, s, two.tiles);
        }
        return One::launch(a, s, one.tiles);
    } else {   // four groups, or two of twice the waves where workgroups are short
        using Two = KGroups<D, BITS, 2, 1>;
        using Four = KGroups<D, BITS, 4, 2>;
        const Cut two = Two::cut(a);
        return two.tiles >= 4 ? Four::launch(a, s, Four::cut(a).tiles) : Two::launch(a, s, two.tiles);
    }
}

template <int D>
static hipError_t launch_k_of(const QuantArgs &a, hipStream_t s)
{
    return a.bits == 2 ? launch_k_bits<D, 2>(a, s) : launch_k_bits<D, 4>(a, s);
}

// the min-max metric's search goes ahead; the indices are then given
static hipError_t search_ahead(QuantArgs &a, hipStream_t s)
{
    if (a.metric != PK_METRIC_MINMAX) return hipSuccess;
    a.idx_given = 1;
    return launch_assign_minmax(a, s);
}

hipError_t launch_quantize_k(const QuantArgs &a_in, hipStream_t s)
{
    QuantArgs a = a_in;
    const hipError_t e = search_ahead(a, s);
    if (e != hipSuccess) return e;
    return a.d == kD ? launch_k_of<kD>(a, s) : a.d == 96 ? launch_k_of<96>(a, s) : launch_k_of<256>(a, s);
}

template <int D, int BITS, int NG, int NT, int NW>
struct VWaves {
    static constexpr int kMultiple = NW / 4 * NT;   // blocks that the workgroup takes at a time
    static size_t lds(int P) { return table_lds_bytes<D>(P) + NW * (size_t)VStaging<D, BITS, NG>::kBytes; }
    static Cut cut(const QuantArgs &a) { return cut_job(a, 64, lds(a.P), NW, D == 256 ? 12 : 16, kMultiple, NT > 1); }
    static hipError_t launch(const QuantArgs &a, hipStream_t s, int tiles)
    {
        return launch_tiled<quantize_v_kernel<D, BITS, NG, NT, NW>, 64 * NW>(a, 64, lds(a.P), lds(NW == 12 ? 128 : 256), s, tiles);
    }
};

template <int D, int BITS, int NG>
static hipError_t launch_v_groups(const QuantArgs &a, hipStream_t s)
{
    // Beside a table that leaves room for two workgroups or one: the waves per workgroup that fill a CU, or four, whichever cut is modelled
    // to take less.  Eight (256 streams x 8192 vectors at 256 patterns 222 us, 250 with four; 288 x 1024 at 200 patterns of 256 channels 83
    // and 120; 8 x 2048 at 136 of 256 17.1 and 15.2); up to 128 patterns of 256 channels twelve (at 128 patterns 512 x 4096 309 and 335; 288 x 64
    // 18 and 12).  With eight waves of up to 128 channels two blocks per table pass.
    using Plain = VWaves<D, BITS, NG, 1, 4>;
    const int blocks = a.nq / 64;
    if (large_table<D>(a.P)) {
        if constexpr (D == 256) {
            return a.P > 128 ? launch_cheaper<VWaves<D, BITS, NG, 1, 8>, Plain>(a, s) : launch_cheaper<VWaves<D, BITS, NG, 1, 12>, Plain>(a, s);
        } else {
            using Eight = VWaves<D, BITS, NG, 2, 8>;
            const Cut eight = Eight::cut(a), plain = Plain::cut(a);
            return eight_waves(eight, plain, blocks) ? Eight::launch(a, s, eight.tiles) : Plain::launch(a, s, plain.tiles);
        }
    }
    const int t = tiles_per_wg(blocks, a.n_streams);
    if constexpr (D != 256) {
        if (two_blocks_per_pass(blocks, a.n_streams, a.P, BITS, a.idx_given != 0)) return VWaves<D, BITS, NG, 2, 4>::launch(a, s, (t + 1) / 2 * 2);
    }
    return Plain::launch(a, s, t);
}

template <int D, int BITS>
static hipError_t launch_v_bits(const QuantArgs &a, hipStream_t s)
{
    if constexpr (D == 96) {
        return a.G == 32 ? launch_v_groups<D, BITS, 3>(a, s) : launch_v_groups<D, BITS, 1>(a, s);
    } else {
        return a.G == 32 ? launch_v_groups<D, BITS, D / 32>(a, s) : a.G == 64 ? launch_v_groups<D, BITS, D / 64>(a, s)
                                                                              : launch_v_groups<D, BITS, D / 128>(a, s);
    }
}

template <int D>
static hipError_t launch_v_of(const QuantArgs &a, hipStream_t s)
{
    return a.bits == 2 ? launch_v_bits<D, 2>(a, s) : launch_v_bits<D, 4>(a, s);
}

hipError_t launch_quantize_v(const QuantArgs &a_in, hipStream_t s)
{
    QuantArgs a = a_in;
    const hipError_t e = search_ahead(a, s);
    if (e != hipSuccess) return e;
    return a.d == kD ? launch_v_of<kD>(a, s) : a.d == 96 ? launch_v_of<96>(a, s) : launch_v_of<256>(a, s);
}

hipError_t launch_tail_copy(const TailCopyArgs &a, hipStream_t s)
{
    const int64_t work = (int64_t)(a.i1 - a.i0) * (a.d / 8);
    if (work <= 0) return hipSuccess;
    const dim3 grid((unsigned)((work + 255) / 256), a.n_streams, 2), block(256);
    if (a.d == kD)
        hipLaunchKernelGGL(tail_copy_kernel<kD>, grid, block, 0, s, a);
    else if (a.d == 96)
        hipLaunchKernelGGL(tail_copy_kernel<96>, grid, block, 0, s, a);
    else
        hipLaunchKernelGGL(tail_copy_kernel<256>, grid, block, 0, s, a);
    return hipGetLastError();
}

}  // namespace pk
