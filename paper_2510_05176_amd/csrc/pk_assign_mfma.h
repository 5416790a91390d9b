// Nearest-pattern search under the Euclidean metric on the matrix cores (Sec. 3.1 Eq. 4 assignment
// step; Sec. 3.2 Eq. 6 argmin in L2 mode).
//
// Ranking uses e = x.m - ||m||^2/2 - ||x||^2/2 = -||x - m||^2 / 2 from v_mfma_f32_16x16x32_f16: the
// accumulator starts at -(||m||^2 + ||x||^2)/2 and the D/32 K-steps add x.m (fp16 products are exact in
// fp32; only the accumulation rounds).  The best and second best value are tracked; a token whose gap
// between the two is not safely above the rounding error of that form is re-evaluated exactly,
// sum_c (x_c - m_c)^2 in binary32 over all patterns, lowest index on ties.  A token that is not
// re-evaluated has a gap larger than any possible ranking error, so the result always equals the
// exact argmin.
//
// Operand layout (lane = 16*kb + n):  A = patterns, row n of the 16-pattern tile, K-step s covers
// channels 32*s + 8*kb + j, KS = D/32 steps (3, 4 or 8 at head dimension 96, 128 or 256);  B = vectors, column n = token n of the 16-token tile, same channels;
// D: column n = token, rows 4*kb + i = patterns 16*tile + 4*kb + i.
#pragma once

#include "pk_internal.h"
#include "pk_lanes.h"

namespace pk {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));

// Halves per pattern row in LDS: D + 16, i.e. 8 words modulo 16 at D = 96, 128 and 256 (56, 72, 136 words), the row skew at
// which 16-byte reads of 16 rows x 4 column groups run at full rate.
template <int D>
constexpr int kTabStrideOf = D + 16;

__host__ __device__ constexpr int pad16(int p) { return (p + 15) & ~15; }

struct PatternTable {
    const __half *lds_rows;   // LDS copy, pad16(P) rows of stride kTabStrideOf<D>, rows past P are zero
    const float *nh;          // LDS [pad16(P)]: -||m_p||^2 / 2, -inf past P
    float norm2_max;          // max_p ||m_p||^2
    int P;
};

__device__ __forceinline__ floatx4_t mfma_f16(const uint4 &a, const uint4 &b, floatx4_t c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a), __builtin_bit_cast(half8_t, b), c, 0, 0, 0);
}

// Stage a pattern table into LDS (nthr threads, a multiple of 64; the loop is guarded) and compute the row norms; red_s
// gets one maximum per wave.  Ends with a barrier.
// Work item i = (row, 16-byte piece): the kLanes lanes of a row (16, or 32 at D = 256; lanes past the row's D / 8 pieces
// idle at D = 96) sum their squares.  kAhead items of a thread are requested before the first is stored: one after the other each
// waited for its own load (a step of 8 sets x 8192 vectors at 64 patterns 14.9 -> 13.3 us, an append of 4 x 131072 vectors at 256 patterns
// 160 -> 155 us).
template <int D = kD>
__device__ __forceinline__ void stage_patterns(const __half *Mg, int P, __half *tab_s, float *nh_s, float *red_s,
                                               int nthr = 256)
{
    constexpr int kLanes = D <= 128 ? 16 : 32, kPieces = D / 8, kStride = kTabStrideOf<D>, kAhead = 8;
    const int tid = threadIdx.x, total = pad16(P) * kLanes;
    float mx = 0.f;
    // total is a multiple of 256, and every kLanes consecutive work items sit in one wave: the row sums
    // below see whole rows (a trailing half round of a 512-thread group has whole waves idle)
    for (int i0 = tid; i0 < total; i0 += kAhead * nthr) {
        uint4 v[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int i = i0 + u * nthr, r = i / kLanes, ch = i % kLanes;
            v[u] = make_uint4(0u, 0u, 0u, 0u);
            if (r < P && (kPieces == kLanes || ch < kPieces)) v[u] = *reinterpret_cast<const uint4 *>(Mg + (int64_t)r * D + ch * 8);
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int i = i0 + u * nthr, r = i / kLanes, ch = i % kLanes;
            if (i >= total) break;
            if (kPieces == kLanes || ch < kPieces) *reinterpret_cast<uint4 *>(tab_s + r * kStride + ch * 8) = v[u];   // rows past P are zero
            const half2_t *h = reinterpret_cast<const half2_t *>(&v[u]);
            float acc = 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k) acc = __builtin_amdgcn_fdot2(h[k], h[k], acc, false);
            acc = row_sum(acc);
            if (kLanes == 32) acc = op_rows(swap16(bits_of(acc), bits_of(acc)), AddF());
            if (ch == 0) nh_s[r] = r < P ? -0.5f * acc : -INFINITY;   // rows past the table never win
            mx = fmaxf(mx, acc);
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
    if ((tid & 63) == 0) red_s[tid >> 6] = mx;
    __syncthreads();
}

// A operand and accumulator start of one 16-pattern tile.
template <int KS>
struct PatternTile {
    uint4 a[KS];
    float4 nh;
};

template <int KS>
__device__ __forceinline__ void load_pattern_tile(const PatternTable &tb, int p0, int n, int kb, PatternTile<KS> &t)
{
    const __half *arow = tb.lds_rows + (p0 + n) * kTabStrideOf<32 * KS> + 8 * kb;
#pragma unroll
    for (int s = 0; s < KS; ++s) t.a[s] = *reinterpret_cast<const uint4 *>(arow + 32 * s);
    t.nh = *reinterpret_cast<const float4 *>(tb.nh + p0 + 4 * kb);
}

// Candidates are ranked as unsigned integer keys: the binary32 pattern of e with the low 8 mantissa bits
// replaced by the pattern index.  e <= 0 up to rounding; among negative floats the unsigned order of the
// patterns is the order of decreasing value, so the smallest key is the nearest pattern.  An e that
// rounding made slightly positive ranks below every negative one, which is right, and can only be
// mis-ordered against another such e: both are then inside the re-evaluation band.
template <int KS>
__device__ __forceinline__ void rank_pattern_tile(const uint4 (&xb)[KS], const PatternTile<KS> &t, float hx, int p0, uint32_t &k1,
                                                  uint32_t &k2)
{
    floatx4_t d = {t.nh.x - hx, t.nh.y - hx, t.nh.z - hx, t.nh.w - hx};
#pragma unroll
    for (int s = 0; s < KS; ++s) d = mfma_f16(t.a[s], xb[s], d);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        // bytes 3..1 of e, byte 0 = index (one byte permute)
        const uint32_t key = __builtin_amdgcn_perm(__float_as_uint(d[i]), (uint32_t)(p0 + i), 0x07060500u);
        k2 = max(min(k1, k2), min(max(k1, k2), key));   // median of three = second smallest so far
        k1 = min(k1, key);
    }
}

// NT 16-token tiles of 32 * KS channels held as B operands xb[j][KS] (K-step s in xb[j][s]); every pattern tile read from the table
// serves all NT of them.  Returns, in every lane of column n, per tile: best index, best squared distance (from
// the expanded form, low 8 mantissa bits dropped), ||x||^2 and whether the token needs the exact re-evaluation.
template <int NT, int KS>
__device__ __forceinline__ void assign_tiles_mfma(const uint4 (&xb)[NT][KS], const PatternTable &tb, int lane, int (&best_i)[NT],
                                                  float (&best_v)[NT], float (&x2)[NT], bool (&flag)[NT])
{
    const int n = lane & 15, kb = lane >> 4;
    float part[NT], hx[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        float acc = 0.f;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const half2_t *h = reinterpret_cast<const half2_t *>(&xb[j][s]);
#pragma unroll
            for (int k = 0; k < 4; ++k) acc = __builtin_amdgcn_fdot2(h[k], h[k], acc, false);
        }
        part[j] = acc;
    }
    const float xx = fold_rows<NT>(part, AddF());   // |x|^2 of the lane's column in tile kb % NT
    spread_rows<NT>(0.5f * xx, hx);

    // the key's index bits are p0 + i here; the lane's 4*kb is added after the loop (no carries: p0 % 16 == 0)
    uint32_t k1[NT], k2[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) k1[j] = k2[j] = 0xffffffffu;   // above every key
    const int Pp = pad16(tb.P);
    if constexpr (KS <= 4) {
        PatternTile<KS> ta, tc;
        load_pattern_tile(tb, 0, n, kb, ta);
        for (int p0 = 0;;) {   // two tiles per round, the next one in flight while the current is ranked
            if (p0 + 16 < Pp) load_pattern_tile(tb, p0 + 16, n, kb, tc);
#pragma unroll
            for (int j = 0; j < NT; ++j) rank_pattern_tile(xb[j], ta, hx[j], p0, k1[j], k2[j]);
            if ((p0 += 16) >= Pp) break;
            if (p0 + 16 < Pp) load_pattern_tile(tb, p0 + 16, n, kb, ta);
#pragma unroll
            for (int j = 0; j < NT; ++j) rank_pattern_tile(xb[j], tc, hx[j], p0, k1[j], k2[j]);
            if ((p0 += 16) >= Pp) break;
        }
    } else {   // 256 channels: a tile is 36 registers, held once
        for (int p0 = 0; p0 < Pp; p0 += 16) {
            PatternTile<KS> ta;
            load_pattern_tile(tb, p0, n, kb, ta);
#pragma unroll
            for (int j = 0; j < NT; ++j) rank_pattern_tile(xb[j], ta, hx[j], p0, k1[j], k2[j]);
        }
    }
    // merge the four lane groups of the columns; from here on row kb speaks for tile kb % NT
    uint32_t a1[NT], a2[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        a1[j] = k1[j] | (uint32_t)kb << 2;
        a2[j] = k2[j] | (uint32_t)kb << 2;
    }
    auto merge = [](rows2 p1, rows2 p2, uint32_t &m1, uint32_t &m2) {
        m1 = min(p1[0], p1[1]);
        m2 = min(min(p2[0], p2[1]), max(p1[0], p1[1]));
    };
    uint32_t m1, m2;
    merge(swap16(a1[0], a1[NT > 1 ? 1 : 0]), swap16(a2[0], a2[NT > 1 ? 1 : 0]), m1, m2);
    if constexpr (NT == 4) {
        uint32_t h1, h2;
        merge(swap16(a1[2], a1[3]), swap16(a2[2], a2[3]), h1, h2);
        merge(swap32(m1, h1), swap32(m2, h2), m1, m2);
    } else {
        merge(swap32(m1, m1), swap32(m2, m2), m1, m2);
    }
    const float best = -2.f * __uint_as_float(m1 & 0xffffff00u), second = -2.f * __uint_as_float(m2 & 0xffffff00u);
    // accumulation error of e is far below 2^-21 (|x|^2 + |m|^2) per chain of four matrix instructions, the keys
    // drop 8 mantissa bits: flag with a wide margin.  A single pattern has nothing to be confused with.
    constexpr float kBand = KS > 4 ? 1.52587890625e-05f : 7.62939453125e-06f;
    const bool open = tb.P > 1 && !(second - best > kBand * (xx + tb.norm2_max) + 6.103515625e-05f * second);
    // (a single pattern could lose to the rows behind the table if e is not a number)
    uint32_t word[NT];
    spread_rows<NT>((m1 & (tb.P > 1 ? 0xffu : 0u)) | (open ? 0x80000000u : 0u), word);
    spread_rows<NT>(best, best_v);
    spread_rows<NT>(xx, x2);
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        best_i[j] = (int)(word[j] & 0xffu);
        flag[j] = (int)word[j] < 0;
    }
}

// One 16-token tile.
template <int KS>
__device__ __forceinline__ void assign_tile_mfma(const uint4 (&xb)[KS], const PatternTable &tb, int lane, int &best_i,
                                                 float &best_v, float &x2, bool &flag)
{
    int bi[1];
    float bv[1], xx[1];
    bool fl[1];
    assign_tiles_mfma<1, KS>(reinterpret_cast<const uint4 (&)[1][KS]>(xb), tb, lane, bi, bv, xx, fl);
    best_i = bi[0];
    best_v = bv[0];
    x2 = xx[0];
    flag = fl[0];
}

// Exact re-evaluation of one token by a whole wave: xrow_s = its D channels (fp16) in LDS.
// Every lane returns the exact argmin (lowest index on ties) and its distance; `none` and infinity for a token that no
// pattern is nearest to: it is not finite, or no pattern is, so that no distance is below infinity.
template <int D>
__device__ __forceinline__ void exact_argmin_wave(const __half *xrow_s, const PatternTable &tb, int lane, int none, int &best_i,
                                                  float &best_d)
{
    float bd = INFINITY;
    int bi = none;
    for (int p = lane; p < tb.P; p += 64) {
        // the pattern rows come from the LDS copy of the table (the same fp16 values): read from global memory they
        // missed L2 often enough to add a fifth to the HBM traffic of a mining step on a large job
        const __half *m = tb.lds_rows + p * kTabStrideOf<D>;
        float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
#pragma unroll 4
        for (int ch = 0; ch < D / 8; ++ch) {   // several row pieces in flight
            const uint4 mv = *reinterpret_cast<const uint4 *>(m + ch * 8);
            const uint4 xv = *reinterpret_cast<const uint4 *>(xrow_s + ch * 8);
            // (one v_fma_mix_f32 per difference instead of two conversions and a subtraction: the same value)
            const float d0 = sub_lo(xv.x, mv.x), d1 = sub_hi(xv.x, mv.x), d2 = sub_lo(xv.y, mv.y), d3 = sub_hi(xv.y, mv.y);
            const float d4 = sub_lo(xv.z, mv.z), d5 = sub_hi(xv.z, mv.z), d6 = sub_lo(xv.w, mv.w), d7 = sub_hi(xv.w, mv.w);
            a0 = fmaf(d0, d0, a0); a1 = fmaf(d1, d1, a1); a2 = fmaf(d2, d2, a2); a3 = fmaf(d3, d3, a3);
            a0 = fmaf(d4, d4, a0); a1 = fmaf(d5, d5, a1); a2 = fmaf(d6, d6, a2); a3 = fmaf(d7, d7, a3);
        }
        const float dist = (a0 + a1) + (a2 + a3);
        if (dist < bd) {
            bd = dist;
            bi = p;
        }
    }
    auto nearer = [&](uint32_t d, uint32_t i) {
        const float od = __uint_as_float(d);
        if (od < bd || (od == bd && (int)i < bi)) {
            bd = od;
            bi = (int)i;
        }
    };
    // lanes n ^ 1 and n ^ 2, mirrored half rows and rows (as in row_sum), then the four rows
    nearer(dpp<0xb1>(bits_of(bd)), dpp<0xb1>((uint32_t)bi));
    nearer(dpp<0x4e>(bits_of(bd)), dpp<0x4e>((uint32_t)bi));
    nearer(dpp<0x141>(bits_of(bd)), dpp<0x141>((uint32_t)bi));
    nearer(dpp<0x140>(bits_of(bd)), dpp<0x140>((uint32_t)bi));
    rows2 od = swap16(bits_of(bd), bits_of(bd)), oi = swap16((uint32_t)bi, (uint32_t)bi);
    nearer(od[0], oi[0]);
    nearer(od[1], oi[1]);
    od = swap32(bits_of(bd), bits_of(bd)), oi = swap32((uint32_t)bi, (uint32_t)bi);
    nearer(od[0], oi[0]);
    nearer(od[1], oi[1]);
    best_i = bi;
    best_d = bd;
}

// Re-evaluate the flagged tokens of a tile.  xrow_s: per-wave LDS scratch of 32 * KS halves.  A token that no pattern is nearest
// to is always flagged (its gap is not a number or infinite); its index becomes `none`.  seen(index): called by the lanes of
// every token that was evaluated again.  UNLIKELY: the loop is put out of the way of the code around it (one token in several
// hundred takes it): a mining step of 8 sets 0.3 % faster; in the quantizers, whose registers are all taken, it costs a spill.
struct Ignore {
    __device__ __forceinline__ void operator()(int) const {}
};
template <int KS, bool UNLIKELY = false, class SEEN = Ignore>
__device__ __forceinline__ void resolve_flagged(const uint4 (&xb)[KS], bool flag, __half *xrow_s, const PatternTable &tb,
                                                int lane, int none, int &best_i, float &best_d, SEEN seen = SEEN())
{
    const int n = lane & 15, kb = lane >> 4;
    unsigned long long todo = __ballot(flag) & 0xffffull;   // one bit per column
    while (UNLIKELY ? __builtin_expect(todo != 0, 0) : todo != 0) {
        const int col = __ffsll((long long)todo) - 1;
        todo &= todo - 1;
        if (n == col) {
#pragma unroll
            for (int s = 0; s < KS; ++s) *reinterpret_cast<uint4 *>(xrow_s + 32 * s + 8 * kb) = xb[s];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        int bi;
        float bd;
        exact_argmin_wave<32 * KS>(xrow_s, tb, lane, none, bi, bd);
        if (n == col) {
            best_i = bi;
            best_d = bd;
            seen(bi);
        }
        __builtin_amdgcn_wave_barrier();
    }
}

}  // namespace pk
