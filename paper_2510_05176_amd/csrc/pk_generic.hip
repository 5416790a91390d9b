// Head dimensions other than 128 (96 and 256, the other two that Sec. 3.3 names): window pattern, decode (with shared prefix
// and with per-sequence fill states) and dequantize, on contiguous and on paged caches; the decode also serves head dimension
// 128 for head counts that the tuned kernel of pk_decode_packed.hip does not take.  (Mining and the quantizers are templates
// on the head dimension in pk_mine.hip and pk_quantize.hip.)  The decode computes in binary32 accuracy throughout.
#pragma clang fp contract(off)

#include "pk_assign_mfma.h"
#include "pk_decode_fields.h"
#include "pk_decode_tail.h"
#include "pk_quant_arith.h"

namespace pk {

namespace {

constexpr int kGenThreads = 256;   // >= the largest head dimension

__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
    return v;
}

// ---------------------------------------------------------------------------------------------- window pattern
__global__ __launch_bounds__(kGenThreads) void gen_window_pattern_kernel(const __half *x, int64_t set_stride, int n, int d,
                                                                        __half *out, int64_t out_stride)
{
    const int c = threadIdx.x;
    if (c >= d) return;
    const __half *xs = x + (int64_t)blockIdx.x * set_stride + c;
    float mn = INFINITY, mx = -INFINITY;
    for (int t = 0; t < n; ++t) {
        const float v = h2f(xs[(int64_t)t * d]);
        mn = fminf(mn, v);
        mx = fmaxf(mx, v);
    }
    out[(int64_t)blockIdx.x * out_stride + c] = __float2half_rn((mn + mx) * 0.5f);
}

// ---------------------------------------------------------------------------------------------- reconstruction
// code of channel c of the packed token at position pos
__device__ __forceinline__ int k_code_at(const CacheView &cv, int64_t pos, int c, int d, int bits)
{
    int code = 0;
    for (int j = 0; j < bits; ++j) code |= (int)((cv.k_codes[(pos * (d / 32) + (c >> 5)) * bits + j] >> (c & 31)) & 1u) << j;
    return code;
}
__device__ __forceinline__ int v_code_at(const CacheView &cv, int64_t pos, int c, int d, int bits)
{
    const uint32_t *vb = reinterpret_cast<const uint32_t *>(cv.v_codes);
    const int64_t word = (((pos >> 4) * 16 + (c & 15)) * (d / 16) + (c >> 4)) * (bits / 2);
    int code = 0;
    for (int j = 0; j < bits; ++j) code |= (int)((vb[word + j / 2] >> (16 * (j % 2) + (int)(pos & 15))) & 1u) << j;
    return code;
}
// K^[c], V^[c] of a packed token: M[k*] + (s * code + z), multiply, add, add in binary32
__device__ __forceinline__ float k_hat(const CacheView &cv, const __half *MK, int64_t pos, int c, int d, int bits, int G)
{
    const int64_t prow = (pos / G) * d + c;
    const float res = h2f(cv.k_scale[prow]) * (float)k_code_at(cv, pos, c, d, bits) + h2f(cv.k_zero[prow]);
    return h2f(MK[(int64_t)cv.k_idx[pos] * d + c]) + res;
}
__device__ __forceinline__ float v_hat(const CacheView &cv, const __half *MV, int64_t pos, int c, int d, int bits, int Gc,
                                       int thresholded)
{
    const int ng = d / Gc;
    const int64_t prow = ((pos >> 4) * ng + c / Gc) * 16 + (pos & 15);
    const float res = h2f(cv.v_scale[prow]) * (float)v_code_at(cv, pos, c, d, bits) + h2f(cv.v_zero[prow]);
    const int vi = cv.v_idx[pos];
    if (thresholded && vi == PK_NO_PATTERN) return res;
    return h2f(MV[(int64_t)vi * d + c]) + res;
}

__global__ __launch_bounds__(kGenThreads) void gen_dequant_kernel(DequantArgs a)
{
    const int t = a.t0 + blockIdx.x, n = blockIdx.y, c = threadIdx.x, d = a.d;
    if (c >= d) return;
    const int set = a.sets.set_of(n);
    const int Gc = a.G < d ? a.G : d;
    const int64_t pos = a.c.map.of(n).pos(t);
    const int64_t orow = ((int64_t)n * (a.t1 - a.t0) + (t - a.t0)) * d + c;
    if (a.k_out) a.k_out[orow] = k_hat(a.c, a.patterns_k + (int64_t)set * a.P * d, pos, c, d, a.bits, a.G);
    if (a.v_out) a.v_out[orow] = v_hat(a.c, a.patterns_v + (int64_t)set * a.P * d, pos, c, d, a.bits, Gc, a.v_thresholded);
}

// ---------------------------------------------------------------------------------------------- decode
// Decode attention (Sec. 3.4) for head dimensions 96 and 256, and at 128 for head counts that the tuned kernel does not take,
// with the accuracy of binary32.  The context of a stream is cut into the same slots as in the tuned path (equal splits of the
// shared prefix's packed part, of the own packed part, then the own tail and the prefix's tail); a workgroup takes one
// slot of one stream for up to eight query heads of the KV head at once (more heads: further workgroups) and leaves an
// unnormalised partial (o, per-pattern softmax mass W, running maximum m in the log2 domain, sum l); a second kernel merges
// the partials and adds W . M_V once per head.  W is summed in LDS as 64-bit fixed point (unit 2^-31, weights are <= 1)
// with integer atomics, so the result does not depend on the order in which the tokens arrive.
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kMassUnit = 2147483648.f;   // 2^31

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// The workgroup's tail slot (own cache, or the shared prefix).  (Without a tail the loop over its tokens has no turn, and the
// partial is empty: the merge skips partials whose sum is zero.)
template <int D>
__device__ __forceinline__ void gen_tail_slot(const DecodeArgs &a, unsigned char *smem, int ns, int which, int h0)
{
    const int nh = min(8, a.n_q_heads / a.n_kv_heads - h0);
    if (nh > 4)
        decode_tail_body<8, D, true>(a, which, ns, h0, nh, *reinterpret_cast<TailShared<8, D> *>(smem));
    else if (nh > 1)
        decode_tail_body<4, D, true>(a, which, ns, h0, nh, *reinterpret_cast<TailShared<4, D> *>(smem));
    else
        decode_tail_body<1, D, true>(a, which, ns, h0, nh, *reinterpret_cast<TailShared<1, D> *>(smem));
}
template <int D>
constexpr size_t gen_tail_lds_bytes(int nh)
{
    return nh > 4 ? sizeof(TailShared<8, D>) : nh > 1 ? sizeof(TailShared<4, D>) : sizeof(TailShared<1, D>);
}

template <int D>
__global__ __launch_bounds__(kGenThreads) void gen_tail_kernel(DecodeArgs a)
{
    extern __shared__ __align__(16) unsigned char gen_decode_smem[];
    gen_tail_slot<D>(a, gen_decode_smem, blockIdx.x, blockIdx.y, blockIdx.z * 8);
}

// Dynamic LDS of the decode kernel: [P][8] q . M_K, [4 waves][nh][w_stride] 64-bit masses, the queries; the waves' outputs
// [4][nh][d] take their place at the end; a tail workgroup has its own layout.
template <int D>
constexpr size_t gen_decode_lds_bytes(int P, int w_stride, int nh)
{
    const size_t q = (size_t)(D + 127) / 128 * 4 * 32 * 16;
    const size_t loop = q + (size_t)P * 8 * 4 + (size_t)4 * nh * w_stride * 8, out = (size_t)4 * nh * D * 4;
    const size_t tail = gen_tail_lds_bytes<D>(nh), most = loop > out ? loop : out;
    return most > tail ? most : tail;
}

__device__ __forceinline__ float other_half(float v)   // the value of column n ^ 8 (row rotation by 8)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x128, 0xf, 0xf, true));
}

// fp16 roundings of x and y, or 2^11 times what those roundings drop (exact, and in range wherever the rounding is)
constexpr float kLowUp = 2048.f;
struct ColumnPart {
    float mul, sub;   // 1, 0 or 2^11, 2^11
};
__device__ __forceinline__ uint32_t split_pair(float x, float y, const ColumnPart &c)
{
    uint32_t hi = cvt2(x, y);
    asm("" : "+v"(hi));   // the very roundings that the first kind uses (folded into the product before, they may be others)
    const half2v h = __builtin_bit_cast(half2v, hi);
    return cvt2(fmaf(-c.sub, (float)h[0], x * c.mul), fmaf(-c.sub, (float)h[1], y * c.mul));
}

// The fields as normal numbers code * 2^(pos - 10).  (Products with subnormal operands are aligned by the exponents as stored and
// cut off there: with the fields as they are the sums of codes came out low by 5e-6 of themselves, 4e-5 of the result.)
__device__ __forceinline__ void fields_to_normal(uint32_t X, uint32_t *out)
{
    fields_to_operand(X, out);
#pragma unroll
    for (int v = 0; v < 8; ++v) out[v] = pk_mul(out[v], 0x74007400u);   // 2^14
}

// The V codes of plane pair F (bits 2F and 2F + 1) as normal numbers (field - 3/2) * 4^F * 2^-11, so that the pairs of a word add up to
// the code less half of the largest one.  One factor for all positions of a word: the other operand then has the whole of
// fp16's range for the weights.
__host__ __device__ constexpr uint32_t half_pair(int e) { return (uint32_t)(e + 15) * 0x04000400u; }   // 2^e twice, -14 <= e <= 15
template <int F>
__device__ __forceinline__ void fields_to_centred(uint32_t X, uint32_t *out)
{
    fields_to_operand(X, out);
    const half2v c = {(_Float16)(-1.5f * (F ? 4.f : 1.f) / 2048.f), (_Float16)(-1.5f * (F ? 4.f : 1.f) / 2048.f)};
#pragma unroll
    for (int v = 0; v < 8; ++v)   // (a field is code * 2^(fpos - 24); the results are exact)
        out[v] = __builtin_bit_cast(uint32_t, __builtin_elementwise_fma(__builtin_bit_cast(half2v, out[v]),
                                                                        __builtin_bit_cast(half2v, half_pair(13 + 2 * F - fpos(v))), c));
}

// Packed part on the matrix cores.  A wave walks 64-token blocks of its own run with its own online softmax; operands and
// lane roles are those of the tuned kernel (pk_decode_packed.hip), with one difference: the sixteen columns (rows on the V
// side) of a tile are eight heads twice, column n with the fp16 rounding of the other operand and column n + 8 with 2^11 times
// what that rounding dropped, again rounded to fp16.  The sum of the two columns is q * s_K exactly (that product of two fp16
// numbers has 22 significant bits) and p * s_V to 23 bits, the codes are exact, and the matrix instruction adds eight products at
// a time to its binary32 accumulator, so that the sums are rounded an eighth as often as the serial sums of the binary32 vector
// arithmetic that this replaces.  The operands are brought
// into fp16's range by powers of two: q * s_K per head and K group, by the largest |q * s_K|; p * s_V per wave, by the largest
// scale met so far (the accumulators follow by an exact multiplication when a block exceeds it), to 2^15, so that a weight has
// its 23 bits down to 2^-27 of the largest and eleven of them down to 2^-39 (a pattern's mass has the unit 2^-31).
// Bound by vector instruction issue (operand building, 1.5 k instructions per block and wave at 256 channels against 64
// matrix instructions).  Replaces a kernel on the vector ALUs (a thread per token, every code taken apart for every head); whole
// decodes, 256 streams x 4096 tokens, 4 heads: d 256, 64-token groups 342 -> 102 us, d 96, 32-token groups 180 -> 74; one
// head 233 -> 92; 7 heads over 32-channel groups at 128 channels (128 streams) 167 -> 64.  Error
// against 64 bits, largest over d 256 / 96 / 128, 2 and 4 bits, 16384 tokens in splits of 8192 (the vector arithmetic's in
// brackets): values about 1 1.1e-7 (1.3e-7), about zero 3.5e-6 (2.4e-5), a first token 9 above the others' scores whose value is small
// 2.6e-7 (1.2e-6), 18 above 7.4e-6 (5.1e-5), keys 20 times as large 3.4e-6 (5.8e-6).
template <int D, int G, int BITS>
__global__ __launch_bounds__(kGenThreads) __attribute__((amdgpu_waves_per_eu(2))) void gen_decode_kernel(DecodeArgs a)
{
    constexpr int KW = (D + 127) / 128;               // plane words of a token per lane and plane: words kb and kb + 4
    constexpr int WPU = BITS / 2;
    constexpr int Gc = G < D ? G : D, NG = D / Gc, TPG = Gc / 16;   // V channel groups, 16-channel tiles of one
    constexpr bool TWO = G == 32;                     // two K groups per block
    extern __shared__ __align__(16) unsigned char gen_decode_smem[];
    __shared__ float stat_m[4][8], stat_l[4][8], stat_pz[4][8][NG];
    const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, kb = lane >> 4, P = a.P;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ns = blockIdx.x, slot = blockIdx.y, h0 = blockIdx.z * 8;   // the workgroup's first head of the KV head's r
    const int seq = ns / a.n_kv_heads, head = ns - seq * a.n_kv_heads;
    const int r = a.n_q_heads / a.n_kv_heads, nh = min(8, r - h0);
    const int n_packed = a.splits_prefix + a.splits_own, n_slots = n_packed + 2;
    if (slot >= n_packed) {
        gen_tail_slot<D>(a, gen_decode_smem, ns, slot - n_packed, h0);
        return;
    }
    const bool pre = slot < a.splits_prefix;
    const CacheView &cv = pre ? a.prefix : a.own;
    int tq = cv.t_quant;
    if (!pre) {
        int tt, ts;
        own_state(a, seq, tq, tt, ts);
    }
    const int stream = pre ? head : ns;
    const int set = pre ? head : a.sets.set_of(ns);
    const int t_begin = (pre ? slot : slot - a.splits_prefix) * a.chunk, t_end = min(tq, t_begin + a.chunk);
    const int64_t pb = ((int64_t)ns * n_slots + slot) * r + h0;   // partial of the workgroup's first query head
    if (t_end <= t_begin) {   // nothing in this slot: the merge skips partials whose sum is zero
        if (tid < nh) {
            a.part_ml[(pb + tid) * 2] = -INFINITY;
            a.part_ml[(pb + tid) * 2 + 1] = 0.f;
        }
        return;
    }

    const int h = n & 7, WS = a.w_stride;
    const bool upper = n >= 8;
    const ColumnPart part = {upper ? kLowUp : 1.f, upper ? kLowUp : 0.f};   // columns 8-15 carry the dropped parts
    const float weight = upper ? 1.f / kLowUp : 1.f;
    const float scale2 = a.softmax_scale * kLog2e;
    uint4 *q_s = reinterpret_cast<uint4 *>(gen_decode_smem);                      // [word j, piece][kb][head]
    float *QMs = reinterpret_cast<float *>(q_s + KW * 4 * 32);                    // [P][8]
    unsigned long long *Ws = reinterpret_cast<unsigned long long *>(QMs + P * 8);   // [wave][nh][WS]
    const bool word_ok = D % 128 == 0 || kb < D / 32;                             // 96 channels: lane group 3 has none
    {
        const __half *qrow = a.q + ((int64_t)seq * a.n_q_heads + head * r + h0 + min(h, nh - 1)) * D;
        const __half *MK = a.patterns_k + (int64_t)set * P * D;
        uint4 qv[KW][4];
#pragma unroll
        for (int j = 0; j < KW; ++j) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                qv[j][i] = make_uint4(0u, 0u, 0u, 0u);
                if (word_ok && h < nh) qv[j][i] = *reinterpret_cast<const uint4 *>(qrow + 32 * (kb + 4 * j) + 8 * i);
                if (wave == 0 && !upper) q_s[(j * 4 + i) * 32 + kb * 8 + h] = qv[j][i];
            }
        }
        for (int tp = wave; tp * 16 < P; tp += 4) {   // q . M_K, one 16-pattern tile per wave and round (fp16 products are exact)
            floatx4 acc = {0.f, 0.f, 0.f, 0.f};
            const int p = tp * 16 + n;
#pragma unroll
            for (int j = 0; j < KW; ++j) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint4 av = make_uint4(0u, 0u, 0u, 0u);
                    if (word_ok && p < P) av = *reinterpret_cast<const uint4 *>(MK + (int64_t)p * D + 32 * (kb + 4 * j) + 8 * i);
                    acc = mfma16(reinterpret_cast<const uint32_t *>(&av), reinterpret_cast<const uint32_t *>(&qv[j][i]), acc);
                }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int pr = tp * 16 + 4 * kb + i;
                if (pr < P && !upper) QMs[pr * 8 + h] = acc[i] * scale2;
            }
        }
        for (int i = lane; i < nh * WS; i += 64) Ws[wave * nh * WS + i] = 0ull;
    }
    __syncthreads();

    const int n_blocks = (t_end - t_begin) >> 6, per = (n_blocks + 3) >> 2;
    const int b0 = wave * per, b1 = min(n_blocks, b0 + per);

    struct Operand {
        uint32_t B[KW][16];   // q * s (columns 0-7) or what its rounding dropped (8-15), operand order, field scale folded in
        float c1, qz;         // factor of a score in the log2 domain; scale2 * q . z
    };
    auto build = [&](int64_t grp, Operand &o) {
        const __half *sp = cv.k_scale + grp * D, *zp = cv.k_zero + grp * D;
        float qs[KW][32];
        float big = 0.f, qz = 0.f;
#pragma unroll
        for (int j = 0; j < KW; ++j) {
            const int w = word_ok ? kb + 4 * j : 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint4 q4 = q_s[(j * 4 + i) * 32 + kb * 8 + h];
                const uint4 s4 = *reinterpret_cast<const uint4 *>(sp + 32 * w + 8 * i), z4 = *reinterpret_cast<const uint4 *>(zp + 32 * w + 8 * i);
                const uint32_t qw[4] = {q4.x, q4.y, q4.z, q4.w}, sw[4] = {s4.x, s4.y, s4.z, s4.w}, zw[4] = {z4.x, z4.y, z4.z, z4.w};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const half2v qh = __builtin_bit_cast(half2v, qw[k]), sh = __builtin_bit_cast(half2v, sw[k]), zh = __builtin_bit_cast(half2v, zw[k]);
                    qz = fmaf((float)qh[0], (float)zh[0], qz);
                    qz = fmaf((float)qh[1], (float)zh[1], qz);
                    const float u = (float)qh[0] * (float)sh[0], v = (float)qh[1] * (float)sh[1];   // exact
                    qs[j][8 * i + 2 * k] = u;
                    qs[j][8 * i + 2 * k + 1] = v;
                    big = fmaxf(fmaxf(big, fabsf(u)), fabsf(v));
                }
            }
        }
        big = fmaxf(big, __shfl_xor(big, 16));
        big = fmaxf(big, __shfl_xor(big, 32));
        qz += __shfl_xor(qz, 16);
        qz += __shfl_xor(qz, 32);
        int e = 7;
        if (big > 0.f) (void)frexpf(big, &e);    // big = m * 2^e, m in [0.5, 1)
        const float up = ldexpf(1.f, 7 - e);     // the largest becomes 64 .. 128, times the field scale (at most 2^8) below 2^15
        o.c1 = ldexpf(scale2 * 4.f, e - 7);     // (a field times its scale is code / 4)
        o.qz = qz * scale2;
#pragma unroll
        for (int j = 0; j < KW; ++j) {
#pragma unroll
            for (int V = 0; V < 16; ++V) {
                const int v = V & 7, odd = V >> 3;
                const float f = up * (float)(1 << (8 - fpos(v)));
                const float x = qs[j][e_lo(v) + odd] * f, y = qs[j][e_lo(v) + 16 + odd] * f;
                o.B[j][V] = split_pair(x, y, part);
            }
        }
    };

    float m_run = 0.f, l_run = 0.f, pz[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) pz[g] = 0.f;
    bool started = false;
    // Values: sum p (s code + z) = sum (p s) (code - mid) + sum p (z + s mid), mid half of the largest code.  (With the code
    // and z as they are, two sums of one sign each all but cancel where V is spread about zero.)
    constexpr float kMid = 0.5f * (float)((1 << BITS) - 1);
    float s_lim = 0.f;   // power of two above the largest V scale so far; the accumulators hold kUp / s_lim / 2048 times the sums
    constexpr float kUp = 32768.f;
    floatx4 O[D / 16];
#pragma unroll
    for (int t = 0; t < D / 16; ++t) O[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    Operand ga, gb;   // gb: second K group of a block
    const uint32_t *vwords = reinterpret_cast<const uint32_t *>(cv.v_codes);
    const StreamMap map = cv.map.of(stream);

    for (int b = b0; b < b1; ++b) {
        const int tb = t_begin + (b << 6);
        const int64_t pos0 = map.pos(tb);   // (a 64-token block never straddles a page)
        // ---- inputs of the block
        uint32_t kw[4][KW][BITS];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int64_t tok = pos0 + 16 * (n >> 2) + 4 * x + (n & 3);
#pragma unroll
            for (int j = 0; j < KW; ++j) {
                const uint32_t *src = cv.k_codes + (tok * (D / 32) + (word_ok ? kb + 4 * j : 0)) * BITS;
#pragma unroll
                for (int k = 0; k < BITS; k += 2) {
                    const uint2 v = *reinterpret_cast<const uint2 *>(src + k);
                    kw[x][j][k] = v.x;
                    kw[x][j][k + 1] = v.y;
                }
            }
        }
        const uint4 ki = *reinterpret_cast<const uint4 *>(cv.k_idx + pos0 + 16 * kb), vi = *reinterpret_cast<const uint4 *>(cv.v_idx + pos0 + 16 * kb);
        const uint32_t kid[4] = {ki.x, ki.y, ki.z, ki.w}, vid[4] = {vi.x, vi.y, vi.z, vi.w};
        // the block's 64 * NG V scales, NG of them per lane
        float s_big = 0.f;
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const float s = h2f(cv.v_scale[(pos0 >> 4) * NG * 16 + g * 64 + lane]);
            s_big = fmaxf(s_big, s < INFINITY ? s : 0.f);   // (an infinite one spoils its own channel group only)
        }

        if (TWO || b == b0 || tb % G == 0) build(pos0 / G, ga);
        if (TWO) build(pos0 / G + 1, gb);

        // ---- scores of the 64 tokens relative to m_run, log2 domain: this lane has tokens 16 kb .. 16 kb + 15 of head h
        float S[16];
        const float c1 = TWO && kb >= 2 ? gb.c1 : ga.c1, base = (TWO && kb >= 2 ? gb.qz : ga.qz) - m_run;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            floatx4 d = {0.f, 0.f, 0.f, 0.f}, d2 = d, e = d, e2 = d;
#pragma unroll
            for (int j = 0; j < KW; ++j) {
#pragma unroll
                for (int f = 0; f < BITS; f += 2) {   // planes f, f + 1
                    uint32_t A16[16];
                    fields_to_normal(bfi(0x55555555u, kw[x][j][f], kw[x][j][f + 1] << 1), A16);
                    fields_to_normal(bfi(0x55555555u, kw[x][j][f] >> 1, kw[x][j][f + 1]), A16 + 8);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if (f == 0) {
                            d = mfma16(&A16[4 * i], &ga.B[j][4 * i], d);
                            if (TWO) d2 = mfma16(&A16[4 * i], &gb.B[j][4 * i], d2);
                        } else {
                            e = mfma16(&A16[4 * i], &ga.B[j][4 * i], e);
                            if (TWO) e2 = mfma16(&A16[4 * i], &gb.B[j][4 * i], e2);
                        }
                    }
                }
            }
            if (BITS == 4) {
                d += 4.f * e;
                d2 += 4.f * e2;
            }
            if (TWO && kb >= 2) d = d2;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int id = min((int)((kid[x] >> (8 * i)) & 255u), P - 1);
                const float dw = d[i] * weight;   // (the same sum, bit for bit, in both halves: the value sides of the two must agree)
                S[4 * x + i] = fmaf(dw + other_half(dw), c1, base + QMs[id * 8 + h]);
            }
        }

        // ---- online softmax (per head)
        float bmax = S[0];
#pragma unroll
        for (int k = 1; k < 16; ++k) bmax = fmaxf(bmax, S[k]);
        if (!started || __ballot(bmax > 0.f) != 0ull) {
            bmax = fmaxf(bmax, __shfl_xor(bmax, 16));
            bmax = fmaxf(bmax, __shfl_xor(bmax, 32));
            const float delta = started ? fmaxf(bmax, 0.f) : bmax;
            const float alpha = started ? __builtin_amdgcn_exp2f(-delta) : 0.f;
            l_run *= alpha;
#pragma unroll
            for (int g = 0; g < NG; ++g) pz[g] *= alpha;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float ar = __shfl(alpha, 4 * kb + i);   // output row 4 kb + i has the head of column 4 kb + i
#pragma unroll
                for (int t = 0; t < D / 16; ++t) O[t][i] *= ar;
            }
            if (started) {
                for (int hh = 0; hh < nh; ++hh) {
                    const double ar = (double)__shfl(alpha, hh);
                    for (int p = lane; p < WS; p += 64) {
                        unsigned long long *w = &Ws[(wave * nh + hh) * WS + p];
                        *w = (unsigned long long)((double)*w * ar);
                    }
                }
            }
            m_run += delta;
#pragma unroll
            for (int k = 0; k < 16; ++k) S[k] -= delta;
            started = true;
        }
        // columns n and n + 8 hold the same weights; of the sums that are not contractions each takes half of the tokens
        float pr[16], own[8];
#pragma unroll
        for (int k = 0; k < 16; ++k) pr[k] = __builtin_amdgcn_exp2f(S[k]);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            own[k] = upper ? pr[k + 8] : pr[k];
            l_run += own[k];
        }
        // ---- softmax mass per V pattern
        if (h < nh) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int id = (int)(((upper ? vid[2 + (k >> 2)] : vid[k >> 2]) >> (8 * (k & 3))) & 255u);
                atomicAdd(&Ws[(wave * nh + h) * WS + min(id, WS - 1)], (unsigned long long)(own[k] * kMassUnit));
            }
        }
        // ---- values
        if (__ballot(s_big > s_lim) != 0ull) {
            const float top = wave_max(s_big);   // positive here
            int e;
            (void)frexpf(top, &e);
            const float lim = ldexpf(1.f, e), f = s_lim / lim;   // (0 the first time: the accumulators are zero)
            s_lim = lim;
#pragma unroll
            for (int t = 0; t < D / 16; ++t) {
#pragma unroll
                for (int i = 0; i < 4; ++i) O[t][i] *= f;
            }
        }
        const float up = s_lim > 0.f ? kUp / s_lim : 0.f;
        float pu[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) pu[k] = pr[k] * up;
        const int64_t unit = (pos0 >> 4) + kb;
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const uint4 *sp = reinterpret_cast<const uint4 *>(cv.v_scale + (unit * NG + g) * 16), *zp = reinterpret_cast<const uint4 *>(cv.v_zero + (unit * NG + g) * 16);
            const uint4 s0 = sp[0], s1 = sp[1], z = zp[upper ? 1 : 0];
            const uint32_t sw[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w}, zw[4] = {z.x, z.y, z.z, z.w};
            uint32_t vw[TPG * WPU];
            const uint2 *vsrc = reinterpret_cast<const uint2 *>(vwords + ((unit * 16 + n) * (D / 16) + g * TPG) * WPU);
#pragma unroll
            for (int i = 0; i < TPG * WPU / 2; ++i) {
                const uint2 v = vsrc[i];
                vw[2 * i] = v.x;
                vw[2 * i + 1] = v.y;
            }
            uint32_t Ap[8];
#pragma unroll
            for (int V = 0; V < 8; ++V) {
                const half2v sh = __builtin_bit_cast(half2v, sw[V]);
                Ap[V] = split_pair(pu[2 * V] * (float)sh[0], pu[2 * V + 1] * (float)sh[1], part);
            }
#pragma unroll
            for (int V = 0; V < 4; ++V) {
                const half2v sh = __builtin_bit_cast(half2v, upper ? sw[V + 4] : sw[V]), zh = __builtin_bit_cast(half2v, zw[V]);
                pz[g] = fmaf(own[2 * V], fmaf((float)sh[0], kMid, (float)zh[0]), pz[g]);
                pz[g] = fmaf(own[2 * V + 1], fmaf((float)sh[1], kMid, (float)zh[1]), pz[g]);
            }
#pragma unroll
            for (int i = 0; i < TPG; ++i) {
                const int t = g * TPG + i;
#pragma unroll
                for (int f = 0; f < WPU; ++f) {
                    // one word = planes 2f (bits 0..15) and 2f + 1 (bits 16..31) of 16 tokens of channel 16 t + n, merged
                    // into 2-bit fields: even tokens in the low half, odd tokens in the high half
                    uint32_t Bv[8];
                    const uint32_t W = vw[i * WPU + f];
                    const uint32_t u = bfi(0x0000AAAAu, W >> 15, W);
                    if (f == 0)
                        fields_to_centred<0>(bfi(0x55550000u, W << 15, u), Bv);
                    else
                        fields_to_centred<1>(bfi(0x55550000u, W << 15, u), Bv);
                    O[t] = mfma16(&Ap[0], &Bv[0], O[t]);
                    O[t] = mfma16(&Ap[4], &Bv[4], O[t]);
                }
            }
        }
    }
    if (!started) m_run = -INFINITY;   // a wave without blocks contributes nothing to the merge

    // ---- merge the four waves of the workgroup
    l_run += other_half(l_run);
    l_run += __shfl_xor(l_run, 16);
    l_run += __shfl_xor(l_run, 32);
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        pz[g] += other_half(pz[g]);
        pz[g] += __shfl_xor(pz[g], 16);
        pz[g] += __shfl_xor(pz[g], 32);
        if (lane < 8) stat_pz[wave][n][g] = pz[g];
    }
    if (lane < 8) {
        stat_m[wave][n] = m_run;
        stat_l[wave][n] = l_run;
    }
    __syncthreads();
    auto top_of = [&](int hh) { return fmaxf(fmaxf(stat_m[0][hh], stat_m[1][hh]), fmaxf(stat_m[2][hh], stat_m[3][hh])); };
    for (int hh = 0; hh < nh; ++hh) {
        const float M = top_of(hh);
        for (int p = tid; p < P; p += kGenThreads) {
            float acc = 0.f;
#pragma unroll
            for (int w = 0; w < 4; ++w) acc = fmaf(__builtin_amdgcn_exp2f(stat_m[w][hh] - M), (float)Ws[(w * nh + hh) * WS + p], acc);
            a.part_w[(pb + hh) * P + p] = acc * (1.f / kMassUnit);
        }
    }
    __syncthreads();
    // every wave leaves its outputs, scaled to the workgroup's reference, in slabs of its own over the start of the dynamic LDS
    float *Os = reinterpret_cast<float *>(gen_decode_smem);
    const float down = s_lim * (2048.f / kUp);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int hh = 4 * kb + i;   // (rows 8-15: the dropped parts)
        const float f = hh < nh ? __builtin_amdgcn_exp2f(stat_m[wave][hh] - top_of(hh)) : 0.f;
#pragma unroll
        for (int t = 0; t < D / 16; ++t) {
            const float v = fmaf(__shfl_xor(O[t][i], 32), 1.f / kLowUp, O[t][i]);
            if (hh < nh) Os[(wave * nh + hh) * D + 16 * t + n] = f * fmaf(v, down, stat_pz[wave][hh][t / TPG]);
        }
    }
    __syncthreads();
    for (int i = tid; i < nh * D; i += kGenThreads)   // waves added in a fixed order
        a.part_o[pb * D + i] = (Os[i] + Os[nh * D + i]) + (Os[2 * nh * D + i] + Os[3 * nh * D + i]);
    if (tid < nh) {
        const float M = top_of(tid);
        float L = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) L = fmaf(__builtin_amdgcn_exp2f(stat_m[w][tid] - M), stat_l[w][tid], L);
        a.part_ml[(pb + tid) * 2] = M;
        a.part_ml[(pb + tid) * 2 + 1] = L;
    }
}

// log-sum-exp merge of the partials of one (sequence, query head) and the pattern part of the values, W . M_V
__global__ __launch_bounds__(kGenThreads) void gen_decode_merge_kernel(DecodeArgs a)
{
    __shared__ float wslot[kMaxSlots];
    __shared__ float Wsum[2][kGenThreads];   // shared prefix, own cache
    __shared__ float red[8];
    const int u = blockIdx.x, tid = threadIdx.x, d = a.d, P = a.P;
    const int seq = u / a.n_q_heads, qh = u - seq * a.n_q_heads;
    const int r = a.n_q_heads / a.n_kv_heads, head = qh / r, hr = qh - head * r;
    const int n = seq * a.n_kv_heads + head;
    const int n_packed = a.splits_prefix + a.splits_own, n_slots = n_packed + 2;
    const int64_t base = (int64_t)n * n_slots;
    float M = -INFINITY;
    for (int s = tid; s < n_slots; s += kGenThreads) {
        const int64_t q = ((base + s) * r + hr) * 2;
        if (a.part_ml[q + 1] > 0.f) M = fmaxf(M, a.part_ml[q]);
    }
    M = wave_max(M);
    if ((tid & 63) == 0) red[tid >> 6] = M;
    __syncthreads();
    M = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    float L = 0.f;
    for (int s = tid; s < n_slots; s += kGenThreads) {
        const int64_t q = ((base + s) * r + hr) * 2;
        const float l = a.part_ml[q + 1];
        const float w = l > 0.f ? exp2f(a.part_ml[q] - M) : 0.f;
        wslot[s] = w;
        L = fmaf(l, w, L);
    }
    L = wave_sum(L);
    if ((tid & 63) == 0) red[4 + (tid >> 6)] = L;
    __syncthreads();
    L = (red[4] + red[5]) + (red[6] + red[7]);
    for (int p = tid; p < P; p += kGenThreads) {
        float wp = 0.f, wo = 0.f;
        for (int s = 0; s < a.splits_prefix; ++s)
            if (wslot[s] > 0.f) wp = fmaf(a.part_w[((base + s) * r + hr) * P + p], wslot[s], wp);
        for (int s = a.splits_prefix; s < n_packed; ++s)
            if (wslot[s] > 0.f) wo = fmaf(a.part_w[((base + s) * r + hr) * P + p], wslot[s], wo);
        Wsum[0][p] = wp;
        Wsum[1][p] = wo;
    }
    __syncthreads();
    if (tid >= d) return;
    float acc = 0.f;
    for (int s = 0; s < n_slots; ++s)
        if (wslot[s] > 0.f) acc = fmaf(a.part_o[((base + s) * r + hr) * d + tid], wslot[s], acc);
    if (a.splits_prefix > 0) {
        const __half *MV = a.patterns_v + (int64_t)head * P * d;
        for (int p = 0; p < P; ++p) acc = fmaf(Wsum[0][p], h2f(MV[(int64_t)p * d + tid]), acc);
    }
    if (a.splits_own > 0) {
        const __half *MV = a.patterns_v + (int64_t)a.sets.set_of(n) * P * d;
        for (int p = 0; p < P; ++p) acc = fmaf(Wsum[1][p], h2f(MV[(int64_t)p * d + tid]), acc);
    }
    a.out[(int64_t)u * d + tid] = L > 0.f ? acc / L : 0.f;
    if (a.lse && tid == 0) a.lse[u] = L > 0.f ? (M + log2f(L)) * kLn2 : -INFINITY;
}

template <int D, int G, int BITS>
hipError_t launch_gen_packed(const DecodeArgs &a, dim3 grid, hipStream_t s)
{
    static LdsOptIn opt_in;
    const int r = a.n_q_heads / a.n_kv_heads, nh = r < 8 ? r : 8;
    constexpr size_t most = gen_decode_lds_bytes<D>(256, 256, 8);
    const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(&gen_decode_kernel<D, G, BITS>), opt_in, most);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((gen_decode_kernel<D, G, BITS>), grid, dim3(kGenThreads), gen_decode_lds_bytes<D>(a.P, a.w_stride, nh), s, a);
    return hipGetLastError();
}
template <int D>
hipError_t launch_gen_decode_of(const DecodeArgs &a, dim3 grid, hipStream_t s)
{
    if constexpr (D != 96) {   // (64 does not divide 96 channels)
        if (a.G == 64) return a.bits == 2 ? launch_gen_packed<D, 64, 2>(a, grid, s) : launch_gen_packed<D, 64, 4>(a, grid, s);
    }
    if (a.G == 32) return a.bits == 2 ? launch_gen_packed<D, 32, 2>(a, grid, s) : launch_gen_packed<D, 32, 4>(a, grid, s);
    if (a.G == 128) return a.bits == 2 ? launch_gen_packed<D, 128, 2>(a, grid, s) : launch_gen_packed<D, 128, 4>(a, grid, s);
    return hipErrorInvalidValue;
}

}  // namespace

// ---------------------------------------------------------------------------------------------- launchers
hipError_t launch_generic_window_pattern(const __half *x, int64_t set_stride, int n_sets, int n, int d, __half *out,
                                         int64_t out_stride, hipStream_t s)
{
    hipLaunchKernelGGL(gen_window_pattern_kernel, dim3(n_sets), dim3(kGenThreads), 0, s, x, set_stride, n, d, out, out_stride);
    return hipGetLastError();
}

hipError_t launch_generic_decode(const DecodeArgs &a, hipStream_t s)
{
    // eight heads of a KV head per workgroup; more (up to 64 by the configuration check) go to further workgroups along z
    const int r = a.n_q_heads / a.n_kv_heads;
    // The tails ride along in the packed kernel's launch, where there is one: apart, 32 streams x 1000 vectors of 256 channels
    // with 232 of them in the tail take 56 us instead of 41, 128 streams 73 instead of 55, 512 streams x 500 of 96 channels
    // 55.5 instead of 52.7, 2048 streams x 600 220 instead of 213.
    const int n_packed = a.splits_prefix + a.splits_own, N = a.n_seq * a.n_kv_heads, hz = (r + 7) / 8;
    hipError_t e;
    if (n_packed > 0) {
        const dim3 grid(N, n_packed + 2, hz);
        e = a.d == kD ? launch_gen_decode_of<kD>(a, grid, s) : a.d == 96 ? launch_gen_decode_of<96>(a, grid, s) : launch_gen_decode_of<256>(a, grid, s);
        if (e != hipSuccess) return e;
    }
    if (n_packed == 0) {
        const dim3 grid(N, 2, hz), block(kGenThreads);
        if (a.d == kD)
            hipLaunchKernelGGL(gen_tail_kernel<kD>, grid, block, gen_tail_lds_bytes<kD>(r), s, a);
        else if (a.d == 96)
            hipLaunchKernelGGL(gen_tail_kernel<96>, grid, block, gen_tail_lds_bytes<96>(r), s, a);
        else
            hipLaunchKernelGGL(gen_tail_kernel<256>, grid, block, gen_tail_lds_bytes<256>(r), s, a);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    hipLaunchKernelGGL(gen_decode_merge_kernel, dim3(a.n_seq * a.n_q_heads), dim3(kGenThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_generic_dequant(const DequantArgs &a, hipStream_t s)
{
    if (a.t1 <= a.t0) return hipSuccess;
    hipLaunchKernelGGL(gen_dequant_kernel, dim3(a.t1 - a.t0, a.n_streams), dim3(kGenThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace pk
