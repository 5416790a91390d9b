// The hot path for head dimensions other than 128 (96 and 256, the other two that Sec. 3.3 names): plain kernels,
// thread <-> channel or thread <-> token (vector), with the Euclidean pattern search on the matrix cores.  They
// compute the same definitions with the same arithmetic where it decides an integer (the quantizer's parameters and
// codes come from the shared pk_quant_arith.h; pattern selection gives the exact argmin of the metric in binary32,
// lowest index on ties) and store the same cache format (head_dim enters the layout formulas), so they meet the
// same parity bars; they are kept simple rather than tuned, and the tuned kernels of the other files keep their
// fixed head dimension.  The decode kernels here also serve head dimension 128 for head counts that the matrix-core
// decode does not take.
// Uniform and ragged appends, decode (with shared prefix and with per-sequence fill states), the window
// pattern and dequantize are covered (mining is in pk_mine.hip for every head dimension), on contiguous and on paged caches.
#pragma clang fp contract(off)

#include "pk_assign_mfma.h"
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
    const int64_t pos = a.c.map.pos(n, t);
    const int64_t orow = ((int64_t)n * (a.t1 - a.t0) + (t - a.t0)) * d + c;
    if (a.k_out) a.k_out[orow] = k_hat(a.c, a.patterns_k + (int64_t)set * a.P * d, pos, c, d, a.bits, a.G);
    if (a.v_out) a.v_out[orow] = v_hat(a.c, a.patterns_v + (int64_t)set * a.P * d, pos, c, d, a.bits, Gc, a.v_thresholded);
}

// ---------------------------------------------------------------------------------------------- decode
// Decode attention (Sec. 3.4) in plain vector arithmetic.  The context of a stream is cut into the same slots as in
// the tuned path (equal splits of the shared prefix's packed part, of the own packed part, then the own tail and
// the prefix's tail); a workgroup takes one slot of one stream for up to R = 8 query heads of the KV head at once (more heads: further workgroups), so
// the codes are taken apart once for all of them, and leaves an unnormalised partial (o, per-pattern softmax mass
// W, running maximum m in the log2 domain, sum l); a second kernel merges the partials and adds W . M_V once per
// head.  Scores: thread <-> token, score = q.M_K[k*] (a table formed once per workgroup) + sum_c q_c (s_c code_c +
// z_c).  Values: thread <-> channel over the tokens of the pass, o += p_t (s_t code_tc + z_t).  The reference of
// the online softmax is the running maximum; when a pass raises it, o, l and W are rescaled.  W is summed in LDS
// as 64-bit fixed point (unit 2^-31, weights are <= 1) with integer atomics, so the result does not depend on the
// order in which the tokens arrive.
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kMassUnit = 2147483648.f;   // 2^31
constexpr int kPass = kGenThreads;           // tokens per pass

__device__ __forceinline__ float half_of(const uint4 &v, int e)   // element e (0..7) of eight packed fp16
{
    const uint32_t w = e < 2 ? v.x : e < 4 ? v.y : e < 6 ? v.z : v.w;
    return h2f(__ushort_as_half((unsigned short)((e & 1) ? w >> 16 : w & 0xffffu)));
}
__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// LDS of a split workgroup, in this order (the 8-byte arrays first)
struct GenDecodeLds {
    unsigned long long *W;   // [P][R]   softmax mass per V pattern and head, fixed point
    long long *pos;          // [kPass]  packed position (or tail ring row) of the pass's tokens
    float *qf;               // [d][R]   the queries, channel-major; heads beyond the workgroup's are zero
    float *QM;               // [P][R]   q . M_K[p]
    float *sc;               // [kPass][R] softmax numerators of the pass
    float *red;              // [4][R]
    __device__ GenDecodeLds(unsigned char *base, int d, int P, int R)
    {
        W = reinterpret_cast<unsigned long long *>(base);
        pos = reinterpret_cast<long long *>(W + (size_t)P * R);
        qf = reinterpret_cast<float *>(pos + kPass);
        QM = qf + (size_t)d * R;
        sc = QM + (size_t)P * R;
        red = sc + (size_t)kPass * R;
    }
};
inline size_t gen_decode_lds_bytes(int d, int P, int R)
{
    return (size_t)P * R * 8 + (size_t)kPass * 8 + ((size_t)d * R + (size_t)P * R + (size_t)kPass * R + 4 * R) * 4;
}

template <int R, int BITS>
__global__ __launch_bounds__(kGenThreads) void gen_decode_split_kernel(DecodeArgs a)
{
    extern __shared__ __align__(16) unsigned char gen_decode_smem[];
    const int tid = threadIdx.x, d = a.d, P = a.P;
    const GenDecodeLds lds(gen_decode_smem, d, P, R);
    const int n = blockIdx.x, slot = blockIdx.y, h0 = blockIdx.z * R;   // the workgroup's first head of the KV head's r
    const int seq = n / a.n_kv_heads, head = n - seq * a.n_kv_heads;
    const int r = a.n_q_heads / a.n_kv_heads, nh = min(R, r - h0);
    const int n_packed = a.splits_prefix + a.splits_own, n_slots = n_packed + 2;
    const bool packed = slot < n_packed;
    const bool pre = slot < a.splits_prefix || slot == n_packed + 1;
    const CacheView &cv = pre ? a.prefix : a.own;
    int tq = cv.t_quant, tt = cv.t_tail, ts = cv.tail_start;
    if (!pre) own_state(a, seq, tq, tt, ts);
    const int stream = pre ? head : n;
    const int set = pre ? head : a.sets.set_of(n);
    int t_begin = 0, t_end = tt;
    if (packed) {
        t_begin = (pre ? slot : slot - a.splits_prefix) * a.chunk;
        t_end = min(tq, t_begin + a.chunk);
    }
    const int64_t pb = ((int64_t)n * n_slots + slot) * r + h0;   // partial of the workgroup's first query head
    if (t_end <= t_begin) {   // nothing in this slot: the merge skips partials whose sum is zero
        if (tid < nh) {
            a.part_ml[(pb + tid) * 2] = -INFINITY;
            a.part_ml[(pb + tid) * 2 + 1] = 0.f;
        }
        return;
    }
    const int Gc = a.G < d ? a.G : d, ng = d / Gc;
    const float scale2 = a.softmax_scale * kLog2e;

    for (int i = tid; i < d * R; i += kGenThreads) {
        const int c = i / R, h = i - c * R;
        lds.qf[i] = h < nh ? h2f(a.q[((int64_t)seq * a.n_q_heads + head * r + h0 + h) * d + c]) : 0.f;
    }
    for (int i = tid; i < P * R; i += kGenThreads) lds.W[i] = 0ull;
    __syncthreads();
    if (packed) {
        const __half *MK = a.patterns_k + (int64_t)set * P * d;
        for (int p = tid; p < P; p += kGenThreads) {
            float s[R];
#pragma unroll
            for (int h = 0; h < R; ++h) s[h] = 0.f;
            for (int c8 = 0; c8 < d / 8; ++c8) {
                const uint4 mv = *reinterpret_cast<const uint4 *>(MK + (int64_t)p * d + 8 * c8);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float x = half_of(mv, e);
#pragma unroll
                    for (int h = 0; h < R; ++h) s[h] = fmaf(lds.qf[(8 * c8 + e) * R + h], x, s[h]);
                }
            }
#pragma unroll
            for (int h = 0; h < R; ++h) lds.QM[p * R + h] = s[h];
        }
        __syncthreads();
    }

    float m_run[R], l_thr[R], acc[R];
#pragma unroll
    for (int h = 0; h < R; ++h) {
        m_run[h] = -INFINITY;
        l_thr[h] = 0.f;
        acc[h] = 0.f;
    }
    // value phase: thread <-> (channel, sub); the subs take the 16-token blocks (tail tokens) of a pass in turn
    const int n_sub = kGenThreads / d;
    const int vsub = tid / d, vc = tid - vsub * d;
    const bool v_active = vsub < n_sub;
    const uint32_t *vwords = reinterpret_cast<const uint32_t *>(cv.v_codes);

    for (int t0 = t_begin; t0 < t_end; t0 += kPass) {
        const int t = t0 + tid;
        const bool live = t < t_end;
        float s[R];
        int64_t where = 0;
#pragma unroll
        for (int h = 0; h < R; ++h) s[h] = -INFINITY;
        if (live && packed) {
            where = cv.map.pos(stream, t);
            const int idx = min((int)cv.k_idx[where], P - 1);
#pragma unroll
            for (int h = 0; h < R; ++h) s[h] = lds.QM[idx * R + h];
            const int64_t prow = (where / a.G) * d;
            for (int w = 0; w < d / 32; ++w) {
                uint32_t pl[BITS];
#pragma unroll
                for (int j = 0; j < BITS; ++j) pl[j] = cv.k_codes[(where * (d / 32) + w) * BITS + j];
#pragma unroll
                for (int o = 0; o < 4; ++o) {
                    const uint4 sv = *reinterpret_cast<const uint4 *>(cv.k_scale + prow + 32 * w + 8 * o);
                    const uint4 zv = *reinterpret_cast<const uint4 *>(cv.k_zero + prow + 32 * w + 8 * o);
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int cc = 8 * o + e;
                        uint32_t code = 0;
#pragma unroll
                        for (int j = 0; j < BITS; ++j) code |= ((pl[j] >> cc) & 1u) << j;
                        const float val = half_of(sv, e) * (float)code + half_of(zv, e);
#pragma unroll
                        for (int h = 0; h < R; ++h) s[h] = fmaf(lds.qf[(32 * w + cc) * R + h], val, s[h]);
                    }
                }
            }
        } else if (live) {
            int sl = ts + t;
            if (sl >= cv.ring_len) sl -= cv.ring_len;
            where = (int64_t)stream * cv.ring_len + sl;
#pragma unroll
            for (int h = 0; h < R; ++h) s[h] = 0.f;
            for (int c8 = 0; c8 < d / 8; ++c8) {
                const uint4 kv = *reinterpret_cast<const uint4 *>(cv.tail_k + where * d + 8 * c8);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float x = half_of(kv, e);
#pragma unroll
                    for (int h = 0; h < R; ++h) s[h] = fmaf(lds.qf[(8 * c8 + e) * R + h], x, s[h]);
                }
            }
        }
        // maximum of the pass per head
#pragma unroll
        for (int h = 0; h < R; ++h) {
            s[h] *= scale2;   // -inf stays -inf
            const float wm = wave_max(s[h]);
            if ((tid & 63) == 0) lds.red[(tid >> 6) * R + h] = wm;
        }
        lds.pos[tid] = where;
        __syncthreads();
        bool raised = false;   // the same in every thread
        float alpha[R];
#pragma unroll
        for (int h = 0; h < R; ++h) {
            const float pm = fmaxf(fmaxf(lds.red[h], lds.red[R + h]), fmaxf(lds.red[2 * R + h], lds.red[3 * R + h]));
            alpha[h] = 1.f;
            if (pm > m_run[h]) {
                alpha[h] = exp2f(m_run[h] - pm);   // 0 the first time
                m_run[h] = pm;
                raised = true;
            }
        }
        if (raised) {
#pragma unroll
            for (int h = 0; h < R; ++h) {
                acc[h] *= alpha[h];
                l_thr[h] *= alpha[h];
            }
            if (packed) {
                for (int p = tid; p < P; p += kGenThreads) {
#pragma unroll
                    for (int h = 0; h < R; ++h)
                        lds.W[p * R + h] = (unsigned long long)((double)lds.W[p * R + h] * (double)alpha[h]);
                }
                __syncthreads();   // before this pass's atomics
            }
        }
        float pw[R];
#pragma unroll
        for (int h = 0; h < R; ++h) {
            pw[h] = live ? exp2f(s[h] - m_run[h]) : 0.f;
            l_thr[h] += pw[h];
            lds.sc[tid * R + h] = pw[h];
        }
        if (live && packed) {
            const int vi = cv.v_idx[where];
            if (!(a.v_thresholded && vi == PK_NO_PATTERN)) {   // a token quantized without a pattern carries no mass
                const int vp = min(vi, P - 1);
#pragma unroll
                for (int h = 0; h < R; ++h) atomicAdd(&lds.W[vp * R + h], (unsigned long long)(pw[h] * kMassUnit));
            }
        }
        __syncthreads();

        const int n_here = min(kPass, t_end - t0);
        if (v_active && packed) {
            for (int b = vsub; 16 * b < n_here; b += n_sub) {
                const int64_t w0 = lds.pos[16 * b];   // the 16 tokens of a block are stored together
                const int64_t word = (((w0 >> 4) * 16 + (vc & 15)) * (d / 16) + (vc >> 4)) * (BITS / 2);
                uint32_t cw[BITS / 2];
#pragma unroll
                for (int j = 0; j < BITS / 2; ++j) cw[j] = vwords[word + j];
                const int64_t prow = ((w0 >> 4) * ng + vc / Gc) * 16;
                const uint4 sv[2] = {*reinterpret_cast<const uint4 *>(cv.v_scale + prow),
                                     *reinterpret_cast<const uint4 *>(cv.v_scale + prow + 8)};
                const uint4 zv[2] = {*reinterpret_cast<const uint4 *>(cv.v_zero + prow),
                                     *reinterpret_cast<const uint4 *>(cv.v_zero + prow + 8)};
#pragma unroll
                for (int k = 0; k < 16; ++k) {
                    uint32_t code = 0;
#pragma unroll
                    for (int j = 0; j < BITS; ++j) code |= ((cw[j / 2] >> (16 * (j % 2) + k)) & 1u) << j;
                    const float val = half_of(sv[k >> 3], k & 7) * (float)code + half_of(zv[k >> 3], k & 7);
#pragma unroll
                    for (int h = 0; h < R; ++h) acc[h] = fmaf(lds.sc[(16 * b + k) * R + h], val, acc[h]);
                }
            }
        } else if (v_active) {
            for (int k = vsub; k < n_here; k += n_sub) {
                const float val = h2f(cv.tail_v[lds.pos[k] * d + vc]);
#pragma unroll
                for (int h = 0; h < R; ++h) acc[h] = fmaf(lds.sc[k * R + h], val, acc[h]);
            }
        }
        __syncthreads();   // sc and pos are rewritten by the next pass
    }

    // the partial: sums over the threads in a fixed order
#pragma unroll
    for (int h = 0; h < R; ++h) {
        const float ws = wave_sum(l_thr[h]);
        if ((tid & 63) == 0) lds.red[(tid >> 6) * R + h] = ws;
    }
    if (v_active && vsub > 0) {
#pragma unroll
        for (int h = 0; h < R; ++h) lds.sc[(vsub * d + vc) * R + h] = acc[h];
    }
    __syncthreads();
    if (tid < d) {
        for (int k = 1; k < n_sub; ++k) {
#pragma unroll
            for (int h = 0; h < R; ++h) acc[h] += lds.sc[(k * d + tid) * R + h];
        }
#pragma unroll
        for (int h = 0; h < R; ++h)
            if (h < nh) a.part_o[(pb + h) * d + tid] = acc[h];
    }
    if (packed) {
        for (int p = tid; p < P; p += kGenThreads) {
#pragma unroll
            for (int h = 0; h < R; ++h)
                if (h < nh) a.part_w[(pb + h) * P + p] = (float)lds.W[p * R + h] * (1.f / kMassUnit);
        }
    }
#pragma unroll
    for (int h = 0; h < R; ++h) {
        if (tid == h && h < nh) {
            a.part_ml[(pb + h) * 2] = m_run[h];
            a.part_ml[(pb + h) * 2 + 1] = (lds.red[h] + lds.red[R + h]) + (lds.red[2 * R + h] + lds.red[3 * R + h]);
        }
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

template <int R>
hipError_t launch_gen_decode_split(const DecodeArgs &a, dim3 grid, size_t lds, hipStream_t s)
{
    if (a.bits == 2)
        hipLaunchKernelGGL((gen_decode_split_kernel<R, 2>), grid, dim3(kGenThreads), lds, s, a);
    else
        hipLaunchKernelGGL((gen_decode_split_kernel<R, 4>), grid, dim3(kGenThreads), lds, s, a);
    return hipGetLastError();
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
    // heads of a KV head per workgroup: the power of two that holds them, eight at most; more heads per KV head
    // (up to 64 by the configuration check) go to further workgroups along z
    const int r = a.n_q_heads / a.n_kv_heads;
    const int R = r > 4 ? 8 : r > 2 ? 4 : r > 1 ? 2 : 1;
    const dim3 grid(a.n_seq * a.n_kv_heads, a.splits_prefix + a.splits_own + 2, (r + R - 1) / R);
    const size_t lds = gen_decode_lds_bytes(a.d, a.P, R);
    hipError_t e = R == 8   ? launch_gen_decode_split<8>(a, grid, lds, s)
                   : R == 4 ? launch_gen_decode_split<4>(a, grid, lds, s)
                   : R == 2 ? launch_gen_decode_split<2>(a, grid, lds, s)
                            : launch_gen_decode_split<1>(a, grid, lds, s);
    if (e != hipSuccess) return e;
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
