// Pattern mining: Lloyd iterations for the K-means objective of Sec. 3.1 Eq. 4, one independent
// problem per pattern set (layer x KV head, K and V separately).
//
// One iteration = mine_step_kernel (assignment step and per-chunk cluster sums, both on the matrix
// cores) followed by mine_update_kernel (fixed-order reduction over the chunks, mean, fp16 rounding).
// Every sum is formed in a fixed order, so results are reproducible bit for bit.
#include <type_traits>

#include "pk_assign_mfma.h"
#include "pk_internal.h"

namespace pk {

namespace {

// patterns[s][p] <- x[s][p], p < P  (initialisation from the first P vectors, where no step follows: a first step reads them itself)
__global__ __launch_bounds__(256) void mine_init_kernel(MineArgs a)
{
    const int s = blockIdx.y;
    const int w = blockIdx.x * 256 + threadIdx.x;
    if (w >= a.P * a.d / 8) return;   // 16-byte pieces; a set's vectors are dense rows, like the patterns
    const uint4 v = *reinterpret_cast<const uint4 *>(a.x + (int64_t)s * a.set_stride + (int64_t)w * 8);
    *reinterpret_cast<uint4 *>(a.patterns + (int64_t)s * a.P * a.d + (int64_t)w * 8) = v;
}

// Assignment step + partial cluster sums of one chunk of one set.  64*NW threads.
// The chunk is walked in sub-tiles of 16*NT*NW vectors: every wave assigns 16*NT of them on the matrix cores
// (NT tiles per pass over the table) and leaves them, with their indices, in an LDS tile.  The cluster sums are a second contraction on the
// matrix cores, sums[p][c] += sum_t onehot[p][t] x[t][c].  The NW waves (4, or 8 when the table is large and
// only one workgroup fits a CU) split the pattern tiles (and, when there are fewer pattern tiles than waves,
// the 8 channel tiles as well), so each wave forms the one-hot operand of its own pattern rows only and keeps
// its accumulator tiles in registers for the whole chunk.  The vector operand is x transposed (the
// contraction runs over vectors, the tile is stored vector-major): it comes out of LDS with the transposing
// 64-bit read, in which lane i of a 16-lane group receives element i of four rows whose 32-byte pieces the
// group's lanes address four to a row.  The one-hot operand is formed in packed fp16 as
// clamp(1 - (idx_t - p)^2, 0, 1), which is exactly 1 or 0 for integers below 256; products are exact and the
// accumulation order is fixed by the instruction sequence, so the sums are reproducible.
// All three head dimensions take this kernel: a search and a cluster-sum kernel of their own, which head dimensions 96 and
// 256 used to have, read the vectors twice and summed them on the vector ALUs; 2 x 10 iterations on 256 sets x 8191
// vectors of 96 channels at 64 patterns 9.40 -> 2.14 ms (step 103 us), of 256 channels (8192 vectors) 19.9 -> 5.0 ms; 64
// sets of 256 channels at 200 patterns 14.0 -> 3.4 ms.  Bound by instruction issue and LDS reads, not by the vectors (39 us
// of traffic in a step at 96 channels).
// Sorted sub-tiles (step_sorts): a wave sums a few pattern tiles only, but walked every vector of the sub-tile and multiplied it by
// a one-hot operand that is mostly zero.  The vectors are stored to the tile in the order of the wave that sums their
// pattern instead (a counting sort: ranks by ballot, the counts of all waves through LDS, a scan), and a wave walks its own run
// of rows, 32 at a time from a multiple of four; rows of its neighbours in the first and last step match none of its
// patterns.  The barrier of the counts replaces the one behind the sums.  The next sub-tile's vectors are requested before the
// search, into a buffer of their own, so that they are in flight for the whole of it (without the sort that gained nothing).
// A quarter (two thirds at 256 patterns) of the matrix instructions less per vector; 256 sets, 2 x 10 iterations: 32768
// vectors at 128 patterns 14.8 -> 13.8 ms (15.1 -> 14.2 on another card); 8 sets x 16384 at 256
// patterns 817 -> 787 us; 64 sets of 256 channels at 200 patterns 3.50 -> 3.16 ms; 256 sets x 8192 at 66, 80, 96 and 112 patterns
// 3.24 -> 3.01, 3.33 -> 3.10, 3.55 -> 3.43 and 3.81 -> 3.81 ms.  With 64 patterns the sort costs more than
// the two steps that it saves (2.6 -> 2.8 ms on 256 sets x 8192), and at 256 channels and 128 patterns it gained nothing
// (2.79 -> 2.80 ms).  Neither matrix cores (24 % busy) nor vector ALUs (44 %) nor HBM (57 %) bound the step at 128
// patterns: two waves per SIMD, a third of their time waiting at barriers and for loads; four waves per SIMD at 96
// channels gained 3 %, at 128 they spill.
// With XC < D (256 channels and more than 128 patterns: the table alone takes 139 KB) the vectors pass through the LDS tile
// XC channels at a time, the sums of those channels being formed between two barriers each; a wave's own rows of that tile
// then serve as its re-evaluation row.
// Dynamic LDS: [table pad16(P) rows] [-norm2/2 pad16(P)] [cnt pad16(P) + 4] [xs 16 NT NW rows of XC]
//              [idx 16 NT NW halves] [xrow NW*D halves, unless XC < D]
template <int XC>
constexpr int kMineXsOf = XC + 16;   // halves per row of the vector tile: 8 words modulo 16, so the eight rows that 32
                                     // lanes of a transposing read touch (8 words each) fall on 64 distinct banks

// sum over the lanes up to this one (the first N lanes, 16 or 64)
template <int N>
__device__ __forceinline__ int wave_scan(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);   // row shifts by 1, 2, 4 and 8
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);
    if constexpr (N > 16) {
        v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
        v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
    }
    return v;
}

typedef _Float16 half2m __attribute__((ext_vector_type(2)));
typedef short short4m __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4m *lds_short4_ptr;

constexpr bool step_sorts(int D, int NPT) { return NPT == 16 || (NPT == 8 && D <= 128); }

template <int D, int NPT, int NW, int NT, int XC>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NT == 1 && NPT <= 4 && D <= 128 ? 4 : 2))) void mine_step_kernel(MineArgs a, int chunk, int outputs)
{
    constexpr int KS = D / 32, kXs = kMineXsOf<XC>;
    extern __shared__ __align__(16) unsigned char smem[];
    const int P = a.P;
    __half *tab_s = reinterpret_cast<__half *>(smem);
    float *norm_s = reinterpret_cast<float *>(smem + (size_t)pad16(P) * kTabStrideOf<D> * 2);
    int *cnt = reinterpret_cast<int *>(norm_s + pad16(P));
    const int kNone = pad16(P);   // index of a vector without a nearest pattern: counted behind the table's rows, summed nowhere
    __half *xs = reinterpret_cast<__half *>(cnt + pad16(P) + 4);
    constexpr int ST = 16 * NT * NW;     // vectors per sub-tile: NT 16-vector tiles per wave
    __half *idx_s = xs + ST * kXs;       // pattern index of every row of the sub-tile, as an fp16 number
    __shared__ float red_s[NW];
    constexpr bool kSort = step_sorts(D, NPT);
    constexpr int kStepUnroll = kSort ? 1 : ST / 32;
    __shared__ int bucket_s[kSort ? NW * NW : 1];   // [bucket][wave]: vectors of the wave's in the bucket (the pattern rows that one wave sums)

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = lane & 15, kb = lane >> 4;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    static_assert(XC == D || 16 * NT * kXs >= D, "a wave's rows of the vector tile hold one vector");
    __half *xrow_s = XC == D ? idx_s + ST + wave * D : xs + wave * NT * 16 * kXs;
    const int ck = blockIdx.x, s = blockIdx.y;
    const int t_begin = ck * chunk, n_tok = min(chunk, a.T - t_begin);
    const __half *xg = a.x + (int64_t)s * a.set_stride + (int64_t)t_begin * D;
    const __half *Mg = a.table + (int64_t)s * a.table_stride;

    auto load_tile = [&](int sub, uint4 (&xb)[NT][KS]) {
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int tok = min(sub * ST + (wave * NT + j) * 16 + n, n_tok - 1);   // rows past the chunk repeat its last vector
#pragma unroll
            for (int k = 0; k < KS; ++k) xb[j][k] = *reinterpret_cast<const uint4 *>(xg + (int64_t)tok * D + 32 * k + 8 * kb);
        }
    };
    constexpr bool kAhead = kSort && D <= 128 && NT > 1;   // a vector buffer more: loads are in flight for a whole sub-tile
    uint4 xb[NT][KS], xn[NT][KS];
    load_tile(0, kAhead ? xn : xb);

    for (int i = tid; i <= kNone; i += 64 * NW) cnt[i] = 0;
    stage_patterns<D>(Mg, P, tab_s, norm_s, red_s, 64 * NW);   // ends with a barrier
    PatternTable tb;
    tb.lds_rows = tab_s;
    tb.nh = norm_s;
    tb.norm2_max = red_s[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) tb.norm2_max = fmaxf(tb.norm2_max, red_s[w]);
    tb.P = P;

    // this wave's share of the sums: PW pattern tiles from pt0, CW channel tiles from ct0.  (With fewer pattern tiles than
    // waves the channel tiles are split too; where they do not divide - 96 channels, one pattern tile - the last wave
    // has none and repeats tile 0 without storing it.)
    constexpr int CT = D / 16, CTX = XC / 16;   // channel tiles of a vector, and of the part of it that is in LDS
    constexpr int PW = NPT >= NW ? NPT / NW : 1;
    constexpr int CW = NPT >= NW ? CT : (CT * NPT + NW - 1) / NW;
    constexpr bool kEven = NPT >= NW || CT * NPT % NW == 0;   // every wave has CW channel tiles of its own
    static_assert(XC == D || CW == CT, "parts of the channels only where a wave takes all of them");
    const int pt0 = NPT >= NW ? wave * PW : wave % NPT;
    const int ct0 = NPT >= NW ? 0 : (wave / NPT) * CW;
    floatx4_t acc[PW][CW];
    half2m prow[PW];   // this lane's pattern row of every tile, as a packed pair
#pragma unroll
    for (int pi = 0; pi < PW; ++pi) {
#pragma unroll
        for (int ci = 0; ci < CW; ++ci) acc[pi][ci] = floatx4_t{0.f, 0.f, 0.f, 0.f};
        const _Float16 v = (_Float16)(float)(16 * (pt0 + pi) + n);
        prow[pi] = half2m{v, v};
    }
    const half2m one2 = {(_Float16)1.f, (_Float16)1.f};

    const int n_sub = (n_tok + ST - 1) / ST;
    for (int sub = 0; sub < n_sub; ++sub) {
        if constexpr (kAhead) {
#pragma unroll
            for (int j = 0; j < NT; ++j) {
#pragma unroll
                for (int k = 0; k < KS; ++k) xb[j][k] = xn[j][k];
            }
            if (sub + 1 < n_sub) load_tile(sub + 1, xn);
        }
        int bi[NT];
        float bv[NT], x2[NT];
        bool flag[NT];
        assign_tiles_mfma<NT, KS>(xb, tb, lane, bi, bv, x2, flag);
        int at[NT];   // row of the tile that takes the lane's vector
        bool lost[NT];   // the lane's vector belongs to no cluster: its row is cleared again (0 * infinity is not 0)
        int step0 = 0, n_steps = ST / 32;   // this wave's 32-vector steps: rows step0 .. step0 + 32 n_steps - 1
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            float bd = fmaxf(bv[j], 0.f);
            if (NPT == 1 && P == 1) flag[j] = !(x2[j] < INFINITY);
            at[j] = (wave * NT + j) * 16 + n;
            const int tok = sub * ST + at[j];
            lost[j] = false;
            resolve_flagged<KS, true>(xb[j], flag[j], xrow_s, tb, lane, kNone, bi[j], bd, [&](int b) { lost[j] = b == kNone; });
            if (kb == 0) {
                if (tok < n_tok) {
                    // per-vector outputs only where somebody reads them: indices from the last step (if asked
                    // for), distances when the objective is reported
                    if (outputs & 1) a.assign[(int64_t)s * a.T + t_begin + tok] = bi[j] < P ? bi[j] : 0x7fffffff;
                    if (outputs & 2) a.best[(int64_t)s * a.T + t_begin + tok] = bd;
                    atomicAdd(&cnt[bi[j]], 1);
                }
            }
        }
        if constexpr (kSort) {
            // lane (n, kb = j) speaks for vector n of tile j: its bucket, and its rank among the wave's vectors of that bucket
            int mine = bi[0];
#pragma unroll
            for (int j = 1; j < NT; ++j) mine = kb == j ? bi[j] : mine;
            const int bucket = min(mine / (16 * PW), NW - 1);   // (a vector without a nearest pattern gets a row too, of zeros)
            int rank = 0;
            int count = 0;   // lane w: vectors in bucket w
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const uint64_t in = __ballot(bucket == w) & ((1ull << 16 * (NT - 1) << 16) - 1);
                const int below = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(in >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)in, 0u));
                rank = bucket == w ? below : rank;
                count = lane == w ? __popcll(in) : count;
            }
            if (lane < NW) bucket_s[lane * NW + wave] = count;
            __syncthreads();   // also: every wave has read the previous sub-tile's rows
            // first row of every (bucket, wave): the sum of all entries before it
            const int own = lane < NW * NW ? bucket_s[lane] : 0;
            const int upto = wave_scan<NW * NW>(own);
            const int first = upto - own;
            const int row = __shfl(first, bucket * NW + wave) + rank;
#pragma unroll
            for (int j = 0; j < NT; ++j) at[j] = __shfl(row, 16 * j + n);
            const int start = __builtin_amdgcn_readlane(first, wave_u * NW), end = __builtin_amdgcn_readlane(upto, wave_u * NW + NW - 1);
            step0 = start & ~3;
            n_steps = end > start ? (end - step0 + 31) / 32 : 0;
            step0 = min(step0, ST - 32 * n_steps);   // the last step stays inside the tile
        }
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const bool in = sub * ST + (wave * NT + j) * 16 + n < n_tok;
            if constexpr (XC == D) {
#pragma unroll
                for (int k = 0; k < KS; ++k)   // a row past the chunk is stored as zeros, so it adds nothing to any sum
                    *reinterpret_cast<uint4 *>(xs + at[j] * kXs + 32 * k + 8 * kb) = in ? xb[j][k] : make_uint4(0u, 0u, 0u, 0u);
            }
            if (kb == 0) idx_s[at[j]] = __float2half_rn((float)bi[j]);   // integers below 2048 are exact
        }
#pragma unroll
        for (int part = 0; part < D / XC; ++part) {   // channels part * XC .. of the vectors
            if constexpr (XC < D) {
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    const bool in = sub * ST + (wave * NT + j) * 16 + n < n_tok;
#pragma unroll
                    for (int k = 0; k < XC / 32; ++k)
                        *reinterpret_cast<uint4 *>(xs + at[j] * kXs + 32 * k + 8 * kb) = in ? xb[j][part * (XC / 32) + k] : make_uint4(0u, 0u, 0u, 0u);
                }
            }
            if (!kAhead && part == D / XC - 1 && sub + 1 < n_sub) load_tile(sub + 1, xb);   // in flight during the accumulation
#pragma unroll
            for (int j = 0; j < NT; ++j) {   // (behind the loads, which the next sub-tile waits for)
                if (__builtin_expect(lost[j], 0)) {
#pragma unroll
                    for (int k = 0; k < XC / 32; ++k) *reinterpret_cast<uint4 *>(xs + at[j] * kXs + 32 * k + 8 * kb) = make_uint4(0u, 0u, 0u, 0u);
                }
            }
            __syncthreads();
#pragma unroll kStepUnroll
            for (int ks = 0; ks < n_steps; ++ks) {
                // 32 rows per step; this lane's k-slots 0-3 are rows ta .. ta+3, its slots 4-7 the ones 16 later
                const int ta = step0 + 32 * ks + 4 * kb;
                const uint2 ia = *reinterpret_cast<const uint2 *>(idx_s + ta);
                const uint2 ib = *reinterpret_cast<const uint2 *>(idx_s + ta + 16);
                const half2m idh[4] = {__builtin_bit_cast(half2m, ia.x), __builtin_bit_cast(half2m, ia.y),
                                       __builtin_bit_cast(half2m, ib.x), __builtin_bit_cast(half2m, ib.y)};
                uint4 av[PW];
#pragma unroll
                for (int pi = 0; pi < PW; ++pi) {
                    uint32_t aop[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const half2m d = idh[j] - prow[pi];
                        half2m oh = one2 - d * d;                       // 1 where the index equals the row, <= 0 elsewhere
                        oh = __builtin_elementwise_min(__builtin_elementwise_max(oh, half2m{(_Float16)0.f, (_Float16)0.f}), one2);   // folds into the clamp bit
                        aop[j] = __builtin_bit_cast(uint32_t, oh);
                    }
                    av[pi] = make_uint4(aop[0], aop[1], aop[2], aop[3]);
                }
                // lane n of group kb addresses the 8-byte piece (n & 3) of row ta + n / 4 and receives column n of rows ta .. ta+3
                const __half *piece = xs + (ta + (n >> 2)) * kXs + 4 * (n & 3);
                constexpr int CP = XC == D ? CW : CTX;   // channel tiles of this part that the wave takes
#pragma unroll
                for (int ci = 0; ci < CP; ++ci) {
                    const int at = XC == D ? (kEven || ct0 + ci < CT ? ct0 + ci : 0) : ci;   // channel tile inside the part
                    const short4m lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(piece + 16 * at));
                    const short4m hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(piece + 16 * kXs + 16 * at));
                    const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
                    const uint4 bop = make_uint4(l2.x, l2.y, h2.x, h2.y);
                    constexpr int kParts = D / XC;
                    const int ai = kParts == 1 ? ci : part * CTX + ci;
#pragma unroll
                    for (int pi = 0; pi < PW; ++pi) acc[pi][ai] = mfma_f16(av[pi], bop, acc[pi][ai]);
                }
            }
            // (sorted: the next sub-tile's barrier behind its search comes before anything is stored to the tile again)
            if (!kSort || XC < D) __syncthreads();
        }
    }
    // partial sums of the chunk: D rows 4kb+i = pattern 16(pt0 + pi) + 4kb + i, column n = channel 16(ct0 + ci) + n
    const int64_t o = ((int64_t)s * a.tsplit + ck) * P;
#pragma unroll
    for (int pi = 0; pi < PW; ++pi) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int pr = 16 * (pt0 + pi) + 4 * kb + i;
            if (pr < P) {
#pragma unroll
                for (int ci = 0; ci < CW; ++ci)
                    if (kEven || ct0 + ci < CT) a.psum[(o + pr) * D + 16 * (ct0 + ci) + n] = acc[pi][ci][i];
            }
        }
    }
    for (int i = tid; i < P; i += 64 * NW) a.pcnt[o + i] = cnt[i];
}

// update step: centroid = mean of members (binary32 division), rounded to fp16;
// an empty cluster keeps its centroid
template <int D>
__global__ __launch_bounds__(D) void mine_update_kernel(MineArgs a)   // thread <-> channel
{
    const int p = blockIdx.x, s = blockIdx.y, c = threadIdx.x;
    const int64_t o0 = (int64_t)s * a.tsplit * a.P + p, step = a.P;
    // chunks in increasing order, up to 32 loads in flight at a time; the order of the additions is fixed
    float sum = 0.f;
    int cnt = 0, ts = 0;
    auto take = [&](auto count) {
        constexpr int N = decltype(count)::value;
        float v[N];
        int k[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            v[u] = a.psum[(o0 + (ts + u) * step) * D + c];
            k[u] = a.pcnt[o0 + (ts + u) * step];
        }
#pragma unroll
        for (int u = 0; u < N; ++u) {
            sum += v[u];
            cnt += k[u];
        }
        ts += N;
    };
    while (ts + 32 <= a.tsplit) take(std::integral_constant<int, 32>());
    if (ts + 16 <= a.tsplit) take(std::integral_constant<int, 16>());
    if (ts + 8 <= a.tsplit) take(std::integral_constant<int, 8>());
    if (ts + 4 <= a.tsplit) take(std::integral_constant<int, 4>());
    if (ts + 2 <= a.tsplit) take(std::integral_constant<int, 2>());
    if (ts < a.tsplit) take(std::integral_constant<int, 1>());
    __half *out = a.patterns + ((int64_t)s * a.P + p) * D + c;
    if (cnt > 0)
        *out = __float2half_rn(sum / (float)cnt);
    else if (a.table != a.patterns)   // (the first step, whose table is not the caller's)
        *out = a.table[(int64_t)s * a.table_stride + p * D + c];
}

// inertia of one assignment step: fixed-order sum of the best distances
__global__ __launch_bounds__(256) void mine_inertia_kernel(MineArgs a, int it)
{
    __shared__ float red[256];
    const int s = blockIdx.x, tid = threadIdx.x;
    const float *b = a.best + (int64_t)s * a.T;
    float acc = 0.f;
    for (int t = tid; t < a.T; t += 256) acc += b[t];
    red[tid] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (tid < w) red[tid] += red[tid + w];
        __syncthreads();
    }
    if (tid == 0) a.inertia[(int64_t)s * a.iters + it] = red[0];
}

// Decode-stage pattern of a window (Sec. 3.1 "Decoding Stage", Eq. 5): per channel (min + max) / 2 over the
// window's vectors, in binary32 (exact for fp16 inputs), rounded to fp16.  One workgroup per window;
// thread <-> (channel, token parity).
__global__ __launch_bounds__(256) void window_pattern_kernel(const __half *x, int64_t set_stride, int n, __half *out,
                                                             int64_t out_stride)
{
    __shared__ float s_mn[kD], s_mx[kD];
    const int c = threadIdx.x & (kD - 1), par = threadIdx.x >> 7;
    const __half *xs = x + (int64_t)blockIdx.x * set_stride + c;
    float mn = INFINITY, mx = -INFINITY;
    for (int t = par; t < n; t += 2) {
        const float v = h2f(xs[(int64_t)t * kD]);
        mn = fminf(mn, v);
        mx = fmaxf(mx, v);
    }
    if (par == 1) {
        s_mn[c] = mn;
        s_mx[c] = mx;
    }
    __syncthreads();
    if (par == 0) {
        mn = fminf(mn, s_mn[c]);
        mx = fmaxf(mx, s_mx[c]);
        out[(int64_t)blockIdx.x * out_stride + c] = __float2half_rn((mn + mx) * 0.5f);
    }
}

// Instantiation for a head dimension and number of patterns: 16 * npt >= P table rows, nw waves, nt 16-vector tiles per wave
// and pass over the table, xc channels of the vectors in LDS at a time.
// wide: eight waves per workgroup where four would leave the chip's wave slots empty (few_chunks below).
struct StepShape {
    int npt, nw, nt, xc;
};
constexpr StepShape step_shape(int D, int P, bool wide = false)
{
    // 8 waves share the table when only one workgroup fits a CU (P > 128, or P > 64 at 256 channels, whose table rows and
    // accumulators are twice as large; at 128 patterns of 128 channels two 4-wave workgroups measured faster than one
    // 8-wave group).  From 128 patterns on a wave assigns two 16-vector tiles per table pass: reading the table out of LDS
    // is what limits the assignment there, and every tile read then serves 32 vectors (at 64 patterns and below, and with
    // the eight-step tiles of 256 channels, the smaller tile and its fewer registers win).
    const int npt = P <= 16 ? 1 : P <= 32 ? 2 : P <= 64 ? 4 : P <= 128 ? 8 : 16;
    const int nw = npt == 16 || (D == 256 && npt == 8) ? 8 : 4;
    const int nt = npt >= 8 && D != 256 ? 2 : 1;
    if (wide) return {npt, 8, 1, D};
    return {npt, nw, nt, D == 256 && npt == 16 ? 64 : D};
}

size_t step_lds_bytes(int D, int P, const StepShape &h)
{
    size_t b = (size_t)pad16(P) * (D + 16) * 2;
    b += (size_t)pad16(P) * 4 + (size_t)(pad16(P) + 4) * 4 + 16 * h.nw * h.nt * (size_t)(h.xc + 16) * 2 + 16 * h.nw * h.nt * 2;
    if (h.xc == D) b += (size_t)h.nw * D * 2;
    return (b + 15) / 16 * 16;
}

}  // namespace

// Workgroups of the step kernel that one compute unit holds at a time: registers allow four 4-wave groups up to 64 patterns
// (two at 256 channels); the table and the vector tile in LDS allow two at 128 patterns and one 8-wave group above.
static int step_groups_per_cu(int P, int d)
{
    const StepShape h = step_shape(d, P);
    return h.nw == 8 ? 1 : h.npt <= 4 && d <= 128 ? 4 : 2;
}

static int mine_chunk(int T, int n_sets, int P, int d)
{
    // One resident round of workgroups over the chip's 256 compute units: all chunks then run side by side and
    // take the same time, and every chunk writes its P*d partial sums once, so fewer, longer chunks also
    // mean less traffic.  At most 64 chunks per set, none shorter than 256 vectors.
    const int64_t slots = 256 * step_groups_per_cu(P, d);
    const int64_t per_set = slots / n_sets > 1 ? slots / n_sets : 1;
    int64_t c = (T + per_set - 1) / per_set;
    if (c < (T + 63) / 64) c = (T + 63) / 64;
    c = (c + 127) / 128 * 128;
    if (c < 256) c = 256;
    return (int)c;
}

static int chunks_of(int T, int n_sets, int P, int d) { return (T + mine_chunk(T, n_sets, P, d) - 1) / mine_chunk(T, n_sets, P, d); }
int mine_tsplit(int T, int n_sets, int P)
{
    // (at 256 channels no more groups fit a CU than at 128, at 96 as many)
    return chunks_of(T, n_sets, P, kD);
}

// All iterations for 16 * NPT patterns or fewer at head dimension D
template <int D, int NPT, bool WIDE>
static hipError_t launch_iterations(const MineArgs &a_in, hipStream_t s)
{
    constexpr StepShape h = step_shape(D, 16 * NPT, WIDE);
    constexpr auto step = mine_step_kernel<D, NPT, h.nw, h.nt, h.xc>;
    static LdsOptIn opt_in;   // the most this instantiation needs: a table of 16 * NPT patterns
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(step), opt_in, step_lds_bytes(D, 16 * NPT, h));
    if (e != hipSuccess) return e;
    MineArgs a = a_in;
    a.tsplit = chunks_of(a.T, a.n_sets, a.P, D);
    const int chunk = mine_chunk(a.T, a.n_sets, a.P, D);
    const size_t lds = step_lds_bytes(D, a.P, h);
    if (!a.init_given && a.iters < 1) {
        hipLaunchKernelGGL(mine_init_kernel, dim3((a.P * D / 8 + 255) / 256, a.n_sets), dim3(256), 0, s, a);
        return hipGetLastError();
    }
    for (int it = 0; it < a.iters; ++it) {
        const bool from_vectors = it == 0 && !a.init_given;
        a.table = from_vectors ? a.x : a.patterns;
        a.table_stride = from_vectors ? a.set_stride : (int64_t)a.P * D;
        const int outputs = (a.assign && it == a.iters - 1 ? 1 : 0) | (a.inertia ? 2 : 0);
        hipLaunchKernelGGL(step, dim3(a.tsplit, a.n_sets), dim3(64 * h.nw), lds, s, a, chunk, outputs);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (a.inertia) {
            hipLaunchKernelGGL(mine_inertia_kernel, dim3(a.n_sets), dim3(256), 0, s, a, it);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        hipLaunchKernelGGL(mine_update_kernel<D>, dim3(a.P, a.n_sets), dim3(D), 0, s, a);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

// Whether the workgroups of a step are so few that eight waves in each still have slots side by side: up to 64 patterns two such groups
// per CU (one at 256 channels, whose vector tile takes the LDS), up to 128 patterns one.  A step then walks half as many
// sub-tiles, one after the other, as with four waves; 10 iterations, four and eight waves: 8 sets x 1024 vectors at 64 patterns 134 and 111 us,
// 8 x 8192 185 and 164, 4 x 32768 258 and 215, 16 x 8192 225 and 220; 8 x 8192 at 128 patterns 242 and 233, of 96 channels at 64 164 and
// 147, of 256 channels 259 and 235.  Not with more groups (32 x 8192 315 and 344; at 128 patterns 16 x 8192 312 and 365), and not beyond
// 128 patterns, where eight waves are the rule and two tiles per table pass worth more.  (Sixteen waves: 168 us for 8 x 8192, 265 for 16 x 8192.)
template <int D, int NPT>
static bool few_chunks(const MineArgs &a)
{
    const int64_t groups = (int64_t)a.n_sets * chunks_of(a.T, a.n_sets, a.P, D);
    return groups <= (NPT <= 4 && D <= 128 ? 512 : 256);
}

template <int D, int NPT>
static hipError_t launch_size(const MineArgs &a, hipStream_t s)
{
    if constexpr (NPT <= 4 || (NPT == 8 && D <= 128)) {
        if (few_chunks<D, NPT>(a)) return launch_iterations<D, NPT, true>(a, s);
    }
    return launch_iterations<D, NPT, false>(a, s);
}

template <int D>
static hipError_t launch_mine_of(const MineArgs &a, hipStream_t s)
{
    switch (step_shape(D, a.P).npt) {
    case 1: return launch_size<D, 1>(a, s);
    case 2: return launch_size<D, 2>(a, s);
    case 4: return launch_size<D, 4>(a, s);
    case 8: return launch_size<D, 8>(a, s);
    default: return launch_size<D, 16>(a, s);
    }
}

hipError_t launch_mine(const MineArgs &a, hipStream_t s)
{
    return a.d == kD ? launch_mine_of<kD>(a, s) : a.d == 96 ? launch_mine_of<96>(a, s) : a.d == 256 ? launch_mine_of<256>(a, s) : hipErrorInvalidValue;
}

hipError_t launch_window_pattern(const __half *x, int64_t set_stride, int n_sets, int n, __half *out, int64_t out_stride,
                                 hipStream_t s)
{
    hipLaunchKernelGGL(window_pattern_kernel, dim3(n_sets), dim3(256), 0, s, x, set_stride, n, out, out_stride);
    return hipGetLastError();
}

}  // namespace pk
