// Centroid-based top-p selection (paper Section 4.2).
//
//   select_scores_kernel   cq_i . ck_j for all pairs, on the matrix cores (not for few rows, select_fused)
//   select_row_kernel      one workgroup per (head, query cluster i):
//       S_ij  = cq_i . ck_j / sqrt(d)                                  (Eq. 1)
//       P'_ij = |K_j| exp(S_ij) / sum_k |K_k| exp(S_ik)                (Eq. 2)
//       sort j by (P' descending, j ascending), exclusive prefix sum of P',
//       keep sorted position t iff the mass before it is < top_p, write the
//       kept j in ascending order to a per-row list.
//   select_compact_kernel  row lengths -> CSR row_ptr, lists -> col_idx,
//       density (Section 5.1).
//
// The row maximum of S is subtracted before exp; it cancels in Eq. 2.
#include <algorithm>
#include <type_traits>

#include "svg2_common.h"

namespace svg2 {

static constexpr int SEL_THREADS = 256;

__device__ __forceinline__ float block_reduce_max(float v, float *s_red)
{
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) s_red[w] = v;
    __syncthreads();
    float r = s_red[0];
    for (int i = 1; i < SEL_THREADS / 64; ++i) r = fmaxf(r, s_red[i]);
    return r;
}

template <typename T> __device__ __forceinline__ T block_reduce_sum(T v, T *s_red)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) s_red[w] = v;
    __syncthreads();
    T r = s_red[0];
    for (int i = 1; i < SEL_THREADS / 64; ++i) r += s_red[i];
    return r;
}

// Exclusive prefix sums of per-thread counts over the workgroup (thread order).
__device__ __forceinline__ int block_exclusive_scan(int v, int *s_red, int *total)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int incl = v;
    for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(incl, o);
        if (lane >= o) incl += u;
    }
    __syncthreads();
    if (lane == 63) s_red[w] = incl;
    __syncthreads();
    int before = 0, all = 0;
    for (int i = 0; i < SEL_THREADS / 64; ++i) {
        if (i < w) before += s_red[i];
        all += s_red[i];
    }
    *total = all;
    return before + incl - v;
}

// Exclusive prefix sums of 256 per-thread floats: the doubling scan x[t] += x[t - o], o = 1, 2, .. 128, by one wavefront
// that holds four elements per lane (element 64 w + lane in register w), so that the eight steps need no barriers.  The
// association of the additions is part of the selection (the mass in front of a cluster is compared with p).
__device__ __forceinline__ float block_exclusive_scan_f32(float v, float *s_scan)
{
    const int tid = threadIdx.x, lane = tid & 63;
    __syncthreads();
    s_scan[tid] = v;
    __syncthreads();
    if (tid < 64) {
        float x[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) x[w] = s_scan[64 * w + lane];
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            float r[4];
#pragma unroll
            for (int w = 0; w < 4; ++w) r[w] = __shfl(x[w], (lane - o) & 63);
#pragma unroll
            for (int w = 3; w >= 0; --w) {
                if (lane >= o) x[w] += r[w];
                else if (w > 0) x[w] += r[w - 1];
            }
        }
        x[3] += x[2]; x[2] += x[1]; x[1] += x[0];                           // o = 64
        x[3] += x[1]; x[2] += x[0];                                         // o = 128
#pragma unroll
        for (int w = 0; w < 4; ++w) s_scan[64 * w + lane] = x[w];
    }
    __syncthreads();
    return s_scan[tid] - v;
}

// scores[h][i][j] = cq_i . ck_j.  grid (ceil(Ck / 128), ceil(Cq / 32), H), a 32 x 32 tile per wavefront.
// Matrix instruction 32x32x2 fp32 with the contraction index in its natural order: each instruction adds the products of
// elements 2 s and 2 s + 1 with a rounding behind each, so a score is bit for bit the chain of fmaf over k = 0 .. d - 1.
// The rows come in whole (coalesced, all requested at once) and go to LDS with their even elements in front of the odd
// ones, so that a lane half reads its share in 16-byte pieces.  What bounds it is that one round trip to memory.  One
// thread per pair inside select_row_kernel made every lane of a load read a row of its own, for every query cluster again:
// 24 heads of 100 x 500 clusters, d = 128: 106 us for scores and rows, 12 + 23 us now; 8 heads of 100 x 2000: 207 us,
// 13 + 38 us now.
typedef __attribute__((ext_vector_type(16))) float f32x16;
template <int D> static constexpr size_t select_scores_lds() { return (size_t)160 * (D + 8) * sizeof(float); }

template <int D>
__global__ __launch_bounds__(256) void select_scores_kernel(const float *__restrict__ cq, const float *__restrict__ ck,
                                                            int Cq, int Ck, float *__restrict__ scores)
{
    constexpr int ROW = D + 8, ODD = D / 2 + 4;         // odd elements start 4 floats further: the halves differ in bank
    constexpr int LPR = D / 4, RPP = 256 / LPR;         // lanes per row, rows per pass of the workgroup
    extern __shared__ __align__(16) float s_x[];        // [32] rows of cq, [128] rows of ck
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5, col = lane & 31;
    const int h = blockIdx.z, i0 = blockIdx.y * 32, j0 = blockIdx.x * 128;
    {
        const int r0 = tid / LPR, c = tid % LPR;
        constexpr int NP = 160 / RPP;
        float4 v[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int r = p * RPP + r0;
            const float *src = r < 32 ? cq + ((size_t)h * Cq + min(i0 + r, Cq - 1)) * D
                                      : ck + ((size_t)h * Ck + min(j0 + r - 32, Ck - 1)) * D;
            v[p] = reinterpret_cast<const float4 *>(src)[c];
        }
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            float *dst = s_x + (p * RPP + r0) * ROW + 2 * c;
            *reinterpret_cast<float2 *>(dst) = make_float2(v[p].x, v[p].z);
            *reinterpret_cast<float2 *>(dst + ODD) = make_float2(v[p].y, v[p].w);
        }
    }
    __syncthreads();
    const int jw = j0 + 32 * wave;
    if (jw >= Ck) return;
    const float4 *qa = reinterpret_cast<const float4 *>(s_x + col * ROW + half * ODD);
    const float4 *kb = reinterpret_cast<const float4 *>(s_x + (32 + 32 * wave + col) * ROW + half * ODD);
    f32x16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < D / 8; ++c) {
        const float4 a = qa[c], b = kb[c];
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b.x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b.y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, b.z, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, b.w, acc, 0, 0, 0);
    }
    if (jw + col >= Ck) return;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int i = i0 + 8 * (r >> 2) + 4 * half + (r & 3);
        if (i < Cq) scores[((size_t)h * Cq + i) * Ck + jw + col] = acc[r];
    }
}

// The lower (keep_min) or the upper one of two sort keys.
__device__ __forceinline__ unsigned long long key_pick(unsigned long long a, unsigned long long b, bool keep_min)
{
    return ((a < b) == keep_min) ? a : b;
}

// the value of lane ^ M, without the LDS crossbar where the hardware has a direct route
template <int M> __device__ __forceinline__ unsigned lane_xor(unsigned x)
{
    const int lane = threadIdx.x & 63;
    if constexpr (M == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);    // the lower half's values, the upper's
        return lane & 32 ? r[0] : r[1];
    } else if constexpr (M == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);    // the even rows' values, the odd ones'
        return lane & 16 ? r[0] : r[1];
    } else if constexpr (M == 8) {
        return (unsigned)__builtin_amdgcn_mov_dpp((int)x, 0x128, 0xF, 0xF, true);       // row_ror:8
    } else if constexpr (M == 4) {
        return (unsigned)__builtin_amdgcn_ds_swizzle((int)x, (4 << 10) | 0x1F);         // xor mask 4
    } else if constexpr (M == 2) {
        return (unsigned)__builtin_amdgcn_mov_dpp((int)x, 0x4E, 0xF, 0xF, true);        // quad_perm [2,3,0,1]
    } else {
        return (unsigned)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xF, 0xF, true);        // quad_perm [1,0,3,2]
    }
}

// Ascending bitonic sort of the first `n` (a power of two, at most 256 E) of 256 E keys, E consecutive ones per thread:
// inside a thread's registers, across the lanes of a wavefront (lane_xor), and only between wavefronts through LDS
// (two barriers each; 3 of the 45 stages at n = 512).  With every stage through LDS and scans of 18 barriers each the row
// kernel took 49 instead of 23 us at 24 heads of 100 x 500 clusters, 97 instead of 38 us at 8 heads of 100 x 2000.
template <int E>
__device__ __forceinline__ void block_sort(unsigned long long (&key)[E], int n, unsigned long long *s_key)
{
    const int tid = threadIdx.x;
    auto lanes = [&](auto m_tag, int m0, bool up) {     // stage of distance M E, if M is among the stages m0, m0 / 2, ..
        constexpr int M = decltype(m_tag)::value;
        if (m0 < M) return;
        const bool keep_min = ((tid & M) == 0) == up;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const unsigned long long other = (unsigned long long)lane_xor<M>((unsigned)(key[e] >> 32)) << 32 |
                                             lane_xor<M>((unsigned)key[e]);
            key[e] = key_pick(key[e], other, keep_min);
        }
    };
    auto inside = [&](int jj, auto up_of) {             // stage of distance jj < E
#pragma unroll
        for (int e = 0; e < E; ++e)
            if ((e & jj) == 0) {
                const unsigned long long a = key[e], b = key[e | jj];
                const bool up = up_of(e);
                key[e] = key_pick(a, b, up);
                key[e | jj] = key_pick(a, b, !up);
            }
    };
#pragma unroll
    for (int k = 2; k <= E; k <<= 1)
#pragma unroll
        for (int jj = k >> 1; jj > 0; jj >>= 1) inside(jj, [&](int e) { return ((tid * E + e) & k) == 0; });
#pragma unroll 1
    for (int k = 2 * E; k <= n; k <<= 1) {
        const bool up = ((tid * E) & k) == 0;
        const int m0 = k / (2 * E);                     // thread tid ^ m, same register, m = m0, m0 / 2, .. 1
#pragma unroll 1
        for (int m = m0; m >= 64; m >>= 1) {
            const bool keep_min = ((tid & m) == 0) == up;
            __syncthreads();
#pragma unroll
            for (int e = 0; e < E; ++e) s_key[e * SEL_THREADS + tid] = key[e];
            __syncthreads();
#pragma unroll
            for (int e = 0; e < E; ++e) key[e] = key_pick(key[e], s_key[e * SEL_THREADS + (tid ^ m)], keep_min);
        }
        lanes(std::integral_constant<int, 32>{}, m0, up);
        lanes(std::integral_constant<int, 16>{}, m0, up);
        lanes(std::integral_constant<int, 8>{}, m0, up);
        lanes(std::integral_constant<int, 4>{}, m0, up);
        lanes(std::integral_constant<int, 2>{}, m0, up);
        lanes(std::integral_constant<int, 1>{}, m0, up);
#pragma unroll
        for (int jj = E >> 1; jj > 0; jj >>= 1) inside(jj, [&](int) { return up; });
    }
}

// `lists` comes in with the scores of the row (as floats; FUSED: they are formed here) and goes out with the kept clusters.  E = next power of two of
// Ck over 256 (at least 1).
// Dynamic LDS layout: u64 key[256 E], later the sorted order as int[256 E] | float P[Ck] | int flag[Ck]
template <int E, bool FUSED>
__global__ __launch_bounds__(SEL_THREADS) void select_row_kernel(
    const float *__restrict__ cq, const float *__restrict__ ck, const int32_t *__restrict__ counts_q, const int32_t *__restrict__ counts_k, int Cq, int Ck, int d, int npow2,
    float top_p, float *__restrict__ p_est, int32_t *lists, int32_t *__restrict__ row_len,
    int32_t *__restrict__ row_keys)
{
    extern __shared__ __align__(16) unsigned char s_raw[];
    unsigned long long *s_key = reinterpret_cast<unsigned long long *>(s_raw);
    int32_t *s_ord = reinterpret_cast<int32_t *>(s_raw);
    float *s_P = reinterpret_cast<float *>(s_key + SEL_THREADS * E);
    int32_t *s_flag = reinterpret_cast<int32_t *>(s_P + Ck);
    __shared__ float s_red[SEL_THREADS / 64];
    __shared__ int32_t s_red_i[SEL_THREADS / 64];
    __shared__ float s_scan[SEL_THREADS];
    __shared__ __align__(16) float s_cq[FUSED ? 128 : 1];

    const int i = blockIdx.x, h = blockIdx.y, tid = threadIdx.x;
    const int32_t *cnt = counts_k + (size_t)h * Ck;
    const int32_t *sc = lists + ((size_t)h * Cq + i) * Ck;
    if (FUSED) {
        if (tid < d) s_cq[tid] = cq[((size_t)h * Cq + i) * d + tid];
        __syncthreads();
    }
    auto score = [&](int j) {                           // cq_i . ck_j
        if (!FUSED) return __int_as_float(sc[j]);
        const float4 *row = reinterpret_cast<const float4 *>(ck + ((size_t)h * Ck + j) * d);
        float acc = 0.f;
#pragma unroll 16
        for (int k = 0; k < d / 4; ++k) {
            const float4 v = row[k], q = reinterpret_cast<const float4 *>(s_cq)[k];
            acc = fmaf(q.x, v.x, acc);
            acc = fmaf(q.y, v.y, acc);
            acc = fmaf(q.z, v.z, acc);
            acc = fmaf(q.w, v.w, acc);
        }
        return acc;
    };

    // Eq. 1
    const float inv_sqrt_d = 1.0f / sqrtf((float)d);
    float mx = -INFINITY;
    for (int j = tid; j < Ck; j += SEL_THREADS) {
        const float s = score(j) * inv_sqrt_d;
        s_P[j] = s;
        if (cnt[j] > 0) mx = fmaxf(mx, s);
    }
    mx = block_reduce_max(mx, s_red);
    // Eq. 2
    float part = 0.f;
    for (int j = tid; j < Ck; j += SEL_THREADS) {
        const int c = cnt[j];
        const float w = (c > 0) ? (float)c * expf(s_P[j] - mx) : 0.f;
        s_P[j] = w;
        part += w;
    }
    const float den = block_reduce_sum<float>(part, s_red);
    const float inv_den = den > 0.f ? 1.0f / den : 0.f;
    for (int j = tid; j < Ck; j += SEL_THREADS) {
        const float p = s_P[j] * inv_den;
        s_P[j] = p;
        if (p_est) p_est[((size_t)h * Cq + i) * Ck + j] = p;
    }
    __syncthreads();

    const bool empty_row = counts_q && counts_q[(size_t)h * Cq + i] == 0;
    const int per = (Ck + SEL_THREADS - 1) / SEL_THREADS;
    const int j0 = min(Ck, tid * per), j1 = min(Ck, j0 + per);
    if (empty_row) {
        for (int j = tid; j < Ck; j += SEL_THREADS) s_flag[j] = 0;
    } else if (top_p >= 1.0f) {
        for (int j = tid; j < Ck; j += SEL_THREADS) s_flag[j] = cnt[j] > 0;
    } else {
        // sort keys: larger P' first, then smaller j.  P' >= 0, so its bit
        // pattern orders like the value.
        unsigned long long key[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int j = tid * E + e;
            key[e] = ~0ull;
            if (j < Ck) key[e] = ((unsigned long long)(0xFFFFFFFFu - __float_as_uint(s_P[j])) << 32) | (unsigned)j;
        }
        block_sort<E>(key, npow2, s_key);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < E; ++e) s_ord[tid * E + e] = (int)(key[e] & 0xFFFFFFFFu);
        for (int j = tid; j < Ck; j += SEL_THREADS) s_flag[j] = 0;
        __syncthreads();
        // exclusive prefix sum of P' in sorted order; thread t owns a contiguous slice
        float sum = 0.f;
        for (int t = j0; t < j1; ++t) sum += s_P[s_ord[t]];
        float run = block_exclusive_scan_f32(sum, s_scan);
        for (int t = j0; t < j1; ++t) {
            const int j = s_ord[t];
            if (run < top_p && cnt[j] > 0) s_flag[j] = 1;
            run += s_P[j];
        }
    }
    __syncthreads();

    // kept clusters in ascending j
    int nk = 0, keys = 0;
    for (int j = j0; j < j1; ++j)
        if (s_flag[j]) { nk += 1; keys += cnt[j]; }
    int total_n;
    int pos = block_exclusive_scan(nk, s_red_i, &total_n);
    int32_t *list = lists + ((size_t)h * Cq + i) * Ck;
    for (int j = j0; j < j1; ++j)
        if (s_flag[j]) list[pos++] = j;
    const int total_keys = block_reduce_sum<int32_t>(keys, s_red_i);
    if (tid == 0) {
        row_len[(size_t)h * Cq + i] = total_n;
        row_keys[(size_t)h * Cq + i] = total_keys;
    }
}

// grid (ceil(Cq / SEL_ROWS), H): a workgroup adds up the lengths of the rows in front of its own and copies its lists,
// one wavefront per row; the first one of a head also forms the density.  (One workgroup per head that copied the rows
// one after the other took 35 to 50 us whatever the number of heads; 6 us now at 24 heads of 100 x 500 clusters.)
static constexpr int SEL_ROWS = 8;

__global__ __launch_bounds__(SEL_THREADS) void select_compact_kernel(
    const int32_t *__restrict__ lists, const int32_t *__restrict__ row_len, const int32_t *__restrict__ row_keys,
    const int32_t *__restrict__ counts_q, const int32_t *__restrict__ counts_k, int Cq, int Ck,
    int32_t *__restrict__ row_ptr, int32_t *__restrict__ col_idx, float *__restrict__ density)
{
    __shared__ int32_t s_red_i[SEL_THREADS / 64];
    __shared__ double s_red[SEL_THREADS / 64];
    const int h = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int32_t *len = row_len + (size_t)h * Cq;
    const int i0 = blockIdx.x * SEL_ROWS, i1 = min(Cq, i0 + SEL_ROWS);
    int before = 0;
    for (int i = tid; i < i0; i += SEL_THREADS) before += len[i];
    before = block_reduce_sum<int32_t>(before, s_red_i);
    int32_t *rp = row_ptr + (size_t)h * (Cq + 1);
    int32_t *ci = col_idx + (size_t)h * Cq * Ck;
    for (int i = i0; i < i1; ++i) {
        const int n = len[i];
        if (tid == 0) rp[i] = before;
        if (wave == (i & (SEL_THREADS / 64 - 1))) {
            const int32_t *list = lists + ((size_t)h * Cq + i) * Ck;
            for (int e = lane; e < n; e += 64) ci[before + e] = list[e];
        }
        before += n;
    }
    if (tid == 0 && i1 == Cq) rp[Cq] = before;
    if (density && blockIdx.x == 0) {
        // work = sum_i |Q_i| * (keys selected for i): integers below 2^53, exact in double
        double w = 0.0, nq = 0.0, nk = 0.0;
        for (int i = tid; i < Cq; i += SEL_THREADS) {
            const int c = counts_q[(size_t)h * Cq + i];
            w += (double)c * (double)row_keys[(size_t)h * Cq + i];
            nq += (double)c;
        }
        for (int j = tid; j < Ck; j += SEL_THREADS) nk += (double)counts_k[(size_t)h * Ck + j];
        w = block_reduce_sum<double>(w, s_red);
        nq = block_reduce_sum<double>(nq, s_red);
        nk = block_reduce_sum<double>(nk, s_red);
        if (tid == 0) density[h] = (nq > 0.0 && nk > 0.0) ? (float)(w / (nq * nk)) : 0.f;
    }
}

static int next_pow2(int x)
{
    int p = 1;
    while (p < x) p <<= 1;
    return p;
}

size_t select_ws_bytes(int H, int Cq, int Ck)
{
    Carver c(nullptr);
    c.take<int32_t>((size_t)H * Cq * Ck);   // scores, then the per-row lists
    c.take<int32_t>((size_t)H * Cq);        // row lengths
    c.take<int32_t>((size_t)H * Cq);        // keys selected per row
    return c.used;
}

static size_t select_lds_bytes(int Ck)
{
    return (size_t)std::max(next_pow2(Ck), SEL_THREADS) * sizeof(unsigned long long) + (size_t)Ck * (sizeof(float) + sizeof(int32_t));
}

// Scores in the row kernel, a key cluster per thread (the same chain of fmaf), or from a kernel of their own?  The former
// saves a launch and a round trip through memory, but every query cluster reads the key centroids again, and a 32 x 128 tile
// of the latter is used as far as Cq and Ck fill it.  Kernel times in us, in the row kernel / in their own (D = 64):
//   1 head x 16 x 32: 11.1 / 12.9     1 x 200 x 256: 14.8 / 17.0     40 x 12 x 64 (480 rows): 13.1 / 15.4
//   24 x 100 x 100 (2400 rows): 24.9 / 22.8     40 x 50 x 128: 22.3 / 19.7     2000 x 10 x 30: 92 / 83
//   2000 x 3 x 5: 28 / 36             30,000 x 1 x 1: 146 / 250
static bool select_fused(int H, int Cq, int Ck)
{
    return (Ck <= SEL_THREADS && (long long)H * Cq <= 1024) || (Ck <= 32 && Cq <= 8);
}

typedef void (*SelectRowKernel)(const float *, const float *, const int32_t *, const int32_t *, int, int, int, int, float,
                                float *, int32_t *, int32_t *, int32_t *);
static SelectRowKernel select_row(int Ck, bool fused)
{
    if (fused) return select_row_kernel<1, true>;
    const int e = next_pow2(Ck) / SEL_THREADS;
    return e <= 1   ? select_row_kernel<1, false>
           : e == 2 ? select_row_kernel<2, false>
           : e == 4 ? select_row_kernel<4, false>
           : e == 8 ? select_row_kernel<8, false>
                    : select_row_kernel<16, false>;
}
static_assert(SVG2_MAX_CLUSTERS == 16 * SEL_THREADS, "16 keys per thread cover the largest number of clusters");

// every LDS size here is below the 64 KB that need no attribute, except these two
int select_prepare()
{
    SVG2_TRY(set_dynamic_lds(reinterpret_cast<const void *>(select_scores_kernel<128>), select_scores_lds<128>()));
    return set_dynamic_lds(reinterpret_cast<const void *>(select_row_kernel<16, false>), select_lds_bytes(SVG2_MAX_CLUSTERS));
}

int select_launch(const float *cq, const float *ck, const int32_t *counts_q, const int32_t *counts_k,
                  int H, int Cq, int Ck, int d, float top_p, int32_t *row_ptr, int32_t *col_idx,
                  float *p_est, float *density, void *ws, hipStream_t st)
{
    Carver c(ws);
    int32_t *lists = c.take<int32_t>((size_t)H * Cq * Ck);
    int32_t *row_len = c.take<int32_t>((size_t)H * Cq);
    int32_t *row_keys = c.take<int32_t>((size_t)H * Cq);
    const bool fused = select_fused(H, Cq, Ck);
    if (!fused) {
        auto scores = d == 128 ? select_scores_kernel<128> : select_scores_kernel<64>;
        hipLaunchKernelGGL(scores, dim3(cdiv(Ck, 128), cdiv(Cq, 32), H), dim3(256),
                           d == 128 ? select_scores_lds<128>() : select_scores_lds<64>(), st, cq, ck, Cq, Ck,
                           reinterpret_cast<float *>(lists));
    }
    hipLaunchKernelGGL(select_row(Ck, fused), dim3(Cq, H), dim3(SEL_THREADS), select_lds_bytes(Ck), st, cq, ck, counts_q,
                       counts_k, Cq, Ck, d, next_pow2(Ck), top_p, p_est, lists, row_len, row_keys);
    hipLaunchKernelGGL(select_compact_kernel, dim3(cdiv(Cq, SEL_ROWS), H), dim3(SEL_THREADS), 0, st, lists, row_len,
                       row_keys, counts_q, counts_k, Cq, Ck, row_ptr, col_idx, density);
    SVG2_HIP_CHECK(hipGetLastError());
    return SVG2_OK;
}

}  // namespace svg2
