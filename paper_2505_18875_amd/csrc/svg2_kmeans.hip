// Per-head Lloyd k-means (paper Section 4.1), batched over heads and over the two sides of a layer (the Q tokens
// and the K tokens are clustered independently, Section 4.1; every kernel here takes both problems in one launch).
//
// One iteration = assign, settle near-ties, update:
//   assign    token x centroid contraction with a fused argmax.
//             bf16 input: MFMA 32x32x16 bf16 with the centroid tile as the A operand (rows) and the tokens as
//             the B operand (columns), so a lane's 16 accumulators are 16 centroids of ONE token.  The
//             accumulators start at -||c||^2 / 2, so argmin ||c||^2 - 2 x.c is the argmax of the accumulator.
//             Each accumulator gets its position written into its 4 lowest mantissa bits; the largest and the
//             second largest of these keys are tracked per token (max3 / med3 chains, no compare-and-select
//             chains), which gives the label and the gap to the runner-up.
//             fp32 input: MFMA 32x32x2 fp32, or with more centroids and tokens 32x32x16 fp16 on operands in two
//             halves, near-ties by the fp32 chain; the centroids of a token dealt out to several wavefronts; a
//             handful of centroids: one token per thread.
//   settle    (bf16) every token whose gap is within the error bound of the fp32 contraction is assigned
//             again in double precision, over all centroids, lowest index winning an exact tie.  Products of
//             two bf16 numbers are exact and their sums fit a double, so these labels are THE argmin of the
//             definition, not an approximation of it; a fraction of a per cent of the tokens take this path.
//   update    segmented sum over the label-sorted token order (counting sort, shared with the permutation
//             stage), in double precision: sums of bf16 values are exact in a double, so the cluster sums do
//             not depend on the order of the additions -- reproducible bit for bit, and the delta update below
//             never drifts.  The pieces of a cluster are summed side by side, so the time does not depend on how
//             skewed the cluster sizes are.  From the second iteration on only the tokens whose label changed are
//             moved between the cluster sums.
//             Shorter heads: straight from the labels, together with the means (kmeans_update_kernel, with a few clusters of few
//             heads kmeans_update_small_kernel), where a workgroup adds all rows of its clusters; the shortest bf16 heads go
//             through all iterations in one workgroup (kmeans_tiny_bf16_kernel).
//   finalize  mean = sum / count in double (an empty cluster keeps its centroid), the fp32 centroid that is
//             handed back, the bf16 copy the next assign reads (rounded from the DOUBLE mean, so it is the
//             correctly rounded bf16 of the mean), and ||c||^2 of that copy.
//
// For bf16 input the assign step sees the centroids rounded to bf16 (both in x.c and in ||c||^2); the
// centroids handed back stay fp32 means.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "svg2_common.h"

namespace svg2 {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(16))) float f32x16;

static constexpr int KM_CMAX = 512;    // centroids resident in LDS at a time (bf16 kernel)
static constexpr int KM_NW = 8;        // wavefronts per workgroup (bf16 kernel)
static constexpr int KM_TB = 2;        // 32-token blocks per wavefront (bf16 kernel)
static constexpr int KM_WG_TOKENS = KM_NW * KM_TB * 32;
static constexpr int KM_UB = 4;        // load instructions in flight per wavefront in the segmented sum
static constexpr int KM_SEG = 256;     // rows per piece of the segmented sum
static constexpr int KM_FULL_EVERY = 16; // iterations between updates that sum every cluster afresh (the others move the changed tokens)
// Workgroups per head and side that walk the list of near-ties: about as many as run at once (5 per CU) in the launch,
// within these limits (24 heads of 16,384 tokens, 100 and 500 centroids: 11.8 us with 26 workgroups, 14.7 with 32, 15.6 with
// 64; 40 heads of 75,600: 23 us with 24, 28 with 32, 27 with 64, 29 with 16).
static constexpr int KM_SETTLE_BLOCKS = 64, KM_SETTLE_MIN = 24, KM_SETTLE_WG = 1280;
// A token is settled in double precision when the gap between its two best keys is at most
//     KM_TIE_KEY * |best key|  +  KM_TIE_ACC * (||x||^2 / 2 + max_j ||c_j||^2).
// First term: the 4 mantissa bits given to the position move a key by less than 16 units in its last place,
// 2^-19 of its value; two keys of at most the best one's magnitude (the runner-up is within the gap of it).
// Second term: the fp32 accumulation of the contraction.  sum_k |x_k c_jk| + ||c_j||^2 / 2 is below the
// bracket; 8 chained matrix instructions with a few units in the last place of the partial sums each are taken
// to stay within 2^-21 of it per accumulator, two accumulators.  (An assumption about the matrix cores'
// internal rounding, which is not documented; the parity tests compare the labels of many heads with the
// double-precision definition and would show a violation as a label that differs away from a tie.)
static constexpr float KM_TIE_KEY = 3.814697265625e-06f;      // 2^-18
static constexpr float KM_TIE_ACC = 9.5367431640625e-07f;     // 2^-20
// -||c||^2 / 2 of the padding rows of a centroid block: stays finite, and wins only where no centroid's key is a larger number
// (centroids that are NaN or beyond the range of fp32): such a token gets cluster 0 or is settled.
static constexpr float KM_PAD_HCN = -3.0e38f;

// One side of a k-means call: all heads of the Q tokens, or of the K tokens.
struct KmSide {
    const void *X;              // [H,N,d] tokens
    const float *init;          // [H,C,d]
    float *centroids;           // [H,C,d] out (may alias init)
    int32_t *labels;            // [H,N] out
    int32_t *counts;            // [H,C] out
    float *objective;           // [H,iters] or null
    int C;
    // workspace
    bf16_t *cb;                 // [H,C,d] centroids rounded to bf16 (bf16 input)
    bf16_t *cbT;                // [H,d/8,C,8] the same, 16-byte chunk-major: chunk q of consecutive centroids is contiguous
    float *ct;                  // [H,2,d/8,C,4] the fp32 centroids, even then odd elements, chunk-major (fp32 input; in
                                // the place of cb and cbT)
    float *hcn;                 // [H,C] -||c||^2 / 2 of the rounded centroids (bf16 input), ||c||^2 (fp32 input)
    double *cn64;               // [H,C] ||c||^2 of the rounded centroids
    double *cd;                 // [H,C,d] centroids in double of the clusters that are empty (what they keep)
    double *csum;               // [H,C,d] cluster sums, kept between iterations
    float *best, *second;       // [H,N] running best / runner-up between centroid chunks (C > KM_CMAX only)
    int32_t *flag_cnt;          // [H] tokens to settle
    int32_t *flag_list;         // [H,N]
    int32_t *labels_alt;        // [H,N] the labels of consecutive iterations alternate between this and `labels`
    int32_t *hist;              // sort scratch
    // two sets of the label-sorted order and its pieces: iteration t uses set t % 2, so the previous
    // iteration's order is still there for the delta update
    int32_t *offsets[2], *perm[2], *first_piece[2], *n_pieces[2];
    int4 *pieces[2];
    double *psum[2];            // [H,max_pieces,d]
    int32_t *moved[2];          // [H,max_pieces] whether the delta update found a token in the piece (else no psum)
    int max_pieces;
    // bf16, KmArgs::lists: the tokens of every group of 64 whose label changed in this iteration, or may still change as they are
    // settled (KM_MV_OPEN), in the place of the second set, which is then not used: [H,N], those of group g from 64 g on (token % 64,
    // previous label << 6, label << 18), and [H, 4 max_pieces] their number
    unsigned *mv_list;
    int32_t *mv_cnt;
};

static constexpr unsigned KM_MV_OPEN = 1u << 30;       // (labels are below 2^12)
static_assert(SVG2_MAX_CLUSTERS <= 1 << 12, "two labels and the position in a group fit an entry");

struct KmArgs {
    KmSide s[2];
    int nsides, H, N, iters;
    int nc[2];                  // wavefronts that share a token block (fp32 assign)
    int split[2];               // whether its operands may be split
    int gc[2];                  // clusters of a workgroup of the update kernel
    bool want_order;            // the caller reads offsets and perm of the last iteration
    bool lists;                 // the assign step lists the tokens whose label changed, the update step reads these lists (bf16)
};

// labels written / read by iteration t
struct KmIter {
    int32_t *lab[2];
    const int32_t *lab_prev[2];
    int t, set;
};

// element `i` (0 or 1) of a two-element array inside a kernel argument: a select, so that the struct stays in
// scalar registers (indexing it with a run-time value would move it to scratch memory)
#define KM_SEL(arr, i) ((i) ? (arr)[1] : (arr)[0])

// v_max / v_min / v_max3 / v_med3 as they are (fmaxf and friends first canonicalise operands the compiler cannot
// prove quiet).  A key that is no number loses against one that is.  Not volatile: the scheduler may place them.
__device__ __forceinline__ float km_max(float a, float b)
{
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float km_min(float a, float b)
{
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float km_max3(float a, float b, float c)
{
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ __forceinline__ float km_med3(float a, float b, float c)
{
    float r;
    asm("v_med3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// the values lanes l and l + 32 hold of x: .x = the lower half's, .y = the upper half's, the same in both lanes (one
// vector instruction; a shuffle across the halves goes through the LDS crossbar and is waited for)
struct KmHalves { unsigned lo, hi; };
__device__ __forceinline__ KmHalves km_halves(unsigned x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return {r[0], r[1]};
}

// sum of a double over the wavefront, in every lane: v += (v of lane ^ o) for o = 32, 16, 8, 4, 2, 1 -- lane swaps and data-parallel
// moves instead of shuffles through the LDS crossbar.  (Behind the steps 32 .. 8 lanes i and i ^ 8 hold the same, so a rotation by
// 4 in a row of 16 is the exchange with lane ^ 4.)
template <int CTRL> __device__ __forceinline__ double km_dpp(double v)
{
    const unsigned long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, false);
    return __longlong_as_double(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double km_join(unsigned lo, unsigned hi) { return __longlong_as_double(((unsigned long long)hi << 32) | lo); }
__device__ __forceinline__ double km_sum_xor32(double v)
{
    const unsigned long long b = __double_as_longlong(v);
    const auto l = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    return km_join(l[0], h[0]) + km_join(l[1], h[1]);
}
__device__ __forceinline__ double km_sum_xor16(double v)
{
    const unsigned long long b = __double_as_longlong(v);
    const auto l = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    return km_join(l[0], h[0]) + km_join(l[1], h[1]);
}
__device__ __forceinline__ double km_wave_sum(double v)
{
    v = km_sum_xor16(km_sum_xor32(v));
    v += km_dpp<0x128>(v);                      // row_ror:8
    v += km_dpp<0x124>(v);                      // row_ror:4
    v += km_dpp<0x4E>(v);                       // quad_perm [2,3,0,1]
    v += km_dpp<0xB1>(v);                       // quad_perm [1,0,3,2]
    return v;
}

// double -> bf16, round to nearest even, in ONE rounding: via float unless the float lands exactly on the midpoint
// of two bf16 values, where the side the double was on decides (and an exact midpoint goes to even).
__device__ __forceinline__ bf16_t f64_to_bf16(double m)
{
    const float f = (float)m;
    const unsigned u = __float_as_uint(f);
    if ((u & 0xFFFFu) != 0x8000u) return (bf16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
    const double fd = (double)f, am = fabs(m), af = fabs(fd);
    const bool up = am > af || (am == af && ((u >> 16) & 1u));
    return (bf16_t)((u >> 16) + (up ? 1u : 0u));
}

// ---------------------------------------------------------------- finalize
// grid (ceil(clusters of both sides / KM_FIN_NW), H), block 64 * KM_FIN_NW: one wavefront per cluster, lane l holds
// elements l (and l + 64).  mode 0: what the first assign step reads, from the caller's centroids.  mode 1: cluster sum
// = sum of the cluster's pieces of set `it.set`.  mode 2 (delta update): cluster sum = previous cluster sum + the pieces
// of the tokens that joined the cluster (set `it.set`) - the pieces of the tokens that left it (the other set), as far
// as a piece has any (`moved`).  All sums are doubles of bf16 / fp32 values, in the order of the pieces.
//
// What bounds it is the bytes it touches (a cluster's double sums in and out, its pieces), so it touches what the next
// step reads and no more: the fp32 centroids go out in the last iteration, and the mean in double is kept only of a
// cluster that has just run empty (it is the previous sum over the previous count).  One workgroup of D threads per
// cluster, all of these written in every iteration and every piece read whether anything moved in it or not, took 24
// instead of 14 us per iteration at 24 heads of 16,384 tokens (100 and 500 clusters, d = 128) and 45 instead of 31 us at
// 40 heads of 75,600.  Only loads that are needed are issued: eight pieces always requested together (the missing ones as
// duplicates of the first) took 25 and 53 us.
static constexpr int KM_FIN_NW = 4;
static constexpr int KM_FIN_UB = 8;             // pieces requested together

// One cluster by one wavefront: s = its new sum (element lane + 64 e), cnt its tokens; s_prev, prev: sum and tokens before, read
// only of a cluster without tokens.
template <bool BF16, int D>
__device__ __forceinline__ void finalize_cluster(const KmArgs &a, const KmSide &S, const KmIter &it, int mode, int h, int j,
                                                 const double (&s)[D / 64], int cnt, const double (&s_prev)[D / 64], int prev)
{
    constexpr int EL = D / 64;
    const int lane = threadIdx.x & 63, C = S.C;
    const size_t idx = ((size_t)h * C + j) * D + lane;
    double c[EL];
    if (mode != 0) {
        if (cnt > 0) {
#pragma unroll
            for (int e = 0; e < EL; ++e) c[e] = s[e] / (double)cnt;
        } else {                                        // an empty cluster keeps its centroid
#pragma unroll
            for (int e = 0; e < EL; ++e) {
                c[e] = it.t == 0 ? (double)S.init[idx + 64 * e]
                       : prev > 0 ? s_prev[e] / (double)prev
                                  : S.cd[idx + 64 * e];
                S.cd[idx + 64 * e] = c[e];
            }
        }
#pragma unroll
        for (int e = 0; e < EL; ++e) {
            S.csum[idx + 64 * e] = cnt > 0 ? s[e] : 0.0;
            if (it.t + 1 == a.iters) S.centroids[idx + 64 * e] = (float)c[e];
        }
        if (lane == 0) S.counts[(size_t)h * C + j] = cnt;
    } else {
#pragma unroll
        for (int e = 0; e < EL; ++e) c[e] = (double)S.init[idx + 64 * e];
    }
    double n2 = 0.0;
#pragma unroll
    for (int e = 0; e < EL; ++e) {
        const int k = lane + 64 * e;
        double cr = (double)(float)c[e];
        if (BF16) {
            const bf16_t b = f64_to_bf16(c[e]);
            S.cb[idx + 64 * e] = b;
            S.cbT[(((size_t)h * (D / 8) + (k >> 3)) * C + j) * 8 + (k & 7)] = b;
            cr = (double)bf16_to_f32(b);
        } else {
            S.ct[((((size_t)h * 2 + (k & 1)) * (D / 8) + (k >> 3)) * C + j) * 4 + ((k >> 1) & 3)] = (float)c[e];
        }
        const double sq = km_wave_sum(cr * cr);
        n2 = e == 0 ? sq : n2 + sq;
    }
    if (lane == 0) {
        S.cn64[(size_t)h * C + j] = n2;
        S.hcn[(size_t)h * C + j] = BF16 ? (float)(-0.5 * n2) : (float)n2;
    }
}

template <bool BF16, int D>
__global__ __launch_bounds__(64 * KM_FIN_NW) void kmeans_finalize_kernel(KmArgs a, KmIter it, int mode)
{
    constexpr int EL = D / 64;
    const int lane = threadIdx.x & 63, h = blockIdx.y, set = it.set;
    const int jj = blockIdx.x * KM_FIN_NW + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int side = jj >= a.s[0].C ? 1 : 0;
    const KmSide S = side ? a.s[1] : a.s[0];
    const int C = S.C, j = side ? jj - a.s[0].C : jj;
    if (side >= a.nsides || j >= C) return;
    if (j == 0 && lane == 0) S.flag_cnt[h] = 0;         // the next assign step starts an empty list
    int cnt = 0, prev = 0;
    double s[EL], s_prev[EL];
#pragma unroll
    for (int e = 0; e < EL; ++e) s[e] = s_prev[e] = 0.0;
    if (mode != 0) {
        const int32_t *off = KM_SEL(S.offsets, set) + (size_t)h * (C + 1);
        cnt = off[j + 1] - off[j];
        if (mode == 2 || (cnt == 0 && it.t > 0)) {
            prev = cnt == 0 ? S.counts[(size_t)h * C + j] : 0;
#pragma unroll
            for (int e = 0; e < EL; ++e) s_prev[e] = S.csum[((size_t)h * C + j) * D + lane + 64 * e];
        }
        if (mode == 2) {
#pragma unroll
            for (int e = 0; e < EL; ++e) s[e] = s_prev[e];
        }
        auto add_pieces = [&](int st, double sign) {
            const int32_t *fp = KM_SEL(S.first_piece, st) + (size_t)h * (C + 1);
            const int p0 = fp[j], np = fp[j + 1] - p0;
            const double *ps = KM_SEL(S.psum, st) + ((size_t)h * S.max_pieces + p0) * D + lane;
            const int32_t *mv = KM_SEL(S.moved, st) + (size_t)h * S.max_pieces + p0;
            // KM_FIN_UB pieces in flight together: the largest cluster of a head has dozens and its wavefront decides
            // how long the launch takes
            for (int p = 0; p < np; p += 64) {
                unsigned long long m = __ballot(p + lane < np && (mode == 1 || mv[min(p + lane, np - 1)] != 0));
                while (m) {
                    double v[KM_FIN_UB][EL];
                    int n = 0;
#pragma unroll
                    for (int u = 0; u < KM_FIN_UB; ++u)
                        if (m) {
                            const int q = p + (int)__builtin_ctzll(m);
                            m &= m - 1;
                            n = u + 1;
#pragma unroll
                            for (int e = 0; e < EL; ++e) v[u][e] = ps[(size_t)q * D + 64 * e];
                        }
#pragma unroll
                    for (int u = 0; u < KM_FIN_UB; ++u)
                        if (u < n) {
#pragma unroll
                            for (int e = 0; e < EL; ++e) s[e] += sign * v[u][e];
                        }
                }
            }
        };
        add_pieces(set, 1.0);
        if (mode == 2) add_pieces(1 - set, -1.0);
    }
    finalize_cluster<BF16, D>(a, S, it, mode, h, j, s, cnt, s_prev, prev);
}

// ---------------------------------------------------------------- assign, bf16 MFMA
// grid (one workgroup per CU), block 64 * KM_NW.  The blocks of KM_WG_TOKENS tokens of all heads of a side form one
// sequence; workgroup w takes the w-th of gridDim.x equal parts of it, on both sides: even workgroups first on the
// second side (the K tokens of a layer: many centroids, bound by the matrix cores) and then on the first (the Q
// tokens: few centroids, waiting for memory), odd workgroups the other way round, so that the two kinds of work
// share the chip at any time.  A part is cut at head boundaries into spans; the head's centroids (up to KM_CMAX
// at a time) are staged in LDS once per span and stay there for all its blocks.  (One workgroup per 4096 tokens of
// one side, placed by the hardware, took 0.59 instead of 0.50 ms per launch on a layer of 40 heads of 75,600 tokens
// with 100 and 500 centroids: the sum of the times the two sides take alone.)  With more than KM_CMAX centroids the running best and runner-up of a token go through `best` / `second`
// between chunks.
//
// A wavefront takes 64 tokens at a time, as two blocks of 32.  Per 32-centroid row block it issues the 2 KS matrix
// instructions of both, then reduces their accumulators to (best, runner-up) with max3 / med3 chains while the other wavefront of
// the SIMD has the matrix cores.
//
// Near-ties (see KM_TIE_*) are listed for kmeans_settle_kernel.
template <int D, bool OBJ>
__global__ __launch_bounds__(64 * KM_NW, 1) void kmeans_assign_bf16_kernel(KmArgs a, KmIter it)
{
    constexpr int KS = D / 16;              // MFMA k-steps
    constexpr int ROW = D + 8;              // LDS row stride in elements (16 bytes of padding)
    extern __shared__ __align__(16) unsigned char s_raw[];
    // -||c||^2 / 2 first: its reads then have offsets below 64 KB, which fit the instruction, and cost no address
    // arithmetic in the step loop
    float *s_hcn = reinterpret_cast<float *>(s_raw);                               // [KM_CMAX]: -||c||^2 / 2
    bf16_t *s_c = reinterpret_cast<bf16_t *>(s_raw + KM_CMAX * sizeof(float));     // [KM_CMAX][ROW]
    __shared__ int s_next;                  // next group of a span that no wavefront has taken yet

    const int N = a.N;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int half = lane >> 5, col = lane & 31;
    const int nbh = (N + KM_WG_TOKENS - 1) / KM_WG_TOKENS;          // token blocks of a head
    const int nb_all = a.H * nbh;                                   // H N d < 2^40: below 2^25
    static_assert(64 * KM_NW == KM_CMAX, "one -||c||^2/2 per thread");

#define KM_FENCE __builtin_amdgcn_sched_barrier(0);
    // this workgroup's part of the block sequence, the same for both sides
    const int part_q = nb_all / (int)gridDim.x, part_r = nb_all % (int)gridDim.x;
    int part_lo = (int)blockIdx.x * part_q + min((int)blockIdx.x, part_r);
    int part_hi = part_lo + part_q + ((int)blockIdx.x < part_r ? 1 : 0);
    // at most as many blocks as CUs over both sides: one block of one side per workgroup (2 heads of 1024 tokens, D = 64:
    // 13.4 us with both sides of a block one after the other in one workgroup and all 512 rows staged, 8.3 us now)
    const bool one_block = (int)gridDim.x == a.nsides * nb_all;
    if (one_block) {
        part_lo = (int)blockIdx.x % nb_all;
        part_hi = part_lo + 1;
    }
#pragma unroll 1
    for (int sd = one_block ? (int)blockIdx.x / nb_all : 0; sd < a.nsides; sd = one_block ? a.nsides : sd + 1) {
    // odd workgroups start with the first side, even ones with the second: while one half of the CUs is on the Q
    // tokens of a layer (few centroids, waits for memory) the other is on the K tokens (many, matrix cores)
    const int side = one_block || (blockIdx.x & 1) ? sd : a.nsides - 1 - sd;
    const KmSide S = side ? a.s[1] : a.s[0];
    int32_t *labels = side ? it.lab[1] : it.lab[0];
    const int32_t *labels_prev = side ? it.lab_prev[1] : it.lab_prev[0];
    const int C = S.C;
    const int nchunk = (C + KM_CMAX - 1) / KM_CMAX;
#pragma unroll 1
    for (int sp = part_lo; sp < part_hi;) {
    // span: blocks blk0 .. blk0 + nblk of head h
    const int h = sp / nbh, blk0 = sp - h * nbh;
    const int nblk = min(nbh - blk0, part_hi - sp);
    sp += nblk;
    const bf16_t *Xh = reinterpret_cast<const bf16_t *>(S.X) + (size_t)h * N * D;
    const bf16_t *cbh = S.cb + (size_t)h * C * D;
    const float *hcnh = S.hcn + (size_t)h * C;
    float obj = 0.f;
    float cmax2 = 0.f;          // largest ||c||^2 of the head (over the chunks so far), for the near-tie bound
    for (int chunk = 0; chunk < nchunk; ++chunk) {
        const int c0 = chunk * KM_CMAX;
        const int cc = min(KM_CMAX, C - c0), ccp = (cc + 31) & ~31;
        const bool last_chunk = chunk + 1 == nchunk;
        __syncthreads();
        // The span is handed out in groups of KM_TB * 32 tokens: wavefront w starts with group w and then takes
        // the next one nobody has taken (the two wavefronts of a SIMD do not run at the same speed, see the
        // priorities below; with a fixed share the fast ones would wait for the slow ones at the end of the span).
        if (tid == 0) s_next = KM_NW;               // read after the barrier behind the staging
        // Two register buffers.  Tokens as the B operand: lane (col, half) holds elements 16 s + 8 half .. + 8 of
        // token `col`.  The KM_TB * KS loads of a group come in four parts; while a group is computed, the parts of
        // the wavefront's next one are requested one by one between its steps (all eight wavefronts of the
        // workgroup asking for a whole group at the same moment queue up in front of the texture unit, and each
        // of them waits for the queue).
        bf16x8 xb[2][KM_TB][KS];
        constexpr int NLD = KM_TB * KS, LPP = NLD / 4;
        auto load_part = [&](auto buf_tag, int g, auto part_tag) {
            constexpr int BUF = decltype(buf_tag)::value, PART = decltype(part_tag)::value;
            const int tok0 = blk0 * KM_WG_TOKENS + g * (KM_TB * 32);
#pragma unroll
            for (int i = PART * LPP; i < (PART + 1) * LPP; ++i) {
                const int tb = i / KS, s = i % KS;
                const int n = min(N - 1, tok0 + tb * 32 + col);
                const uint4 v = reinterpret_cast<const uint4 *>(Xh + (size_t)n * D + 8 * half)[2 * s];
                __builtin_memcpy(&xb[BUF][tb][s], &v, 16);
            }
        };
        auto load_x = [&](auto buf_tag, int g) {
            load_part(buf_tag, g, std::integral_constant<int, 0>{});
            load_part(buf_tag, g, std::integral_constant<int, 1>{});
            load_part(buf_tag, g, std::integral_constant<int, 2>{});
            load_part(buf_tag, g, std::integral_constant<int, 3>{});
        };
        // stage the chunk (rows past the last centroid are zero and can never win).  A thread requests all its
        // pieces before it stores the first, so the block waits for one round trip to memory, not sixteen;
        // no branches (a row past the end re-reads the last one and is zeroed in registers), and every workgroup
        // starts at another row, so that the workgroups of a head that run side by side do not ask the same L2
        // channel for the same line at the same moment.
        {
            constexpr int PER = KM_CMAX * (D / 8) / (64 * KM_NW);
            // the addresses are formed here, in every chunk: formed once in front of the chunk loop (where the
            // compiler would move them) they would sit in scratch memory while the token blocks are computed
            int tid_o = tid;
            asm volatile("" : "+v"(tid_o));
            auto stage = [&](auto nv_tag) {
                constexpr int NV = decltype(nv_tag)::value, ROWS = NV * 64 * KM_NW / (D / 8);
                static_assert((ROWS & (ROWS - 1)) == 0, "row rotation wraps with a mask");
                const int rot = (int)(blockIdx.x * 37u);
                uint4 v[NV];
#pragma unroll
                for (int i = 0; i < NV; ++i) {
                    const int e = tid_o + i * 64 * KM_NW, r = ((e / (D / 8)) + rot) & (ROWS - 1);
                    v[i] = reinterpret_cast<const uint4 *>(cbh + (size_t)(c0 + min(r, cc - 1)) * D)[e % (D / 8)];
                }
                // in the same round trip: this thread's -||c||^2/2 and the wavefront's first block of tokens
                const float hv = hcnh[c0 + min(tid_o, cc - 1)];
                load_x(std::integral_constant<int, 0>{}, wave);
#pragma unroll
                for (int i = 0; i < NV; ++i) {
                    const int e = tid_o + i * 64 * KM_NW, r = ((e / (D / 8)) + rot) & (ROWS - 1);
                    if (r >= cc) v[i] = make_uint4(0, 0, 0, 0);
                    *reinterpret_cast<uint4 *>(&s_c[r * ROW + (e % (D / 8)) * 8]) = v[i];
                }
                s_hcn[tid] = tid < cc ? hv : KM_PAD_HCN;
            };
            // few centroids: a quarter of the rows is all there is to stage (at D = 128 a second form costs registers
            // that the step loop does not have)
            if (D == 64 && ccp <= KM_CMAX / 4) stage(std::integral_constant<int, PER / 4>{});
            else stage(std::integral_constant<int, PER>{});
        }
        __syncthreads();
        {
            float m = cmax2;
#pragma unroll
            for (int k = 0; k < KM_CMAX / 64; ++k) {
                const int t = lane + 64 * k;
                m = fmaxf(m, t < cc ? -2.f * s_hcn[t] : 0.f);
            }
            for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
            cmax2 = m;
        }

        // What a block of tokens writes (label; running pair or the near-tie list) is held back until the tokens of
        // the next block have been waited for: that wait is for ALL outstanding memory operations, and behind the
        // stores it would last a round trip to memory although the tokens arrived long ago.
        // The halves of a wavefront hold the same results; lane l writes those of token l of the group.
        static_assert(KM_TB == 2, "a lane writes one token");
        int pend_tok0 = 0, pend_c[KM_TB], pend_prev = 0;
        float pend_T[KM_TB], pend_U[KM_TB];
        bool pend_f[KM_TB], pend = false;
        auto flush = [&]() {
            if (!pend) return;
            pend = false;
            const int n = pend_tok0 + lane, c = half ? pend_c[1] : pend_c[0];
            const bool flagged = half ? pend_f[1] : pend_f[0];
            if (n < N) {
                labels[(size_t)h * N + n] = c;
                if (!last_chunk) {
                    S.best[(size_t)h * N + n] = half ? pend_T[1] : pend_T[0];
                    S.second[(size_t)h * N + n] = half ? pend_U[1] : pend_U[0];
                } else if (flagged) {
                    const int pos = atomicAdd(&S.flag_cnt[h], 1);
                    S.flag_list[(size_t)h * N + pos] = n;
                }
            }
            if (a.lists && last_chunk && pend_tok0 < N) {
                int sd_o = side;                                // (read here from the arguments, not held in registers)
                asm volatile("" : "+s"(sd_o));
                unsigned *mv_list = sd_o ? a.s[1].mv_list : a.s[0].mv_list;
                int32_t *mv_cnt = sd_o ? a.s[1].mv_cnt : a.s[0].mv_cnt;
                const int mvs = 4 * (sd_o ? a.s[1].max_pieces : a.s[0].max_pieces);
                const bool moved = n < N && (flagged || c != pend_prev);
                const unsigned long long m = __ballot(moved);
                if (moved)
                    mv_list[(size_t)h * N + pend_tok0 + __popcll(m & ((1ull << lane) - 1ull))] =
                        (unsigned)lane | (unsigned)pend_prev << 6 | (unsigned)c << 18 | (flagged ? KM_MV_OPEN : 0u);
                if (lane == 0) mv_cnt[(size_t)h * mvs + pend_tok0 / 64] = __popcll(m);
            }
        };
        // Accumulator i of a lane is centroid 8 (i/4) + 4 half + i%4 of the row block; its key is the accumulator
        // with i in its 4 lowest mantissa bits, compared as a float.  best = largest key seen, second = runner-up,
        // bbase = first centroid of the row block the best came from (the same number in every lane: the select
        // then takes it from a scalar register).
        auto compute = [&](auto buf_tag, int g) -> int {
            constexpr int BUF = decltype(buf_tag)::value;
            // the group after this one (taken here, so that the answer is there when the first step wants it)
            int g_next = 0;
            if (lane == 0) g_next = atomicAdd(&s_next, 1);
            g_next = __builtin_amdgcn_readfirstlane(g_next);
            const int tok0 = blk0 * KM_WG_TOKENS + g * (KM_TB * 32);
            float best[KM_TB], second[KM_TB];
            int bbase[KM_TB];
#pragma unroll
            for (int tb = 0; tb < KM_TB; ++tb) {
                best[tb] = -INFINITY;
                second[tb] = -INFINITY;
                bbase[tb] = 0;
            }
            // The two wavefronts of a SIMD (w and w + 4) get different priorities: with equal ones they fall into
            // step, both in their matrix instructions and then both in their reductions, and each unit idles
            // while the other works.
            if (wave & 4) __builtin_amdgcn_s_setprio(2); else __builtin_amdgcn_s_setprio(0);
            const int nrb = ccp / 32;
            // steps after which the four parts of the next block are requested: spread over the first half of a
            // long block (the loads then have the second half to land in), all at once when the block is short
            const int pstep = nrb >= 8 ? nrb / 8 : 0;
            // everything this wavefront has requested so far -- the tokens of this block -- has to be there; said
            // here, in front of the loop, the compiler places no wait inside it
            __builtin_amdgcn_s_waitcnt(0x0F70);
            flush();
            bf16x8 am[KS];
            f32x16 cinit;
            auto fetch_c = [&](int rb) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float4 v = *reinterpret_cast<const float4 *>(&s_hcn[rb * 32 + 8 * g + 4 * half]);
                    cinit[4 * g] = v.x; cinit[4 * g + 1] = v.y; cinit[4 * g + 2] = v.z; cinit[4 * g + 3] = v.w;
                }
            };
            auto fetch_a = [&](int rb, int s) {
                const uint4 v = *reinterpret_cast<const uint4 *>(&s_c[(rb * 32 + col) * ROW + 8 * half + 16 * s]);
                __builtin_memcpy(&am[s], &v, 16);
            };
            // (largest, runner-up) of A's keys and the running pair.  Two keys at a time against the largest so far: max3 is
            // the new largest, med3 what of the three may be the runner-up, and the medians meet the runner-up two by two:
            // 2.5 instructions per pair of keys.  (Groups of four, each reduced to a pair of its own and the pairs merged, took 3.75:
            // 487 instead of 480 us per launch at 40 heads of 75,600 tokens, 100 and 500 centroids.)
            auto reduce = [&](const f32x16 &A, float &bst, float &snd, int &bse, int rbase) {
                float key[16], med[8], top = bst;
#pragma unroll
                for (int i = 0; i < 16; ++i) key[i] = __uint_as_float((__float_as_uint(A[i]) & 0xFFFFFFF0u) | (unsigned)i);
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    med[i] = km_med3(top, key[2 * i], key[2 * i + 1]);
                    top = km_max3(top, key[2 * i], key[2 * i + 1]);
                    if (i & 1) snd = km_max3(snd, med[i - 1], med[i]);
                }
                bse = top > bst ? rbase : bse;
                bst = top;
            };
            // One step = one 32-centroid row block against both token blocks: 2 KS matrix instructions back to back,
            // the LDS reads of the next row block's operands, then the two top-2 reductions on the vector ALU
            // while the other wavefront of the SIMD has the matrix cores.  (Interleaving the reduction of one token
            // block with the matrix instructions of the other, chunk by chunk, was measured slower: 0.49 against
            // 0.42 ms for the K side of the Wan-like layer.)
            fetch_c(0);
#pragma unroll
            for (int s = 0; s < KS; ++s) fetch_a(0, s);
#pragma unroll 1
            for (int rb = 0; rb < nrb; ++rb) {
                f32x16 acc[KM_TB];
#pragma unroll
                for (int s = 0; s < KS; ++s)
#pragma unroll
                    for (int q = 0; q < KM_TB; ++q)
                        acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(am[s], xb[BUF][q][s], s == 0 ? cinit : acc[q], 0, 0, 0);
                KM_FENCE
                if (rb + 1 < nrb) {
                    fetch_c(rb + 1);
#pragma unroll
                    for (int s = 0; s < KS; ++s) fetch_a(rb + 1, s);
                }
                {
                    using NB = std::integral_constant<int, BUF ^ 1>;
                    if (rb == 0) load_part(NB{}, g_next, std::integral_constant<int, 0>{});
                    if (rb == pstep) load_part(NB{}, g_next, std::integral_constant<int, 1>{});
                    if (rb == 2 * pstep) load_part(NB{}, g_next, std::integral_constant<int, 2>{});
                    if (rb == 3 * pstep) {
                        load_part(NB{}, g_next, std::integral_constant<int, 3>{});
                        pend_prev = labels_prev[(size_t)h * N + min(N - 1, tok0 + lane)];
                    }
                }
                KM_FENCE
                const int rbase = c0 + rb * 32;
#pragma unroll
                for (int q = 0; q < KM_TB; ++q) reduce(acc[q], best[q], second[q], bbase[q], rbase);
                KM_FENCE
            }
            KM_FENCE
#pragma unroll
            for (int tb = 0; tb < KM_TB; ++tb) {
                const unsigned kb = __float_as_uint(best[tb]);
                const int cown = bbase[tb] + 4 * half + (int)(((kb & 12u) << 1) | (kb & 3u));
                // the two lane halves of a token hold disjoint centroids
                const KmHalves hb = km_halves(kb), hs = km_halves(__float_as_uint(second[tb])),
                               hi = km_halves((unsigned)cown);
                const float b0 = __uint_as_float(hb.lo), b1 = __uint_as_float(hb.hi);
                float T = km_max(b0, b1), U = km_max3(km_min(b0, b1), __uint_as_float(hs.lo), __uint_as_float(hs.hi));
                int cidx = (b1 > b0) ? (int)hi.hi : (int)hi.lo;
                const int n = tok0 + tb * 32 + col;
                if (chunk > 0) {
                    // best and runner-up over the earlier chunks (read here, behind the loop: a load in front of
                    // it would make every step of the loop wait for all outstanding loads, the prefetch included)
                    const int nn = min(N - 1, n);
                    const float cb = S.best[(size_t)h * N + nn], cs = S.second[(size_t)h * N + nn];
                    const int cl = labels[(size_t)h * N + nn];
                    U = km_max3(km_min(T, cb), U, cs);
                    if (!(T > cb)) cidx = cl;
                    T = km_max(T, cb);
                }
                bool flagged = false;
                float x2 = 0.f;
                if (last_chunk) {
                    // ||x||^2, two elements per instruction (this lane's half of the token, then both halves)
#pragma unroll
                    for (int s = 0; s < KS; ++s)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const bf16x2_t p2 = {xb[BUF][tb][s][2 * e], xb[BUF][tb][s][2 * e + 1]};
                            x2 = __builtin_amdgcn_fdot2_f32_bf16(p2, p2, x2, false);
                        }
                    {
                        const KmHalves hx = km_halves(__float_as_uint(x2));
                        x2 = __uint_as_float(hx.lo) + __uint_as_float(hx.hi);
                    }
                    // runner-up within the error of this contraction: the token is settled in double precision
                    // (a tie, including an exact one, always is)
                    const float tau = KM_TIE_KEY * fabsf(T) + KM_TIE_ACC * (0.5f * x2 + cmax2);
                    flagged = !(T - U > tau);
                    if (OBJ && S.objective && half == 0 && n < N) obj += x2 - 2.f * T;
                }
                pend_c[tb] = cidx < C ? cidx : 0; pend_T[tb] = T; pend_U[tb] = U; pend_f[tb] = flagged;
            }
            pend_tok0 = tok0;
            pend = true;
            return g_next;
        };
        // The tokens of the group after the one being computed are ALWAYS requested (past the end of the span the
        // addresses are clamped and the values unused): with a conditional prefetch the compiler has to place waits
        // that are also right for the path without it.
        const int ng = nblk * KM_NW;
#pragma unroll 1
        for (int g = wave; g < ng;) {
            g = compute(std::integral_constant<int, 0>{}, g);
            if (g < ng) g = compute(std::integral_constant<int, 1>{}, g);
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);     // the last, unused request: the registers are reused from here on
        flush();
    }
    if (OBJ && S.objective) {
        for (int o = 32; o > 0; o >>= 1) obj += __shfl_xor(obj, o);
        if (lane == 0) atomicAdd(S.objective + (size_t)h * a.iters + it.t, obj);
    }
    }   // spans
    }   // sides
#undef KM_FENCE
}

// ---------------------------------------------------------------- settle near-ties, bf16 input
// grid (workgroups per head and side, H * sides), block 256: one workgroup per listed token at a time.  The argmin of the
// distance ||c_j||^2 - 2 x.c_j over EVERY centroid in double precision, lowest index on an exact tie.  x and c are bf16
// numbers: every product is exact, and so are the sums of 128 of them while the products span no more than some 30 binary
// orders; beyond that the sums round, which is why every distance is formed by the same chain of additions.
//
// What the launch takes is the time of ONE token (a head lists a few dozen), so the token is first compared with all
// centroids in fp32 (wavefront w takes the centroid groups 64 (w + 4 i) .. + 64, lane l of it centroid l of the group,
// read from the chunk-major copy so that the 64 lanes of a load read 1 KB of consecutive memory; two products per
// instruction), and only the centroids within the error of that are measured in double, one per lane, the token's elements read
// from LDS ahead of the chain (as they were needed: 15.4 instead of 14.7 us at 24 heads of 16,384 tokens, 32 workgroups). With every
// centroid measured in double, a few thousand instructions per group, the launch took 20 instead of 12 us there, 27 instead
// of 13 us on average over 8 heads of 37,800 in 100 and in 2000, and 28 instead of 23 us at 40 heads of 75,600.
//
// Error of the fp32 value x.c - ||c||^2 / 2: D / 2 steps with at most two roundings each of partial sums below ||x||^2 / 2 +
// ||c||^2, below 2^-17 of that at D = 128; two values are compared, and the margin is twice what that makes.
static constexpr float KM_SETTLE_MARGIN = 3.0517578125e-05f;  // 2^-15

template <int D>
__global__ __launch_bounds__(256, 5) void kmeans_settle_kernel(KmArgs a, KmIter it)
{
    __shared__ __align__(16) double s_x[D];
    __shared__ __align__(16) bf16_t s_xb[D];
    __shared__ float s_v[SVG2_MAX_CLUSTERS];
    __shared__ float s_top[4], s_cmax[4];
    __shared__ double s_best[4];
    __shared__ int s_bj[4];
    const int side = blockIdx.y % a.nsides, h = blockIdx.y / a.nsides;
    const KmSide S = side ? a.s[1] : a.s[0];
    int32_t *labels = side ? it.lab[1] : it.lab[0];
    const int N = a.N, C = S.C;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int cnt = min(S.flag_cnt[h], N);
    const bf16_t *Xh = reinterpret_cast<const bf16_t *>(S.X) + (size_t)h * N * D;
    const uint4 *ct = reinterpret_cast<const uint4 *>(S.cbT) + (size_t)h * (D / 8) * C;
    const bf16_t *cbh = S.cb + (size_t)h * C * D;
    const double *cn = S.cn64 + (size_t)h * C;
    for (int t = blockIdx.x; t < cnt; t += gridDim.x) {
        const int n = S.flag_list[(size_t)h * N + t];
        __syncthreads();                            // the previous token's LDS is no longer read
        if (tid < D) {
            const bf16_t xb = Xh[(size_t)n * D + tid];
            s_xb[tid] = xb;
            s_x[tid] = (double)bf16_to_f32(xb);
        }
        __syncthreads();
        float x2 = 0.f;
#pragma unroll
        for (int e = 0; e < D / 64; ++e) {
            const float x = bf16_to_f32(s_xb[lane + 64 * e]);
            x2 = fmaf(x, x, x2);
        }
        float top = -INFINITY, cmax = 0.f;
        for (int j0 = 64 * wave; j0 < C; j0 += 256) {
            const int j = min(j0 + lane, C - 1);
            const float c2 = (float)cn[j];
            float dot = 0.f;
#pragma unroll 1
            for (int q0 = 0; q0 < D / 8; q0 += 8) {     // eight pieces at a time: fewer registers, more workgroups per CU
                uint4 w4[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) w4[q] = ct[(size_t)(q0 + q) * C + j];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const uint4 xq = reinterpret_cast<const uint4 *>(s_xb)[q0 + q];
                    const unsigned w[4] = {w4[q].x, w4[q].y, w4[q].z, w4[q].w}, u[4] = {xq.x, xq.y, xq.z, xq.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        bf16x2_t p, r;
                        __builtin_memcpy(&p, &w[e], 4);
                        __builtin_memcpy(&r, &u[e], 4);
                        dot = __builtin_amdgcn_fdot2_f32_bf16(p, r, dot, false);
                    }
                }
            }
            const float v = fmaf(-0.5f, c2, dot);   // the larger, the closer
            s_v[j0 + lane < C ? j0 + lane : C - 1] = v;     // (the lanes past the end hold the last centroid as well)
            top = fmaxf(top, v);
            cmax = fmaxf(cmax, c2);
        }
        for (int o = 32; o > 0; o >>= 1) {
            top = fmaxf(top, __shfl_xor(top, o));
            cmax = fmaxf(cmax, __shfl_xor(cmax, o));
            x2 += __shfl_xor(x2, o);
        }
        if (lane == 0) { s_top[wave] = top; s_cmax[wave] = cmax; }
        __syncthreads();
        top = fmaxf(fmaxf(s_top[0], s_top[1]), fmaxf(s_top[2], s_top[3]));
        cmax = fmaxf(fmaxf(s_cmax[0], s_cmax[1]), fmaxf(s_cmax[2], s_cmax[3]));
        const float least = top - KM_SETTLE_MARGIN * (0.5f * x2 + cmax);

        double best = INFINITY;
        int bj = 0x7FFFFFFF;
        for (int j0 = 64 * wave; j0 < C; j0 += 256) {
            // (what is no number is measured too)
            const int j = j0 + lane;
            if (j >= C || s_v[j] < least) continue;
            // one chain of additions per centroid, k = 0 .. D - 1, so that equal centroids tie whatever the sum rounds;
            // the token comes from LDS eight elements ahead of their use
            const uint4 *row = reinterpret_cast<const uint4 *>(cbh + (size_t)j * D);
            double dot = 0.0;
#pragma unroll 1
            for (int q0 = 0; q0 < D / 8; q0 += 8) {
                asm volatile("" ::: "memory");      // (read here, not held in 2 D registers across the groups)
                uint4 w4[8];
                double2 x2d[2][4];
#pragma unroll
                for (int q = 0; q < 8; ++q) w4[q] = row[q0 + q];
                auto load_x = [&](int q) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) x2d[q & 1][e] = reinterpret_cast<const double2 *>(s_x)[4 * (q0 + q) + e];
                };
                load_x(0);
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    if (q < 7) load_x(q + 1);
                    __builtin_amdgcn_sched_barrier(0);
                    const unsigned w[4] = {w4[q].x, w4[q].y, w4[q].z, w4[q].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        dot = fma(x2d[q & 1][e].x, (double)__uint_as_float(w[e] << 16), dot);
                        dot = fma(x2d[q & 1][e].y, (double)__uint_as_float(w[e] & 0xFFFF0000u), dot);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            const double dist = cn[j] - 2.0 * dot;
            // ascending j: strict < keeps the lower index
            if (dist < best) { best = dist; bj = j; }
        }
        for (int o = 32; o > 0; o >>= 1) {
            const double ob = __shfl_xor(best, o);
            const int oj = __shfl_xor(bj, o);
            if (ob < best || (ob == best && oj < bj)) { best = ob; bj = oj; }
        }
        if (lane == 0) { s_best[wave] = best; s_bj[wave] = bj; }
        __syncthreads();
        if (tid == 0) {
#pragma unroll
            for (int w = 1; w < 4; ++w)
                if (s_best[w] < best || (s_best[w] == best && s_bj[w] < bj)) { best = s_best[w]; bj = s_bj[w]; }
            labels[(size_t)h * N + n] = bj < C ? bj : 0;    // (no distance is a finite number: cluster 0)
        }
    }
}

// ---------------------------------------------------------------- assign, fp32
// grid (token blocks, H, sides), block 64 * KF_NW; the side with more work (the last one: the K tokens of a layer) comes
// first.  The centroid tile is the A operand, 32 tokens are the B operand, a lane's 16 accumulators are 16 centroids of ONE token.
//
// With more than KF_SPLIT centroids the operands are taken as two fp16 halves (f32_split: x to 2^-23) and a product as hi hi +
// hi lo + lo hi, three 32x32x16 instructions that take a fifth of the time of the eight 32x32x2 fp32 ones, which bound the kernel.
// A token is brought to 2^14 .. 2^15 by a power of two, the centroids of a head by one that follows from their largest norm.  The rule
// (`split`): tokens of a block and the largest centroid finite and within 2^+-KF_EXP, some token of the block with |x|^2 at least KF_FAR of the
// largest ||c||^2 (else most distances are near-ties, below), no near-ties in numbers in an iteration before.  Anything else, up to KF_SPLIT
// centroids, where splitting 32 tokens costs what it saves (2 x 1000 in 60: 69.5
// against 67.4 us per five iterations; one head of 700 in 24 54.8 against 53.0), and calls with little to do (kmeans_f32_split) go
// through the fp32 instruction: contraction index in its natural order (lane half h supplies the elements of parity h), the
// instruction adds its two products one after the other with a rounding behind each, so an accumulator is bit for bit the chain
// of fmaf over k = 0 .. D - 1.  That chain decides the label in either case: the split products leave the tokens whose two best distances
// are closer than KF_TIE D |x| max |c| + 2^-22 (|best| + |second|) to it.  The first term is four times the most that two dot products may
// be apart: D roundings of 2^-24 |x| |c| for the chain, which partial sums in one direction nearly reach, and twice that for the split
// products (2^-21 for the parts and lo lo; their sums measured at less than the chain's: of differences of two distances 0.5e-6 of
// |x|^2 + |c|^2 on 7.7 million tokens next to a border, 0.7e-6 by the chain).  The second term is for the rounding of the distances themselves.
// Up to KF_TIES such tokens of a block are taken one at a time; a block with more goes through the fp32 instruction as well, and in the
// iterations that follow through that alone (a word of flag_list per block).  Tokens that come twice as centroids, and tokens far from the
// origin, are near-ties all of them.  Five iterations, us, fp32 instruction alone / one token at a time without a limit / now: 4 x 9601 in 500, D =
// 128, a third of the tokens equal 575 / 1069 / 477, all equal 536 / 2497 / 422, one centroid 2^10 times as long 536 / 2487 / 388; 24 x 16,384, D = 64, a
// third equal 1924 / 3626 / 1482.  (The update step is faster than it was with the first figure.)  With limits of 1, 2, 4 tokens: 6 x 12,000 in 1000,
// D = 64, one token in twenty equal 846, 753, 690, offset of 30 deviations 671, 755, 1038; 4 x 9601 in 500, D = 128, the same, 575, 490, 445 and 444, 439, 439.
//
// The centroids need no LDS: they come from a chunk-major copy (`ct`, consecutive lanes read consecutive 16 bytes) with two
// register buffers, the halves of a row block, each requested again as soon as it has been used.  What decides for few tokens is how
// many SIMDs have work, so the row blocks of a token block are dealt out to up to four wavefronts (KF_NW / nc token blocks
// per workgroup, nc wavefronts each, kmeans_f32_share) and the shares compared through LDS.  k-means of five iterations, D = 128,
// fp32 instruction -> split: 4 x 9601 in 500 centroids 406 -> 304 us, 24 x 16,384 in
// 500 2769 -> 1410, 6 x 12,000 in 1000 1021 -> 659.  One
// token per thread with the centroids in LDS took 770 us per iteration for 4 heads of 9601 tokens against 100 and 500.
static constexpr int KF_NW = 4;
static constexpr int KF_SPLIT = 64;             // most centroids that go through the fp32 instruction whatever the values
static constexpr int KF_EXP = 40;
static constexpr float KF_FAR = 0x1p-8f;
static constexpr int KF_TIES64 = 2, KF_TIES128 = 4;
static constexpr long long KF_SPLIT_BLOCKS = 1024;      // token blocks of 128 elements, over all heads
static constexpr float KF_TIE = 7.152557373046875e-07f;  // 4 (1 + 2) 2^-24
static constexpr int KF_CHAINS = 4;                     // centroids of a lane side by side

template <int D, bool OBJ>
__global__ __launch_bounds__(64 * KF_NW, D == 64 ? 4 : 2) void kmeans_assign_f32_kernel(KmArgs a, KmIter it)
{
    constexpr int NB = D / 16;                  // float4 per register buffer: half of a lane's half row
    __shared__ float s_cn[SVG2_MAX_CLUSTERS];
    __shared__ float s_best[KF_NW][32], s_second[KF_NW][32];
    __shared__ int s_idx[KF_NW][32];
    __shared__ unsigned s_most[KF_NW];
    const int side = (int)(gridDim.z - 1 - blockIdx.z);
    const KmSide S = side ? a.s[1] : a.s[0];
    int32_t *labels = side ? it.lab[1] : it.lab[0];
    const int N = a.N, C = S.C, h = blockIdx.y, tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, col = lane & 31;
    const int nrb = (C + 31) / 32;
    const int nc = KM_SEL(a.nc, side);
    const int wc = wave % nc, wt = wave / nc;
    const int wg_tok0 = (int)blockIdx.x * (KF_NW / nc) * 32;
    if (wg_tok0 >= N) return;                   // the grid is sized for the larger nc
    const int n0 = wg_tok0 + wt * 32, n = n0 + col;

    float x[D / 2];                             // x[s]: element 2 s + half of the token
    auto load_x = [&]() {
        const float4 *src = reinterpret_cast<const float4 *>(static_cast<const float *>(S.X) +
                                                             ((size_t)h * N + min(n, N - 1)) * D + half * (D / 2));
#pragma unroll
        for (int k = 0; k < D / 8; ++k) {
            // the lane halves load half a row each and trade its odd elements for the other half's even ones
            const float4 v = src[k];
            const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v.x), __float_as_uint(v.y), false, false);
            const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(v.z), __float_as_uint(v.w), false, false);
            x[2 * k] = __uint_as_float(p[0]); x[D / 4 + 2 * k] = __uint_as_float(p[1]);
            x[2 * k + 1] = __uint_as_float(q[0]); x[D / 4 + 2 * k + 1] = __uint_as_float(q[1]);
        }
    };
    load_x();
    const char *ct = reinterpret_cast<const char *>(S.ct + (size_t)h * D * C);
    auto load_c = [&](float4 (&buf)[NB], int rb, int hf) {
        const unsigned off = 16u * (unsigned)(half * (D / 8) * C + min(rb * 32 + col, C - 1));     // (a head is 2 MB at most)
#pragma unroll
        for (int i = 0; i < NB; ++i) buf[i] = *reinterpret_cast<const float4 *>(ct + 16 * (size_t)(hf * NB + i) * C + off);
    };
    float4 bufA[NB], bufB[NB];                  // the two halves of a row block
    load_c(bufA, min(wc, nrb - 1), 0);
    unsigned cn_most = 0;                       // largest ||c||^2, as bits
    for (int c = tid; c < 32 * nrb; c += 64 * KF_NW) {
        const float v = c < C ? S.hcn[(size_t)h * C + c] : INFINITY;
        s_cn[c] = v;
        if (c < C) cn_most = max(cn_most, __float_as_uint(v));
    }
    const bool may_split = KM_SEL(a.split, side);
    int32_t *ties = S.flag_list + (size_t)h * N + n0;          // of this token block: whether it had many in an iteration before
    if (may_split) {
        for (int o = 32; o > 0; o >>= 1) cn_most = max(cn_most, (unsigned)__shfl_xor((int)cn_most, o));
        if (lane == 0) s_most[wave] = cn_most;
    }
    float x2 = 0.f;
    if ((OBJ && S.objective) || may_split) {
#pragma unroll
        for (int k = 0; k < D / 2; ++k) x2 = fmaf(x[k], x[k], x2);
        x2 += __shfl_xor(x2, 32);
    }
    __syncthreads();

    float best = INFINITY, second = INFINITY;           // (second: of the split loop only)
    int bidx = 0;
    // accumulator i is centroid 8 (i / 4) + 4 half + i % 4 of the row block: ascending in a lane, so strict <
    // keeps the lowest index; the padding rows of the last block are at infinity
    auto compare = [&](const f32x16 &acc, int rb, float mul, auto with_second) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int j = rb * 32 + 8 * (i >> 2) + 4 * half + (i & 3);
            const float dist = fmaf(mul, acc[i], s_cn[j]);
            if constexpr (decltype(with_second)::value) second = __builtin_amdgcn_fmed3f(best, second, dist);
            if (dist < best) { best = dist; bidx = j; }
        }
    };
    // the two lane halves, then the wavefronts of a token block, hold disjoint centroids of the same token
    auto merge = [&](float ob, int oj, float os) {
        second = fminf(fminf(second, os), fmaxf(best, ob));
        if (ob < best || (ob == best && oj < bidx)) { best = ob; bidx = oj; }
    };
    auto merge_halves = [&]() {
        merge(__shfl_xor(best, 32), __shfl_xor(bidx, 32), __shfl_xor(second, 32));
        if (nc > 1 && half == 0) { s_best[wave][col] = best; s_idx[wave][col] = bidx; s_second[wave][col] = second; }
    };
    auto merge_waves = [&]() {
        for (int w = 1; w < nc; ++w) {
            const int o = wave - wc + (wc + w) % nc;
            merge(s_best[o][col], s_idx[o][col], s_second[o][col]);
        }
    };
    // split operands or not (the comment above)
    float x_up = 1.f, c_up = 1.f;
    bool split = false, tied = false;
    unsigned near = 0;
    if (may_split) {
        cn_most = s_most[0];
#pragma unroll
        for (int w = 1; w < KF_NW; ++w) cn_most = max(cn_most, s_most[w]);
        unsigned xb = 0;
#pragma unroll
        for (int k = 0; k < D / 2; ++k) xb = max(xb, __float_as_uint(x[k]) & 0x7FFFFFFFu);
        xb = max(xb, (unsigned)__shfl_xor((int)xb, 32));
        const int xe = xb == 0 ? 0 : (int)(xb >> 23) - 127, ce = (int)(cn_most >> 23) - 127;
        tied = it.t > 0 && n0 < N && *ties != 0;
        split = !tied && abs(ce) <= 2 * KF_EXP && __all(abs(xe) <= KF_EXP) && __any(x2 >= KF_FAR * __uint_as_float(cn_most));
        x_up = __uint_as_float((unsigned)(127 + 14 - xe) << 23);
        c_up = __uint_as_float((unsigned)(127 + 15 - ((ce + 2) >> 1)) << 23);       // |c| < 2^((ce + 1) / 2)
    }
    if (split) {
        f16x8 xh[D / 16], xl[D / 16];
#pragma unroll
        for (int t = 0; t < D / 16; ++t)
#pragma unroll
            for (int e = 0; e < 8; ++e) f32_split(x[8 * t + e], x_up, xh[t], xl[t], e);
        const float mul = -2.f * (1.f / x_up) * (1.f / c_up);
        auto half_block = [&](f32x16 &acc, float4 (&buf)[NB], int hf) {
            // (pinned: the compiler otherwise splits ahead of the loads' turn, all halves at once, and spills)
#pragma unroll
            for (int i = 0; i < NB; ++i) asm volatile("" : "+v"(buf[i].x), "+v"(buf[i].y), "+v"(buf[i].z), "+v"(buf[i].w));
#pragma unroll
            for (int t = 0; t < NB / 2; ++t) {
                const float c[8] = {buf[2 * t].x, buf[2 * t].y, buf[2 * t].z, buf[2 * t].w,
                                    buf[2 * t + 1].x, buf[2 * t + 1].y, buf[2 * t + 1].z, buf[2 * t + 1].w};
                f16x8 ch, cl;
#pragma unroll
                for (int e = 0; e < 8; ++e) f32_split(c[e], c_up, ch, cl, e);
                const int i = hf * (NB / 2) + t;
                acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(cl, xh[i], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(ch, xl[i], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(ch, xh[i], acc, 0, 0, 0);
            }
        };
        load_c(bufB, min(wc, nrb - 1), 1);
        for (int rb = wc; rb < nrb; rb += nc) {
            const int next = min(rb + nc, nrb - 1);     // (past the last row block: a valid one, not used)
            f32x16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            half_block(acc, bufA, 0);
            __builtin_amdgcn_sched_barrier(0);
            load_c(bufA, next, 0);
            __builtin_amdgcn_sched_barrier(0);
            half_block(acc, bufB, 1);
            __builtin_amdgcn_sched_barrier(0);
            load_c(bufB, next, 1);
            __builtin_amdgcn_sched_barrier(0);
            compare(acc, rb, mul, std::true_type{});
            __builtin_amdgcn_sched_barrier(0);
        }
        merge_halves();
#pragma unroll
        for (int k = 0; k < D / 2; ++k) x[k] = 0.f;             // (read again below, not held over the loop)
    }
    if (may_split) {                                            // (the same for the workgroup)
        if (nc > 1) __syncthreads();
        if (split) {
            merge_waves();
            const float tie = KF_TIE * D * __builtin_amdgcn_sqrtf(x2) * __builtin_amdgcn_sqrtf(__uint_as_float(cn_most)) +
                              0x1p-22f * (fabsf(best) + fabsf(second));
            near = (unsigned)__ballot(n < N && !(second - best > tie));
            if (__popc(near) > (D == 64 ? KF_TIES64 : KF_TIES128)) {
                split = false;
                tied = true;
                best = second = INFINITY;
                bidx = 0;
                load_x();
                load_c(bufA, min(wc, nrb - 1), 0);
            }
        }
        if (lane == 0 && wc == 0 && n0 < N) *ties = tied;
    }
    if (nc > 1 && may_split ? __syncthreads_or(!split) : !split) {
        if (!split) {
            for (int rb = wc; rb < nrb; rb += nc) {
                load_c(bufB, rb, 1);
                __builtin_amdgcn_sched_barrier(0);
                f32x16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(bufA[i].x, x[4 * i], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(bufA[i].y, x[4 * i + 1], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(bufA[i].z, x[4 * i + 2], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(bufA[i].w, x[4 * i + 3], acc, 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                load_c(bufA, min(rb + nc, nrb - 1), 0);     // (past the last row block: a valid one, not used)
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(bufB[i].x, x[4 * (NB + i)], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(bufB[i].y, x[4 * (NB + i) + 1], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(bufB[i].z, x[4 * (NB + i) + 2], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(bufB[i].w, x[4 * (NB + i) + 3], acc, 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                compare(acc, rb, -2.f, std::false_type{});
            }
            merge_halves();
        }
        if (nc > 1) __syncthreads();
        if (!split) merge_waves();
    }
    if (wc != 0) return;
    // elements 8 q .. 8 q + 7 of the chain of fmaf for centroid j
    auto chain8 = [&](float &dot, int q, int j, const float4 &x0, const float4 &x1) {
        const float4 ev = *reinterpret_cast<const float4 *>(ct + 16 * ((size_t)q * C + j));
        const float4 od = *reinterpret_cast<const float4 *>(ct + 16 * ((size_t)(D / 8 + q) * C + j));
        dot = fmaf(ev.x, x0.x, dot); dot = fmaf(od.x, x0.y, dot);
        dot = fmaf(ev.y, x0.z, dot); dot = fmaf(od.y, x0.w, dot);
        dot = fmaf(ev.z, x1.x, dot); dot = fmaf(od.z, x1.y, dot);
        dot = fmaf(ev.w, x1.z, dot); dot = fmaf(od.w, x1.w, dot);
    };
    // Near-ties of the split products go by the chain of fmaf, as all tokens do without them: a token at a time, KF_CHAINS centroids per
    // lane (one after the other, its loads all requested at once: 6 x 12,000 in 1000 721 instead of 621 us, 1 x 12,000 287 instead of 222).
    if (split) {
        for (; near; near &= near - 1) {
            const int c32 = __builtin_ctz(near);
            const float *xr = static_cast<const float *>(S.X) + ((size_t)h * N + n0 + c32) * D;     // (uniform)
            float tb = INFINITY;
            int tj = 0;
            for (int j0 = lane; j0 < C; j0 += 64 * KF_CHAINS) {
                float dot[KF_CHAINS] = {};
#pragma unroll 2
                for (int q = 0; q < D / 8; ++q) {
                    const float4 x0 = *reinterpret_cast<const float4 *>(xr + 8 * q), x1 = *reinterpret_cast<const float4 *>(xr + 8 * q + 4);
#pragma unroll
                    for (int u = 0; u < KF_CHAINS; ++u) chain8(dot[u], q, min(j0 + 64 * u, C - 1), x0, x1);
                }
#pragma unroll
                for (int u = 0; u < KF_CHAINS; ++u) {
                    const int j = min(j0 + 64 * u, C - 1);      // (past the last one: that one again, which changes nothing)
                    const float dist = fmaf(-2.f, dot[u], s_cn[j]);
                    if (dist < tb) { tb = dist; tj = j; }
                }
            }
            for (int o = 32; o > 0; o >>= 1) {
                const float ob = __shfl_xor(tb, o);
                const int oj = __shfl_xor(tj, o);
                if (ob < tb || (ob == tb && oj < tj)) { tb = ob; tj = oj; }
            }
            if (col == c32) { best = tb; bidx = tj; }
        }
    }
    if (half == 0 && n < N) labels[(size_t)h * N + n] = bidx;
    if (OBJ && S.objective) {
        if (split) {
            // The distance of the chain, whatever found the label: hi hi + hi lo + lo hi lacks lo lo, which is a square for a token near its
            // centroid, so all distances were too large by up to 2^-22 |x|^2.
            const float *xr = static_cast<const float *>(S.X) + ((size_t)h * N + min(n, N - 1)) * D;
            float dot = 0.f;
            for (int q = 0; q < D / 8; ++q) {
                const float4 x0 = *reinterpret_cast<const float4 *>(xr + 8 * q), x1 = *reinterpret_cast<const float4 *>(xr + 8 * q + 4);
                chain8(dot, q, bidx, x0, x1);
            }
            best = fmaf(-2.f, dot, s_cn[bidx]);
        }
        float v = (half == 0 && n < N) ? x2 + best : 0.f;
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
        if (lane == 0) atomicAdd(S.objective + (size_t)h * a.iters + it.t, v);
    }
}

// A handful of centroids: one token per thread, the centroids in LDS, the same chain of fmaf over k.  The 32-row tile of the
// matrix instruction would be mostly padding: 24 heads of 16,384 tokens, D = 128: 32 instead of 63 us with 2 centroids, 55
// instead of 63 with 12; one head of 4096, D = 64: 4.6 instead of 5.2 us with 4.  With more than four centroids it takes
// many tokens, or the wavefronts that share a token block there are faster (one head of 4096, D = 64: 5.4 against 5.2 us
// with 6 centroids, 8.3 against 5.0 with 12; 4 heads of 9601, D = 128: 10.3 against 12.7 with 6, 14.5 against 13.2 with 12).
static constexpr int KF_FEW = 12, KF_FEW_ANY = 4, KF_FEW_TOKENS = 8192;  // .. and tokens of all heads per centroid

static bool kmeans_f32_few(int H, int N, int C)
{
    return C <= KF_FEW_ANY || (C <= KF_FEW && (long long)H * N >= (long long)KF_FEW_TOKENS * C);
}

template <int D, bool OBJ>
__global__ __launch_bounds__(128) void kmeans_assign_f32_few_kernel(KmArgs a, KmIter it, int side)
{
    __shared__ __align__(16) float s_c[KF_FEW][D];
    __shared__ float s_cn[KF_FEW];
    const KmSide S = side ? a.s[1] : a.s[0];
    int32_t *labels = side ? it.lab[1] : it.lab[0];
    const int N = a.N, C = S.C, h = blockIdx.y, tid = threadIdx.x, n = blockIdx.x * 128 + tid;
    const float4 *xr = reinterpret_cast<const float4 *>(static_cast<const float *>(S.X) + ((size_t)h * N + min(n, N - 1)) * D);
    float x[D];
#pragma unroll
    for (int k = 0; k < D / 4; ++k) {
        const float4 v = xr[k];
        x[4 * k] = v.x; x[4 * k + 1] = v.y; x[4 * k + 2] = v.z; x[4 * k + 3] = v.w;
    }
    for (int e = tid; e < C * D; e += 128) {
        const int j = e / D, k = e % D;
        s_c[j][k] = S.ct[((((size_t)h * 2 + (k & 1)) * (D / 8) + (k >> 3)) * C + j) * 4 + ((k >> 1) & 3)];
    }
    if (tid < C) s_cn[tid] = S.hcn[(size_t)h * C + tid];
    __syncthreads();
    float best = INFINITY;
    int bidx = 0;
    for (int j = 0; j < C; ++j) {
        float dot = 0.f;
#pragma unroll
        for (int k = 0; k < D; ++k) dot = fmaf(x[k], s_c[j][k], dot);
        const float dist = fmaf(-2.f, dot, s_cn[j]);
        if (dist < best) { best = dist; bidx = j; }
    }
    if (n < N) labels[(size_t)h * N + n] = bidx;
    if (OBJ && S.objective) {
        float x2 = 0.f;
#pragma unroll
        for (int k = 0; k < D; ++k) x2 = fmaf(x[k], x[k], x2);
        float v = n < N ? x2 + best : 0.f;
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
        if ((tid & 63) == 0) atomicAdd(S.objective + (size_t)h * a.iters + it.t, v);
    }
}

// ---------------------------------------------------------------- update
// Segmented sum over the sorted order, one wavefront per piece (at most KM_SEG rows of one cluster).  A row is LPR
// lanes of 16 bytes; 64 / LPR rows are read per instruction and KM_UB instructions are in flight before their
// values are added, in double precision.
//   DELTA = false  grid (ceil(max_pieces / 4), H, sides): every row of the piece (set `it.set`).
//   DELTA = true   grid (.., H, 2 * sides), z = 2 * side + dir: only the rows of a piece whose label in `other`
//                  differs from the piece's cluster.  dir 0: the new order (set) against the previous labels --
//                  the tokens that JOINED the cluster; dir 1: the previous order (other set) against the new
//                  labels -- the tokens that LEFT it.  A wavefront first scans its piece one row per lane and
//                  packs the rows that qualify into a list, then reads only those rows of X.
//
template <typename T> __device__ __forceinline__ void add_row(const uint4 &v, double (&acc)[16 / sizeof(T)])
{
    const unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if constexpr (sizeof(T) == 2) {
            acc[2 * q] += (double)__uint_as_float(w[q] << 16);
            acc[2 * q + 1] += (double)__uint_as_float(w[q] & 0xFFFF0000u);
        } else {
            acc[q] += (double)__uint_as_float(w[q]);
        }
    }
}

// acc = sum of the rows row(0) .. row(cnt - 1) of Xh, by one wavefront: the elements part * EPL .. of every lane whose row part that is
template <typename T, int D, int UB, typename R>
__device__ __forceinline__ void sum_rows(const T *Xh, int cnt, R row, double (&acc)[16 / sizeof(T)])
{
    constexpr int EPL = 16 / sizeof(T);            // elements per lane
    constexpr int LPR = D / EPL;                   // lanes per row
    constexpr int RPI = 64 / LPR;                  // rows per instruction
    const int lane = threadIdx.x & 63, sub = lane / LPR, part = lane % LPR;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[e] = 0.0;
    for (int r = 0; r < cnt; r += RPI * UB) {
        uint4 v[UB];
#pragma unroll
        for (int u = 0; u < UB; ++u)
            v[u] = reinterpret_cast<const uint4 *>(Xh + (size_t)row(min(r + u * RPI + sub, cnt - 1)) * D)[part];
#pragma unroll
        for (int u = 0; u < UB; ++u)
            if (r + u * RPI + sub < cnt) add_row<T>(v[u], acc);
    }
    // lanes with the same `part` hold the same columns
#pragma unroll
    for (int o = LPR; o < 64; o <<= 1)
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] += __shfl_xor(acc[e], o);
}

// One piece (rows row0 .. + nrows of the sorted order pm) of cluster cl by one wavefront: acc = the sum of its rows that
// qualify, the elements part * EPL .. of every lane whose row part that is; returns how many rows there are (0: no acc).
template <typename T, int D, bool DELTA>
__device__ __forceinline__ int sum_piece(const T *Xh, const int32_t *pm, const int32_t *other, int cl, int row0, int nrows,
                                         int32_t *list, double (&acc)[16 / sizeof(T)])
{
    const int lane = threadIdx.x & 63;
    int cnt = nrows;
    if (DELTA) {
        const unsigned long long lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
        cnt = 0;
        // the rows of the piece and then their other labels are requested together: two memory round trips
        // for the piece instead of two per 64 rows
        constexpr int NG = KM_SEG / 64;
        int srcs[NG], oth[NG];
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            const int rr = i * 64 + lane;
            srcs[i] = (rr < nrows) ? pm[row0 + rr] : 0;
        }
#pragma unroll
        for (int i = 0; i < NG; ++i) oth[i] = other[srcs[i]];
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            if (i * 64 >= nrows) break;
            const bool take = i * 64 + lane < nrows && oth[i] != cl;
            const unsigned long long m = __ballot(take);
            if (take) list[cnt + __popcll(m & lt_mask)] = srcs[i];
            cnt += __popcll(m);
        }
        if (cnt == 0) return 0;
    }
    sum_rows<T, D, KM_UB>(Xh, cnt, [&](int r) { return DELTA ? list[r] : pm[row0 + r]; }, acc);
    return cnt;
}

template <typename T, int D, bool DELTA>
__global__ __launch_bounds__(256) void kmeans_segsum_kernel(KmArgs a, KmIter it)
{
    constexpr int EPL = 16 / sizeof(T), LPR = D / EPL;
    __shared__ int32_t s_list[DELTA ? 4 : 1][DELTA ? KM_SEG : 1];
    const int side = DELTA ? blockIdx.z >> 1 : blockIdx.z, dir = DELTA ? (blockIdx.z & 1) : 0;
    const KmSide S = side ? a.s[1] : a.s[0];
    const int set = dir ? 1 - it.set : it.set;
    const int h = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, N = a.N;
    const int piece = blockIdx.x * 4 + wave;
    if (piece >= KM_SEL(S.n_pieces, set)[h]) return;
    const int4 desc = KM_SEL(S.pieces, set)[(size_t)h * S.max_pieces + piece];
    const int32_t *other = nullptr;
    if (DELTA)
        other = (dir ? (side ? it.lab[1] : it.lab[0]) : (side ? it.lab_prev[1] : it.lab_prev[0])) + (size_t)h * N;
    double acc[EPL];
    const int cnt = sum_piece<T, D, DELTA>(reinterpret_cast<const T *>(S.X) + (size_t)h * N * D,
                                           KM_SEL(S.perm, set) + (size_t)h * N, other, desc.x, desc.y, desc.z,
                                           s_list[DELTA ? wave : 0], acc);
    if (DELTA) {
        if (lane == 0) KM_SEL(S.moved, set)[(size_t)h * S.max_pieces + piece] = cnt;
        if (cnt == 0) return;
    }
    if (lane < LPR) {
        double *out = KM_SEL(S.psum, set) + ((size_t)h * S.max_pieces + piece) * D + lane * EPL;
#pragma unroll
        for (int e = 0; e < EPL; e += 2) *reinterpret_cast<double2 *>(out + e) = make_double2(acc[e], acc[e + 1]);
    }
}

// The whole update step of a cluster in one workgroup, for heads of at most KM_SMALL_N tokens, straight from the labels: the
// wavefronts go through the labels of the head, list the cluster's tokens (mode 1) or those that joined and those that left it
// (mode 2) in token order, sum the lists in pieces of KM_SEG rows, and the first wavefront adds these in their order and finishes the
// cluster.  So an iteration needs no sort; the last one sorts for the order that is handed on.
//
// A workgroup has to be able to walk a cluster that holds most of the head about as fast as the pieces would be walked side
// by side: four wavefronts up to 2048 tokens, sixteen above, where fewer such workgroups run at once.  Five iterations in us,
// clusters of about equal size, then one of all tokens; the kernels of the longer heads / this one:
//   40 heads x 2048, bf16, D = 128, 50 clusters (2000): 201 / 168, 169 / 155      100 x 1100, 64, 30 (3000): 168 / 145, 152 / 141
//   40 x 2048, 128, 100 (4000): 198 / 189, 181 / 191                              24 x 4096, 128, 30 (720): 225 / 230, 170 / 164
// the same workgroup behind a sort / this one:
//   1 head x 4096, fp32, D = 64, 16 clusters: 105 / 77, 99 / 69                   1 x 2048, bf16, 128, 100: 137 / 112, 156 / 122
//   1 x 4096, bf16, 128, 100: 155 / 128, 159 / 126                                40 x 4096, 128, 12: 255 / 237, 200 / 175
static constexpr int KM_SMALL_N = 4096, KM_SMALL_N4 = 2048;     // tokens of a head, with 16 and with 4 wavefronts
static constexpr int KM_SMALL_WG = 512, KM_SMALL_WG4 = 3072;    // .. and clusters of all heads

static bool kmeans_update_small(int H, int N, int C)
{
    return N <= KM_SMALL_N && (long long)C * H <= (N <= KM_SMALL_N4 ? KM_SMALL_WG4 : KM_SMALL_WG);
}

template <typename T, int D, bool BF16, int NW>
__global__ __launch_bounds__(64 * NW) void kmeans_update_small_kernel(KmArgs a, KmIter it, int mode)
{
    constexpr int EPL = 16 / sizeof(T), LPR = D / EPL, RPI = 64 / LPR, EL = D / 64;
    constexpr int NMAX = NW == 4 ? KM_SMALL_N4 : KM_SMALL_N, NG = NMAX / (64 * NW);    // groups of 64 labels per wavefront
    constexpr int NP = 2 * NMAX / KM_SEG + 2;                                          // most pieces of a cluster, joined and left
    __shared__ __align__(16) double s_ps[NP][D];
    __shared__ uint16_t s_list[2 * NMAX];           // those that joined, then those that left
    __shared__ int32_t s_cnt[3][NW];                // per wavefront: joined, left, in the cluster
    const int h = blockIdx.y, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), N = a.N;
    const int side = (int)blockIdx.x >= a.s[0].C ? 1 : 0;
    const KmSide S = side ? a.s[1] : a.s[0];
    const int j = (int)blockIdx.x - (side ? a.s[0].C : 0);
    const T *Xh = reinterpret_cast<const T *>(S.X) + (size_t)h * N * D;
    const int32_t *lab = (side ? it.lab[1] : it.lab[0]) + (size_t)h * N;
    const int32_t *prev = mode == 2 ? (side ? it.lab_prev[1] : it.lab_prev[0]) + (size_t)h * N : lab;
    unsigned long long in[NG], out[NG];
    {
        int l[NG], p[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const int n = min((wave * NG + g) * 64 + lane, N - 1);
            l[g] = lab[n];
            p[g] = prev[n];
        }
        int n_in = 0, n_out = 0, n_all = 0;
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const bool ok = (wave * NG + g) * 64 + lane < N;
            in[g] = __ballot(ok && l[g] == j && (mode != 2 || p[g] != j));
            out[g] = __ballot(ok && l[g] != j && p[g] == j);
            n_in += __popcll(in[g]);
            n_out += __popcll(out[g]);
            n_all += __popcll(__ballot(ok && l[g] == j));
        }
        if (lane == 0) { s_cnt[0][wave] = n_in; s_cnt[1][wave] = n_out; s_cnt[2][wave] = n_all; }
    }
    __syncthreads();
    int tot_in = 0, tot_out = 0, cnt = 0, at_in = 0, at_out = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        at_in += w < wave ? s_cnt[0][w] : 0;
        at_out += w < wave ? s_cnt[1][w] : 0;
        tot_in += s_cnt[0][w];
        tot_out += s_cnt[1][w];
        cnt += s_cnt[2][w];
    }
    at_out += tot_in;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const unsigned long long lt = (1ull << lane) - 1ull;
        const int n = (wave * NG + g) * 64 + lane;
        if (in[g] >> lane & 1) s_list[at_in + __popcll(in[g] & lt)] = (uint16_t)n;
        if (out[g] >> lane & 1) s_list[at_out + __popcll(out[g] & lt)] = (uint16_t)n;
        at_in += __popcll(in[g]);
        at_out += __popcll(out[g]);
    }
    __syncthreads();
    const int np_in = (tot_in + KM_SEG - 1) / KM_SEG, np = np_in + (tot_out + KM_SEG - 1) / KM_SEG;
    double s_prev[EL];
    int n_prev = 0;
#pragma unroll
    for (int e = 0; e < EL; ++e) s_prev[e] = 0.0;
    if (wave == 0 && it.t > 0) {            // used behind the last barrier
        n_prev = S.counts[(size_t)h * S.C + j];
#pragma unroll
        for (int e = 0; e < EL; ++e) s_prev[e] = S.csum[((size_t)h * S.C + j) * D + lane + 64 * e];
    }
    const int sub = lane / LPR, part = lane % LPR;
    for (int q = wave; q < np; q += NW) {
        const int r0 = q < np_in ? q * KM_SEG : tot_in + (q - np_in) * KM_SEG;
        const int r1 = min(r0 + KM_SEG, q < np_in ? tot_in : tot_in + tot_out);
        double acc[EPL];
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] = 0.0;
        for (int r = r0; r < r1; r += RPI * KM_UB) {
            uint4 v[KM_UB];
#pragma unroll
            for (int u = 0; u < KM_UB; ++u)
                v[u] = reinterpret_cast<const uint4 *>(Xh + (size_t)s_list[min(r + u * RPI + sub, r1 - 1)] * D)[part];
#pragma unroll
            for (int u = 0; u < KM_UB; ++u)
                if (r + u * RPI + sub < r1) add_row<T>(v[u], acc);
        }
        // lanes with the same `part` hold the same columns
#pragma unroll
        for (int o = LPR; o < 64; o <<= 1)
#pragma unroll
            for (int e = 0; e < EPL; ++e) acc[e] += __shfl_xor(acc[e], o);
        if (lane < LPR) {
#pragma unroll
            for (int e = 0; e < EPL; e += 2)
                *reinterpret_cast<double2 *>(&s_ps[q][lane * EPL + e]) = make_double2(acc[e], acc[e + 1]);
        }
    }
    __syncthreads();
    if (wave != 0) return;
    double s[EL];
#pragma unroll
    for (int e = 0; e < EL; ++e) s[e] = mode == 2 ? s_prev[e] : 0.0;
    for (int q = 0; q < np; ++q)
#pragma unroll
        for (int e = 0; e < EL; ++e) s[e] += q < np_in ? s_ps[q][lane + 64 * e] : -s_ps[q][lane + 64 * e];
    if (j == 0 && lane == 0) S.flag_cnt[h] = 0;         // the next assign step starts an empty list
    finalize_cluster<BF16, D>(a, S, it, mode, h, j, s, cnt, s_prev, n_prev);
}

// The update step of up to KU_G clusters of a head in one workgroup, straight from the labels (mode 1: all tokens of the clusters, mode 2:
// those that joined and those that left one): the wavefronts go through the labels of the head, each through its share of
// them, and list the tokens in token order; the lists are sorted by (cluster, joined / left) in LDS, stably, summed in pieces of
// KU_PIECE rows by one wavefront each, KU_SLOTS pieces at a time, and the pieces added to the clusters' sums in their order -- so
// that fp32 sums are the same in every run.  A wavefront whose list is full waits for the next round of this.  At the
// end the wavefronts finish the clusters.  So an iteration needs no sort; the last one sorts for the order that is handed on.
//
// What bounds it is the chain of round trips (labels, rows) and the labels, which every workgroup reads whole; sort, sums and means of
// the longer heads are a chain of three to five launches.  Five iterations in us, those / this kernel:
//   24 heads x 16,384, bf16, D = 128, 100 / 500 clusters: 384 / 334, 568 / 505      24 x 9601, 500: 446 / 368      6 x 11,000, 150: 257 / 203
//   24 x 30,000, 500: 823 / 762      2 x 30,000, 300: 295 / 250      4 x 20,000, D = 64, 1000: 369 / 283      4 x 9601, fp32, 500: 540 / 488
// Beyond KU_N tokens the labels cost as much as is gained (8 x 37,800, 500: 523 / 499; 1 x 75,600: 341 / 357; 1 x 118,800, 64: 237 / 439).
// All tokens are summed this way (mode 1) up to KU_FULL_N: a workgroup then has all rows of its clusters to add, about 100 rows per us, and of
// a cluster that holds most of a long head the pieces side by side are faster.  Two iterations, bf16, D = 128, sorted in the first / not at
// all: 12 heads x 4096 tokens, 100 clusters: 97 / 70 us, all tokens in one cluster 85 / 93; 12 x 5000 88 / 69, in one 81 / 104; 12 x 8000 97 / 82, in one 84 / 135.
// The same holds for the many tokens that move in the second iteration, and with clusters large enough for those of all later ones.  So the
// second iteration goes by the sorted order from KU_SECOND_SIZE tokens per cluster on (the first one has left its order, beyond KU_FULL_N), every
// iteration from KU_SIZE on.  D = 128, centroids drawn from the tokens, cluster sizes alike / Zipf; sorted, by the labels, now:
//   two iterations: bf16 4 x 17,000 in 8 122, 125, 121 / 128, 168, 125; 24 x 32,000 in 16 215, 232, 216 / 223, 302, 224; fp32 1 x 32,000 in 32
//   120, 153, 120 / 118, 120, 118; 4 x 32,000 in 4 141, 193, 139 / 145, 270, 145
//   five: bf16 24 x 32,000 in 16 483, 439, 422 / 495, 540, 464; fp32 4 x 32,000 in 16 325, 340, 304 / 349, 419, 339, in 8 308, 396, 307 / 325, 418, 326
// What remains is tokens that move at once between two of many clusters: a third of them in the second of two iterations, fp32, D = 128,
// sorted / by labels 12 x 12,000 in 100 254 / 277, 24 x 16,384 in 500 1406 / 1181.
// bf16 heads of more than KU_LISTS_N tokens: the assign step lists the tokens that moved (KU_LISTS, kmeans_update_lists).  With four
// wavefronts in place of eight, so that all workgroups of 24 heads of 16,384 tokens run at once, a late iteration
// took 21 instead of 26 us and the first of them 97 instead of 60; with 32 clusters to a workgroup and several workgroups for the tokens
// of few clusters 34 and 88.
// As few workgroups as give every CU one read the labels (three times as many: 24 x 16,384, 500 clusters: 544; 6 x 11,000, 150: 232).
static constexpr int KU_N = 32768, KU_FULL_N = 4096, KU_LISTS_N = 8192;
static constexpr int KU_SIZE = 2048, KU_SECOND_SIZE = 256;      // tokens per cluster: most, and most in the second iteration
static constexpr int KU_NW = 8;                 // wavefronts
static constexpr int KU_G = 16;                 // most clusters of a workgroup
static constexpr int KU_CAP = 448;              // entries of a wavefront's list (three workgroups fit a CU)
static constexpr int KU_PIECE = 64, KU_SLOTS = 16, KU_UB = 4;
static constexpr int KU_LB = 4;                 // groups of 64 labels requested together
static constexpr int KU_B = 2 * KU_G;           // (cluster, left) pairs
static_assert(KU_B * KU_NW == 256 && KU_B <= 32, "the scan below: four wavefronts, a lane of half a wavefront per pair");
static_assert(KU_SLOTS == KU_G, "the sums of the clusters go out through the pieces' LDS");

enum { KU_ALL = 0, KU_LABELS = 1, KU_LISTS = 2 };     // all tokens; those that moved, by the labels; by the assign step's lists

template <typename T, int D, bool BF16, int MODE>
__global__ __launch_bounds__(64 * KU_NW, 6) void kmeans_update_kernel(KmArgs a, KmIter it)
{
    constexpr bool DELTA = MODE != KU_ALL;
    constexpr int EPL = 16 / sizeof(T), LPR = D / EPL, EL = D / 64;
    __shared__ __align__(16) double s_ps[KU_SLOTS][D];
    __shared__ int32_t s_ent[KU_NW][KU_CAP];    // listed tokens
    __shared__ uint8_t s_bkt[KU_NW][KU_CAP];    // and their 2 * cluster + left
    __shared__ int32_t s_tok[KU_NW * KU_CAP];   // sorted
    __shared__ int32_t s_hist[KU_NW][KU_B];
    __shared__ int32_t s_start[KU_B + 1], s_fp[KU_B + 1], s_tot[KU_B], s_sum[4];
    __shared__ int32_t s_more;
    const int h = blockIdx.y, N = a.N, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ng0 = (a.s[0].C + a.gc[0] - 1) / a.gc[0];
    const int side = (int)blockIdx.x >= ng0 ? 1 : 0;
    const KmSide S = side ? a.s[1] : a.s[0];
    const int gc = KM_SEL(a.gc, side), c0 = ((int)blockIdx.x - (side ? ng0 : 0)) * gc, nc = min(gc, S.C - c0);
    const T *Xh = reinterpret_cast<const T *>(S.X) + (size_t)h * N * D;
    const int32_t *lab = (side ? it.lab[1] : it.lab[0]) + (size_t)h * N;
    const int32_t *prev = (side ? it.lab_prev[1] : it.lab_prev[0]) + (size_t)h * N;
    const unsigned long long lt = (1ull << lane) - 1ull;
    // this wavefront's share of the tokens, whole groups of 64
    const int ngrp = (N + 63) / 64, per = (ngrp + KU_NW - 1) / KU_NW, hi = min(ngrp, (wave + 1) * per);
    int pos = min(ngrp, wave * per);
    const unsigned *mv = S.mv_list + (size_t)h * N;
    const int32_t *mvc = S.mv_cnt + (size_t)h * 4 * S.max_pieces;
    int ent = 0;                                // lists: next entry of the 64 groups from pos on

    // thread (msub, mk): element mk of the sums of the clusters msub, msub + NSUB, ..
    constexpr int NSUB = 64 * KU_NW / D, JN = KU_G / NSUB;
    const int mk = tid % D, msub = tid / D;
    double csum[JN];
#pragma unroll
    for (int i = 0; i < JN; ++i) {
        const int j = msub + NSUB * i;
        csum[i] = DELTA && j < nc ? S.csum[((size_t)h * S.C + c0 + j) * D + mk] : 0.0;
    }
    int total = 0;                              // wavefront 0, lane b: entries of pair b so far

    for (bool more = true; more;) {
        int cnt = 0;
        if (tid < KU_B * KU_NW) (&s_hist[0][0])[tid] = 0;
        if (tid == 0) s_more = 0;
        __syncthreads();
        auto put = [&](bool take, int n, int pair) {
            const unsigned long long m = __ballot(take);
            if (m == 0) return;
            if (take) {
                const int at = cnt + __popcll(m & lt);
                s_ent[wave][at] = n;
                s_bkt[wave][at] = (uint8_t)pair;
                atomicAdd(&s_hist[wave][pair], 1);
            }
            cnt += __popcll(m);
        };
        constexpr int MOST = DELTA ? 128 : 64;  // entries of a group at most
        if constexpr (MODE == KU_LISTS) {
            while (pos < hi && cnt + MOST <= KU_CAP) {
                int incl = pos + lane < hi ? mvc[pos + lane] : 0;
                const int own = incl;
                for (int o = 1; o < 64; o <<= 1) {
                    const int u = __shfl_up(incl, o);
                    if (lane >= o) incl += u;
                }
                const int excl = incl - own, all = __builtin_amdgcn_readlane(incl, 63);
                while (ent < all && cnt + MOST <= KU_CAP) {
                    unsigned w[KU_LB];
                    int n0[KU_LB];
#pragma unroll
                    for (int u = 0; u < KU_LB; ++u) {
                        const int e = min(ent + 64 * u + lane, all - 1);
                        int g = 0;                          // groups whose entries end in front of e
#pragma unroll
                        for (int o = 32; o > 0; o >>= 1)
                            if (__shfl(incl, g + o - 1) <= e) g += o;
                        n0[u] = 64 * (pos + g);
                        w[u] = mv[n0[u] + e - __shfl(excl, g)];
                    }
#pragma unroll
                    for (int u = 0; u < KU_LB; ++u)
                        if (ent < all && cnt + MOST <= KU_CAP) {
                            const bool ok = ent + lane < all;
                            const int n = n0[u] + (int)(w[u] & 63u), p = (int)(w[u] >> 6 & 4095u) - c0;
                            int l = (int)(w[u] >> 18 & 4095u) - c0;
                            if (w[u] & KM_MV_OPEN) l = lab[n] - c0;
                            put(ok && l != p && (unsigned)l < (unsigned)nc, n, 2 * l);
                            put(ok && l != p && (unsigned)p < (unsigned)nc, n, 2 * p + 1);
                            ent += 64;
                        }
                }
                if (ent >= all) {
                    ent = 0;
                    pos += 64;
                }
            }
        } else {
            while (pos < hi && cnt + MOST <= KU_CAP) {
                int tl[KU_LB], tp[KU_LB];
#pragma unroll
                for (int u = 0; u < KU_LB; ++u) {
                    const int n = min(64 * (pos + u) + lane, N - 1);
                    tl[u] = lab[n];
                    if (DELTA) tp[u] = prev[n];
                }
#pragma unroll
                for (int u = 0; u < KU_LB; ++u)
                    if (pos < hi && cnt + MOST <= KU_CAP) {
                        const int n = 64 * pos + lane;
                        const bool ok = n < N && (!DELTA || tl[u] != tp[u]);
                        put(ok && (unsigned)(tl[u] - c0) < (unsigned)nc, n, 2 * (tl[u] - c0));
                        if (DELTA) put(ok && (unsigned)(tp[u] - c0) < (unsigned)nc, n, 2 * (tp[u] - c0) + 1);
                        ++pos;
                    }
            }
        }
        if (pos < hi && lane == 0) s_more = 1;
        __syncthreads();
        // ---- sort by pair, then wavefront, then token
        {
            int v = 0, incl = 0;
            if (tid < 256) {
                v = s_hist[tid % KU_NW][tid / KU_NW];
                incl = v;
                for (int o = 1; o < 64; o <<= 1) {
                    const int u = __shfl_up(incl, o);
                    if (lane >= o) incl += u;
                }
                if (lane == 63) s_sum[wave] = incl;
            }
            __syncthreads();
            if (tid < 256) {
                int first = incl - v;
#pragma unroll
                for (int w = 0; w < 3; ++w) first += w < wave ? s_sum[w] : 0;
                s_hist[tid % KU_NW][tid / KU_NW] = first;
                if (tid % KU_NW == 0) s_start[tid / KU_NW] = first;
                if (tid == 255) s_start[KU_B] = first + v;
            }
            __syncthreads();
        }
        if (wave == 0) {
            const int size = lane < KU_B ? s_start[lane + 1] - s_start[lane] : 0, np = (size + KU_PIECE - 1) / KU_PIECE;
            total += size;
            int incl = np;
            for (int o = 1; o < KU_B; o <<= 1) {
                const int u = __shfl_up(incl, o);
                if (lane >= o) incl += u;
            }
            if (lane < KU_B) {
                s_fp[lane] = incl - np;
                s_tot[lane] = total;
                if (lane == KU_B - 1) s_fp[KU_B] = incl;
            }
        }
        for (int e0 = 0; e0 < cnt; e0 += 64) {
            const bool ok = e0 + lane < cnt;
            const int n = ok ? s_ent[wave][e0 + lane] : 0, b = ok ? s_bkt[wave][e0 + lane] : 0;
            unsigned long long peers = __ballot(ok);
#pragma unroll
            for (int q = 1; q < KU_B; q <<= 1) {
                const unsigned long long m = __ballot((b & q) != 0);
                peers &= (b & q) ? m : ~m;
            }
            const int rank = __popcll(peers & lt);
            if (ok) s_tok[s_hist[wave][b] + rank] = n;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (ok && rank == 0) s_hist[wave][b] += __popcll(peers);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        // ---- sums
        more = s_more != 0;
        const int np = s_fp[KU_B];
        for (int r0 = 0; r0 < np; r0 += KU_SLOTS) {
            for (int q = r0 + wave; q < min(np, r0 + KU_SLOTS); q += KU_NW) {
                const int fp = s_fp[lane % KU_B];
                const int b = __popcll(__ballot(lane < KU_B && fp <= q)) - 1;   // (the last of equal ones has the pieces)
                const int row0 = s_start[b] + (q - s_fp[b]) * KU_PIECE;
                double acc[EPL];
                sum_rows<T, D, KU_UB>(Xh, min(KU_PIECE, s_start[b + 1] - row0), [&](int r) { return s_tok[row0 + r]; }, acc);
                if (lane < LPR) {
#pragma unroll
                    for (int e = 0; e < EPL; e += 2)
                        *reinterpret_cast<double2 *>(&s_ps[q - r0][lane * EPL + e]) = make_double2(acc[e], acc[e + 1]);
                }
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < JN; ++i) {
                const int b = 2 * (msub + NSUB * i);
                const int p0 = s_fp[b], p1 = s_fp[b + 1], p2 = s_fp[b + 2];
                for (int p = max(p0, r0); p < min(p1, r0 + KU_SLOTS); ++p) csum[i] += s_ps[p - r0][mk];
                for (int p = max(p1, r0); p < min(p2, r0 + KU_SLOTS); ++p) csum[i] -= s_ps[p - r0][mk];
            }
            __syncthreads();
        }
    }
    if (c0 == 0 && tid == 0) S.flag_cnt[h] = 0;     // the next assign step starts an empty list
#pragma unroll
    for (int i = 0; i < JN; ++i) s_ps[msub + NSUB * i][mk] = csum[i];
    __syncthreads();
    for (int j = wave; j < nc; j += KU_NW) {
        const int joined = s_tot[2 * j], left = s_tot[2 * j + 1];
        // nothing moved: sum, mean and what the next assign step reads of them stay
        if (DELTA && joined + left == 0 && it.t + 1 < a.iters) continue;
        const int n_prev = it.t > 0 ? S.counts[(size_t)h * S.C + c0 + j] : 0, size = (DELTA ? n_prev : 0) + joined - left;
        double sum[EL], s_prev[EL];
#pragma unroll
        for (int e = 0; e < EL; ++e) {
            sum[e] = s_ps[j][lane + 64 * e];
            s_prev[e] = size == 0 && it.t > 0 ? S.csum[((size_t)h * S.C + c0 + j) * D + lane + 64 * e] : 0.0;
        }
        finalize_cluster<BF16, D>(a, S, it, DELTA ? 2 : 1, h, c0 + j, sum, size, s_prev, n_prev);
    }
}

// Whether the assign step of bf16 heads lists the tokens that moved.  The update kernel then reads a few per cent of what the labels of two iterations are; the assign step pays for
// it with a comparison per token, which up to KU_LISTS_N tokens is what is gained (24 heads x 6000, 200 clusters, five iterations: 240
// us by the labels, 247 by lists; 24 x 8000, 500: 349 / 351; 40 x 9000, D = 64, 100: 247 / 241).
//   24 x 16,384, D = 128, 100 / 500 clusters: 339 / 321, 505 / 491      2 x 30,000, 300: 261 / 235      24 x 30,000, 100, Zipf sizes: 520 / 480
// Beyond KU_N tokens, where the labels are too much for every workgroup to read, it is the sorted order that they replace.  A
// workgroup has all rows of its clusters to add, so it takes clusters that are not too large for that:
//   8 x 37,800, 1000 / 2000 clusters: 837 / 730, 1392 / 1222 (Zipf sizes 842 / 758, 1436 / 1297)      8 x 75,600, 4000: 3951 / 3648
//   1 x 118,800, 500, Zipf sizes (not taken): 392 / 513      8 x 37,800, 100 (not taken): 379 / 391
static constexpr int KU_LISTS_SIZE = 64;        // tokens per cluster, beyond KU_N tokens
static bool kmeans_update_direct(int H, int N, int call, int cmin)
{
    return !kmeans_update_small(H, N, call) && N <= KU_N && N <= (long long)KU_SIZE * cmin;
}
static bool kmeans_update_lists(int H, int N, int call, int cmin)
{
    return N > KU_LISTS_N && (kmeans_update_direct(H, N, call, cmin) || (N > KU_N && N <= (long long)KU_LISTS_SIZE * cmin));
}

// Clusters of a workgroup of the update kernel: as many as leave a workgroup per CU over all heads and sides, and no more than a sixteenth
// of the side's (few large clusters: their tokens are shared out over more CUs) unless there are four workgroups per CU without that.
// (With the sixteenth always, many heads of few clusters were a workgroup per cluster, each reading all labels.  Five iterations, sorted / by
// a sixteenth / now, fp32, D = 64: 1000 x 256 in 20 341 / 677 / 240 us, 5000 x 64 in 8 683 / 1173 / 321, 100 x 3000 in 31 253 / 278 / 229; bf16, D = 128:
// 1000 x 256 in 40 566 / 918 / 428, 100 x 3000 in 31 275 / 310 / 255, 200 x 4096 in 16 459 / 461 / 408.)
static int kmeans_update_group(int H, int C, int call)
{
    int g = KU_G;
    while (g > 1 && ((long long)call * H < 256ll * g || (16 * g > C && (long long)H * cdiv(C, g) < 1024))) g >>= 1;
    return g;
}

// ---------------------------------------------------------------- all iterations of a short head, bf16
// grid (H, sides), block 1024: a head of at most KM_TINY_N tokens goes through all its iterations in one workgroup --
// wavefront w holds tokens 64 w .. + 64 as the B operand of the assign step, and centroids, labels, order and the
// sums of the pieces (KM_TINY_SEG rows of one cluster) stay in LDS.  Same labels, order, cluster sums and means as the kernels above:
// near-ties are settled in double precision over every centroid, and the sums of the bf16 rows are exact.
//
// Such a head is bound by launches that depend on each other (four of 4 to 8 us per iteration), here by the chain of short
// phases between barriers, most of all the sums: 12 us per iteration at D = 64 and 32 clusters.  Up to KM_TINY_CD / D clusters, beyond which
// the pieces and means of one workgroup take longer than the launches.  Five iterations in us, the launches / this kernel:
//   1 head x 1024, D = 64, 16 clusters: 104 / 48      2 x 1024, 64, 32: 98 / 59       2 x 1024, 64, 64: 102 / 87
//   128 x 1024, 64, 32: 167 / 68                      2 x 1024, 128, 32: 125 / 101    2 x 1024, 128, 64: 116 / 124 (not taken)
//   2000 x 300, 64, 8: 556 / 262                      one cluster of all tokens, 2 x 1024, 64, 32: 104 / 49
static constexpr int KM_TINY_N = 1024, KM_TINY_CD = 4096, KM_TINY_SEG = 64, KM_TINY_NW = KM_TINY_N / 64;

static size_t kmeans_tiny_lds(int d, int C)
{
    const size_t cp = (size_t)(C + 31) / 32 * 32;
    return (KM_TINY_NW + C) * (size_t)d * sizeof(double) + cp * (d + 8) * sizeof(bf16_t) + cp * sizeof(float) + (C + 1) * sizeof(double) +
           (size_t)KM_TINY_NW * C * sizeof(int32_t) + 2 * (size_t)(C + 1) * sizeof(int32_t) + (3 * (size_t)KM_TINY_N + KM_TINY_NW + C) * sizeof(int32_t);
}

template <int D>
__global__ __launch_bounds__(64 * KM_TINY_NW) void kmeans_tiny_bf16_kernel(KmArgs a)
{
    constexpr int KS = D / 16, ROW = D + 8, EL = D / 64, NW = KM_TINY_NW;
    constexpr int LPR = D / 8, RPI = 64 / LPR;      // lanes per row and rows per load instruction of the sums
    extern __shared__ __align__(16) unsigned char s_raw[];
    __shared__ int32_t s_nflag;
    const KmSide S = blockIdx.y ? a.s[1] : a.s[0];
    const int h = blockIdx.x, N = a.N, C = S.C, CP = (C + 31) & ~31, set = (a.iters - 1) & 1;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, col = lane & 31;
    double *s_ps = reinterpret_cast<double *>(s_raw);                               // [NW + C][D] sums of the pieces
    double *s_cn = s_ps + (NW + C) * D;                                             // [C] ||c||^2
    bf16_t *s_c = reinterpret_cast<bf16_t *>(s_cn + C + (C & 1));                   // [CP][ROW]
    float *s_hcn = reinterpret_cast<float *>(s_c + CP * ROW);                       // [CP] -||c||^2 / 2
    int32_t *s_hist = reinterpret_cast<int32_t *>(s_hcn + CP);                      // [NW][C]
    int32_t *s_off = s_hist + NW * C, *s_fp = s_off + C + 1;                        // [C + 1] first row, first piece
    int32_t *s_lab = s_fp + C + 1, *s_perm = s_lab + KM_TINY_N, *s_flag = s_perm + KM_TINY_N;
    int32_t *s_pc = s_flag + KM_TINY_N;                                             // [NW + C] cluster of a piece
    const bf16_t *Xh = reinterpret_cast<const bf16_t *>(S.X) + (size_t)h * N * D;
    const int n_own = wave * 64 + lane;
    int nbits = 0;
    while ((1 << nbits) < C) ++nbits;

    bf16x8 xb[D == 64 ? 2 : 1][KS];             // lane (col, half): elements 16 s + 8 half .. + 8 of token 64 w + 32 b + col
    float x2[2];                                // ||x||^2
    auto load_x = [&](int b) {
        bf16x8 (&x)[KS] = xb[D == 64 ? b : 0];
        int n = min(N - 1, wave * 64 + 32 * b + col);
        asm volatile("" : "+v"(n));
        const uint4 *src = reinterpret_cast<const uint4 *>(Xh + (size_t)n * D + 8 * half);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const uint4 v = src[2 * s];
            __builtin_memcpy(&x[s], &v, 16);
        }
        float q = 0.f;
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bf16x2_t p2 = {x[s][2 * e], x[s][2 * e + 1]};
                q = __builtin_amdgcn_fdot2_f32_bf16(p2, p2, q, false);
            }
        const KmHalves hx = km_halves(__float_as_uint(q));
        x2[b] = __uint_as_float(hx.lo) + __uint_as_float(hx.hi);
    };
    if (D == 64) { load_x(0); load_x(1); }      // (at D = 128 read again in every iteration: 64 registers)
    for (int e = tid; e < (CP - C) * ROW; e += 64 * NW) s_c[C * ROW + e] = 0;
    for (int j = C + tid; j < CP; j += 64 * NW) s_hcn[j] = KM_PAD_HCN;
    // centroid c[] (element lane + 64 e) of cluster j as the next assign step reads it
    auto put_centroid = [&](int j, const double (&c)[EL]) {
        double n2 = 0.0;
#pragma unroll
        for (int e = 0; e < EL; ++e) {
            const bf16_t b = f64_to_bf16(c[e]);
            s_c[j * ROW + lane + 64 * e] = b;
            const double cr = (double)bf16_to_f32(b), sq = km_wave_sum(cr * cr);
            n2 = e == 0 ? sq : n2 + sq;
        }
        if (lane == 0) {
            s_cn[j] = n2;
            s_hcn[j] = (float)(-0.5 * n2);
        }
    };
    for (int j = wave; j < C; j += NW) {
        double c[EL];
#pragma unroll
        for (int e = 0; e < EL; ++e) c[e] = (double)S.init[((size_t)h * C + j) * D + lane + 64 * e];
        put_centroid(j, c);
    }

#pragma unroll 1
    for (int t = 0; t < a.iters; ++t) {
        if (tid == 0) s_nflag = 0;
        for (int c = lane; c < C; c += 64) s_hist[wave * C + c] = 0;
        __syncthreads();
        // ---- assign: as in kmeans_assign_bf16_kernel
        float cmax2 = 0.f;
        for (int j = lane; j < C; j += 64) cmax2 = fmaxf(cmax2, -2.f * s_hcn[j]);
        for (int o = 32; o > 0; o >>= 1) cmax2 = fmaxf(cmax2, __shfl_xor(cmax2, o));
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            if (D != 64) load_x(b);
            const bf16x8 (&x)[KS] = xb[D == 64 ? b : 0];
            float best = -INFINITY, second = -INFINITY;
            int bbase = 0;
#pragma unroll 1
            for (int rb = 0; rb < CP / 32; ++rb) {
                f32x16 acc;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float4 v = *reinterpret_cast<const float4 *>(&s_hcn[rb * 32 + 8 * g + 4 * half]);
                    acc[4 * g] = v.x; acc[4 * g + 1] = v.y; acc[4 * g + 2] = v.z; acc[4 * g + 3] = v.w;
                }
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    bf16x8 am;
                    const uint4 v = *reinterpret_cast<const uint4 *>(&s_c[(rb * 32 + col) * ROW + 8 * half + 16 * s]);
                    __builtin_memcpy(&am, &v, 16);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(am, x[s], acc, 0, 0, 0);
                }
                const float before = best;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const float key = __uint_as_float((__float_as_uint(acc[i]) & 0xFFFFFFF0u) | (unsigned)i);
                    second = km_med3(best, second, key);
                    best = km_max(best, key);
                }
                bbase = best > before ? rb * 32 : bbase;
            }
            const unsigned kb = __float_as_uint(best);
            const int cown = bbase + 4 * half + (int)(((kb & 12u) << 1) | (kb & 3u));
            const KmHalves hb = km_halves(kb), hs = km_halves(__float_as_uint(second)), hi = km_halves((unsigned)cown);
            const float b0 = __uint_as_float(hb.lo), b1 = __uint_as_float(hb.hi);
            const float T = km_max(b0, b1), U = km_max3(km_min(b0, b1), __uint_as_float(hs.lo), __uint_as_float(hs.hi));
            const int n = wave * 64 + 32 * b + col;
            if (half == 0 && n < N) {
                const int cidx = (b1 > b0) ? (int)hi.hi : (int)hi.lo;
                s_lab[n] = cidx < C ? cidx : 0;
                const float tau = KM_TIE_KEY * fabsf(T) + KM_TIE_ACC * (0.5f * x2[b] + cmax2);
                if (!(T - U > tau)) s_flag[atomicAdd(&s_nflag, 1)] = n;
            }
        }
        __syncthreads();
        // ---- settle: a wavefront per listed token, a centroid per lane, every distance by the same chain of additions
        const int nflag = s_nflag;
        for (int f = wave; f < nflag; f += NW) {
            const int n = s_flag[f];
            const uint4 *xr = reinterpret_cast<const uint4 *>(Xh + (size_t)n * D);
            const uint4 *cr = reinterpret_cast<const uint4 *>(s_c + min(lane, C - 1) * ROW);
            double dot = 0.0;
#pragma unroll 1
            for (int q0 = 0; q0 < D / 8; q0 += 8) {
                uint4 xv[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) xv[q] = xr[q0 + q];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    __builtin_amdgcn_sched_barrier(0);
                    const uint4 cv = cr[q0 + q];
                    const unsigned u[4] = {xv[q].x, xv[q].y, xv[q].z, xv[q].w}, w[4] = {cv.x, cv.y, cv.z, cv.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        dot = fma((double)__uint_as_float(u[e] << 16), (double)__uint_as_float(w[e] << 16), dot);
                        dot = fma((double)__uint_as_float(u[e] & 0xFFFF0000u), (double)__uint_as_float(w[e] & 0xFFFF0000u), dot);
                    }
                }
            }
            double best = INFINITY;
            int bj = 0x7FFFFFFF;
            const double dist = s_cn[min(lane, C - 1)] - 2.0 * dot;
            if (lane < C && dist < best) { best = dist; bj = lane; }
            for (int o = 32; o > 0; o >>= 1) {
                const double ob = __shfl_xor(best, o);
                const int oj = __shfl_xor(bj, o);
                if (ob < best || (ob == best && oj < bj)) { best = ob; bj = oj; }
            }
            if (lane == 0) s_lab[n] = bj < C ? bj : 0;  // (no distance is a finite number: cluster 0)
        }
        if (nflag > 0) __syncthreads();
        // ---- stable counting sort: a wavefront's 64 tokens are one group
        const bool valid = n_own < N;
        const int l = valid ? s_lab[n_own] : 0;
        unsigned long long peers = __ballot(valid);
        for (int b = 0; b < nbits; ++b) {
            const unsigned long long m = __ballot((l >> b) & 1);
            peers &= (l >> b) & 1 ? m : ~m;
        }
        const int rank = __popcll(peers & ((1ull << lane) - 1ull));
        if (valid && rank == 0) s_hist[wave * C + l] = __popcll(peers);
        __syncthreads();
        if (wave == 0) {                        // (C <= 64: one lane per cluster)
            int size = 0, cnt[NW];
#pragma unroll
            for (int w = 0; w < NW; ++w) cnt[w] = lane < C ? s_hist[w * C + lane] : 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                if (lane < C) s_hist[w * C + lane] = size;
                size += cnt[w];
            }
            const int np = (size + KM_TINY_SEG - 1) / KM_TINY_SEG;
            int isz = size, inp = np;
            for (int o = 1; o < 64; o <<= 1) {
                const int us = __shfl_up(isz, o), up = __shfl_up(inp, o);
                if (lane >= o) { isz += us; inp += up; }
            }
            if (lane < C) {
                s_off[lane] = isz - size;
                s_fp[lane] = inp - np;
                for (int p = inp - np; p < inp; ++p) s_pc[p] = lane;
                if (lane == C - 1) { s_off[C] = isz; s_fp[C] = inp; }
            }
        }
        __syncthreads();
        if (valid) s_perm[s_off[l] + s_hist[wave * C + l] + rank] = n_own;
        __syncthreads();
        // ---- sums of the pieces, in double precision
        for (int p = wave; p < s_fp[C]; p += NW) {
            const int c = s_pc[p], r0 = s_off[c] + (p - s_fp[c]) * KM_TINY_SEG, rows = min(KM_TINY_SEG, s_off[c + 1] - r0);
            const int sub = lane / LPR, part = lane % LPR;
            double acc[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] = 0.0;
#pragma unroll 1
            for (int r = 0; r < rows; r += RPI * KM_UB) {
                uint4 v[KM_UB];
#pragma unroll
                for (int u = 0; u < KM_UB; ++u)
                    v[u] = reinterpret_cast<const uint4 *>(Xh + (size_t)s_perm[r0 + min(r + u * RPI + sub, rows - 1)] * D)[part];
#pragma unroll
                for (int u = 0; u < KM_UB; ++u) {
                    if (r + u * RPI + sub >= rows) continue;
                    const unsigned w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        acc[2 * q] += (double)__uint_as_float(w[q] << 16);
                        acc[2 * q + 1] += (double)__uint_as_float(w[q] & 0xFFFF0000u);
                    }
                }
            }
            // lanes with the same `part` hold the same columns
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if (LPR == 8) acc[e] += km_dpp<0x128>(acc[e]);      // row_ror:8
                acc[e] = km_sum_xor32(km_sum_xor16(acc[e]));
            }
            if (lane < LPR) {
#pragma unroll
                for (int e = 0; e < 8; ++e) s_ps[p * D + lane * 8 + e] = acc[e];
            }
        }
        __syncthreads();
        // ---- means: one wavefront per cluster (always the same one: what an empty cluster keeps is read back by its writer)
        for (int j = wave; j < C; j += NW) {
            const int cnt = s_off[j + 1] - s_off[j];
            const size_t idx = ((size_t)h * C + j) * D + lane;
            double c[EL];
#pragma unroll
            for (int e = 0; e < EL; ++e) {
                double sum = 0.0;
                for (int p = s_fp[j]; p < s_fp[j + 1]; ++p) sum += s_ps[p * D + lane + 64 * e];
                c[e] = cnt > 0 ? sum / (double)cnt : t == 0 ? (double)S.init[idx + 64 * e] : S.cd[idx + 64 * e];
                S.cd[idx + 64 * e] = c[e];
                if (t + 1 == a.iters) S.centroids[idx + 64 * e] = (float)c[e];
            }
            put_centroid(j, c);
        }
    }
    // (the last iteration's labels, offsets and order are complete since the barrier behind the scatter)
    if (n_own < N) {
        S.labels[(size_t)h * N + n_own] = s_lab[n_own];
        KM_SEL(S.perm, set)[(size_t)h * N + n_own] = s_perm[n_own];
    }
    for (int c = tid; c <= C; c += 64 * NW) KM_SEL(S.offsets, set)[(size_t)h * (C + 1) + c] = s_off[c];
    for (int c = tid; c < C; c += 64 * NW) S.counts[(size_t)h * C + c] = s_off[c + 1] - s_off[c];
}

__global__ void kmeans_zero_kernel(float *p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.f;
}

// ---------------------------------------------------------------- host side
static void kmeans_carve_side(Carver &c, KmSide &k, int H, int N, int d, int C)
{
    k.C = C;
    k.max_pieces = cdiv(N, KM_SEG) + C;
    k.cb = c.take<bf16_t>((size_t)H * C * d);
    k.cbT = c.take<bf16_t>((size_t)H * C * d);          // right behind cb, so the two hold H C d floats
    k.ct = reinterpret_cast<float *>(k.cb);
    k.hcn = c.take<float>((size_t)H * C);
    k.cn64 = c.take<double>((size_t)H * C);
    k.cd = c.take<double>((size_t)H * C * d);
    k.csum = c.take<double>((size_t)H * C * d);
    for (int s = 0; s < 2; ++s) {
        k.offsets[s] = c.take<int32_t>((size_t)H * (C + 1));
        k.perm[s] = c.take<int32_t>((size_t)H * N);
        k.first_piece[s] = c.take<int32_t>((size_t)H * (C + 1));
        k.n_pieces[s] = c.take<int32_t>((size_t)H);
        k.pieces[s] = c.take<int4>((size_t)H * k.max_pieces);
        k.psum[s] = c.take<double>((size_t)H * k.max_pieces * d);
        k.moved[s] = c.take<int32_t>((size_t)H * k.max_pieces);
    }
    k.labels_alt = c.take<int32_t>((size_t)H * N);
    k.flag_cnt = c.take<int32_t>((size_t)H);
    k.mv_list = reinterpret_cast<unsigned *>(k.perm[1]);        // (the memory, whatever perm[1] points to later)
    k.mv_cnt = reinterpret_cast<int32_t *>(k.pieces[1]);        // 16 bytes per 256 tokens and more
    k.flag_list = c.take<int32_t>((size_t)H * N);
    k.best = c.take<float>(C > KM_CMAX ? (size_t)H * N : 0);
    k.second = c.take<float>(C > KM_CMAX ? (size_t)H * N : 0);
    k.hist = reinterpret_cast<int32_t *>(c.take<char>(permute_ws_bytes(H, N, C)));
}

size_t kmeans_ws_bytes(int dtype, int H, int N, int d, int C)
{
    (void)dtype;
    Carver c(nullptr);
    KmSide k;
    kmeans_carve_side(c, k, H, N, d, C);
    return c.used;
}

size_t kmeans_pair_ws_bytes(int dtype, int H, int N, int d, int Cq, int Ck)
{
    return kmeans_ws_bytes(dtype, H, N, d, Cq) + kmeans_ws_bytes(dtype, H, N, d, Ck);
}

// dynamic LDS of the bf16 assign kernel
template <int D> static constexpr size_t kmeans_assign_lds()
{
    return (size_t)KM_CMAX * (D + 8) * sizeof(bf16_t) + KM_CMAX * sizeof(float);
}

int kmeans_prepare(int dtype, int d)
{
    if (dtype != SVG2_BF16) return SVG2_OK;
    const void *tiny = d == 128 ? reinterpret_cast<const void *>(kmeans_tiny_bf16_kernel<128>)
                                : reinterpret_cast<const void *>(kmeans_tiny_bf16_kernel<64>);
    SVG2_TRY(set_dynamic_lds(tiny, kmeans_tiny_lds(d, KM_TINY_CD / d)));
    if (d == 128) {
        SVG2_TRY(set_dynamic_lds(reinterpret_cast<const void *>(kmeans_assign_bf16_kernel<128, true>), kmeans_assign_lds<128>()));
        SVG2_TRY(set_dynamic_lds(reinterpret_cast<const void *>(kmeans_assign_bf16_kernel<128, false>), kmeans_assign_lds<128>()));
    } else {
        SVG2_TRY(set_dynamic_lds(reinterpret_cast<const void *>(kmeans_assign_bf16_kernel<64, true>), kmeans_assign_lds<64>()));
        SVG2_TRY(set_dynamic_lds(reinterpret_cast<const void *>(kmeans_assign_bf16_kernel<64, false>), kmeans_assign_lds<64>()));
    }
    return SVG2_OK;
}

// number of compute units of the current device (the bf16 assign kernel runs one workgroup on each)
int device_cu_count(int *ncu)
{
    static std::atomic<int> known[64];
    int dev = -1;
    SVG2_HIP_CHECK(hipGetDevice(&dev));
    int n = (dev >= 0 && dev < 64) ? known[dev].load() : 0;
    if (n <= 0) {
        SVG2_HIP_CHECK(hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev));
        SVG2_REQUIRE(n > 0, SVG2_HIP_ERROR, "device %d reports %d compute units", dev, n);
        if (dev >= 0 && dev < 64) known[dev].store(n);
    }
    *ncu = n;
    return SVG2_OK;
}

// Wavefronts that share a token block of the fp32 assign step: every one of them loads (and splits) the tokens, so a share has at
// least 8 row blocks from 512 wavefronts on, and from 4096 wavefronts on none is shared further; as few as one row block with fewer
// (k-means of five iterations with one, two, four wavefronts, us: 4 x 9601 in 500 288, 275, 290; in 100 192, 203, 201; 6 x 12,000 in
// 1000 653, 602, 625; 24 x 16,384 in 500 1327, 1489, 1910; 3 x 3000 in 300 131, 106, 118; 1 x 12,000 in 1000 300, 211, 206, all D = 128;
// 1 x 4096 in 200, D = 64 84, 75, 69).  Without splitting a share has at least four row blocks where the token blocks alone are enough
// for two wavefronts per SIMD, and as few as one otherwise.  Splitting pays from one token block of 128 elements per SIMD
// on (fp32 instruction / split, D = 128: 4 x 9601 in 100 224 / 195, in 500 406 / 304, 6 x 12,000 in 1000 1021 / 659; below: 1 x 12,000 in 1000 270 / 256
// and 291 / 397 with one token in twenty equal, 1 x 9601 in 500 185 / 193, 4 x 4000 in 300 147 / 150; D = 64: 6 x 12,000 in 1000 583 / 479, 24 x 16,384
// in 500 1443 / 870; below: 4 x 9601 in 500 263 / 246 and 268 / 363, 1 x 12,000 in 1000 186 / 251).
// The grid has 64 KF_NW threads per 32 (KF_NW / nc) tokens of a head, 2 nc N, and one grid dimension takes less than 2^32: 2 N with one
// wavefront per block, and what is shared is 4096 wavefronts at most.
static constexpr bool kmeans_f32_split(int H, int N, int C, int d)
{
    return C > KF_SPLIT && H * (((long long)N + 31) / 32) * d >= KF_SPLIT_BLOCKS * 128;
}
static constexpr int kmeans_f32_share(int H, int N, int C, int d)
{
    const int nrb = (C + 31) / 32;
    const long long blocks = H * (((long long)N + 31) / 32);
    int nc = 1;
    while (nc < KF_NW && 2 * nc <= nrb &&
           (!kmeans_f32_split(H, N, C, d) ? nrb > 4 * nc || blocks * nc < 2048 : blocks * nc < 512 || (nrb >= 16 * nc && blocks * nc < 4096)))
        nc *= 2;
    return nc;
}
static_assert(kmeans_f32_share(1, 1000, 4096, 64) == 4 && kmeans_f32_share(1, 32767, 4096, 128) == 4 && kmeans_f32_share(1, 32768, 4096, 128) == 4 &&
              kmeans_f32_share(1, 65537, 4096, 128) == 2 && kmeans_f32_share(1, 131072, 4096, 128) == 1 && kmeans_f32_share(1, 131072, 64, 64) == 1 &&
              kmeans_f32_share(1, 1 << 30, 4096, 64) == 1, "the grid of the fp32 assign step stays below 2^32 threads");

template <typename T, int D, bool BF16>
static int kmeans_run(KmArgs a, hipStream_t st)
{
    const int H = a.H, N = a.N, iters = a.iters, ns = a.nsides;
    int ncu = 0;
    if (BF16) SVG2_TRY(device_cu_count(&ncu));
    int call = 0, cmin = a.s[0].C, pmax = 0, ncmax = 1;
    bool any_obj = false, any_few = false;
    for (int s = 0; s < ns; ++s) {
        call += a.s[s].C;
        cmin = std::min(cmin, a.s[s].C);
    }
    int ngroups = 0;
    for (int s = 0; s < ns; ++s) {
        a.gc[s] = kmeans_update_group(H, a.s[s].C, call);
        ngroups += cdiv(a.s[s].C, a.gc[s]);
        any_few |= !BF16 && kmeans_f32_few(H, N, a.s[s].C);
        a.split[s] = kmeans_f32_split(H, N, a.s[s].C, D);
        a.nc[s] = kmeans_f32_share(H, N, a.s[s].C, D);
        ncmax = std::max(ncmax, a.nc[s]);
        pmax = std::max(pmax, a.s[s].max_pieces);
        if (a.s[s].objective) {
            any_obj = true;
            hipLaunchKernelGGL(kmeans_zero_kernel, dim3(cdiv(H * iters, 256)), dim3(256), 0, st, a.s[s].objective, H * iters);
        }
    }
    if constexpr (BF16) {
        int cmax = 0;
        for (int s = 0; s < ns; ++s) cmax = std::max(cmax, a.s[s].C);
        if (N <= KM_TINY_N && cmax * D <= KM_TINY_CD && !any_obj) {
            ProfileSpan sp(SVG2_K_KMEANS_ASSIGN, st);
            hipLaunchKernelGGL((kmeans_tiny_bf16_kernel<D>), dim3(H, ns), dim3(64 * KM_TINY_NW), kmeans_tiny_lds(D, cmax), st, a);
            return SVG2_OK;
        }
    }
    const dim3 fin_grid(cdiv(call, KM_FIN_NW), H);
    const bool small = kmeans_update_small(H, N, call), direct = kmeans_update_direct(H, N, call, cmin);
    const bool lists = BF16 && kmeans_update_lists(H, N, call, cmin);
    {
        ProfileSpan sp(SVG2_K_KMEANS_FINALIZE, st);
        hipLaunchKernelGGL((kmeans_finalize_kernel<BF16, D>), fin_grid, dim3(64 * KM_FIN_NW), 0, st, a, KmIter{}, 0);
    }
    for (int t = 0; t < iters; ++t) {
        // Update step: the first iteration, and every KM_FULL_EVERY-th after that, sums every cluster afresh; the
        // others only move the tokens whose label changed (a quarter in the second iteration, a few per cent from
        // the third on) between the cluster sums, which reads a fraction of X.
        const bool full = t % KM_FULL_EVERY == 0;
        // sums and means straight from the labels, or by the label-sorted order (in the second iteration of few large clusters, where
        // the first one has left its order)
        const bool by_order = t == 1 && N > KU_FULL_N && N > (long long)KU_SECOND_SIZE * cmin;
        const bool straight = small || (full ? direct && N <= KU_FULL_N : (direct || lists) && !by_order);
        a.lists = lists && !by_order;
        KmIter it;
        it.t = t;
        it.set = t & 1;
        for (int s = 0; s < 2; ++s) {
            // the labels of iteration t go to the caller's buffer when iters - 1 - t is even, else to the scratch
            // buffer: the last iteration lands in the caller's buffer, the previous labels are always the other one
            const bool alt = (iters - 1 - t) & 1;
            it.lab[s] = alt ? a.s[s].labels_alt : a.s[s].labels;
            it.lab_prev[s] = alt ? a.s[s].labels : a.s[s].labels_alt;
        }
        if (BF16) {
            const long long nb_all = (long long)H * cdiv(N, KM_WG_TOKENS);
            // a block of one side per workgroup while there are CUs enough for that, else a share of both sides
            const dim3 grid((unsigned)(ns * nb_all <= ncu ? ns * nb_all : std::min<long long>(ncu, nb_all)));
            auto kern = any_obj ? kmeans_assign_bf16_kernel<D, true> : kmeans_assign_bf16_kernel<D, false>;
            {
                ProfileSpan sp(SVG2_K_KMEANS_ASSIGN, st);
                hipLaunchKernelGGL(kern, grid, dim3(64 * KM_NW), kmeans_assign_lds<D>(), st, a, it);
            }
            {
                ProfileSpan sp(SVG2_K_KMEANS_SETTLE, st);
                hipLaunchKernelGGL((kmeans_settle_kernel<D>), dim3(std::max(KM_SETTLE_MIN, std::min(KM_SETTLE_BLOCKS, KM_SETTLE_WG / (H * ns))), H * ns), dim3(256),
                                   0, st, a, it);
            }
        } else {
            ProfileSpan sp(SVG2_K_KMEANS_ASSIGN, st);
            auto kern = any_obj ? kmeans_assign_f32_kernel<D, true> : kmeans_assign_f32_kernel<D, false>;
            const dim3 grid(cdiv(N, 32 * (KF_NW / ncmax)), H, ns);
            if (!any_few) {
                hipLaunchKernelGGL(kern, grid, dim3(64 * KF_NW), 0, st, a, it);
            } else {
                auto few = any_obj ? kmeans_assign_f32_few_kernel<D, true> : kmeans_assign_f32_few_kernel<D, false>;
                for (int s = 0; s < ns; ++s) {
                    if (kmeans_f32_few(H, N, a.s[s].C)) {
                        hipLaunchKernelGGL(few, dim3(cdiv(N, 128), H), dim3(128), 0, st, a, it, s);
                        continue;
                    }
                    KmArgs one = a;                     // that side alone
                    KmIter one_it = it;
                    one.s[0] = a.s[s]; one.nc[0] = a.nc[s]; one.split[0] = a.split[s]; one_it.lab[0] = it.lab[s];
                    hipLaunchKernelGGL(kern, dim3(grid.x, H), dim3(64 * KF_NW), 0, st, one, one_it);
                }
            }
        }
        // label-sorted order of the tokens and its pieces, then the segmented sum over it; or sums and means straight from the labels
        SortArgs sa = {};
        for (int s = 0; s < ns; ++s) {
            const KmSide &k = a.s[s];
            sa.s[s].labels = it.lab[s];
            sa.s[s].C = k.C;
            sa.s[s].hist = k.hist;
            sa.s[s].offsets = k.offsets[it.set];
            sa.s[s].perm = k.perm[it.set];
            sa.s[s].inv_perm = nullptr;
            sa.s[s].pieces = straight ? nullptr : k.pieces[it.set];      // (straight: the order is handed on, not read here)
            sa.s[s].first_piece = k.first_piece[it.set];
            sa.s[s].n_pieces = k.n_pieces[it.set];
            sa.s[s].max_pieces = k.max_pieces;
            sa.s[s].seg = KM_SEG;
        }
        if (!straight || (t + 1 == iters && a.want_order)) {
            ProfileSpan sp(SVG2_K_KMEANS_SORT, st);
            SVG2_TRY(sort_launch(sa, ns, H, N, st));
        }
        if (straight) {
            ProfileSpan sp(full ? SVG2_K_KMEANS_SEGSUM_FULL : SVG2_K_KMEANS_SEGSUM_DELTA, st);
            if (small && N <= KM_SMALL_N4)
                hipLaunchKernelGGL((kmeans_update_small_kernel<T, D, BF16, 4>), dim3(call, H), dim3(256), 0, st, a, it, full ? 1 : 2);
            else if (small)
                hipLaunchKernelGGL((kmeans_update_small_kernel<T, D, BF16, 16>), dim3(call, H), dim3(1024), 0, st, a, it, full ? 1 : 2);
            else if (full)
                hipLaunchKernelGGL((kmeans_update_kernel<T, D, BF16, KU_ALL>), dim3(ngroups, H), dim3(64 * KU_NW), 0, st, a, it);
            else if (a.lists)
                hipLaunchKernelGGL((kmeans_update_kernel<T, D, BF16, BF16 ? KU_LISTS : KU_LABELS>), dim3(ngroups, H), dim3(64 * KU_NW), 0, st, a, it);
            else
                hipLaunchKernelGGL((kmeans_update_kernel<T, D, BF16, KU_LABELS>), dim3(ngroups, H), dim3(64 * KU_NW), 0, st, a, it);
            continue;
        }
        if (full) {
            ProfileSpan sp(SVG2_K_KMEANS_SEGSUM_FULL, st);
            hipLaunchKernelGGL((kmeans_segsum_kernel<T, D, false>), dim3(cdiv(pmax, 4), H, ns), dim3(256), 0, st, a, it);
        } else {
            ProfileSpan sp(SVG2_K_KMEANS_SEGSUM_DELTA, st);
            hipLaunchKernelGGL((kmeans_segsum_kernel<T, D, true>), dim3(cdiv(pmax, 4), H, 2 * ns), dim3(256), 0, st, a, it);
        }
        {
            ProfileSpan sp(SVG2_K_KMEANS_FINALIZE, st);
            hipLaunchKernelGGL((kmeans_finalize_kernel<BF16, D>), fin_grid, dim3(64 * KM_FIN_NW), 0, st, a, it,
                               full ? 1 : 2);
        }
    }
    return SVG2_OK;
}

static int kmeans_dispatch(const KmArgs &a, int dtype, int d, hipStream_t st)
{
    int rc;
    if (dtype == SVG2_BF16) rc = d == 128 ? kmeans_run<bf16_t, 128, true>(a, st) : kmeans_run<bf16_t, 64, true>(a, st);
    else rc = d == 128 ? kmeans_run<float, 128, false>(a, st) : kmeans_run<float, 64, false>(a, st);
    if (rc != SVG2_OK) return rc;
    SVG2_HIP_CHECK(hipGetLastError());
    return SVG2_OK;
}

static void kmeans_fill_side(KmSide &k, const void *X, const float *init, float *centroids, int32_t *labels,
                             int32_t *counts, float *objective)
{
    k.X = X;
    k.init = init;
    k.centroids = centroids;
    k.labels = labels;
    k.counts = counts;
    k.objective = objective;
}

int kmeans_launch(const void *X, int dtype, int H, int N, int d, int C, int iters, const float *init,
                  float *centroids, int32_t *labels, int32_t *counts, float *objective, void *ws, hipStream_t st)
{
    KmArgs a = {};
    a.nsides = 1; a.H = H; a.N = N; a.iters = iters;
    Carver c(ws);
    kmeans_carve_side(c, a.s[0], H, N, d, C);
    kmeans_fill_side(a.s[0], X, init, centroids, labels, counts, objective);
    a.s[1] = a.s[0];
    return kmeans_dispatch(a, dtype, d, st);
}

int kmeans_pair_launch(const void *Q, const void *K, int dtype, int H, int N, int d, int Cq, int Ck, int iters,
                       float *cq_inout, float *ck_inout, int32_t *labels_q, int32_t *labels_k, int32_t *counts_q,
                       int32_t *counts_k, int32_t *offsets_q, int32_t *offsets_k, int32_t *perm_q, int32_t *perm_k,
                       void *ws, hipStream_t st)
{
    KmArgs a = {};
    a.nsides = 2; a.H = H; a.N = N; a.iters = iters;
    Carver c(ws);
    kmeans_carve_side(c, a.s[0], H, N, d, Cq);
    kmeans_carve_side(c, a.s[1], H, N, d, Ck);
    kmeans_fill_side(a.s[0], Q, cq_inout, cq_inout, labels_q, counts_q, nullptr);
    kmeans_fill_side(a.s[1], K, ck_inout, ck_inout, labels_k, counts_k, nullptr);
    // the set of the last iteration is the caller's
    const int last = (iters - 1) & 1;
    a.s[0].offsets[last] = offsets_q;
    a.s[0].perm[last] = perm_q;
    a.s[1].offsets[last] = offsets_k;
    a.s[1].perm[last] = perm_k;
    a.want_order = true;
    return kmeans_dispatch(a, dtype, d, st);
}

}  // namespace svg2
