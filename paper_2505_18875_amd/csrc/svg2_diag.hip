// Two pieces around the layer path that the paper uses but that are not on the per-step hot path:
//
//   attention recall (Section 3.1)   the share of a query's true attention mass that its
//                                    selected keys capture.  With lse_sel the log-sum-exp of the
//                                    scores over the selected keys (svg2_sparse_attn's lse) and
//                                    lse_all the one over all keys (the dense special case),
//                                    recall = exp(lse_sel - lse_all).
//   k-means++ seeding (Section 4.3)  the initialisation an un-cached k-means starts from: the
//                                    first centre is a given token, every further centre is drawn
//                                    with probability D2 / sum(D2), D2 = squared distance to the
//                                    nearest centre so far.  The uniform random numbers are an
//                                    input, so the draw is reproducible and can be checked.  All
//                                    arithmetic is fp64 (the draw compares a running sum of D2
//                                    with a threshold; fp32 would move the boundaries).
#include <algorithm>

#include "svg2_common.h"

namespace svg2 {

static constexpr int DG_BLOCK = 1024;       // tokens per workgroup in the recall kernel (256 threads x 4)

// ---------------------------------------------------------------- recall
// grid (nblk, H), block 256
__global__ __launch_bounds__(256) void recall_rows_kernel(const float *__restrict__ lse_sel,
                                                          const float *__restrict__ lse_all, int N, int nblk,
                                                          float *__restrict__ recall, float *__restrict__ partial)
{
    __shared__ float s_red[256];
    const int h = blockIdx.y, tid = threadIdx.x;
    float acc = 0.f;
    for (int k = 0; k < 4; ++k) {
        const int n = blockIdx.x * DG_BLOCK + k * 256 + tid;
        if (n < N) {
            const float a = lse_sel[(size_t)h * N + n], b = lse_all[(size_t)h * N + n];
            const float r = (a == -INFINITY) ? 0.f : expf(a - b);
            if (recall) recall[(size_t)h * N + n] = r;
            acc += r;
        }
    }
    s_red[tid] = acc;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {         // fixed order: reproducible
        if (tid < o) s_red[tid] += s_red[tid + o];
        __syncthreads();
    }
    if (tid == 0) partial[(size_t)h * nblk + blockIdx.x] = s_red[0];
}

// grid (H), block 64
__global__ void recall_mean_kernel(const float *__restrict__ partial, int N, int nblk, float *__restrict__ mean)
{
    const int h = blockIdx.x;
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int b = 0; b < nblk; ++b) s += (double)partial[(size_t)h * nblk + b];
        mean[h] = (float)(s / (double)N);
    }
}

size_t recall_ws_bytes(int H, int N) { return align256((size_t)H * cdiv(N, DG_BLOCK) * sizeof(float)); }

int recall_launch(const float *lse_sel, const float *lse_all, int H, int N, float *recall, float *recall_mean,
                  void *ws, hipStream_t st)
{
    const int nblk = cdiv(N, DG_BLOCK);
    float *partial = static_cast<float *>(ws);
    hipLaunchKernelGGL(recall_rows_kernel, dim3(nblk, H), dim3(256), 0, st, lse_sel, lse_all, N, nblk, recall, partial);
    hipLaunchKernelGGL(recall_mean_kernel, dim3(H), dim3(64), 0, st, partial, N, nblk, recall_mean);
    SVG2_HIP_CHECK(hipGetLastError());
    return SVG2_OK;
}

// ---------------------------------------------------------------- k-means++
// A draw is a chain: find the token (from the sums of D2 that the draw before it left), then measure the tokens against
// it.  One launch does both: every workgroup finds the token by itself -- a few hundred block sums and one block of D2,
// read by all of them -- and then updates its own block, so no second kernel waits for the first.  D2, the block
// sums and the change flags alternate between two buffers, because a block that is being updated may still be read
// by the workgroups that look for the token; a chunk of D2 is written only where it differs from what the buffer
// holds (it changed in this draw or in the last one).
//
// Most tokens are not nearer to the new centre than to an older one, and a 4-bit copy of the tokens is enough to see
// it: with x^ = s_x q_x the copy (q_x 4-bit integers, one scale per token), r_x >= ||x - x^||, and c^, r_c the
// same for the centre in 8 bits, ||x - c|| >= ||x^ - c^|| - r_x - r_c, where ||x^ - c^||^2 takes one integer dot
// product (v_dot8_i32_i4, twice for the two halves of c's digits).  Only the tokens whose bound is below D2 are
// read and measured, in double precision; the others are exactly those that a measurement would have left as they are
// (margins for the rounding of the bound are in the constants), so the draws do not depend on it.  A token costs D / 2
// + 20 bytes per draw instead of its row.
//
// What bounds a draw now is the chain: launch, two round trips to find the token, one for its row, one or two for the
// rows that are measured.  24 heads of 16,384 tokens (d = 128, bf16, 64 components, 500 draws): 13 us per draw against
// 101 us with two kernels and every row read (6.46 / 50.6 ms in all).  Of the 13 us about 3 are the launch, 3 the
// bound over all tokens (28 MB, which the L2s of the 8 XCDs keep between the draws; read from memory it would be 4), 3
// the search, 4 the measuring.  The step kernel is held to 64 registers so that six workgroups of five wavefronts fit
// a CU: with two more rows in flight per group it spills (11.3 ms), with fewer workgroups resident it takes 6.7 ms.
static constexpr int KPP_CHUNK = 256;       // tokens a workgroup handles at a time, one per thread
static constexpr int KPP_TARGET_WGS = 1536; // workgroups of a launch: six per CU, all resident at once

template <int CTRL> __device__ __forceinline__ float dpp_f32(float v)
{
    return __uint_as_float(__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), CTRL, 0xF, 0xF, false));
}
template <int CTRL> __device__ __forceinline__ double dpp_f64(double v)
{
    const unsigned long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, false);
    return __longlong_as_double(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}
// over groups of LPT = 8 or 16 lanes, result in every lane: quad_perm [1,0,3,2] and [2,3,0,1], row_half_mirror, row_mirror
template <int LPT> __device__ __forceinline__ double group_sum(double v)
{
    v += dpp_f64<0xB1>(v);
    v += dpp_f64<0x4E>(v);
    v += dpp_f64<0x141>(v);
    if (LPT == 16) v += dpp_f64<0x140>(v);
    return v;
}
template <int LPT> __device__ __forceinline__ float group_sum(float v)
{
    v += dpp_f32<0xB1>(v);
    v += dpp_f32<0x4E>(v);
    v += dpp_f32<0x141>(v);
    if (LPT == 16) v += dpp_f32<0x140>(v);
    return v;
}
template <int LPT> __device__ __forceinline__ float group_max(float v)
{
    v = fmaxf(v, dpp_f32<0xB1>(v));
    v = fmaxf(v, dpp_f32<0x4E>(v));
    v = fmaxf(v, dpp_f32<0x141>(v));
    if (LPT == 16) v = fmaxf(v, dpp_f32<0x140>(v));
    return v;
}

// 8 consecutive elements: as loaded (16-byte loads), and as floats
template <typename T> struct Raw8 { uint4 w[sizeof(T) / 2]; };
template <typename T> __device__ __forceinline__ Raw8<T> load_raw(const T *p)
{
    Raw8<T> r;
#pragma unroll
    for (int i = 0; i < (int)sizeof(T) / 2; ++i) r.w[i] = reinterpret_cast<const uint4 *>(p)[i];
    return r;
}
__device__ __forceinline__ void to_floats(const Raw8<bf16_t> &r, float (&out)[8])
{
    const unsigned w[4] = {r.w[0].x, r.w[0].y, r.w[0].z, r.w[0].w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        out[2 * q] = __uint_as_float(w[q] << 16);
        out[2 * q + 1] = __uint_as_float(w[q] & 0xFFFF0000u);
    }
}
__device__ __forceinline__ void to_floats(const Raw8<float> &r, float (&out)[8])
{
    __builtin_memcpy(out, r.w, 32);
}
template <typename T> __device__ __forceinline__ void load_8(const T *p, float (&out)[8]) { to_floats(load_raw(p), out); }

// smallest bf16 number that is not below v (v >= 0)
__device__ __forceinline__ unsigned bf16_up(float v) { return (__float_as_uint(v) + 0xFFFFu) >> 16; }
__device__ __forceinline__ float bf16_lo(unsigned w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(unsigned w) { return __uint_as_float(w & 0xFFFF0000u); }

// A row v ~ scale * q, q integers in -MAXQ .. MAXQ: what the bound needs besides the digits.
struct KppRow {
    float scale, r;     // r >= ||v - scale q||; both are bf16 numbers
    int q2;             // sum of q^2
};

// Digits of the 8 elements of a lane and the row's KppRow (in every lane of the group)
template <int LPT, int MAXQ> __device__ __forceinline__ KppRow kpp_digits(const float (&x)[8], int (&q)[8])
{
    float m = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) m = fmaxf(m, fabsf(x[j]));
    KppRow row;
    row.scale = bf16_lo(bf16_up(group_max<LPT>(m) * (1.0f / MAXQ)));
    const float inv = row.scale > 0.f ? 1.0f / row.scale : 0.f;
    float e2 = 0.f, q2 = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        q[j] = max(-MAXQ, min(MAXQ, (int)rintf(x[j] * inv)));
        const float e = fmaf(-row.scale, (float)q[j], x[j]);
        e2 = fmaf(e, e, e2);
        q2 += (float)(q[j] * q[j]);
    }
    q2 = group_sum<LPT>(q2);                    // at most 128 * 119^2: exact
    e2 = group_sum<LPT>(e2);
    row.q2 = (int)q2;
    // the error of e (2^-24 |x| per element) and of the sums is far inside these margins
    row.r = bf16_lo(bf16_up(1.0001f * sqrtf(e2) + 1e-6f * sqrtf(row.scale * row.scale * q2 + e2)));
    return row;
}
__device__ __forceinline__ unsigned pack_nibbles(const int (&q)[8])
{
    unsigned w = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) w |= (unsigned)(q[j] & 15) << (4 * j);
    return w;
}

struct KppBufs {
    double *d2[2], *csum[2];    // [H,N]; [H,nch] sums of D2 over the chunks
    int32_t *chg[2];            // [H,nch] the chunk's D2 changed in the draw that wrote the flag
    uint4 *dig;                 // [H,D/32,N] 4-bit digits: 16-byte piece p of consecutive tokens is contiguous
    uint2 *row;                 // [H,N] scale and r (bf16), sum of q^2 (16 bits) and D2 rounded up (bf16)
    int32_t *picked;            // [H,C]
    int nch, cpw;               // chunks per head, chunks per workgroup
    // kpp_loop_kernel
    unsigned long long *rec[2]; // [H,nch,2] the sum of a chunk's D2: high half and number of draws so far, low half and the same
    int32_t *fail;              // [H] a workgroup has given up waiting
};

// What the workgroups of a head exchange inside a launch (D2, the records) goes through relaxed atomics at device scope: these are
// coherent over the L2s of the XCDs, location by location.  Order between locations: a wavefront waits for its stores
// (vmcnt) in front of the barrier behind which a record is written, and reads on only once it has seen the record.
__device__ __forceinline__ double kpp_get(const double *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void kpp_put(double *p, double v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void kpp_put_rec(unsigned long long *r, double sum, unsigned draws)
{
    const unsigned long long b = __double_as_longlong(sum);
    __hip_atomic_store(r, (b & 0xFFFFFFFF00000000ull) | draws, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(r + 1, (b << 32) | draws, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// sum over the first 256 threads, in every thread (fixed order)
__device__ __forceinline__ double block_sum_256(double v, double *s_w)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    __syncthreads();
    if ((threadIdx.x & 63) == 0 && threadIdx.x < 256) s_w[threadIdx.x >> 6] = v;
    __syncthreads();
    return ((s_w[0] + s_w[1]) + s_w[2]) + s_w[3];
}

// First draw: token floor(u N); every token's D2 against it and its digits.  grid (workgroups, H), block 256.
template <typename T, int D>
__global__ __launch_bounds__(256) void kpp_first_kernel(const T *__restrict__ X, const double *__restrict__ u, KppBufs w,
                                                        int N, int C, float *__restrict__ centroids, bool again)
{
    if (again && !w.fail[blockIdx.y]) return;
    constexpr int LPT = D / 8, G = 256 / LPT, UB = 4;       // lanes per token, tokens per pass, passes in flight
    __shared__ double s_w[4];
    const int h = blockIdx.y, tid = threadIdx.x, grp = tid / LPT, part = tid % LPT;
    const T *Xh = X + (size_t)h * N * D;
    const int pick = max(0, min(N - 1, (int)floor(u[(size_t)h * C] * (double)N)));
    float c[8];
    load_8(Xh + (size_t)pick * D + part * 8, c);
    if (blockIdx.x == 0 && grp == 0) {
        if (part == 0) {
            w.picked[(size_t)h * C] = pick;
            if (!again) w.fail[h] = 0;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) centroids[(size_t)h * C * D + part * 8 + j] = c[j];
    }
    if (C == 1) return;
    for (int ch = (int)blockIdx.x * w.cpw; ch < min(w.nch, ((int)blockIdx.x + 1) * w.cpw); ++ch) {
        const int n_lo = ch * KPP_CHUNK, n_hi = min(N, n_lo + KPP_CHUNK);
        double acc = 0.0;
        for (int n0 = n_lo; n0 < n_hi; n0 += G * UB) {
            float x[UB][8];
#pragma unroll
            for (int b = 0; b < UB; ++b) load_8(Xh + (size_t)min(n_hi - 1, n0 + b * G + grp) * D + part * 8, x[b]);
#pragma unroll
            for (int b = 0; b < UB; ++b) {
                const int n = n0 + b * G + grp;
                double a = 0.0;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const double t = (double)x[b][j] - (double)c[j];
                    a = fma(t, t, a);
                }
                a = group_sum<LPT>(a);
                int q[8];
                const KppRow row = kpp_digits<LPT, 7>(x[b], q);
                if (n < n_hi) {
                    if (!(a < INFINITY)) a = INFINITY;      // (a distance that is not a number never lowers D2)
                    reinterpret_cast<unsigned *>(w.dig + ((size_t)h * (D / 32) + part / 4) * N + n)[part % 4] = pack_nibbles(q);
                    if (part == 0) {
                        w.d2[0][(size_t)h * N + n] = a;
                        w.row[(size_t)h * N + n] = make_uint2((__float_as_uint(row.scale) >> 16) | __float_as_uint(row.r),
                                                              (unsigned)row.q2 | (bf16_up((float)a) << 16));
                        acc += a;
                    }
                }
            }
        }
        const double sum = block_sum_256(acc, s_w);
        if (tid == 0) {
            w.csum[0][(size_t)h * w.nch + ch] = sum;
            w.chg[0][(size_t)h * w.nch + ch] = 1;
            kpp_put_rec(w.rec[0] + ((size_t)h * w.nch + ch) * 2, sum, 1);
            kpp_put_rec(w.rec[1] + ((size_t)h * w.nch + ch) * 2, 0.0, 0);
        }
    }
}

// Inclusive sums over the wavefront's lanes
__device__ __forceinline__ double wave_scan(double v, int lane)
{
    for (int s = 1; s < 64; s <<= 1) {
        const double t = __shfl_up(v, s);
        if (lane >= s) v += t;
    }
    return v;
}

// The token of a draw, found by one wavefront: the first token whose running sum of D2 exceeds uk * sum(D2), from the
// sums cs[nch] of the chunks and then the tokens dh[N] of the chunk in which the running sum crosses.
template <typename F>
__device__ __forceinline__ int kpp_pick(F dh, const double *cs, int N, int nch, double uk, int lane)
{
    constexpr int M = KPP_CHUNK / 64;
    const int per = (nch + 63) / 64, b0 = min(nch, lane * per), b1 = min(nch, b0 + per);
    double loc = 0.0;
#pragma unroll 4
    for (int b = b0; b < b1; ++b) loc += cs[b];
    const double incl = wave_scan(loc, lane), total = __shfl(incl, 63);
    const double target = uk * total;
    int pick = -1;
    if (total > 0.0) {
        double run = incl - loc;
        int mine = nch;
        for (int b = b0; b < b1; ++b) {
            const double v = cs[b];
            if (run + v > target) { mine = b; break; }
            run += v;
        }
        // the first lane that found a chunk has the first chunk, and the running sum in front of it
        const unsigned long long found = __ballot(mine < nch);
        const int src = found ? __ffsll((long long)found) - 1 : 0;
        double base = __shfl(run, src);
        for (int ch = __shfl(mine, src); ch < nch; ++ch) {      // a second pass only if rounding pushed the crossing on
            double v[M], lb = 0.0;
#pragma unroll
            for (int i = 0; i < M; ++i) {
                const int n = ch * KPP_CHUNK + lane * M + i;
                v[i] = n < N ? dh(n) : 0.0;
                lb += v[i];
            }
            const double li = wave_scan(lb, lane);
            double r = base + (li - lb);
            int tok = -1;
#pragma unroll
            for (int i = 0; i < M; ++i) {
                r += v[i];
                if (tok < 0 && r > target && v[i] > 0.0) tok = ch * KPP_CHUNK + lane * M + i;
            }
            const unsigned long long hit = __ballot(tok >= 0);
            if (hit) {
                pick = __shfl(tok, __ffsll((long long)hit) - 1);
                break;
            }
            base += __shfl(li, 63);
        }
        if (pick < 0) {                         // rounding left the running sum at the threshold: last token with D2 > 0
            for (int n = lane; n < N; n += 64)
                if (dh(n) > 0.0) pick = n;
            for (int s = 32; s > 0; s >>= 1) pick = max(pick, __shfl_xor(pick, s));
        }
    }
    if (pick < 0) pick = (int)floor(uk * (double)N);        // every D2 is zero
    return max(0, min(N - 1, pick));
}

// Whether the bound rules a token out: not nearer to the centre than to an older one.  dot = q_x . q_c.
__device__ __forceinline__ bool kpp_ruled_out(uint2 row, int dot, float c_scale, float c_r, float c_n2)
{
    // ||x^ - c^||^2 from below (its three terms are each within 3 units in the last place of n2)
    const float scale = bf16_lo(row.x), r = bf16_hi(row.x), d2_up = bf16_hi(row.y);
    const float n2 = fmaf(scale * scale, (float)(row.y & 0xFFFFu), c_n2);
    const float t = fmaf(-2.0f * scale * c_scale, (float)dot, n2) - 1e-6f * n2;
    const float lb = sqrtf(fmaxf(t, 0.f)) - (r + c_r);
    // only if the bound is an ordinary number and says so (inputs that are no numbers are measured).  Below 1e-18 squares of
    // digit errors and scales can underflow: what is lost of r is up to 1.2e-18 and of the terms of n2 up to 1e-31, against
    // margins of 5e-16 and 1e-24 at t = 1e-18.
    return t > 1e-18f && t < 1e37f && lb > 0.f && lb * lb > 1.00001f * d2_up;
}

// Draw k >= 1.  grid (workgroups, H), block 320: wavefront 4 finds the token and the digits of the centre while
// wavefronts 0..3 wait for what the bound needs of their tokens (one wavefront that did both would wait for its bulk
// loads first: a wavefront's loads return in order).  The last draw has nothing to update and is launched with one
// workgroup per head.
template <typename T, int D>
__global__ __launch_bounds__(320, 8) void kpp_step_kernel(const T *__restrict__ X, const double *__restrict__ u, KppBufs w,
                                                          int N, int C, int k, float *__restrict__ centroids)
{
    constexpr int LPT = D / 8, G = 256 / LPT, UB = 4 / sizeof(T);       // UB: rows in flight per group of lanes
    constexpr int NW = D / 8, NQ = D / 32;      // digit words and 16-byte pieces per token
    __shared__ __align__(16) int s_c[2 * NW];   // digits of the centre: high, then low halves
    __shared__ double2 s_cd[D / 2];             // the centre: elements 8 p + 2 j, + 1 at j * LPT + p
    __shared__ KppRow s_row;
    __shared__ double s_new[KPP_CHUNK];         // lowered D2 of a token, or negative
    __shared__ uint16_t s_left[KPP_CHUNK];
    __shared__ double s_w[4];
    __shared__ int s_nleft, s_chg;

    const int h = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
    const int grp = tid / LPT, part = tid % LPT;
    const bool finder = tid >= 256;
    const int o = k & 1, nch = w.nch;
    const T *Xh = X + (size_t)h * N * D;
    const double *dh = (o ? w.d2[0] : w.d2[1]) + (size_t)h * N;
    const double *cs = (o ? w.csum[0] : w.csum[1]) + (size_t)h * nch;
    const int32_t *fl = (o ? w.chg[0] : w.chg[1]) + (size_t)h * nch;
    const uint4 *qh = w.dig + (size_t)h * NQ * N;
    uint2 *rh = w.row + (size_t)h * N;
    const bool last = k + 1 == C;
    const int ch_lo = (int)blockIdx.x * w.cpw, ch_hi = last ? ch_lo : min(nch, ch_lo + w.cpw);

    uint2 row = {};
    uint4 dig[NQ] = {};
    int chg_old = 0;
    auto load_tok = [&](int ch) {               // one token per thread
        const int n = min(N - 1, ch * KPP_CHUNK + tid);
        row = rh[n];
#pragma unroll
        for (int p = 0; p < NQ; ++p) dig[p] = qh[(size_t)p * N + n];
        chg_old = fl[ch];
    };
    if (!finder) {
        load_tok(ch_lo);
    } else {
        const int pick = kpp_pick([&](int n) { return dh[n]; }, cs, N, nch, u[(size_t)h * C + k], lane);
        float c[8];
        load_8(Xh + (size_t)pick * D + part * 8, c);
        // digits q = 16 hi + lo with hi in -7 .. 7, lo in -8 .. 7
        int q[8], hi[8], lo[8];
        const KppRow r = kpp_digits<LPT, 119>(c, q);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            hi[j] = (q[j] + 8) >> 4;
            lo[j] = q[j] - 16 * hi[j];
        }
        if (lane < LPT) {
            s_c[part] = (int)pack_nibbles(hi);
            s_c[NW + part] = (int)pack_nibbles(lo);
#pragma unroll
            for (int j = 0; j < 4; ++j) s_cd[j * LPT + part] = make_double2((double)c[2 * j], (double)c[2 * j + 1]);
            if (part == 0) { s_row = r; s_nleft = 0; s_chg = 0; }
            if (blockIdx.x == 0) {
                if (part == 0) w.picked[(size_t)h * C + k] = pick;
#pragma unroll
                for (int j = 0; j < 8; ++j) centroids[((size_t)h * C + k) * D + part * 8 + j] = c[j];
            }
        }
    }
    if (last) return;
    __syncthreads();
    const float c_scale = s_row.scale, c_r = s_row.r, c_n2 = c_scale * c_scale * (float)s_row.q2;

    // ---- D2[n] = min(D2[n], ||x_n - c||^2) for the tokens of the workgroup's chunks, and the chunks' sums
    for (int ch = ch_lo; ch < ch_hi; ++ch) {
        if (ch > ch_lo && !finder) load_tok(ch);
        const int c0 = ch * KPP_CHUNK;
        const bool in = !finder && c0 + tid < N;
        int dot = 0, dlo = 0;
#pragma unroll
        for (int p = 0; p < NQ; ++p) {
            const int4 a = *reinterpret_cast<const int4 *>(&s_c[4 * p]);
            dot = __builtin_amdgcn_sdot8((int)dig[p].x, a.x, dot, false);
            dot = __builtin_amdgcn_sdot8((int)dig[p].y, a.y, dot, false);
            dot = __builtin_amdgcn_sdot8((int)dig[p].z, a.z, dot, false);
            dot = __builtin_amdgcn_sdot8((int)dig[p].w, a.w, dot, false);
        }
#pragma unroll
        for (int p = 0; p < NQ; ++p) {
            const int4 a = *reinterpret_cast<const int4 *>(&s_c[NW + 4 * p]);
            dlo = __builtin_amdgcn_sdot8((int)dig[p].x, a.x, dlo, false);
            dlo = __builtin_amdgcn_sdot8((int)dig[p].y, a.y, dlo, false);
            dlo = __builtin_amdgcn_sdot8((int)dig[p].z, a.z, dlo, false);
            dlo = __builtin_amdgcn_sdot8((int)dig[p].w, a.w, dlo, false);
        }
        dot = 16 * dot + dlo;
        const bool left = in && !kpp_ruled_out(row, dot, c_scale, c_r, c_n2);
        const unsigned long long m = __ballot(left);
        int pos = 0;
        if (lane == 0 && m) pos = atomicAdd(&s_nleft, __popcll(m));
        pos = __builtin_amdgcn_readfirstlane(pos) + __popcll(m & ((1ull << lane) - 1ull));
        if (left) s_left[pos] = (uint16_t)tid;
        if (!finder) s_new[tid] = -1.0;
        __syncthreads();
        const int nleft = s_nleft;
        if (!finder && nleft > 0) {
            for (int i0 = 0; i0 < nleft; i0 += G * UB) {
                Raw8<T> raw[UB];
                double old[UB];
                int at[UB];
#pragma unroll
                for (int b = 0; b < UB; ++b) {
                    at[b] = s_left[min(nleft - 1, i0 + b * G + grp)];
                    raw[b] = load_raw(Xh + (size_t)(c0 + at[b]) * D + part * 8);
                    old[b] = dh[c0 + at[b]];
                }
#pragma unroll
                for (int b = 0; b < UB; ++b) {
                    if (i0 + b * G >= nleft) break;
                    asm volatile("" ::: "memory");      // the centre is read from LDS as it is used: 16 registers less
                    float x[8];
                    to_floats(raw[b], x);
                    double a = 0.0;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const double2 c = s_cd[j * LPT + part];
                        const double e0 = (double)x[2 * j] - c.x, e1 = (double)x[2 * j + 1] - c.y;
                        a = fma(e0, e0, a);
                        a = fma(e1, e1, a);
                    }
                    a = group_sum<LPT>(a);
                    if (part == 0 && i0 + b * G + grp < nleft && a < old[b]) {
                        s_new[at[b]] = a;
                        s_chg = 1;
                    }
                }
            }
        }
        __syncthreads();
        const bool chg = s_chg != 0;
        double v = 0.0;
        if (in && (chg || chg_old)) {           // the buffer that is written holds D2 of two draws ago
            v = s_new[tid];
            if (v < 0.0) v = dh[c0 + tid];
            else rh[c0 + tid].y = (row.y & 0xFFFFu) | (bf16_up((float)v) << 16);
            (o ? w.d2[1] : w.d2[0])[(size_t)h * N + c0 + tid] = v;
        }
        double sum = cs[ch];
        if (chg) sum = block_sum_256(v, s_w);   // (chg is the same in every thread)
        if (tid == 0) {
            (o ? w.csum[1] : w.csum[0])[(size_t)h * nch + ch] = sum;
            (o ? w.chg[1] : w.chg[0])[(size_t)h * nch + ch] = chg;
            s_nleft = 0;                        // (read behind the next chunk's first barrier only)
        }
        if (ch + 1 < ch_hi) {
            __syncthreads();
            if (tid == 0) s_chg = 0;
        }
    }
}

// All draws but the first in one launch: the workgroups of a head stay and wait for each other.  grid (workgroups, heads), block
// 512.  A workgroup has cpw chunks of its head, KPP_SLOTS pairs at a time (wavefronts 0..3 the even ones, 4..7 the odd ones, a
// token per thread and pair); with HELD these are all it has, and their digits and rows stay in registers, their D2 in LDS.
//
// A draw: wavefront 0 waits for the records of all chunks of the head, finds the token as kpp_step_kernel does, and puts the centre
// and its digits into LDS; all wavefronts rule out tokens by the bound and list the others; the list is measured by
// all; changed D2 goes to memory, then the sum of every chunk as a record (of a head with one workgroup both stay in LDS).  Two generations of D2 and
// of the records take turns: a workgroup that writes those of draw k has seen all records of draw k - 1, so every one
// has finished reading those of draw k - 2.
//
// The wait is bounded.  The launch takes at most one workgroup per CU of two that fit, counted on the CUs that the stream may use
// (kpp_stream_cus), so the workgroups of a head get onto the chip together -- unless other launches wait in the same way
// (several seedings at once on other streams) or the process has been kept to less than half of the CUs from outside (HSA_CU_MASK, which
// no call tells).  Workgroups that wait for one another in vain give up after KPP_PATIENCE looks, set fail[h], and the head is done again by
// a single workgroup, which waits for nobody (HELD = false, `again`; 24 heads of 16,384: 60 instead of 9 us per draw, one of 65,536: 146
// instead of 6).
//
// What bounds a draw is its chain of round trips: record out and seen, the D2 of one chunk, the new centre's row, the rows that are
// measured, D2 out.  us per draw, a launch for each / this kernel: 24 heads of 16,384 tokens (d = 128, bf16, 64 components) 13.0 /
// 8.7, 40 of 9000 14.9 / 9.2, 10 of 30,000 (d = 64) 8.4 / 7.6, 4 of 4096 (d = 64, fp32) 6.0 / 4.7, 1000 of 900 (one workgroup
// each) 32.5 / 15.2.  Beyond 65,536 tokens (more than KPP_LOOKS records to a lane) and beyond a workgroup per CU a launch
// for each draw stays: one head of 75,600 7.1 / 7.5.
static constexpr int KPP_SLOTS = 4;
static constexpr int KPP_HELD_CHUNKS = 2 * KPP_SLOTS;       // chunks of a workgroup whose digits fit its registers
static constexpr int KPP_LOOKS = 4;                         // records a lane looks at together
// looks of a draw, about a microsecond each: a draw takes 9 us, all draws of the heads in front of one, which it may have to let
// pass, 5 to 10 ms
static constexpr unsigned KPP_PATIENCE = 1u << 14;

template <typename T, int D, bool HELD>
__global__ __launch_bounds__(512, 4) void kpp_loop_kernel(const T *__restrict__ X, const double *__restrict__ u, KppBufs w, int N,
                                                          int C, unsigned patience, float *__restrict__ centroids, bool again)
{
    constexpr int LPT = D / 8, G = 512 / LPT, UB = 4 / sizeof(T);       // UB: rows in flight per group of lanes
    constexpr int NW = D / 8, NQ = D / 32;      // digit words and 16-byte pieces per token
    constexpr int TOK = 512 * KPP_SLOTS;        // tokens at a time
    extern __shared__ __align__(16) double s_cs[];      // [nch] sums of the chunks
    __shared__ __align__(16) int s_c[2 * NW];   // digits of the centre: high, then low halves
    __shared__ double2 s_cd[D / 2];             // the centre: elements 8 p + 2 j, + 1 at j * LPT + p
    __shared__ KppRow s_row;
    __shared__ double s_d2[TOK];
    __shared__ uint2 s_tok[TOK];                // KppBufs::row of the tokens
    __shared__ uint16_t s_left[TOK];
    __shared__ double s_w[KPP_SLOTS][8];
    __shared__ int s_nleft, s_stop, s_chg[2 * KPP_SLOTS];

    const int h = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int pair = wave >> 2, gt = tid & 255;
    const int grp = tid / LPT, part = tid % LPT;
    if (again && !w.fail[h]) return;
    const int nch = w.nch;
    const T *Xh = X + (size_t)h * N * D;
    const uint4 *qh = w.dig + (size_t)h * NQ * N;
    uint2 *rh = w.row + (size_t)h * N;
    // chunk i of the workgroup: neighbours go to different workgroups (the tokens near a centre often lie together)
    const int nwg = gridDim.x;
    const bool alone = HELD && nwg == 1;        // the D2 of the whole head is in LDS, token n at s_d2[n]
    auto chunk = [&](int i) { return (int)blockIdx.x + nwg * i; };

    uint4 dig[KPP_SLOTS][NQ] = {};
    unsigned chg_old = 0xFFFFFFFFu;             // HELD: bit s: the chunk of slot s changed in the draw before
    auto load_tokens = [&](int i0, const double *d2) {
#pragma unroll
        for (int s = 0; s < KPP_SLOTS; ++s) {
            const int n = min(N - 1, chunk(i0 + 2 * s + pair) * KPP_CHUNK + gt);
            s_tok[s * 512 + tid] = rh[n];
            s_d2[s * 512 + tid] = kpp_get(d2 + n);
#pragma unroll
            for (int p = 0; p < NQ; ++p) dig[s][p] = qh[(size_t)p * N + n];
        }
    };
    if (HELD) load_tokens(0, w.d2[0] + (size_t)h * N);
    if (tid == 0) s_stop = 0;

#pragma unroll 1
    for (int k = 1; k < C; ++k) {
        const int o = k & 1;
        const double *dh = (o ? w.d2[0] : w.d2[1]) + (size_t)h * N;
        double *dn = (o ? w.d2[1] : w.d2[0]) + (size_t)h * N;
        if (wave == 0) {
            const unsigned long long *rec = (o ? w.rec[0] : w.rec[1]) + (size_t)h * nch * 2;
            bool stop = false;
            unsigned looks = 0;
            for (int b0 = 0; (nwg > 1 || k == 1) && b0 < nch && !stop; b0 += 64 * KPP_LOOKS) {
                unsigned long long hi[KPP_LOOKS], lo[KPP_LOOKS];
                for (;;) {
                    bool all = patience > 0;
#pragma unroll
                    for (int i = 0; i < KPP_LOOKS; ++i) {
                        const int b = min(b0 + 64 * i + lane, nch - 1);
                        hi[i] = __hip_atomic_load(rec + 2 * b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        lo[i] = __hip_atomic_load(rec + 2 * b + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
#pragma unroll
                    for (int i = 0; i < KPP_LOOKS; ++i) all &= (unsigned)hi[i] == (unsigned)k && (unsigned)lo[i] == (unsigned)k;
                    if (__all(all)) break;
                    // (a head that has been given up: its other workgroups need not wait as long)
                    if (++looks >= patience || ((looks & 255) == 0 &&
                                                __hip_atomic_load(w.fail + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
                        stop = true;
                        break;
                    }
                }
#pragma unroll
                for (int i = 0; i < KPP_LOOKS; ++i)
                    if (b0 + 64 * i + lane < nch)
                        s_cs[b0 + 64 * i + lane] = __longlong_as_double((hi[i] & 0xFFFFFFFF00000000ull) | (lo[i] >> 32));
            }
            if (stop) {
                if (lane == 0) {
                    __hip_atomic_store(w.fail + h, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    s_stop = 1;
                }
            } else {
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                const int pick = kpp_pick([&](int n) { return alone ? s_d2[n] : kpp_get(dh + n); }, s_cs, N, nch, u[(size_t)h * C + k], lane);
                float c[8];
                load_8(Xh + (size_t)pick * D + part * 8, c);
                // digits q = 16 hi + lo with hi in -7 .. 7, lo in -8 .. 7
                int q[8], hi[8], lo[8];
                const KppRow r = kpp_digits<LPT, 119>(c, q);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    hi[j] = (q[j] + 8) >> 4;
                    lo[j] = q[j] - 16 * hi[j];
                }
                if (lane < LPT) {
                    s_c[part] = (int)pack_nibbles(hi);
                    s_c[NW + part] = (int)pack_nibbles(lo);
#pragma unroll
                    for (int j = 0; j < 4; ++j) s_cd[j * LPT + part] = make_double2((double)c[2 * j], (double)c[2 * j + 1]);
                    if (part == 0) s_row = r;
                    if (blockIdx.x == 0) {
                        if (part == 0) w.picked[(size_t)h * C + k] = pick;
#pragma unroll
                        for (int j = 0; j < 8; ++j) centroids[((size_t)h * C + k) * D + part * 8 + j] = c[j];
                    }
                }
            }
        }
        if (k + 1 == C) return;                 // (the last centre has nobody to be measured against)
        for (int i1 = 0; chunk(i1) < nch; i1 += KPP_HELD_CHUNKS) {
            if (!HELD) {
                __syncthreads();                // (the tokens before: what is in LDS has been read)
                load_tokens(i1, dh);
            }
            if (tid == 0) s_nleft = 0;
            if (tid < 2 * KPP_SLOTS) s_chg[tid] = 0;
            __syncthreads();
            if (s_stop) return;
            const float c_scale = s_row.scale, c_r = s_row.r, c_n2 = c_scale * c_scale * (float)s_row.q2;
            // ---- the bound, as in kpp_step_kernel
#pragma unroll
            for (int s = 0; s < KPP_SLOTS; ++s) {
                const int ch = chunk(i1 + 2 * s + pair);
                if (ch >= nch) break;
                int dot = 0, dlo = 0;
#pragma unroll
                for (int p = 0; p < NQ; ++p) {
                    const int4 a = *reinterpret_cast<const int4 *>(&s_c[4 * p]), b = *reinterpret_cast<const int4 *>(&s_c[NW + 4 * p]);
                    dot = __builtin_amdgcn_sdot8((int)dig[s][p].x, a.x, dot, false);
                    dot = __builtin_amdgcn_sdot8((int)dig[s][p].y, a.y, dot, false);
                    dot = __builtin_amdgcn_sdot8((int)dig[s][p].z, a.z, dot, false);
                    dot = __builtin_amdgcn_sdot8((int)dig[s][p].w, a.w, dot, false);
                    dlo = __builtin_amdgcn_sdot8((int)dig[s][p].x, b.x, dlo, false);
                    dlo = __builtin_amdgcn_sdot8((int)dig[s][p].y, b.y, dlo, false);
                    dlo = __builtin_amdgcn_sdot8((int)dig[s][p].z, b.z, dlo, false);
                    dlo = __builtin_amdgcn_sdot8((int)dig[s][p].w, b.w, dlo, false);
                }
                const bool left = ch * KPP_CHUNK + gt < N && !kpp_ruled_out(s_tok[s * 512 + tid], 16 * dot + dlo, c_scale, c_r, c_n2);
                const unsigned long long m = __ballot(left);
                int pos = 0;
                if (lane == 0 && m) pos = atomicAdd(&s_nleft, __popcll(m));
                pos = __builtin_amdgcn_readfirstlane(pos) + __popcll(m & ((1ull << lane) - 1ull));
                if (left) s_left[pos] = (uint16_t)(s * 512 + tid);
            }
            __syncthreads();
            // ---- measure what is left
            const int nleft = s_nleft;
            for (int i0 = 0; i0 < nleft; i0 += G * UB) {
                Raw8<T> raw[UB];
                int at[UB];
#pragma unroll
                for (int b = 0; b < UB; ++b) {
                    at[b] = s_left[min(nleft - 1, i0 + b * G + grp)];
                    const int n = chunk(i1 + (at[b] >> 8)) * KPP_CHUNK + (at[b] & 255);
                    raw[b] = load_raw(Xh + (size_t)n * D + part * 8);
                }
#pragma unroll
                for (int b = 0; b < UB; ++b) {
                    if (i0 + b * G >= nleft) break;
                    float x[8];
                    to_floats(raw[b], x);
                    double a = 0.0;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const double2 c = s_cd[j * LPT + part];
                        const double e0 = (double)x[2 * j] - c.x, e1 = (double)x[2 * j + 1] - c.y;
                        a = fma(e0, e0, a);
                        a = fma(e1, e1, a);
                    }
                    a = group_sum<LPT>(a);
                    if (part == 0 && i0 + b * G + grp < nleft && a < s_d2[at[b]]) {
                        s_d2[at[b]] = a;
                        s_chg[at[b] >> 8] = 1;
                    }
                }
            }
            __syncthreads();
            // ---- hand on: D2 of the chunks that changed in this draw or the last (the generation that is written is two draws
            // old), and the sums
#pragma unroll
            for (int s = 0; s < KPP_SLOTS; ++s) {
                const int ch = chunk(i1 + 2 * s + pair), n = ch * KPP_CHUNK + gt;
                if (ch >= nch) break;
                const bool chg = s_chg[2 * s + pair] != 0;
                double v = 0.0;
                if (n < N) {
                    v = s_d2[s * 512 + tid];
                    if (!HELD || (!alone && (chg || (chg_old >> s & 1)))) kpp_put(dn + n, v);
                    if (chg) {
                        const unsigned y = (s_tok[s * 512 + tid].y & 0xFFFFu) | (bf16_up((float)v) << 16);
                        s_tok[s * 512 + tid].y = y;
                        if (!HELD) rh[n].y = y;
                    }
                }
                if (chg) {
                    for (int x = 32; x > 0; x >>= 1) v += __shfl_xor(v, x);
                    if (lane == 0) s_w[s][wave] = v;
                }
                chg_old = (chg_old & ~(1u << s)) | ((unsigned)chg << s);
            }
            __builtin_amdgcn_s_waitcnt(0x0F70); // vmcnt(0): D2 is in place ..
            __syncthreads();                    // .. all of the workgroup's
            if (gt < KPP_SLOTS) {
                const int ch = chunk(i1 + 2 * gt + pair);
                if (ch < nch) {
                    const double *sw = &s_w[gt][4 * pair];
                    const double sum = s_chg[2 * gt + pair] ? ((sw[0] + sw[1]) + sw[2]) + sw[3] : s_cs[ch];
                    if (nwg > 1) kpp_put_rec((o ? w.rec[1] : w.rec[0]) + ((size_t)h * nch + ch) * 2, sum, (unsigned)k + 1);
                    else s_cs[ch] = sum;        // (nobody else wants it)
                }
            }
        }
        __syncthreads();                        // s_cs, s_w, s_chg and the centre have been read
    }
}

// Chunks per workgroup: as many as it takes to have at most KPP_TARGET_WGS workgroups (each of them repeats the search
// for the token of the draw).
static KppBufs kpp_carve(void *ws, int H, int N, int d, int C, size_t *total)
{
    KppBufs k;
    k.nch = (int)(((long long)N + KPP_CHUNK - 1) / KPP_CHUNK);
    k.cpw = (int)(((long long)H * k.nch + KPP_TARGET_WGS - 1) / KPP_TARGET_WGS);
    Carver c(ws);
    for (int i = 0; i < 2; ++i) {
        k.d2[i] = c.take<double>((size_t)H * N);
        k.csum[i] = c.take<double>((size_t)H * k.nch);
        k.chg[i] = c.take<int32_t>((size_t)H * k.nch);
    }
    k.dig = c.take<uint4>((size_t)H * N * (d / 32));
    k.row = c.take<uint2>((size_t)H * N);
    k.picked = c.take<int32_t>((size_t)H * C);
    for (int i = 0; i < 2; ++i) k.rec[i] = c.take<unsigned long long>((size_t)H * k.nch * 2);
    k.fail = c.take<int32_t>((size_t)H);
    *total = c.used;
    return k;
}

// (the size query does not name d: the larger of the two head dimensions)
size_t kpp_ws_bytes(int H, int N, int C)
{
    size_t total;
    (void)kpp_carve(nullptr, H, N, 128, C, &total);
    return total;
}

// CUs that launches on the stream may use: those of its mask (hipExtStreamCreateWithCUMask), else all of the device.  A stream that is
// captured is not asked; its graph may run on any.
static int kpp_stream_cus(hipStream_t st, int *ncu)
{
    SVG2_TRY(device_cu_count(ncu));
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    uint32_t mask[32] = {};
    if (hipStreamIsCapturing(st, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone &&
        hipExtStreamGetCUMask(st, 32, mask) == hipSuccess) {
        int n = 0;
        for (uint32_t m : mask) n += __builtin_popcount(m);
        if (n > 0) *ncu = std::min(*ncu, n);
    } else {
        (void)hipGetLastError();                // (not an error of this call)
    }
    return SVG2_OK;
}

// Chunks per workgroup of kpp_loop_kernel, 0 if a launch per draw is the better way (see there): a single workgroup for a head
// that it can hold; as few chunks as leave a workgroup per CU otherwise.
static int kpp_loop_chunks(int H, int nch, int ncu)
{
    if (nch <= KPP_HELD_CHUNKS) return nch;
    if (nch > 64 * KPP_LOOKS) return 0;
    for (int cpw = 2; cpw <= KPP_HELD_CHUNKS; cpw += 2)
        if ((long long)H * cdiv(nch, cpw) <= ncu) return cpw;
    return 0;
}

template <typename T, int D>
static int kpp_run(const T *X, int H, int N, int C, const double *u, float *centroids, int32_t *picked, void *ws,
                   unsigned patience, hipStream_t st)
{
    size_t total;
    KppBufs w = kpp_carve(ws, H, N, D, C, &total);
    if (picked) w.picked = picked;
    const int nwg = cdiv(w.nch, w.cpw);
    hipLaunchKernelGGL((kpp_first_kernel<T, D>), dim3(C > 1 ? nwg : 1, H), dim3(256), 0, st, X, u, w, N, C, centroids, false);
    int cpw = 0, ncu = 0;
    SVG2_TRY(kpp_stream_cus(st, &ncu));
    if (C > 2) cpw = kpp_loop_chunks(H, w.nch, ncu);
    const size_t lds = (size_t)w.nch * sizeof(double);
    if (cpw > 0) {
        // (a head in one workgroup has nobody to wait for)
        hipLaunchKernelGGL((kpp_loop_kernel<T, D, true>), dim3(cdiv(w.nch, cpw), H), dim3(512), lds, st, X, u, w, N, C,
                           cpw < w.nch ? patience : KPP_PATIENCE, centroids, false);
        if (cpw < w.nch) {                      // heads that were given up
            hipLaunchKernelGGL((kpp_first_kernel<T, D>), dim3(nwg, H), dim3(256), 0, st, X, u, w, N, C, centroids, true);
            hipLaunchKernelGGL((kpp_loop_kernel<T, D, false>), dim3(1, H), dim3(512), lds, st, X, u, w, N, C, KPP_PATIENCE,
                               centroids, true);
        }
    } else {
        for (int k = 1; k < C; ++k)
            hipLaunchKernelGGL((kpp_step_kernel<T, D>), dim3(k + 1 < C ? nwg : 1, H), dim3(320), 0, st, X, u, w, N, C, k,
                               centroids);
    }
    SVG2_HIP_CHECK(hipGetLastError());
    return SVG2_OK;
}

static int kpp_dispatch(const void *X, int dtype, int H, int N, int d, int C, const double *u, float *centroids,
                        int32_t *picked, void *ws, unsigned patience, hipStream_t st)
{
    if (dtype == SVG2_BF16) {
        const bf16_t *x = static_cast<const bf16_t *>(X);
        return d == 128 ? kpp_run<bf16_t, 128>(x, H, N, C, u, centroids, picked, ws, patience, st)
                        : kpp_run<bf16_t, 64>(x, H, N, C, u, centroids, picked, ws, patience, st);
    }
    const float *x = static_cast<const float *>(X);
    return d == 128 ? kpp_run<float, 128>(x, H, N, C, u, centroids, picked, ws, patience, st)
                    : kpp_run<float, 64>(x, H, N, C, u, centroids, picked, ws, patience, st);
}

int kpp_launch(const void *X, int dtype, int H, int N, int d, int C, const double *u, float *centroids, int32_t *picked,
               void *ws, hipStream_t st)
{
    return kpp_dispatch(X, dtype, H, N, d, C, u, centroids, picked, ws, KPP_PATIENCE, st);
}

}  // namespace svg2

#ifdef SVG2_TEST_HOOKS
// svg2_kmeans_pp_init with checked arguments and a patience of its own: with 0 a workgroup gives its head up at its first look
// for the others' sums, and every head of several workgroups is done again.
extern "C" int svg2_test_kmeans_pp_init(const void *X, int dtype, int H, int N, int d, int C, const double *u, float *centroids,
                                        int32_t *picked, void *ws, unsigned patience, void *stream)
{
    return svg2::kpp_dispatch(X, dtype, H, N, d, C, u, centroids, picked, ws, patience, static_cast<hipStream_t>(stream));
}

// Workgroups that wait for one another in a call on the stream; 0: none do.
extern "C" int svg2_test_kmeans_pp_waiting(int H, int N, void *stream)
{
    int ncu = 0;
    if (svg2::kpp_stream_cus(static_cast<hipStream_t>(stream), &ncu) != SVG2_OK) return -1;
    const int nch = svg2::cdiv(N, svg2::KPP_CHUNK), cpw = svg2::kpp_loop_chunks(H, nch, ncu);
    return cpw > 0 && cpw < nch ? H * svg2::cdiv(nch, cpw) : 0;
}

// Byte of the workspace at which svg2_test_kmeans_pp_init leaves one int32 per head: 1 if the head has been given up.
extern "C" size_t svg2_test_kmeans_pp_given_up(int H, int N, int d, int C)
{
    size_t total;
    char *base = reinterpret_cast<char *>(256);         // (any aligned address: nothing is read)
    return (size_t)(reinterpret_cast<char *>(svg2::kpp_carve(base, H, N, d, C, &total).fail) - base);
}
#endif
