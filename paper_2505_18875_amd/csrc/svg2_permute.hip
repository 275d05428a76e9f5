// Semantic-aware permutation (paper Section 4.1) as a stable counting sort of
// token ids by cluster label, plus the row gather that applies it.
//
//   hist     per (head, chunk): histogram of labels              (LDS atomics)
//   scan     per head: totals -> offsets (exclusive scan over clusters) and
//            the first output slot of every (chunk, cluster)
//   scatter  per (head, chunk): one wavefront walks its chunk in token order,
//            ranking equal labels inside each group of 64 with ballots, so the
//            order inside a cluster stays the original token order
//   (short heads: all three in one workgroup per head, permute_sort_head_kernel)
//   gather   dst[r,:] = src[perm[r],:], 16 bytes per lane, rows coalesced on
//            the write side
//
// Everything is integer work: results are unique and reproducible bit for bit.
#include <algorithm>
#include <mutex>

#include "svg2_common.h"

namespace svg2 {

static constexpr int PERM_CHUNK = 1024;     // tokens per chunk (one wavefront in scatter)

// Scratch of svg2_permute_noalloc: the per-(head, chunk, cluster) histogram of the counting sort lives in this
// file-scope array instead of a caller's workspace.  Every GPU the library runs on holds its own copy until the
// process ends.  In host code the name is only a handle: the device address is looked up once per device
// (hipGetSymbolAddress) and that pointer is what kernels get.
static __device__ __align__(256) unsigned char scratch[SVG2_PERMUTE_NOALLOC_SCRATCH_BYTES];

// Every kernel of the sort takes up to two independent problems ("sides": the Q tokens and the K tokens of a
// layer, which share H and N but not C) and picks its side with blockIdx.z, so that both sorts of a layer -- or of
// a k-means iteration -- cost one launch per step instead of two.
__global__ __launch_bounds__(256) void permute_hist_kernel(SortArgs a, int N, int nchunks)
{
    extern __shared__ int32_t s_hist[];
    const SortSide S = blockIdx.z ? a.s[1] : a.s[0];      // (a select of scalars, not an indexed copy)
    const int chunk = blockIdx.x, h = blockIdx.y, C = S.C;
    for (int c = threadIdx.x; c < C; c += blockDim.x) s_hist[c] = 0;
    __syncthreads();
    const int n0 = chunk * PERM_CHUNK;
    const int n1 = min(N, n0 + PERM_CHUNK);
    const int32_t *lab = S.labels + (size_t)h * N;
    for (int n = n0 + threadIdx.x; n < n1; n += blockDim.x) atomicAdd(&s_hist[lab[n]], 1);
    __syncthreads();
    int32_t *out = S.hist + ((size_t)h * nchunks + chunk) * C;
    for (int c = threadIdx.x; c < C; c += blockDim.x) out[c] = s_hist[c];
}

static constexpr int SCAN_THREADS = 1024;
static constexpr int SCAN_UB = 16;

// Exclusive prefix sum over the workgroup's threads; *total = sum of all.
__device__ __forceinline__ int scan_threads(int v, int32_t *s_wave, int *total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int incl = v;
    for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(incl, o);
        if (lane >= o) incl += u;
    }
    __syncthreads();                                    // s_wave of an earlier call has been read
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < SCAN_THREADS / 64; ++w) {
        const int u = s_wave[w];
        before += w < wave ? u : 0;
        all += u;
    }
    *total = all;
    return before + incl - v;
}

// s_tot[0 .. C): sizes of the clusters -> first sorted row of each; offsets[h] is written.  If the side asks for it
// (S.pieces), every cluster is also cut into pieces of at most S.seg sorted rows (never crossing a cluster boundary) for
// the segmented sum of the k-means update step: pieces[h][first_piece[c] + t] = (cluster, first row, rows, 0),
// first_piece[h][C] = n_pieces[h] = number of pieces of the head.
__device__ __forceinline__ void scan_clusters(const SortSide &S, int h, int N, int32_t *s_tot, int32_t *s_wave)
{
    const int tid = threadIdx.x, C = S.C, seg = S.seg;
    int32_t *off = S.offsets + (size_t)h * (C + 1);
    int carry = 0, carry_p = 0;
    for (int cb = 0; cb < C; cb += SCAN_THREADS) {
        const int c = cb + tid;
        const int size = c < C ? s_tot[c] : 0;
        int all;
        const int start = carry + scan_threads(size, s_wave, &all);
        carry += all;
        if (c < C) {
            s_tot[c] = start;
            off[c] = start;
        }
        if (S.pieces == nullptr) continue;
        const int np = (size + seg - 1) / seg;
        const int first = carry_p + scan_threads(np, s_wave, &all);
        carry_p += all;
        if (c < C) S.first_piece[(size_t)h * (C + 1) + c] = first;
        for (int t = 0; t < np; ++t)
            S.pieces[(size_t)h * S.max_pieces + first + t] = make_int4(c, start + t * seg, min(seg, size - t * seg), 0);
    }
    if (tid == 0) {
        off[C] = N;
        if (S.pieces) {
            S.first_piece[(size_t)h * (C + 1) + C] = carry_p;
            S.n_pieces[h] = carry_p;
        }
    }
    __syncthreads();
}

// One workgroup per head and side.  hist[h][k][c] becomes the first sorted row that chunk k writes for cluster c.  What
// bounds it is the chain of round trips to memory: the chunks of a cluster are dealt out to as many threads as there
// are (1024 over the clusters), SCAN_UB loads of a thread are issued before they are used.  (256 threads, each with all
// chunks of its clusters: 22 instead of 13 us at 40 heads of 75,600 tokens in 100 and 500 clusters, 24 instead of 12 us on
// average over 8 heads of 37,800 in 100 and in 2000.)
__global__ __launch_bounds__(SCAN_THREADS) void permute_scan_kernel(SortArgs a, int N, int nchunks)
{
    extern __shared__ int32_t s_tot[];                 // [C] totals, then exclusive offsets
    __shared__ int32_t s_part[SCAN_THREADS];
    __shared__ int32_t s_wave[SCAN_THREADS / 64];
    const SortSide S = blockIdx.z ? a.s[1] : a.s[0];      // (a select of scalars, not an indexed copy)
    const int h = blockIdx.x, tid = threadIdx.x, C = S.C;
    int32_t *hh = S.hist + (size_t)h * nchunks * C;
    int cw = SCAN_THREADS;                              // clusters side by side; the threads form SCAN_THREADS / cw parts
    while (cw > 64 && cw / 2 >= C) cw >>= 1;
    const int parts = SCAN_THREADS / cw, part = tid / cw, cl = tid & (cw - 1);
    const int per = (nchunks + parts - 1) / parts, k_lo = min(nchunks, part * per), k_hi = min(nchunks, k_lo + per);
    for (int cb = 0; cb < C; cb += cw) {                // (more than one pass only with parts = 1)
        const int c = cb + cl;
        int run = 0;
        if (c < C)
            for (int k0 = k_lo; k0 < k_hi; k0 += SCAN_UB) {
                int v[SCAN_UB];
#pragma unroll
                for (int u = 0; u < SCAN_UB; ++u) v[u] = (k0 + u < k_hi) ? hh[(size_t)(k0 + u) * C + c] : 0;
#pragma unroll
                for (int u = 0; u < SCAN_UB; ++u) run += v[u];
            }
        s_part[tid] = run;
        __syncthreads();
        if (part == 0 && c < C) {
            for (int q = 1; q < parts; ++q) run += s_part[q * cw + cl];
            s_tot[c] = run;
        }
        if (cb + cw < C) __syncthreads();
    }
    __syncthreads();
    scan_clusters(S, h, N, s_tot, s_wave);
    for (int cb = 0; cb < C; cb += cw) {
        const int c = cb + cl;
        if (c >= C) break;
        int pos = s_tot[c];
        for (int q = 0; q < part; ++q) pos += s_part[q * cw + cl];
        for (int k0 = k_lo; k0 < k_hi; k0 += SCAN_UB) {
            int v[SCAN_UB];
#pragma unroll
            for (int u = 0; u < SCAN_UB; ++u) v[u] = (k0 + u < k_hi) ? hh[(size_t)(k0 + u) * C + c] : 0;
#pragma unroll
            for (int u = 0; u < SCAN_UB; ++u) {
                if (k0 + u < k_hi) hh[(size_t)(k0 + u) * C + c] = pos;
                pos += v[u];
            }
        }
    }
}

// Stable ranks of one chunk: a wavefront walks it in token order, 64 tokens at a time; lr[] holds the labels of the
// chunk, s_cur[c] the next free sorted row of cluster c (of this chunk alone).
__device__ __forceinline__ void scatter_chunk(const int (&lr)[PERM_CHUNK / 64], int n0, int n1, int nbits, int32_t *s_cur,
                                              int32_t *__restrict__ pm, int32_t *__restrict__ ip)
{
    const int lane = threadIdx.x & 63;
    const unsigned long long lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
    for (int i = 0; i < PERM_CHUNK / 64; ++i) {
        const int g = n0 + i * 64;
        if (g >= n1) break;
        const int n = g + lane;
        const bool valid = n < n1;
        const int l = lr[i];
        // lanes holding the same label as this one (what bounds the kernel: four vector instructions per bit and group)
        const unsigned long long live = __ballot(valid);
        unsigned lo = (unsigned)live, hi = (unsigned)(live >> 32);
        for (int b = 0; b < nbits; ++b) {
            const unsigned bit = (unsigned)__builtin_amdgcn_sbfe(l, b, 1);      // 0 or all ones
            const unsigned long long m = __ballot(bit != 0);
            lo &= ~((unsigned)m ^ bit);
            hi &= ~((unsigned)(m >> 32) ^ bit);
        }
        const unsigned long long peers = (unsigned long long)hi << 32 | lo;
        if (valid) {
            const int pos = s_cur[l] + __popcll(peers & lt_mask);
            pm[pos] = n;
            if (ip) ip[n] = pos;
        }
        // the first lane of every peer group advances that cluster's cursor; LDS operations of one wavefront complete in
        // order, so it is enough that the compiler keeps theirs
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (valid && (peers & lt_mask) == 0) s_cur[l] += __popcll(peers);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

__device__ __forceinline__ void load_chunk_labels(int (&lr)[PERM_CHUNK / 64], const int32_t *lab, int n0, int n1)
{
    // all labels of the chunk are requested up front (one memory round trip instead of one per group of 64)
#pragma unroll
    for (int i = 0; i < PERM_CHUNK / 64; ++i) {
        const int n = n0 + i * 64 + (threadIdx.x & 63);
        lr[i] = (n < n1) ? lab[n] : 0;
    }
}

__global__ __launch_bounds__(64) void permute_scatter_kernel(SortArgs a, int N, int nchunks)
{
    extern __shared__ int32_t s_cur[];                 // [C] next free sorted row per cluster
    const SortSide S = blockIdx.z ? a.s[1] : a.s[0];      // (a select of scalars, not an indexed copy)
    const int chunk = blockIdx.x, h = blockIdx.y, lane = threadIdx.x, C = S.C;
    const int32_t *base = S.hist + ((size_t)h * nchunks + chunk) * C;
    const int n0 = chunk * PERM_CHUNK, n1 = min(N, n0 + PERM_CHUNK);
    int lr[PERM_CHUNK / 64];
    load_chunk_labels(lr, S.labels + (size_t)h * N, n0, n1);
    for (int c = lane; c < C; c += 64) s_cur[c] = base[c];
    __syncthreads();
    scatter_chunk(lr, n0, n1, S.nbits, s_cur, S.perm + (size_t)h * N, S.inv_perm ? S.inv_perm + (size_t)h * N : nullptr);
}

// The whole sort of a head in one workgroup, for heads of at most 16 wavefronts x 1024 tokens whose histograms fit
// SORT1_LDS: wavefront w counts, ranks and scatters chunk w (`chunk` tokens, as few as give every wavefront one), the
// histograms and their scan stay in LDS.  Three launches that each wait for a few round trips to memory become one:
// 2 heads of 1024 tokens in 16 and 32 clusters 17 -> 5.4 us, 24 heads of 16,384 in 100 and 500 29 -> 19 us.
// With more tokens the heads alone do not fill the chip and the three kernels spread better.
static constexpr int SORT1_WAVES = SCAN_THREADS / 64;
static constexpr size_t SORT1_LDS = 60 * 1024;

__global__ __launch_bounds__(SCAN_THREADS) void permute_sort_head_kernel(SortArgs a, int N, int chunk, int nchunks)
{
    extern __shared__ int32_t s_hist[];                // [nchunks + 1][C], the last row the totals
    __shared__ int32_t s_wave[SCAN_THREADS / 64];
    const SortSide S = blockIdx.z ? a.s[1] : a.s[0];      // (a select of scalars, not an indexed copy)
    const int h = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, C = S.C;
    const int n0 = wave * chunk, n1 = min(N, n0 + chunk);       // (a wavefront past the last chunk: n1 <= n0)
    int32_t *s_tot = s_hist + (size_t)nchunks * C, *s_own = s_hist + (size_t)wave * C;
    int lr[PERM_CHUNK / 64];
    load_chunk_labels(lr, S.labels + (size_t)h * N, n0, n1);
    for (int e = tid; e < nchunks * C; e += SCAN_THREADS) s_hist[e] = 0;
    __syncthreads();
    // the lanes that hold the first lane's label count together: atomics on one address run one after the other (24 heads of
    // 16,384 tokens, 90 % of them in one cluster: 13.7 instead of 24.0 us, the three kernels 19.9; even: 13.8 instead of 13.1)
#pragma unroll
    for (int i = 0; i < PERM_CHUNK / 64; ++i) {
        const int g = n0 + i * 64, l = lr[i], l0 = __builtin_amdgcn_readfirstlane(l);
        if (g >= n1) break;
        const unsigned long long same = __ballot(g + lane < n1 && l == l0);
        if (lane == 0) atomicAdd(&s_own[l0], __popcll(same));
        else if (g + lane < n1 && l != l0) atomicAdd(&s_own[l], 1);
    }
    __syncthreads();
    for (int c = tid; c < C; c += SCAN_THREADS) {
        int run = 0;
        for (int k = 0; k < nchunks; ++k) {
            const int v = s_hist[k * C + c];
            s_hist[k * C + c] = run;
            run += v;
        }
        s_tot[c] = run;
    }
    __syncthreads();
    scan_clusters(S, h, N, s_tot, s_wave);
    if (n0 >= n1) return;
    for (int c = lane; c < C; c += 64) s_own[c] += s_tot[c];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    scatter_chunk(lr, n0, n1, S.nbits, s_own, S.perm + (size_t)h * N, S.inv_perm ? S.inv_perm + (size_t)h * N : nullptr);
}

// dst[h, r, :] = src[h, perm[h, r], :] for up to three tensors, each with its permutation, in one launch; a row is
// `lanes_per_row` lanes of 16 bytes, and a lane has GATHER_UB rows in flight.  Large layers run at the rate of a large copy
// (two tensors of 8 heads of 118,800 rows, fp32: 386 us), small ones at the latency of two dependent loads: 4 heads of 9601
// rows in fp32, D = 128: 12.4 us, one head of 4096 in bf16: 3.0 us.  (One row at a time, 256 rows per workgroup whatever the
// size: 22 and 7.6 us.  With the rows in flight as HIP's uint4, a class whose arrays the compiler moves to LDS: 22 and 10.2
// us, and 20.7 instead of 9.8 us for one head of 118,800 rows of 128 bytes.)
static constexpr int GATHER_UB = 4;

typedef __attribute__((ext_vector_type(4))) unsigned gather_vec;
struct GatherPtrs {
    const gather_vec *src[3];
    gather_vec *dst[3];
    const int32_t *perm[3];
};

__global__ __launch_bounds__(256) void permute_gather_kernel(GatherPtrs p, int N, int lanes_per_row, int rows_per_block)
{
    const int h = blockIdx.y, t = blockIdx.z;
    const gather_vec *src = (t == 0 ? p.src[0] : t == 1 ? p.src[1] : p.src[2]) + (size_t)h * N * lanes_per_row;
    gather_vec *dst = (t == 0 ? p.dst[0] : t == 1 ? p.dst[1] : p.dst[2]) + (size_t)h * N * lanes_per_row;
    const int32_t *pm = (t == 0 ? p.perm[0] : t == 1 ? p.perm[1] : p.perm[2]) + (size_t)h * N;
    const int r0 = blockIdx.x * rows_per_block;
    const int r1 = min(N, r0 + rows_per_block);
    const int rows_per_pass = 256 / lanes_per_row;
    const int sub = threadIdx.x / lanes_per_row, part = threadIdx.x % lanes_per_row;
    for (int r = r0 + sub; r < r1; r += GATHER_UB * rows_per_pass) {
        int s[GATHER_UB];
        gather_vec v[GATHER_UB];
#pragma unroll
        for (int u = 0; u < GATHER_UB; ++u) s[u] = pm[min(r + u * rows_per_pass, r1 - 1)];
#pragma unroll
        for (int u = 0; u < GATHER_UB; ++u) v[u] = src[(size_t)s[u] * lanes_per_row + part];
#pragma unroll
        for (int u = 0; u < GATHER_UB; ++u)
            if (r + u * rows_per_pass < r1) dst[(size_t)(r + u * rows_per_pass) * lanes_per_row + part] = v[u];
    }
}

size_t permute_ws_bytes(int H, int N, int C)
{
    const int nchunks = cdiv(N, PERM_CHUNK);
    return align256((size_t)H * nchunks * C * sizeof(int32_t));
}

// The counting sort of one or two sides (labels -> offsets, perm, inv_perm; pieces if asked for): one
// launch or three.
// The caller fills labels, C, hist, offsets, perm, inv_perm and the piece fields of every side; nbits is set here.
int sort_launch(SortArgs a, int nsides, int H, int N, hipStream_t st)
{
    const int nchunks = cdiv(N, PERM_CHUNK);
    int cmax = 0;
    for (int s = 0; s < nsides; ++s) {
        int nbits = 0;
        while ((1 << nbits) < a.s[s].C) ++nbits;
        a.s[s].nbits = nbits;
        cmax = std::max(cmax, a.s[s].C);
    }
    const size_t lds = (size_t)cmax * sizeof(int32_t);
    // one workgroup per head, if the histograms of as many wavefronts as the tokens need fit its LDS
    const int waves = std::min<int>(SORT1_WAVES, (int)(SORT1_LDS / lds) - 1), groups = cdiv(N, 64);
    if (waves >= 1 && cdiv(groups, waves) * 64 <= PERM_CHUNK) {
        const int chunk = cdiv(groups, waves) * 64, nch = cdiv(N, chunk);
        hipLaunchKernelGGL(permute_sort_head_kernel, dim3(H, 1, nsides), dim3(SCAN_THREADS), (nch + 1) * lds, st, a, N, chunk,
                           nch);
        SVG2_HIP_CHECK(hipGetLastError());
        return SVG2_OK;
    }
    hipLaunchKernelGGL(permute_hist_kernel, dim3(nchunks, H, nsides), dim3(256), lds, st, a, N, nchunks);
    hipLaunchKernelGGL(permute_scan_kernel, dim3(H, 1, nsides), dim3(SCAN_THREADS), lds, st, a, N, nchunks);
    hipLaunchKernelGGL(permute_scatter_kernel, dim3(nchunks, H, nsides), dim3(64), lds, st, a, N, nchunks);
    SVG2_HIP_CHECK(hipGetLastError());
    return SVG2_OK;
}

static void gather_launch(const int32_t *const *perm, int H, int N, int n_tensors, const void *const *src,
                          void *const *dst, int dtype, int d, hipStream_t st)
{
    GatherPtrs p = {};
    for (int t = 0; t < n_tensors; ++t) {
        p.src[t] = static_cast<const gather_vec *>(src[t]);
        p.dst[t] = static_cast<gather_vec *>(dst[t]);
        p.perm[t] = perm[t];
    }
    const int row_bytes = d * (dtype == SVG2_BF16 ? 2 : 4);
    const int lanes_per_row = row_bytes / 16;
    // 256 rows per workgroup, fewer (down to what it has in flight at once) where that leaves CUs without work
    int rows_per_block = 256;
    while (rows_per_block > GATHER_UB * (256 / lanes_per_row) && (long long)cdiv(N, rows_per_block) * H * n_tensors < 2048)
        rows_per_block /= 2;
    hipLaunchKernelGGL(permute_gather_kernel, dim3(cdiv(N, rows_per_block), H, n_tensors), dim3(256), 0, st, p, N,
                       lanes_per_row, rows_per_block);
}

int permute_launch(const int32_t *labels, int H, int N, int C, int32_t *offsets, int32_t *perm,
                   int32_t *inv_perm, int n_tensors, const void *const *src, void *const *dst,
                   int dtype, int d, void *ws, hipStream_t st)
{
    SortArgs a = {};
    a.s[0].labels = labels;
    a.s[0].C = C;
    a.s[0].hist = static_cast<int32_t *>(ws);
    a.s[0].offsets = offsets;
    a.s[0].perm = perm;
    a.s[0].inv_perm = inv_perm;
    {
        ProfileSpan sp(SVG2_K_PERMUTE_SORT, st);
        SVG2_TRY(sort_launch(a, 1, H, N, st));
    }
    if (n_tensors > 0) {
        ProfileSpan sp(SVG2_K_PERMUTE_GATHER, st);
        const int32_t *perms[2] = {perm, perm};
        gather_launch(perms, H, N, n_tensors, src, dst, dtype, d, st);
    }
    SVG2_HIP_CHECK(hipGetLastError());
    return SVG2_OK;
}

// The permuted copies of a layer (Section 4.1: pi_q for Q, pi_k shared by K and V).
int gather_pair_launch(const int32_t *perm_q, const int32_t *perm_k, int H, int N, const void *Q, const void *K,
                       const void *V, void *Qp, void *Kp, void *Vp, int dtype, int d, hipStream_t st)
{
    ProfileSpan sp(SVG2_K_PERMUTE_GATHER, st);
    const int32_t *perm[3] = {perm_q, perm_k, perm_k};
    const void *src[3] = {Q, K, V};
    void *dst[3] = {Qp, Kp, Vp};
    gather_launch(perm, H, N, 3, src, dst, dtype, d, st);
    SVG2_HIP_CHECK(hipGetLastError());
    return SVG2_OK;
}

// Device address of `scratch` on the current device (looked up on the first call per device, then kept).
static constexpr int PERM_MAX_DEVICES = 64;
static std::mutex g_scratch_mu;
static void *g_scratch_ptr[PERM_MAX_DEVICES] = {};

int permute_static_scratch(void **out)
{
    int dev = -1;
    SVG2_HIP_CHECK(hipGetDevice(&dev));
    SVG2_REQUIRE(dev >= 0 && dev < PERM_MAX_DEVICES, SVG2_INVALID_ARG, "device ordinal %d is outside 0..%d", dev,
                 PERM_MAX_DEVICES - 1);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        SVG2_HIP_CHECK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        SVG2_REQUIRE(p != nullptr, SVG2_HIP_ERROR, "hipGetSymbolAddress returned a null address for the scratch array");
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return SVG2_OK;
}

}  // namespace svg2
