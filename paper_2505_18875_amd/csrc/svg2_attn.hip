// Block-sparse attention over variable-size clusters (paper Section 4.3).
//
// A work item is (head, tile of up to BM consecutive rows of ONE query
// cluster).  Its keys are the rows of the key clusters selected for that query
// cluster (one CSR row), taken as one virtual concatenated sequence that is
// consumed 64 keys at a time: a 64-key tile may straddle cluster boundaries,
// so short key clusters cost no padding; only the last tile of a work item is
// ragged and masked.  This plays the role of the per-token sparse load the
// paper describes, re-thought for LDS staging.
//
//   attn_plan_kernel   per head: tile descriptors (cluster, first row, rows)
//                      and, for every CSR entry, (first key row, keys before
//                      it in its CSR row).
//   attn_bf16_kernel   MFMA 32x32x16 bf16, FlashAttention-style online softmax
//                      in fp32.  Scores are computed transposed (S^T = K Q^T):
//                      a lane then holds 32 keys of ONE query, so row max / row
//                      sum stay in registers, and the probabilities are
//                      already laid out as the B operand of O^T += V^T P^T.
//                      V^T comes out of LDS through the transposing 64-bit
//                      read (ds_read_b64_tr_b16).
//   attn_f32_kernel    fp32 storage: operands in three bf16 parts or, where these would lose bits, MFMA 32x32x2 fp32; the keys of
//                      a work item split over the wavefronts.
//
// The result of sorted row r is stored at row perm_q[r] (Section 4.1: the
// inverse query permutation restores the original order).
//
// Gather-free variant (perm_k given): Q, K and V stay in token order and the
// kernels go through perm_q / perm_k when they fetch a row -- the per-token
// sparse load of Section 4.3 -- so no permuted copies are needed.
#include <algorithm>
#include <type_traits>

#include "svg2_attn_shared.h"

namespace svg2 {


// Launch shape of the bf16 kernel.  Measured on the Wan-like layer (8-head probe, ms sparse / dense):
// 4 wavefronts, 2 buffers, 2 workgroups per CU 7.76 / 24.5;  8 wavefronts, 3 buffers, 1 workgroup per CU
// (half the L2 -> LDS traffic, but 8 wavefronts behind one barrier) 8.17 / 25.7.
static constexpr int ATT_NSTG = 2;         // K and V tile buffers in LDS (each); the schedule is written for two
static constexpr int ATT_RUN_LDS = 1920;     // runs of a work item kept in LDS (15 KB: two workgroups of 80 KB still fit a CU)
static constexpr int ATT_OPS_B = 16;       // vector operations of a block's probabilities done early (see phase B)
// The reference level of a query starts as the maximum of its first score block; a block whose maximum is more than 2^8
// above it takes it up to that maximum, where the largest probability is 1 again.  (A level that may lag by more loses
// precision: the probability that decides the row is then a rounded bf16 number.  With 2^40, log-sum-exp is off by up to
// 2^-8 and its rms error over rows of ordinary layers is 1.1 to 1.25 times what it is with 2^8; 2^40 also leaves V only
// 2^87 over the row length.)  The block's maximum itself is not looked for in every block: a probability above 2^8 makes
// the block's sum at least 2^8, and only then is it taken.  (In every block it cost 8 v_max3 and a chain of eight dependent
// instructions per 32 keys: 3.21 against 3.10 ms for dense attention of 24 heads of 16,384 tokens, with the same bits.)
static constexpr float ATT_LEVEL_LOG2 = 8.0f;
static constexpr float ATT_LEVEL_SUM = 256.0f;

// ---------------------------------------------------------------- plan
// grid (1 + ceil(Cq / 4), H), block 256.  Workgroup 0 of a head writes its tiles, the others take four CSR rows each, one
// per wavefront.  A cluster with many tiles and a run with many key tiles have their entries written by the whole
// wavefront.  (One workgroup per head for all rows took 45 to 60 us whatever the number of heads, each wavefront a
// quarter of the rows with three dependent round trips to memory each: 24 heads of 9601 tokens, 100 x 500 clusters: 51 us,
// 6 us now; dense attention of 24 heads of 9601 tokens: 13 us, 5 us now.)
static constexpr int PLAN_OWN = 4;              // up to this many entries are written by the lane that holds the cluster

__global__ __launch_bounds__(256) void attn_plan_kernel(const int32_t *__restrict__ offsets_q,
                                                        const int32_t *__restrict__ offsets_k,
                                                        const int32_t *__restrict__ row_ptr,
                                                        const int32_t *__restrict__ col_idx, int Cq, int Ck, int BM,
                                                        int max_tiles, int4 *__restrict__ tiles,
                                                        int32_t *__restrict__ n_tiles, int2 *__restrict__ runs,
                                                        int32_t *__restrict__ row_keys,
                                                        int32_t *__restrict__ cl_first, int key_tiles,
                                                        int32_t *__restrict__ tile_run, unsigned *__restrict__ range)
{
    __shared__ int32_t s_wave[4];
    const int h = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

    if (blockIdx.x == 0) {
        if (range && tid < F32_RANGE) range[(size_t)h * F32_RANGE + tid] = 0;      // (attn_range fills it in the next launch)
        // tiles: running count over clusters, 256 clusters per pass
        const int32_t *oq = offsets_q + (size_t)h * (Cq + 1);
        int4 *tl = tiles + (size_t)h * max_tiles;
        int carry = 0;
        for (int c0 = 0; c0 < Cq; c0 += 256) {
            const int c = c0 + tid;
            const int start = (c < Cq) ? oq[c] : 0;
            const int size = (c < Cq) ? oq[c + 1] - start : 0;
            const int nt = (size + BM - 1) / BM;
            int incl = nt;
            for (int o = 1; o < 64; o <<= 1) {
                const int v = __shfl_up(incl, o);
                if (lane >= o) incl += v;
            }
            __syncthreads();                            // the pass before has read s_wave
            if (lane == 63) s_wave[wave] = incl;
            __syncthreads();
            int base = carry;
            for (int w = 0; w < 4; ++w) {
                if (w < wave) base += s_wave[w];
                carry += s_wave[w];
            }
            const int first = base + incl - nt;
            if (c < Cq) cl_first[(size_t)h * Cq + c] = first;
            if (nt <= PLAN_OWN)
                for (int t = 0; t < nt; ++t) tl[first + t] = make_int4(c, start + t * BM, min(BM, size - t * BM), 0);
            for (unsigned long long big = __ballot(nt > PLAN_OWN); big; big &= big - 1) {
                const int src = __builtin_ctzll(big);
                const int bn = __shfl(nt, src), bf = __shfl(first, src), bs = __shfl(start, src), bz = __shfl(size, src);
                for (int t = lane; t < bn; t += 64)
                    tl[bf + t] = make_int4(c - lane + src, bs + t * BM, min(BM, bz - t * BM), 0);
            }
        }
        if (tid == 0) n_tiles[h] = carry;
        return;
    }

    // runs: one wavefront per CSR row, 64 entries per pass
    const int i = ((int)blockIdx.x - 1) * 4 + wave;
    if (i >= Cq) return;
    const int32_t *ok = offsets_k + (size_t)h * (Ck + 1);
    const int32_t *rp = row_ptr + (size_t)h * (Cq + 1);
    const int32_t *ci = col_idx + (size_t)h * Cq * Ck;
    int2 *rn = runs + (size_t)h * Cq * Ck;
    int32_t *tr = tile_run + ((size_t)h * Cq + i) * key_tiles;
    const int e0 = rp[i], e1 = rp[i + 1];
    int carry = 0;
    for (int e = e0; e < e1; e += 64) {
        const int idx = e + lane;
        int start = 0, len = 0;
        if (idx < e1) {
            const int j = ci[idx];
            start = ok[j];
            len = ok[j + 1] - start;
        }
        int incl = len;
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(incl, o);
            if (lane >= o) incl += v;
        }
        const int before = carry + incl - len;          // keys of the row in front of this run
        if (idx < e1) rn[idx] = make_int2(start, before);
        // the 64-key tiles whose first key lies in this run start their row look-up here
        const int t0 = (before + ATT_BN - 1) / ATT_BN;
        const int t1 = min((before + len + ATT_BN - 1) / ATT_BN, key_tiles);
        if (t1 - t0 <= PLAN_OWN)
            for (int t = t0; t < t1; ++t) tr[t] = idx - e0;
        for (unsigned long long big = __ballot(t1 - t0 > PLAN_OWN); big; big &= big - 1) {
            const int src = __builtin_ctzll(big);
            const int b0 = __shfl(t0, src), b1 = __shfl(t1, src);
            for (int t = b0 + lane; t < b1; t += 64) tr[t] = e - e0 + src;
        }
        carry += __shfl(incl, 63);
    }
    if (lane == 0) row_keys[(size_t)h * Cq + i] = carry;
}

// tile_base[h] = number of tiles of heads < h, tile_base[H] = all tiles; and
// order[0 .. all tiles): the work items sorted by decreasing number of key tiles (longest first), so that the
// last workgroups of a launch are short ones.  The tiles of one query cluster stay together (they read the
// same keys); among clusters of equal length the order is whatever the atomics give -- it only decides when a
// work item runs, never what it computes.  One workgroup; with more clusters than ORD_MAX_CLUSTERS the list
// keeps its head-major order.  What bounds it is round trips to memory, so a thread requests what it needs of ORD_UB clusters
// together, keeps it between counting and placing, and the tiles of a cluster of more than ORD_OWN are written by the whole
// wavefront (of every cluster: 28 instead of 22 us at 24 heads of 118,800).  One cluster of a thread at a time, counted and placed
// from memory, and a scan with twenty barriers took 10.1 instead of 7.9 us at 24 heads of 16,384 tokens in 100 clusters, 34.5 instead
// of 23.6 us at 40 heads of 75,600.
static constexpr int ORD_BUCKETS = 2048;
static constexpr int ORD_MAX_CLUSTERS = 1 << 20;
static constexpr int ORD_UB = 4;                // clusters of a thread at a time
static constexpr int ORD_OWN = 96;              // tiles of a cluster that its thread writes by itself

// exclusive prefix sum over 1024 threads; *total = sum of all
__device__ __forceinline__ int ord_scan(int v, int32_t *s_wave, int *total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int incl = v;
    for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(incl, o);
        if (lane >= o) incl += u;
    }
    __syncthreads();                            // s_wave of an earlier call has been read
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
        const int u = s_wave[w];
        before += w < wave ? u : 0;
        all += u;
    }
    *total = all;
    return before + incl - v;
}

// Range of the K and V values of a head (fp32 storage), for the rule that lets the attention kernel split them (below), of |x| as
// bits, so that a NaN or an infinity is above every number:
//   [0], [1]  largest of K, of V         [2], [3]  minus the smallest of K, of V, zeros left out (0: zeros alone)
// Workgroups 1 .. of the order kernel's launch, RANGE_PASSES rows per row slot: one pass over K and V next to the one workgroup
// that sorts the list, which takes longer.
static constexpr int RANGE_PASSES = 4;
__device__ __forceinline__ void f32_range(unsigned bits, unsigned &most, unsigned &least)
{
    const unsigned b = bits & 0x7FFFFFFFu;
    most = max(most, b);
    least = max(least, 0u - b);
}
static inline int attn_range_blocks(int H, int N, int d) { return 2 * H * cdiv(N, RANGE_PASSES * (1024 / (d / 4))); }

__device__ __forceinline__ void attn_range(int blk, const float *__restrict__ K, const float *__restrict__ V, int H, int N, int d,
                                           unsigned *__restrict__ range, unsigned *s_max)
{
    const int tid = threadIdx.x, lpr = d / 4, step = 1024 / lpr, nb = (N + RANGE_PASSES * step - 1) / (RANGE_PASSES * step);
    const int side = blk / (H * nb), h = blk / nb % H, r0 = blk % nb * RANGE_PASSES * step;
    const uint4 *X = reinterpret_cast<const uint4 *>((side ? V : K) + (size_t)h * N * d);
    if (tid < 2) s_max[tid] = 0;
    __syncthreads();
    uint4 v[RANGE_PASSES];
#pragma unroll
    for (int p = 0; p < RANGE_PASSES; ++p) v[p] = X[(size_t)min(r0 + p * step + tid / lpr, N - 1) * lpr + tid % lpr];
    unsigned most = 0, least = 0;               // least: minus the smallest
#pragma unroll
    for (int p = 0; p < RANGE_PASSES; ++p) {
        f32_range(v[p].x, most, least); f32_range(v[p].y, most, least);
        f32_range(v[p].z, most, least); f32_range(v[p].w, most, least);
    }
    for (int o = 32; o > 0; o >>= 1) {
        most = max(most, (unsigned)__shfl_xor((int)most, o));
        least = max(least, (unsigned)__shfl_xor((int)least, o));
    }
    if ((tid & 63) == 0) { atomicMax(&s_max[0], most); atomicMax(&s_max[1], least); }
    __syncthreads();
    if (tid < 2) atomicMax(&range[(size_t)h * F32_RANGE + 2 * tid + side], s_max[tid]);
}

__global__ __launch_bounds__(1024) void attn_order_kernel(const int32_t *__restrict__ offsets_q,
                                                          const int32_t *__restrict__ n_tiles, int32_t *tile_base,
                                                          const int32_t *__restrict__ row_keys,
                                                          const int32_t *__restrict__ cl_first, int H, int Cq, int BM,
                                                          int32_t *__restrict__ order, const float *__restrict__ K,
                                                          const float *__restrict__ V, int N, int d, unsigned *__restrict__ range)
{
    __shared__ int32_t s_cnt[ORD_BUCKETS];
    __shared__ int32_t s_wave[16];
    if (blockIdx.x > 0) {                       // (fp32 storage only)
        attn_range((int)blockIdx.x - 1, K, V, H, N, d, range, reinterpret_cast<unsigned *>(s_cnt));
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63;
    for (int b = tid; b < ORD_BUCKETS; b += 1024) s_cnt[b] = 0;
    int all = 0;
    for (int h0 = 0; h0 < H; h0 += 1024) {
        const int h = h0 + tid;
        int sum;
        const int before = ord_scan(h < H ? n_tiles[h] : 0, s_wave, &sum);
        if (h < H) tile_base[h] = all + before;
        all += sum;
    }
    if (tid == 0) tile_base[H] = all;
    __syncthreads();                            // tile_base is read by other threads of this workgroup below
    const long long ncl = (long long)H * Cq;
    if (ncl > ORD_MAX_CLUSTERS) {
        for (int v = tid; v < all; v += 1024) order[v] = v;
        return;
    }
    // clusters i0 + tid + 1024 u: tiles, bucket (the one with the most key tiles is bucket 0), first tile in head-major order
    struct Cluster { int nt, bucket, first; };
    Cluster c[ORD_UB];
    auto load = [&](int i0) {
        int kt[ORD_UB], q0[ORD_UB], q1[ORD_UB], tb[ORD_UB], cf[ORD_UB];
#pragma unroll
        for (int u = 0; u < ORD_UB; ++u) {
            const int i = min(i0 + tid + 1024 * u, (int)ncl - 1), h = i / Cq;
            const int32_t *oq = offsets_q + (size_t)i + h;              // [H][Cq + 1]
            kt[u] = row_keys[i];
            q0[u] = oq[0];
            q1[u] = oq[1];
            tb[u] = tile_base[h];
            cf[u] = cl_first[i];
        }
#pragma unroll
        for (int u = 0; u < ORD_UB; ++u) {
            c[u].nt = i0 + tid + 1024 * u < ncl ? (q1[u] - q0[u] + BM - 1) / BM : 0;
            c[u].bucket = ORD_BUCKETS - 1 - min((kt[u] + ATT_BN - 1) / ATT_BN, ORD_BUCKETS - 1);
            c[u].first = tb[u] + cf[u];
        }
    };
    for (int i0 = 0; i0 < (int)ncl; i0 += 1024 * ORD_UB) {
        load(i0);
#pragma unroll
        for (int u = 0; u < ORD_UB; ++u)
            if (c[u].nt > 0) atomicAdd(&s_cnt[c[u].bucket], c[u].nt);
    }
    __syncthreads();
    {
        static_assert(ORD_BUCKETS == 2048, "two buckets per thread");
        const int a0 = s_cnt[2 * tid], a1 = s_cnt[2 * tid + 1];
        int sum;
        const int excl = ord_scan(a0 + a1, s_wave, &sum);
        s_cnt[2 * tid] = excl;
        s_cnt[2 * tid + 1] = excl + a0;
    }
    __syncthreads();
    for (int i0 = 0; i0 < (int)ncl; i0 += 1024 * ORD_UB) {
        if (ncl > 1024 * ORD_UB) load(i0);      // (else: what was loaded for the counting)
#pragma unroll
        for (int u = 0; u < ORD_UB; ++u) {
            const int nt = c[u].nt, pos = nt > 0 ? atomicAdd(&s_cnt[c[u].bucket], nt) : 0;
            if (nt <= ORD_OWN)
                for (int t = 0; t < nt; ++t) order[pos + t] = c[u].first + t;
            for (unsigned long long big = __ballot(nt > ORD_OWN); big; big &= big - 1) {
                const int src = __builtin_ctzll(big);
                const int bn = __shfl(nt, src), bp = __shfl(pos, src), bf = __shfl(c[u].first, src);
                for (int t = lane; t < bn; t += 64) order[bp + t] = bf + t;
            }
        }
    }
}

// ---------------------------------------------------------------- bf16 MFMA kernel

// acc + both bf16 halves of w (v_dot2c_f32_bf16 with a vector of ones): the row sum is taken
// over the rounded probabilities, the same values the matrix cores multiply with V
__device__ __forceinline__ float add_bf16x2(unsigned w, float acc)
{
    bf16x2 x;
    __builtin_memcpy(&x, &w, 4);
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
    return __builtin_amdgcn_fdot2_f32_bf16(x, ones, acc, false);
}

// RUN_CAP: the launch was sized for at most ATT_RUN_LDS runs in LDS (more than that many key clusters); a work item
// with more runs then reads them from global memory.  Without it the table always fits and that path does not exist.
// At D = 64 a third workgroup fits a CU as long as a wavefront takes 168 registers at most (the compiler takes 154): dense
// attention of 20 heads of 4000 tokens took 138 us with 183 registers and two workgroups, 118 now.
template <int D, bool RUN_CAP>
__global__ __launch_bounds__(64 * ATT_NW, D == 64 ? 3 : 2) void attn_bf16_kernel(
    const bf16_t *__restrict__ Q, const bf16_t *__restrict__ K, const bf16_t *__restrict__ V, int H, int N, int Cq,
    int Ck, const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ perm_q,
    const int32_t *__restrict__ perm_k, const int4 *__restrict__ tiles, const int32_t *__restrict__ tile_base,
    const int32_t *__restrict__ order, int max_tiles,
    const int2 *__restrict__ runs, const int32_t *__restrict__ row_keys, const int32_t *__restrict__ tile_run,
    int key_tiles, float scale_log2, int group, bf16_t *__restrict__ O, float *__restrict__ lse)
{
    constexpr int KS = D / 16;                 // k-steps of QK^T
    constexpr int DVB = D / 32;                // 32-row blocks of O^T
    constexpr int RB = 2 * D;                  // bytes per K / V row
    constexpr int CPR = D / 8;                 // 16-byte chunks per row
    constexpr int RPI = 1024 / RB;             // rows one direct-to-LDS load instruction fills (64 lanes x 16 B)
    constexpr int NW = ATT_NW, NSTG = ATT_NSTG;
    constexpr int NPASS = ATT_BN / (NW * RPI); // such instructions per wavefront, tile and tensor
    static_assert(NPASS >= 1, "a tile needs at least one load instruction per wavefront");
    constexpr int TILE_B = ATT_BN * RB;        // bytes of one K or V tile in LDS

    // LDS: K tiles [NSTG][64][D] and V tiles [NSTG][64][D], rows unpadded (the direct loads
    // fill 1024 contiguous bytes per instruction); bank conflicts are avoided by
    // storing 16-byte chunk c of row r at position c ^ swz(r):
    //   K  swz = (r / (256 / RB)) % CPR        the 16 rows of one ds_read_b128 pass differ
    //   V  swz = 4 * ((r / (256 / RB)) % (CPR / 4))   the 4 rows of one transposing pass differ
    extern __shared__ __align__(16) unsigned char s_raw[];
    unsigned char *sK = s_raw;                                      // [NSTG][TILE_B]
    unsigned char *sV = s_raw + NSTG * TILE_B;                      // [NSTG][TILE_B]
    int32_t *s_rows = reinterpret_cast<int32_t *>(s_raw + 2 * NSTG * TILE_B);   // [2][64]
    int2 *s_run = reinterpret_cast<int2 *>(s_rows + 2 * ATT_BN);    // [nnz + 1]

    // ---- which work item.  All tiles of all heads form one list; tiles that share keys are neighbours in it and share
    // an L2, and every XCD gets the same amount of work whatever the per-head densities are.
    const int pos = attn_list_pos(group);
    if (pos >= tile_base[H]) return;
    const int v = order[pos];                   // longest work items first (attn_order_kernel)
    int h = 0;
    for (int step = 1 << 15; step > 0; step >>= 1)
        if (h + step < H && tile_base[h + step] <= v) h += step;
    const int t = v - tile_base[h];
    const int4 desc = tiles[(size_t)h * max_tiles + t];
    const int ci = desc.x, row0 = desc.y, nrows = desc.z;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // wavefront-uniform: lives in a scalar register
    const int half = lane >> 5, col = lane & 31;

    const int e0 = row_ptr[(size_t)h * (Cq + 1) + ci];
    const int nnz = row_ptr[(size_t)h * (Cq + 1) + ci + 1] - e0;
    const int L = row_keys[(size_t)h * Cq + ci];
    const int2 *rn = runs + (size_t)h * Cq * Ck + e0;
    const int32_t *trh = tile_run + ((size_t)h * Cq + ci) * key_tiles;      // run in which each key tile starts
    // The run table of the work item (nnz entries + a closing one) is staged in LDS when it fits the share of LDS
    // that still lets two workgroups run on a CU; a query cluster that selects more key clusters than that reads
    // its runs from global memory (slow look-ups, same result).
    const bool runs_in_lds = !RUN_CAP || nnz + 1 <= ATT_RUN_LDS;
    if (runs_in_lds) {
        for (int e = tid; e < nnz; e += 64 * NW) s_run[e] = rn[e];
        if (tid == 0) s_run[nnz] = make_int2(0, L);
    }
    auto run_at = [&](int c) -> int2 {
        if (!RUN_CAP || runs_in_lds) return s_run[c];
        return c < nnz ? rn[c] : make_int2(0, L);
    };

    const bf16_t *Qh = Q + (size_t)h * N * D;
    const bf16_t *Kh = K + (size_t)h * N * D;
    const bf16_t *Vh = V + (size_t)h * N * D;

    // ---- queries as the B operand of S^T = K Q^T: this wavefront owns 32 rows of the tile
    bf16x8 qreg[KS];
    {
        int r = row0 + min(nrows - 1, wave * 32 + col);
        if (perm_k) r = perm_q[(size_t)h * N + r];      // gather-free: Q is in token order
        const uint4 *src = reinterpret_cast<const uint4 *>(Qh + (size_t)r * D + 8 * half);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const uint4 w = src[2 * s];
            __builtin_memcpy(&qreg[s], &w, 16);
        }
    }
    const bool wave_active = wave * 32 < nrows;

    f32x16 oacc[DVB];
    float m_run = -INFINITY, l_run = 0.f;
#pragma unroll
    for (int b = 0; b < DVB; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[b][i] = 0.f;

    // ---- loader.  The permuted K / V row of every key slot of a tile is looked up by
    // ONE wavefront (wave kt % NW, lane = slot) ahead of time and parked in s_rows.  The
    // rows then go from global memory straight into LDS (no staging registers): load
    // instruction (wave, p) fills LDS rows (NW p + wave) * RPI .. + RPI of the tile, lane l
    // the chunk position l % CPR of row l / CPR, so it fetches the global chunk that the
    // swizzle puts there.  K tiles are fetched two tiles ahead of their use and V tiles
    // one tile ahead (see the schedule below), so the byte offsets of a tile's rows are
    // kept in registers from its K fetch to its V fetch.
    const char *Kb = reinterpret_cast<const char *>(Kh);
    const char *Vb = reinterpret_cast<const char *>(Vh);
    const int32_t *pkh = perm_k ? perm_k + (size_t)h * N : nullptr;
    int cur = 0;                                // per-lane cursor into the run table, only moves forward
    int lk_hint = -1;                           // run in which the tile looked up next starts (-1: not known)
    const int ld_row = lane / CPR;                                  // row inside the instruction's group
    const int ld_swz = ((wave * RPI + ld_row) / (256 / RB));
    const unsigned ld_koff = (unsigned)(((lane % CPR) ^ (ld_swz % CPR)) * 16);
    const unsigned ld_voff = (unsigned)(((lane % CPR) ^ (4 * (ld_swz % (CPR / 4)))) * 16);
    __syncthreads();                            // s_run visible

#define ATT_ROWS(KT)                                                                       \
    if (wave == ((KT) & (NW - 1))) {                                                       \
        const int kk = (KT) * ATT_BN + lane;                                               \
        int row_ = 0;                                                                      \
        if (kk < L) {                                                                      \
            while (kk >= run_at(cur + 1).y) ++cur;                                         \
            const int2 rs_ = run_at(cur);                                                  \
            row_ = rs_.x + kk - rs_.y;                                                     \
        }                                                                                  \
        if (perm_k) {                           /* gather-free: sorted row -> token */     \
            row_ = pkh[row_];                                                              \
            asm volatile("" : "+v"(row_));      /* the wait for this load stays inside the branch */ \
        }                                                                                  \
        s_rows[((KT) & 1) * ATT_BN + lane] = row_ * RB;     /* byte offset of the row */   \
    }
// second and third step of the look-up of a tile's rows (first step: lk_rs_ = s_run[cur], lk_nb_ = start of the next run)
#define ATT_LOOKUP_FINISH(KT)                                                              \
    {                                                                                      \
        const int kk = (KT) * ATT_BN + lane;                                               \
        if (kk < L) {                                                                      \
            while (kk >= lk_nb_) {                                                         \
                ++cur;                                                                     \
                lk_rs_ = run_at(cur);                                                      \
                lk_nb_ = run_at(cur + 1).y;                                                \
            }                                                                              \
            lk_row_ = lk_rs_.x + kk - lk_rs_.y;                                            \
        }                                                                                  \
        if (perm_k) lk_row_ = pkh[lk_row_];     /* gather-free: sorted row -> token */     \
    }
#define ATT_LOOKUP_STORE(KT)                                                               \
    {                                                                                      \
        asm volatile("" : "+v"(lk_row_));       /* the value is first touched here, so the wait for it comes here */ \
        s_rows[((KT) & 1) * ATT_BN + lane] = lk_row_ * RB;                                 \
    }
#define ATT_OFFS(KT, OFF)                                                                  \
    _Pragma("unroll") for (int p_ = 0; p_ < NPASS; ++p_)                                   \
        OFF[p_] = (unsigned)s_rows[((KT) & 1) * ATT_BN + (NW * p_ + wave) * RPI + ld_row];
#define ATT_FETCH(OFF, SRC, LOFF, DST)                                                     \
    _Pragma("unroll") for (int p_ = 0; p_ < NPASS; ++p_)                                   \
        load_to_lds_16(SRC, OFF[p_] + LOFF, DST + ((NW * p_ + wave) * RPI) * RB);

// one load instruction (pass P) of a tile: DSTB = byte offset of the tile's buffer in LDS
#define ATT_FETCH1(P, OFF, SRC, LOFF, DSTB)                                                \
    load_to_lds_16(SRC, OFF[P] + LOFF, s_raw + (DSTB) + ((NW * (P) + wave) * RPI) * RB);

    const int ntile = (L + ATT_BN - 1) / ATT_BN;
    unsigned off_nx[NPASS];                     // row offsets of the tile whose V is fetched next
    ATT_ROWS(0)
    ATT_ROWS(1)
    __syncthreads();
    if (ntile > 0) {
        ATT_OFFS(0, off_nx)
        ATT_FETCH(off_nx, Kb, ld_koff, sK)
        ATT_FETCH(off_nx, Vb, ld_voff, sV)
    }
    if (ntile > 1) {
        ATT_OFFS(1, off_nx)
        ATT_FETCH(off_nx, Kb, ld_koff, sK + TILE_B)
    }
    __syncthreads();                            // everyone has read the rows of tiles 0 and 1
    if (ntile > 2) { ATT_ROWS(2) }
    if (ntile > 3 && 3 < key_tiles && wave == (3 & (NW - 1))) lk_hint = trh[3];      // tile 3 is looked up during tile 0
    // off_nx stays live: it holds the rows of tile 1, whose V is requested during tile 0
    // per-lane LDS read offsets (bytes, buffer 0): K operand of k-step s, V^T operand of column block b
    int koff[KS], voff[DVB];
    {
        const int kz = (col / (256 / RB)) % CPR;
#pragma unroll
        for (int s = 0; s < KS; ++s) koff[s] = col * RB + (((2 * s + half) ^ kz) * 16);
        const int r16 = lane & 15;
        const int kr0 = 4 * half + (r16 >> 2);
        const int vz = 4 * ((kr0 / (256 / RB)) % (CPR / 4));
        const int cl = 2 * ((lane >> 4) & 1) + ((r16 & 3) >> 1);
#pragma unroll
        for (int b = 0; b < DVB; ++b) voff[b] = kr0 * RB + ((((4 * b) ^ vz) + cl) * 16) + (r16 & 1) * 8;
        // fold the address of the LDS buffer in once and make the sums opaque: otherwise the compiler re-adds the
        // (link-time constant) base in front of every LDS read
        const int lds_base = (int)(unsigned)(size_t)(const lds_u8 *)s_raw;
#pragma unroll
        for (int s = 0; s < KS; ++s) { koff[s] += lds_base; asm volatile("" : "+v"(koff[s])); }
#pragma unroll
        for (int b = 0; b < DVB; ++b) { voff[b] += lds_base; asm volatile("" : "+v"(voff[b])); }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);         // vmcnt(0): queries and the first tiles have landed
    __syncthreads();

    // ---- schedule.  The key sequence is consumed in blocks of 32 keys (two per 64-key
    // tile).  Per block j the work is S_j = K_j Q^T (KS matrix instructions),
    // P_j = exp2(S_j - m) (vector ALU, 6 operations per pair of scores: two fma,
    // two exp2, one pack to bf16, one row-sum dot) and O^T += V_j^T P_j^T (NPV matrix
    // instructions).  The blocks are software-pipelined so that every matrix instruction
    // has about the same amount of independent vector work in its shadow:
    //
    //   phase A(j):  S_{j+1} = K_{j+1} Q^T   ||  last two thirds of P_j, LDS reads of V_j^T
    //   phase B(j):  O^T += V_j^T P_j^T      ||  first third of P_{j+1}, LDS reads of K_{j+2}
    //
    // The instruction stream is laid out by hand (ATT_FENCE keeps the compiler from moving
    // code across chunk boundaries).  The reference level m of a query is the maximum of its
    // first score block; it only moves to a block maximum more than 2^8 above it (ATT_LEVEL_LOG2),
    // which is looked for at the end of phase A, before the block is accumulated, if the block's
    // sum says that there may be one.
    // Accumulator i of a block is key 8 (i/4) + 4 half + i%4.
    //
    // Tile t lives in K buffer t % 2 and V buffer t % 2.  One barrier per tile: at the top of
    // tile t every wavefront has finished tile t - 1 and all fetches issued during tile t - 1
    // have landed.  V_{t+1} and K_{t+2} are requested during tile t (K is read one and a half
    // blocks ahead of V, so it is fetched a tile earlier): the V loads one by one after every
    // other matrix instruction of the first phase A, the K loads likewise in the first phase B.
    // Issued in one burst at the top of the tile, the load instructions of all wavefronts of a
    // CU queue up behind each other (a CU accepts one 1 KB load per ~17 cycles) while no matrix
    // instruction is in flight.  The rows of tile t + 3 are looked up by one wavefront in three
    // steps between the phases (request the run, resolve it, park the row offsets in s_rows), so
    // that neither the LDS latency nor the latency of the gathered index is waited for.
#define ATT_FENCE __builtin_amdgcn_sched_barrier(0);
// An empty volatile asm that "modifies" a value: the value has to exist at this point of the
// program, so optimisation passes that work above the instruction scheduler cannot sink the
// vector work out of the chunk it was written in.
#define ATT_PIN(X) asm volatile("" : "+v"(X));
    constexpr int NPV = 2 * DVB;
    constexpr int NOPS = 48;                    // vector operations of one block's probabilities
    constexpr int OPS_B = ATT_OPS_B;            // of which phase B (of the block before) does the first OPS_B
    const lds_u8 *lds = (const lds_u8 *)0;      // koff / voff are complete LDS addresses
    f32x16 s0, s1;                              // scores of block 0 / block 1 of a tile
    unsigned pw0[8], pw1[8];                    // probabilities of block 0 / block 1, two bf16 per word
    bf16x8 ka[KS], va[NPV];                     // K operands of the next score block, V^T operands of this one
    float psum = 0.f, t0 = 0.f, t1 = 0.f;

    // operation `op` (0..47) of the probabilities of one block: S -> pw
    auto exp_op = [&](const f32x16 &S, unsigned *pw, int op) {
        const int e = op / 6, k = op % 6;
        if (k == 0) { t0 = fmaf(S[2 * e], scale_log2, -m_run); ATT_PIN(t0) }
        else if (k == 1) { t1 = fmaf(S[2 * e + 1], scale_log2, -m_run); ATT_PIN(t1) }
        else if (k == 2) { t0 = __builtin_amdgcn_exp2f(t0); ATT_PIN(t0) }
        else if (k == 3) { t1 = __builtin_amdgcn_exp2f(t1); ATT_PIN(t1) }
        else if (k == 4) { pw[e] = pack_bf16x2(t0, t1); ATT_PIN(pw[e]) }
        else { psum = add_bf16x2(pw[e], psum); ATT_PIN(psum) }
    };
    auto mask_block = [&](f32x16 &S, int base, int rem) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if (base + 8 * (i >> 2) + 4 * half + (i & 3) >= rem) S[i] = -INFINITY;
    };
    // Sum of a block's probabilities 2^8 or more, infinite or not a number: take the level of every query whose block
    // maximum is more than 2^8 above it up to that maximum, bring the accumulators along and form the block's
    // probabilities again.  S still holds the scores, and the block has not been accumulated yet.
    auto relevel = [&](const f32x16 &S, unsigned *pw) {
        float mx = fmaxf(S[0], S[1]);
#pragma unroll
        for (int i = 2; i < 16; ++i) mx = fmaxf(mx, S[i]);
        const float mx_s = max_xor32(mx) * scale_log2;
        const bool upd = mx_s > m_run + ATT_LEVEL_LOG2;
        if (!__any(upd)) return;
        const float m_new = upd ? mx_s : m_run;
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
        m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int b = 0; b < DVB; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) oacc[b][i] *= alpha;
        psum = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            pw[e] = pack_bf16x2(__builtin_amdgcn_exp2f(fmaf(S[2 * e], scale_log2, -m_run)),
                                __builtin_amdgcn_exp2f(fmaf(S[2 * e + 1], scale_log2, -m_run)));
            psum = add_bf16x2(pw[e], psum);
        }
    };
    // K operands of a score block: KBYTE = byte offset of the block's first row in LDS
    auto load_k = [&](auto kbyte_tag, int s) {
        constexpr int KBYTE = decltype(kbyte_tag)::value;
        const u32x4 w = lds_read_b128((lds + koff[s]) + KBYTE);
        __builtin_memcpy(&ka[s], &w, 16);
    };
    // V^T operand idx of a block (ks = idx / DVB: 16 keys, b = idx % DVB: 32 output columns)
    auto load_v = [&](auto vbyte_tag, int idx) {
        constexpr int VBYTE = decltype(vbyte_tag)::value;
        const int ks = idx / DVB, b = idx % DVB;
        const s16x4 lo = lds_read_tr16((lds + voff[b]) + (VBYTE + (ks * 16) * RB));
        const s16x4 hi = lds_read_tr16((lds + voff[b]) + (VBYTE + (ks * 16 + 8) * RB));
        __builtin_memcpy(&va[idx], &lo, 8);
        __builtin_memcpy(reinterpret_cast<char *>(&va[idx]) + 8, &hi, 8);
    };
    // phase A: Sacc = K Q^T from ka[] (if DO_S)  ||  operations OPS_B..47 of pw = exp2(Sexp - m), V^T operands from
    // VBYTE, the check of the block's sum
    auto phase_a = [&](auto do_s_tag, auto vbyte_tag, auto vfetch_tag, f32x16 &Sacc, const f32x16 &Sexp, unsigned *pw) {
        constexpr bool DO_S = decltype(do_s_tag)::value;
        constexpr int VFETCH = decltype(vfetch_tag)::value;     // >= 0: LDS byte offset of the V buffer to fill
        constexpr int KPF = KS / NPASS;                         // k-steps per load instruction
        bool high = false;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            if (DO_S) {
                if (s == 0) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) Sacc[i] = 0.f;
                }
                Sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[s], qreg[s], Sacc, 0, 0, 0);
            }
            ATT_FENCE
#pragma unroll
            for (int idx = (2 * NPV * s) / KS; idx < (2 * NPV * (s + 1)) / KS && idx < NPV; ++idx)
                load_v(vbyte_tag, idx);         // all issued in the first half, so they have landed by phase B
#pragma unroll
            for (int op = OPS_B + ((NOPS - OPS_B) * s) / (KS - 1);
                 op < OPS_B + ((NOPS - OPS_B) * (s + 1)) / (KS - 1) && op < NOPS; ++op)
                exp_op(Sexp, pw, op);
            // compared in front of the last matrix instruction, branched on behind it
            if (s == KS - 2) high = __any(!(psum < ATT_LEVEL_SUM));
            if constexpr (VFETCH >= 0) {
                if (s % KPF == KPF - 1) { ATT_FETCH1(s / KPF, off_nx, Vb, ld_voff, VFETCH) }
            }
            ATT_FENCE
        }
        if (__builtin_expect(high, 0)) relevel(Sexp, pw);       // rare
        l_run += psum;
        psum = 0.f;
    };
    // phase B: O^T += V^T P^T from va[] and pr[]  ||  operations 0..OPS_B-1 of pn = exp2(Snext - m) (if DO_P); K operands
    // of the block after Snext from KBYTE (if DO_K)
    auto phase_b = [&](auto do_p_tag, auto do_k_tag, auto kbyte_tag, auto kfetch_tag, auto slot_tag, bool do_kfetch,
                       const unsigned *pr, const f32x16 &Snext, unsigned *pn) {
        constexpr bool DO_P = decltype(do_p_tag)::value;
        constexpr bool DO_K = decltype(do_k_tag)::value;
        constexpr int KFETCH = decltype(kfetch_tag)::value;     // >= 0: LDS byte offset of the K buffer to fill
        constexpr int SLOT = decltype(slot_tag)::value;         // which half of s_rows holds that tile's rows
        constexpr int KF0 = NPV / 4;                            // first matrix instruction followed by a load
#pragma unroll
        for (int idx = 0; idx < NPV; ++idx) {
            bf16x8 pb;
            __builtin_memcpy(&pb, pr + 4 * (idx / DVB), 16);
            oacc[idx % DVB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[idx], pb, oacc[idx % DVB], 0, 0, 0);
            ATT_FENCE
            if (DO_K) {
#pragma unroll
                for (int s = (KS * idx) / NPV; s < (KS * (idx + 1)) / NPV; ++s) load_k(kbyte_tag, s);
            }
            if (DO_P && idx > 0) {
#pragma unroll
                for (int op = OPS_B * (idx - 1) / (NPV - 1); op < OPS_B * idx / (NPV - 1); ++op) exp_op(Snext, pn, op);
            }
            if constexpr (KFETCH >= 0) {
                if (do_kfetch) {
                    if (idx == 0) {
#pragma unroll
                        for (int p_ = 0; p_ < NPASS; ++p_)
                            off_nx[p_] = (unsigned)s_rows[SLOT * ATT_BN + (NW * p_ + wave) * RPI + ld_row];
                    }
                    if (idx >= KF0 && idx < KF0 + NPASS) { ATT_FETCH1(idx - KF0, off_nx, Kb, ld_koff, KFETCH) }
                }
            }
            ATT_FENCE
        }
    };
    using T = std::true_type;

    // ---- prologue: S of block 0 of tile 0, its maximum, the first third of its probabilities,
    // K operands of block 1
    if (wave_active && ntile > 0) {
#pragma unroll
        for (int s = 0; s < KS; ++s) load_k(std::integral_constant<int, 0>{}, s);
#pragma unroll
        for (int i = 0; i < 16; ++i) s0[i] = 0.f;
#pragma unroll
        for (int s = 0; s < KS; ++s) s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[s], qreg[s], s0, 0, 0, 0);
#pragma unroll
        for (int s = 0; s < KS; ++s) load_k(std::integral_constant<int, 32 * RB>{}, s);
        if (L < 32) mask_block(s0, 0, L);
        float mx = fmaxf(s0[0], s0[1]);
#pragma unroll
        for (int i = 2; i < 16; ++i) mx = fmaxf(mx, s0[i]);
        m_run = max_xor32(mx) * scale_log2;     // key 0 exists, so the maximum is finite
#pragma unroll
        for (int op = 0; op < OPS_B; ++op) exp_op(s0, pw0, op);
    }

    // One tile: tile kt sits in K / V buffer BUF = kt % NSTG.  HAS_NEXT: tile kt + 1 exists.
    // At the top, the fetches issued during the tile before (V of this tile, K of the next) must
    // have landed.
#define ATT_TILE(BUF, HAS_NEXT)                                                            \
    {                                                                                      \
        __builtin_amdgcn_s_waitcnt(0x0F70);     /* vmcnt(0) */                             \
        __syncthreads();                                                                   \
        /* fetches of this tile: V of the next tile (it exists: HAS_NEXT) into the other V buffer, K of the  \
           tile after it into this tile's K buffer; spread over the first two phases so that the load        \
           instructions of the wavefronts of a CU do not queue up behind each other at the top of a tile */  \
        constexpr int VF_ = HAS_NEXT ? NSTG * TILE_B + ((BUF + 1) % NSTG) * TILE_B : -1;   \
        constexpr int KF_ = HAS_NEXT ? BUF * TILE_B : -1;                                  \
        const bool do_kf_ = HAS_NEXT && kt + NSTG < ntile;                                 \
        /* rows of tile kt + 3 (needed by the K fetch of the next tile): one wavefront looks them up, in   \
           three steps between the phases so that the LDS and memory latencies are not waited for */     \
        const bool lk_ = HAS_NEXT && kt + NSTG + 1 < ntile && wave == ((kt + NSTG + 1) & (NW - 1)); \
        int2 lk_rs_ = make_int2(0, 0);                                                     \
        int lk_nb_ = 0, lk_row_ = 0;                                                       \
        if (lk_) {                                                                         \
            cur = max(cur, lk_hint);            /* start at the tile's first run, not where this lane was 4 tiles ago */ \
            lk_rs_ = run_at(cur);                                                          \
            lk_nb_ = run_at(cur + 1).y;                                                    \
        }                                                                                  \
        if (wave_active) {                                                                 \
            using HN = std::integral_constant<bool, HAS_NEXT>;                             \
            constexpr int KB_ = ((BUF + 1) % NSTG) * TILE_B, VB_ = NSTG * TILE_B + BUF * TILE_B; \
            phase_a(T{}, std::integral_constant<int, VB_>{}, std::integral_constant<int, VF_>{}, s1, s0, pw0); \
            if (!HAS_NEXT) mask_block(s1, 32, L - kt * ATT_BN);                            \
            if (lk_) { ATT_LOOKUP_FINISH(kt + NSTG + 1) }                                  \
            phase_b(T{}, HN{}, std::integral_constant<int, KB_>{}, std::integral_constant<int, KF_>{}, \
                    std::integral_constant<int, BUF>{}, do_kf_, pw0, s1, pw1);             \
            phase_a(HN{}, std::integral_constant<int, VB_ + 32 * RB>{}, std::integral_constant<int, -1>{}, s0, s1, pw1); \
            if (HAS_NEXT && kt + 2 == ntile && L - (kt + 1) * ATT_BN < 32)                 \
                mask_block(s0, 0, L - (kt + 1) * ATT_BN);                                  \
            phase_b(HN{}, HN{}, std::integral_constant<int, KB_ + 32 * RB>{}, std::integral_constant<int, -1>{}, \
                    std::integral_constant<int, 0>{}, false, pw1, s0, pw0);                \
            /* stored at the end of the tile: the wait for the gathered index (all loads: the compiler  \
               does not know which are outstanding) then falls together with the one at the top */      \
            if (lk_) { ATT_LOOKUP_STORE(kt + NSTG + 1) }                                   \
        } else if (HAS_NEXT) {      /* a wavefront without query rows still loads its share of the tiles */ \
            ATT_FETCH(off_nx, Vb, ld_voff, sV + ((BUF + NSTG - 1) % NSTG) * TILE_B)        \
            if (do_kf_) {                                                                  \
                ATT_OFFS(kt + NSTG, off_nx)                                                \
                ATT_FETCH(off_nx, Kb, ld_koff, sK + BUF * TILE_B)                          \
            }                                                                              \
            if (lk_) {                                                                     \
                ATT_LOOKUP_FINISH(kt + NSTG + 1)                                           \
                ATT_LOOKUP_STORE(kt + NSTG + 1)                                            \
            }                                                                              \
        }                                                                                  \
        /* where the tile that the next tile looks up starts (from the plan, global memory): requested here, \
           used behind the wait at the top of the next tile */                                              \
        {                                                                                  \
            const int tn_ = kt + NSTG + 2;                                                 \
            lk_hint = -1;                                                                  \
            if (HAS_NEXT && tn_ < ntile && tn_ < key_tiles && wave == (tn_ & (NW - 1))) lk_hint = trh[tn_]; \
        }                                                                                  \
        ++kt;                                                                              \
    }
    static_assert(NSTG == 2, "the fetch schedule below is written for two buffers");
    int kt = 0;
    while (kt < ntile - 1) {                    // every tile but the last
        ATT_TILE(0, true)
        if (kt >= ntile - 1) break;
        ATT_TILE(1, true)
    }
    if (ntile > 0) {                            // the last tile: nothing follows it, maybe ragged; one copy for both buffers
        if (kt % NSTG != 0) {
#pragma unroll
            for (int b = 0; b < DVB; ++b) voff[b] += TILE_B;
        }
        ATT_TILE(0, false)
    }
#undef ATT_TILE
#undef ATT_FENCE
#undef ATT_PIN
#undef ATT_ROWS
#undef ATT_OFFS
#undef ATT_LOOKUP_FINISH
#undef ATT_LOOKUP_STORE
#undef ATT_FETCH
#undef ATT_FETCH1

    // ---- epilogue: normalise, store at the original row
    {
        const int rl = wave * 32 + col;
        if (rl < nrows) {
            const int r = row0 + rl;
            const size_t dst = (size_t)h * N + (perm_q ? perm_q[(size_t)h * N + r] : r);
            const float l_tot = sum_xor32(l_run);
            const float inv = (l_tot > 0.f) ? 1.0f / l_tot : 0.f;
#pragma unroll
            for (int b = 0; b < DVB; ++b)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int dv0 = b * 32 + 8 * g + 4 * half;
                    unsigned lo = (unsigned)f32_to_bf16(oacc[b][4 * g + 0] * inv) |
                                  ((unsigned)f32_to_bf16(oacc[b][4 * g + 1] * inv) << 16);
                    unsigned hi = (unsigned)f32_to_bf16(oacc[b][4 * g + 2] * inv) |
                                  ((unsigned)f32_to_bf16(oacc[b][4 * g + 3] * inv) << 16);
                    *reinterpret_cast<uint2 *>(O + dst * D + dv0) = make_uint2(lo, hi);
                }
            if (lse && half == 0)
                lse[dst] = (l_tot > 0.f) ? (m_run + log2f(l_tot)) * 0.6931471805599453f : -INFINITY;
        }
    }
}

// ---------------------------------------------------------------- fp32 kernel
// grid (tile list), block 64 * NW.  A work item is 32 consecutive rows of one query cluster; its key sequence is
// cut into blocks of 32 keys which the wavefronts take in turn (wavefront w: blocks w, w + NW, ..), each with its own
// running softmax over its share of the keys; the shares are put together through LDS at the end.  So a short layer
// (one head of 4096 tokens is 128 work items) still puts work on 512 SIMDs, and no wavefront waits for another
// before the end.  The list runs longest first: 1400 work items of very different lengths on 256 CUs in head-major order
// left the last third of the launch half empty (4 heads of 9601 tokens, d = 128: 0.80 ms, 0.66 ms in this order).  Eight
// wavefronts share a work item rather than four for the small layers, where a CU has one at most (one head of 4096 tokens,
// d = 64: 31 instead of 35 us).
//
// S^T = K Q^T: accumulator i is key 8 (i / 4) + 4 half + i % 4 of query `col`, which is what O^T += V^T P^T wants as its other
// operand.  Row m of output block b is column DVB m + b, so that one load of DVB consecutive floats is the operand of all DVB
// blocks, and the DVB accumulators of a row are consecutive floats of the result.
//
// Operands in three parts (the first of the two loops).  The fp32 instruction takes 13 times as long as the bf16 one for the same
// work, so where the values allow it a value x is taken as the sum of three bf16, each rounded to nearest from what the ones before
// leave: exactly x.  Of the nine products of two operands the six of 2^-17 and more go through the 32x32x16 instruction, the other
// three are below 2^-24 of it, without a common sign.  Small products have an accumulator of their own, the second product of 16 keys is
// summed from zero: added one by one to a long sum, the third parts of V rows that are alike would be rounded away each time (V rows
// all the same, 9601 keys: 8.7e-7 instead of 1.3e-7).  The rule: every K and V value of the head and Q value of the tile is zero or
// between 2^-60 and 2^40 and the scale no more than 2^40, so that no part is subnormal and no sum overflows; infinities, NaN and the rest go
// through the fp32 instruction: the second loop.  Error of O against 64 bits, of the fp32 instruction's, over 600 to 9601 keys, scores of
// deviation 0 to 8, means, channels of any size in Q and K, V rows alike: 0.38 to 0.93, of the log-sum-exp 0.42 to 1.03; with V values of all
// sizes no element further off.  (Two fp16 halves, hi hi + hi lo + lo hi, took 0.41 instead of 0.56 ms below, but lost what lies
// 2^-28 below the largest value of K, of V or of a Q row.)
//
// Time: 4 heads of 9601 tokens in 100 and 500 clusters, D = 128, 31 % selected (58 GFLOP; a seventh of the rows of the 32-row tiles is
// padding) 0.61 -> 0.56 ms with the plan, one head of 4096 at D = 64 38 -> 36 us;
// dense, D = 128, 4 x 9601 1.59 -> 1.39 ms, 2 x 3000 124 -> 103 us.  What bounds the first loop is the vector ALU, 5.5 instructions per
// value for the parts, and the matrix cores behind one another with two wavefronts per SIMD.  K goes by whole
// rows straight to LDS (a wavefront's own 32 rows, fetched while the block before is in its second product) instead of 16 bytes of a row per
// lane, and the rows of a block are found from one load of 64 runs issued a block ahead, not by a walk through memory.  V
// goes to registers, requested in front of the first product; Q, split, is read from LDS, which leaves the registers for that.
// The second loop has K and V in two register buffers each: a 32-key block is 128 matrix instructions (8192 cycles, D = 128), which cover
// its 32 loads.  One query per thread with K and V in LDS took 13.8 ms on the same shape.
// No more wavefronts than a head has key blocks, rounded up to a power of two (5000 heads of 16 tokens, D = 64: 58 us with one,
// 105 with eight), and four instead of eight in short heads that are work items enough without (3000 heads of 100 tokens, 10
// and 20 clusters, a quarter selected: 302 instead of 495 us; 200 of 500, 30 and 60 clusters, D = 128: 208 instead of 276).
static constexpr unsigned F32_LEAST = (127 - 60) << 23, F32_MOST = (127 + 40) << 23;       // 2^-60, 2^40 as bits
static constexpr float F32_SCALE = 1099511627776.f;                                        // 2^40
static constexpr int F32_NW = 8, F32_MANY = 1024, F32_SHORT = 512;
static constexpr int F32_BM = 32;

// elements 2 i and 2 i + 1 of the three parts of a and b; the differences are exact
__device__ __forceinline__ void f32_split3(float a, float b, u32x4 (&part)[3], int i)
{
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        const unsigned w = pack_bf16x2(a, b);
        part[p][i] = w;
        a -= __uint_as_float(w << 16);
        b -= __uint_as_float(w & 0xFFFF0000u);
    }
}

// products of two operands in three parts: large += first parts, small += the others, smallest first
__device__ __forceinline__ void f32_mfma3(const u32x4 (&x)[3], const u32x4 (&y)[3], f32x16 &large, f32x16 &small)
{
    auto mfma = [&](int i, int j, f32x16 &acc) {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x[i]), __builtin_bit_cast(bf16x8, y[j]), acc, 0, 0, 0);
    };
    mfma(2, 0, small);
    mfma(0, 2, small);
    mfma(1, 1, small);
    mfma(1, 0, small);
    mfma(0, 1, small);
    mfma(0, 0, large);
}

template <int D, int NW>
__global__ __launch_bounds__(64 * NW, D == 64 && NW == F32_NW ? 4 : 2) void attn_f32_kernel(
    const float *__restrict__ Q, const float *__restrict__ K, const float *__restrict__ V, int H, int N, int Cq, int Ck,
    const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ perm_q, const int32_t *__restrict__ perm_k,
    const int4 *__restrict__ tiles, const int32_t *__restrict__ tile_base, const int32_t *__restrict__ order, int max_tiles,
    const int2 *__restrict__ runs, const int32_t *__restrict__ row_keys, const int32_t *__restrict__ tile_run,
    int key_tiles, float scale_log2, int group, const unsigned *__restrict__ range, float *__restrict__ O, float *__restrict__ lse)
{
    constexpr int DVB = D / 32;                 // output blocks of 32 columns
    constexpr int NB = D / 16;                  // float4 per register buffer: half of a lane's share of K or V
    constexpr int ROW = D + 4;                  // LDS row of the final sum, padded
    constexpr int RB = D * 4;                   // bytes per row
    typedef float fvec __attribute__((ext_vector_type(DVB)));
    extern __shared__ __align__(16) float s_o[];        // [NW][32][ROW]
    __shared__ float s_m[NW][32], s_l[NW][32];
    // the list of all heads' tiles, longest first, handed out in groups of `group` per XCD (as in the bf16 kernel)
    const int tid = threadIdx.x;
    const int pos = attn_list_pos(group);
    if (pos >= tile_base[H]) return;
    const int v = order[pos];
    int h = 0;
    for (int step = 1 << 15; step > 0; step >>= 1)
        if (h + step < H && tile_base[h + step] <= v) h += step;
    const int4 desc = tiles[(size_t)h * max_tiles + (v - tile_base[h])];
    const int ci = desc.x, row0 = desc.y, nrows = desc.z;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, col = lane & 31;
    const int e0 = row_ptr[(size_t)h * (Cq + 1) + ci];
    const int nnz = row_ptr[(size_t)h * (Cq + 1) + ci + 1] - e0;
    const int L = row_keys[(size_t)h * Cq + ci];
    const int2 *rn = runs + (size_t)h * Cq * Ck + e0;
    const int32_t *trh = tile_run + ((size_t)h * Cq + ci) * key_tiles;
    const int32_t *pkh = perm_k ? perm_k + (size_t)h * N : nullptr;
    const char *Kb = reinterpret_cast<const char *>(K + (size_t)h * N * D);
    const char *Vb = reinterpret_cast<const char *>(V + (size_t)h * N * D);
    const int nblk = (L + 31) / 32;

    int qrow = row0 + min(nrows - 1, col);
    if (perm_k) qrow = perm_q[(size_t)h * N + qrow];    // gather-free: Q is in token order
    const float *Qr = Q + ((size_t)h * N + qrow) * D;
    // Split operands or not: the same for all wavefronts of the work item (same Q rows, same head)
    // split Q in LDS behind the wavefronts' K blocks: lane's part of step t is elements 16 t + 8 half .. of its row
    u32x4 *s_q = reinterpret_cast<u32x4 *>(s_o + (size_t)NW * 32 * D);
    bool split = false;
    if (NW == F32_NW && range) {
        float q[D / 2];
#pragma unroll
        for (int t = 0; t < D / 16; ++t) {
            const float4 *src = reinterpret_cast<const float4 *>(Qr + 16 * t + 8 * half);
            const float4 w0 = src[0], w1 = src[1];
            q[8 * t] = w0.x; q[8 * t + 1] = w0.y; q[8 * t + 2] = w0.z; q[8 * t + 3] = w0.w;
            q[8 * t + 4] = w1.x; q[8 * t + 5] = w1.y; q[8 * t + 6] = w1.z; q[8 * t + 7] = w1.w;
        }
        const unsigned *rg = range + (size_t)h * F32_RANGE;
        unsigned most = max(rg[0], rg[1]), least = max(rg[2], rg[3]);
#pragma unroll
        for (int k = 0; k < D / 2; ++k) f32_range(__float_as_uint(q[k]), most, least);
        split = __all(most <= F32_MOST && least <= 0u - F32_LEAST) && scale_log2 <= F32_SCALE;
        if (split) {
#pragma unroll
            for (int t = 0; t < D / 16; ++t)
                if (t % NW == wave) {           // (wave-uniform; every wavefront holds the same row parts)
                    u32x4 part[3];
#pragma unroll
                    for (int e = 0; e < 4; ++e) f32_split3(q[8 * t + 2 * e], q[8 * t + 2 * e + 1], part, e);
#pragma unroll
                    for (int i = 0; i < 3; ++i) s_q[(3 * t + i) * 64 + lane] = part[i];
                }
            __syncthreads();
        }
    }
    f32x16 oacc[DVB];
#pragma unroll
    for (int b = 0; b < DVB; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[b][i] = 0.f;
    float m = -INFINITY, l = 0.f;

    // byte offset of the row of key 32 j + col (past the end: the last key's row, so that nothing but selected rows is
    // ever read here; its score is masked)
    auto row_off = [&](int j) -> unsigned {
        const int kk = min(32 * j + col, L - 1);
        // run in which the 64-key tile starts (the table ends at N keys; a row may have more, if its list names a
        // cluster twice)
        int c = trh[min(j >> 1, key_tiles - 1)];
        while (c + 1 < nnz && kk >= rn[c + 1].y) ++c;
        const int2 rs = rn[c];
        int r = rs.x + kk - rs.y;
        if (perm_k) r = pkh[r];                 // gather-free: sorted row -> token
        return (unsigned)r * RB;
    };
    // V of contraction steps 8 hf .. 8 hf + 7: step i takes key 8 (i / 4) + 4 half + i % 4, columns DVB col ..
    auto load_v = [&](fvec (&buf)[8], unsigned off, int hf) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int st = 8 * hf + i;
            const unsigned r = (unsigned)__shfl((int)off, 8 * (st / 4) + 4 * half + st % 4);
            buf[i] = *reinterpret_cast<const fvec *>(Vb + (r + (unsigned)(col * (4 * DVB))));
        }
    };
    // scores of a block -> its probabilities, running level and sum
    auto softmax = [&](f32x16 &S) {
        float mx = fmaxf(S[0], S[1]);
#pragma unroll
        for (int i = 2; i < 16; ++i) mx = fmaxf(mx, S[i]);
        mx = fmaxf(m, max_xor32(mx) * scale_log2);
        if (__any(mx > m)) {
            const float alpha = __builtin_amdgcn_exp2f(m - mx);
            m = mx;
            l *= alpha;
#pragma unroll
            for (int b = 0; b < DVB; ++b)
#pragma unroll
                for (int i = 0; i < 16; ++i) oacc[b][i] *= alpha;
        }
        const float m_ref = (m == -INFINITY) ? 0.f : m;         // scores of -inf alone so far: weights 0, not NaN
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            S[i] = __builtin_amdgcn_exp2f(fmaf(S[i], scale_log2, -m_ref));
            l += S[i];
        }
    };
    // keys past the end: no score, and no value either (zero times an infinite one would be NaN)
    auto mask = [&](f32x16 &S, fvec (&v0)[8], fvec (&v1)[8], int j) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if (32 * j + 8 * (i >> 2) + 4 * half + (i & 3) >= L) {
                S[i] = -INFINITY;
                (i < 8 ? v0 : v1)[i & 7] = fvec{};
            }
    };
#define F32_FENCE __builtin_amdgcn_sched_barrier(0);

    if (NW == F32_NW && split) {
        fvec vA[8], vB[8];
        float *sk = s_o + wave * (32 * D);      // this wavefront's K block
        constexpr int CPR = D / 4;              // 16-byte chunks per row
        // chunk c of row r sits at c ^ (r % 16): 16 rows read at one chunk hit different banks
        const unsigned chunk = 16u * (unsigned)((lane % CPR) ^ (lane / CPR));
        auto fetch_k = [&](unsigned off) {
            unsigned x = chunk;
            asm volatile("" : "+v"(x));
            unsigned o[CPR / 2];
#pragma unroll
            for (int i = 0; i < CPR / 2; ++i) o[i] = (unsigned)__shfl((int)off, i * (64 / CPR) + lane / CPR);
#pragma unroll
            for (int i = 0; i < CPR / 2; ++i)           // (row i * (64 / CPR) + lane / CPR)
                load_to_lds_16(Kb, o[i] + (x ^ (16u * (i * (64 / CPR) % 16))), reinterpret_cast<const unsigned char *>(sk) + 1024 * i);
        };
        const float *krow = sk + col * D;
        const unsigned kx = (unsigned)(col % 16 ^ 2 * half);
        auto qk = [&](f32x16 &S) {
            unsigned x = kx;
            asm volatile("" : "+v"(x));         // (the addresses are formed here, not held in registers)
            f32x16 small = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < D / 16; ++t) {
                u32x4 kp[3];
#pragma unroll
                for (int e4 = 0; e4 < 2; ++e4) {
                    const float4 w = *reinterpret_cast<const float4 *>(krow + 4 * (x ^ (unsigned)(4 * t + e4)));      // chunk 4 t + 2 half + e4
                    f32_split3(w.x, w.y, kp, 2 * e4);
                    f32_split3(w.z, w.w, kp, 2 * e4 + 1);
                }
                const u32x4 qp[3] = {s_q[3 * t * 64 + lane], s_q[(3 * t + 1) * 64 + lane], s_q[(3 * t + 2) * 64 + lane]};
                f32_mfma3(kp, qp, S, D == 128 ? small : S);         // (D == 64: no registers left)
            }
            if (D == 128)
#pragma unroll
                for (int i = 0; i < 16; ++i) S[i] += small[i];
        };
        // The products of 16 keys are summed by themselves and meet the running sum as one: term by term the third parts of values
        // that many keys share would be rounded away, one key like the other.
        auto pv = [&](const f32x16 &P, const fvec (&v)[8], int hf) {
            u32x4 pp[3];
#pragma unroll
            for (int i = 0; i < 4; ++i) f32_split3(P[8 * hf + 2 * i], P[8 * hf + 2 * i + 1], pp, i);
#pragma unroll
            for (int b = 0; b < DVB; ++b) {
                u32x4 vp[3];
#pragma unroll
                for (int i = 0; i < 4; ++i) f32_split3(v[2 * i][b], v[2 * i + 1][b], vp, i);
                f32x16 sum = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                f32_mfma3(vp, pp, sum, sum);
#pragma unroll
                for (int i = 0; i < 16; ++i) oacc[b][i] += sum[i];
            }
        };
        // The rows of a block two ahead, in two steps between which its loads are on their way: the 64 runs from the one in which the
        // 64-key tile starts, one per lane; then each lane counts those that start at or before its key.
        auto first_run = [&](int j) -> int { return trh[min(min(j, nblk - 1) >> 1, key_tiles - 1)]; };
        auto load_runs = [&](int c0) -> int2 { return rn[min(c0 + lane, nnz - 1)]; };
        auto find_rows = [&](int j, int c0, const int2 &rv) -> unsigned {
            if (j >= nblk) return 0;
            const int kk = min(32 * j + col, L - 1), last = min(32 * j + 31, L - 1);
            const int start = c0 + lane < nnz ? rv.y : 0x7FFFFFFF;
            int c = 0, i = 1;
            for (; i < 64; ++i) {
                const int s = __builtin_amdgcn_readlane(start, i);
                if (s > last) break;
                c += kk >= s;
            }
            if (i == 64) return row_off(j);     // (runs of one key, or of none)
            int r = __shfl(rv.x - rv.y, c) + kk;
            if (perm_k) r = pkh[r];
            return (unsigned)r * RB;
        };
        unsigned off = 0, off_n = 0;
        int c0 = 0;
        if (wave < nblk) {
            off = row_off(wave);
            fetch_k(off);
            off_n = row_off(min(wave + NW, nblk - 1));
            c0 = first_run(wave + 2 * NW);
        }
        for (int j = wave; j < nblk; j += NW) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // block j of K is in LDS, its rows are known
            load_v(vA, off, 0);
            load_v(vB, off, 1);
            const int2 rv = load_runs(c0);
            F32_FENCE
            f32x16 S = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            qk(S);
            F32_FENCE
            // V is waited for here, in front of the fetches of the next K, which the compiler does not see
#pragma unroll
            for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(vA[i]), "+v"(vB[i]));
            F32_FENCE
            if (j + NW < nblk) fetch_k(off_n);
            const unsigned off_2 = find_rows(j + 2 * NW, c0, rv);
            c0 = first_run(j + 3 * NW);
            F32_FENCE
            if (j == nblk - 1) mask(S, vA, vB, j);
            softmax(S);
            F32_FENCE
            pv(S, vA, 0);
            pv(S, vB, 1);
            F32_FENCE
            off = off_n;
            off_n = off_2;
        }
    } else {
        float4 bufA[NB], bufB[NB];
        fvec vA[8], vB[8];
        float q[D / 2];                         // this lane's half of the row
#pragma unroll
        for (int k = 0; k < D / 8; ++k) {
            const float4 w = reinterpret_cast<const float4 *>(Qr + half * (D / 2))[k];
            q[4 * k] = w.x; q[4 * k + 1] = w.y; q[4 * k + 2] = w.z; q[4 * k + 3] = w.w;
        }
        auto load_k = [&](float4 (&buf)[NB], unsigned off, int hf) {
            const float4 *src = reinterpret_cast<const float4 *>(Kb + (off + (unsigned)(half * (RB / 2) + hf * (RB / 4))));
#pragma unroll
            for (int i = 0; i < NB; ++i) buf[i] = src[i];
        };
        auto qk = [&](f32x16 &S, const float4 (&buf)[NB], int hf) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                S = __builtin_amdgcn_mfma_f32_32x32x2f32(buf[i].x, q[4 * (hf * NB + i)], S, 0, 0, 0);
                S = __builtin_amdgcn_mfma_f32_32x32x2f32(buf[i].y, q[4 * (hf * NB + i) + 1], S, 0, 0, 0);
                S = __builtin_amdgcn_mfma_f32_32x32x2f32(buf[i].z, q[4 * (hf * NB + i) + 2], S, 0, 0, 0);
                S = __builtin_amdgcn_mfma_f32_32x32x2f32(buf[i].w, q[4 * (hf * NB + i) + 3], S, 0, 0, 0);
            }
        };
        auto pv = [&](const f32x16 &P, const fvec (&v)[8], int hf) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int b = 0; b < DVB; ++b) oacc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[i][b], P[8 * hf + i], oacc[b], 0, 0, 0);
        };
        unsigned off = 0;
        if (wave < nblk) {
            off = row_off(wave);
            load_k(bufA, off, 0);
        }
        for (int j = wave; j < nblk; j += NW) {
            load_k(bufB, off, 1);
            const unsigned off_n = row_off(min(j + NW, nblk - 1));
            F32_FENCE
            f32x16 S = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            qk(S, bufA, 0);
            F32_FENCE
            load_v(vA, off, 0);
            F32_FENCE
            qk(S, bufB, 1);
            F32_FENCE
            load_v(vB, off, 1);
            F32_FENCE
            if (j == nblk - 1) mask(S, vA, vB, j);
            softmax(S);
            F32_FENCE
            pv(S, vA, 0);
            F32_FENCE
            load_k(bufA, off_n, 0);             // (after the last block: a valid row, not used)
            F32_FENCE
            pv(S, vB, 1);
            F32_FENCE
            off = off_n;
        }
    }
#undef F32_FENCE

    // ---- the shares of the wavefronts: common level, scaled accumulators to LDS, sum, store
    l = sum_xor32(l);
    if (half == 0) { s_m[wave][col] = m; s_l[wave][col] = l; }
    __syncthreads();
    float m_all = s_m[0][col];
#pragma unroll
    for (int w = 1; w < NW; ++w) m_all = fmaxf(m_all, s_m[w][col]);
    const float f = (m == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m - m_all);
    float *so = s_o + (size_t)(wave * 32 + col) * ROW;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int row = 8 * (i >> 2) + 4 * half + (i & 3);
        fvec v;
#pragma unroll
        for (int b = 0; b < DVB; ++b) v[b] = oacc[b][i] * f;
        *reinterpret_cast<fvec *>(so + DVB * row) = v;
    }
    __syncthreads();
    constexpr int LPR = D / 4;                  // lanes per row of the result
    for (int r = tid / LPR; r < nrows; r += 64 * NW / LPR) {
        const int c4 = (tid % LPR) * 4;
        float mm = s_m[0][r], lt = 0.f;
#pragma unroll
        for (int w = 1; w < NW; ++w) mm = fmaxf(mm, s_m[w][r]);
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            lt += s_l[w][r] * (s_m[w][r] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(s_m[w][r] - mm));
            const float4 v = *reinterpret_cast<const float4 *>(s_o + (size_t)(w * 32 + r) * ROW + c4);
            acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
        }
        const size_t dst = (size_t)h * N + (perm_q ? perm_q[(size_t)h * N + row0 + r] : row0 + r);
        // (no key: 0; keys without any weight, or scores that are no numbers: the softmax is undefined)
        const float inv = (lt > 0.f) ? 1.0f / lt : L > 0 ? NAN : 0.f;
        *reinterpret_cast<float4 *>(O + dst * D + c4) = make_float4(acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv);
        if (lse && c4 == 0) lse[dst] = (lt > 0.f) ? (mm + log2f(lt)) * 0.6931471805599453f : -INFINITY;
    }
}

// ---------------------------------------------------------------- host side

size_t attn_ws_bytes(int dtype, int H, int N, int d, int Cq, int Ck)
{
    (void)d;
    return attn_carve(nullptr, dtype, H, N, Cq, Ck).bytes;
}

static size_t attn_lds_bytes(int d, int Ck)
{
    return (size_t)2 * ATT_NSTG * ATT_BN * d * sizeof(bf16_t) + 2 * ATT_BN * sizeof(int32_t) +
           (size_t)std::min(Ck + 1, ATT_RUN_LDS) * sizeof(int2);
}

// The ranges that let a head's operands be split: none for short heads, where looking at K and V costs more than it saves (with operands in
// two fp16 halves, which were faster yet: 1000 heads of 256 tokens, D = 128: 537 instead of 430 us; 5000 of 16, D = 64: 134 instead of 55); 200 of 600,
// fp32 instruction / split, D = 64 221 / 190, D = 128 459 / 431 us, and 247 and 513 where an infinity is found in every head.  Heads
// with a range have eight wavefronts per work item (attn_f32_nw), which share a CU with no other at D = 128.
static unsigned *attn_range_of(const AttnWs &a, int N) { return N > F32_SHORT ? a.range : nullptr; }

// (split Q lies behind the K blocks; the padding of the final sum's rows is not there yet)
static size_t attn_f32_lds_bytes(int d, int nw, bool ranged)
{
    const size_t sum = (size_t)nw * F32_BM * (d + 4) * sizeof(float);
    return ranged ? std::max(sum, (size_t)nw * F32_BM * d * sizeof(float) + 3 * F32_BM * d * sizeof(bf16_t)) : sum;
}

static int attn_f32_nw(int H, int N)
{
    const bool many = (long long)H * cdiv(N, F32_BM) >= F32_MANY && N <= F32_SHORT;
    int nw = 1;
    while (nw < (many ? F32_NW / 2 : F32_NW) && 32 * nw < N) nw *= 2;
    return nw;
}

int attn_prepare(int dtype, int d)
{
    if (dtype != SVG2_BF16) {
        // (with fewer wavefronts than F32_NW less than 64 KB of LDS except at D = 128 and four)
        if (d == 128) {
            SVG2_TRY(set_dynamic_lds(reinterpret_cast<const void *>(attn_f32_kernel<128, 4>), attn_f32_lds_bytes(d, 4, false)));
            return set_dynamic_lds(reinterpret_cast<const void *>(attn_f32_kernel<128, F32_NW>), attn_f32_lds_bytes(d, F32_NW, true));
        }
        return set_dynamic_lds(reinterpret_cast<const void *>(attn_f32_kernel<64, F32_NW>), attn_f32_lds_bytes(d, F32_NW, true));
    }
    const size_t lds = attn_lds_bytes(d, SVG2_MAX_CLUSTERS);
    if (d == 128) {
        SVG2_TRY(set_dynamic_lds(reinterpret_cast<const void *>(attn_bf16_kernel<128, true>), lds));
        SVG2_TRY(set_dynamic_lds(reinterpret_cast<const void *>(attn_bf16_kernel<128, false>), lds));
    } else {
        SVG2_TRY(set_dynamic_lds(reinterpret_cast<const void *>(attn_bf16_kernel<64, true>), lds));
        SVG2_TRY(set_dynamic_lds(reinterpret_cast<const void *>(attn_bf16_kernel<64, false>), lds));
    }
    return SVG2_OK;
}

int attn_plan_launch(const void *Kp, const void *Vp, int dtype, int H, int N, int d, int Cq, int Ck, const int32_t *offsets_q, const int32_t *offsets_k,
                     const int32_t *row_ptr, const int32_t *col_idx, void *ws, hipStream_t st)
{
    const AttnWs a = attn_carve(ws, dtype, H, N, Cq, Ck);
    hipLaunchKernelGGL(attn_plan_kernel, dim3(1 + cdiv(Cq, 4), H), dim3(256), 0, st, offsets_q, offsets_k, row_ptr, col_idx,
                       Cq, Ck, attn_bm(dtype), a.max_tiles, a.tiles, a.n_tiles, a.runs, a.row_keys, a.cl_first,
                       a.key_tiles, a.tile_run, attn_range_of(a, N));
    const bool f32 = attn_range_of(a, N) != nullptr;
    hipLaunchKernelGGL(attn_order_kernel, dim3(1 + (f32 ? attn_range_blocks(H, N, d) : 0)), dim3(1024), 0, st, offsets_q, a.n_tiles,
                       a.tile_base, a.row_keys, a.cl_first, H, Cq, attn_bm(dtype), a.order,
                       f32 ? static_cast<const float *>(Kp) : nullptr, f32 ? static_cast<const float *>(Vp) : nullptr, N, d, a.range);
    SVG2_HIP_CHECK(hipGetLastError());
    return SVG2_OK;
}

int attn_main_launch(const void *Qp, const void *Kp, const void *Vp, int dtype, int H, int N, int d, int Cq, int Ck,
                     const int32_t *row_ptr, const int32_t *perm_q, const int32_t *perm_k, float scale, void *O,
                     float *lse, void *ws, hipStream_t st)
{
    const AttnWs a = attn_carve(ws, dtype, H, N, Cq, Ck);
    const int max_tiles = a.max_tiles;
    int4 *tiles = a.tiles;
    int32_t *tile_base = a.tile_base;
    int2 *runs = a.runs;
    int32_t *row_keys = a.row_keys;
    if (!(scale > 0.f)) scale = 1.0f / sqrtf((float)d);
    const int total = H * max_tiles;
    const int group = ATT_GROUP;
    if (dtype == SVG2_BF16) {
        const float scale_log2 = scale * 1.4426950408889634f;
        const bf16_t *q = static_cast<const bf16_t *>(Qp), *k = static_cast<const bf16_t *>(Kp),
                     *v = static_cast<const bf16_t *>(Vp);
        bf16_t *o = static_cast<bf16_t *>(O);
        const size_t lds = attn_lds_bytes(d, Ck);
        const bool cap = Ck + 1 > ATT_RUN_LDS;
        auto kern = d == 128 ? (cap ? attn_bf16_kernel<128, true> : attn_bf16_kernel<128, false>)
                             : (cap ? attn_bf16_kernel<64, true> : attn_bf16_kernel<64, false>);
        hipLaunchKernelGGL(kern, attn_list_grid(total), dim3(64 * ATT_NW), lds, st, q, k, v, H, N, Cq, Ck, row_ptr, perm_q, perm_k, tiles,
                           tile_base, a.order, max_tiles, runs, row_keys, a.tile_run, a.key_tiles, scale_log2, group, o, lse);
    } else {
        const float *q = static_cast<const float *>(Qp), *k = static_cast<const float *>(Kp),
                    *v = static_cast<const float *>(Vp);
        float *o = static_cast<float *>(O);
        static_assert(F32_BM == attn_bm(SVG2_F32), "the plan cuts query clusters into the tiles of this kernel");
        const int nw = attn_f32_nw(H, N);
        static_assert(F32_SHORT >= 32 * F32_NW / 2, "a head with a range (attn_range_of) has eight wavefronts per work item");
        auto kern = d == 128 ? (nw == 1   ? attn_f32_kernel<128, 1>
                                : nw == 2 ? attn_f32_kernel<128, 2>
                                : nw == 4 ? attn_f32_kernel<128, 4>
                                          : attn_f32_kernel<128, F32_NW>)
                             : (nw == 1   ? attn_f32_kernel<64, 1>
                                : nw == 2 ? attn_f32_kernel<64, 2>
                                : nw == 4 ? attn_f32_kernel<64, 4>
                                          : attn_f32_kernel<64, F32_NW>);
        hipLaunchKernelGGL(kern, attn_list_grid(total), dim3(64 * nw), attn_f32_lds_bytes(d, nw, attn_range_of(a, N) != nullptr), st, q, k, v, H, N, Cq, Ck,
                           row_ptr, perm_q, perm_k, tiles, tile_base, a.order, max_tiles, runs, row_keys, a.tile_run,
                           a.key_tiles, scale * 1.4426950408889634f, group, attn_range_of(a, N), o, lse);
    }
    SVG2_HIP_CHECK(hipGetLastError());
    return SVG2_OK;
}

int attn_launch(const void *Qp, const void *Kp, const void *Vp, int dtype, int H, int N, int d, int Cq, int Ck,
                const int32_t *offsets_q, const int32_t *offsets_k, const int32_t *row_ptr,
                const int32_t *col_idx, const int32_t *perm_q, const int32_t *perm_k, float scale, void *O,
                float *lse, void *ws, hipStream_t st)
{
    const int rc = attn_plan_launch(Kp, Vp, dtype, H, N, d, Cq, Ck, offsets_q, offsets_k, row_ptr, col_idx, ws, st);
    if (rc != SVG2_OK) return rc;
    return attn_main_launch(Qp, Kp, Vp, dtype, H, N, d, Cq, Ck, row_ptr, perm_q, perm_k, scale, O, lse, ws, st);
}

}  // namespace svg2
