// One reassignment step of the paper's Algorithm 2 on gfx950, for one
// clustering problem or for many independent ones at once.
//
//   1. V from the labels (Sec. 4.1): cluster sizes by a reduction of the label
//      array, then V in CSR form.  V's values are all 1/|c| within a row, so
//      the CSR arrays reduce to the row pointers (cluster offsets) and the
//      column indices (point indices grouped by cluster, stable).
//   2. E = K V^T (Eq. dist_sp_1).  K is symmetric, so row c of E^T is the sum
//      of the K rows of cluster c's members, scaled by 1/|c|.  Walking V's CSR
//      rows visits K's rows cluster by cluster: every row read has one label
//      for the whole wavefront, and each lane keeps a running compensated sum
//      per column in registers that is flushed once per cluster segment.  K is
//      read exactly once, in 1 KiB contiguous pieces per wavefront.
//   3. ||c_c||^2 = (V z)_c with z_i = E_{i,a(i)} (Eq. c_norm, Eq. cnorms_gemv):
//      the sweep folds z into per-segment partials as it flushes, a small
//      kernel reduces them per cluster.
//   4. D_ic = K_ii - 2 E_ic + ||c_c||^2 (Eq. dist_sp_1), argmin over c, the new
//      cluster-size histogram, the number of changed labels and the FP64
//      objective of the input labels, fused in one pass over the points.
//
// Every kernel takes an instance set: either one problem passed by value, or a
// device table of live problems whose blocks are laid end to end in one grid
// (a block finds its problem by binary search in a prefix array; blocks past
// the live total exit).  The table is rewritten on the device between steps,
// so a captured sequence of launches can be replayed while problems converge
// one by one.
//
// No floating-point atomics are used: every reduction runs in a fixed order,
// so a step is bitwise repeatable.
#include "iterate.h"

namespace kkm {

namespace {

constexpr int kPtsPerBlock = 256;          // points per block in the label kernels
constexpr int kSweepThreads = 256;         // 4 waves
constexpr int kAssignPts = 64;             // points per assignment workgroup (4 waves share them)
constexpr int kAssignStageK = 128;         // largest k whose D rows are staged in LDS
constexpr int kSmallThreads = 1024;        // the one-workgroup CSR build
constexpr int64_t kSmallPts = 8192;        // its most points

// The problem and the block index within it for a flattened grid position g;
// false when g lies past the live problems of a table.  MULTI selects the
// table form at compile time: a run-time choice between the two sources would
// leave the problem's fields in vector registers.
template <bool MULTI>
__device__ __forceinline__ bool locate(const InstSet &s, const int64_t *start, int64_t g, Inst &in,
                                       int64_t &local) {
    if constexpr (MULTI) {
        if (g >= uniform_load(start + s.count)) return false;
        const int32_t b = find_inst(start, s.count, g);
        local = g - uniform_load(start + b);
        in = uniform_load(s.table + b);
    } else {
        local = g;
        in = s.one;
    }
    return true;
}

// ---------------------------------------------------------------- 1. V in CSR form

// Per-block label histogram (column-major [k][nblk]) and range check.
template <bool MULTI>
__global__ __launch_bounds__(kPtsPerBlock) void v_block_hist(InstSet s, const int32_t *labels_all) {
    extern __shared__ int32_t sh[];  // [k] + 1
    Inst in;
    int64_t lb;
    if (!locate<MULTI>(s, s.blk_start, blockIdx.x, in, lb)) return;
    const int32_t k = in.k;
    const int32_t *labels = labels_all + in.lab_off;
    int32_t *hist = sh;
    int32_t *bad = sh + k;
    for (int c = threadIdx.x; c < k; c += blockDim.x) hist[c] = 0;
    if (threadIdx.x == 0) *bad = 0;
    __syncthreads();
    const int64_t i = lb * kPtsPerBlock + threadIdx.x;
    if (i < in.n) {
        const int32_t c = labels[i];
        if (c < 0 || c >= k)
            atomicAdd(bad, 1);
        else
            atomicAdd(&hist[c], 1);
    }
    __syncthreads();
    for (int c = threadIdx.x; c < k; c += blockDim.x) in.blk_hist[(int64_t)c * in.nblk + lb] = hist[c];
    if (threadIdx.x == 0) in.blk_bad[lb] = *bad;
}

// One workgroup per (problem, cluster): exclusive prefix of its per-block counts
// (in place) and its size.  Cluster 0's workgroup also folds the range check.
template <bool MULTI>
__global__ __launch_bounds__(256) void v_cluster_scan(InstSet s) {
    __shared__ int32_t part[256];
    __shared__ int32_t carry;
    Inst in;
    int64_t c;
    if (!locate<MULTI>(s, s.cl_start, blockIdx.x, in, c)) return;
    const int64_t nblk = in.nblk;
    int32_t *row = in.blk_hist + c * nblk;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int64_t base = 0; base < nblk; base += 256) {
        const int64_t i = base + threadIdx.x;
        const int32_t v = (i < nblk) ? row[i] : 0;
        part[threadIdx.x] = v;
        __syncthreads();
        // Hillis-Steele inclusive scan over 256 entries
        for (int off = 1; off < 256; off <<= 1) {
            const int32_t add = (threadIdx.x >= off) ? part[threadIdx.x - off] : 0;
            __syncthreads();
            part[threadIdx.x] += add;
            __syncthreads();
        }
        if (i < nblk) row[i] = carry + part[threadIdx.x] - v;
        __syncthreads();
        if (threadIdx.x == 255) carry += part[255];
        __syncthreads();
    }
    if (threadIdx.x == 0) in.counts[c] = carry;
    if (c == 0) {
        int32_t t = 0;
        for (int64_t i = threadIdx.x; i < nblk; i += 256) t += in.blk_bad[i];
        part[threadIdx.x] = t;
        __syncthreads();
        if (threadIdx.x == 0) {
            int32_t u = 0;
            for (int w = 0; w < 256; ++w) u += part[w];
            *in.err = u;
        }
    }
}

// Stable scatter of point indices into V's CSR order.  Block 0 of each problem
// also publishes the row pointers and clears the step's counters.
template <bool MULTI>
__global__ __launch_bounds__(kPtsPerBlock) void v_scatter(InstSet s, const int32_t *labels_all) {
    extern __shared__ int32_t sh[];  // off[k+1], wcnt[4][k]
    Inst in;
    int64_t lb;
    if (!locate<MULTI>(s, s.blk_start, blockIdx.x, in, lb)) return;
    const int32_t k = in.k;
    const int32_t *labels = labels_all + in.lab_off;
    int32_t *off = sh;
    int32_t *wcnt = sh + (k + 1);
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    if (*in.err != 0) return;

    // exclusive scan of the cluster sizes (k <= KKM_MAX_K; one thread, then share)
    if (tid == 0) {
        int32_t run = 0;
        for (int c = 0; c < k; ++c) {
            off[c] = run;
            run += in.counts[c];
        }
        off[k] = run;
    }
    for (int c = tid; c < 4 * k; c += kPtsPerBlock) wcnt[c] = 0;
    __syncthreads();
    if (lb == 0) {
        for (int c = tid; c <= k; c += kPtsPerBlock) in.offsets[c] = off[c];
        for (int c = tid; c < k; c += kPtsPerBlock) in.counts_out[c] = 0;
        if (tid == 0) *in.n_changed = 0;
    }

    const int64_t i = lb * kPtsPerBlock + tid;
    const bool valid = i < in.n;
    const int32_t c = valid ? labels[i] : -1;
    // rank among equal labels earlier in this wave
    const uint64_t peers = label_peers(valid, c, label_bits(k));
    const int32_t rank = __popcll(peers & ((lane == 0) ? 0ull : (~0ull >> (64 - lane))));
    if (valid && rank == 0) wcnt[wave * k + c] = __popcll(peers);
    __syncthreads();
    if (valid) {
        int32_t before = 0;
        for (int w = 0; w < wave; ++w) before += wcnt[w * k + c];
        const int64_t pos = off[c] + in.blk_hist[(int64_t)c * in.nblk + lb] + before + rank;
        in.perm[pos] = (int32_t)i;
    }
}

// The three kernels above in one workgroup, for one small problem: below about
// 8000 points each of them is a launch whose few workgroups wait on memory
// (2.5 + 4.1 + 3.4 us and their gaps at n = 1000; here 3.6).  Each wave takes a contiguous
// stretch of points, 64 at a time, so its running counts need no barrier; the
// labels are read once.  Same row pointers and the same stable order, so the
// same V.
constexpr int kSmallGroups = kSmallPts / kSmallThreads;  // 64-point groups per wave

// What the wave's lanes read and wrote in LDS before it comes before what they
// read and write after it.
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__global__ __launch_bounds__(kSmallThreads) void v_csr_small(Inst in, const int32_t *labels) {
    extern __shared__ int32_t sh[];  // run[k], wcnt[16][k]
    __shared__ int32_t bad;
    const int32_t k = in.k;
    const int32_t n = (int32_t)in.n;
    constexpr int NW = kSmallThreads / kWave;
    int32_t *run = sh, *wcnt = sh + k;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int groups = (n + kSmallThreads - 1) / kSmallThreads;
    const int32_t i0 = wave * groups * kWave + lane;
    int32_t c[kSmallGroups], rank[kSmallGroups];
#pragma unroll
    for (int g = 0; g < kSmallGroups; ++g) {
        const int32_t i = i0 + g * kWave;
        c[g] = (g < groups && i < n) ? labels[i] : -1;
    }
    for (int t = tid; t < NW * k; t += kSmallThreads) wcnt[t] = 0;
    if (tid == 0) bad = 0;
    __syncthreads();
    const int bits = label_bits(k);
    int32_t nbad = 0;
#pragma unroll
    for (int g = 0; g < kSmallGroups; ++g) {
        if (g >= groups) break;
        const bool in_n = i0 + g * kWave < n;
        const bool valid = in_n && c[g] >= 0 && c[g] < k;
        nbad += __popcll(__ballot(in_n && !valid));
        const uint64_t peers = label_peers(valid, c[g], bits);
        const int32_t below = __popcll(peers & ((lane == 0) ? 0ull : (~0ull >> (64 - lane))));
        int32_t *const count = &wcnt[wave * k + (valid ? c[g] : 0)];
        const int32_t before = *count;  // read by a label's lanes,
        rank[g] = before + below;
        wave_fence();
        if (valid && below == 0) *count = before + __popcll(peers);  // then written by its first
        wave_fence();
    }
    if (nbad && lane == 0) atomicAdd(&bad, nbad);
    __syncthreads();
    nbad = bad;
    if (tid == 0) {
        in.err[0] = nbad;
        in.err[1] = 0;  // the assignment's arrival counter
    }
    if (nbad != 0) return;  // uniform
    for (int t = tid; t < k; t += kSmallThreads) {
        int32_t sum = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const int32_t v = wcnt[w * k + t];
            wcnt[w * k + t] = sum;
            sum += v;
        }
        run[t] = sum;
    }
    __syncthreads();
    // sizes -> exclusive prefix (row pointers), one wave
    if (wave == 0) {
        int32_t base = 0;
        for (int32_t t0 = 0; t0 < k; t0 += kWave) {
            const int32_t v = (t0 + lane < k) ? run[t0 + lane] : 0;
            int32_t x = v;
#pragma unroll
            for (int off = 1; off < kWave; off <<= 1) {
                const int32_t y = __shfl_up(x, off, kWave);
                if (lane >= off) x += y;
            }
            if (t0 + lane < k) {
                run[t0 + lane] = base + x - v;
                in.offsets[t0 + lane] = base + x - v;
            }
            base += __shfl(x, kWave - 1, kWave);
        }
        if (lane == 0) in.offsets[k] = base;
    }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < kSmallGroups; ++g)
        if (g < groups && i0 + g * kWave < n)
            in.perm[run[c[g]] + wcnt[wave * k + c[g]] + rank[g]] = i0 + g * kWave;
}

// ---------------------------------------------------------------- 2. row sweep of K

// Entries of K as FP32 (4 per 16-byte load) or bfloat16 (8 per 16-byte load),
// widened to float for the sums.
template <typename T> struct KRow;
template <> struct KRow<float> {
    static constexpr int E = 4;
    // 16-byte rows go through 64-bit global addresses: measured faster for FP32
    // K than buffer loads (25.7 vs 26.3 ms per 160 GB sweep)
    static constexpr bool kBuffer = false;
    static __device__ __forceinline__ void load_vec(const float *row, int64_t col, int64_t n,
                                                    float (&v)[E]) {
        if (col + E - 1 < n) {
            const f32x4 w = *reinterpret_cast<const f32x4 *>(row + col);
#pragma unroll
            for (int u = 0; u < E; ++u) v[u] = w[u];
        } else {
#pragma unroll
            for (int u = 0; u < E; ++u) v[u] = (col + u < n) ? row[col + u] : 0.f;
        }
    }
    // element loads of a row of any alignment (0 past column n)
    static __device__ __forceinline__ void load(const float *row, int64_t col, int64_t n,
                                                float (&v)[E]) {
#pragma unroll
        for (int u = 0; u < E; ++u) v[u] = (col + u < n) ? row[col + u] : 0.f;
    }
    // 16-byte load at byte offset voff of the row described by r (0 past its end)
    static __device__ __forceinline__ void load_buf(__amdgpu_buffer_rsrc_t r, uint32_t voff,
                                                    float (&v)[E]) {
        const auto w = __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, 0);
#pragma unroll
        for (int u = 0; u < E; ++u) v[u] = __uint_as_float(w[u]);
    }
};
template <> struct KRow<uint16_t> {
    static constexpr int E = 8;
    // buffer loads: one shared 32-bit lane offset instead of a 64-bit address
    // per row lets the unpacked rows fit 80 VGPRs (6 waves per SIMD instead of
    // 4); measured 13.2 vs 15.1 ms per 80 GB sweep
    static constexpr bool kBuffer = true;
    static __device__ __forceinline__ void load(const uint16_t *row, int64_t col, int64_t n,
                                                float (&v)[E]) {
#pragma unroll
        for (int u = 0; u < E; ++u)
            v[u] = (col + u < n) ? __uint_as_float((uint32_t)row[col + u] << 16) : 0.f;
    }
    static __device__ __forceinline__ void load_buf(__amdgpu_buffer_rsrc_t r, uint32_t voff,
                                                    float (&v)[E]) {
        const auto w = __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, 0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            v[2 * u] = __uint_as_float(w[u] << 16);
            v[2 * u + 1] = __uint_as_float(w[u] & 0xffff0000u);
        }
    }
};

// Buffer resource of one K row (gfx9 raw buffer: stride 0, range in bytes,
// 32-bit data format word).  Loads through it take one 32-bit lane offset
// shared by every row, and return 0 beyond the range.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void *row, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(row), (short)0, (int)bytes,
                                             0x00020000);
}

// The E entries of one K row at this lane's columns.  VEC: rows 16-byte
// aligned (ldk a multiple of E); otherwise element loads.
template <typename T, bool VEC>
__device__ __forceinline__ void load_row(const T *row, int64_t col, int64_t n, uint32_t voff,
                                         uint32_t rbytes, float (&v)[KRow<T>::E]) {
    if constexpr (VEC && KRow<T>::kBuffer)
        KRow<T>::load_buf(row_rsrc(row, rbytes), voff, v);
    else if constexpr (VEC)
        KRow<T>::load_vec(row, col, n, v);
    else
        KRow<T>::load(row, col, n, v);
}

// One work item = (column strip, chunk of L positions in V's CSR order).  Each
// lane owns E consecutive columns (one 16-byte load per row); a wave covers
// 64 E columns and the workgroup 256 E columns of every row it visits.  A chunk
// may span several clusters: the running sums are flushed to the partial-buffer
// slot (chunk + cluster) whenever the cluster changes; the slot is unique per
// (chunk, cluster) pair.
template <typename T, bool VEC>
__device__ __forceinline__ void sweep_item(const Inst &in, int64_t item, const int32_t *labels_all) {
    constexpr int E = KRow<T>::E;
    if (*in.err != 0) return;
    const int64_t n = in.n;
    const int32_t k = in.k;
    const int64_t L = in.L;
    const T *__restrict__ K = static_cast<const T *>(in.K);
    const int64_t ldk = in.ldk;
    const int32_t *__restrict__ perm = in.perm;
    const int32_t *__restrict__ offsets = in.offsets;
    const int32_t *__restrict__ labels = labels_all + in.lab_off;
    const int64_t nws = in.nws;
    const int64_t strip = (uint32_t)item % (uint32_t)in.nstrip;
    const int64_t q = (uint32_t)item / (uint32_t)in.nstrip;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int64_t wave_strip = strip * (kSweepThreads / kWave) + (tid >> 6);
    const int64_t col = wave_strip * (kWave * E) + (int64_t)lane * E;
    const int64_t p_begin = q * L;
    const int64_t p_end = min(n, p_begin + L);
    // VEC: every row is read with 16-byte buffer loads at this lane's byte
    // offset; columns in [n, ldk) are read but never used (their sums are not
    // stored and their labels are -1), and the range ends the row at ldk.
    const uint32_t voff = (uint32_t)(col * (int64_t)sizeof(T));
    const uint32_t rbytes = (uint32_t)(ldk * (int64_t)sizeof(T));

    // labels of this lane's columns (for z: the own-cluster entries)
    int32_t own[E];
#pragma unroll
    for (int u = 0; u < E; ++u) own[u] = (col + u < n) ? labels[col + u] : -1;

    // cluster holding position p_begin: last c with offsets[c] <= p_begin
    int32_t lo = 0, hi = k - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (offsets[mid] <= p_begin) lo = mid;
        else hi = mid - 1;
    }
    int32_t c = lo;

    int64_t p = p_begin;
    while (p < p_end) {
        while (offsets[c + 1] <= p) ++c;  // skip empty clusters
        const int64_t seg_end = min(p_end, (int64_t)offsets[c + 1]);
        float sum[E], e[E];
#pragma unroll
        for (int u = 0; u < E; ++u) sum[u] = e[u] = 0.f;
        for (; p + 8 <= seg_end; p += 8) {
            // pairwise sum of 8 rows, ((r0+r1)+(r2+r3)) + ((r4+r5)+(r6+r7)), taken
            // as two halves so that only four rows are unpacked at a time
            float blk[E];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float v[4][E];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int64_t j = __builtin_amdgcn_readfirstlane(perm[p + 4 * h + r]);
                    load_row<T, VEC>(K + j * ldk, col, n, voff, rbytes, v[r]);
                }
#pragma unroll
                for (int u = 0; u < E; ++u) {
                    const float q = (v[0][u] + v[1][u]) + (v[2][u] + v[3][u]);
                    blk[u] = h ? blk[u] + q : q;
                }
            }
#pragma unroll
            for (int u = 0; u < E; ++u) {
                float t, er;
                two_sum(sum[u], blk[u], t, er);
                sum[u] = t;
                e[u] += er;
            }
        }
        if (p < seg_end) {
            float blk[E];
#pragma unroll
            for (int u = 0; u < E; ++u) blk[u] = 0.f;
            for (; p < seg_end; ++p) {
                const int64_t j = __builtin_amdgcn_readfirstlane(perm[p]);
                float v[E];
                load_row<T, VEC>(K + j * ldk, col, n, voff, rbytes, v);
#pragma unroll
                for (int u = 0; u < E; ++u) blk[u] += v[u];
            }
#pragma unroll
            for (int u = 0; u < E; ++u) {
                float t, er;
                two_sum(sum[u], blk[u], t, er);
                sum[u] = t;
                e[u] += er;
            }
        }
        float tot[E];
#pragma unroll
        for (int u = 0; u < E; ++u) tot[u] = sum[u] + e[u];
        const int64_t slot = q + c;
        if (col < n) {
            float *dst = in.P + slot * in.ldp + col;
            if (col + E - 1 < n) {
#pragma unroll
                for (int u = 0; u < E; u += 4) {
                    const f32x4 w = {tot[u], tot[u + 1], tot[u + 2], tot[u + 3]};
                    *reinterpret_cast<f32x4 *>(dst + u) = w;
                }
            } else {
#pragma unroll
                for (int u = 0; u < E; ++u)
                    if (col + u < n) dst[u] = tot[u];
            }
        }
        float z = 0.f;
#pragma unroll
        for (int u = 0; u < E; ++u)
            if (own[u] == c) z += tot[u];
        z = wave_sum(z);
        if (lane == 0 && wave_strip < nws) in.Zp[slot * nws + wave_strip] = z;
    }
}

// One workgroup per item.  For a table the grid covers the items of every
// problem the table can hold and workgroups past the live total exit.  (A
// persistent grid looping over contiguous item ranges measured 4.5% slower:
// its loop raised the kernel from 64 to 76 VGPRs, 6 waves per SIMD instead of
// 8.)
template <typename T, bool VEC, bool MULTI>
__global__ __launch_bounds__(kSweepThreads) void spmm_row_sweep(InstSet s,
                                                                const int32_t *labels_all) {
    Inst in;
    int64_t item;
    if (!locate<MULTI>(s, s.item_start, blockIdx.x, in, item)) return;
    sweep_item<T, VEC>(in, item, labels_all);
}

// The sweep of a small problem: one workgroup per (64 E columns, chunk of at
// most 64 positions), its eight waves taking the chunk's blocks of up to eight
// rows in turn; wave 0 then adds the block sums, segment by segment, in their
// order.  Blocks, order and compensation are sweep_item's, so the partial sums
// are the same bit for bit.  sweep_item walks the chunk in one wave, a chain of
// index and row loads of which a small K has too few workgroups to hide
// (n = 1000: 16 workgroups, 18 us, here 7.9; n = 3001: 38 us for 36 MB, here 12).
constexpr int kSmallWaves = 8;    // (16: 2 workgroups per CU, n = 3001 12.0 -> 14.7 us)
constexpr int kSmallBlocks = 16;  // block sums staged per round

template <typename T, bool VEC>
__global__ __launch_bounds__(kSmallWaves *kWave) void spmm_small_sweep(Inst in, const int32_t *labels) {
    constexpr int E = KRow<T>::E;
    __shared__ __attribute__((aligned(16))) float bs[kSmallBlocks][kWave * E];
    __shared__ int32_t offsets[KKM_MAX_K + 1];
    const int64_t n = in.n;
    const T *__restrict__ K = static_cast<const T *>(in.K);
    const int64_t ldk = in.ldk;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t strip = (uint32_t)blockIdx.x % (uint32_t)in.nws;
    const int64_t q = (uint32_t)blockIdx.x / (uint32_t)in.nws;
    const int64_t col = strip * (kWave * E) + (int64_t)lane * E;
    const int32_t p_begin = (int32_t)(q * in.L);
    const int32_t p_end = (int32_t)min(n, q * in.L + in.L);
    const uint32_t voff = (uint32_t)(col * (int64_t)sizeof(T));
    const uint32_t rbytes = (uint32_t)(ldk * (int64_t)sizeof(T));
    // the chunk's rows (at most 64), one per lane
    const int32_t bad = *in.err;
    const int32_t rows = in.perm[min(p_begin + lane, p_end - 1)];
    for (int t = threadIdx.x; t <= in.k; t += kSmallWaves * kWave) offsets[t] = in.offsets[t];
    if (bad != 0) return;
    int32_t own[E];
#pragma unroll
    for (int u = 0; u < E; ++u) own[u] = (wave == 0 && col + u < n) ? labels[col + u] : -1;
    __syncthreads();
    // cluster holding position p_begin: last c with offsets[c] <= p_begin
    int32_t lo = 0, hi = in.k - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (__builtin_amdgcn_readfirstlane(offsets[mid]) <= p_begin) lo = mid;
        else hi = mid - 1;
    }
    int32_t c = lo;
    auto end_of = [&](int32_t cl) { return __builtin_amdgcn_readfirstlane(offsets[cl + 1]); };
    int32_t c_end = end_of(c);

    float sum[E], e[E];
#pragma unroll
    for (int u = 0; u < E; ++u) sum[u] = e[u] = 0.f;
    int32_t p = p_begin;
    while (p < p_end) {
        // this round's blocks: up to eight rows of one segment each
        int32_t pr = p, cr = c, cr_end = c_end, nb = 0;
        while (pr < p_end && nb < kSmallBlocks) {
            while (cr_end <= pr) cr_end = end_of(++cr);  // skip empty clusters
            const int32_t cnt = min(8, min(p_end, cr_end) - pr);
            if ((nb & (kSmallWaves - 1)) == wave) {
                float blk[E];
                const int l0 = pr - p_begin;
                if (cnt == 8) {
                    float v[8][E];
#pragma unroll
                    for (int r = 0; r < 8; ++r) {
                        const int64_t j = __builtin_amdgcn_readlane(rows, l0 + r);
                        load_row<T, VEC>(K + j * ldk, col, n, voff, rbytes, v[r]);
                    }
#pragma unroll
                    for (int u = 0; u < E; ++u) {
                        const float h0 = (v[0][u] + v[1][u]) + (v[2][u] + v[3][u]);
                        const float h1 = (v[4][u] + v[5][u]) + (v[6][u] + v[7][u]);
                        blk[u] = h0 + h1;
                    }
                } else {
#pragma unroll
                    for (int u = 0; u < E; ++u) blk[u] = 0.f;
                    for (int r = 0; r < cnt; ++r) {
                        const int64_t j = __builtin_amdgcn_readlane(rows, l0 + r);
                        float v[E];
                        load_row<T, VEC>(K + j * ldk, col, n, voff, rbytes, v);
#pragma unroll
                        for (int u = 0; u < E; ++u) blk[u] += v[u];
                    }
                }
#pragma unroll
                for (int u = 0; u < E; u += 4)
                    *reinterpret_cast<f32x4 *>(&bs[nb][lane * E + u]) =
                        f32x4{blk[u], blk[u + 1], blk[u + 2], blk[u + 3]};
            }
            ++nb;
            pr += cnt;
        }
        __syncthreads();
        if (wave == 0) {
            int32_t pw = p;
            f32x4 ahead[E / 4];
            auto fetch = [&](int b) {
#pragma unroll
                for (int u = 0; u < E / 4; ++u) ahead[u] = *reinterpret_cast<const f32x4 *>(&bs[b][lane * E + 4 * u]);
            };
            fetch(0);
            for (int b = 0; b < nb; ++b) {
                f32x4 v[E / 4];
#pragma unroll
                for (int u = 0; u < E / 4; ++u) v[u] = ahead[u];
                fetch(min(b + 1, kSmallBlocks - 1));
                while (c_end <= pw) c_end = end_of(++c);
                const int32_t seg_end = min(p_end, c_end);
                pw += min(8, seg_end - pw);
#pragma unroll
                for (int u = 0; u < E; ++u) {
                    float t, er;
                    two_sum(sum[u], v[u / 4][u % 4], t, er);
                    sum[u] = t;
                    e[u] += er;
                }
                if (pw < seg_end) continue;
                const int64_t slot = q + c;
                float *dst = in.P + slot * in.ldp + col;
                float tot[E];
                float z = 0.f;
#pragma unroll
                for (int u = 0; u < E; ++u) {
                    tot[u] = sum[u] + e[u];
                    if (own[u] == c) z += tot[u];
                    sum[u] = e[u] = 0.f;
                }
                if (col + E - 1 < n) {
#pragma unroll
                    for (int u = 0; u < E; u += 4)
                        *reinterpret_cast<f32x4 *>(dst + u) = f32x4{tot[u], tot[u + 1], tot[u + 2], tot[u + 3]};
                } else {
#pragma unroll
                    for (int u = 0; u < E; ++u)
                        if (col + u < n) dst[u] = tot[u];
                }
                z = wave_sum(z);
                if (lane == 0) in.Zp[slot * in.nws + strip] = z;
            }
        }
        p = pr;
        c = cr;
        c_end = cr_end;
        if (p < p_end) __syncthreads();  // the sums are read before the next round writes its own
    }
}

// ---------------------------------------------------------------- 3. centroid norms

// One workgroup per (problem, cluster): ||c_c||^2 = (1/|c|^2) sum_{i in c} S_ic,
// summing the z partials of the cluster's segments in a fixed order.
template <bool MULTI>
__global__ __launch_bounds__(256) void centroid_norms(InstSet s) {
    __shared__ float ss[256], sc[256];
    Inst in;
    int64_t c;
    if (!locate<MULTI>(s, s.cl_start, blockIdx.x, in, c)) return;
    if (*in.err != 0) return;
    const int64_t nws = in.nws;
    const int64_t a = in.offsets[c], e = in.offsets[c + 1];
    const int64_t cnt = e - a;
    float sum = 0.f, comp = 0.f;
    if (cnt > 0) {
        const int64_t q0 = a / in.L, q1 = (e - 1) / in.L;
        const int64_t total = (q1 - q0 + 1) * nws;
        const float *z = in.Zp + (q0 + c) * nws;  // the cluster's slots follow each other
        // eight loads at a time: few clusters mean few workgroups, each a chain
        // of loads (n = 60000, k = 10: 17 -> 6.7 us)
        for (int64_t t = threadIdx.x; t < total; t += 8 * 256) {
            float v[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) v[r] = (t + 256 * r < total) ? z[t + 256 * r] : 0.f;
#pragma unroll
            for (int r = 0; r < 8; ++r) {  // adding 0 past the end changes nothing
                float u, er;
                two_sum(sum, v[r], u, er);
                sum = u;
                comp += er;
            }
        }
    }
    ss[threadIdx.x] = sum;
    sc[threadIdx.x] = comp;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (threadIdx.x < h) {
            float u, er;
            two_sum(ss[threadIdx.x], ss[threadIdx.x + h], u, er);
            ss[threadIdx.x] = u;
            sc[threadIdx.x] += sc[threadIdx.x + h] + er;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        float v = 0.f;
        if (cnt > 0) {
            const float fc = (float)cnt;
            v = ((ss[0] + sc[0]) / fc) / fc;
        }
        in.ctilde[c] = v;
        if (in.ctilde_out) in.ctilde_out[c] = v;
    }
}

// The same norm by one wave, from the cluster's `total` own-cluster sums z:
// lane l stands for the 256 threads' sums l, l + 64, l + 128 and l + 192, added
// in the tree's order, so the bits are the same.  Lane 0 holds the result.
__device__ __forceinline__ float cluster_norm_wave(const float *z, int32_t total, int32_t cnt, int lane) {
    float s[4], m[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) s[u] = m[u] = 0.f;
    for (int32_t t = 0; t < total; t += 256) {
        float x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = (t + lane + 64 * u < total) ? z[t + lane + 64 * u] : 0.f;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            float w, er;
            two_sum(s[u], x[u], w, er);
            s[u] = w;
            m[u] += er;
        }
    }
    auto join = [](float &s0, float &m0, float s1, float m1) {
        float u, er;
        two_sum(s0, s1, u, er);
        s0 = u;
        m0 += m1 + er;
    };
    join(s[0], m[0], s[2], m[2]);
    join(s[1], m[1], s[3], m[3]);
    join(s[0], m[0], s[1], m[1]);
#pragma unroll
    for (int h = kWave / 2; h > 0; h >>= 1) {
        const float s1 = __shfl_down(s[0], h, kWave), m1 = __shfl_down(m[0], h, kWave);
        join(s[0], m[0], s1, m1);
    }
    const float fc = (float)cnt;
    return ((s[0] + m[0]) / fc) / fc;
}

// ---------------------------------------------------------------- 4. distances + argmin + histogram

// What each assignment workgroup leaves for the end of the step: its part of J
// and of the changed labels, over V's column indices (the sweep was their last
// reader), and its cluster sizes (at most 64: bytes) over the CSR build's block
// histograms, [k][4 nblk].  Sums in a fixed order instead of atomics: with a
// workgroup per 64 points the atomics on k sizes were half of the assignment's
// time (n = 100000, k = 64: 52 us with them, 28 us without).
struct AssignPart {
    double J;
    int64_t changed;
};
__device__ __forceinline__ AssignPart *assign_parts(const Inst &in) { return reinterpret_cast<AssignPart *>(in.perm); }
__device__ __forceinline__ uint8_t *assign_sizes(const Inst &in, int32_t c) {
    return reinterpret_cast<uint8_t *>(in.blk_hist + (int64_t)c * in.nblk);
}
__device__ __forceinline__ int64_t assign_blocks(const Inst &in) { return (in.n + kAssignPts - 1) / kAssignPts; }

// ACROSS: the value was stored by another workgroup of the same launch.
template <bool ACROSS, typename T> __device__ __forceinline__ T part_load(const T *p) {
    if constexpr (ACROSS) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return *p;
}
template <bool ACROSS, typename T> __device__ __forceinline__ void part_store(T *p, T v) {
    if constexpr (ACROSS) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *p = v;
}

// J of the input labels and the number of changed labels, by the first 256
// threads of a workgroup (all of its threads call).
template <bool ACROSS>
__device__ __forceinline__ void finish_objective(const Inst &in, double *wJ, long long *wC) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid < kPtsPerBlock) {
        const AssignPart *part = assign_parts(in);
        const int64_t nb = assign_blocks(in);
        double J = 0.0;
        long long changed = 0;
        for (int64_t t = tid; t < nb; t += kPtsPerBlock) {
            J += part_load<ACROSS>(&part[t].J);
            changed += part_load<ACROSS>(&part[t].changed);
        }
        J = wave_sum(J);
        changed = wave_sum(changed);
        if (lane == 0) {
            wJ[wave] = J;
            wC[wave] = changed;
        }
    }
    __syncthreads();
    if (tid == 0) {
        double tj = 0.0;
        long long tc = 0;
        for (int w = 0; w < kPtsPerBlock / kWave; ++w) {
            tj += wJ[w];
            tc += wC[w];
        }
        *in.J_in = tj;
        *in.n_changed = tc;
    }
}

// Size of cluster c, by LANES lanes of a wave (this one is `sub`); lane 0 of
// them writes it.  The blocks' bytes are read four at a time, those past the
// last block left out.
template <bool ACROSS, int LANES>
__device__ __forceinline__ void finish_size(const Inst &in, int32_t c, int sub) {
    const uint32_t *row = reinterpret_cast<const uint32_t *>(assign_sizes(in, c));
    const int64_t nb = assign_blocks(in);
    uint32_t sum = 0;
    for (int64_t t = sub; 4 * t < nb; t += LANES) {
        const uint32_t w = part_load<ACROSS>(row + t);
        const int64_t left = nb - 4 * t;
        sum += (w & 0xFFu) + (left > 1 ? (w >> 8) & 0xFFu : 0u) + (left > 2 ? (w >> 16) & 0xFFu : 0u) +
               (left > 3 ? w >> 24 : 0u);
    }
#pragma unroll
    for (int off = LANES / 2; off > 0; off >>= 1) sum += __shfl_xor(sum, off, kWave);
    if (sub == 0) in.counts_out[c] = (int32_t)sum;
}

// 64 points per workgroup, one per lane, the clusters dealt to the NW waves in
// turn.  A thread per point summing every cluster's partials alone waited load
// batch after load batch in n/256 workgroups; here a wave's chain is k / NW
// clusters long, the next cluster's loads in flight (n = 3001, k = 12: 18 ->
// 9.4 us with the norms and sums included; n = 60000, k = 10: 63 -> 18 us; n =
// 100000, k = 64: 73 -> 29 us, 57 MB moved).  D's rows (a contiguous stretch of
// 64 k floats) leave through LDS as whole lines when k <= 128.
//
// SMALL (one problem whose slots x strips of own-cluster sums are few): each
// wave also computes the centroid norms of its clusters, and the last workgroup
// to arrive adds up the parts, so neither takes a launch.  With few workgroups
// the fence that orders the parts costs less than a launch; with hundreds it
// does not.
template <int NW, bool MULTI, bool SMALL>
__global__ __launch_bounds__(NW *kWave) void assign_fused(InstSet s, const int32_t *labels_in_all,
                                                          int32_t *labels_out_all, int stage_d) {
    static_assert(kPtsPerBlock == 4 * kAssignPts && NW * kWave >= kPtsPerBlock, "four workgroups per label block");
    extern __shared__ int32_t sh[];  // off[k+1], hist[k], ct[k], first[k], slots[k], D rows
    __shared__ float wbest[NW][kAssignPts], wown[NW][kAssignPts];
    __shared__ int32_t warg[NW][kAssignPts];
    __shared__ double wJ[4];
    __shared__ long long wC[4];
    __shared__ int32_t last;
    constexpr int NT = NW * kWave;
    Inst in;
    int64_t lb;
    // the label blocks' grid, four workgroups to a block
    if (!locate<MULTI>(s, s.blk_start, blockIdx.x >> 2, in, lb)) return;
    lb = 4 * lb + (blockIdx.x & 3);
    if (lb * kAssignPts >= in.n) return;  // uniform
    const int32_t k = in.k;
    const int64_t ldp = in.ldp;
    const int32_t *__restrict__ labels_in = labels_in_all + in.lab_off;
    int32_t *__restrict__ labels_out = labels_out_all + in.lab_off;
    int32_t *off = sh;
    int32_t *hist = sh + (k + 1);
    float *ct = reinterpret_cast<float *>(hist + k);
    int32_t *first = hist + 2 * k, *slots = hist + 3 * k;
    float *dst = reinterpret_cast<float *>(hist + 4 * k);  // row stride odd: no bank conflicts
    const int dld = k | 1;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // what every point needs, loaded at once: a chain of dependent loads is most
    // of this kernel's time when the problem is small
    const int32_t bad = *in.err;
    const int64_t i = lb * kAssignPts + lane;
    const bool valid = i < in.n;
    const float dii = in.diag[min(i, in.n - 1)];
    const int32_t a_in = valid ? labels_in[i] : -1;
    for (int c = tid; c <= k; c += NT) off[c] = in.offsets[c];
    for (int c = tid; c < k; c += NT) {
        hist[c] = 0;
        if constexpr (!SMALL) ct[c] = in.ctilde[c];
    }
    if (bad != 0) {
        if (lb == 0 && tid == 0) {
            *in.n_changed = -1;
            *in.J_in = __builtin_nan("");
        }
        return;
    }
    __syncthreads();
    // segment (q, c) of the sweep sits in slot q + c: cluster c has the slots of
    // the chunks its positions lie in (positions and L fit 32 bits)
    for (int c = tid; c < k; c += NT) {
        const uint32_t lo = (uint32_t)off[c], hi = (uint32_t)off[c + 1], L = (uint32_t)in.L;
        const uint32_t q0 = lo / L;
        first[c] = (int32_t)q0 + c;
        slots[c] = hi > lo ? (int32_t)((hi - 1) / L - q0) + 1 : 0;
    }
    __syncthreads();

    float best = __builtin_inff(), own = 0.f;
    int32_t arg = -1;
    const float empty_d = (in.empty_policy == KKM_EMPTY_ZERO_CENTROID) ? dii : __builtin_inff();
    const float *__restrict__ Pi = in.P + min(i, in.n - 1);
    // the first eight partials of a cluster (or of none: c >= k)
    struct Head {
        int32_t s0, m, cnt;
        float v[8];
    };
    auto load8 = [&](const float *Ps, int32_t t0, int32_t m, float (&v)[8]) {
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = (t0 + u < m) ? Ps[(t0 + u) * ldp] : 0.f;
    };
    auto head_of = [&](int32_t c, Head &h) {
        h.s0 = c < k ? __builtin_amdgcn_readfirstlane(first[c]) : 0;
        h.m = c < k ? __builtin_amdgcn_readfirstlane(slots[c]) : 0;
        h.cnt = c < k ? __builtin_amdgcn_readfirstlane(off[c + 1] - off[c]) : 0;
        load8(Pi + h.s0 * ldp, 0, h.m, h.v);
    };
    Head cur, ahead;
    head_of(wave, cur);
#pragma unroll 1
    for (int32_t c = wave; c < k; c += NW) {
        head_of(c + NW, ahead);  // the next cluster's loads wait with this one's
        float dic = empty_d, norm = 0.f;
        if (cur.m > 0) {
            // S_ic: the compensated sum of the cluster's partials in CSR order
            float sum = 0.f, comp = 0.f;
            auto add = [&](const float (&v)[8]) {
#pragma unroll
                for (int u = 0; u < 8; ++u) {  // adding 0 past the last slot changes nothing
                    float x, er;
                    two_sum(sum, v[u], x, er);
                    sum = x;
                    comp += er;
                }
            };
            if constexpr (SMALL)  // the cluster's slots follow each other
                norm = __shfl(cluster_norm_wave(in.Zp + (int64_t)cur.s0 * in.nws, cur.m * (int32_t)in.nws,
                                                cur.cnt, lane), 0, kWave);
            else
                norm = ct[c];
            add(cur.v);
            for (int32_t t0 = 8; t0 < cur.m; t0 += 8) {
                float v[8];
                load8(Pi + cur.s0 * ldp, t0, cur.m, v);
                add(v);
            }
            dic = fmaf(-2.0f, (sum + comp) / (float)cur.cnt, dii) + norm;
        }
        if constexpr (SMALL)
            if (lb == 0 && lane == 0 && in.ctilde_out) in.ctilde_out[c] = norm;
        if (stage_d)
            dst[lane * dld + c] = dic;
        else if (in.D_out && valid)
            in.D_out[i * k + c] = dic;
        if (c == a_in) own = dic;
        if (dic < best) {
            best = dic;
            arg = c;
        }
        cur = ahead;
    }
    wbest[wave][lane] = best;
    warg[wave][lane] = arg;
    wown[wave][lane] = own;  // 0 but in the wave of the point's own cluster
    __syncthreads();
    if (wave == 0) {
        double own_d = 0.0;
        long long changed = 0;
        if (valid) {
            for (int w = 1; w < NW; ++w) {
                const float b = wbest[w][lane];
                const int32_t a = warg[w][lane];
                own += wown[w][lane];
                if (b < best || (b == best && a >= 0 && a < arg)) {  // ties: the lowest index
                    best = b;
                    arg = a;
                }
            }
            if (arg < 0) arg = a_in;
            labels_out[i] = arg;
            atomicAdd(&hist[arg], 1);
            changed = (arg != a_in);
            own_d = (double)own;
        }
        const double wj = wave_sum(own_d);
        const long long wc = wave_sum(changed);
        if (lane == 0) {
            part_store<SMALL>(&assign_parts(in)[lb].J, wj);
            part_store<SMALL>(&assign_parts(in)[lb].changed, (int64_t)wc);
        }
    }
    if (stage_d) {
        // element e of the block's rows is (e / k, e % k): stepped, not divided
        const int total = (int)min((int64_t)kAssignPts, in.n - lb * kAssignPts) * k;
        float *out = in.D_out + lb * kAssignPts * (int64_t)k;
        const int dr = NT / k, dc = NT % k;
        int r = tid / k, c = tid % k;
        for (int e = tid; e < total; e += NT) {
            out[e] = dst[r * dld + c];
            r += dr;
            c += dc;
            if (c >= k) {
                c -= k;
                ++r;
            }
        }
    }
    __syncthreads();
    if constexpr (!SMALL) {
        for (int c = tid; c < k; c += NT) part_store<SMALL>(assign_sizes(in, c) + lb, (uint8_t)hist[c]);
    } else {
        // every part leaves by the wave whose first lane then arrives, so that its
        // release waits for all of them: a wave waits for its own stores only, and
        // a barrier for none
        if (wave == 0)
            for (int c = lane; c < k; c += kWave) part_store<SMALL>(assign_sizes(in, c) + lb, (uint8_t)hist[c]);
        if (tid == 0)
            last = __hip_atomic_fetch_add(in.err + 1, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) ==
                   (int32_t)assign_blocks(in) - 1;
        __syncthreads();
        if (!last) return;  // uniform
        for (int32_t c = tid >> 4; c < k; c += NT / 16)  // 16 lanes read up to 64 blocks' sizes at once
            finish_size<true, 16>(in, c, tid & 15);
        finish_objective<true>(in, wJ, wC);
    }
}

// The end of a step: one workgroup per (problem, cluster) adds the cluster's
// size, cluster 0's also the objective and the changed count (a kernel of its
// own: a device-wide release fence in every assignment workgroup of a large
// problem costs far more than this launch).
template <bool MULTI>
__global__ __launch_bounds__(kPtsPerBlock) void step_finish(InstSet s) {
    __shared__ double wJ[kPtsPerBlock / kWave];
    __shared__ long long wC[kPtsPerBlock / kWave];
    Inst in;
    int64_t c;
    if (!locate<MULTI>(s, s.cl_start, blockIdx.x, in, c)) return;
    if (*in.err != 0) return;  // the assignment has published NaN
    if (threadIdx.x < kWave) finish_size<false, kWave>(in, (int32_t)c, threadIdx.x);
    if (c == 0) finish_objective<false>(in, wJ, wC);
}

// Geometry shared by the workspace sizing and the kernels.
int64_t chunk_rows(int64_t n) {
    // the largest power of two in [64, 4096] that still gives about 8192 sweep
    // workgroups of 1024 FP32 columns (the partial sums cost slots * n floats)
    const int64_t nstrip = (n + 1023) / 1024;
    int64_t L = 4096;
    while (L > 64 && ((n + L - 1) / L) * nstrip < 8192) L >>= 1;
    return L;
}

}  // namespace

InstGeom inst_geometry(int64_t n, int32_t k, int64_t L) {
    InstGeom g;
    g.n = n;
    g.k = k;
    g.L = (L > 0) ? L : chunk_rows(n);
    g.nblk = (n + kPtsPerBlock - 1) / kPtsPerBlock;
    g.nchunk = (n + g.L - 1) / g.L;
    g.slots = g.nchunk + k;
    g.ldp = (n + 63) & ~int64_t(63);
    g.nws_max = (n + kWave * 4 - 1) / (kWave * 4);  // FP32 K: the most wave strips
    return g;
}

size_t inst_workspace_bytes(const InstGeom &g) {
    size_t bytes = 0;
    inst_carve(nullptr, g, nullptr, &bytes);
    return bytes;
}

void inst_carve(void *base, const InstGeom &g, Inst *in, size_t *bytes) {
    Carver c(base);
    int32_t *perm = c.take<int32_t>((size_t)g.n);
    int32_t *offsets = c.take<int32_t>((size_t)g.k + 1);
    int32_t *counts = c.take<int32_t>((size_t)g.k);
    int32_t *blk_hist = c.take<int32_t>((size_t)g.k * (size_t)g.nblk);
    int32_t *blk_bad = c.take<int32_t>((size_t)g.nblk);
    int32_t *err = c.take<int32_t>(2);  // bad labels; the assignment's arrival counter
    float *P = c.take<float>((size_t)g.slots * (size_t)g.ldp);
    float *Zp = c.take<float>((size_t)g.slots * (size_t)g.nws_max);
    float *ctilde = c.take<float>((size_t)g.k);
    if (bytes) *bytes = c.bytes();
    if (!in) return;
    in->n = g.n;
    in->k = g.k;
    in->L = g.L;
    in->nblk = g.nblk;
    in->ldp = g.ldp;
    in->perm = perm;
    in->offsets = offsets;
    in->counts = counts;
    in->blk_hist = blk_hist;
    in->blk_bad = blk_bad;
    in->err = err;
    in->P = P;
    in->Zp = Zp;
    in->ctilde = ctilde;
}

int64_t inst_sweep_items(const InstGeom &g, int32_t k_store) {
    const int64_t cols = (int64_t)kSweepThreads * ((k_store == KKM_BF16) ? 8 : 4);
    return ((g.n + cols - 1) / cols) * g.nchunk;
}

void inst_set_store(Inst *in, int32_t k_store) {
    const int64_t E = (k_store == KKM_BF16) ? 8 : 4;
    in->nstrip = (in->n + kSweepThreads * E - 1) / (kSweepThreads * E);
    in->nws = (in->n + kWave * E - 1) / (kWave * E);
}

namespace {

// One problem small enough for the one-workgroup CSR build (its labels wait in
// registers, eight per thread; k bounds its LDS): 5 us at n = 3001 for the three
// launches' 11 us and their gaps.
bool small_csr(int64_t n, int32_t k) { return n <= kSmallPts && k <= 256; }

// Centroid norms and J inside the assignment: every workgroup reads all the
// own-cluster sums, so only while those are few.
bool small_norms(const Inst &in) {
    return small_csr(in.n, in.k) && ((in.n + in.L - 1) / in.L + in.k) * in.nws <= 4096;
}

// Chunks of at most 64 positions of a K small enough that the sweep's
// workgroups do not fill the chip: the eight-wave sweep.
bool small_sweep(const Inst &in) { return in.L <= kWave && in.n <= kSmallPts; }

template <bool MULTI>
kkm_status csr_launch(const InstSet &s, int64_t total_blocks, int64_t total_clusters, int32_t max_k,
                      const int32_t *labels_in, hipStream_t stream) {
    const dim3 pb(kPtsPerBlock);
    hipLaunchKernelGGL(v_block_hist<MULTI>, dim3((unsigned)total_blocks), pb,
                       (size_t)(max_k + 1) * sizeof(int32_t), stream, s, labels_in);
    KKM_HIP(hipGetLastError());
    hipLaunchKernelGGL(v_cluster_scan<MULTI>, dim3((unsigned)total_clusters), dim3(256), 0, stream, s);
    KKM_HIP(hipGetLastError());
    hipLaunchKernelGGL(v_scatter<MULTI>, dim3((unsigned)total_blocks), pb,
                       (size_t)(max_k + 1 + 4 * max_k) * sizeof(int32_t), stream, s, labels_in);
    KKM_HIP(hipGetLastError());
    return KKM_OK;
}

// V of one problem.
kkm_status csr_one(const InstSet &s, const int32_t *labels_in, hipStream_t stream) {
    const Inst &in = s.one;
    if (!small_csr(in.n, in.k)) return csr_launch<false>(s, in.nblk, in.k, in.k, labels_in, stream);
    hipLaunchKernelGGL(v_csr_small, dim3(1), dim3(kSmallThreads),
                       (size_t)(1 + kSmallThreads / kWave) * in.k * sizeof(int32_t), stream, in,
                       labels_in);
    KKM_HIP(hipGetLastError());
    return KKM_OK;
}

// Four waves cover up to 8 clusters in two rounds; sixteen take more, while the
// workgroups are few: with many the chip is full either way and large workgroups
// fill it worse (n = 100000, k = 64: 52 us with sixteen, 29 us with four; n =
// 3001, k = 12: 9.4 us with sixteen).  The results do not depend on it.
constexpr int64_t kAssignWide = 128;  // label blocks
template <bool MULTI, bool SMALL>
kkm_status assign_launch(const InstSet &s, int64_t total_blocks, int32_t max_k, const int32_t *labels_in,
                         int32_t *labels_out, hipStream_t stream) {
    const int stage_d = !MULTI && s.one.D_out && max_k <= kAssignStageK;
    size_t lds = (size_t)(5 * max_k + 1) * sizeof(int32_t);
    if (stage_d) lds += (size_t)kAssignPts * (max_k | 1) * sizeof(float);
    const dim3 grid((unsigned)(4 * total_blocks));
    if (max_k <= 8 || total_blocks > kAssignWide)
        hipLaunchKernelGGL((assign_fused<4, MULTI, SMALL>), grid, dim3(4 * kWave), lds, stream, s, labels_in,
                           labels_out, stage_d);
    else
        hipLaunchKernelGGL((assign_fused<16, MULTI, SMALL>), grid, dim3(16 * kWave), lds, stream, s, labels_in,
                           labels_out, stage_d);
    KKM_HIP(hipGetLastError());
    return KKM_OK;
}

// Centroid norms, assignment and objective.
template <bool MULTI>
kkm_status finish_launch(const InstSet &s, int64_t total_blocks, int64_t total_clusters, int32_t max_k,
                         const int32_t *labels_in, int32_t *labels_out, hipStream_t stream) {
    if (!MULTI && small_norms(s.one))
        return assign_launch<false, true>(s, total_blocks, max_k, labels_in, labels_out, stream);
    hipLaunchKernelGGL(centroid_norms<MULTI>, dim3((unsigned)total_clusters), dim3(256), 0, stream, s);
    KKM_HIP(hipGetLastError());
    KKM_TRY((assign_launch<MULTI, false>(s, total_blocks, max_k, labels_in, labels_out, stream)));
    hipLaunchKernelGGL(step_finish<MULTI>, dim3((unsigned)total_clusters), dim3(kPtsPerBlock), 0, stream, s);
    KKM_HIP(hipGetLastError());
    return KKM_OK;
}

template <bool MULTI>
kkm_status step_launch_t(const InstSet &s, int64_t total_blocks, int64_t total_clusters,
                         int64_t sweep_grid, int32_t max_k, int32_t k_store, bool vec,
                         const int32_t *labels_in, int32_t *labels_out, hipStream_t stream) {
    const TimedSpan whole = timing_begin(TK_ITERATE, stream);
    if constexpr (MULTI)
        KKM_TRY(csr_launch<true>(s, total_blocks, total_clusters, max_k, labels_in, stream));
    else
        KKM_TRY(csr_one(s, labels_in, stream));
    const TimedSpan span = timing_begin(TK_SWEEP, stream);
    if (!MULTI && small_sweep(s.one)) {
        const dim3 sg((unsigned)(s.one.nws * ((s.one.n + s.one.L - 1) / s.one.L))), sb(kSmallWaves * kWave);
        if (k_store == KKM_F32 && vec)
            hipLaunchKernelGGL((spmm_small_sweep<float, true>), sg, sb, 0, stream, s.one, labels_in);
        else if (k_store == KKM_F32)
            hipLaunchKernelGGL((spmm_small_sweep<float, false>), sg, sb, 0, stream, s.one, labels_in);
        else if (vec)
            hipLaunchKernelGGL((spmm_small_sweep<uint16_t, true>), sg, sb, 0, stream, s.one, labels_in);
        else
            hipLaunchKernelGGL((spmm_small_sweep<uint16_t, false>), sg, sb, 0, stream, s.one, labels_in);
    } else {
        const dim3 sg((unsigned)sweep_grid), sb(kSweepThreads);
        if (k_store == KKM_F32 && vec)
            hipLaunchKernelGGL((spmm_row_sweep<float, true, MULTI>), sg, sb, 0, stream, s, labels_in);
        else if (k_store == KKM_F32)
            hipLaunchKernelGGL((spmm_row_sweep<float, false, MULTI>), sg, sb, 0, stream, s, labels_in);
        else if (vec)
            hipLaunchKernelGGL((spmm_row_sweep<uint16_t, true, MULTI>), sg, sb, 0, stream, s, labels_in);
        else
            hipLaunchKernelGGL((spmm_row_sweep<uint16_t, false, MULTI>), sg, sb, 0, stream, s, labels_in);
    }
    KKM_HIP(hipGetLastError());
    timing_end(span, stream);
    KKM_TRY(finish_launch<MULTI>(s, total_blocks, total_clusters, max_k, labels_in, labels_out, stream));
    timing_end(whole, stream);
    return KKM_OK;
}

}  // namespace

kkm_status step_launch(const InstSet &s, int64_t total_blocks, int64_t total_clusters,
                       int64_t sweep_grid, int32_t max_k, int32_t k_store, bool vec,
                       const int32_t *labels_in, int32_t *labels_out, hipStream_t stream) {
    if (s.table)
        return step_launch_t<true>(s, total_blocks, total_clusters, sweep_grid, max_k, k_store,
                                   vec, labels_in, labels_out, stream);
    return step_launch_t<false>(s, total_blocks, total_clusters, sweep_grid, max_k, k_store, vec,
                                labels_in, labels_out, stream);
}

// One step of a single problem whose sweep is supplied by the caller: the CSR
// build of V, then `sweep` (it fills in.P and in.Zp as spmm_row_sweep does:
// slot q + c of P holds, for every column, the sum over the positions of
// chunk q in cluster c, and Zp[(q + c) nws + w] that slot's own-cluster sum
// over the w-th strip of in.n / in.nws columns), then the centroid norms, the
// fused assignment and the objective.
kkm_status step_launch_custom(const Inst &in, const int32_t *labels_in, int32_t *labels_out,
                              const std::function<kkm_status(hipStream_t)> &sweep,
                              hipStream_t stream) {
    InstSet s{};
    s.count = 1;
    s.one = in;
    const TimedSpan whole = timing_begin(TK_ITERATE, stream);
    KKM_TRY(csr_one(s, labels_in, stream));
    KKM_TRY(sweep(stream));  // times its own launches
    KKM_TRY(finish_launch<false>(s, in.nblk, in.k, in.k, labels_in, labels_out, stream));
    timing_end(whole, stream);
    return KKM_OK;
}

// V in CSR form for one problem (used by the feature-space Lloyd iterations):
// the first three kernels of a step on a set of one.
kkm_status vcsr_build(const int32_t *labels, int64_t n, int32_t k, int32_t *blk_hist,
                      int32_t *blk_bad, int32_t *err, int32_t *counts, int32_t *perm,
                      int32_t *offsets, int32_t *counts_out, int64_t *n_changed,
                      hipStream_t stream) {
    InstSet s{};
    s.count = 1;
    Inst &in = s.one;
    in.n = n;
    in.k = k;
    in.nblk = (n + kPtsPerBlock - 1) / kPtsPerBlock;
    in.blk_hist = blk_hist;
    in.blk_bad = blk_bad;
    in.err = err;
    in.counts = counts;
    in.perm = perm;
    in.offsets = offsets;
    in.counts_out = counts_out;
    in.n_changed = n_changed;
    return csr_launch<false>(s, in.nblk, k, k, labels, stream);
}

size_t iterate_workspace_bytes(int64_t n, int32_t k) {
    return inst_workspace_bytes(inst_geometry(n, k, 0));
}

kkm_status iterate_launch(const void *K, int32_t k_store, int64_t ldk, const float *diagK,
                          int64_t n, int32_t k, const int32_t *labels_in, int32_t empty_policy,
                          int32_t *labels_out, int32_t *counts_out, int64_t *n_changed,
                          double *J_in, float *D_out, float *ctilde_out, void *ws,
                          size_t ws_bytes, hipStream_t stream) {
    const InstGeom g = inst_geometry(n, k, 0);
    size_t need = 0;
    inst_carve(nullptr, g, nullptr, &need);
    if (ws == nullptr || ws_bytes < need) {
        set_error("kkm_iterate: workspace of %zu bytes is smaller than %zu", ws_bytes, need);
        return KKM_ERR_NOMEM;
    }
    InstSet s{};
    s.count = 1;
    Inst &in = s.one;
    inst_carve(ws, g, &in, nullptr);
    in.K = K;
    in.ldk = ldk;
    in.diag = diagK;
    in.lab_off = 0;
    in.empty_policy = empty_policy;
    in.counts_out = counts_out;
    in.n_changed = n_changed;
    in.J_in = J_in;
    in.D_out = D_out;
    in.ctilde_out = ctilde_out;
    inst_set_store(&in, k_store);
    const int E = (k_store == KKM_BF16) ? 8 : 4;
    const bool vec = ((ldk % E) == 0) && ((reinterpret_cast<uintptr_t>(K) & 15) == 0);
    return step_launch(s, g.nblk, k, inst_sweep_items(g, k_store), k, k_store, vec, labels_in,
                       labels_out, stream);
}

}  // namespace kkm
