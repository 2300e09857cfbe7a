// Cheap iterations of the learned warm start: Lloyd's algorithm (the three
// phases of the paper's Sec. 2.1) with explicit centroids on the feature rows
// F = phi_theta(X) (n x f).  One step costs O(n f k) instead of the O(n^2) of
// an exact step.  Per step:
//   1. V in CSR form from the labels (shared with the exact step);
//   2. centroid sums: chunks of CSR positions, running per-feature sums flushed
//      at cluster boundaries (slot chunk + cluster), then a fixed-order reduce
//      that also forms ||c_c||^2;
//   3. G = F C^T on MFMA (FP32), d_ic = ||f_i||^2 - 2 G_ic + ||c_c||^2 and its
//      argmin (lowest index on ties, an empty cluster at +inf) from the
//      accumulators, changed count.
//
// All of it reads F's rows (51 MB at n = 50000, f = 256, which stay in the
// last-level cache) and is bound by how many of those loads are in flight: none
// sits behind a branch, where the compiler would wait for each before the next.
#include "gemm_small.h"

namespace kkm {

kkm_status vcsr_build(const int32_t *labels, int64_t n, int32_t k, int32_t *blk_hist,
                      int32_t *blk_bad, int32_t *err, int32_t *counts, int32_t *perm,
                      int32_t *offsets, int32_t *counts_out, int64_t *n_changed,
                      hipStream_t stream);

namespace {

constexpr int64_t kRows = 64;  // CSR positions per centroid-sum chunk

struct LloydWs {
    int32_t *blk_hist, *blk_bad, *err, *counts, *perm, *offsets, *counts_out;
    int64_t *changed;
    float *fn, *Cp, *C, *cn;
    int32_t *lab[2];
    double *part, *obj;
};

LloydWs carve_lloyd(void *base, int64_t n, int64_t f, int32_t k, size_t *bytes) {
    const int64_t nblk = (n + 255) / 256;
    const int64_t slots = (n + kRows - 1) / kRows + k;
    Carver c(base);
    LloydWs w;
    w.blk_hist = c.take<int32_t>((size_t)(k * nblk));
    w.blk_bad = c.take<int32_t>((size_t)nblk);
    w.err = c.take<int32_t>(1);
    w.counts = c.take<int32_t>((size_t)k);
    w.perm = c.take<int32_t>((size_t)n);
    w.offsets = c.take<int32_t>((size_t)k + 1);
    w.counts_out = c.take<int32_t>((size_t)k);
    w.changed = c.take<int64_t>(1);
    w.fn = c.take<float>((size_t)n);
    w.Cp = c.take<float>((size_t)(slots * f));
    w.C = c.take<float>((size_t)(k * f));
    w.cn = c.take<float>((size_t)k);
    w.lab[0] = c.take<int32_t>((size_t)n);
    w.lab[1] = c.take<int32_t>((size_t)n);
    w.part = c.take<double>((size_t)((n + 63) / 64));
    w.obj = c.take<double>(1);
    if (bytes) *bytes = c.bytes();
    return w;
}

// Four columns of a row in flight per lane (a row's sum is in column order).
__global__ __launch_bounds__(256) void feature_sqnorms(const float *F, int64_t n, int64_t f, int64_t ldf, float *fn) {
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= n) return;
    const float *x = F + row * ldf;
    float s = 0.f;
    for (int64_t t = lane; t < f; t += 4 * kWave) {
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = x[min(t + u * kWave, f - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (t + u * kWave < f) s = fmaf(v[u], v[u], s);
    }
    s = wave_sum(s);
    if (lane == 0) fn[row] = s;
}

// One wave per (chunk of kRows CSR positions, block of 256 features): lane l
// owns features 4l .. 4l+3 of the block; rows are read sixteen at a time and
// summed in order per cluster segment, flushed to slot chunk + cluster.  VEC:
// rows of whole 16-byte quads.  (n = 50000, f = 256: 28.6 us with each load
// behind a branch, 14.4 us so.)
template <bool VEC>
__global__ __launch_bounds__(256) void centroid_partials(const float *F, int64_t n, int64_t f,
                                                         int64_t ldf, int32_t k, int64_t nchunk,
                                                         const int32_t *perm,
                                                         const int32_t *offsets, float *Cp) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int64_t q = (int64_t)blockIdx.x * 4 + wave;
    if (q >= nchunk) return;
    const int64_t t0 = (int64_t)blockIdx.y * 256 + lane * 4;
    const int64_t p0 = q * kRows, p1 = min(n, p0 + kRows);
    static_assert(kRows == kWave, "a chunk's rows, one per lane");
    const int32_t rows = perm[min(p0 + lane, n - 1)];
    // each position's cluster: the last c with offsets[c] <= position
    int32_t lo = 0, hi = k - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (offsets[mid] <= min(p0 + lane, n - 1)) lo = mid;
        else hi = mid - 1;
    }
    const int cnt = (int)(p1 - p0);
    constexpr int U = 16;
    f32x4 v[U];
    auto fetch = [&](int first) {  // rows first .. of the chunk, its last again past it
#pragma unroll
        for (int r = 0; r < U; ++r) {
            const int64_t j = __builtin_amdgcn_readlane(rows, min(first + r, cnt - 1));
            v[r] = line4<VEC>(F + j * ldf, 0, t0, f, true);
        }
    };
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    for (int g = 0; g < cnt; g += U) {
        fetch(g);
#pragma unroll
        for (int r = 0; r < U; ++r)
            if (g + r < cnt) {  // uniform
                const int32_t c = __builtin_amdgcn_readlane(lo, g + r);
#pragma unroll
                for (int u = 0; u < 4; ++u) s[u] += v[r][u];
                if (g + r + 1 == cnt || __builtin_amdgcn_readlane(lo, min(g + r + 1, kWave - 1)) != c) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        if (t0 + u < f) Cp[(q + c) * f + t0 + u] = s[u];
                        s[u] = 0.f;
                    }
                }
            }
    }
}

// One workgroup per cluster: centroid = sum of its chunk partials / |c|, and
// ||c||^2.  Thread t takes features 4 (t % 64) .. + 3 of each 256-feature
// block and chunks t / 64, t / 64 + 4, ...; the four chunk lanes are then
// added pairwise in a fixed order.
__global__ __launch_bounds__(256) void centroid_finalize(const float *Cp, int64_t f, int32_t k,
                                                         const int32_t *offsets, float *C,
                                                         float *cn) {
    __shared__ f32x4 part[4][64];
    __shared__ float sh[256];
    const int c = blockIdx.x;
    const int tid = threadIdx.x, fq = tid & 63, cl = tid >> 6;
    const int64_t a = offsets[c], b = offsets[c + 1];
    const int64_t q0 = (b > a) ? a / kRows : 0, q1 = (b > a) ? (b - 1) / kRows : -1;
    const bool vec = (f & 3) == 0 && (reinterpret_cast<uintptr_t>(Cp) & 15) == 0;
    float sq = 0.f;
    for (int64_t f0 = 0; f0 < f; f0 += 256) {
        const int64_t t0 = f0 + 4 * fq;
        f32x4 s = {0.f, 0.f, 0.f, 0.f};
        for (int64_t q = q0 + cl; q <= q1; q += 4 * 8) {  // eight chunks in flight, added in order
            f32x4 v[8];
            auto load = [&](auto whole) {
#pragma unroll
                for (int r = 0; r < 8; ++r)
                    v[r] = line4<decltype(whole)::value>(Cp, (min(q + 4 * r, q1) + c) * f, t0, f, true);
            };
            if (vec)  // uniform
                load(std::true_type{});
            else
                load(std::false_type{});
#pragma unroll
            for (int r = 0; r < 8; ++r)
                if (q + 4 * r <= q1) s += v[r];
        }
        part[cl][fq] = s;
        __syncthreads();
        if (cl == 0) {
            const f32x4 tot = (part[0][fq] + part[1][fq]) + (part[2][fq] + part[3][fq]);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (t0 + u >= f) break;
                // sum / |c| (an empty cluster keeps a zero centroid)
                const float v = (b > a) ? tot[u] / (float)(b - a) : 0.f;
                C[(int64_t)c * f + t0 + u] = v;
                sq = fmaf(v, v, sq);
            }
        }
        __syncthreads();
    }
    sh[tid] = sq;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (tid < h) sh[tid] += sh[tid + h];
        __syncthreads();
    }
    if (tid == 0) cn[c] = sh[0];
}

// The product G = F C^T and the assignment in one kernel: a workgroup takes 128
// points, a wave 32 of them, and 32 MT clusters at a time; a lane holds 16
// clusters of one point per MFMA block and keeps the smallest distance so far
// (clusters in ascending order, strictly smaller wins), the point's two lanes
// are joined at the end.  G never reaches memory: as a product of 64 x 256
// tiles, its store and a pass over it these were 37 + 14 us at n = 50000, k =
// 32, f = 256; here 18 us for 51 MB of F.
//
// 64 features are staged at a time, the next 64 in registers.  NATURAL: the
// MFMA chain takes features in order, else within each 32 as 0, 16, 1, 17, ...
// (large problems: whole 16-byte reads of LDS rows; the order decides the last
// bit of a distance).
//
// part (nullable): per 64 points, the sum of the chosen distances in FP64;
// summed over all points it is the objective of the new labels once no label
// changes.
constexpr int NP = 128;       // points per workgroup
constexpr int NK = 64;        // features staged at a time
constexpr int NLD = NK + 4;

template <int MT, bool NATURAL>
__global__ __launch_bounds__(256) void feature_nearest(const float *F, int64_t ldf, int64_t f, int vec_f,
                                                       const float *C, int vec_c, const float *fn, const float *cn,
                                                       const int32_t *offsets, int64_t n, int32_t k,
                                                       const int32_t *labels_in, int32_t *labels_out,
                                                       int64_t *changed, double *part) {
    __shared__ __attribute__((aligned(16))) float a[32 * MT][NLD];
    __shared__ __attribute__((aligned(16))) float b[NP][NLD];
    __shared__ float cnorm[32 * MT];
    __shared__ double dm[NP];
    __shared__ long long wc[4];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int64_t n0 = (int64_t)blockIdx.x * NP;
    const int lr = tid >> 4, lc = (tid & 15) * 4;  // 16 threads x 4 floats per row
    constexpr int RA = 2 * MT, RB = NP / 16;
    f32x4 ra[RA], rb[RB];
    auto gload = [&](int32_t c0, int64_t k0) {
        auto load = [&](auto vf, auto vc) {
#pragma unroll
            for (int u = 0; u < RA; ++u)
                ra[u] = line4<decltype(vc)::value>(C, (int64_t)(c0 + lr + 16 * u) * f, k0 + lc, f, c0 + lr + 16 * u < k);
#pragma unroll
            for (int u = 0; u < RB; ++u)
                rb[u] = line4<decltype(vf)::value>(F, (n0 + lr + 16 * u) * ldf, k0 + lc, f, n0 + lr + 16 * u < n);
        };
        if (vec_f && vec_c)  // uniform
            load(std::true_type{}, std::true_type{});
        else
            load(std::false_type{}, std::false_type{});
    };
    // feature kk of a 32-wide slab sits where the fragment reads want it
    auto store = [&](float *row, f32x4 v) {
        if constexpr (NATURAL) {  // MFMA s takes 2s + half: even features first, then odd ones
            float *at = row + (lc & 32) + ((lc & 31) >> 1);
            at[0] = v[0];
            at[1] = v[2];
            at[16] = v[1];
            at[17] = v[3];
        } else {
            *reinterpret_cast<f32x4 *>(row + lc) = v;
        }
    };
    const int64_t i = n0 + 32 * wave + l32;
    const bool valid = i < n;
    const float fi = fn[min(i, n - 1)];
    const int32_t l_in = labels_in[min(i, n - 1)];
    float best = __builtin_inff();
    int32_t arg = -1;
    for (int32_t c0 = 0; c0 < k; c0 += 32 * MT) {
        f32x16 acc[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[m][r] = 0.f;
        gload(c0, 0);
        // an empty cluster is never chosen: its norm is +inf
        if (tid < 32 * MT) {
            const int32_t c = min(c0 + tid, k - 1);
            const bool there = c0 + tid < k && offsets[c + 1] != offsets[c];
            const float v = cn[c];
            cnorm[tid] = there ? v : __builtin_inff();
        }
        for (int64_t k0 = 0; k0 < f; k0 += NK) {
#pragma unroll
            for (int u = 0; u < RA; ++u)
                store(a[lr + 16 * u], mask4(ra[u], k0 + lc, f, c0 + lr + 16 * u < k));
#pragma unroll
            for (int u = 0; u < RB; ++u)
                store(b[lr + 16 * u], mask4(rb[u], k0 + lc, f, n0 + lr + 16 * u < n));
            __syncthreads();
            if (k0 + NK < f) gload(c0, k0 + NK);
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2) {
                if (s2 && k0 + 32 >= f) break;  // uniform: a slab of zeros
                f32x4 bv[4], av[MT][4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    bv[u] = *reinterpret_cast<const f32x4 *>(&b[32 * wave + l32][32 * s2 + 16 * half + 4 * u]);
#pragma unroll
                    for (int m = 0; m < MT; ++m)
                        av[m][u] = *reinterpret_cast<const f32x4 *>(&a[32 * m + l32][32 * s2 + 16 * half + 4 * u]);
                }
#pragma unroll
                for (int s = 0; s < 16; ++s)
#pragma unroll
                    for (int m = 0; m < MT; ++m)
                        acc[m] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[m][s >> 2][s & 3], bv[s >> 2][s & 3], acc[m], 0, 0, 0);
            }
            __syncthreads();
        }
        // register r of a lane: cluster 8 (r / 4) + 4 half + r % 4 of its block
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int cl = 32 * m + 8 * (r >> 2) + 4 * half + (r & 3);
                const float d = fmaf(-2.0f, acc[m][r], fi) + cnorm[cl];
                if (d < best) {
                    best = d;
                    arg = c0 + cl;
                }
            }
        __syncthreads();  // the norms are read before the next clusters' are written
    }
    {
        const float ob = __shfl_xor(best, 32, kWave);
        const int32_t oa = __shfl_xor(arg, 32, kWave);
        if (oa >= 0 && (arg < 0 || ob < best || (ob == best && oa < arg))) {
            best = ob;
            arg = oa;
        }
    }
    if (arg < 0) arg = l_in;
    long long ch = 0;
    if (half == 0) {
        if (valid) {
            labels_out[i] = arg;
            ch = (arg != l_in);
        }
        dm[32 * wave + l32] = valid ? (double)fmaxf(best, 0.0f) : 0.0;
    }
    ch = wave_sum(ch);
    if (lane == 0) wc[wave] = ch;
    __syncthreads();
    if (part && wave < NP / kWave && n0 + wave * kWave < n) {
        const double w = wave_sum(dm[wave * kWave + lane]);
        if (lane == 0) part[(n0 >> 6) + wave] = w;
    }
    if (tid == 0) {
        const long long t = wc[0] + wc[1] + wc[2] + wc[3];
        if (t) atomicAdd((unsigned long long *)changed, (unsigned long long)t);
    }
}

kkm_status nearest_launch(const float *F, int64_t ldf, int64_t f, const float *C, const float *fn, const float *cn,
                          const int32_t *offsets, int64_t n, int32_t k, const int32_t *labels_in, int32_t *labels_out,
                          int64_t *changed, double *part, hipStream_t s) {
    const int vf = vec_ok(F, ldf, f), vc = vec_ok(C, f, f);
    const dim3 g((unsigned)((n + NP - 1) / NP)), b(256);
    const bool natural = !(k >= 32 && n >= 256 && (int64_t)k * n >= (1 << 20));
    // one block of clusters at a time where that covers them all
#define KKM_NEAREST(MTV, NATV) \
    hipLaunchKernelGGL((feature_nearest<MTV, NATV>), g, b, 0, s, F, ldf, f, vf, C, vc, fn, cn, offsets, n, k, \
                       labels_in, labels_out, changed, part)
    if (k <= 32 && natural) KKM_NEAREST(1, true);
    else if (k <= 32) KKM_NEAREST(1, false);
    else if (natural) KKM_NEAREST(2, true);
    else KKM_NEAREST(2, false);
#undef KKM_NEAREST
    KKM_HIP(hipGetLastError());
    return KKM_OK;
}

// Sum of the parts of 64 points, four at a time first.
__global__ __launch_bounds__(256) void sum_blocks(const double *part, int64_t np, double *out) {
    __shared__ double sh[256];
    double s = 0.0;
    for (int64_t i = 4 * threadIdx.x; i < np; i += 4 * 256) {
        double w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) w[u] = i + u < np ? part[i + u] : 0.0;
        s += (w[0] + w[1]) + (w[2] + w[3]);
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (threadIdx.x < h) sh[threadIdx.x] += sh[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = sh[0];
}

// ---------------------------------------------------------------- k-means++ seeding
//
// Seeding by D^2 sampling (Arthur and Vassilvitskii, 2007; the K-means++ the
// paper's Sec. 2.1 mentions): the first seed is row floor(u_0 n); seed t+1 is
// the first row i whose running sum of dmin exceeds u_{t+1} * sum(dmin), where
// dmin_i is the squared distance of row i to its nearest seed so far.  The
// uniforms u_t come from the caller.  Sums run in FP64 in a fixed order.

// The running sum is kept in three levels of FP64 sums: blocks of kKppRows
// rows, groups of kKppGroup rows (one update workgroup), and the total.  The
// update kernel writes the first two; a one-workgroup select kernel then
// locates the crossing level by level with block scans: ranges of groups,
// then groups, then blocks, then rows.  Each level takes the first element
// whose inclusive running sum passes the target, or its last element if
// rounding leaves the target at its very end.

constexpr int kKppRows = 4;
constexpr int kKppGroup = 256;
constexpr int kKppPerGroup = kKppGroup / kKppRows;  // block sums per group

struct KppSums {
    double *bsum;  // [ceil(n / kKppRows)]
    double *gsum;  // [ceil(n / kKppGroup)]
};

// Scan of one value per thread over the first 256 threads of a workgroup (fixed
// order; all of its threads call): returns the inclusive sum, with the exclusive sum in *excl and the total in
// *total.  The exclusive sum of thread i is bit for bit the inclusive sum of
// thread i-1, and the total that of thread 255, so "the first thread whose
// running sum passes a target" is well defined and consistent with the total.
__device__ double block_scan256(double v, double *sh, double *excl, double *total) {
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const double o = __shfl_up(v, off, kWave);
        if (lane >= off) v += o;
    }
    const double prev = __shfl_up(v, 1, kWave);
    if (lane == kWave - 1 && w < 4) sh[w] = v;
    __syncthreads();
    double base = 0.0;
    for (int q = 0; q < 4; ++q)
        if (q < w) base += sh[q];
    double t = 0.0;
    for (int q = 0; q < 4; ++q) t += sh[q];
    *total = t;
    *excl = (lane == 0) ? base : base + prev;
    __syncthreads();
    return base + v;
}

// Smallest index among a workgroup's first 256 threads whose pred is true, or -1.
__device__ int first_true256(bool pred, int *shi) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const unsigned long long m = __ballot(pred);
    if (lane == 0 && w < 4) shi[w] = m ? w * kWave + __ffsll((long long)m) - 1 : -1;
    __syncthreads();
    int r = -1;
    for (int q = 3; q >= 0; --q)
        if (shi[q] >= 0) r = shi[q];
    __syncthreads();
    return r;
}

// Index in [lo, hi) of the first element whose inclusive running sum, added
// to *run, passes target (the last one if none does), with *run advanced to
// the exclusive running sum before it.  hi - lo may exceed 256 (chunks of 256).
__device__ int64_t kpp_locate(const double *vals, int64_t lo, int64_t hi, double target, double *run,
                              double *sh, int *shi) {
    const int tid = threadIdx.x;
    double base = *run;
    if (hi - lo == 1) {  // the scan of one value
        const double v = vals[lo];
        if (!(base + v > target)) *run = (base + v) - v;
        return lo;
    }
    for (int64_t c0 = lo; c0 < hi; c0 += 256) {
        const int64_t i = c0 + tid;
        const bool in = tid < 256 && i < hi;
        const double x = vals[min(i, hi - 1)];
        const double v = in ? x : 0.0;
        double excl, tot;
        const double incl = block_scan256(v, sh, &excl, &tot);
        const int f = first_true256(in && base + incl > target, shi);
        if (f >= 0) {
            if (tid == f) sh[4] = base + excl;
            __syncthreads();
            *run = sh[4];
            __syncthreads();
            return c0 + f;
        }
        base += tot;
    }
    // rounding left the target at the very end
    *run = base - vals[hi - 1];
    return hi - 1;
}

// A seed from the sums, by the first 256 threads of a workgroup (all call);
// thread 0 writes it.
__device__ void kpp_select_seed(const KppSums &q, const float *dmin, int64_t n, double u, int32_t *seed_out) {
    __shared__ double sh[8];
    __shared__ int shi[4];
    const int64_t nb = (n + kKppRows - 1) / kKppRows, ng = (n + kKppGroup - 1) / kKppGroup;
    const int tid = threadIdx.x;
    // ranges of groups, one per thread
    const int64_t per = (ng + 255) / 256;
    const int64_t g0 = min(ng, (int64_t)min(tid, 256) * per), g1 = min(ng, g0 + per);
    double s = 0.0;
    for (int64_t g = g0; g < g1; ++g) s += q.gsum[g];
    double excl, total;
    const double incl = block_scan256(s, sh, &excl, &total);
    if (!(total > 0.0)) {
        if (tid == 0) *seed_out = (int32_t)min((int64_t)(u * (double)n), n - 1);
        return;  // every row coincides with a seed
    }
    const double target = u * total;
    int r = first_true256(g0 < g1 && incl > target, shi);
    if (r < 0) r = (int)((ng - 1) / per);  // the last non-empty range
    if (tid == r) sh[4] = excl;
    __syncthreads();
    double run = sh[4];
    __syncthreads();
    const int64_t rg0 = (int64_t)r * per, rg1 = min(ng, rg0 + per);
    const int64_t g = kpp_locate(q.gsum, rg0, rg1, target, &run, sh, shi);
    const int64_t b = kpp_locate(q.bsum, g * kKppPerGroup, min(nb, (g + 1) * kKppPerGroup), target,
                                 &run, sh, shi);
    if (tid == 0) {
        const int64_t r1 = min(n, (b + 1) * kKppRows);
        float x[kKppRows];
#pragma unroll
        for (int j = 0; j < kKppRows; ++j) x[j] = dmin[min(b * kKppRows + j, n - 1)];
        int64_t row = -1;
#pragma unroll
        for (int j = 0; j < kKppRows; ++j) {
            run += (double)x[j];
            if (row < 0 && b * kKppRows + j < r1 && run > target) row = b * kKppRows + j;
        }
        *seed_out = (int32_t)(row < 0 ? r1 - 1 : row);
    }
}

__global__ __launch_bounds__(256) void kpp_select(KppSums q, const float *dmin, int64_t n, double u,
                                                  int32_t *seed_out) {
    kpp_select_seed(q, dmin, n, u, seed_out);
}

// Block and group sums of the calling workgroup (thread i < 256 holds the
// updated dmin of row blockIdx.x * kKppGroup + i, 0 past n; all threads call).
__device__ void kpp_sums(double v, int64_t n, const KppSums &q) {
    __shared__ double sh[4];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (w < 4) {
        const int64_t row = (int64_t)blockIdx.x * kKppGroup + tid;
        const int g = lane & ~(kKppRows - 1);
        const double v0 = __shfl(v, g, kWave), v1 = __shfl(v, g + 1, kWave);
        const double v2 = __shfl(v, g + 2, kWave), v3 = __shfl(v, g + 3, kWave);
        const double bs = (v0 + v1) + (v2 + v3);
        const bool head = (lane & (kKppRows - 1)) == 0;
        if (head && row < n) q.bsum[row / kKppRows] = bs;
        const double ws = wave_sum(head ? bs : 0.0);
        if (lane == 0) sh[w] = ws;
    }
    __syncthreads();
    if (tid == 0) q.gsum[blockIdx.x] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// One seed: the select of seed t from the last step's sums (SELECT: every
// workgroup does it for itself; workgroup 0 records it), then dmin_i = min over seeds
// 0..t of |F_i - F_seed|^2 and the new sums.  `was` and `now` alternate between
// two sets, so no workgroup overwrites what another still reads.  Wave w of a
// workgroup takes rows 32w .. 32w+31 of its group, kKppPass at a time with all
// their loads in flight, the first of them before the seed is known; a row's
// squared distance is summed over 16-byte slices (lane l: columns 4l + 256j ..)
// and then across the wave, the lanes halving the rows they stand for at each
// step of the tree (same pairs, so the same sum; 17 exchanges for 16 rows where
// a tree per row took 96).  (A select kernel and an update with each load
// behind a branch were 5.8 + 21 us and two launches per seed at n = 50000, f =
// 256; here 16 us in all.  1024 threads of 16 rows each are as fast alone and
// slower beside other restarts.)
constexpr int kKppPass = 16;

struct KppState {
    float *dmin;
    KppSums q;
};

// Every workgroup's own select reads all the group sums, n / 256 of them n / 256
// times over a launch, so it pays for few groups; past them the select is a
// launch of its own again (SELECT false), in front of an update of 256 threads.
// Per seed, own select / two launches: n = 50000, f = 16 9.9 / 12.9 us, f = 256
// 14.8 / 16.4; n = 100000 14.3 / 14.3 and 22.8 / 23.7; n = 150000 22 / 16 and 36 / 33;
// n = 10^6 121 / 51 and 222 / 192; n = 4 10^6, f = 16 1053 / 194.
constexpr int64_t kKppOwnSelect = 384;  // groups
template <bool SELECT> constexpr int kpp_threads() { return SELECT ? 512 : 256; }

template <bool VEC, bool SELECT>
__global__ __launch_bounds__(kpp_threads<SELECT>()) void kpp_step(const float *F, int64_t n, int64_t f, int64_t ldf,
                                                                  int32_t *seeds, int t, int64_t first, double u,
                                                                  KppState was, KppState now) {
    constexpr int kKppWaveRows = kKppGroup / (kpp_threads<SELECT>() / kWave);
    constexpr int passes = SELECT ? 1 : kKppWaveRows / kKppPass;  // unrolled
    __shared__ float dist[kKppGroup];
    __shared__ int32_t chosen;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t r0 = (int64_t)blockIdx.x * kKppGroup + kKppWaveRows * w;
    f32x4 x[kKppPass];
    auto fetch = [&](int p, int64_t c0) {
#pragma unroll
        for (int j = 0; j < kKppPass; ++j)
            x[j] = line4<VEC>(F + min(r0 + p + j, n - 1) * ldf, 0, c0 + 4 * lane, f, true);
    };
    fetch(0, 0);
    int64_t seed = first;
    if constexpr (SELECT) {
        kpp_select_seed(was.q, was.dmin, n, u, &chosen);
        __syncthreads();
        seed = __builtin_amdgcn_readfirstlane(chosen);
    } else if (t > 0) {
        seed = seeds[t];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0 && (SELECT || t == 0)) seeds[t] = (int32_t)seed;
    const float *c = F + seed * ldf;
#pragma unroll passes
    for (int p = 0; p < kKppWaveRows; p += kKppPass) {
        float d[kKppPass];
#pragma unroll
        for (int j = 0; j < kKppPass; ++j) d[j] = 0.f;
        for (int64_t c0 = 0; c0 < f; c0 += 4 * kWave) {
            if (p > 0 || c0 > 0) fetch(p, c0);
            const f32x4 cv = line4<VEC>(c, 0, c0 + 4 * lane, f, true);
#pragma unroll
            for (int j = 0; j < kKppPass; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float df = c0 + 4 * lane + e < f ? x[j][e] - cv[e] : 0.f;
                    d[j] = fmaf(df, df, d[j]);
                }
        }
        // value 0 of lane l after the steps 32, 16, 8, 4: row l / 4
        auto halve = [&](auto half_rows) {
            constexpr int H = decltype(half_rows)::value, off = 4 * H;
            const bool up = lane & off;
#pragma unroll
            for (int j = 0; j < H; ++j) {
                const float keep = up ? d[j + H] : d[j], give = up ? d[j] : d[j + H];
                d[j] = keep + __shfl_xor(give, off, kWave);
            }
        };
        static_assert(kKppPass == 16, "four steps");
        halve(std::integral_constant<int, 8>{});
        halve(std::integral_constant<int, 4>{});
        halve(std::integral_constant<int, 2>{});
        halve(std::integral_constant<int, 1>{});
        float s = d[0] + __shfl_xor(d[0], 2, kWave);
        s += __shfl_xor(s, 1, kWave);
        if (!(lane & 3)) dist[kKppWaveRows * w + p + (lane >> 2)] = s;
    }
    __syncthreads();
    const int64_t row = (int64_t)blockIdx.x * kKppGroup + threadIdx.x;
    double v = 0.0;
    if (threadIdx.x < kKppGroup && row < n) {
        const float mine = dist[threadIdx.x];
        const float m = (t == 0) ? mine : fminf(was.dmin[row], mine);
        now.dmin[row] = m;
        v = (double)m;
    }
    kpp_sums(v, n, now.q);
}

// ---------------------------------------------------------------- seeding on K
//
// The same D^2 sampling in the kernel's feature space, with no features: the
// squared distance of point i to seed s is K_ii + K_ss - 2 K_si (row s of K,
// read along the row), clamped at 0.  O(n) per seed, O(nk) for the labels.

__device__ __forceinline__ float kentry(const float *K, int64_t idx) { return K[idx]; }
__device__ __forceinline__ float kentry(const uint16_t *K, int64_t idx) {
    return __uint_as_float((uint32_t)K[idx] << 16);
}

// dmin_i = min over seeds 0..t of the distance, one thread per row; the sums
// as for the feature rows.
template <typename T>
__global__ __launch_bounds__(256) void kkpp_update(const T *K, int64_t ldk, const float *diag,
                                                   int64_t n, const int32_t *seeds, int t,
                                                   float *dmin, KppSums q) {
    const int64_t i = (int64_t)blockIdx.x * kKppGroup + threadIdx.x;
    const int64_t sd = seeds[t];
    double v = 0.0;
    if (i < n) {
        const float d = fmaxf(diag[i] + diag[sd] - 2.0f * kentry(K, sd * ldk + i), 0.0f);
        const float m = (t == 0) ? d : fminf(dmin[i], d);
        dmin[i] = m;
        v = (double)m;
    }
    kpp_sums(v, n, q);
}

// label_i = index of the nearest seed (lowest on ties)
template <typename T>
__global__ __launch_bounds__(256) void kkpp_assign(const T *K, int64_t ldk, const float *diag,
                                                   int64_t n, int32_t k, const int32_t *seeds,
                                                   int32_t *labels) {
    extern __shared__ int32_t ss[];
    for (int t = threadIdx.x; t < k; t += 256) ss[t] = seeds[t];
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float di = diag[i];
    float best = __builtin_inff();
    int32_t arg = 0;
    for (int32_t t = 0; t < k; ++t) {
        const int64_t sd = ss[t];
        const float d = fmaxf(di + diag[sd] - 2.0f * kentry(K, sd * ldk + i), 0.0f);
        if (d < best) {
            best = d;
            arg = t;
        }
    }
    labels[i] = arg;
}

__global__ void gather_seed_rows(const float *F, int64_t ldf, int64_t f, const int32_t *seeds,
                                 float *C) {
    const int64_t c = blockIdx.x;
    const int64_t src = seeds[c];
    for (int64_t t = threadIdx.x; t < f; t += blockDim.x) C[c * f + t] = F[src * ldf + t];
}

__global__ void row_sqnorms_small(const float *C, int64_t k, int64_t f, float *cn) {
    const int64_t c = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (c >= k) return;
    float s = 0.f;
    for (int64_t t = lane; t < f; t += kWave) s = fmaf(C[c * f + t], C[c * f + t], s);
    s = wave_sum(s);
    if (lane == 0) cn[c] = s;
}

__global__ void iota_i32(int32_t *p, int64_t count) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = (int32_t)i;
}

__global__ void fill_one_i32(int32_t *p, int32_t v) { *p = v; }

}  // namespace

}  // namespace kkm

using namespace kkm;

// Block and group sums of a second set (none for one seed).
static int64_t kpp_second(int64_t n, int32_t k) {
    return k > 1 ? (n + kKppRows - 1) / kKppRows + (n + kKppGroup - 1) / kKppGroup : 0;
}

extern "C" size_t kkm_feature_kmeanspp_workspace_bytes(int64_t n, int64_t f, int32_t k) {
    if (n < 1 || f < 1 || k < 1) return 0;
    Carver c(nullptr);
    c.take<float>((size_t)n);                                  // dmin
    c.take<double>((size_t)((n + kKppRows - 1) / kKppRows));   // block sums
    c.take<double>((size_t)((n + kKppGroup - 1) / kKppGroup)); // group sums
    c.take<float>((size_t)(k * f));                            // seed rows
    c.take<float>((size_t)k);                                  // their norms
    c.take<float>((size_t)n);                                  // row norms
    c.take<double>((size_t)kpp_second(n, k));                  // the second set of sums
    c.take<int32_t>((size_t)k + 1);                            // offsets 0..k
    c.take<int32_t>((size_t)n);                                // placeholder input labels
    c.take<int64_t>(1);                                        // changed count
    return c.bytes();
}

extern "C" kkm_status kkm_feature_kmeanspp(const float *F, int64_t n, int64_t f, int64_t ldf,
                                           int32_t k, const double *uniforms, int32_t *seeds,
                                           int32_t *labels_out, void *ws, size_t ws_bytes,
                                           void *stream) {
    if (n < 1 || f < 1 || ldf < f || k < 1 || k > n || !F || !uniforms || !seeds || !labels_out) {
        set_error("kkm_feature_kmeanspp: bad sizes or NULL pointer");
        return KKM_ERR_ARG;
    }
    for (int32_t t = 0; t < k; ++t)
        if (!(uniforms[t] >= 0.0 && uniforms[t] < 1.0)) {
            set_error("kkm_feature_kmeanspp: uniforms must lie in [0, 1)");
            return KKM_ERR_ARG;
        }
    const size_t need = kkm_feature_kmeanspp_workspace_bytes(n, f, k);
    if (!ws || ws_bytes < need) {
        set_error("kkm_feature_kmeanspp: workspace of %zu bytes is smaller than %zu", ws_bytes, need);
        return KKM_ERR_NOMEM;
    }
    hipStream_t s = (hipStream_t)stream;
    Carver c(ws);
    float *dmin = c.take<float>((size_t)n);
    const int64_t ng = (n + kKppGroup - 1) / kKppGroup;
    KppSums q;
    q.bsum = c.take<double>((size_t)((n + kKppRows - 1) / kKppRows));
    q.gsum = c.take<double>((size_t)ng);
    float *C = c.take<float>((size_t)(k * f));
    float *cn = c.take<float>((size_t)k);
    float *fn = c.take<float>((size_t)n);
    double *sums2 = c.take<double>((size_t)kpp_second(n, k));
    int32_t *offs = c.take<int32_t>((size_t)k + 1);
    int32_t *lab_in = c.take<int32_t>((size_t)n);
    int64_t *changed = c.take<int64_t>(1);
    const int64_t first = (int64_t)(uniforms[0] * (double)n);
    // the row norms' place holds the second set of distances until they are needed
    const KppState st[2] = {{dmin, q}, {fn, KppSums{sums2, sums2 + (n + kKppRows - 1) / kKppRows}}};
    for (int32_t t = 0; t + 1 < k; ++t) {
        const KppState &was = st[(t + 1) & 1], &now = st[t & 1];
        const bool select = t > 0 && ng <= kKppOwnSelect;
        if (t > 0 && !select)
            hipLaunchKernelGGL(kpp_select, dim3(1), dim3(256), 0, s, was.q, was.dmin, n, uniforms[t], seeds + t);
        auto step = [&](auto vec, auto sel) {
            constexpr bool V = decltype(vec)::value, S = decltype(sel)::value;
            hipLaunchKernelGGL((kpp_step<V, S>), dim3((unsigned)ng), dim3(kpp_threads<S>()), 0, s, F, n, f, ldf, seeds, t,
                               first < n ? first : n - 1, uniforms[t], was, now);
        };
        if (vec_ok(F, ldf, f) && select)
            step(std::true_type{}, std::true_type{});
        else if (vec_ok(F, ldf, f))
            step(std::true_type{}, std::false_type{});
        else if (select)
            step(std::false_type{}, std::true_type{});
        else
            step(std::false_type{}, std::false_type{});
        KKM_HIP(hipGetLastError());
    }
    if (k > 1) {
        const KppState &was = st[(k - 2) & 1];
        hipLaunchKernelGGL(kpp_select, dim3(1), dim3(256), 0, s, was.q, was.dmin, n, uniforms[k - 1], seeds + k - 1);
    } else {
        hipLaunchKernelGGL(fill_one_i32, dim3(1), dim3(1), 0, s, seeds, (int32_t)(first < n ? first : n - 1));
    }
    KKM_HIP(hipGetLastError());
    // labels: nearest seed (lowest index on ties), via the Lloyd assignment
    hipLaunchKernelGGL(gather_seed_rows, dim3((unsigned)k), dim3(256), 0, s, F, ldf, f, seeds, C);
    hipLaunchKernelGGL(row_sqnorms_small, dim3((unsigned)((k + 3) / 4)), dim3(256), 0, s, C,
                       (int64_t)k, f, cn);
    hipLaunchKernelGGL(feature_sqnorms, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, F, n, f,
                       ldf, fn);
    hipLaunchKernelGGL(iota_i32, dim3((unsigned)((k + 1 + 255) / 256)), dim3(256), 0, s, offs,
                       (int64_t)k + 1);
    hipLaunchKernelGGL(iota_i32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, lab_in, n);
    KKM_HIP(hipGetLastError());
    KKM_TRY(nearest_launch(F, ldf, f, C, fn, cn, offs, n, k, lab_in, labels_out, changed, nullptr, s));
    return KKM_OK;
}

extern "C" size_t kkm_kernel_kmeanspp_workspace_bytes(int64_t n, int32_t k) {
    if (n < 1 || k < 1) return 0;
    Carver c(nullptr);
    c.take<float>((size_t)n);                                   // dmin
    c.take<double>((size_t)((n + kKppRows - 1) / kKppRows));    // block sums
    c.take<double>((size_t)((n + kKppGroup - 1) / kKppGroup));  // group sums
    return c.bytes();
}

extern "C" kkm_status kkm_kernel_kmeanspp(const void *K, int32_t k_store, int64_t ldk,
                                          const float *diagK, int64_t n, int32_t k,
                                          const double *uniforms, int32_t *seeds,
                                          int32_t *labels_out, void *ws, size_t ws_bytes,
                                          void *stream) {
    if (n < 1 || k < 1 || k > n || ldk < n || !K || !diagK || !uniforms || !seeds ||
        !labels_out) {
        set_error("kkm_kernel_kmeanspp: bad sizes or NULL pointer");
        return KKM_ERR_ARG;
    }
    if (k_store != KKM_F32 && k_store != KKM_BF16) {
        set_error("kkm_kernel_kmeanspp: K must be stored as KKM_F32 or KKM_BF16");
        return KKM_ERR_ARG;
    }
    if (k > KKM_MAX_K) {
        set_error("kkm_kernel_kmeanspp: k=%d exceeds KKM_MAX_K=%d", k, KKM_MAX_K);
        return KKM_ERR_UNSUPPORTED;
    }
    for (int32_t t = 0; t < k; ++t)
        if (!(uniforms[t] >= 0.0 && uniforms[t] < 1.0)) {
            set_error("kkm_kernel_kmeanspp: uniforms must lie in [0, 1)");
            return KKM_ERR_ARG;
        }
    const size_t need = kkm_kernel_kmeanspp_workspace_bytes(n, k);
    if (!ws || ws_bytes < need) {
        set_error("kkm_kernel_kmeanspp: workspace of %zu bytes is smaller than %zu", ws_bytes,
                  need);
        return KKM_ERR_NOMEM;
    }
    hipStream_t s = (hipStream_t)stream;
    Carver c(ws);
    float *dmin = c.take<float>((size_t)n);
    KppSums q;
    q.bsum = c.take<double>((size_t)((n + kKppRows - 1) / kKppRows));
    q.gsum = c.take<double>((size_t)((n + kKppGroup - 1) / kKppGroup));
    const int64_t first = (int64_t)(uniforms[0] * (double)n);
    hipLaunchKernelGGL(fill_one_i32, dim3(1), dim3(1), 0, s, seeds,
                       (int32_t)(first < n ? first : n - 1));
    const dim3 g((unsigned)((n + kKppGroup - 1) / kKppGroup)), b(256);
    for (int32_t t = 0; t + 1 < k; ++t) {
        if (k_store == KKM_F32)
            hipLaunchKernelGGL(kkpp_update<float>, g, b, 0, s, static_cast<const float *>(K), ldk,
                               diagK, n, seeds, t, dmin, q);
        else
            hipLaunchKernelGGL(kkpp_update<uint16_t>, g, b, 0, s,
                               static_cast<const uint16_t *>(K), ldk, diagK, n, seeds, t, dmin, q);
        hipLaunchKernelGGL(kpp_select, dim3(1), dim3(256), 0, s, q, dmin, n, uniforms[t + 1],
                           seeds + t + 1);
        KKM_HIP(hipGetLastError());
    }
    const size_t lds = sizeof(int32_t) * (size_t)k;
    if (k_store == KKM_F32)
        hipLaunchKernelGGL(kkpp_assign<float>, g, b, lds, s, static_cast<const float *>(K), ldk,
                           diagK, n, k, seeds, labels_out);
    else
        hipLaunchKernelGGL(kkpp_assign<uint16_t>, g, b, lds, s, static_cast<const uint16_t *>(K),
                           ldk, diagK, n, k, seeds, labels_out);
    KKM_HIP(hipGetLastError());
    return KKM_OK;
}

extern "C" size_t kkm_feature_lloyd_workspace_bytes(int64_t n, int64_t f, int32_t k) {
    if (n < 1 || f < 1 || k < 1) return 0;
    size_t bytes = 0;
    carve_lloyd(nullptr, n, f, k, &bytes);
    return bytes;
}

extern "C" kkm_status kkm_feature_lloyd(const float *F, int64_t n, int64_t f, int64_t ldf,
                                        int32_t k, const int32_t *labels0, int32_t max_iter,
                                        int32_t *labels_out, int32_t *iters,
                                        int64_t *changed_trace, double *objective, void *ws,
                                        size_t ws_bytes,
                                        void *stream) {
    if (n < 1 || f < 1 || ldf < f || k < 1 || k > n || max_iter < 0 || !F || !labels0 ||
        !labels_out || !iters) {
        set_error("kkm_feature_lloyd: bad sizes or NULL pointer");
        return KKM_ERR_ARG;
    }
    if (k > KKM_MAX_K) {
        set_error("kkm_feature_lloyd: k=%d exceeds KKM_MAX_K=%d", k, KKM_MAX_K);
        return KKM_ERR_UNSUPPORTED;
    }
    size_t need = 0;
    LloydWs w = carve_lloyd(ws, n, f, k, &need);
    if (!ws || ws_bytes < need) {
        set_error("kkm_feature_lloyd: workspace of %zu bytes is smaller than %zu", ws_bytes, need);
        return KKM_ERR_NOMEM;
    }
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(feature_sqnorms, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, F, n, f,
                       ldf, w.fn);
    KKM_HIP(hipGetLastError());
    KKM_HIP(hipMemcpyAsync(w.lab[0], labels0, (size_t)n * 4, hipMemcpyDeviceToDevice, s));
    const int64_t nchunk = (n + kRows - 1) / kRows;
    int cur = 0;
    int32_t t = 0;
    int64_t hc = -1;
    int32_t herr = 0;
    for (; t < max_iter; ++t) {
        KKM_TRY(vcsr_build(w.lab[cur], n, k, w.blk_hist, w.blk_bad, w.err, w.counts, w.perm,
                           w.offsets, w.counts_out, w.changed, s));
        if (t == 0) {
            KKM_HIP(hipMemcpyAsync(&herr, w.err, sizeof herr, hipMemcpyDeviceToHost, s));
            KKM_HIP(hipStreamSynchronize(s));
            if (herr) {
                set_error("kkm_feature_lloyd: a label of labels0 lies outside [0, %d)", k);
                return KKM_ERR_LABEL;
            }
        }
        const dim3 cg((unsigned)((nchunk + 3) / 4), (unsigned)((f + 255) / 256));
        if (vec_ok(F, ldf, f))
            hipLaunchKernelGGL(centroid_partials<true>, cg, dim3(256), 0, s, F, n, f, ldf, k, nchunk, w.perm,
                               w.offsets, w.Cp);
        else
            hipLaunchKernelGGL(centroid_partials<false>, cg, dim3(256), 0, s, F, n, f, ldf, k, nchunk, w.perm,
                               w.offsets, w.Cp);
        hipLaunchKernelGGL(centroid_finalize, dim3((unsigned)k), dim3(256), 0, s, w.Cp, f, k,
                           w.offsets, w.C, w.cn);
        KKM_HIP(hipGetLastError());
        KKM_TRY(nearest_launch(F, ldf, f, w.C, w.fn, w.cn, w.offsets, n, k, w.lab[cur], w.lab[cur ^ 1], w.changed,
                               w.part, s));
        KKM_HIP(hipMemcpyAsync(&hc, w.changed, sizeof hc, hipMemcpyDeviceToHost, s));
        KKM_HIP(hipStreamSynchronize(s));
        if (changed_trace) changed_trace[t] = hc;
        cur ^= 1;
        if (hc == 0) {
            ++t;
            break;
        }
    }
    KKM_HIP(hipMemcpyAsync(labels_out, w.lab[cur], (size_t)n * 4, hipMemcpyDeviceToDevice, s));
    double obj = 0.0;
    if (objective && t > 0) {
        // sum_i min_c d_ic of the last step (the objective of labels_out when it changed nothing)
        hipLaunchKernelGGL(sum_blocks, dim3(1), dim3(256), 0, s, w.part, (n + 63) / 64, w.obj);
        KKM_HIP(hipGetLastError());
        KKM_HIP(hipMemcpyAsync(&obj, w.obj, sizeof obj, hipMemcpyDeviceToHost, s));
    }
    KKM_HIP(hipStreamSynchronize(s));
    *iters = t;
    if (objective) *objective = (t > 0) ? obj : __builtin_nan("");
    return KKM_OK;
}
