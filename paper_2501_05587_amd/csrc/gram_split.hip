// The split product of the kernel matrix (gram_split.h): its prologue and its
// launches, in a translation unit of its own so that the library's sources
// compile in parallel.
#include "gram_split.h"

namespace kkm {
namespace gt {

namespace {

// One thread per (row, 8 features): a wave writes the three planes of one
// group's slab whole.  Rows past n are zeros.  Workgroup 0 clears the flag.
__global__ __launch_bounds__(256) void split_rows(const float *X, int64_t n, int64_t d, int64_t ldx,
                                                  int64_t groups, int64_t nslab, unsigned char *Xs,
                                                  int32_t *flag) {
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *flag = 0;
    const int lane = threadIdx.x & 63;
    const int64_t g = blockIdx.x;
    const int64_t slab = (int64_t)blockIdx.y * 4 + (threadIdx.x >> 6);
    if (slab >= nslab) return;
    const int r = lane >> 2, c = (lane & 3) ^ ((r >> 2) & 3);
    const int64_t row = g * SPG + r;
    split_chunk(X + min(row, n - 1) * ldx, d, slab * SPK + 8 * c, row < n, Xs + (slab * groups + g) * SPB + lane * 16);
}

// Squared norms (Gaussian; as the FP32 product's prologue) and the flag, one
// wave per row.
__global__ __launch_bounds__(256) void split_stats(const float *X, int64_t n, int64_t d, int64_t ldx,
                                                   float *nrm, int32_t *flag) {
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= n) return;
    const float *x = X + row * ldx;
    if (nrm) sqnorm_row(x, d, nrm + row, lane);
    if (split_row_bad(x, d, lane) && lane == 0) atomicOr(flag, 1);
}

template <typename OUT, bool FULL>
__global__ __launch_bounds__(GTHREADS, 2) void gram_split_mfma(SplitTile x, Epi e, TileOrder o) {
    __shared__ __attribute__((aligned(1024))) SplitLds lds;
    int64_t bi, bj;
    if (!tile_of_block(o, bi, bj)) return;
    if (*x.flag != 0) return;
    split_tile<OUT, FULL>(x, e, bi, bj, lds);
}

template <bool FULL>
void launch_product(int32_t k_store, const SplitTile &x, const Epi &e, const TileOrder &order, hipStream_t stream) {
    const dim3 g((unsigned)(order.per_xcd * 8)), b(GTHREADS);
    if (k_store == KKM_F32)
        hipLaunchKernelGGL((gram_split_mfma<float, FULL>), g, b, 0, stream, x, e, order);
    else
        hipLaunchKernelGGL((gram_split_mfma<uint16_t, FULL>), g, b, 0, stream, x, e, order);
}

}  // namespace

size_t split_bytes(int64_t n, int64_t d) {
    return (size_t)split_groups(n) * (size_t)split_slabs(d) * SPB;
}

// Below about 3500 points a tile per CU or two is all there is, and the
// prologue and the flagged launch cost what the product saves unless rows are
// long; rows of less than half a slab are mostly padding, and sums of one or two
// products gain nothing in exactness.  FP32 kernel / split, us, Gaussian: n =
// 2304, d = 65 37 / 33, d = 128 35 / 34, d = 784 129 / 90; n = 3584, d = 16 28 / 29,
// d = 64 34 / 35, d = 128 50 / 45; n = 60000, d = 16 2701 / 2773 (bfloat16 K 2534 /
// 1831), d = 128 5286 / 4551, d = 784 25530 / 18607.
bool split_pays(int64_t n, int64_t d) { return d >= 16 && split_room(n, d); }

// The workspace has room for it for shorter rows too: its size is what it was
// when they took the split.
bool split_room(int64_t n, int64_t d) { return n >= 3584 || (n >= 2304 && d > 64); }

kkm_status launch_gram_split(int32_t k_store, bool full, const F32Tile &a, const TileOrder &order,
                             unsigned char *Xs, float *nrm, int32_t *flag, hipStream_t stream) {
    const int64_t groups = split_groups(a.e.n), nslab = split_slabs(a.d);
    hipLaunchKernelGGL(split_rows, dim3((unsigned)groups, (unsigned)((nslab + 3) / 4)), dim3(256), 0, stream, a.X,
                       a.e.n, a.d, a.ldx, groups, nslab, Xs, flag);
    KKM_HIP(hipGetLastError());
    hipLaunchKernelGGL(split_stats, dim3((unsigned)((a.e.n + 3) / 4)), dim3(256), 0, stream, a.X, a.e.n, a.d,
                       a.ldx, a.e.kernel == KKM_GAUSS ? nrm : nullptr, flag);
    KKM_HIP(hipGetLastError());
    const SplitTile x{Xs, groups * SPB, nslab, flag};
    const TimedSpan span = timing_begin(TK_GRAM, stream);
    if (full)
        launch_product<true>(k_store, x, a.e, order, stream);
    else
        launch_product<false>(k_store, x, a.e, order, stream);
    KKM_HIP(hipGetLastError());
    launch_gram_f32_flagged(k_store, full, a, order, flag, stream);
    KKM_HIP(hipGetLastError());
    timing_end(span, stream);
    return KKM_OK;
}

}  // namespace gt
}  // namespace kkm
