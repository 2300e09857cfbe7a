// The split product of the kernel matrix (gram_split.h): its prologue and its
// launches, in a translation unit of its own so that the library's sources
// compile in parallel.
#include "gram_split.h"

namespace kkm {
namespace gt {

namespace {

// One thread per (row, 8 features): a wave writes the three planes of one
// group's slab whole.  Rows past n are zeros.
__global__ __launch_bounds__(256) void split_rows(const float *X, int64_t n, int64_t d, int64_t ldx,
                                                  int64_t groups, int64_t nslab, unsigned char *Xs) {
    const int lane = threadIdx.x & 63;
    const int64_t g = blockIdx.x;
    const int r = lane >> 2, c = (lane & 3) ^ ((r >> 2) & 3);
    const int64_t row = g * SPG + r;
    for (int64_t slab = (int64_t)blockIdx.y * 4 + (threadIdx.x >> 6); slab < nslab; slab += 4 * (int64_t)gridDim.y) {
        float v[8];
        split_load(X + min(row, n - 1) * ldx, d, slab * SPK + 8 * c, v);
        split_store(v, d, slab * SPK + 8 * c, row < n, Xs + (slab * groups + g) * SPB + lane * 16);
    }
}

// Squared norms (Gaussian; as the FP32 product's prologue) and the rows' marks,
// one wave per row.
__global__ __launch_bounds__(256) void split_stats(const float *X, int64_t n, int64_t d, int64_t ldx,
                                                   bool norm, float *nrm) {
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= n) return;
    split_row_stats(X + row * ldx, d, norm, nrm + row, lane);
}

template <typename OUT, bool FULL, bool PRE>
__global__ __launch_bounds__(GTHREADS, 2) void gram_split_mfma(SplitTile x, F32Tile a, TileOrder o) {
    __shared__ __attribute__((aligned(1024))) SplitOrF32Lds lds;
    int64_t bi, bj;
    if (!tile_of_block(o, bi, bj)) return;
    if (outside_split(a.e, bi * GM, bj * GM))
        f32_tile<OUT, FULL>(a, bi, bj, lds.f);
    else
        split_tile<OUT, FULL, PRE>(x, a, bi, bj, lds.s);
}

template <bool FULL, bool PRE>
void launch_product(int32_t k_store, const SplitTile &x, const F32Tile &a, const TileOrder &order, hipStream_t stream) {
    const dim3 g((unsigned)(order.per_xcd * 8)), b(GTHREADS);
    if (k_store == KKM_F32)
        hipLaunchKernelGGL((gram_split_mfma<float, FULL, PRE>), g, b, 0, stream, x, a, order);
    else
        hipLaunchKernelGGL((gram_split_mfma<uint16_t, FULL, PRE>), g, b, 0, stream, x, a, order);
}

}  // namespace

size_t split_bytes(int64_t n, int64_t d) {
    return (size_t)split_groups(n) * (size_t)split_slabs(d) * SPB;
}

kkm_status launch_gram_split(int32_t k_store, bool full, const F32Tile &a, const TileOrder &order,
                             unsigned char *Xs, float *nrm, hipStream_t stream) {
    const int64_t groups = split_groups(a.e.n), nslab = split_slabs(a.d);
    if (Xs) {
        const unsigned gy = (unsigned)((nslab + 3) / 4 < 65535 ? (nslab + 3) / 4 : 65535);
        hipLaunchKernelGGL(split_rows, dim3((unsigned)groups, gy), dim3(256), 0, stream, a.X, a.e.n, a.d, a.ldx, groups,
                           nslab, Xs);
        KKM_HIP(hipGetLastError());
    }
    hipLaunchKernelGGL(split_stats, dim3((unsigned)((a.e.n + 3) / 4)), dim3(256), 0, stream, a.X, a.e.n, a.d,
                       a.ldx, a.e.kernel == KKM_GAUSS, nrm);
    KKM_HIP(hipGetLastError());
    const SplitTile x = split_source(Xs, a.e.n, a.d);
    const TimedSpan span = timing_begin(TK_GRAM, stream);
    if (full && Xs)
        launch_product<true, true>(k_store, x, a, order, stream);
    else if (full)
        launch_product<true, false>(k_store, x, a, order, stream);
    else if (Xs)
        launch_product<false, true>(k_store, x, a, order, stream);
    else
        launch_product<false, false>(k_store, x, a, order, stream);
    KKM_HIP(hipGetLastError());
    timing_end(span, stream);
    return KKM_OK;
}

}  // namespace gt
}  // namespace kkm
