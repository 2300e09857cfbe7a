// MFMA products for the learned feature map.  FP32 (the loss of a large batch
// and its gradient): 64 x 64 output tile per 256-thread workgroup, 4
// waves as 2 x 2, each one 32 x 32 MFMA block; k staged in LDS in slabs of 32.
// BF16 (operands rounded to nearest even): the 32 x 32 tiles of gemm_small.h,
// or the wider tiles below for a layer forward of many rows.
#include "gemm_small.h"

namespace kkm {

namespace {

constexpr int TM = 64, TK = 32, TLD = TK + 1;

// Stage a 64 x 32 operand slab (rows r0.., k k0..) into LDS as [row][k].
template <bool KCONTIG>
__device__ __forceinline__ void stage(const float *P, int64_t ld, int64_t rows, int64_t K,
                                      int64_t r0, int64_t k0, float (*S)[TLD]) {
    const int t = threadIdx.x;
    if (KCONTIG) {
        const int r = t >> 2, c = (t & 3) * 8;  // 8 consecutive k of one row
        const int64_t gr = r0 + r;
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            const int64_t gk = k0 + c + v;
            S[r][c + v] = (gr < rows && gk < K) ? P[gr * ld + gk] : 0.f;
        }
    } else {
        const int kk = t >> 3, c = (t & 7) * 8;  // 8 consecutive rows of one k
        const int64_t gk = k0 + kk;
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            const int64_t gr = r0 + c + v;
            S[c + v][kk] = (gr < rows && gk < K) ? P[gk * ld + gr] : 0.f;
        }
    }
}

template <bool AK, bool BK>
__global__ __launch_bounds__(256) void gemm_f32(GemmArgs g, int epi) {
    __shared__ float As[TM][TLD], Bs[TM][TLD];
    __shared__ double red[4];
    const int64_t m0 = (int64_t)blockIdx.y * TM, n0 = (int64_t)blockIdx.x * TM;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int half = lane >> 5, l32 = lane & 31;

    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;

    for (int64_t k0 = 0; k0 < g.K; k0 += TK) {
        stage<AK>(g.A, g.lda, g.M, g.K, m0, k0, As);
        stage<BK>(g.B, g.ldb, g.N, g.K, n0, k0, Bs);
        __syncthreads();
        const float *ra = As[wm * 32 + l32];
        const float *rb = Bs[wn * 32 + l32];
#pragma unroll
        for (int s = 0; s < TK / 2; ++s)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(ra[2 * s + half], rb[2 * s + half], acc, 0, 0, 0);
        __syncthreads();
    }

    // accumulator register r of lane l: row 8*(r/4) + 4*(l/32) + r%4, column l%32
    double sq = 0.0;
    const int64_t n = n0 + wn * 32 + l32;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int64_t m = m0 + wm * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
        if (m >= g.M || n >= g.N) continue;
        const float v = g.alpha * acc[r];
        if (epi == EPI_STORE) {
            g.C[m * g.ldc + n] = v;
        } else {  // EPI_LOSS
            const float e = v - g.Kb[m * g.ldkb + n];
            g.C[m * g.ldc + n] = e;
            sq += (double)e * (double)e;
        }
    }
    if (epi == EPI_LOSS) {
        sq = wave_sum(sq);
        if (lane == 0) red[wave] = sq;
        __syncthreads();
        if (tid == 0)
            g.part[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
    }
}

// ---------------------------------------------------------------- wide tiles
//
// Both operands k-contiguous (A(m,k) = A[m*lda+k], B(n,k) = B[n*ldb+k]) and
// many rows: a 64 x 256 output tile per workgroup, wave w owning columns
// 64w .. 64w+63 as 2 x 2 blocks of 32 x 32, or for a narrow layer a 64 x 64 tile,
// a wave owning one block.  k-slabs of 64 floats per row are
// loaded a slab ahead into registers without branches (behind one each load
// would be waited for before the next), rounded to bfloat16 and staged in LDS,
// so a fragment is one 16-byte read.  MFMA s (s = 0, 1) of each 32 k takes
// k = 16h + 8s .. 16h + 8s + 7 from lane half h; of a narrow layer, k = 16s + 8h ..
// 16s + 8h + 7, the order of the small tiles.  (32768 x 512 x 512: 98 us
// with FP32 slabs of 32, rounded per fragment, and branches; 72 us so.)

constexpr int WM = 64, WK = 64, WLD = WK + 8;

template <int WN> struct WideLds {
    __bf16 a[WM][WLD];
    __bf16 b[WN][WLD];
};

template <int WN>
__global__ __launch_bounds__(256, 2) void gemm_wide(GemmArgs g, bool act, int vec) {
    static_assert(WN == 256 || WN == 64, "four waves of 2 x 2 blocks or of one");
    constexpr bool WIDE = WN == 256;
    constexpr int NB = WIDE ? 2 : 1;  // blocks a wave owns each way
    __shared__ __attribute__((aligned(16))) WideLds<WN> lds;
    const int64_t m0 = (int64_t)blockIdx.y * WM, n0 = (int64_t)blockIdx.x * WN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int half = lane >> 5, l32 = lane & 31;
    const int lr = tid >> 4, lc = (tid & 15) * 4;  // 16 threads x 4 floats per row of a slab
    constexpr int RA = WM / 16, RB = WN / 16;
    const int wm = WIDE ? 0 : 32 * (wave >> 1), wn = WIDE ? 64 * wave : 32 * (wave & 1);  // the wave's rows and columns
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

    f32x4 ra[RA], rb[RB];
    auto gload = [&](int64_t k0) {
        auto load = [&](auto v) {
            constexpr bool V = decltype(v)::value;
#pragma unroll
            for (int u = 0; u < RA; ++u)
                ra[u] = line4<V>(g.A, (m0 + lr + 16 * u) * g.lda, k0 + lc, g.K, m0 + lr + 16 * u < g.M);
#pragma unroll
            for (int u = 0; u < RB; ++u)
                rb[u] = line4<V>(g.B, (n0 + lr + 16 * u) * g.ldb, k0 + lc, g.K, n0 + lr + 16 * u < g.N);
        };
        if (vec)  // uniform
            load(std::true_type{});
        else
            load(std::false_type{});
    };
    auto sstore = [&](int64_t k0) {
#pragma unroll
        for (int u = 0; u < RA; ++u)
            *reinterpret_cast<bf16x4 *>(&lds.a[lr + 16 * u][lc]) =
                __builtin_convertvector(mask4(ra[u], k0 + lc, g.K, m0 + lr + 16 * u < g.M), bf16x4);
#pragma unroll
        for (int u = 0; u < RB; ++u)
            *reinterpret_cast<bf16x4 *>(&lds.b[lr + 16 * u][lc]) =
                __builtin_convertvector(mask4(rb[u], k0 + lc, g.K, n0 + lr + 16 * u < g.N), bf16x4);
    };

    f32x16 acc[NB][NB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    gload(0);
    for (int64_t k0 = 0; k0 < g.K; k0 += WK) {
        sstore(k0);
        __syncthreads();
        if (k0 + WK < g.K) gload(k0 + WK);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (k0 + 16 * (s & 2) >= g.K) break;  // uniform: 32 zeros
            const int at = WIDE ? 16 * (s & 2) + 16 * half + 8 * (s & 1) : 16 * s + 8 * half;
            bf16x8 x[NB], y[NB];
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                x[i] = *reinterpret_cast<const bf16x8 *>(&lds.a[wm + i * 32 + l32][at]);
                y[i] = *reinterpret_cast<const bf16x8 *>(&lds.b[wn + i * 32 + l32][at]);
            }
#pragma unroll
            for (int mi = 0; mi < NB; ++mi)
#pragma unroll
                for (int ni = 0; ni < NB; ++ni)
                    acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[mi], y[ni], acc[mi][ni], 0, 0, 0);
        }
        __syncthreads();
    }

    // accumulator register r of lane l: row 8*(r/4) + 4*(l/32) + r%4, column l%32
#pragma unroll
    for (int ni = 0; ni < NB; ++ni) {
        const int64_t n = n0 + wn + ni * 32 + l32;
        const float bias = g.bias[min(n, g.N - 1)];
#pragma unroll
        for (int mi = 0; mi < NB; ++mi)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t m = m0 + wm + mi * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                if (m >= g.M || n >= g.N) continue;
                const float z = acc[mi][ni][r] + bias;
                if (g.C) g.C[m * g.ldc + n] = z;
                if (act) g.C2[m * g.ldc2 + n] = gelu(z);
            }
    }
}

// Products that take the wide tiles: a layer forward (both operands
// k-contiguous, a bias, GELU or not) of many rows.
bool gemm_wide_fits(GemmOp op, bool ak, bool bk, GemmEpi epi, const GemmArgs &g) {
    return op == GEMM_BF16 && ak && bk && (epi == EPI_BIAS || epi == EPI_BIAS_GELU) && g.alpha == 1.0f &&
           g.M >= 32 && g.N >= 256 && g.M * g.N >= (1 << 20);
}
// The same for a layer of fewer than 256 columns.  With few rows its 64 x 64 tiles
// leave most of the chip idle while they walk k, and the 32 x 32 tiles that stage
// it at once are faster; with many those wait on their 66 KiB of LDS, two
// workgroups a CU, and load for 512 k whatever k is.  A forward of three layers,
// 32 x 32 tiles / these: d = 64, widths 64, 64, 32: 8192 rows 21.9 / 17.7 us, 32768
// 61 / 20; 128, 128, 64: 4096 rows 22.5 / 22.0, 32768 115 / 35; d = 1024, 64, 64, 16:
// 4096 rows 24 / 30, 8192 36 / 32; 250, 250, 50: 2000 rows 37 / 44, 4096 58 / 46; d =
// 50, 50, 50, 50: 8192 rows 31 / 22; d = 784, 250, 250, 10, the last layer alone:
// 8192 rows 54 / 58, 32768 162 / 156.
bool gemm_narrow_fits(GemmOp op, bool ak, bool bk, GemmEpi epi, const GemmArgs &g) {
    return op == GEMM_BF16 && ak && bk && (epi == EPI_BIAS || epi == EPI_BIAS_GELU) && g.alpha == 1.0f &&
           g.N < 256 && g.M <= 65535 * WM && (g.M >= 16384 || (g.M >= 4096 && g.M * g.N >= (3 << 17)));
}

template <int WN>
kkm_status gemm_wide_launch(GemmEpi epi, const GemmArgs &g, hipStream_t stream) {
    const dim3 grid((unsigned)((g.N + WN - 1) / WN), (unsigned)((g.M + WM - 1) / WM));
    hipLaunchKernelGGL(gemm_wide<WN>, grid, dim3(256), 0, stream, g, epi == EPI_BIAS_GELU,
                       vec_ok(g.A, g.lda, g.K) && vec_ok(g.B, g.ldb, g.K));
    KKM_HIP(hipGetLastError());
    return KKM_OK;
}

template <bool AK, bool BK, int KS, int EPI>
__global__ __launch_bounds__(SNT) void gemm_small(SmallGemm g) {
    __shared__ __attribute__((aligned(16))) SmallLds lds;
    small_tile<AK, BK, KS, EPI>(g, blockIdx.x, AdamArgs{}, lds);
}

template <bool AK, bool BK, int KS, int EPI>
kkm_status gemm_small_launch(const SmallGemm &g, hipStream_t stream) {
    hipLaunchKernelGGL((gemm_small<AK, BK, KS, EPI>), dim3((unsigned)small_tiles(g)), dim3(SNT), 0, stream, g);
    KKM_HIP(hipGetLastError());
    return KKM_OK;
}

// The BF16 forms the network uses (all with alpha = 1).  A training step of a
// large batch takes them for its products below the wide tiles' sizes; with 64 x
// 64 tiles that staged FP32 slabs of 32 k it was, d = 128, widths 512, 512, 256: B =
// 257 453 us, here 247; B = 512 647 / 367; B = 1024 1019 / 639; B = 4096 4642 / 3693.
kkm_status gemm_bf16_small(bool ak, bool bk, GemmEpi epi, const GemmArgs &g, hipStream_t stream) {
    SmallGemm s = small_gemm(ak, bk, g.A, g.lda, g.B, g.ldb, g.M, g.N, g.K, g.C, g.ldc);
    s.C2 = g.C2;
    if (g.alpha == 1.0f && ak && bk && epi == EPI_BIAS_GELU && (!g.C || g.ldc == g.ldc2)) {
        s.x = g.bias;
        s.ldc = g.ldc2;
        return gemm_small_launch<true, true, SK, SE_BIAS_GELU>(s, stream);
    }
    if (g.alpha == 1.0f && ak && bk && epi == EPI_BIAS) {
        s.x = g.bias;
        return gemm_small_launch<true, true, SK, SE_BIAS>(s, stream);
    }
    if (g.alpha == 1.0f && ak && !bk && epi == EPI_GELU_BWD && g.ldz == g.ldc) {
        s.x = g.Zp;
        return gemm_small_launch<true, false, SK, SE_GELU_BWD>(s, stream);
    }
    if (g.alpha == 1.0f && !ak && !bk && epi == EPI_STORE)
        return gemm_small_launch<false, false, 256, SE_GRAD>(s, stream);
    set_error("internal: BF16 product in a form no kernel takes");
    return KKM_ERR_UNSUPPORTED;
}

}  // namespace

kkm_status gemm_launch(GemmOp op, bool ak, bool bk, GemmEpi epi, const GemmArgs &g,
                       hipStream_t stream) {
    if (g.M <= 0 || g.N <= 0) return KKM_OK;
    if (gemm_wide_fits(op, ak, bk, epi, g)) return gemm_wide_launch<256>(epi, g, stream);
    if (gemm_narrow_fits(op, ak, bk, epi, g)) return gemm_wide_launch<64>(epi, g, stream);
    if (op == GEMM_BF16) return gemm_bf16_small(ak, bk, epi, g, stream);
    const dim3 grid((unsigned)((g.N + TM - 1) / TM), (unsigned)((g.M + TM - 1) / TM));
    const dim3 blk(256);
    if (ak && bk && epi == EPI_LOSS)
        hipLaunchKernelGGL((gemm_f32<true, true>), grid, blk, 0, stream, g, (int)epi);
    else if (ak && !bk && epi == EPI_STORE)
        hipLaunchKernelGGL((gemm_f32<true, false>), grid, blk, 0, stream, g, (int)epi);
    else {
        set_error("internal: FP32 product in a form no kernel takes");
        return KKM_ERR_UNSUPPORTED;
    }
    KKM_HIP(hipGetLastError());
    return KKM_OK;
}

}  // namespace kkm
