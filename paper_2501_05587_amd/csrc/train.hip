// One training step of the feature network on a small batch (up to 256 rows)
// in seven launches:
//   1. Z1 = XB W1^T + b1, H1 = GELU(Z1)      and the batch's kernel values KB
//   2. Z2 = H1 W2^T + b2, H2 = GELU(Z2)
//   3. Phi = H2 W3^T + b3
//   4. G = Phi Phi^T - KB (in LDS), its squares, dPhi = (4/B^2) G Phi
//   5. dZ2 = (dPhi W3) * GELU'(Z2)
//   6. dZ1 = (dZ2 W2) * GELU'(Z1)            and W3, b3 with their Adam update
//   7. W2, b2, W1, b1 with their Adam update and the loss
// A layer's weights are updated one launch after their last use, straight from
// the accumulators of their gradient.
//
// A step of 64 rows multiplies 0.2 GFLOP over 13 MB of weights and moments, so
// it is bound by launches and by the latency of each one's chain of loads.  As
// 18 launches of 64 x 64 tiles (8 workgroups for a layer, a 32-wide slab of k
// staged and waited for at a time) it took 301 us; here 45 us.  Each
// product takes 32 x 32 tiles and stages up to 512 k at once, so a tile waits
// for memory once and the MFMA chain of a tile is k / 32 instructions.
//
// Every sum keeps its order: the 16x16x32 BF16 MFMA adds its k in the order in
// which two 32x32x16 do, and the FP32 MFMAs (32x32x2, 16x16x4) round as a chain
// of fused multiply-adds in k order (checked bit for bit on gfx950).
#include "gemm_small.h"
#include "gram_tile.h"

namespace kkm {

namespace {

constexpr int FK = 256;  // features staged at a time for the kernel values
constexpr int FLDK = FK + 4;

union TrainLds {
    SmallLds h;
    struct {
        float a[ST][FLDK], b[ST][FLDK], nrm[2 * ST];
    } f;
};

// The bias gradient of a layer (column sums of dZ [rows, cols], in row order),
// one column per thread, 32 rows' loads in flight; then Adam or a store.
struct SmallBias {
    const float *dZ;
    int64_t rows, cols;
    float *p, *am, *av;  // Adam: the biases and their moments; else p receives the gradient
};
template <bool ADAM>
__device__ __forceinline__ void small_bias(const SmallBias &b, int64_t blk, const AdamArgs &ad) {
    const int64_t c = blk * SNT + threadIdx.x;
    if (c >= b.cols) return;
    float s = 0.f;
    for (int64_t r0 = 0; r0 < b.rows; r0 += 32) {
        float v[32];
#pragma unroll
        for (int u = 0; u < 32; ++u) v[u] = b.dZ[min(r0 + u, b.rows - 1) * b.cols + c];
#pragma unroll
        for (int u = 0; u < 32; ++u)
            if (r0 + u < b.rows) s += v[u];
    }
    if constexpr (ADAM) {
        float p = b.p[c], mo = b.am[c], ve = b.av[c];
        adam_one(p, mo, ve, s, ad);
        b.p[c] = p;
        b.am[c] = mo;
        b.av[c] = ve;
    } else {
        b.p[c] = s;
    }
}

// A 32 x 32 tile of the batch's kernel values, as the FP32 Gram kernel
// computes them: within each slab of 32 features its MFMAs take them in the
// order 0, 16, 1, 17, ...
__device__ __forceinline__ void batch_kernel_tile(const TrainStep &t, int64_t tile, TrainLds &lds) {
    const int64_t tn = (t.B + ST - 1) / ST;
    const int64_t m0 = (tile / tn) * ST, n0 = (tile % tn) * ST;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4, i = lane & 15;
    const int wm = 16 * ((wave >> 1) & 1), wn = 16 * (wave & 1);
    const SmallOperand x{t.XB, t.ldx, t.B, t.d, vec_ok(t.XB, t.ldx, t.d)};
    constexpr int U = FK / 64;
    f32x4 ra[U], rb[U];
    auto load = [&](int64_t k0) {
        small_load<true, FK>(x, m0, k0, ra);
        small_load<true, FK>(x, n0, k0, rb);
    };
    load(0);
    // the squared norms of the 64 rows, eight per wave, a wave per row at a
    // time, from the staged rows (zeros past d add nothing)
    float s8[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) s8[u] = 0.f;
    const int first = wave * 8;
    const float *nrow = first < ST ? lds.f.a[first] : lds.f.b[first - ST];
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    const int kq = (q >> 1) + 16 * (q & 1);
    for (int64_t k0 = 0; k0 < t.d; k0 += FK) {
        const int klim = (int)((min((int64_t)FK, t.d - k0) + 31) & ~int64_t(31));
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = tid + SNT * u, r = e / (FK / 4), k = 4 * (e % (FK / 4));
            if (k < klim) {
                *reinterpret_cast<f32x4 *>(&lds.f.a[r][k]) = small_mask<true, FK>(x, m0, k0, u, ra[u]);
                *reinterpret_cast<f32x4 *>(&lds.f.b[r][k]) = small_mask<true, FK>(x, n0, k0, u, rb[u]);
            }
        }
        __syncthreads();
        if (k0 + FK < t.d) load(k0 + FK);
        if (t.kern.kernel == KKM_GAUSS)
            for (int l = lane; l < klim; l += kWave)
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const float x = nrow[u * FLDK + l];
                    s8[u] = fmaf(x, x, s8[u]);
                }
        if (wave < 4) {
            const float *pa = &lds.f.a[wm + i][kq], *pb = &lds.f.b[wn + i][kq];
            for (int s = 0; s < klim; s += 32)
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(pa[s + 2 * u], pb[s + 2 * u], acc, 0, 0, 0);
        }
        __syncthreads();
    }
    if (t.kern.kernel == KKM_GAUSS) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            s8[u] = wave_sum(s8[u]);
            if (lane == 0) lds.f.nrm[first + u] = s8[u];
        }
        __syncthreads();
    }
    if (wave >= 4) return;
    const int64_t n = n0 + wn + i;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int mr = wm + 4 * q + r;
        const int64_t m = m0 + mr;
        if (m >= t.B || n >= t.B) continue;
        const float b = acc[r];
        const bool gauss = t.kern.kernel == KKM_GAUSS;
        float v = gt::kappa_from_dot(b, gauss ? lds.f.nrm[mr] : 0.f, gauss ? lds.f.nrm[ST + wn + i] : 0.f,
                                     t.kern.kernel, t.kern.gamma, t.kern.coef0, t.kern.degree);
        if (gauss && m == n) v = isfinite(b) ? 1.0f : __builtin_nanf("");
        t.KB[m * t.ldkb + n] = v;
    }
}

// ---------------------------------------------------------------- the launches

// Launches 1-3 and 5: a layer forward, or its input gradient.  The first nkb
// workgroups of launch 1 compute the kernel values instead.
template <bool BK, int EPI, bool KERN>
__global__ __launch_bounds__(SNT) void train_layer(SmallGemm g, TrainStep t, int64_t nkb) {
    __shared__ __attribute__((aligned(16))) TrainLds lds;
    if (KERN && blockIdx.x < nkb)
        batch_kernel_tile(t, blockIdx.x, lds);
    else
        small_tile<true, BK, SK, EPI>(g, blockIdx.x - nkb, AdamArgs{}, lds.h);
}

// Launch 6: the first layer's dZ, and the last layer's weights.
template <bool ADAM>
__global__ __launch_bounds__(SNT) void train_mid(SmallGemm dz, int64_t ndz, SmallGemm dw, SmallBias db,
                                                 int64_t ndb, AdamArgs ad) {
    __shared__ __attribute__((aligned(16))) SmallLds lds;
    int64_t b = blockIdx.x;
    if (b < ndz) return small_tile<true, false, SK, SE_GELU_BWD>(dz, b, ad, lds);
    b -= ndz;
    if (b < ndb) return small_bias<ADAM>(db, b, ad);
    small_tile<false, false, (int)kSmallBatch, ADAM ? SE_ADAM : SE_GRAD>(dw, b - ndb, ad, lds);
}

// Launch 7: the other layers' weights, and the loss.
template <bool ADAM>
__global__ __launch_bounds__(SNT) void train_last(SmallBias db2, int64_t nb2, SmallBias db1, int64_t nb1,
                                                  SmallGemm dw2, int64_t n2, SmallGemm dw1, AdamArgs ad,
                                                  const double *part, int64_t np, double scale, double *loss) {
    __shared__ __attribute__((aligned(16))) SmallLds lds;
    int64_t b = blockIdx.x;
    if (b == 0) {
        if (threadIdx.x == 0) {
            double s = 0.0;
            for (int64_t p = 0; p < np; ++p) s += part[p];
            *loss = s * scale;
        }
        return;
    }
    b -= 1;
    if (b < nb2) return small_bias<ADAM>(db2, b, ad);
    b -= nb2;
    if (b < nb1) return small_bias<ADAM>(db1, b, ad);
    b -= nb1;
    // one body for both: each has its own copy of some forty scalars otherwise
    const bool second = b < n2;
    small_tile<false, false, (int)kSmallBatch, ADAM ? SE_ADAM : SE_GRAD>(second ? dw2 : dw1, second ? b : b - n2, ad, lds);
}

// Launch 4: one workgroup per 16 rows.  G's rows stay in LDS: the waves take
// its 16 x 16 tiles in turn (Phi staged KC columns at a time so that all B rows
// fit), then dPhi's.
constexpr int LR = 16;                                    // rows per workgroup
constexpr int LPhi = (int)kSmallBatch * (128 + 4);        // floats staged: 128 rows of 256, 256 of 128
constexpr int LG = (int)kSmallBatch + 4;                  // stride of G's rows
constexpr int LT = (int)kSmallBatch / 16 / (SNT / kWave); // most tiles of G per wave

__global__ __launch_bounds__(SNT) void train_loss(TrainStep t, int kc, float alpha) {
    __shared__ __attribute__((aligned(16))) float phi[LPhi];
    __shared__ float G[LR][LG];
    __shared__ double red[SNT / kWave];
    const int64_t r0 = (int64_t)blockIdx.x * LR;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4, i = lane & 15;
    const int B = (int)t.B;
    const int nt = (B + 15) / 16;  // column tiles of G
    const int ld = kc + 4;
    f32x4 acc[LT], kb[LT];
#pragma unroll
    for (int u = 0; u < LT; ++u) {
        acc[u] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int c = min(16 * (wave + u * (SNT / kWave)) + i, B - 1);
#pragma unroll
        for (int r = 0; r < 4; ++r) kb[u][r] = t.KB[min(r0 + 4 * q + r, (int64_t)(B - 1)) * t.ldkb + c];
    }
    const int kv = kc / 4, dr = SNT / kv, dk = SNT % kv;
    const bool vec = (t.out & 3) == 0;  // Phi is the workspace's own, 256-byte aligned
    // the sums of NT of the wave's tiles over the staged columns
    auto sums = [&](auto tiles, int klim) {
        constexpr int NT = decltype(tiles)::value;
        const float *pa = phi + (int)(r0 + i) * ld + q;
        const float *pb = phi + (16 * wave + i) * ld + q;
        const int step = 16 * (SNT / kWave) * ld;
        auto step4 = [&](int s) {
            const float a = pa[s];
#pragma unroll
            for (int u = 0; u < NT; ++u)
                acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, pb[u * step + s], acc[u], 0, 0, 0);
        };
        int s = 0;
        for (; s + 64 <= klim; s += 64)  // LDS reads of sixteen steps in flight
#pragma unroll
            for (int u = 0; u < 16; ++u) step4(s + 4 * u);
        for (; s < klim; s += 4) step4(s);
    };
    const int mine = (nt - wave + SNT / kWave - 1) / (SNT / kWave);  // tiles of this wave (<= 0: none)
    for (int64_t k0 = 0; k0 < t.out; k0 += kc) {
        auto stage = [&](auto vector) {
            int r = tid / kv, k = tid % kv;  // stepped, not divided
            while (r < 16 * nt) {            // eight loads in flight
                f32x4 v[8];
                int rr[8], kk[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    rr[u] = r;
                    kk[u] = 4 * k;
                    v[u] = line4<decltype(vector)::value>(t.Phi, r * t.out, k0 + kk[u], t.out, r < B);
                    r += dr;
                    k += dk;
                    if (k >= kv) {
                        k -= kv;
                        ++r;
                    }
                }
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (rr[u] < 16 * nt)
                        *reinterpret_cast<f32x4 *>(&phi[rr[u] * ld + kk[u]]) =
                            mask4(v[u], k0 + kk[u], t.out, rr[u] < B);
            }
        };
        if (vec)
            stage(std::true_type{});
        else
            stage(std::false_type{});
        __syncthreads();
        const int klim = (int)min((int64_t)kc, t.out - k0);
        static_assert(LT == 2, "one or two tiles per wave");
        if (mine >= 2)
            sums(std::integral_constant<int, 2>{}, klim);
        else if (mine == 1)
            sums(std::integral_constant<int, 1>{}, klim);
        __syncthreads();
    }
    double sq = 0.0;
#pragma unroll
    for (int u = 0; u < LT; ++u) {
        const int ct = wave + u * (SNT / kWave);
        if (ct >= nt) continue;
        const int c = 16 * ct + i;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t m = r0 + 4 * q + r;
            float e = 0.f;
            if (m < B && c < B) {
                e = acc[u][r] - kb[u][r];
                sq += (double)e * (double)e;
            }
            G[4 * q + r][c] = e;  // 0 past the batch: dPhi's chain takes whole steps of 4
        }
    }
    sq = wave_sum(sq);
    if (lane == 0) red[wave] = sq;
    __syncthreads();
    if (tid == 0) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < SNT / kWave; ++w) s += red[w];
        t.part[blockIdx.x] = s;
    }
    // dPhi: k runs over the batch, 16 steps of 4 in flight; Phi from LDS where
    // all its columns are staged (rows past the batch are zeros there)
    const bool whole = kc >= t.out;
    for (int64_t c0 = 16 * wave; c0 < t.out; c0 += 16 * (SNT / kWave)) {
        const int64_t c = c0 + i;
        f32x4 d = {0.f, 0.f, 0.f, 0.f};
        for (int s = 0; s < B; s += 64) {
            float b[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int k = s + 4 * u + q;
                float x;
                if (whole)  // uniform
                    x = phi[min(k, B - 1) * ld + min((int)c, ld - 1)];
                else
                    x = t.Phi[min(k, B - 1) * t.out + min(c, t.out - 1)];
                b[u] = k < B ? x : 0.f;
            }
#pragma unroll
            for (int u = 0; u < 16; ++u)
                if (s + 4 * u < B) d = __builtin_amdgcn_mfma_f32_16x16x4f32(G[i][s + 4 * u + q], b[u], d, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t m = r0 + 4 * q + r;
            if (m < B && c < t.out) t.dPhi[m * t.out + c] = alpha * d[r];
        }
    }
}

}  // namespace

kkm_status train_step_small(const TrainStep &t, const AdamArgs *adam, hipStream_t s) {
    const AdamArgs ad = adam ? *adam : AdamArgs{};
    const dim3 b(SNT);
    auto grid = [](int64_t n) { return dim3((unsigned)n); };

    SmallGemm g = small_gemm(true, true, t.XB, t.ldx, t.th + t.oW1, t.d, t.B, t.h1, t.d, t.Z1, t.h1);
    g.C2 = t.H1;
    g.x = t.th + t.ob1;
    const int64_t bt = (t.B + ST - 1) / ST;
    const int64_t nkb = t.kern.kernel >= 0 ? bt * bt : 0;
    hipLaunchKernelGGL((train_layer<true, SE_BIAS_GELU, true>), grid(nkb + small_tiles(g)), b, 0, s, g, t, nkb);
    KKM_HIP(hipGetLastError());
    g = small_gemm(true, true, t.H1, t.h1, t.th + t.oW2, t.h1, t.B, t.h2, t.h1, t.Z2, t.h2);
    g.C2 = t.H2;
    g.x = t.th + t.ob2;
    hipLaunchKernelGGL((train_layer<true, SE_BIAS_GELU, false>), grid(small_tiles(g)), b, 0, s, g, t, (int64_t)0);
    KKM_HIP(hipGetLastError());
    g = small_gemm(true, true, t.H2, t.h2, t.th + t.oW3, t.h2, t.B, t.out, t.h2, t.Phi, t.out);
    g.x = t.th + t.ob3;
    hipLaunchKernelGGL((train_layer<true, SE_BIAS, false>), grid(small_tiles(g)), b, 0, s, g, t, (int64_t)0);
    KKM_HIP(hipGetLastError());

    const double b2 = (double)t.B * (double)t.B;
    // the widest stretch of Phi's columns whose rows (whole tiles of 16) fit
    const int rows = (int)((t.B + 15) & ~int64_t(15));
    int kc = LPhi / rows - 4;
    kc = kc > 256 ? 256 : kc & ~3;
    hipLaunchKernelGGL(train_loss, grid((t.B + LR - 1) / LR), b, 0, s, t, kc, (float)(4.0 / b2));
    KKM_HIP(hipGetLastError());

    g = small_gemm(true, false, t.dPhi, t.out, t.th + t.oW3, t.h2, t.B, t.h2, t.out, t.dZ2, t.h2);
    g.x = t.Z2;
    hipLaunchKernelGGL((train_layer<false, SE_GELU_BWD, false>), grid(small_tiles(g)), b, 0, s, g, t, (int64_t)0);
    KKM_HIP(hipGetLastError());

    float *dst = adam ? t.th : t.grad;
    auto weights = [&](const float *dZ, int64_t rows_w, const float *in, int64_t ldin, int64_t cols, int64_t off) {
        SmallGemm w = small_gemm(false, false, dZ, rows_w, in, ldin, rows_w, cols, t.B, dst + off, cols);
        w.am = t.am + (adam ? off : 0);
        w.av = t.av + (adam ? off : 0);
        return w;
    };
    auto bias = [&](const float *dZ, int64_t cols, int64_t off) {
        return SmallBias{dZ, t.B, cols, dst + off, t.am + (adam ? off : 0), t.av + (adam ? off : 0)};
    };
    auto bias_blocks = [](int64_t cols) { return (cols + SNT - 1) / SNT; };

    g = small_gemm(true, false, t.dZ2, t.h2, t.th + t.oW2, t.h1, t.B, t.h1, t.h2, t.dZ1, t.h1);
    g.x = t.Z1;
    const SmallGemm w3 = weights(t.dPhi, t.out, t.H2, t.h2, t.h2, t.oW3);
    const int64_t nb3 = bias_blocks(t.out);
    const dim3 mid = grid(small_tiles(g) + nb3 + small_tiles(w3));
    const SmallBias db3 = bias(t.dPhi, t.out, t.ob3);
    if (adam)
        hipLaunchKernelGGL(train_mid<true>, mid, b, 0, s, g, small_tiles(g), w3, db3, nb3, ad);
    else
        hipLaunchKernelGGL(train_mid<false>, mid, b, 0, s, g, small_tiles(g), w3, db3, nb3, ad);
    KKM_HIP(hipGetLastError());

    const SmallGemm w2 = weights(t.dZ2, t.h2, t.H1, t.h1, t.h1, t.oW2);
    const SmallGemm w1 = weights(t.dZ1, t.h1, t.XB, t.ldx, t.d, t.oW1);
    const SmallBias db2 = bias(t.dZ2, t.h2, t.ob2), db1 = bias(t.dZ1, t.h1, t.ob1);
    const int64_t nb2 = bias_blocks(t.h2), nb1 = bias_blocks(t.h1);
    const dim3 lastg = grid(1 + nb2 + nb1 + small_tiles(w2) + small_tiles(w1));
    const int64_t np = (t.B + LR - 1) / LR;
    if (adam)
        hipLaunchKernelGGL(train_last<true>, lastg, b, 0, s, db2, nb2, db1, nb1, w2, small_tiles(w2), w1, ad,
                           t.part, np, 1.0 / b2, t.loss);
    else
        hipLaunchKernelGGL(train_last<false>, lastg, b, 0, s, db2, nb2, db1, nb1, w2, small_tiles(w2), w1, ad,
                           t.part, np, 1.0 / b2, t.loss);
    KKM_HIP(hipGetLastError());
    return KKM_OK;
}

}  // namespace kkm
