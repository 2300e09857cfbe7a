// 32 x 32 tiles of a product with bfloat16 operands, for small shapes: up to
// 512 k are staged in LDS at once (bfloat16, rounded to nearest even), so that
// a workgroup waits for memory once or twice where slabs of 32 k waited at
// every slab (64 x 64 tiles, M = 64, N = K = 512: 35 us in 8 workgroups; here
// 32 workgroups, 5.5 us).  Eight waves load, four hold a 16 x 16 quadrant
// each.  The 16x16x32 MFMA adds its k in the order in which two 32x32x16 do
// (checked bit for bit on gfx950), so results are those of the larger tiles.
// Internal to the library.
#pragma once

#include "gemm.h"

namespace kkm {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int ST = 32;          // tile edge
constexpr int SNT = 512;        // threads: all load, four waves hold a 16 x 16 quadrant each
constexpr int SK = 512;         // k staged at a time
constexpr int SLDK = SK + 8;    // LDS row stride (bf16): 16-byte reads of 16 rows hit all banks once

struct SmallLds {
    __bf16 a[ST][SLDK], b[ST][SLDK];
};

enum SmallEpi { SE_BIAS, SE_BIAS_GELU, SE_GELU_BWD, SE_GRAD, SE_ADAM };

// An operand: P(r, k) = P[r * ld + k] (KC, k contiguous) or P[k * ld + r].
struct SmallOperand {
    const float *P;
    int64_t ld, rows, K;
    int vec;
};

// C[m][n] = sum_k A(m,k) B(n,k), operands rounded to bfloat16.
struct SmallGemm {
    SmallOperand A, B;
    int64_t M, N, K;
    float *C;           // SE_BIAS / SE_BIAS_GELU: Z; SE_GELU_BWD / SE_GRAD: C; SE_ADAM: the weights
    float *C2;          // SE_BIAS_GELU: H
    const float *x;     // bias, or Z of the GELU derivative
    float *am, *av;     // SE_ADAM: moments
    int64_t ldc;
    int64_t tn;         // tiles along n
};

// Lines of `len` elements, ld apart, that 16-byte loads can read whole.
__host__ __device__ inline int vec_ok(const float *p, int64_t ld, int64_t len) {
    return (ld & 3) == 0 && (len & 3) == 0 && (reinterpret_cast<uintptr_t>(p) & 15) == 0;
}

// 4 consecutive elements e0 .. e0+3 of the line at base + at; any valid
// element of `base` in the place of those past `len` or of a line that is not
// there (!in).  VEC: whole quads, 16-byte aligned.  No branch, and the caller
// masks when it uses them: behind a branch or a select the compiler waits for
// each load before the next, and a workgroup's loads no longer overlap (K =
// 512: 7.6 us a layer, so 5.5).
template <bool VEC>
__device__ __forceinline__ f32x4 line4(const float *base, int64_t at, int64_t e0, int64_t len, bool in) {
    if constexpr (VEC) return *reinterpret_cast<const f32x4 *>(base + (in && e0 < len ? at + e0 : 0));
    f32x4 v;
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = base[in && e0 + u < len ? at + e0 + u : 0];
    return v;
}
__device__ __forceinline__ f32x4 mask4(f32x4 v, int64_t e0, int64_t len, bool in) {
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = in && e0 + u < len ? v[u] : 0.f;
    return v;
}

// The calling thread's share of rows r0 .. r0+31, k k0 .. k0+KS-1: KC: KS/64
// groups of 4 k of one row; else a block of KS/64 k x 4 rows.
template <bool KC, int KS>
__device__ __forceinline__ void small_at(int u, int64_t r0, int64_t k0, int64_t &r, int64_t &k) {
    const int t = threadIdx.x;
    if constexpr (KC) {
        const int e = t + SNT * u;
        r = r0 + e / (KS / 4);
        k = k0 + 4 * (e % (KS / 4));
    } else {
        r = r0 + 4 * (t & 7);
        k = k0 + (KS / 64) * (t >> 3) + u;
    }
}
template <bool KC, int KS>
__device__ __forceinline__ void small_load(const SmallOperand &o, int64_t r0, int64_t k0, f32x4 (&v)[KS / 64]) {
    auto load = [&](auto vec) {
        constexpr bool V = decltype(vec)::value;
#pragma unroll
        for (int u = 0; u < KS / 64; ++u) {
            int64_t r, k;
            small_at<KC, KS>(u, r0, k0, r, k);
            v[u] = KC ? line4<V>(o.P, r * o.ld, k, o.K, r < o.rows) : line4<V>(o.P, k * o.ld, r, o.rows, k < o.K);
        }
    };
    if (o.vec)  // uniform
        load(std::true_type{});
    else
        load(std::false_type{});
}
template <bool KC, int KS>
__device__ __forceinline__ f32x4 small_mask(const SmallOperand &o, int64_t r0, int64_t k0, int u, f32x4 v) {
    int64_t r, k;
    small_at<KC, KS>(u, r0, k0, r, k);
    return KC ? mask4(v, k, o.K, r < o.rows) : mask4(v, r, o.rows, k < o.K);
}

// ... and into LDS as bfloat16 [row][k]; klim: k staged (a multiple of 32).
template <bool KC, int KS>
__device__ __forceinline__ void small_stage(const SmallOperand &o, int64_t r0, int64_t k0,
                                            const f32x4 (&v)[KS / 64], int klim, __bf16 (*S)[SLDK]) {
    const int t = threadIdx.x;
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    if constexpr (KC) {
#pragma unroll
        for (int u = 0; u < KS / 64; ++u) {
            const int e = t + SNT * u;
            const int r = e / (KS / 4), k = 4 * (e % (KS / 4));
            if (k < klim)
                *reinterpret_cast<bf16x4 *>(&S[r][k]) =
                    __builtin_convertvector(small_mask<KC, KS>(o, r0, k0, u, v[u]), bf16x4);
        }
    } else {
        constexpr int U = KS / 64;
        typedef __bf16 bf16xu __attribute__((ext_vector_type(U)));
        const int k = U * (t >> 3), r = 4 * (t & 7);
        if (k < klim) {
            f32x4 m[U];
#pragma unroll
            for (int u = 0; u < U; ++u) m[u] = small_mask<KC, KS>(o, r0, k0, u, v[u]);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                bf16xu w;
#pragma unroll
                for (int u = 0; u < U; ++u) w[u] = (__bf16)m[u][e];
                *reinterpret_cast<bf16xu *>(&S[r + e][k]) = w;
            }
        }
    }
}

// Tile `tile` of a product, by the workgroup's 512 threads.
template <bool AK, bool BK, int KS, int EPI>
__device__ __forceinline__ void small_tile(const SmallGemm &g, int64_t tile, const AdamArgs &ad, SmallLds &lds) {
    const int64_t m0 = (tile / g.tn) * ST, n0 = (tile % g.tn) * ST;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4, i = lane & 15;
    const int wm = 16 * ((wave >> 1) & 1), wn = 16 * (wave & 1);
    f32x4 ra[KS / 64], rb[KS / 64];
    small_load<AK, KS>(g.A, m0, 0, ra);
    small_load<BK, KS>(g.B, n0, 0, rb);

    // what the epilogue reads, in flight with the operands (the last row or
    // column where the tile passes the edge)
    const int64_t n = n0 + wn + i, nc = min(n, g.N - 1);
    float x0[4], x1[4], x2[4];
    bool in[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t m = m0 + wm + 4 * q + r, at = min(m, g.M - 1) * g.ldc + nc;
        in[r] = wave < 4 && m < g.M && n < g.N;
        x0[r] = x1[r] = x2[r] = 0.f;
        if constexpr (EPI == SE_BIAS || EPI == SE_BIAS_GELU) x0[r] = g.x[nc];
        if constexpr (EPI == SE_GELU_BWD) x0[r] = g.x[at];
        if constexpr (EPI == SE_ADAM) {
            x0[r] = g.C[at];
            x1[r] = g.am[at];
            x2[r] = g.av[at];
        }
    }

    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int64_t k0 = 0; k0 < g.K; k0 += KS) {
        const int klim = (int)((min((int64_t)KS, g.K - k0) + 31) & ~int64_t(31));
        small_stage<AK, KS>(g.A, m0, k0, ra, klim, lds.a);
        small_stage<BK, KS>(g.B, n0, k0, rb, klim, lds.b);
        __syncthreads();
        if (k0 + KS < g.K) {
            small_load<AK, KS>(g.A, m0, k0 + KS, ra);
            small_load<BK, KS>(g.B, n0, k0 + KS, rb);
        }
        if (wave < 4) {
            const __bf16 *pa = &lds.a[wm + i][8 * q], *pb = &lds.b[wn + i][8 * q];
            auto step = [&](int s) {
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8 *>(pa + s),
                                                              *reinterpret_cast<const bf16x8 *>(pb + s),
                                                              acc, 0, 0, 0);
            };
            int s = 0;
            for (; s + 256 <= klim; s += 256)  // LDS reads of eight steps in flight
#pragma unroll
                for (int u = 0; u < 8; ++u) step(s + 32 * u);
            for (; s + 64 <= klim; s += 64) {
                step(s);
                step(s + 32);
            }
            if (s < klim) step(s);
        }
        __syncthreads();
    }
    // register r of lane (q, i): row 4q + r, column i of the wave's quadrant
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if (!in[r]) continue;
        const int64_t at = (m0 + wm + 4 * q + r) * g.ldc + n;
        if constexpr (EPI == SE_BIAS) {
            g.C[at] = acc[r] + x0[r];
        } else if constexpr (EPI == SE_BIAS_GELU) {
            const float z = acc[r] + x0[r];
            if (g.C) g.C[at] = z;
            g.C2[at] = gelu(z);
        } else if constexpr (EPI == SE_GELU_BWD) {
            g.C[at] = acc[r] * gelu_grad(x0[r]);
        } else if constexpr (EPI == SE_GRAD) {
            g.C[at] = acc[r];
        } else {
            adam_one(x0[r], x1[r], x2[r], acc[r], ad);
            g.C[at] = x0[r];
            g.am[at] = x1[r];
            g.av[at] = x2[r];
        }
    }
}

SmallGemm small_gemm(bool ak, bool bk, const float *A, int64_t lda, const float *B, int64_t ldb, int64_t M,
                     int64_t N, int64_t K, float *C, int64_t ldc) {
    SmallGemm g{};
    g.A = SmallOperand{A, lda, M, K, vec_ok(A, lda, ak ? K : M)};
    g.B = SmallOperand{B, ldb, N, K, vec_ok(B, ldb, bk ? K : N)};
    g.M = M;
    g.N = N;
    g.K = K;
    g.C = C;
    g.ldc = ldc;
    g.tn = (N + ST - 1) / ST;
    return g;
}

int64_t small_tiles(const SmallGemm &g) { return g.tn * ((g.M + ST - 1) / ST); }

}  // namespace

}  // namespace kkm
