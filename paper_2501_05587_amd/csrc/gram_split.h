// The FP32 product of the kernel matrix on the bfloat16 matrix units: every
// FP32 value is the sum of three bfloat16 values, x = h + m + l exactly (each the
// rounding of what the ones before left: 8 bits of the 24), and
//   x y = h h' + (h m' + m h' + m m' + h l' + l h' + m l' + l m') + l l'
// with l l' below 2^-33 |x y|.  Eight v_mfma_f32_32x32x16_bf16 with exact products
// and FP32 sums take the place of eight v_mfma_f32_32x32x2_f32 at a sixteenth of
// their cost each (2.5 PFLOP/s against 157 TFLOP/s).
//
// The products h h' have sums of their own, a slab's 32 features from zero and
// the slabs' rounded to nearest: these products have 16 bits, so that FP32 adds a
// few of them without rounding.  All the others are below 2^-6 of them, and the
// roundings of their sum below 2^-29.  The two meet once, in the last slab.  So
// a single product is rounded once, as the FP32 matrix unit rounds it, and a sum
// less often: with one sum for all of them, a slab with one feature that both
// rows have cost two roundings more, and sparse rows were less exact than on the
// FP32 unit.  Without m l' and l m' (below 2^-24 |x y| together) a single product
// was off by up to 1.5 times as much.
// Error against 64 bits, relative in norm, of X X^T, n = 3600, here / FP32 matrix
// unit / six products with one sum a slab: normal points d = 16 3.2e-8 / 7.4e-8 /
// 3.4e-8, d = 128 5.4e-8 / 2.0e-7 / 8.0e-8, d = 784 9.9e-8 / 4.9e-7 / 1.2e-7; one
// entry in five not zero d = 64 2.9e-8 / 3.9e-8 / 5.1e-8, d = 784 5.3e-8 / 1.2e-7 /
// 9.8e-8; one feature 2.5e-8 / 2.5e-8 / 3.5e-8.  The matrix unit sums eight products
// at a time and cuts each off at 2^-24 of the largest one's power of two, so of few
// features that differ by many powers of two the FP32 unit's chain is the more
// exact where it happens to add the small ones first (feature k scaled by 4^k, d =
// 16 5.7e-8 / 2.5e-8; log-normal values over 2^+-4, d = 64 7.1e-8 / 6.8e-8, from d =
// 128 on 0.92 to 0.14 of it); the bound of the sum is no larger.
//
// n = 60000, d = 784: 25.4 -> 18.7 ms, 1.21 PFLOP/s of bfloat16 products, the
// rate that a plain bfloat16 product of 8192^3 reaches on this card (1.13).
//
// Values whose low parts would leave the bfloat16 range, and infinities and
// NaNs (inf - inf inside a split), are left to the FP32 unit: the prologue marks
// their rows in the sign of the squared norm, and a tile with a marked row is the
// FP32 kernel's tile.
//
// The parts are laid out once (PRE) where the workspace has room for them, else
// split while they are staged: the same parts, so the same K bit for bit (n =
// 60000, d = 784 18.8 / 22.1 ms, d = 128 4.6 / 5.0; n = 3584, d = 128 42 / 41 us).
//
// Per 32-feature slab a 128 x 128 tile stages 2 x 24 KiB with direct
// global-to-LDS loads, already in LDS order (the prologue wrote them so), single
// buffered: two workgroups per CU (128 accumulators a lane) hide each other's
// loads behind 64 MFMAs a wave and slab.  The bound is the matrix units' power.
// Shared by the single- and many-instance Gram kernels.  Internal to the library.
#pragma once

#include "gram_tile.h"

namespace kkm {
namespace gt {

namespace {

// Rows are grouped by 16; a slab of 32 features of a group is three planes (h,
// m, l) of 16 x 64 bytes.  16-byte chunk c of row r sits at chunk position
// c ^ (r / 4 % 4), which spreads the fragment reads of 16 rows over all banks.
constexpr int SPG = 16;                       // rows per group
constexpr int SPK = 32;                       // features per slab
constexpr int SPP = SPG * SPK * 2;            // bytes of one plane of a group
constexpr int SPB = 3 * SPP;                  // bytes of a group's slab
constexpr int SPT = GM / SPG * SPB;           // bytes of a tile operand's slab

struct SplitLds {
    union {
        unsigned char op[2][SPT];
        float T[epi_lds_bytes(1) / sizeof(float)];  // the epilogue's tile
    };
    float rn[2 * GM], rs[2 * GM];
};

// A matrix split and laid out: Xs [slab][group][plane][16 rows x 64 bytes].
struct SplitTile {
    const unsigned char *Xs;
    int64_t slab_bytes;       // groups * SPB
    int64_t nslab;
};

union SplitOrF32Lds {
    SplitLds s;
    F32Lds f;
};

__host__ __device__ inline int64_t split_groups(int64_t n) { return (n + GM - 1) / GM * (GM / SPG); }
__host__ __device__ inline int64_t split_slabs(int64_t d) { return (d + SPK - 1) / SPK; }
__host__ __device__ inline SplitTile split_source(const unsigned char *Xs, int64_t n, int64_t d) {
    return SplitTile{Xs, split_groups(n) * SPB, split_slabs(d)};
}

// Where chunk c of row r (of 128) of a tile operand's slab sits.
__device__ __forceinline__ int split_at(int r, int c) {
    return (r / SPG) * SPB + (r % SPG) * (SPK * 2) + ((c ^ ((r >> 2) & 3)) * 16);
}

// The three parts of the eight features k0 .. k0+7 of a row, x (zeros past d, or
// all zeros if !in), 16 bytes each, SPP apart.
__device__ __forceinline__ void split_store(const float (&x)[8], int64_t d, int64_t k0, bool in, unsigned char *dst) {
    bf16x8 h, m, l;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const float v = (in && k0 + u < d) ? x[u] : 0.f;
        h[u] = (__bf16)v;
        const float v1 = v - (float)h[u];
        m[u] = (__bf16)v1;
        l[u] = (__bf16)(v1 - (float)m[u]);
    }
    *reinterpret_cast<bf16x8 *>(dst) = h;
    *reinterpret_cast<bf16x8 *>(dst + SPP) = m;
    *reinterpret_cast<bf16x8 *>(dst + 2 * SPP) = l;
}
__device__ __forceinline__ void split_load(const float *x, int64_t d, int64_t k0, float (&v)[8]) {
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = x[min(k0 + u, d - 1)];
}

// Whether a row (one whole wave) has a value outside the split's range: neither
// zero nor between 2^-45 and 2^50 in size, or not finite.  Within it the parts
// hold every bit, no product or sum that counts is subnormal, and no sum of
// fewer than 2^27 features overflows.
__device__ __forceinline__ bool split_row_bad(const float *x, int64_t d, int lane) {
    bool bad = false;
    for (int64_t k = lane; k < d; k += kWave) {
        const float v = fabsf(x[k]);
        bad |= !(v == 0.f || (v >= 0x1p-45f && v <= 0x1p50f));
    }
    return __ballot(bad) != 0;
}

// A row's squared norm (or 0) and, in its sign, whether the row is outside the
// split's range, by one whole wave.
__device__ __forceinline__ void split_row_stats(const float *x, int64_t d, bool norm, float *nrm, int lane) {
    float s = 0.f;
    if (norm) sqnorm_row(x, d, &s, lane);  // lane 0's
    const bool bad = split_row_bad(x, d, lane);
    if (lane == 0) *nrm = bad ? __uint_as_float(__float_as_uint(s) | 0x80000000u) : fabsf(s);
}

// Whether the tile (rows m0.., columns n0..) has a row outside the split's
// range (the whole workgroup calls).
__device__ __forceinline__ bool outside_split(const Epi &e, int64_t m0, int64_t n0) {
    const int t = threadIdx.x;
    const int64_t g = (t < GM) ? m0 + t : n0 + (t - GM);
    return __syncthreads_or(g < e.n && (__float_as_uint(e.nrm[g]) >> 31) != 0) != 0;
}

// One 128 x 128 tile (bi, bj) and its epilogue.  FULL: tiles below the diagonal
// swap the order of mixed terms, so they round as their mirror above does.
// !PRE: the rows are split as they are staged.
template <typename OUT, bool FULL, bool PRE>
__device__ __forceinline__ void split_tile(const SplitTile &x, const F32Tile &src, int64_t bi, int64_t bj,
                                           SplitLds &lds) {
    const Epi &e = src.e;
    const int64_t m0 = bi * GM, n0 = bj * GM;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave >> 1, wc = wave & 1;
    const int half = lane >> 5, l32 = lane & 31;

    // each wave copies a quarter of both operands' slabs, 1 KiB at a time
    constexpr int Q = SPT / 4, NB = Q / 1024;
    const unsigned char *ga = x.Xs + bi * SPT + wave * Q + lane * 16;
    const unsigned char *gb = x.Xs + bj * SPT + wave * Q + lane * 16;
    typedef __attribute__((address_space(3))) void lds_void;
    typedef const __attribute__((address_space(1))) void glb_void;
    auto fetch = [&](int64_t kt) {
        if constexpr (!PRE) {
            // two chunks of 8 features of each operand per thread, all their loads in flight
            float v[2][2][8];
            const int64_t k0 = kt * SPK + 8 * (tid & 3);
            auto load = [&](auto vec) {
#pragma unroll
                for (int o = 0; o < 2; ++o)
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const int64_t row = (o ? n0 : m0) + (tid >> 2) + 64 * u;
                        const float *p = src.X + min(row, e.n - 1) * src.ldx;
                        if constexpr (decltype(vec)::value) {
                            const f32x4 q0 = *reinterpret_cast<const f32x4 *>(p + k0);
                            const f32x4 q1 = *reinterpret_cast<const f32x4 *>(p + k0 + 4);
#pragma unroll
                            for (int c = 0; c < 4; ++c) v[o][u][c] = q0[c], v[o][u][4 + c] = q1[c];
                        } else {
                            split_load(p, src.d, k0, v[o][u]);
                        }
                    }
            };
            if (src.vec_x && (kt + 1) * SPK <= src.d)  // uniform
                load(std::true_type{});
            else
                load(std::false_type{});
#pragma unroll
            for (int o = 0; o < 2; ++o)
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int r = (tid >> 2) + 64 * u;
                    split_store(v[o][u], src.d, k0, (o ? n0 : m0) + r < e.n, lds.op[o] + split_at(r, tid & 3));
                }
            return;
        }
#pragma unroll
        for (int b = 0; b < NB; ++b)
            __builtin_amdgcn_global_load_lds((glb_void *)(ga + b * 1024), (lds_void *)(&lds.op[0][wave * Q + b * 1024]),
                                             16, 0, 0);
#pragma unroll
        for (int b = 0; b < NB; ++b)
            __builtin_amdgcn_global_load_lds((glb_void *)(gb + b * 1024), (lds_void *)(&lds.op[1][wave * Q + b * 1024]),
                                             16, 0, 0);
        ga += x.slab_bytes;
        gb += x.slab_bytes;
    };

    // hi: the products h h'; lo: all the others
    f32x16 hi[2][2], lo[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) hi[i][j][r] = lo[i][j][r] = 0.f;

    stage_norms(e, m0, n0, lds.rn, lds.rs);
    // lane half h of MFMA s takes the 8 features of chunk 2s + h of its row
    const int swz = (l32 >> 2) & 3;
    const int frag = (l32 >> 4) * SPB + (l32 & 15) * 64;
    const unsigned char *As = lds.op[0] + wr * (4 * SPB) + frag, *Bs = lds.op[1] + wc * (4 * SPB) + frag;
    auto frag_of = [&](const unsigned char *op, int i, int p, int chunk) {
        return *reinterpret_cast<const bf16x8 *>(op + i * (2 * SPB) + p * SPP + chunk);
    };
    for (int64_t kt = 0; kt < x.nslab; ++kt) {
        fetch(kt);
        if constexpr (PRE) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int chunk = ((2 * s + half) ^ swz) * 16;
            // plane p of A's rows times plane q of B's
            auto product = [&](int p, int q) {
                bf16x8 a[2], b[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    a[i] = frag_of(As, i, p, chunk);
                    b[i] = frag_of(Bs, i, q, chunk);
                }
#pragma unroll
                for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                    for (int ni = 0; ni < 2; ++ni)
                        lo[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[mi], b[ni], lo[mi][ni], 0, 0, 0);
            };
            // a mixed pair: a tile below the diagonal takes it the other way round
            auto mixed = [&](int p, int q) {
                const int u = FULL && bi > bj ? q : p, v = FULL && bi > bj ? p : q;
                product(u, v);
                product(v, u);
            };
            mixed(1, 2);  // the small terms first
            mixed(0, 2);
            product(1, 1);
            mixed(0, 1);
        }
        // the rest joins the running sum before the last slab's h h': one rounding
        // less where those are most of it (features scaled from 2^-30 to 1, d = 128:
        // error in norm 4.1e-8; joined after them 4.8e-8, the FP32 unit 4.5e-8)
        if (kt + 1 == x.nslab)  // uniform
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) hi[i][j][r] += lo[i][j][r];
        // h h' of the slab, from zero, then rounded to nearest into the running sum:
        // the matrix unit's own additions to a long sum cut it off
#pragma unroll
        for (int mi = 0; mi < 2; ++mi) {
            f32x16 t[2];
#pragma unroll
            for (int ni = 0; ni < 2; ++ni) {
#pragma unroll
                for (int r = 0; r < 16; ++r) t[ni][r] = 0.f;
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const int chunk = ((2 * s + half) ^ swz) * 16;
                    t[ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_of(As, mi, 0, chunk), frag_of(Bs, ni, 0, chunk),
                                                                    t[ni], 0, 0, 0);
                }
            }
#pragma unroll
            for (int ni = 0; ni < 2; ++ni)
#pragma unroll
                for (int r = 0; r < 16; ++r) hi[mi][ni][r] += t[ni][r];
        }
        __syncthreads();  // every read of the slab is done
    }
    f32x16(&acc)[2][2] = hi;
    // FP32 K and the FULL shape: the tile staged whole, as the FP32 kernel's (in
    // halves FULL was 64 us at n = 5000, d = 32 where it is 53, and the FP32 kernel
    // 50); bfloat16 K: in halves, which hold it whole as bfloat16
    constexpr int HV = sizeof(OUT) == 2 ? 2 : 1;
    static_assert(sizeof(lds.T) >= epi_lds_bytes_bf16, "bfloat16 epilogue tile does not fit");
    if (FULL && bi != bj)
        epilogue<OUT, true, 1>(e, acc, m0, n0, false, wr, wc, lane, lds.T, lds.rn, lds.rs);
    else
        epilogue<OUT, false, HV>(e, acc, m0, n0, bi == bj, wr, wc, lane, lds.T, lds.rn, lds.rs);
}

}  // namespace

}  // namespace gt
}  // namespace kkm
