// Device code shared by the kernels of liblqfire: the discrete Landau-de
// Gennes force of one site, raw buffer access, block reductions and the FIRE
// controller.
#pragma once

#include <hip/hip_runtime.h>

#include "lq_internal.h"

namespace lq {

__device__ __forceinline__ double fma_t(double a, double b, double c) { return fma(a, b, c); }
__device__ __forceinline__ float fma_t(float a, float b, float c) { return fmaf(a, b, c); }

// Raw buffer access to one field (5 components, 5 N elements): the resource
// covers exactly the field, so an offset past its end reads 0 and drops the
// store; the component offset c N sizeof(T) goes in the scalar offset and the
// site offset in one 32-bit vector register.  A field must fit in 2^32 bytes.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t field_rsrc(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}
template <typename T>
__device__ __forceinline__ T bld(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, (int)soff, 0));
    } else {
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, (int)voff, (int)soff, 0));
    }
}
// Stores of the streamed fields: POL is the buffer instruction's
// cache-policy operand, 2 (bit 1) the non-temporal policy on gfx950, 0 the
// default one.
template <typename T, int POL>
__device__ __forceinline__ void bst_p(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, T v) {
    if constexpr (sizeof(T) == 4) {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, (int)voff, (int)soff, POL);
    } else {
        typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, (int)voff, (int)soff, POL);
    }
}
// Cache policy of a step kernel's state stores.  Non-temporal stores keep
// the written state from displacing lines the step still reuses: measured
// faster for the one-constant and the FP64 kernels (5% on the 256^3 boxes).
// The FP32 L2/L3 kernels measured faster with the default policy at every
// size (14% on the 128^3 bulk box, whose two state buffers fit in the
// 256 MiB Infinity Cache, 2-4% on the 512^3 patterned wall).  Rows that are no
// whole number of half lines (ROWS: they are) end tiles inside a line; the L2
// merges the two tiles' parts under the default policy, while non-temporal
// parts leave it one by one (FP32 200^3 270 -> 233 us per step, 230x187x141
// 243 -> 198, FP64 230x187x141 420 -> 388; rows of 64 bytes' multiples are
// faster non-temporal, FP64 200^3 505 and 520).  Where both state buffers fit
// in the Infinity Cache the step kernels take the default policy too: the
// next step then reads what this one wrote from there (FP32 128^3 66.1 -> 52.5,
// 112^3 57.1 -> 40.4; FP64 128x128x60 57.7 -> 48.9; FP64 L2/L3 96^3 69.3 -> 56.3,
// L4 96^3 102 -> 91; beyond it FP64 L2/L3 128^3 122.6 and 128.2, 256^3 FP32 414 and
// 420).  FP64 L2/L3 with ragged rows: 201x163x95 240 -> 228.  The force alone
// stays non-temporal (FP64 230x187x141 101 and 139 us).  A compile-time choice: a
// run-time one put a branch in the march loop that cost 1.5%.
template <typename T, bool L23, bool ROWS>
constexpr int store_policy() { return (L23 && sizeof(T) == 4) || !ROWS ? 0 : 2; }
// (15 values a site and buffer, also for gradient descent, whose steps use ten of them.)
template <typename T>
__host__ __device__ inline bool state_fits_cache(int64_t N) { return 2 * 15 * N * (int64_t)sizeof(T) <= (int64_t)256 << 20; }
template <typename T>
inline bool whole_rows(int nx) { return ((size_t)nx * sizeof(T)) % 64 == 0; }

// Barrier for data exchanged through LDS only: waits for this wave's LDS
// operations, not for its global loads and stores (which __syncthreads()
// would drain, stalling every plane on memory latency).
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

__device__ __forceinline__ int wrapc(int g, int n, int per) {
    if (g >= 0 && g < n) return g;
    if (!per) return -1;
    g %= n;
    return g < 0 ? g + n : g;
}

// Coordinate of a padded position g >= -1 of a tile or brick: wrapped, or -1 off
// an open edge.  Positions past n, where the tile hangs over the box, belong to
// no site's neighbourhood: -1, so that they load nothing.
__device__ __forceinline__ int wrap1(int g, int n, int per) {
    g = g < 0 ? (per ? n - 1 : -1) : g;
    g = g == n ? (per ? 0 : -1) : g;
    return g > n ? -1 : g;
}

__device__ __forceinline__ bool has_nb(uint32_t m, int k, int s) {
    return (m >> (2 * k + (s < 0 ? 1 : 0))) & 1u;
}

__device__ __forceinline__ int n_choices(uint32_t m, int k) {
    return (int)((m >> (2 * k)) & 1u) + (int)((m >> (2 * k + 1)) & 1u);
}

// Coefficients of C_k(x) = ap Q(x+e_k) + a0 Q(x) + am Q(x-e_k): the mean of
// the allowed one-sided differences along axis k.
template <typename T>
__device__ __forceinline__ void mean_diff_coef(uint32_t m, int k, T& ap, T& a0, T& am) {
    bool p = has_nb(m, k, +1), n = has_nb(m, k, -1);
    if (p && n) {
        ap = T(0.5); a0 = T(0); am = T(-0.5);
    } else if (p) {
        ap = T(1); a0 = T(-1); am = T(0);
    } else if (n) {
        ap = T(0); a0 = T(1); am = T(-1);
    } else {
        ap = T(0); a0 = T(0); am = T(0);
    }
}

template <typename T>
__device__ __forceinline__ void full_of(const T q[5], T Q[3][3]) {
    Q[0][0] = q[0]; Q[0][1] = q[1]; Q[0][2] = q[2];
    Q[1][0] = q[1]; Q[1][1] = q[3]; Q[1][2] = q[4];
    Q[2][0] = q[2]; Q[2][1] = q[4]; Q[2][2] = -q[0] - q[3];
}

template <typename T>
__device__ __forceinline__ void pT(const T G[3][3], T g[5]) {
    g[0] = G[0][0] - G[2][2];
    g[1] = G[0][1] + G[1][0];
    g[2] = G[0][2] + G[2][0];
    g[3] = G[1][1] - G[2][2];
    g[4] = G[1][2] + G[2][1];
}

// d(bulk)/dq = P^T (A Q + B Q^2 + C tr(Q^2) Q), written out in the five
// components: P^T Q = M q and P^T S = (Sxx - Szz, 2 Sxy, 2 Sxz, Syy - Szz,
// 2 Syz) for the symmetric S = Q^2.
template <typename T>
__device__ __forceinline__ void bulk_grad(const T q[5], T A, T B, T C, T g[5]) {
    const T zz = -q[0] - q[3];
    const T s01 = q[1] * q[1], s02 = q[2] * q[2], s04 = q[4] * q[4];
    const T t2 = q[0] * q[0] + q[3] * q[3] + zz * zz + T(2) * (s01 + s02 + s04);
    const T Sxx = q[0] * q[0] + s01 + s02;
    const T Syy = s01 + q[3] * q[3] + s04;
    const T Szz = s02 + s04 + zz * zz;
    const T Sxy = q[0] * q[1] + q[1] * q[3] + q[2] * q[4];
    const T Sxz = q[0] * q[2] + q[1] * q[4] + q[2] * zz;
    const T Syz = q[1] * q[2] + q[3] * q[4] + q[4] * zz;
    const T a = A + C * t2;
    g[0] = a * (T(2) * q[0] + q[3]) + B * (Sxx - Szz);
    g[1] = T(2) * (a * q[1] + B * Sxy);
    g[2] = T(2) * (a * q[2] + B * Sxz);
    g[3] = a * (q[0] + T(2) * q[3]) + B * (Syy - Szz);
    g[4] = T(2) * (a * q[4] + B * Syz);
}

// The bond (L1) metric: sum_ij dQ_ij^2 = d^T M d; returns M d.
template <typename T>
__device__ __forceinline__ void metric(const T d[5], T o[5]) {
    o[0] = T(2) * d[0] + d[3];
    o[1] = T(2) * d[1];
    o[2] = T(2) * d[2];
    o[3] = d[0] + T(2) * d[3];
    o[4] = T(2) * d[4];
}

// Same-axis part of L2/L3 along axis j: sum_i dQ_ij^2 (column j of dQ);
// returns its gradient / 2 with respect to d.
template <typename T>
__device__ __forceinline__ void column_metric(int j, const T d[5], T o[5]) {
    if (j == 0) {
        o[0] = d[0]; o[1] = d[1]; o[2] = d[2]; o[3] = T(0); o[4] = T(0);
    } else if (j == 1) {
        o[0] = T(0); o[1] = d[1]; o[2] = T(0); o[3] = d[3]; o[4] = d[4];
    } else {
        T s = d[0] + d[3];
        o[0] = s; o[1] = T(0); o[2] = d[2]; o[3] = s; o[4] = d[4];
    }
}

// h_j = P^T H_j with H_j,ab = sum_{k != j} [L2 delta_bj C_k,ak + L3 delta_bk C_k,aj]:
// the derivative of the cross-axis L2/L3 energy of one site with respect to
// its mean difference C_j, mapped to q components.
template <typename T>
__device__ __forceinline__ void cross_h(int j, const T Ck[3][5], T L2, T L3, T h[5]) {
    T H[3][3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) H[a][b] = T(0);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        if (k == j) continue;
        T C[3][3];
        full_of(Ck[k], C);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            H[a][j] += L2 * C[a][k];
            H[a][k] += L3 * C[a][j];
        }
    }
    pT(H, h);
}

// Levi-Civita symbol
__host__ __device__ constexpr int eps3(int a, int b, int c) { return ((a - b) * (b - c) * (c - a)) / 2; }

// Chiral term (L4) of Eq. (fdistortionFull), E4(x) = L4/2 eps_lik Q_lj(x) C_k,ij(x).
// Its derivative with respect to the site tensor: P^T of sum_ik eps_aik C_k,ib.
template <typename T>
__device__ __forceinline__ void chiral_site(const T C[3][5], T h[5]) {
    T H[3][3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) H[a][b] = T(0);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        T Ck[3][3];
        full_of(C[k], Ck);
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                if (eps3(a, i, k) == 0) continue;
#pragma unroll
                for (int b = 0; b < 3; ++b) H[a][b] += T(eps3(a, i, k)) * Ck[i][b];
            }
    }
    pT(H, h);
}

// Derivative of E4(x) with respect to the tensor of a site that enters C_k(x)
// with coefficient 1: P^T of sum_l eps_lak Q_lb(x).
template <typename T>
__device__ __forceinline__ void chiral_nb(int k, const T qx[5], T h[5]) {
    T Qx[3][3], H[3][3];
    full_of(qx, Qx);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            T v = T(0);
#pragma unroll
            for (int l = 0; l < 3; ++l)
                if (eps3(l, a, k) != 0) v += T(eps3(l, a, k)) * Qx[l][b];
            H[a][b] = v;
        }
    pT(H, h);
}

// ---------------------------------------------------------------------------
// The force reads its neighbourhood through a stencil view P: P.at(dx, dy, dz,
// c) and P.mask(dx, dy, dz) at offsets in {-1, 0, 1} around the centre (the
// views of the two families of kernels are defined beside them).
__device__ __forceinline__ void unit(int k, int s, int& dx, int& dy, int& dz) {
    dx = k == 0 ? s : 0;
    dy = k == 1 ? s : 0;
    dz = k == 2 ? s : 0;
}

// The FP32 L2/L3 kernels evaluate boundary sites branch-free: every stencil
// position holds a finite value (0 where no simulated site is), so a term
// whose coefficient is 0 adds exactly nothing, and the LDS reads of all
// terms can be in flight together (the branch per term serialized them on
// LDS latency; measured 33% faster on the 128^3 colloid slab).  In FP64 the
// branch-free form needs more registers than the kernel has and measured
// slower, so the FP64 kernels read only the terms that are present.
template <typename T>
constexpr bool branch_free() { return sizeof(T) == 4; }

// mean differences C_k (k != skip) at offset o of the stencil
template <typename T, class ST>
__device__ __forceinline__ void mean_diffs(const ST& P, int ox, int oy, int oz,
                                           int skip, uint32_t m, T Ck[3][5]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        if (k == skip) {
#pragma unroll
            for (int c = 0; c < 5; ++c) Ck[k][c] = T(0);
            continue;
        }
        T ap, a0, am;
        mean_diff_coef(m, k, ap, a0, am);
        int ex, ey, ez;
        unit(k, 1, ex, ey, ez);
#pragma unroll
        for (int c = 0; c < 5; ++c) {
            T v = a0 * P.at(ox, oy, oz, c);
            if (branch_free<T>() || ap != T(0)) v = fma_t(ap, P.at(ox + ex, oy + ey, oz + ez, c), v);
            if (branch_free<T>() || am != T(0)) v = fma_t(am, P.at(ox - ex, oy - ey, oz - ez, c), v);
            Ck[k][c] = v;
        }
    }
}

// K (upper triangle) and b of one site's anchoring form
template <typename T>
struct AnchRow {
    T k[15], b[5];
};

// Loads the force's copy of anchoring row arow1 - 1 (zeros for arow1 == 0:
// the offset lies past the end of the buffer).
template <typename T>
__device__ __forceinline__ void anch_load(const LatDev& L, int arow1, AnchRow<T>& A) {
    constexpr uint32_t ROW = ANCH_FSTRIDE * sizeof(T);  // 80 or 160 bytes: whole 16-byte pieces
    const __amdgpu_buffer_rsrc_t r = field_rsrc(L.anch_force, (uint32_t)L.n_anch * ROW);
    const uint32_t off = arow1 > 0 ? (uint32_t)(arow1 - 1) * ROW : 0xFFFFFFFFu;
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef double f64x2 __attribute__((ext_vector_type(2)));
    T v[ANCH_FSTRIDE];
#pragma unroll
    for (int i = 0; i < (int)(ROW / 16); ++i) {
        // whole-vector casts: a bit cast of one subscripted element of the
        // loaded vector is not reliably compiled
        const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, i * 16, 0);
        if constexpr (sizeof(T) == 4) {
            const f32x4 x = __builtin_bit_cast(f32x4, w);
            v[4 * i + 0] = x.x; v[4 * i + 1] = x.y; v[4 * i + 2] = x.z; v[4 * i + 3] = x.w;
        } else {
            const f64x2 x = __builtin_bit_cast(f64x2, w);
            v[2 * i + 0] = x.x; v[2 * i + 1] = x.y;
        }
    }
#pragma unroll
    for (int i = 0; i < 15; ++i) A.k[i] = v[i];
#pragma unroll
    for (int i = 0; i < 5; ++i) A.b[i] = v[15 + i];
}

// -dE/dq at the stencil centre (a simulated site with mask m0).  Where m0
// carries the anchoring bit, the site's anchoring form is AR (wide tiles,
// loaded ahead by the caller) or row arow1 - 1 of the FP64 forms, read here
// (bricks, and narrow tiles, where early loads measure within 2% either way; FP64
// L2/L3: the 40 registers of an early row are what keeps that kernel from two
// waves per SIMD).
template <typename T, bool L23, bool L4, bool BULK, int W, class ST>
__device__ __forceinline__ void site_force(const ST& P, uint32_t m0,
                                           const LatDev& L, const AnchRow<T>& AR, int arow1, T F[5]) {
    const T A = T(L.A), B = T(L.B), C = T(L.C), L1 = T(L.L1);
    T q0[5];
    P.load5(0, 0, 0, q0);
    T g[5];
    bulk_grad(q0, A, B, C, g);
    // external fields: a constant force per simulated site
#pragma unroll
    for (int c = 0; c < 5; ++c) g[c] -= T(L.ext[c]);
    if (BULK) {
        // every bond has weight 1: the L1 term is -L1 M (sum of neighbours - 6 q)
        T S[3][5];  // q(+e_k) + q(-e_k)
#pragma unroll
        for (int c = 0; c < 5; ++c) {
            S[0][c] = P.at(1, 0, 0, c) + P.at(-1, 0, 0, c);
            S[1][c] = P.at(0, 1, 0, c) + P.at(0, -1, 0, c);
            S[2][c] = P.at(0, 0, 1, c) + P.at(0, 0, -1, c);
            F[c] = fma_t(T(-6), q0[c], (S[0][c] + S[1][c]) + S[2][c]);
        }
        T o[5];
        metric(F, o);
#pragma unroll
        for (int c = 0; c < 5; ++c) g[c] = fma_t(-L1, o[c], g[c]);
        if (L23) {
            // In the bulk every mean difference is central and both L2/L3
            // parts depend on L2 + L3 only.  Same-axis part: (L2 + L3) times
            // the sum over axes k of column k of (2 q - S_k).  Cross-axis
            // part: the sum over x = centre -+ e_j of +-1/2 h_j(x) collapses
            // to -1/4 (L2 + L3) sum_{j<k} X_jk, where X_jk = P^T H with
            // H_aj = D_ak, H_ak = D_aj, and D the full tensor of the mixed
            // second difference q(+j+k) - q(+j-k) - q(-j+k) + q(-j-k).
            // Written out, X_xy = (D1, D0 + D3, D4, D1, D2),
            // X_xz = (0, D4, -D3, -D2, D1), X_yz = (-D4, D2, D1, 0, -D0).
            T d[3][5];
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int c = 0; c < 5; ++c) d[k][c] = fma_t(T(2), q0[c], -S[k][c]);
            const T s2 = d[2][0] + d[2][3];
            T col[5];
            col[0] = d[0][0] + s2;
            col[1] = d[0][1] + d[1][1];
            col[2] = d[0][2] + d[2][2];
            col[3] = d[1][3] + s2;
            col[4] = d[1][4] + d[2][4];
            auto mix = [&](int j, int k, int c) {
                int pj[3], pk[3];
                unit(j, 1, pj[0], pj[1], pj[2]);
                unit(k, 1, pk[0], pk[1], pk[2]);
                return (P.at(pj[0] + pk[0], pj[1] + pk[1], pj[2] + pk[2], c) -
                        P.at(pj[0] - pk[0], pj[1] - pk[1], pj[2] - pk[2], c)) -
                       (P.at(pk[0] - pj[0], pk[1] - pj[1], pk[2] - pj[2], c) -
                        P.at(-pj[0] - pk[0], -pj[1] - pk[1], -pj[2] - pk[2], c));
            };
            T X[5];
            X[0] = mix(0, 1, 1) - mix(1, 2, 4);
            X[1] = (mix(0, 1, 0) + mix(0, 1, 3)) + (mix(0, 2, 4) + mix(1, 2, 2));
            X[2] = (mix(0, 1, 4) - mix(0, 2, 3)) + mix(1, 2, 1);
            X[3] = mix(0, 1, 1) - mix(0, 2, 2);
            X[4] = (mix(0, 1, 2) + mix(0, 2, 1)) - mix(1, 2, 0);
            const T L23s = T(L.L2) + T(L.L3);
#pragma unroll
            for (int c = 0; c < 5; ++c) g[c] = fma_t(L23s, fma_t(T(-0.25), X[c], col[c]), g[c]);
        }
    } else {
        // bond sums: L1 and the same-axis part of L2/L3.  Branch-free (FP32
        // L2/L3): an absent bond gets weight 0; the other kernels skip it.
        constexpr bool BF = L23 && branch_free<T>();
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int s = -1; s <= 1; s += 2) {
                if (!BF && !has_nb(m0, k, s)) continue;
                int dx, dy, dz;
                unit(k, s, dx, dy, dz);
                uint32_t mn = P.mask(dx, dy, dz);
                T w = (n_choices(m0, k) == 2 ? T(0.5) : T(1)) + (n_choices(mn, k) == 2 ? T(0.5) : T(1));
                w = has_nb(m0, k, s) ? w : T(0);
                T d[5], o[5];
#pragma unroll
                for (int c = 0; c < 5; ++c) d[c] = q0[c] - P.at(dx, dy, dz, c);
                metric(d, o);
                T wl = w * L1;
#pragma unroll
                for (int c = 0; c < 5; ++c) g[c] = fma_t(wl, o[c], g[c]);
                if (L23) {
                    column_metric(k, d, o);
                    T wl23 = w * (T(L.L2) + T(L.L3));
#pragma unroll
                    for (int c = 0; c < 5; ++c) g[c] = fma_t(wl23, o[c], g[c]);
                }
                // one bond's reads at a time in flight: hoisting every
                // stencil read of the branch-free form spills registers
                if (BF) __builtin_amdgcn_sched_barrier(0);
            }
    }
    if (L23 && !BULK) {
        const T L2 = T(L.L2), L3 = T(L.L3);
        // cross-axis part: every site x whose mean difference C_j contains
        // Q(centre).  The branch per site x also keeps the branch-free form
        // to one mean-difference evaluation's reads in flight at a time
        // (without it every read of all seven is hoisted and registers spill).
#pragma unroll
        for (int j = 0; j < 3; ++j) {
#pragma unroll
            for (int s = -1; s <= 1; s += 2) {
                // x = centre - s e_j uses Q(centre) with coefficient a_{j,s}(x)
                int dx, dy, dz;
                unit(j, -s, dx, dy, dz);
                uint32_t mx = P.mask(dx, dy, dz);
                T ap, a0, am;
                mean_diff_coef(mx, j, ap, a0, am);
                const T coef = s > 0 ? ap : am;
                if (coef == T(0)) continue;
                T Ck[3][5], h[5];
                mean_diffs(P, dx, dy, dz, j, mx, Ck);
                cross_h(j, Ck, L2, L3, h);
#pragma unroll
                for (int c = 0; c < 5; ++c) g[c] = fma_t(coef, h[c], g[c]);
            }
            T ap, a0, am;
            mean_diff_coef(m0, j, ap, a0, am);
            if (a0 != T(0)) {
                T Ck[3][5], h[5];
                mean_diffs(P, 0, 0, 0, j, m0, Ck);
                cross_h(j, Ck, L2, L3, h);
#pragma unroll
                for (int c = 0; c < 5; ++c) g[c] = fma_t(a0, h[c], g[c]);
            }
        }
    }
    if (L4) {
        if (L.L4 != 0.0) {
            // chiral term: the site's own tensor, then every C_k(x) holding Q(centre)
            const T hL4 = T(0.5 * L.L4);
            T Cc[3][5], h[5];
            mean_diffs(P, 0, 0, 0, -1, m0, Cc);
            chiral_site(Cc, h);
#pragma unroll
            for (int c = 0; c < 5; ++c) g[c] = fma_t(hL4, h[c], g[c]);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
#pragma unroll
                for (int s = -1; s <= 1; s += 2) {
                    int dx, dy, dz;
                    unit(k, -s, dx, dy, dz);
                    T ap, a0, am;
                    mean_diff_coef(P.mask(dx, dy, dz), k, ap, a0, am);
                    const T coef = s > 0 ? ap : am;
                    if (coef == T(0)) continue;
                    T qx[5];
                    P.load5(dx, dy, dz, qx);
                    chiral_nb(k, qx, h);
#pragma unroll
                    for (int c = 0; c < 5; ++c) g[c] = fma_t(hL4 * coef, h[c], g[c]);
                }
                T ap, a0, am;
                mean_diff_coef(m0, k, ap, a0, am);
                if (a0 != T(0)) {
                    chiral_nb(k, q0, h);
#pragma unroll
                    for (int c = 0; c < 5; ++c) g[c] = fma_t(hL4 * a0, h[c], g[c]);
                }
            }
        }
    }
    // d/dq of 1/2 q^T K q + b^T q = K q + b, K from its upper triangle
    if (!BULK && W == 1 && !(L23 && sizeof(T) == 8) && (m0 & M_ANCH)) {
        T Kq[5];
#pragma unroll
        for (int a = 0; a < 5; ++a) Kq[a] = AR.b[a];
        int t = 0;
#pragma unroll
        for (int a = 0; a < 5; ++a)
#pragma unroll
            for (int b = a; b < 5; ++b, ++t) {
                const T k = AR.k[t];
                Kq[a] = fma_t(k, q0[b], Kq[a]);
                if (b != a) Kq[b] = fma_t(k, q0[a], Kq[b]);
            }
#pragma unroll
        for (int c = 0; c < 5; ++c) g[c] += Kq[c];
    }
    if (!BULK && (W == 0 || (L23 && sizeof(T) == 8)) && (m0 & M_ANCH)) {
        // the row of the FP64 form, read here
        const int at = arow1 - 1;
        if (at >= 0) {
            const double* d = L.anch_data + ANCH_STRIDE * (int64_t)at;
            T Kq[5];
#pragma unroll
            for (int a = 0; a < 5; ++a) Kq[a] = T(d[15 + a]);
            int t = 0;
#pragma unroll
            for (int a = 0; a < 5; ++a)
#pragma unroll
                for (int b = a; b < 5; ++b, ++t) {
                    const T k = T(d[t]);
                    Kq[a] = fma_t(k, q0[b], Kq[a]);
                    if (b != a) Kq[b] = fma_t(k, q0[a], Kq[b]);
                }
#pragma unroll
            for (int c = 0; c < 5; ++c) g[c] += Kq[c];
        }
    }
#pragma unroll
    for (int c = 0; c < 5; ++c) F[c] = -g[c];
}

// ---------------------------------------------------------------------------
// Wave reductions over data-parallel primitives: within rows of 16 lanes by
// shifts, then across the four rows by broadcasts of each row's last lane, so
// that lane 63 holds the result (a lane that a move leaves out adds the
// identity 0; maxima are of non-negative values).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_move(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROWS, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, ROWS, 0xf, true);
    return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
}
// result in lane 63
__device__ __forceinline__ double wave_sum(double v) {
    v += dpp_move<0x111, 0xf>(v);  // row_shr:1
    v += dpp_move<0x112, 0xf>(v);  // row_shr:2
    v += dpp_move<0x114, 0xf>(v);  // row_shr:4
    v += dpp_move<0x118, 0xf>(v);  // row_shr:8
    v += dpp_move<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
    v += dpp_move<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
    return v;
}
__device__ __forceinline__ double wave_max(double v) {
    v = fmax(v, dpp_move<0x111, 0xf>(v));
    v = fmax(v, dpp_move<0x112, 0xf>(v));
    v = fmax(v, dpp_move<0x114, 0xf>(v));
    v = fmax(v, dpp_move<0x118, 0xf>(v));
    v = fmax(v, dpp_move<0x142, 0xa>(v));
    v = fmax(v, dpp_move<0x143, 0xc>(v));
    return v;
}

// Block reduction of 4 values in a fixed order: 3 sums and a max
// (LAST_MAX, the step partials), or 4 sums (the energy terms).  LDS_ONLY: the
// block's global loads and stores stay in flight across it.
template <bool LAST_MAX = true, bool LDS_ONLY = false>
__device__ __forceinline__ void block_reduce4(double r[4], double (*scratch)[4]) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    double a = wave_sum(r[0]), b = wave_sum(r[1]), c = wave_sum(r[2]);
    double d = LAST_MAX ? wave_max(r[3]) : wave_sum(r[3]);
    if (lane == 63) {
        scratch[wv][0] = a; scratch[wv][1] = b; scratch[wv][2] = c; scratch[wv][3] = d;
    }
    if (LDS_ONLY) lds_barrier();
    else __syncthreads();
    if (threadIdx.x == 0) {
        const int nw = (blockDim.x + 63) >> 6;
        double s0 = 0, s1 = 0, s2 = 0, s3 = 0;
        for (int w = 0; w < nw; ++w) {
            s0 += scratch[w][0]; s1 += scratch[w][1]; s2 += scratch[w][2];
            s3 = LAST_MAX ? fmax(s3, scratch[w][3]) : s3 + scratch[w][3];
        }
        r[0] = s0; r[1] = s1; r[2] = s2; r[3] = s3;
    }
}

// FIRE controller (Algorithm 1), run by one thread after the grid reduction.
// Steering and restart decided here are applied to v by the next step kernel
// (or by the finalize kernel) as v <- c_v v + c_F F.
__device__ inline void fire_control(FireDev* st, double P, double nF2, double nv2, double maxF) {
    st->P = P; st->nF2 = nF2; st->nv2 = nv2; st->maxF = maxF;
    if (st->init_pending) {
        st->init_pending = 0;
        if (!(isfinite(nF2) && isfinite(nv2) && isfinite(maxF))) {
            st->status = LQ_NONFINITE; st->done = 1;
        } else if (maxF < st->tol) {
            st->status = LQ_CONVERGED; st->done = 1;
        } else if (st->step >= st->max_steps) {
            st->status = LQ_MAX_STEPS; st->done = 1;
        }
        return;
    }
    st->step += 1;
    st->cur = 1 - st->cur;
    if (!(isfinite(P) && isfinite(nF2) && isfinite(nv2) && isfinite(maxF))) {
        st->status = LQ_NONFINITE;
        st->done = 1;
        st->c_v = 1.0; st->c_F = 0.0;
        return;
    }
    if (st->method != LQ_METHOD_FIRE) {
        // gradient descent and Nesterov: fixed dt and momentum, no steering
    } else if (P > 0.0) {
        double nF = sqrt(nF2), nv = sqrt(nv2);
        st->c_v = 1.0 - st->alpha;
        st->c_F = st->alpha * nv / nF;
        st->n_pos += 1;
        if (st->n_pos > st->n_min) {
            st->dt = fmin(st->dt * st->f_inc, st->dt_max);
            st->alpha = st->alpha * st->f_alpha;
        }
    } else {
        st->c_v = 0.0; st->c_F = 0.0;
        st->dt = st->dt * st->f_dec;
        st->alpha = st->alpha0;
        st->n_pos = 0;
        st->restarts += 1;
    }
    if (maxF < st->tol) {
        st->status = LQ_CONVERGED; st->done = 1;
    } else if (st->step >= st->max_steps) {
        st->status = LQ_MAX_STEPS; st->done = 1;
    } else if (st->step >= st->stop_at) {
        st->done = 1;
    }
}

// Sums the partials of nblocks blocks in block order (every block of a
// kernel that calls this gets the same sums: they depend on the block size
// and nblocks only); the first `stride` threads read.
__device__ __forceinline__ void sum_partials(const double* partials, int nblocks, double s[4],
                                             double (*scratch)[4], int stride) {
    for (int b = (int)threadIdx.x < stride ? (int)threadIdx.x : nblocks; b < nblocks; b += stride) {
        const double* p = partials + 4 * (int64_t)b;
        s[0] += p[0]; s[1] += p[1]; s[2] += p[2]; s[3] = fmax(s[3], p[3]);
    }
    __syncthreads();
    block_reduce4(s, scratch);
}


// After the k_steps step kernels of a call: the controller on the last
// step's reduction (the same sums, in the same order, as in a step kernel
// of NT threads; its first `stride` threads sum), or the state the run
// stopped with, into st[0].  Every wave reads the stop word, so it stays as it
// is here: the start of the next call clears it.
template <int NT>
__device__ __forceinline__ void dc_final(FireDev* st, const double* partials, int nblocks, int k_steps,
                                         double (*scratch)[4], int stride = NT) {
    DcCtl* ctl = (DcCtl*)(st + 2);
    if (ctl->halt) {
        if (threadIdx.x == 0) {
            const int sl = ctl->slot;
            if (sl != 0) st[0] = st[sl];
        }
        return;
    }
    if (k_steps <= 0) return;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    sum_partials(partials + 4 * (int64_t)(k_steps & 1) * nblocks, nblocks, s, scratch, stride);
    if (threadIdx.x == 0) {
        FireDev c = st[k_steps >= 2 ? ((k_steps - 1) & 1) : 0];
        fire_control(&c, s[0], s[1], s[2], s[3]);
        st[0] = c;
    }
}

// Blocks are dispatched round-robin over the 8 XCDs: XCD x runs the blocks
// x, x + 8, ...  They take the x-th contiguous share of the work (the first
// nblocks % 8 shares one longer), so that neighbouring tiles share an L2.
__device__ __forceinline__ int xcd_block(int block, int nblocks) {
    const int x = block & 7, q = nblocks >> 3, r = nblocks & 7;
    return x * q + (x < r ? x : r) + (block >> 3);
}

// The member m of a batch with off[m] <= b < off[m + 1] (off[0] = 0): every
// wave compares 64 offsets at a time, one memory latency for up to 64 members.
__device__ __forceinline__ int member_of(const int* __restrict__ off, int n, int b) {
    int m = -1;
    for (int i = 0; i < n; i += 64) {
        const int lane = i + (int)(threadIdx.x & 63);
        const bool le = lane < n && off[lane] <= b;
        m += __builtin_popcountll(__builtin_amdgcn_ballot_w64(le));
    }
    return m;
}

}  // namespace lq
