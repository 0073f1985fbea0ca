// HIP kernels of liblqfire for gfx950: the discrete Landau-de Gennes force,
// the fused force + FIRE step, the FIRE controller, the energy and helpers.
//
// The energy is the paper's discretization (sec. III.B): bulk Eq. (fphase),
// distortion Eq. (fdistortionFull) (L6 = 0) from one-sided differences
// Eq. (onesidedderivatives) averaged over every allowed forward/backward
// choice per axis, plus anchoring (sec. II.A.4) and external fields
// (sec. II.A.3).  Because the choices on different axes are independent, the
// average factorizes:
//   - products of differences along one axis k average to the mean over the
//     allowed choices of that axis, which turns the L1 term and the same-axis
//     part of L2/L3 into bond sums, bond (x, x+e_k) weighted
//     w = 1/n_k(x) + 1/n_k(x+e_k) with n_k the number of allowed choices;
//   - products of differences along two different axes j != k average to
//     C_j C_k, with C_k the mean of the allowed one-sided differences of
//     axis k (a central difference in the bulk).
// The forces are the exact negative gradient of that energy with respect to
// the five components q (sec. III.B), i.e. P^T applied to dE/dQ where
// P^T G = (Gxx - Gzz, Gxy + Gyx, Gxz + Gzx, Gyy - Gzz, Gyz + Gzy).
//
// FIRE (Algorithm 1) is fused with the force: the kernel of step t reads
// q, v, F of step t-1 with the steering coefficients (c_v, c_F) and dt
// decided by the controller of step t-1, applies steering, the first half
// kick and the drift to every site it needs (its tile plus a one-site halo,
// recomputed in LDS), evaluates the force at the new positions, applies the
// second half kick and writes q, v, F to the other buffer.  Per-block FP64
// partial sums of F.v, |F|^2, |v|^2 and max|F_i| are combined at the start of
// the next step kernel, every block of which runs the controller.  The host
// never waits between steps.  The same march runs gradient descent and
// Nesterov's accelerated gradient (a compile-time mode) and the force alone.
// Further kernels: the energy (FP64 per-term sums), the uniaxial initial
// state, the FIRE bookkeeping, batched steps over many lattices, and the
// director / defect extraction.
//
// Layout: SoA fields [5][nz][ny][nx].  A block owns an X x Y column tile and
// marches zc planes along z, keeping the drifted q of four planes with their
// halo in LDS: the force of plane f reads planes f-1, f, f+1 while plane f+1
// is being written, so that one barrier per plane suffices.
// This header holds the kernels' templates; march_f32.hip and march_f64.hip
// instantiate them for one element type each.
#pragma once

#include <hip/hip_runtime.h>

#include "lq_internal.h"
#include "lq_site.h"

namespace lq {

// ---------------------------------------------------------------------------
// Stencil view used by the force: offsets (dx, dy, dz) in {-1, 0, 1} around
// the centre, read from the LDS slots of the planes below, at and above the
// centre.  BULK: every site of the padded tile is simulated with all six
// neighbours, so masks are compile-time constants.
template <typename T, bool L23, bool BULK, int W>
struct Stencil {
    T (*q)[5][Tile<T, L23, W>::PY][Tile<T, L23, W>::PX];
    uint8_t (*m)[Tile<T, L23, W>::PY][Tile<T, L23, W>::PX];
    int s[3];  // LDS slots of the planes below, at and above the centre
    int cx, cy;
    __device__ __forceinline__ T at(int dx, int dy, int dz, int c) const {
        return q[s[dz + 1]][c][cy + dy][cx + dx];
    }
    __device__ __forceinline__ uint32_t mask(int dx, int dy, int dz) const {
        if (BULK) return (uint32_t)M_FULL;
        return (uint32_t)m[s[dz + 1]][cy + dy][cx + dx];
    }
    __device__ __forceinline__ void load5(int dx, int dy, int dz, T o[5]) const {
#pragma unroll
        for (int c = 0; c < 5; ++c) o[c] = at(dx, dy, dz, c);
    }
};

// ---------------------------------------------------------------------------
// The z-marching kernel.  MODE_FORCE: F = force(q) only.  MODE_FIRE,
// MODE_GD, MODE_NAG: one fused minimizer step between the two buffers of b:
//   FIRE      v1 = c_v v + c_F F + dt/2 F, q' = q + dt v1, F' = F(q'),
//             v' = v1 + dt/2 F'   (Algorithm 1, steering of the previous step
//             applied first);
//   GD        q' = q + dt F, F' = F(q');
//   Nesterov  m' = mu m + dt F, q' = q + m', F' = F(q' + mu m')  (m in the
//             v buffers; the stencil holds the look-ahead point q' + mu m').
//
// A block owns an X x Y column tile and the planes z0 .. z0+zc-1.  Plane i
// of the march (global z = z0 - 1 + i, i = 0 .. zc+1) is loaded into
// registers (the block's own sites, plus the one-site ring around the tile
// spread over all threads one (site, component) pair at a time), then drifted
// (steering, first half kick, q += dt v) into an LDS slot.  Loads run one
// plane ahead of the drift, so the loads of plane i+1 are in flight while the
// force of plane i-1 is evaluated.  Steps march upwards and downwards in turn
// (`down`, by the parity of the step count): the planes that one step wrote
// last are the first that the next one reads, while the Infinity Cache still
// holds them.  That pays where the state is stored with the default policy (us
// per step, FP32 L2/L3 201x163x95 slab 145.7 -> 134.3, 256^3 437 -> 426;
// one-constant 230x187x141 FP32 198 -> 181, FP64 371 -> 361) and is neutral
// with the non-temporal one.  Upwards always march the FP64 L4 kernels
// (201x163x95 with a colloid 358, in turn 363) and, where the cache holds the
// state, the L2/L3 kernels of narrow tiles, which lose to the choice itself (TURN:
// a kernel has it; FP32 3x64x4000 297, in turn 316, 5x400x200 130 and 139; FP64
// 60x132x132 with a sphere 148 and 151).  Beyond the cache those march in turn too
// (FP64 50x250x250 211, upwards 221; FP32 34x300x300 139 and 147), as do wide tiles
// on either side of its size (FP32 L2/L3 128^3 slab 63 us a step, 78 upwards).
template <typename T, bool L23, int W>
__device__ __forceinline__ void ring_pos(int r, int& px, int& py) {
    constexpr int PX = Tile<T, L23, W>::PX, PY = Tile<T, L23, W>::PY;
    if (r < PX) { px = r; py = 0; }
    else if (r < 2 * PX) { px = r - PX; py = PY - 1; }
    else if (r < 2 * PX + PY - 2) { px = 0; py = r - 2 * PX + 1; }
    else { px = PX - 1; py = r - 2 * PX - (PY - 2) + 1; }
}

// Positions of a tile that hangs over the box's edge: the FP64 step kernels with
// L4 load nothing there (SKIP; 101x90x67 74.7 -> 71.9 us per step), the others
// a wrapped site (FP32 one-constant 230x187x141 202 us, 218 without; FP32 L2/L3
// and the force alone 2-3% faster too; FP32 with L4, FIRE and gradient descent:
// 201x163x95 172 and 121, 181 and 136 without; 24x400x400 290, 318 without).
template <bool SKIP>
__device__ __forceinline__ int wrapt(int g, int n, int per) { return SKIP ? wrap1(g, n, per) : wrapc(g, n, per); }

// Plane f (1-based within the march) of a chunk takes the bulk evaluation.
__device__ __forceinline__ bool bulk_plane_of(const PlaneBits& b, int f) {
    const int i = f - 1;
    if (i < 0 || i >= CHUNK_MAX) return false;
    const uint64_t w = i < 64 ? b.w[0] : (i < 128 ? b.w[1] : (i < 192 ? b.w[2] : b.w[3]));
    return (w >> (i & 63)) & 1u;
}

#ifndef LQ_PREFETCH
#define LQ_PREFETCH 1
#endif
static_assert(LQ_PREFETCH == 1 || LQ_PREFETCH == 2, "prefetch depth is 1 or 2 planes");

template <typename T, bool L23, bool L4, int MODE, bool BULK, int W, bool ROWS>
__device__ __forceinline__ void march(const LatDev& L, const T* __restrict__ q_in,
                                      const T* __restrict__ v_in, const T* __restrict__ F_in,
                                      T* __restrict__ q_out, T* __restrict__ v_out,
                                      T* __restrict__ F_out, T cv, T cF, T dt, T hdt, int x0, int y0,
                                      int z0, int zc, bool down, T (*sq)[5][Tile<T, L23, W>::PY][Tile<T, L23, W>::PX],
                                      uint8_t (*sm)[Tile<T, L23, W>::PY][Tile<T, L23, W>::PX], double red[4],
                                      const PlaneBits plane_bulk) {
    using G = Tile<T, L23, W>;
    constexpr int NS = 4;
    constexpr int PF = LQ_PREFETCH;  // planes of raw data in flight
    constexpr int TX = G::X, NTHREADS = G::N, RING = G::RING;
    constexpr int RING_ITEMS = G::RING_ITEMS, ITEMS_PER_THREAD = G::IPT;
    constexpr bool STEP = MODE != MODE_FORCE;
    constexpr bool USES_V = MODE == MODE_FIRE || MODE == MODE_NAG;
    constexpr bool ZERO_SOLID = !BULK && L23 && branch_free<T>();
    constexpr bool SKIP = L4 && STEP && sizeof(T) == 8;
    const int64_t N = L.N;
    const int nxy = L.nx * L.ny;
    const int tx = threadIdx.x % TX, ty = threadIdx.x / TX;
    const int gx = x0 + tx, gy = y0 + ty;
    const bool own_xy = gx < L.nx && gy < L.ny;
    int sxy_own;
    {
        const int wx = wrapt<SKIP>(gx, L.nx, L.per[0]), wy = wrapt<SKIP>(gy, L.ny, L.per[1]);
        sxy_own = (wx >= 0 && wy >= 0) ? wx + L.nx * wy : -1;
    }
    // ring items of this thread
    int it_c[ITEMS_PER_THREAD], it_px[ITEMS_PER_THREAD], it_py[ITEMS_PER_THREAD], it_sxy[ITEMS_PER_THREAD];
#pragma unroll
    for (int j = 0; j < ITEMS_PER_THREAD; ++j) {
        const int k = threadIdx.x + j * NTHREADS;
        it_c[j] = -1; it_px[j] = 0; it_py[j] = 0; it_sxy[j] = -1;
        if (k < RING_ITEMS) {
            it_c[j] = k / RING;
            ring_pos<T, L23, W>(k % RING, it_px[j], it_py[j]);
            const int wx = wrapt<SKIP>(x0 - 1 + it_px[j], L.nx, L.per[0]);
            const int wy = wrapt<SKIP>(y0 - 1 + it_py[j], L.ny, L.per[1]);
            it_sxy[j] = (wx >= 0 && wy >= 0) ? wx + L.nx * wy : -1;
        }
    }
    // raw data of a plane still to drift (PF planes are in flight)
    struct Raw {
        T q[5], v[5], f[5];
        T iq[ITEMS_PER_THREAD], iv[ITEMS_PER_THREAD], iF[ITEMS_PER_THREAD];
        uint32_t m, im[ITEMS_PER_THREAD];
    };

    const uint32_t cs = (uint32_t)N * (uint32_t)sizeof(T);  // bytes per component
    const uint32_t fb = 5u * cs;                               // bytes per field
    const __amdgpu_buffer_rsrc_t rq_in = field_rsrc(q_in, fb);
    const __amdgpu_buffer_rsrc_t rv_in = field_rsrc(USES_V ? v_in : q_in, fb);
    const __amdgpu_buffer_rsrc_t rF_in = field_rsrc(STEP ? F_in : q_in, fb);
    const __amdgpu_buffer_rsrc_t rq_out = field_rsrc(STEP ? q_out : F_out, fb);
    const __amdgpu_buffer_rsrc_t rv_out = field_rsrc(USES_V ? v_out : F_out, fb);
    const __amdgpu_buffer_rsrc_t rF_out = field_rsrc(F_out, fb);
    const __amdgpu_buffer_rsrc_t rmask = field_rsrc(L.mask, (uint32_t)N);
    constexpr uint32_t NONE = 0xFFFFFFFFu;  // past every resource: loads give 0, stores drop
    // global z of plane i of the march (1 .. zc: the chunk's planes)
    auto z_of = [&](int i) { return down ? z0 + zc - i : z0 - 1 + i; };
    // Branch-free loads: an invalid position gets an offset past the end of the
    // buffer instead of a branch, so the wait counts stay exact and the stores
    // of the previous plane can drain while this plane is drifted.
    auto load = [&](int i, Raw& R) {
        const int wz = (i >= 0 && i <= zc + 1) ? wrapc(z_of(i), L.nz, L.per[2]) : -1;
        const bool ok = sxy_own >= 0 && wz >= 0;
        const uint32_t site = (uint32_t)(sxy_own + nxy * wz);
        const uint32_t off = ok ? site * (uint32_t)sizeof(T) : NONE;
#pragma unroll
        for (int c = 0; c < 5; ++c) {
            R.q[c] = bld<T>(rq_in, off, c * cs);
            if (USES_V) R.v[c] = bld<T>(rv_in, off, c * cs);
            if (STEP) R.f[c] = bld<T>(rF_in, off, c * cs);
        }
        if (!BULK) R.m = __builtin_amdgcn_raw_buffer_load_b8(rmask, (int)(ok ? site : NONE), 0, 0);
#pragma unroll
        for (int j = 0; j < ITEMS_PER_THREAD; ++j) {
            const bool okj = it_sxy[j] >= 0 && wz >= 0;
            const uint32_t t = (uint32_t)(it_sxy[j] + nxy * wz);
            const uint32_t offj = okj ? ((uint32_t)it_c[j] * (uint32_t)N + t) * (uint32_t)sizeof(T) : NONE;
            R.iq[j] = bld<T>(rq_in, offj, 0u);
            if (USES_V) R.iv[j] = bld<T>(rv_in, offj, 0u);
            if (STEP) R.iF[j] = bld<T>(rF_in, offj, 0u);
            // the branch-free kernels zero the sites that are not simulated,
            // so they need the mask of every ring item
            if (!BULK) R.im[j] = __builtin_amdgcn_raw_buffer_load_b8(rmask, (int)(okj && (ZERO_SOLID || it_c[j] == 0) ? t : NONE), 0, 0);
        }
    };
    // drift the registers into LDS slot; returns the own site's q' and v1
    // (FIRE: v after the first half kick; Nesterov: m')
    auto drift = [&](const Raw& R, int slot, T qn[5], T v1[5], uint32_t& m) {
#pragma unroll
        for (int c = 0; c < 5; ++c) {
            T x;
            if (MODE == MODE_FIRE) {
                const T vm = fma_t(cv, R.v[c], cF * R.f[c]);
                v1[c] = fma_t(hdt, R.f[c], vm);
                qn[c] = fma_t(dt, v1[c], R.q[c]);
                x = qn[c];
            } else if (MODE == MODE_GD) {
                qn[c] = fma_t(dt, R.f[c], R.q[c]);
                v1[c] = T(0);
                x = qn[c];
            } else if (MODE == MODE_NAG) {
                v1[c] = fma_t(cv, R.v[c], dt * R.f[c]);
                qn[c] = R.q[c] + v1[c];
                x = fma_t(cv, v1[c], qn[c]);
            } else {
                qn[c] = R.q[c];
                v1[c] = T(0);
                x = qn[c];
            }
            // branch-free kernels: a site that is not simulated holds 0 in
            // LDS, whatever its stored tensor (the force reads it with weight 0)
            if (ZERO_SOLID) x = (R.m & M_SIM) ? x : T(0);
            sq[slot][c][ty + 1][tx + 1] = x;
        }
        m = BULK ? (uint32_t)M_FULL : R.m;
        if (!BULK) sm[slot][ty + 1][tx + 1] = (uint8_t)R.m;
#pragma unroll
        for (int j = 0; j < ITEMS_PER_THREAD; ++j) {
            if (it_c[j] < 0) continue;
            T x = R.iq[j];
            if (MODE == MODE_FIRE) {
                const T vm = fma_t(cv, R.iv[j], cF * R.iF[j]);
                x = fma_t(dt, fma_t(hdt, R.iF[j], vm), x);
            } else if (MODE == MODE_GD) {
                x = fma_t(dt, R.iF[j], x);
            } else if (MODE == MODE_NAG) {
                const T mj = fma_t(cv, R.iv[j], dt * R.iF[j]);
                x = fma_t(cv, mj, x + mj);
            }
            if (ZERO_SOLID) x = (R.im[j] & M_SIM) ? x : T(0);
            sq[slot][it_c[j]][it_py[j]][it_px[j]] = x;
            if (!BULK && it_c[j] == 0) sm[slot][it_py[j]][it_px[j]] = (uint8_t)R.im[j];
        }
    };
    auto slot_of = [](int i) { return (i + NS) & (NS - 1); };
    // plane of the chunk (1-based from its bottom, as the plane flags count)
    auto plane_of = [&](int f) { return down ? zc + 1 - f : f; };

    // Loads run one plane ahead: iteration j drifts plane j (loaded during
    // iteration j-1), issues the loads of plane j+1, and evaluates and stores
    // the force of plane j-1 from the LDS planes j-2 .. j.  Every path into
    // the drift has the same stores queued behind the loads it waits for
    // (the prologue stores to an offset past the end of the buffers, which
    // the hardware drops), so the wait lets those stores drain.  Planes
    // outside 0 .. zc+1 load from out-of-range offsets; forces outside
    // 1 .. zc are stored nowhere.
    // v1 and mask of the own site: `older` is the plane whose force is
    // evaluated in this iteration, `newer` the plane just drifted.
    T v1_older[5], v1_newer[5], q_older[5], q_newer[5];
    uint32_t m_older = 0, m_newer = 0;
    // anchoring row (1 + row, 0: none) of the own site: loaded right after
    // the drift, once the mask is known, so that it has arrived by the time
    // the force of that plane is evaluated in the next iteration
    const __amdgpu_buffer_rsrc_t ranch = field_rsrc(L.anch_index, (uint32_t)N * 4u);
    int a_older = 0, a_newer = 0;
#pragma unroll
    for (int c = 0; c < 5; ++c) { v1_older[c] = T(0); v1_newer[c] = T(0); q_older[c] = T(0); q_newer[c] = T(0); }
    // One iteration of the march: drift plane j from R (loaded PF iterations
    // earlier), reload R with plane j + PF, and evaluate and store the force of
    // plane j - 1 from the LDS planes j - 2 .. j.
    T fmax_abs = T(0);  // max |F| in the field's own type (exact), folded into red[3] at the end
    auto plane = [&](int j, Raw& R) {
        if (!L23) __builtin_amdgcn_s_setprio(0);  // drift and loads at the normal priority
        // anchoring forms of plane j - 1, whose force this iteration
        // evaluates.  Wide tiles issue them first, so that they arrive while
        // plane j is drifted and the block meets at the barrier.  Narrow tiles
        // read the FP64 rows inside the force instead (us per FIRE step with
        // and without: FP32 60x300x300 169.0 and 169.4, L4 262 and 268; FP64 390.6
        // and 389.2).  So do the FP64 L2/L3 kernels (registers; see site_force).
        AnchRow<T> A;
        if (!BULK && W == 1 && !(L23 && sizeof(T) == 8)) {
            const int f = j - 1;
            const bool bulk_plane = bulk_plane_of(plane_bulk, plane_of(f));
            // only waves with an anchored site issue the loads
            if (!bulk_plane && __builtin_amdgcn_ballot_w64((m_newer & M_ANCH) != 0) != 0)
                anch_load(L, (m_newer & M_ANCH) ? a_newer : 0, A);
        }
#pragma unroll
        for (int c = 0; c < 5; ++c) { v1_older[c] = v1_newer[c]; q_older[c] = q_newer[c]; }
        m_older = m_newer;
        a_older = a_newer;
        drift(R, slot_of(j), q_newer, v1_newer, m_newer);
        if (!BULK) {
            const bool anch = own_xy && j >= 1 && j <= zc && (m_newer & M_ANCH);
            const uint32_t sj = (uint32_t)(gx + L.nx * gy + nxy * z_of(j));
            a_newer = (int)__builtin_amdgcn_raw_buffer_load_b32(ranch, (int)(anch ? sj * 4u : NONE), 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        load(j + PF, R);
        __builtin_amdgcn_sched_barrier(0);  // the loads stay ahead of this plane's stores
        lds_barrier();
        // one-constant kernels: waves past the barrier (force and stores) go
        // before waves still drifting, so each plane's stores leave sooner
        // (measured 0.7% on the 256^3 multi-colloid step; not for L2/L3)
        if (!L23) __builtin_amdgcn_s_setprio(1);
        {
            const int f = j - 1;  // plane whose force is evaluated
            const bool in_chunk = f >= 1;
            const int s = gx + L.nx * gy + nxy * z_of(f);
            const uint32_t off = (own_xy && in_chunk) ? (uint32_t)s * (uint32_t)sizeof(T) : NONE;
            const bool live = own_xy && in_chunk && (m_older & M_SIM);
            Stencil<T, L23, BULK, W> P;
            P.q = sq; P.m = sm;
            P.s[0] = slot_of(down ? f + 1 : f - 1); P.s[1] = slot_of(f); P.s[2] = slot_of(down ? f - 1 : f + 1);
            P.cx = tx + 1; P.cy = ty + 1;
            T F[5];
            // a plane whose 3 x 3 x 3 neighbourhoods are all full bulk sites
            // takes the bulk evaluation also inside a boundary tile (wide
            // tiles only.  That was settled when small boxes marched on narrow
            // tiles, few of whose planes qualify.  Boxes that march on them
            // now would gain with L2/L3: with a sphere and two walls 60x300x300
            // takes 241 us a step in FP32 and 866 in FP64, 174 and 420 with the
            // bulk evaluation; one-constant 169 and 389, 174 and 391).  The first two
            // iterations have no plane of the chunk to evaluate (their stores
            // are dropped): the L2/L3 kernels compute no force there (in the
            // one-constant kernels the branch split the loop body and measured
            // 3% slower than the two wasted evaluations).
            if (L23 && !in_chunk) {
#pragma unroll
                for (int c = 0; c < 5; ++c) F[c] = T(0);
            } else if (W == 1 && !BULK && bulk_plane_of(plane_bulk, plane_of(f))) {
                Stencil<T, L23, true, W> PB;
                PB.q = sq; PB.m = sm;
                PB.s[0] = P.s[0]; PB.s[1] = P.s[1]; PB.s[2] = P.s[2];
                PB.cx = P.cx; PB.cy = P.cy;
                site_force<T, L23, L4, true, W>(PB, (uint32_t)M_FULL, L, A, 0, F);
            } else {
                site_force<T, L23, L4, BULK, W>(P, m_older, L, A, a_older, F);
            }
            {
                constexpr int POL = store_policy<T, L23, ROWS>();
#pragma unroll
                for (int c = 0; c < 5; ++c) {
                    const T Fc = live ? F[c] : T(0);
                    if (MODE == MODE_FIRE || MODE == MODE_NAG) {
                        const T v2 = live ? (MODE == MODE_FIRE ? fma_t(hdt, F[c], v1_older[c]) : v1_older[c]) : T(0);
                        const T qc = live ? (MODE == MODE_FIRE ? P.at(0, 0, 0, c) : q_older[c]) : T(0);
                        bst_p<T, POL>(rq_out, off, c * cs, qc);
                        bst_p<T, POL>(rv_out, off, c * cs, v2);
                        bst_p<T, POL>(rF_out, off, c * cs, Fc);
                        const double fd = (double)Fc, vd = (double)v2;
                        red[0] = fma(fd, vd, red[0]);
                        red[1] = fma(fd, fd, red[1]);
                        red[2] = fma(vd, vd, red[2]);
                        fmax_abs = fmax(fmax_abs, fabs(Fc));
                    } else if (MODE == MODE_GD) {
                        const T qc = live ? P.at(0, 0, 0, c) : T(0);
                        bst_p<T, POL>(rq_out, off, c * cs, qc);
                        bst_p<T, POL>(rF_out, off, c * cs, Fc);
                        const double fd = (double)Fc;
                        red[1] = fma(fd, fd, red[1]);
                        fmax_abs = fmax(fmax_abs, fabs(Fc));
                    } else {
                        bst_p<T, POL>(rF_out, off, c * cs, Fc);
                    }
                }
            }
        }
    };
    Raw RA, RB;
    load(0, RA);
    if (PF == 2) load(1, RB);
    __builtin_amdgcn_sched_barrier(0);  // keep the dropped stores behind the loads
#pragma unroll
    for (int c = 0; c < 5; ++c) {
        bst_p<T, 2>(rF_out, NONE, c * cs, T(0));
        if (STEP) bst_p<T, 2>(rq_out, NONE, c * cs, T(0));
        if (USES_V) bst_p<T, 2>(rv_out, NONE, c * cs, T(0));
    }
    __builtin_amdgcn_sched_barrier(0);
    if (PF == 1) {
#pragma clang loop unroll(disable)
        for (int j = 0; j <= zc + 1; ++j) plane(j, RA);
    } else {
#pragma clang loop unroll(disable)
        for (int j = 0; j <= zc + 1; j += 2) {
            plane(j, RA);
            if (j + 1 <= zc + 1) plane(j + 1, RB);
        }
    }
    red[3] = fmax(red[3], (double)fmax_abs);
}

// Start of step kernel k (1-based within a call) of a lattice: the
// controller on the reduction of step k - 1, in every block (the same sums
// in the same order give every block the same result), so that no block
// waits for a last one to finish the previous kernel.  Block 0 keeps the
// new state in st[(k - 1) & 1].  Returns true (every thread) when the run has
// stopped; the step's parameters go to cd (dt, c_v, c_F, mu) and ci (cur with
// the parity of the step count in bit 1, stop; ci[2] takes the stop word).
__device__ bool dc_begin(FireDev* st, const double* partials, int nblocks, int k, int bid,
                         double (*scratch)[4], double* cd, int* ci) {
    DcCtl* ctl = (DcCtl*)(st + 2);
    // one read of the stop word per block: waves that read it apart could see
    // different values while block 0 of this kernel sets it
    if (threadIdx.x == 0) ci[2] = ((volatile const DcCtl*)ctl)->halt;
    __syncthreads();
    if (ci[2]) return true;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    if (k >= 2) sum_partials(partials + 4 * (int64_t)((k - 1) & 1) * nblocks, nblocks, s, scratch, blockDim.x);
    if (threadIdx.x == 0) {
        FireDev c = st[k >= 2 ? (k & 1) : 0];
        if (k >= 2 && !c.done) fire_control(&c, s[0], s[1], s[2], s[3]);
        const int stop = c.done ? 1 : 0;
        if (bid == 0) {
            if (k >= 2) st[(k - 1) & 1] = c;
            if (stop) {
                ctl->slot = k >= 2 ? ((k - 1) & 1) : 0;
                ctl->halt = 1;
            }
        }
        cd[0] = c.dt; cd[1] = c.c_v; cd[2] = c.c_F; cd[3] = c.mu;
        ci[0] = c.cur | (int)(c.step & 1) << 1; ci[1] = stop;
    }
    __syncthreads();
    return ci[1] != 0;
}

// One block of the force / FIRE step: tile `bid` of lattice L.  `nblocks`
// is the lattice's own tile count; partials are indexed by tile, so the
// reduction order does not depend on how blocks are dispatched.  The
// controller of step k - 1 runs at the start (dc_begin); the partials of
// step k go to slot k & 1.  TURN: steps march up and down in turn.  BATCH: the
// kernel serves members of any size, and L4 says only that they may be chiral;
// each marches in the direction that its kernel alone takes, since the order of
// a block's sums follows the march.
template <typename T, bool L23, bool L4, int MODE, int W, bool ROWS, bool TURN, bool BATCH = false>
__device__ __forceinline__ void step_block(const LatDev& L, const Bufs<T>& b, const T* __restrict__ qin,
                                           T* __restrict__ Fout, double* partials, FireDev* st,
                                           int nblocks, int bid, int k) {
    constexpr int NS = 4;
    using G = Tile<T, L23, W>;
    constexpr int PX = G::PX, PY = G::PY;
    __shared__ T sq[NS][5][PY][PX];
    __shared__ uint8_t sm[NS][PY][PX];
    __shared__ double scratch[G::N / 64][4];
    __shared__ double ctl_d[4];
    __shared__ int ctl_i[3];

    constexpr bool STEP = MODE != MODE_FORCE;
    const T *q_in, *v_in = nullptr, *F_in = nullptr;
    T *q_out = nullptr, *v_out = nullptr, *F_out;
    T cv = T(1), cF = T(0), dt = T(0), hdt = T(0);
    bool down = false;
    if (STEP) {
        if (dc_begin(st, partials, nblocks, k, bid, scratch, ctl_d, ctl_i)) return;
        const int cur = ctl_i[0] & 1;
        const bool upwards = !TURN || (L4 && sizeof(T) == 8 && (!BATCH || L.L4 != 0.0)) ||
                             (BATCH && L23 && W == 0 && state_fits_cache<T>(L.N));
        down = !upwards && (ctl_i[0] & 2) != 0;
        const double dtd = ctl_d[0], c_v = ctl_d[1], c_F = ctl_d[2], mu = ctl_d[3];
        // selects rather than indexing by cur, which would put b in scratch
        q_in = cur ? b.q[1] : b.q[0]; v_in = cur ? b.v[1] : b.v[0]; F_in = cur ? b.F[1] : b.F[0];
        q_out = cur ? b.q[0] : b.q[1]; v_out = cur ? b.v[0] : b.v[1]; F_out = cur ? b.F[0] : b.F[1];
        dt = T(dtd); hdt = T(0.5 * dtd);
        if (MODE == MODE_FIRE) { cv = T(c_v); cF = T(c_F); }
        if (MODE == MODE_NAG) cv = T(mu);
    } else {
        q_in = qin;
        F_out = Fout;
    }
    double red[4] = {0.0, 0.0, 0.0, 0.0};
    // the block's chunks one after the other: a packed plan (FP64 L2/L3 only)
    // gives some blocks two; every other plan one per block, chunk bid (the
    // loop costs the other kernels registers)
    constexpr bool PACKED = L23 && sizeof(T) == 8;
    const int i0 = PACKED ? L.first[bid] : bid, i1 = PACKED ? L.first[bid + 1] : bid + 1;
    for (int i = i0; i < i1; ++i) {
        if (i > i0) __syncthreads();  // every wave is done with the LDS planes of the previous chunk
        const Chunk ch = L.chunks[i];
        const int x0 = ch.x0, y0 = ch.y0, z0 = ch.z0, zc = ch.zc;
        if (L.tile_bulk[i]) {
            PlaneBits all;
#pragma unroll
            for (int w = 0; w < PLANE_WORDS; ++w) all.w[w] = ~(uint64_t)0;
            march<T, L23, L4, MODE, true, W, ROWS>(L, q_in, v_in, F_in, q_out, v_out, F_out, cv, cF, dt, hdt, x0, y0, z0,
                                             zc, down, sq, sm, red, all);
        } else {
            march<T, L23, L4, MODE, false, W, ROWS>(L, q_in, v_in, F_in, q_out, v_out, F_out, cv, cF, dt, hdt, x0, y0, z0,
                                              zc, down, sq, sm, red, L.tile_planes[i]);
        }
    }
    if (STEP) {
        block_reduce4(red, scratch);
        if (threadIdx.x == 0) {
            double* p = partials + 4 * ((int64_t)(k & 1) * nblocks + bid);
            p[0] = red[0]; p[1] = red[1]; p[2] = red[2]; p[3] = red[3];
        }
    }
}

// L4: the kernel evaluates the chiral term (a kernel of its own, so that the
// common L2/L3 kernels do not carry its registers).  TWO: held to two waves
// per SIMD (the FP64 L2/L3 kernel for lattices whose one-wave chunks would be
// short; LatDev::two_waves).
template <typename T, bool L23, bool L4, int MODE, int W, bool TWO = false, bool ROWS = true, bool TURN = true>
__global__ __launch_bounds__((Tile<T, L23, W>::N)) __attribute__((amdgpu_waves_per_eu(L4 ? 1 : (TWO ? 2 : Tile<T, L23, W>::WAVES)))) void k_march(LatDev L, Bufs<T> b, const T* __restrict__ qin,
                                                    T* __restrict__ Fout, double* partials,
                                                    FireDev* st, int k) {
    const int nblocks = (int)gridDim.x;
    const int bid = xcd_block((int)blockIdx.x, nblocks);
    step_block<T, L23, L4, MODE, W, ROWS, TURN>(L, b, qin, Fout, partials, st, nblocks, bid, k);
}

// ---------------------------------------------------------------------------
// Batched steps: one launch advances every member of a batch of lattices by
// one FIRE step.  Block b belongs to the member m with off[m] <= b <
// off[m+1]; each member keeps its own controller and partials, so
// its trajectory is bit for bit the one it has alone.
template <typename T, bool L23, int W>
__global__ __launch_bounds__((Tile<T, L23, W>::N)) __attribute__((amdgpu_waves_per_eu(Tile<T, L23, W>::WAVES))) void k_march_batch(const MemberDev* __restrict__ mem,
                                                          const int* __restrict__ off, int n_members, int k) {
    const int m = member_of(off, n_members, (int)blockIdx.x);
    const MemberDev& M = mem[m];
    Bufs<T> b;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        b.q[i] = (T*)M.q[i]; b.v[i] = (T*)M.v[i]; b.F[i] = (T*)M.F[i];
    }
    const LatDev& L = M.L;
    step_block<T, L23, L23, MODE_FIRE, W, true, true, true>(L, b, nullptr, nullptr, M.partials, M.st, M.nblocks,
                                          (int)blockIdx.x - off[m], k);
}

// ---------------------------------------------------------------------------
// launchers of one element type

// Resident blocks per compute unit of the fused FIRE step kernel.
template <typename T, bool L23, bool L4, int W, bool TWO = false>
static int blocks_per_cu() {
    int n = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_march<T, L23, L4, MODE_FIRE, W, TWO>,
                                                                Tile<T, L23, W>::N, 0);
    return e == hipSuccess && n > 0 ? n : 1;
}
template <typename T>
static int blocks_per_cu_t(bool l23, bool l4, int wide) {
    if (!l23) return wide ? blocks_per_cu<T, false, false, 1>() : blocks_per_cu<T, false, false, 0>();
    if (l4) return wide ? blocks_per_cu<T, true, true, 1>() : blocks_per_cu<T, true, true, 0>();
    return wide ? blocks_per_cu<T, true, false, 1>() : blocks_per_cu<T, true, false, 0>();
}
template <typename T, bool L23, bool L4, int MODE, int W, bool TWO, bool ROWS>
static void launch_one(const LatDev& L, const Bufs<T>& b, const void* q, void* F, double* partials, FireDev* st, int k,
                       hipStream_t s) {
    constexpr bool F64 = sizeof(T) == 8;
    const dim3 g((unsigned)n_step_blocks(L));
    // narrow L2/L3 steps within the cache (its FP64 kernels store with ROWS false there)
    if constexpr (L23 && W == 0 && MODE != MODE_FORCE && !(F64 && (L4 || ROWS))) {
        if (state_fits_cache<T>(L.N)) {
            k_march<T, L23, L4, MODE, W, TWO, ROWS, false><<<g, Tile<T, L23, W>::N, 0, s>>>(L, b, (const T*)q, (T*)F,
                                                                                          partials, st, k);
            return;
        }
    }
    k_march<T, L23, L4, MODE, W, TWO, ROWS><<<g, Tile<T, L23, W>::N, 0, s>>>(L, b, (const T*)q, (T*)F, partials, st, k);
}

template <typename T, int MODE, int W>
static void launch_march(const LatDev& L, bool l23, const Bufs<T>& b, const void* q, void* F, double* partials,
                         FireDev* st, int k, hipStream_t s) {
    constexpr bool STEP = MODE != MODE_FORCE, F64 = sizeof(T) == 8;
    // the store policy (store_policy): the force and the FP32 L2/L3/L4 kernels have one
    const bool rows = !STEP || (whole_rows<T>(L.nx) && !state_fits_cache<T>(L.N));
    if (l23 && L.L4 != 0.0) {
        if (rows) launch_one<T, true, true, MODE, W, false, true>(L, b, q, F, partials, st, k, s);
        else launch_one<T, true, true, MODE, W, false, !(F64 && STEP)>(L, b, q, F, partials, st, k, s);
    } else if (l23) {
        if constexpr (F64 && W == 1) {
            if (L.two_waves) {
                if (rows) launch_one<T, true, false, MODE, W, true, true>(L, b, q, F, partials, st, k, s);
                else launch_one<T, true, false, MODE, W, true, !(F64 && STEP)>(L, b, q, F, partials, st, k, s);
                return;
            }
        }
        if (rows) launch_one<T, true, false, MODE, W, false, true>(L, b, q, F, partials, st, k, s);
        else launch_one<T, true, false, MODE, W, false, !(F64 && STEP)>(L, b, q, F, partials, st, k, s);
    } else {
        if (rows) launch_one<T, false, false, MODE, W, false, true>(L, b, q, F, partials, st, k, s);
        else launch_one<T, false, false, MODE, W, false, !STEP>(L, b, q, F, partials, st, k, s);
    }
}

template <typename T, int MODE>
static void launch_march_any(const LatDev& L, bool l23, const Bufs<T>& b, const void* q, void* F, double* partials,
                             FireDev* st, int k, hipStream_t s) {
    if (L.kind == KIND_WIDE) launch_march<T, MODE, 1>(L, l23, b, q, F, partials, st, k, s);
    else launch_march<T, MODE, 0>(L, l23, b, q, F, partials, st, k, s);
}

template <typename T, int W>
static void launch_batch_group(bool l23, const MemberDev* mem, const BatchGroup& g, int k, hipStream_t s) {
    if (g.n <= 0) return;
    if (l23) k_march_batch<T, true, W><<<g.blocks, Tile<T, true, W>::N, 0, s>>>(mem, g.off, g.n, k);
    else k_march_batch<T, false, W><<<g.blocks, Tile<T, false, W>::N, 0, s>>>(mem, g.off, g.n, k);
}

template <typename T>
static void launch_march_mode(const LatDev& L, bool l23, int mode, const void* bufs, const void* q, void* F,
                              double* partials, FireDev* st, int k, hipStream_t s) {
    const Bufs<T> none{};
    const Bufs<T>& b = bufs ? *(const Bufs<T>*)bufs : none;
    if (mode == MODE_FORCE) launch_march_any<T, MODE_FORCE>(L, l23, b, q, F, partials, st, k, s);
    else if (mode == MODE_GD) launch_march_any<T, MODE_GD>(L, l23, b, q, F, partials, st, k, s);
    else if (mode == MODE_NAG) launch_march_any<T, MODE_NAG>(L, l23, b, q, F, partials, st, k, s);
    else launch_march_any<T, MODE_FIRE>(L, l23, b, q, F, partials, st, k, s);
}

}  // namespace lq
