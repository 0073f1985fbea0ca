// Brick kernels: the force, and the fused minimizer steps, of small lattices.
//
// A small box does not fill the GPU, so its step lasts as long as one block's
// chain of dependent waits, not as long as its bytes take.  A marching block
// (march.h) waits for memory once per plane; here a block owns one
// X x Y x Z brick with one thread per site, loads the brick and its one-site
// halo at once (each thread its own site and IPT halo sites), drifts them into
// LDS and evaluates the force after a single barrier.  The controller of the
// step before runs beside those loads; which of the two buffers holds the state
// follows from the parity of the step within the call.
//
// What bounds a step: up to about 32^3 sites one block's chain (launch, loads,
// controller, drift, force, reduction); then the loads, which the Infinity
// Cache serves.  One MI355X, us per FIRE step, marching kernels and bricks:
//   one-constant FP64  32^3 bulk 15.9 and 7.6, with a colloid 20.0 and 8.3
//                      (8.9 and 9.6 with the controller behind the loads);
//                      64^3 29.6 and 17.1
//   one-constant FP32  32^3 16.7 and 7.4; 64^3 21.5 and 12.4; 75x81x93 32.1 and 27.2
//   L2/L3 FP64         32^3 17.8 and 8.0, with a colloid 51.9 and 16.9
// and 20 FP32 boxes of 16 to 64 sites a side in one batch 61 and 36.  Brick
// shapes for 44^3 and 64^3 FP32 one-constant: 8x4x4 11.5 and 22.7, 8x8x4 9.6 and
// 15.8, 16x4x4 10.7 and 17.0, 16x8x4 9.2 and 12.4, 16x8x8 12.6 and 13.6.
#include <hip/hip_runtime.h>

#include "lq_internal.h"
#include "lq_site.h"

namespace lq {

// Lattices of at most this many bricks run the controller in one wave: us per
// step, behind the loads and in one wave, one-constant FP64 32^3 (64 bricks)
// 8.9 and 7.6, 44^3 (198) 10.7 and 9.7, 64^3 (512) 17.4 and 17.5, 80^3 (1000)
// 31.5 and 36.0.
constexpr int WAVE_SUMS = 256;

// The neighbourhood of one site in the brick's padded LDS copy.
template <typename T, bool L23, bool BULK>
struct BrickStencil {
    using G = Brick<L23>;
    T (*q)[G::PZ][G::PY][G::PX];
    uint8_t (*m)[G::PY][G::PX];
    int cx, cy, cz;
    __device__ __forceinline__ T at(int dx, int dy, int dz, int c) const { return q[c][cz + dz][cy + dy][cx + dx]; }
    __device__ __forceinline__ uint32_t mask(int dx, int dy, int dz) const {
        if (BULK) return (uint32_t)M_FULL;
        return (uint32_t)m[cz + dz][cy + dy][cx + dx];
    }
    __device__ __forceinline__ void load5(int dx, int dy, int dz, T o[5]) const {
#pragma unroll
        for (int c = 0; c < 5; ++c) o[c] = at(dx, dy, dz, c);
    }
};

// a / d for a < 2^16 (a lattice's bricks) and magic = floor(2^32 / d) + 1: exact,
// since the error a (magic - 2^32 / d) / 2^32 < 2^-16 stays below 1 / d.
__device__ __forceinline__ int fast_div(int a, uint64_t magic) { return (int)(((uint64_t)(uint32_t)a * magic) >> 32); }

// Padded position of halo site h: the six faces (one-constant kernels, whose
// stencil has no diagonal), or the whole shell of the padded brick.
template <bool L23>
__device__ __forceinline__ void halo_pos(int h, int& px, int& py, int& pz) {
    using G = Brick<L23>;
    if constexpr (L23) {
        constexpr int CAP = G::PX * G::PY, RING = 2 * G::PX + 2 * G::Y;
        if (h < 2 * CAP) {
            pz = h < CAP ? 0 : G::PZ - 1;
            const int r = h < CAP ? h : h - CAP;
            px = r % G::PX; py = r / G::PX;
            return;
        }
        h -= 2 * CAP;
        pz = 1 + h / RING;
        const int r = h % RING;
        if (r < 2 * G::PX) {
            px = r % G::PX; py = r < G::PX ? 0 : G::PY - 1;
        } else {
            px = (r & 1) ? G::PX - 1 : 0; py = 1 + ((r - 2 * G::PX) >> 1);
        }
    } else {
        constexpr int FZ = G::X * G::Y, FY = G::X * G::Z;
        if (h < 2 * FZ) {
            pz = h < FZ ? 0 : G::PZ - 1;
            const int r = h < FZ ? h : h - FZ;
            px = 1 + r % G::X; py = 1 + r / G::X;
        } else if (h < 2 * FZ + 2 * FY) {
            h -= 2 * FZ;
            py = h < FY ? 0 : G::PY - 1;
            const int r = h < FY ? h : h - FY;
            px = 1 + r % G::X; pz = 1 + r / G::X;
        } else {
            h -= 2 * FZ + 2 * FY;
            px = (h & 1) ? G::PX - 1 : 0;
            const int r = h >> 1;
            py = 1 + r % G::Y; pz = 1 + r / G::Y;
        }
    }
}

template <typename T, bool L23, bool L4, int MODE>
__device__ __forceinline__ void brick_block(const LatDev& L, const Bufs<T>& b, const T* __restrict__ qin,
                                            T* __restrict__ Fout, double* partials, FireDev* st, int nblocks,
                                            int bid, int k) {
    using G = Brick<L23>;
    constexpr int NT = G::N, IPT = G::IPT;
    constexpr bool STEP = MODE != MODE_FORCE;
    constexpr bool USES_V = MODE == MODE_FIRE || MODE == MODE_NAG;
    constexpr bool ZERO_SOLID = L23 && branch_free<T>();
    __shared__ T sq[5][G::PZ][G::PY][G::PX];
    __shared__ uint8_t sm[G::PZ][G::PY][G::PX];
    __shared__ double scratch[NT / 64][4];
    __shared__ struct {
        FireDev st;
        int32_t halt;
    } ctl;
    constexpr int CTL_WORDS = sizeof(FireDev) / 4;
    static_assert(offsetof(DcCtl, halt) == 0 && sizeof(FireDev) % 8 == 0 && CTL_WORDS < 64 && CTL_WORDS < NT, "one word per lane");
    const int tid = threadIdx.x;

    // The controller's reads: the state word by word (lane CTL_WORDS: the stop
    // word) and the partial sums of step k - 1.  Few of them (WAVE_SUMS) the
    // first wave sums and runs the controller on while the other waves issue
    // their loads; many are summed by the whole block, behind those loads.
    const bool wave_ctl = nblocks <= WAVE_SUMS;
    const double* part = partials + 4 * (int64_t)((k - 1) & 1) * nblocks;
    uint32_t word = 0;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    auto add = [&](int i) {
        const double* p = part + 4 * (int64_t)i;
        s[0] += p[0]; s[1] += p[1]; s[2] += p[2]; s[3] = fmax(s[3], p[3]);
    };
    auto control = [&]() {  // one thread
        if (k >= 2 && !ctl.halt && !ctl.st.done) fire_control(&ctl.st, s[0], s[1], s[2], s[3]);
    };
    if (STEP) {
        // one load for all words: st[slot] then the stop word behind st[1]
        if (tid <= CTL_WORDS)
            word = ((const uint32_t*)st)[tid < CTL_WORDS ? (k >= 2 ? (k & 1) : 0) * CTL_WORDS + tid : 2 * CTL_WORDS];
        if (wave_ctl) {
            if (tid < 64) {
                if (k >= 2) {
                    for (int i = tid; i < nblocks; i += 64) add(i);
                    s[0] = wave_sum(s[0]); s[1] = wave_sum(s[1]); s[2] = wave_sum(s[2]); s[3] = wave_max(s[3]);
                }
                if (tid <= CTL_WORDS) ((uint32_t*)&ctl)[tid] = word;
                // lane 63 reads what the lanes of its wave wrote: a compiler
                // fence that no lane's path may be moved across, and a wait
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_wave_barrier();
                if (tid == 63) control();
            }
        } else if (k >= 2 && tid < nblocks) {
            const double* p = part + 4 * (int64_t)tid;
            s[0] = p[0]; s[1] = p[1]; s[2] = p[2]; s[3] = p[3];
        }
        __builtin_amdgcn_sched_barrier(0);
    }

    // brick (bx, by, bz) = bid in x-fastest order
    const int nbx = (L.nx + G::X - 1) / G::X, nby = (L.ny + G::Y - 1) / G::Y;
    const int row = fast_div(bid, L.magic_x), bz = fast_div(bid, L.magic_xy);
    const int x0 = (bid - row * nbx) * G::X, y0 = (row - bz * nby) * G::Y, z0 = bz * G::Z;
    const int64_t N = L.N;
    const uint32_t cs = (uint32_t)N * (uint32_t)sizeof(T);  // bytes per component
    const uint32_t fb = 5u * cs;                               // bytes per field
    const int cur = (k - 1) & 1;  // buffer 0 holds the state when a call starts
    const T* q_in = !STEP ? qin : (cur ? b.q[1] : b.q[0]);
    const T* v_in = cur ? b.v[1] : b.v[0];
    const T* F_in = cur ? b.F[1] : b.F[0];
    T* q_out = cur ? b.q[0] : b.q[1];
    T* v_out = cur ? b.v[0] : b.v[1];
    T* F_out = !STEP ? Fout : (cur ? b.F[0] : b.F[1]);
    const __amdgpu_buffer_rsrc_t rq_in = field_rsrc(q_in, fb);
    const __amdgpu_buffer_rsrc_t rv_in = field_rsrc(USES_V ? v_in : q_in, fb);
    const __amdgpu_buffer_rsrc_t rF_in = field_rsrc(STEP ? F_in : q_in, fb);
    const __amdgpu_buffer_rsrc_t rmask = field_rsrc(L.mask, (uint32_t)N);
    constexpr uint32_t NONE = 0xFFFFFFFFu;  // past every resource: loads give 0, stores drop

    // item 0: the own site; items 1 .. IPT: halo sites
    const int tx = tid % G::X, ty = (tid / G::X) % G::Y, tz = tid / (G::X * G::Y);
    int px[IPT + 1], py[IPT + 1], pz[IPT + 1];
    uint32_t site[IPT + 1];
    bool used[IPT + 1];
    T rq[IPT + 1][5], rv[IPT + 1][5], rf[IPT + 1][5];
    uint32_t rm[IPT + 1];
#pragma unroll
    for (int j = 0; j <= IPT; ++j) {
        const int h = tid + (j - 1) * NT;
        used[j] = j == 0 || h < G::HALO;
        px[j] = tx + 1; py[j] = ty + 1; pz[j] = tz + 1;
        if (j > 0) halo_pos<L23>(used[j] ? h : 0, px[j], py[j], pz[j]);
        const int wx = wrap1(x0 + px[j] - 1, L.nx, L.per[0]), wy = wrap1(y0 + py[j] - 1, L.ny, L.per[1]),
                  wz = wrap1(z0 + pz[j] - 1, L.nz, L.per[2]);
        const bool ok = used[j] && wx >= 0 && wy >= 0 && wz >= 0;
        site[j] = ok ? (uint32_t)(wx + L.nx * (wy + L.ny * wz)) : NONE;
        const uint32_t off = ok ? site[j] * (uint32_t)sizeof(T) : NONE;
#pragma unroll
        for (int cc = 0; cc < 5; ++cc) {
            rq[j][cc] = bld<T>(rq_in, off, cc * cs);
            if (USES_V) rv[j][cc] = bld<T>(rv_in, off, cc * cs);
            if (STEP) rf[j][cc] = bld<T>(rF_in, off, cc * cs);
        }
        rm[j] = __builtin_amdgcn_raw_buffer_load_b8(rmask, (int)site[j], 0, 0);
    }
    // anchoring row of the own site (1 + row, 0: none; no table when nothing is anchored)
    const __amdgpu_buffer_rsrc_t ranch = field_rsrc(L.anch_index, (uint32_t)N * 4u);
    const int arow1 = (int)__builtin_amdgcn_raw_buffer_load_b32(
        ranch, (int)(L.n_anch > 0 && site[0] != NONE ? site[0] * 4u : NONE), 0, 0);
    // the force form of the own plane; a wave lies in one plane of the brick
    static_assert((G::X * G::Y) % 64 == 0, "a wave's sites share a plane");
    const bool bulk = (L.tile_bulk[bid] >> __builtin_amdgcn_readfirstlane(tz)) & 1;
    __builtin_amdgcn_sched_barrier(0);

    T cv = T(1), cF = T(0), dt = T(0), hdt = T(0);
    if (STEP) {
        if (!wave_ctl) {
            if (tid <= CTL_WORDS) ((uint32_t*)&ctl)[tid] = word;
            if (k >= 2) {
                for (int i = tid + NT; i < nblocks; i += NT) add(i);
                block_reduce4<true, true>(s, scratch);
            } else {
                lds_barrier();
            }
            if (tid == 0) control();
        }
        lds_barrier();
        const int halt = ctl.halt, stop = halt || ctl.st.done;
        if (bid == 0 && !halt) {
            // block 0 keeps the new state
            if (k >= 2 && tid < CTL_WORDS) ((uint32_t*)(st + ((k - 1) & 1)))[tid] = ((const uint32_t*)&ctl)[tid];
            if (stop && tid == 0) {
                DcCtl* dc = (DcCtl*)(st + 2);
                dc->slot = k >= 2 ? ((k - 1) & 1) : 0;
                dc->halt = 1;
            }
        }
        if (stop) return;
        const double dtd = ctl.st.dt;
        dt = T(dtd); hdt = T(0.5 * dtd);
        if (MODE == MODE_FIRE) { cv = T(ctl.st.c_v); cF = T(ctl.st.c_F); }
        if (MODE == MODE_NAG) cv = T(ctl.st.mu);
    }

    T v1[5], qn[5];  // own site: v after the first half kick (Nesterov: m'), q'
#pragma unroll
    for (int j = 0; j <= IPT; ++j) {
        if (!used[j]) continue;
#pragma unroll
        for (int cc = 0; cc < 5; ++cc) {
            T x = rq[j][cc], qj = x, vj = T(0);
            if (MODE == MODE_FIRE) {
                vj = fma_t(hdt, rf[j][cc], fma_t(cv, rv[j][cc], cF * rf[j][cc]));
                x = qj = fma_t(dt, vj, x);
            } else if (MODE == MODE_GD) {
                x = qj = fma_t(dt, rf[j][cc], x);
            } else if (MODE == MODE_NAG) {
                vj = fma_t(cv, rv[j][cc], dt * rf[j][cc]);
                qj = x + vj;
                x = fma_t(cv, vj, qj);
            }
            if (j == 0) { v1[cc] = vj; qn[cc] = qj; }
            if (ZERO_SOLID) x = (rm[j] & M_SIM) ? x : T(0);
            sq[cc][pz[j]][py[j]][px[j]] = x;
        }
        sm[pz[j]][py[j]][px[j]] = (uint8_t)rm[j];
    }
    lds_barrier();

    const bool own = x0 + tx < L.nx && y0 + ty < L.ny && z0 + tz < L.nz;
    const bool live = own && (rm[0] & M_SIM);
    double red[4] = {0.0, 0.0, 0.0, 0.0};
    T fmax_abs = T(0);
    // waves that lie past the box's edge have no force to evaluate (L2/L3 FP64
    // 17^3 12.1 -> 7.3 us per step, 50^3 18.2 -> 15.5; the one-constant force is
    // too cheap for the branch, 16^3 7.1 and 7.3)
    if (!L23 || __builtin_amdgcn_ballot_w64(own) != 0) {
        T F[5];
        AnchRow<T> none;
        if (bulk) {
            BrickStencil<T, L23, true> P;
            P.q = sq; P.m = sm; P.cx = tx + 1; P.cy = ty + 1; P.cz = tz + 1;
            site_force<T, L23, L4, true, 0>(P, (uint32_t)M_FULL, L, none, 0, F);
        } else {
            BrickStencil<T, L23, false> P;
            P.q = sq; P.m = sm; P.cx = tx + 1; P.cy = ty + 1; P.cz = tz + 1;
            site_force<T, L23, L4, false, 0>(P, rm[0], L, none, arow1, F);
        }
        const __amdgpu_buffer_rsrc_t rq_out = field_rsrc(STEP ? q_out : F_out, fb);
        const __amdgpu_buffer_rsrc_t rv_out = field_rsrc(USES_V ? v_out : F_out, fb);
        const __amdgpu_buffer_rsrc_t rF_out = field_rsrc(F_out, fb);
        const uint32_t off = own ? site[0] * (uint32_t)sizeof(T) : NONE;
#pragma unroll
        for (int cc = 0; cc < 5; ++cc) {
            const T Fc = live ? F[cc] : T(0);
            bst_p<T, 0>(rF_out, off, cc * cs, Fc);
            if (!STEP) continue;
            bst_p<T, 0>(rq_out, off, cc * cs, live ? qn[cc] : T(0));
            const double fd = (double)Fc;
            red[1] = fma(fd, fd, red[1]);
            fmax_abs = fmax(fmax_abs, fabs(Fc));
            if (USES_V) {
                const T v2 = live ? (MODE == MODE_FIRE ? fma_t(hdt, F[cc], v1[cc]) : v1[cc]) : T(0);
                bst_p<T, 0>(rv_out, off, cc * cs, v2);
                const double vd = (double)v2;
                red[0] = fma(fd, vd, red[0]);
                red[2] = fma(vd, vd, red[2]);
            }
        }
    }
    if (STEP) {
        red[3] = (double)fmax_abs;
        block_reduce4<true, true>(red, scratch);
        if (tid == 0) {
            double* p = partials + 4 * ((int64_t)(k & 1) * nblocks + bid);
            p[0] = red[0]; p[1] = red[1]; p[2] = red[2]; p[3] = red[3];
        }
    }
}

template <typename T, bool L23, bool L4, int MODE>
__global__ __launch_bounds__(Brick<L23>::N) __attribute__((amdgpu_waves_per_eu(!L23 && sizeof(T) == 4 ? 6 : 1))) void k_brick(LatDev L, Bufs<T> b, const T* __restrict__ qin,
                                                        T* __restrict__ Fout, double* partials, FireDev* st,
                                                        int k) {
    brick_block<T, L23, L4, MODE>(L, b, qin, Fout, partials, st, L.nblocks, xcd_block((int)blockIdx.x, L.nblocks), k);
}

// One FIRE step of every member of a batch group: block b of the launch is
// brick b - off[m] of the member m with off[m] <= b < off[m + 1].
template <typename T, bool L23>
__global__ __launch_bounds__(Brick<L23>::N) __attribute__((amdgpu_waves_per_eu(!L23 && sizeof(T) == 4 ? 6 : 1))) void k_brick_batch(const MemberDev* __restrict__ mem,
                                                              const int* __restrict__ off, int n_members, int k) {
    const int blk = xcd_block((int)blockIdx.x, (int)gridDim.x);
    const int m = member_of(off, n_members, blk);
    const MemberDev& M = mem[m];
    Bufs<T> b;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        b.q[i] = (T*)M.q[i]; b.v[i] = (T*)M.v[i]; b.F[i] = (T*)M.F[i];
    }
    brick_block<T, L23, L23, MODE_FIRE>(M.L, b, nullptr, nullptr, M.partials, M.st, M.nblocks, blk - off[m], k);
}

// The controller on a call's last step (dc_final), with the step kernels' sums.
template <int NT>
__device__ __forceinline__ void brick_final(FireDev* st, const double* partials, int nblocks, int k_steps) {
    __shared__ double scratch[NT / 64][4];
    dc_final<NT>(st, partials, nblocks, k_steps, scratch, nblocks <= WAVE_SUMS ? 64 : NT);
}
template <int NT>
__global__ __launch_bounds__(NT) void k_brick_control(FireDev* st, const double* partials, int nblocks, int k_steps) {
    brick_final<NT>(st, partials, nblocks, k_steps);
}
template <int NT>
__global__ __launch_bounds__(NT) void k_brick_batch_control(const MemberDev* __restrict__ mem, int k_steps) {
    const MemberDev& M = mem[blockIdx.x];
    brick_final<NT>(M.st, M.partials, M.nblocks, k_steps);
}

// ---------------------------------------------------------------------------
// launchers
template <typename T, int MODE>
static void launch_brick(const LatDev& L, bool l23, const Bufs<T>& b, const void* q, void* F, double* partials,
                         FireDev* st, int k, hipStream_t s) {
    const dim3 g((unsigned)L.nblocks);
    if (l23 && L.L4 != 0.0)
        k_brick<T, true, true, MODE><<<g, Brick<true>::N, 0, s>>>(L, b, (const T*)q, (T*)F, partials, st, k);
    else if (l23)
        k_brick<T, true, false, MODE><<<g, Brick<true>::N, 0, s>>>(L, b, (const T*)q, (T*)F, partials, st, k);
    else
        k_brick<T, false, false, MODE><<<g, Brick<false>::N, 0, s>>>(L, b, (const T*)q, (T*)F, partials, st, k);
}

void launch_brick_forces(const LatDev& L, bool l23, int prec, const void* q, void* F, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    if (prec == LQ_F64) launch_brick<double, MODE_FORCE>(L, l23, Bufs<double>{}, q, F, nullptr, nullptr, 1, s);
    else launch_brick<float, MODE_FORCE>(L, l23, Bufs<float>{}, q, F, nullptr, nullptr, 1, s);
}

template <int MODE>
static void launch_brick_mode(const LatDev& L, bool l23, int prec, const void* bufs, double* partials, FireDev* st,
                              int k, hipStream_t s) {
    if (prec == LQ_F64)
        launch_brick<double, MODE>(L, l23, *(const Bufs<double>*)bufs, nullptr, nullptr, partials, st, k, s);
    else
        launch_brick<float, MODE>(L, l23, *(const Bufs<float>*)bufs, nullptr, nullptr, partials, st, k, s);
}

void launch_brick_step(const LatDev& L, bool l23, int prec, int method, const void* bufs, double* partials,
                       FireDev* st, int k, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    if (method == LQ_METHOD_GD) launch_brick_mode<MODE_GD>(L, l23, prec, bufs, partials, st, k, s);
    else if (method == LQ_METHOD_NESTEROV) launch_brick_mode<MODE_NAG>(L, l23, prec, bufs, partials, st, k, s);
    else launch_brick_mode<MODE_FIRE>(L, l23, prec, bufs, partials, st, k, s);
}

void launch_brick_control(bool l23, FireDev* st, const double* partials, int nblocks, int k_steps, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    if (l23) k_brick_control<Brick<true>::N><<<1, Brick<true>::N, 0, s>>>(st, partials, nblocks, k_steps);
    else k_brick_control<Brick<false>::N><<<1, Brick<false>::N, 0, s>>>(st, partials, nblocks, k_steps);
}

void launch_brick_batch_control(bool l23, const MemberDev* mem, int n, int k_steps, void* stream) {
    if (n <= 0) return;
    hipStream_t s = (hipStream_t)stream;
    if (l23) k_brick_batch_control<Brick<true>::N><<<n, Brick<true>::N, 0, s>>>(mem, k_steps);
    else k_brick_batch_control<Brick<false>::N><<<n, Brick<false>::N, 0, s>>>(mem, k_steps);
}

void launch_brick_batch(bool l23, int prec, const MemberDev* mem, const int* off, int n, int bricks, int k,
                        void* stream) {
    if (n <= 0) return;
    hipStream_t s = (hipStream_t)stream;
    if (prec == LQ_F64) {
        if (l23) k_brick_batch<double, true><<<bricks, Brick<true>::N, 0, s>>>(mem, off, n, k);
        else k_brick_batch<double, false><<<bricks, Brick<false>::N, 0, s>>>(mem, off, n, k);
    } else {
        if (l23) k_brick_batch<float, true><<<bricks, Brick<true>::N, 0, s>>>(mem, off, n, k);
        else k_brick_batch<float, false><<<bricks, Brick<false>::N, 0, s>>>(mem, off, n, k);
    }
}

}  // namespace lq
