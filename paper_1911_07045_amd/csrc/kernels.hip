// Bookkeeping kernels of the minimizers (initial state and reduction, the final
// controller and state of a call, batches) and the launch sequences of the step
// kernels (march.h, brick.hip).
#include <hip/hip_runtime.h>

#include "lq_internal.h"
#include "lq_site.h"

namespace lq {

template <int NT>
__global__ __launch_bounds__(NT) void k_dc_control(FireDev* st, const double* partials, int nblocks, int k_steps) {
    __shared__ double scratch[NT / 64][4];
    dc_final<NT>(st, partials, nblocks, k_steps, scratch);
}

// The same for every member of a batch group (one block per member).
template <int NT>
__global__ __launch_bounds__(NT) void k_batch_dc_control(const MemberDev* __restrict__ mem, int k_steps) {
    __shared__ double scratch[NT / 64][4];
    const MemberDev& M = mem[blockIdx.x];
    dc_final<NT>(M.st, M.partials, M.nblocks, k_steps, scratch);
}

__global__ void k_batch_begin(const MemberDev* __restrict__ mem, int n_members, int64_t n_steps) {
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= n_members) return;
    FireDev* st = mem[m].st;
    ((DcCtl*)(st + 2))->halt = 0;
    if (st->status == LQ_RUNNING) {
        st->done = 0;
        st->stop_at = st->step + n_steps;
        if (n_steps <= 0) st->done = 1;
    }
}

// State of every member into its buffer 0 with pending steering applied.
template <typename T>
__global__ __launch_bounds__(256) void k_batch_finalize(const MemberDev* __restrict__ mem,
                                                        const int* __restrict__ off, int n_members) {
    const int m = member_of(off, n_members, (int)blockIdx.x);
    const MemberDev& M = mem[m];
    const FireDev* st = M.st;
    const int cur = st->cur;
    const T cv = T(st->c_v), cF = T(st->c_F);
    const int64_t n = 5 * M.L.N;
    const int nb = off[m + 1] - off[m];
    T* q0 = (T*)M.q[0]; T* v0 = (T*)M.v[0]; T* F0 = (T*)M.F[0];
    const T* qc = (const T*)M.q[cur]; const T* vc = (const T*)M.v[cur]; const T* Fc = (const T*)M.F[cur];
    for (int64_t i = ((int)blockIdx.x - off[m]) * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)nb * blockDim.x) {
        const T v = vc[i], f = Fc[i];
        const T vm = fma_t(cv, v, cF * f);
        if (cur) { q0[i] = qc[i]; F0[i] = f; }
        v0[i] = vm;
    }
}

// Resets the pending steering of every member and gathers the controller
// states into one array (pinned host memory).
__global__ void k_batch_reset_gather(const MemberDev* __restrict__ mem, int n_members, FireDev* out) {
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= n_members) return;
    FireDev* st = mem[m].st;
    st->cur = 0;
    st->c_v = 1.0;
    st->c_F = 0.0;
    out[m] = *st;
    __threadfence_system();
}

// ---------------------------------------------------------------------------
// lq_fire_init reduction: block partials of |F|^2, |v|^2, F.v, max|F_i| of the
// initial state; then one block sums them in block order and runs the
// controller's initial convergence test.
template <typename T>
__global__ __launch_bounds__(256) void k_init_reduce(const T* __restrict__ F, const T* __restrict__ v,
                                                     int64_t n, double* partials) {
    __shared__ double scratch[4][4];
    double r[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        double f = (double)F[i], w = v ? (double)v[i] : 0.0;
        r[0] = fma(f, w, r[0]);
        r[1] = fma(f, f, r[1]);
        r[2] = fma(w, w, r[2]);
        r[3] = fmax(r[3], fabs(f));
        if (f != f) r[3] = f;
    }
    block_reduce4(r, scratch);
    if (threadIdx.x == 0) {
        double* p = partials + 4 * (int64_t)blockIdx.x;
        p[0] = r[0]; p[1] = r[1]; p[2] = r[2]; p[3] = r[3];
    }
}

__global__ __launch_bounds__(256) void k_init_control(const double* partials, int nblocks, FireDev* st) {
    __shared__ double scratch[4][4];
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    sum_partials(partials, nblocks, s, scratch, 256);
    if (threadIdx.x == 0) {
        FireDev c = *st;
        fire_control(&c, s[0], s[1], s[2], s[3]);
        *st = c;
    }
}

__global__ void k_begin(FireDev* st, int64_t n_steps) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        ((DcCtl*)(st + 2))->halt = 0;
        if (st->status == LQ_RUNNING) {
            st->done = 0;
            st->stop_at = st->step + n_steps;
            if (n_steps <= 0) st->done = 1;
        }
    }
}

// Brings the current state into buffer 0 and applies the pending steering.
// Gradient descent leaves v untouched (with_v = false).  VL values (16 bytes)
// per lane where every buffer is 16-byte aligned: 4.4 -> 5.1 TB/s on the 256^3
// FP32 box.
template <typename T, int VL>
__global__ __launch_bounds__(256) void k_finalize(Bufs<T> b, int64_t n, const FireDev* st, int with_v) {
    struct alignas(sizeof(T) * VL) Vec {
        T e[VL];
    };
    const int cur = st->cur;
    const T cv = T(st->c_v), cF = T(st->c_F);
    auto at = [](T* p, int64_t i) -> Vec& { return ((Vec*)p)[i]; };
    const int64_t t0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, nt = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = t0; i < n / VL; i += nt) {
        const Vec f = at(b.F[cur], i);
        if (cur) {
            at(b.q[0], i) = at(b.q[1], i);
            at(b.F[0], i) = f;
        }
        if (with_v) {
            Vec v = at(b.v[cur], i);
#pragma unroll
            for (int k = 0; k < VL; ++k) v.e[k] = fma_t(cv, v.e[k], cF * f.e[k]);
            at(b.v[0], i) = v;
        }
    }
    for (int64_t i = n / VL * VL + t0; i < n; i += nt) {
        const T f = b.F[cur][i];
        if (cur) {
            b.q[0][i] = b.q[1][i];
            b.F[0][i] = f;
        }
        if (with_v) b.v[0][i] = fma_t(cv, b.v[cur][i], cF * f);
    }
}

// y = q + mu m: the Nesterov look-ahead point of a resumed state.
template <typename T>
__global__ __launch_bounds__(256) void k_lookahead(const T* __restrict__ q, const T* __restrict__ m, T mu,
                                                   T* __restrict__ y, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        y[i] = fma_t(mu, m[i], q[i]);
}

// After the finalize: no steering is pending, the state is in buffer 0.  The
// result also goes to host (pinned memory that the host reads after the call).
__global__ void k_reset_mix(FireDev* st, FireDev* host) {
    __shared__ FireDev c;
    constexpr int WORDS = sizeof(FireDev) / 4;
    const int t = threadIdx.x;
    if (t < WORDS) ((uint32_t*)&c)[t] = ((const uint32_t*)st)[t];
    __syncthreads();
    if (t == 0) {
        c.cur = 0;
        c.c_v = 1.0;
        c.c_F = 0.0;
    }
    __syncthreads();
    if (t < WORDS) {
        const uint32_t w = ((const uint32_t*)&c)[t];
        ((uint32_t*)st)[t] = w;
        ((uint32_t*)host)[t] = w;
    }
    __threadfence_system();
}

__global__ __launch_bounds__(256) void k_fill_zero(uint32_t* p, int64_t n_words) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n_words;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

// q = 3/2 S (n n - I/3) at simulated sites, 0 inside objects.  Products are
// rounded one by one (no contraction) so that the state is reproducible.
template <typename T>
__global__ __launch_bounds__(256) void k_uniaxial(LatDev L, const double* __restrict__ dirs, double S,
                                                  T* __restrict__ q) {
#pragma clang fp contract(off)
    const int64_t N = L.N;
    for (int64_t s = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; s < N;
         s += (int64_t)gridDim.x * blockDim.x) {
        double r[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
        if (L.mask[s] & M_SIM) {
            double nx = dirs[s], ny = dirs[N + s], nz = dirs[2 * N + s];
            double h = 1.5 * S;
            r[0] = h * (nx * nx - 1.0 / 3.0);
            r[1] = h * nx * ny;
            r[2] = h * nx * nz;
            r[3] = h * (ny * ny - 1.0 / 3.0);
            r[4] = h * ny * nz;
        }
        for (int c = 0; c < 5; ++c) q[c * N + s] = T(r[c]);
    }
}

// ---------------------------------------------------------------------------
// launchers
static int hip_status(hipError_t e) { return e == hipSuccess ? LQ_OK : LQ_EHIP; }

int64_t n_step_blocks(const LatDev& L) { return L.nblocks; }

int step_blocks_per_cu(int prec, bool l23, bool l4, int wide, bool two) {
    return prec == LQ_F64 ? march_blocks_per_cu_f64(l23, l4, wide, two) : march_blocks_per_cu_f32(l23, l4, wide);
}

int64_t n_energy_blocks(const LatDev& L) {
    int64_t b = (L.N + 255) / 256;
    return b < 2048 ? b : 2048;
}

static int grid_1d(int64_t n) {
    int64_t b = (n + 255) / 256;
    return (int)(b < 4096 ? (b > 0 ? b : 1) : 4096);
}

int launch_forces(const LatDev& L, bool l23, int prec, const void* q, void* F, void* stream) {
    if (L.kind == KIND_BRICK) launch_brick_forces(L, l23, prec, q, F, stream);
    else if (prec == LQ_F64) launch_march_f64(L, l23, MODE_FORCE, nullptr, q, F, nullptr, nullptr, 0, stream);
    else launch_march_f32(L, l23, MODE_FORCE, nullptr, q, F, nullptr, nullptr, 0, stream);
    return hip_status(hipGetLastError());
}

// Index of step kernel i (1-based) of a call as the step kernels use it:
// only whether it is the first, and its parity, matter (kept within int).
static int step_index(int64_t i) { return i <= 1 ? (int)i : 2 + (int)(i & 1); }

int launch_fire_steps(const LatDev& L, bool l23, int prec, int method, const void* bufs, double* partials,
                      FireDev* st, int64_t n_steps, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    const int mode = method == LQ_METHOD_GD ? MODE_GD : (method == LQ_METHOD_NESTEROV ? MODE_NAG : MODE_FIRE);
    for (int64_t i = 1; i <= n_steps; ++i) {
        const int k = step_index(i);
        if (L.kind == KIND_BRICK) launch_brick_step(L, l23, prec, method, bufs, partials, st, k, stream);
        else if (prec == LQ_F64) launch_march_f64(L, l23, mode, bufs, nullptr, nullptr, partials, st, k, stream);
        else launch_march_f32(L, l23, mode, bufs, nullptr, nullptr, partials, st, k, stream);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return LQ_EHIP;
    }
    // the controller on the last step's reduction, with the step kernel's block size
    if (L.kind == KIND_BRICK) {
        launch_brick_control(l23, st, partials, (int)n_step_blocks(L), step_index(n_steps), stream);
        return hip_status(hipGetLastError());
    }
    const int nt = tile_threads(prec, l23, L.kind), nb = (int)n_step_blocks(L), kl = step_index(n_steps);
    if (nt == 1024) k_dc_control<1024><<<1, 1024, 0, s>>>(st, partials, nb, kl);
    else if (nt == 512) k_dc_control<512><<<1, 512, 0, s>>>(st, partials, nb, kl);
    else if (nt == 256) k_dc_control<256><<<1, 256, 0, s>>>(st, partials, nb, kl);
    else return LQ_EINVAL;
    return hip_status(hipGetLastError());
}

int launch_fire_init_reduce(const LatDev& L, int prec, const void* F, const void* v,
                            double* partials, FireDev* st, void* stream);

int launch_begin(FireDev* st, int64_t n_steps, void* stream) {
    k_begin<<<1, 64, 0, (hipStream_t)stream>>>(st, n_steps);
    return hip_status(hipGetLastError());
}

template <typename T>
static void finalize_t(const Bufs<T>& b, int64_t n, const FireDev* st, int with_v, hipStream_t s) {
    uintptr_t any = 0;
    for (int i = 0; i < 2; ++i) any |= (uintptr_t)b.q[i] | (uintptr_t)b.v[i] | (uintptr_t)b.F[i];
    if (any % 16 == 0) {
        constexpr int VL = 16 / (int)sizeof(T);
        k_finalize<T, VL><<<grid_1d((n + VL - 1) / VL), 256, 0, s>>>(b, n, st, with_v);
    } else {
        k_finalize<T, 1><<<grid_1d(n), 256, 0, s>>>(b, n, st, with_v);
    }
}

int launch_finalize(const LatDev& L, int prec, bool with_v, const void* bufs, FireDev* st, FireDev* host, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    if (prec == LQ_F64) finalize_t(*(const Bufs<double>*)bufs, 5 * L.N, st, with_v, s);
    else finalize_t(*(const Bufs<float>*)bufs, 5 * L.N, st, with_v, s);
    if (hipGetLastError() != hipSuccess) return LQ_EHIP;
    k_reset_mix<<<1, 64, 0, s>>>(st, host);
    return hip_status(hipGetLastError());
}

int launch_lookahead(const LatDev& L, int prec, const void* q, const void* m, double mu, void* y,
                     void* stream) {
    hipStream_t s = (hipStream_t)stream;
    const int64_t n = 5 * L.N;
    if (prec == LQ_F64)
        k_lookahead<double><<<grid_1d(n), 256, 0, s>>>((const double*)q, (const double*)m, mu, (double*)y, n);
    else
        k_lookahead<float><<<grid_1d(n), 256, 0, s>>>((const float*)q, (const float*)m, (float)mu, (float*)y, n);
    return hip_status(hipGetLastError());
}

int launch_fill_zero(void* p, int64_t bytes, void* stream) {
    const int64_t w = bytes / 4;
    k_fill_zero<<<grid_1d(w), 256, 0, (hipStream_t)stream>>>((uint32_t*)p, w);
    return hip_status(hipGetLastError());
}

int launch_uniaxial(const LatDev& L, int prec, const double* dirs, double S, void* q,
                    void* stream) {
    hipStream_t s = (hipStream_t)stream;
    if (prec == LQ_F64) k_uniaxial<double><<<grid_1d(L.N), 256, 0, s>>>(L, dirs, S, (double*)q);
    else k_uniaxial<float><<<grid_1d(L.N), 256, 0, s>>>(L, dirs, S, (float*)q);
    return hip_status(hipGetLastError());
}

// The final controller of every member of a group, with the group's block size.
static void launch_batch_control(int nt, const MemberDev* mem, int n, int k, hipStream_t s) {
    if (n <= 0) return;
    if (nt == 1024) k_batch_dc_control<1024><<<n, 1024, 0, s>>>(mem, k);
    else if (nt == 512) k_batch_dc_control<512><<<n, 512, 0, s>>>(mem, k);
    else k_batch_dc_control<256><<<n, 256, 0, s>>>(mem, k);
}

int launch_batch_steps(int prec, bool l23, const MemberDev* mem, const BatchGroup group[N_KINDS],
                       const int* fin_off, int total_fin, FireDev* gather, int64_t n_steps, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    const MemberDev* gm[N_KINDS];
    int n_members = 0;
    for (int g = 0; g < N_KINDS; ++g) {
        gm[g] = mem + n_members;
        n_members += group[g].n;
    }
    const int nb = (n_members + 63) / 64;
    k_batch_begin<<<nb, 64, 0, s>>>(mem, n_members, n_steps);
    if (hipGetLastError() != hipSuccess) return LQ_EHIP;
    for (int64_t i = 1; i <= n_steps; ++i) {
        const int k = step_index(i);
        for (int w = KIND_NARROW; w <= KIND_WIDE; ++w) {
            if (prec == LQ_F64) launch_march_batch_f64(l23, gm[w], group[w], w, k, stream);
            else launch_march_batch_f32(l23, gm[w], group[w], w, k, stream);
        }
        launch_brick_batch(l23, prec, gm[KIND_BRICK], group[KIND_BRICK].off, group[KIND_BRICK].n,
                           group[KIND_BRICK].blocks, k, stream);
        if (hipGetLastError() != hipSuccess) return LQ_EHIP;
    }
    for (int w = KIND_NARROW; w <= KIND_WIDE; ++w)
        launch_batch_control(tile_threads(prec, l23, w), gm[w], group[w].n, step_index(n_steps), s);
    launch_brick_batch_control(l23, gm[KIND_BRICK], group[KIND_BRICK].n, step_index(n_steps), stream);
    if (hipGetLastError() != hipSuccess) return LQ_EHIP;
    if (prec == LQ_F64) k_batch_finalize<double><<<total_fin, 256, 0, s>>>(mem, fin_off, n_members);
    else k_batch_finalize<float><<<total_fin, 256, 0, s>>>(mem, fin_off, n_members);
    if (hipGetLastError() != hipSuccess) return LQ_EHIP;
    k_batch_reset_gather<<<nb, 64, 0, s>>>(mem, n_members, gather);
    return hip_status(hipGetLastError());
}

int launch_fire_init_reduce(const LatDev& L, int prec, const void* F, const void* v,
                            double* partials, FireDev* st, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    const int64_t n = 5 * L.N;
    const int g = (int)n_energy_blocks(L);
    if (prec == LQ_F64) k_init_reduce<double><<<g, 256, 0, s>>>((const double*)F, (const double*)v, n, partials);
    else k_init_reduce<float><<<g, 256, 0, s>>>((const float*)F, (const float*)v, n, partials);
    if (hipGetLastError() != hipSuccess) return LQ_EHIP;
    k_init_control<<<1, 256, 0, s>>>(partials, g, st);
    return hip_status(hipGetLastError());
}

}  // namespace lq
