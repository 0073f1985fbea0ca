// Observables of a state: the energy (FP64 per-term sums) and the director and
// defect extraction.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "lq_internal.h"
#include "lq_site.h"

namespace lq {

// ---------------------------------------------------------------------------
// Energy, in FP64: per-term block partials, summed in block order by a second
// kernel of one block.  (With the sum in the last block to take a ticket, the
// blocks' atomics and fences on one address took 25 ns each, 100 of the 110 us
// of a 128^3 energy.)  Bound by the L1 data path, 82% busy with 18 loads a site,
// beside a vector ALU that is 61% busy, two fifths of it FP64 arithmetic (256^3
// FP32 one-constant 440 -> 146 us per call, 130 of them this kernel, where its
// 336 MB take 68; L2/L3 578 -> 221; 128^3 110 -> 41, of which 20 are two launches
// and a wait); loading the neighbours one plane ahead measured equal to 15%
// slower, 2048 or 8192 blocks instead of 4096 equal or slower.  A thread owns one
// column (x, y) and walks zc planes of it upwards with the own and the next
// plane's q in registers.  A block takes 256 columns of one run of planes, or
// (PACKED) the columns' runs follow each other over the threads: boxes of few
// columns would leave most of such blocks idle (3x3x100000 FP32 207 us, packed 32;
// L2/L3 280 and 40; 4x4x30000 77 and 26), while in full blocks z is uniform (256^3
// FP32 145.9, packed 147.0).  Bonds are taken once, from their lower end, with the
// weights of both ends (1/n_k each, 1/2 in the bulk); the cross-axis and chiral
// terms need the mean differences of the site and so both neighbours of every
// axis.
template <typename T, bool L23, bool PACKED>
__global__ __launch_bounds__(256) void k_energy(LatDev L, const T* __restrict__ q, int zc, double* partials) {
    __shared__ double scratch[4][4];
    const int nxy = L.nx * L.ny;
    const int bid = xcd_block((int)blockIdx.x, (int)gridDim.x);
    int run, p;
    if (PACKED) {
        const int item = bid * 256 + (int)threadIdx.x;
        run = item / nxy;
        p = item - run * nxy;
    } else {
        const int cols = (nxy + 255) / 256;
        run = bid / cols;
        p = (bid - run * cols) * 256 + (int)threadIdx.x;
    }
    const int z0 = run * zc, z1 = min(z0 + zc, L.nz);
    const bool own = p < nxy && z0 < L.nz;
    const int x = p % L.nx, y = p / L.nx;
    const uint32_t cs = (uint32_t)L.N * (uint32_t)sizeof(T);
    const __amdgpu_buffer_rsrc_t rq = field_rsrc(q, 5u * cs);
    const __amdgpu_buffer_rsrc_t rm = field_rsrc(L.mask, (uint32_t)L.N);
    constexpr uint32_t NONE = 0xFFFFFFFFu;  // past every resource: loads give 0
    // plane offsets of the x and y neighbours, -1 off an open edge
    const int xp = x + 1 < L.nx ? p + 1 : (L.per[0] ? p + 1 - L.nx : -1);
    const int xm = x > 0 ? p - 1 : (L.per[0] ? p - 1 + L.nx : -1);
    const int yp = y + 1 < L.ny ? p + L.nx : (L.per[1] ? p + L.nx - nxy : -1);
    const int ym = y > 0 ? p - L.nx : (L.per[1] ? p - L.nx + nxy : -1);
    auto site = [&](int at, int z) -> uint32_t {
        const int wz = wrapc(z, L.nz, L.per[2]);
        return own && at >= 0 && wz >= 0 ? (uint32_t)(at + nxy * wz) : NONE;
    };
    auto mask = [&](uint32_t s) { return (uint32_t)__builtin_amdgcn_raw_buffer_load_b8(rm, (int)s, 0, 0); };
    auto load = [&](uint32_t s, double o[5]) {
        const uint32_t off = s == NONE ? NONE : s * (uint32_t)sizeof(T);
#pragma unroll
        for (int c = 0; c < 5; ++c) o[c] = (double)bld<T>(rq, off, c * cs);
    };
    // sum_ij dQ_ij^2 / 2 and column j's sum_i dQ_ij^2
    auto half_norm = [](const double d[5]) {
        return fma(d[0], d[0] + d[3], fma(d[3], d[3], fma(d[1], d[1], fma(d[2], d[2], d[4] * d[4]))));
    };
    double e_b = 0.0, e_d = 0.0, e_a = 0.0, e_x = 0.0;
    double q0[5], qz[5], qb[5];
    load(site(p, z0), q0);
    uint32_t m = mask(site(p, z0));
    if (L23) load(site(p, z0 - 1), qb);
    for (int z = z0; z < z1; ++z) {
        double qx[5], qy[5], qxm[5], qym[5];
        load(site(p, z + 1), qz);
        load(site(xp, z), qx);
        load(site(yp, z), qy);
        const uint32_t mz = mask(site(p, z + 1)), mx = mask(site(xp, z)), my = mask(site(yp, z));
        if (L23) {
            load(site(xm, z), qxm);
            load(site(ym, z), qym);
        }
        if (m & M_SIM) {
            // tr Q^2 = 2 h with h = half_norm(q); tr Q^3 = 3 det Q (traceless)
            const double zz = -q0[0] - q0[3];
            const double t2 = 2.0 * half_norm(q0);
            const double det = q0[0] * fma(q0[3], zz, -q0[4] * q0[4]) - q0[1] * fma(q0[1], zz, -q0[4] * q0[2]) +
                               q0[2] * fma(q0[1], q0[4], -q0[3] * q0[2]);
            e_b += t2 * fma(0.25 * L.C, t2, 0.5 * L.A) + L.B * det;
            double ed = 0.0;
            auto bond = [&](int k, const double n[5], uint32_t mn) {
                if (!has_nb(m, k, 1)) return;
                double d[5];
#pragma unroll
                for (int c = 0; c < 5; ++c) d[c] = n[c] - q0[c];
                const double w = (n_choices(m, k) == 2 ? 0.5 : 1.0) + (n_choices(mn, k) == 2 ? 0.5 : 1.0);
                double e = L.L1 * half_norm(d);
                if (L23) {
                    const double s = d[0] + d[3];
                    const double col = k == 0 ? fma(d[0], d[0], fma(d[1], d[1], d[2] * d[2]))
                                     : k == 1 ? fma(d[1], d[1], fma(d[3], d[3], d[4] * d[4]))
                                              : fma(s, s, fma(d[2], d[2], d[4] * d[4]));
                    e = fma(0.5 * (L.L2 + L.L3), col, e);
                }
                ed = fma(w, e, ed);
            };
            bond(0, qx, mx);
            bond(1, qy, my);
            bond(2, qz, mz);
            if (L23) {
                double Cm[3][5];
                const double* qp[3] = {qx, qy, qz};
                const double* qm[3] = {qxm, qym, qb};
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    double ap, a0, am;
                    mean_diff_coef(m, k, ap, a0, am);
#pragma unroll
                    for (int c = 0; c < 5; ++c) {
                        double v = a0 * q0[c];
                        if (ap != 0.0) v = fma(ap, qp[k][c], v);
                        if (am != 0.0) v = fma(am, qm[k][c], v);
                        Cm[k][c] = v;
                    }
                }
                // sum_{j<k} L2 sum_i C_j,ij C_k,ik + L3 sum_i C_j,ik C_k,ij
                double Cf[3][3][3];
#pragma unroll
                for (int k = 0; k < 3; ++k) full_of(Cm[k], Cf[k]);
                double s2 = 0.0, s3 = 0.0;
#pragma unroll
                for (int j = 0; j < 3; ++j)
#pragma unroll
                    for (int k = j + 1; k < 3; ++k)
#pragma unroll
                        for (int i = 0; i < 3; ++i) {
                            s2 = fma(Cf[j][i][j], Cf[k][i][k], s2);
                            s3 = fma(Cf[j][i][k], Cf[k][i][j], s3);
                        }
                ed += L.L2 * s2 + L.L3 * s3;
                if (L.L4 != 0.0) {
                    // chiral term L4/2 eps_lik Q_lj C_k,ij
                    double Q[3][3], e4 = 0.0;
                    full_of(q0, Q);
#pragma unroll
                    for (int l = 0; l < 3; ++l)
#pragma unroll
                        for (int i = 0; i < 3; ++i)
#pragma unroll
                            for (int k = 0; k < 3; ++k) {
                                if (eps3(l, i, k) == 0) continue;
#pragma unroll
                                for (int j = 0; j < 3; ++j) e4 += eps3(l, i, k) * Q[l][j] * Cf[k][i][j];
                            }
                    ed += 0.5 * L.L4 * e4;
                }
            }
            e_d += ed;
            double qe = 0.0;
#pragma unroll
            for (int c = 0; c < 5; ++c) qe = fma(L.ext[c], q0[c], qe);
            e_x -= qe;
            if (m & M_ANCH) {
                const int at = L.anch_index[site(p, z)] - 1;
                if (at >= 0) {
                    // 1/2 q^T K q + b^T q + c
                    const double* d = L.anch_data + ANCH_STRIDE * (int64_t)at;
                    double quad = 0.0, lin = 0.0;
                    int t = 0;
                    for (int a = 0; a < 5; ++a) {
                        lin += d[15 + a] * q0[a];
                        for (int b = a; b < 5; ++b, ++t) quad += (b == a ? 0.5 : 1.0) * d[t] * q0[a] * q0[b];
                    }
                    e_a += quad + lin + d[20];
                }
            }
        }
        m = mz;
#pragma unroll
        for (int c = 0; c < 5; ++c) {
            if (L23) qb[c] = q0[c];
            q0[c] = qz[c];
        }
    }
    double r[4] = {e_b, e_d, e_a, e_x};
    block_reduce4<false>(r, scratch);
    if (threadIdx.x == 0) {
        double* o = partials + 4 * (int64_t)bid;
        o[0] = r[0]; o[1] = r[1]; o[2] = r[2]; o[3] = r[3];
    }
}

constexpr int SUM_THREADS = 512;

// out may be host memory
__global__ __launch_bounds__(SUM_THREADS) void k_energy_sum(const double* partials, int n, EnergyOut* out) {
    __shared__ double scratch[SUM_THREADS / 64][4];
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (int b = threadIdx.x; b < n; b += SUM_THREADS) {
        const double* o = partials + 4 * (int64_t)b;
        s[0] += o[0]; s[1] += o[1]; s[2] += o[2]; s[3] += o[3];
    }
    block_reduce4<false>(s, scratch);
    if (threadIdx.x == 0) {
        out->bulk = s[0]; out->elastic = s[1]; out->anch = s[2]; out->ext = s[3];
        __threadfence_system();
    }
}

// ---------------------------------------------------------------------------
// Director and defect extraction (Eq. Qtensor and the text after it; the
// display of directors and defects in sec. IV): per simulated site the
// largest eigenvalue of Q and its eigenvector, and whether that eigenvalue
// lies below a threshold.  FP64 arithmetic.  For a traceless symmetric Q
// with p = sqrt(tr(Q^2)/6) the eigenvalues are 2p cos((acos(r) + 2 pi m)/3),
// r = det(Q)/(2 p^3) (the trigonometric solution of the characteristic
// cubic), m = 0 giving the largest.  The eigenvector is the largest cross
// product of two rows of Q - lambda I; when Q - lambda I has rank one (the
// largest eigenvalue is doubly degenerate) any vector normal to its
// non-zero row is an eigenvector.  n and -n being equal, the sign makes the
// largest-magnitude component positive.
//
// The cosine: c = cos(acos(r)/3) is the largest root of 4 c^3 - 3 c = r, taken
// by Newton's iteration in FP64 from a start good to 3e-5 (acos from Abramowitz
// and Stegun 4.4.45, cos from its series).  The derivative 12 c^2 - 3 enters in
// FP32: with its 1e-7 the truncation errors fall as 3e-5, 1e-8, 1e-15, below 1e-20
// for r >= -0.98, and the rounding of the last FP64 correction (about one spacing
// of the result) is what remains.  (Below that the root is nearly double and takes
// the rounding of r to its square root: the caller goes by sqrt, acos and cos.)
// With acos and cos for every site the kernel was bound by its arithmetic (192^3
// FP32 121 -> 103 us per call, 128^3 79 -> 52, 20 of them launches and the wait);
// now the vector ALU is 58% busy and the memory gives 3.3 of 4.9 TB/s.
__device__ __forceinline__ double cos_third(double r) {
    const float x = fabsf((float)r);
    float t = __builtin_amdgcn_sqrtf(fmaxf(1.0f - x, 0.0f)) *
              fmaf(fmaf(fmaf(-0.0187293f, x, 0.0742610f), x, -0.2121144f), x, 1.5707288f);
    t = (r < 0.0 ? 3.14159265f - t : t) * 0.333333333f;
    const float t2 = t * t;
    double c = (double)fmaf(t2, fmaf(t2, fmaf(t2, fmaf(t2, 2.48015873e-5f, -1.38888889e-3f), 4.16666667e-2f), -0.5f), 1.0f);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const double c2 = c * c;
        const double f = fma(c, fma(4.0, c2, -3.0), -r);
        c -= f * (double)__builtin_amdgcn_rcpf(fmaf(12.0f, (float)c2, -3.0f));
    }
    return c;
}

template <typename T>
__global__ __launch_bounds__(256) void k_directors(LatDev L, const T* __restrict__ q, T* __restrict__ dirs,
                                                   T* __restrict__ lmax, uint8_t* __restrict__ defect,
                                                   double thr, uint32_t* counts) {
    __shared__ unsigned int block_count;
    if (threadIdx.x == 0) block_count = 0;
    __syncthreads();
    const int64_t N = L.N;
    unsigned int mine = 0;
    for (int64_t s = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; s < N;
         s += (int64_t)gridDim.x * blockDim.x) {
        double n[3] = {0.0, 0.0, 0.0}, lam = 0.0;
        const bool sim = (L.mask[s] & M_SIM) != 0;
        if (sim) {
            double v[5];
            for (int c = 0; c < 5; ++c) v[c] = (double)q[c * N + s];
            double Q[3][3];
            full_of(v, Q);
            double p2 = 0.0;
            for (int i = 0; i < 3; ++i)
                for (int j = 0; j < 3; ++j) p2 += Q[i][j] * Q[i][j];
            if (p2 > 0.0) {
                // products of five entries of Q below stay in range for p2 in
                // [1e-80, 1e80]; other tensors are scaled by their largest entry
                double unit = 1.0;
                if (!(p2 >= 1e-80 && p2 <= 1e80)) {
                    for (int c = 0; c < 5; ++c) unit = c == 0 ? fabs(v[0]) : fmax(unit, fabs(v[c]));
                    if (unit > 0.0 && unit <= 1e300) {
                        p2 = 0.0;
                        for (int i = 0; i < 3; ++i)
                            for (int j = 0; j < 3; ++j) {
                                Q[i][j] /= unit;
                                p2 += Q[i][j] * Q[i][j];
                            }
                    } else {
                        unit = 1.0;
                    }
                }
                const double det = Q[0][0] * (Q[1][1] * Q[2][2] - Q[1][2] * Q[2][1]) -
                                   Q[0][1] * (Q[1][0] * Q[2][2] - Q[1][2] * Q[2][0]) +
                                   Q[0][2] * (Q[1][0] * Q[2][1] - Q[1][1] * Q[2][0]);
                // ps = p2 / 6, p = sqrt(ps) and rp = 1 / p, each rounded once:
                // with rsqrt(ps) as it comes the eigenvalues' mean error was 9.3e-17,
                // 6.7e-17 with a square root and a division, which take longer
                double ps = p2 * (1.0 / 6.0);
                ps = fma(fma(-6.0, ps, p2), 1.0 / 6.0, ps);
                double rp = rsqrt(ps), p = ps * rp;
                p = fma(fma(-p, p, ps), 0.5 * rp, p);
                rp = fma(fma(-p, rp, 1.0), rp, rp);
                const double r = 0.5 * det * rp * rp * rp;
                if (r >= -0.98 && rp > 0.0) {
                    lam = 2.0 * p * cos_third(fmin(1.0, r));
                } else {  // also where entries are infinite: p and rp are not numbers
                    p = sqrt(p2 / 6.0);
                    lam = 2.0 * p * cos(acos(fmin(1.0, fmax(-1.0, det / (2.0 * p * p * p)))) / 3.0);
                }
                double A[3][3];
                for (int i = 0; i < 3; ++i)
                    for (int j = 0; j < 3; ++j) A[i][j] = Q[i][j] - (i == j ? lam : 0.0);
                lam *= unit;
                double best = -1.0;
                for (int a = 0; a < 3; ++a)
                    for (int b = a + 1; b < 3; ++b) {
                        const double c[3] = {A[a][1] * A[b][2] - A[a][2] * A[b][1],
                                             A[a][2] * A[b][0] - A[a][0] * A[b][2],
                                             A[a][0] * A[b][1] - A[a][1] * A[b][0]};
                        const double c2 = c[0] * c[0] + c[1] * c[1] + c[2] * c[2];
                        if (c2 > best) { best = c2; n[0] = c[0]; n[1] = c[1]; n[2] = c[2]; }
                    }
                if (!(best > 0.0)) {
                    // rank one: a vector normal to the largest row
                    int a = 0;
                    double rb = -1.0;
                    for (int i = 0; i < 3; ++i) {
                        const double r2 = A[i][0] * A[i][0] + A[i][1] * A[i][1] + A[i][2] * A[i][2];
                        if (r2 > rb) { rb = r2; a = i; }
                    }
                    int e = 0;
                    for (int k = 1; k < 3; ++k)
                        if (fabs(A[a][k]) < fabs(A[a][e])) e = k;
                    double u[3] = {0.0, 0.0, 0.0};
                    u[e] = 1.0;
                    n[0] = A[a][1] * u[2] - A[a][2] * u[1];
                    n[1] = A[a][2] * u[0] - A[a][0] * u[2];
                    n[2] = A[a][0] * u[1] - A[a][1] * u[0];
                    best = n[0] * n[0] + n[1] * n[1] + n[2] * n[2];
                }
                const double inv = best > 0.0 ? rsqrt(best) : 0.0;
                int big = 0;
                for (int k = 1; k < 3; ++k)
                    if (fabs(n[k]) > fabs(n[big])) big = k;
                const double sg = n[big] < 0.0 ? -inv : inv;
                for (int k = 0; k < 3; ++k) n[k] *= sg;
            }
        }
        const bool is_defect = sim && lam < thr;
        mine += is_defect ? 1u : 0u;
        if (dirs)
            for (int k = 0; k < 3; ++k) dirs[k * N + s] = T(n[k]);
        if (lmax) lmax[s] = T(lam);
        if (defect) defect[s] = is_defect ? 1 : 0;
    }
    if (counts) {
        atomicAdd(&block_count, mine);
        __syncthreads();
        if (threadIdx.x == 0) counts[blockIdx.x] = block_count;
    }
}

// Sum of the blocks' defect counts; total may be host memory.
__global__ __launch_bounds__(256) void k_count_sum(const uint32_t* counts, int n, unsigned long long* total) {
    __shared__ unsigned long long sum;
    if (threadIdx.x == 0) sum = 0;
    __syncthreads();
    unsigned long long mine = 0;
    for (int b = threadIdx.x; b < n; b += 256) mine += counts[b];
    atomicAdd(&sum, mine);
    __syncthreads();
    if (threadIdx.x == 0) {
        *total = sum;
        __threadfence_system();
    }
}

// ---------------------------------------------------------------------------
// launchers

// Work split of the energy kernel: runs of zc planes of a column, so short that
// some 4096 blocks share the lattice (small ones: one plane a run); packed where
// blocks of 256 columns would leave more than a fifth of their threads idle.
struct EnergySplit {
    bool packed;
    int zc;
    int64_t blocks;
};
static EnergySplit energy_split(const LatDev& L) {
    const int64_t nxy = (int64_t)L.nx * L.ny, cols = (nxy + 255) / 256;
    EnergySplit e;
    e.packed = 4 * 256 * cols > 5 * nxy;
    const int64_t threads = (e.packed ? nxy : 256 * cols) * L.nz;
    e.zc = (int)std::min<int64_t>((threads + 4096 * 256 - 1) / (4096 * 256), L.nz);
    const int64_t runs = (L.nz + e.zc - 1) / e.zc;
    e.blocks = e.packed ? (nxy * runs + 255) / 256 : cols * runs;
    return e;
}

// Blocks of the director kernel (a grid-stride loop over the sites).
static int director_blocks(const LatDev& L) { return (int)std::min<int64_t>((L.N + 255) / 256, 4096); }
int64_t n_observe_bytes(const LatDev& L) {
    return std::max<int64_t>(energy_split(L).blocks * 4 * (int64_t)sizeof(double), director_blocks(L) * (int64_t)sizeof(uint32_t));
}

int launch_directors(const LatDev& L, int prec, const void* q, void* dirs, void* lmax, uint8_t* defect,
                     double thr, uint32_t* counts, unsigned long long* total, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    const int g = director_blocks(L);
    uint32_t* c = total ? counts : nullptr;
    if (prec == LQ_F64)
        k_directors<double><<<g, 256, 0, s>>>(L, (const double*)q, (double*)dirs, (double*)lmax, defect, thr, c);
    else
        k_directors<float><<<g, 256, 0, s>>>(L, (const float*)q, (float*)dirs, (float*)lmax, defect, thr, c);
    if (hipGetLastError() != hipSuccess) return LQ_EHIP;
    if (total) k_count_sum<<<1, 256, 0, s>>>(counts, g, total);
    return hipGetLastError() == hipSuccess ? LQ_OK : LQ_EHIP;
}

template <typename T, bool L23>
static void energy_t(const LatDev& L, const EnergySplit& e, const void* q, double* partials, hipStream_t s) {
    if (e.packed) k_energy<T, L23, true><<<dim3((unsigned)e.blocks), 256, 0, s>>>(L, (const T*)q, e.zc, partials);
    else k_energy<T, L23, false><<<dim3((unsigned)e.blocks), 256, 0, s>>>(L, (const T*)q, e.zc, partials);
}

int launch_energy(const LatDev& L, bool l23, int prec, const void* q, double* partials, EnergyOut* out,
                  void* stream) {
    hipStream_t s = (hipStream_t)stream;
    const EnergySplit e = energy_split(L);
    if (prec == LQ_F64) {
        if (l23) energy_t<double, true>(L, e, q, partials, s);
        else energy_t<double, false>(L, e, q, partials, s);
    } else {
        if (l23) energy_t<float, true>(L, e, q, partials, s);
        else energy_t<float, false>(L, e, q, partials, s);
    }
    if (hipGetLastError() != hipSuccess) return LQ_EHIP;
    k_energy_sum<<<1, SUM_THREADS, 0, s>>>(partials, (int)e.blocks, out);
    return hipGetLastError() == hipSuccess ? LQ_OK : LQ_EHIP;
}

}  // namespace lq
