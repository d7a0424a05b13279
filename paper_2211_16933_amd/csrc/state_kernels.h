// Kernels around the stage kernel: initial states, conserved densities, per-cell moments and
// the base of the stochastic rounding stream.  Included by elb.hip only.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>

#include "elb_kernels.h"

namespace elb {

// Base of the stochastic rounding stream for the next replay of a captured graph.
__global__ void k_set_seed(unsigned *base, unsigned value)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) *base = value;
}

// --------------------------------------------------------------------------------------
// Check of the fields a state is set from: the first cell without finite n > 0, u, T > 0 and
// the first with a reduced density of 0.99 or more (UINT_MAX: none) and the smallest relaxation
// time.  One cell at a time on the host, or one partial result per block of k_check_state.
// --------------------------------------------------------------------------------------
constexpr int CHECK_THREADS = 256, CHECK_BLOCKS = 64, CHECK_HOST_CELLS = 2048;

struct StateCheck {
    double min_tau;
    unsigned bad, dense;

    __host__ __device__ void clear()
    {
        min_tau = 1e300;
        bad = dense = 0xffffffffu;
    }
    __host__ __device__ void cell(unsigned i, double vn, double vu, double vT, double b, double mu_ref)
    {
        if (!(vn > 0) || !(vT > 0) || !(fabs(vn) < HUGE_VAL) || !(fabs(vu) < HUGE_VAL) || !(fabs(vT) < HUGE_VAL)) {
            bad = i < bad ? i : bad;
            return;
        }
        const double eta = 0.25 * b * vn;
        if (eta >= 0.99) {
            dense = i < dense ? i : dense;
            return;
        }
        const double chi = 0.5 * (2.0 - eta) / ((1.0 - eta) * (1.0 - eta) * (1.0 - eta));
        const double y = b * vn * chi;
        const double cm = (4.0 / 25.0) * (1.0 + 12.0 / M_PI);
        min_tau = fmin(min_tau, mu_ref * (1.0 + 0.8 * y + cm * y * y) / (vn * chi * sqrt(vT)));
    }
    __host__ __device__ void add(const StateCheck &o)
    {
        min_tau = fmin(min_tau, o.min_tau);
        bad = o.bad < bad ? o.bad : bad;
        dense = o.dense < dense ? o.dense : dense;
    }
};

__global__ __launch_bounds__(CHECK_THREADS) void k_check_state(const double *fields, int nx, double b, double mu_ref,
                                                               StateCheck *part)
{
    __shared__ StateCheck sh[CHECK_THREADS];
    StateCheck s;
    s.clear();
    for (int i = blockIdx.x * CHECK_THREADS + threadIdx.x; i < nx; i += gridDim.x * CHECK_THREADS)
        s.cell(i, fields[i], fields[(size_t)nx + i], fields[2 * (size_t)nx + i], b, mu_ref);
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int h = CHECK_THREADS / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) sh[threadIdx.x].add(sh[threadIdx.x + h]);
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// --------------------------------------------------------------------------------------
// Equilibrium initialisation: phi_k = n g_k(u,T), theta_k = 2 T n g_k, g_k = sum_l Bt[l][k]
// c_l(u, T) in FP64 (QP-strided table), minus the per-column reference (zero in FP64 storage);
// with bookkeeping also the conserved densities (n, n u, (n u^2 + 3 n T)/2).  Interior rows of
// level 0 and the ghost rows (end states, or periodic images) of all three levels: the
// interior of the other two is written by the first stages before anything reads it.
//
// Two forms with the same arithmetic.  k_init_equilibrium: a thread per (row, node), which runs
// its row's coefficient chain beside the sum over l; a launch takes 5 to 50 us (Q = 8 to 200,
// tables cold) until the chip is full, then 320 us at 65536 cells, Q = 96.  k_init_tiles, for rows Q N >= INIT_TILES: the chain of a row once, by one
// thread, into LDS, then the product with Bt, each thread 8 rows of 4 nodes, so that a table
// value serves 8 rows and a coefficient read 4 nodes.  65536 cells, Q = 96: 100 us (FP64 117);
// Q = 12: 14 us against 16, below the line.  Setting a state took three launches of the first
// form, one per level: 950 us at 65536 cells, Q = 96; 91 at 160 cells, Q = 200, now 51.
// --------------------------------------------------------------------------------------
constexpr double INIT_TILES = 1e8;
constexpr int INIT_THREADS = 256, INIT_RJ = 8, INIT_KJ = 4;

// rows per block of k_init_tiles, within 64 KB of coefficients
inline int init_rows(int Q) { return Q >= 200 ? 32 : Q >= 64 ? 64 : 128; }

struct InitArgs {
    void *psi[3];
    double *U[3];        // bookkeeping mode, else NULL
    const double *fields;  // n [nx], u [nx], T [nx]
    const double *Bt, *sq, *rsq, *ref;
    int *flag;
    double ghost[2][3];
    int nx, Q, QP, N, periodic;
};

// n, u, T of storage row r (interior, periodic image or end state)
__device__ inline void init_fields(const InitArgs &a, int r, double &n, double &u, double &T)
{
    const int cell = r - NG;
    if (a.periodic || (cell >= 0 && cell < a.nx)) {
        const int i = row_of(cell, a.nx, a.periodic) - NG;
        n = a.fields[i];
        u = a.fields[(size_t)a.nx + i];
        T = a.fields[2 * (size_t)a.nx + i];
    } else {
        const double *g = a.ghost[cell < 0 ? 0 : 1];
        n = g[0]; u = g[1]; T = g[2];
    }
}

// the two distribution values of (row r, node k), and with k == 0 the conserved densities
template <typename R>
__device__ inline void init_store(const InitArgs &a, int r, int k, double n, double u, double T, double g)
{
    const bool ghost = r < NG || r >= a.nx + NG;
    const R phi = (R)(n * g - a.ref[k]), theta = (R)(2.0 * T * n * g - a.ref[a.Q + k]);
    auto put = [&](void *psi, double *U) {
        R *o = static_cast<R *>(psi) + (size_t)r * 2 * a.Q + k;
        o[0] = phi;
        o[a.Q] = theta;
        if (U && k == 0) {
            U[3 * (size_t)r + 0] = n;
            U[3 * (size_t)r + 1] = n * u;
            U[3 * (size_t)r + 2] = 0.5 * (n * u * u + 3.0 * n * T);
        }
    };
    put(a.psi[0], a.U[0]);
    if (ghost) {
        put(a.psi[1], a.U[1]);
        put(a.psi[2], a.U[2]);
    }
}

template <typename R>
__global__ __launch_bounds__(INIT_THREADS) void k_init_equilibrium(InitArgs a)
{
    const size_t idx = (size_t)blockIdx.x * INIT_THREADS + threadIdx.x;  // rows * Q may pass 2^31
    if (idx < 4) a.flag[idx] = 0;
    const int Q = a.Q, QP = a.QP;
    if (idx >= (size_t)(a.nx + 2 * NG) * Q) return;
    const int r = (int)(idx / Q), k = (int)(idx - (size_t)r * Q);
    double n, u, T;
    init_fields(a, r, n, u, T);
    double cm = 1.0, cc = u;
    double g = a.Bt[k] * cm;
    if (a.N >= 1) g += a.Bt[QP + k] * cc;
    for (int l = 1; l < a.N; ++l) {
        double cn = (u * cc + (T - 1.0) * a.sq[l] * cm) * a.rsq[l + 1];
        cm = cc;
        cc = cn;
        g += a.Bt[(l + 1) * QP + k] * cc;
    }
    init_store<R>(a, r, k, n, u, T, g);
}

template <typename R>
__global__ __launch_bounds__(INIT_THREADS) void k_init_tiles(InitArgs a, int rows)
{
    extern __shared__ double coef[];  // [N + 1][rows]
    __shared__ double f_n[128], f_u[128], f_T[128], sq_s[MAXQP], rsq_s[MAXQP];
    constexpr int RJ = INIT_RJ, KJ = INIT_KJ;
    const int r0 = blockIdx.x * rows;
    const int nr = min(rows, a.nx + 2 * NG - r0);
    const int t = threadIdx.x;
    if (blockIdx.x == 0 && t < 4) a.flag[t] = 0;
    if (t <= a.N) {
        sq_s[t] = a.sq[t];
        rsq_s[t] = a.rsq[t];
    }
    __syncthreads();
    if (t < rows) {
        double n, u, T;
        init_fields(a, r0 + min(t, nr - 1), n, u, T);
        f_n[t] = n;
        f_u[t] = u;
        f_T[t] = T;
        double cm = 1.0, cc = u;
        coef[t] = cm;
        coef[rows + t] = cc;
        for (int l0 = 1; l0 < a.N; l0 += 8) {  // the constants of 8 steps are read together
            double s8[8], r8[8];
#pragma unroll
            for (int d = 0; d < 8; ++d) {
                s8[d] = sq_s[min(l0 + d, a.N)];
                r8[d] = rsq_s[min(l0 + d + 1, a.N)];
            }
#pragma unroll
            for (int d = 0; d < 8; ++d)
                if (l0 + d < a.N) {
                    double cn = (u * cc + (T - 1.0) * s8[d] * cm) * r8[d];
                    cm = cc;
                    cc = cn;
                    coef[(l0 + d + 1) * rows + t] = cc;
                }
        }
    }
    __syncthreads();
    const int Q = a.Q, QK = Q / KJ;  // every compiled Q is a multiple of 4
    for (int it = t; it < QK * (rows / RJ); it += INIT_THREADS) {
        const int grp = it / QK, k = it - grp * QK;  // nodes k, k + QK, ...
        const double *c = coef + grp * RJ;
        double g[KJ][RJ];
#pragma unroll
        for (int m = 0; m < KJ; ++m)
#pragma unroll
            for (int j = 0; j < RJ; ++j) g[m][j] = 0.0;
        constexpr int LB = 4;  // orders whose table values are in flight together
        for (int l = 0; l <= a.N; l += LB) {
            double b[LB][KJ];
#pragma unroll
            for (int d = 0; d < LB; ++d)
#pragma unroll
                for (int m = 0; m < KJ; ++m) b[d][m] = a.Bt[min(l + d, a.N) * a.QP + k + m * QK];
#pragma unroll
            for (int d = 0; d < LB; ++d)
                if (l + d <= a.N)
#pragma unroll
                    for (int m = 0; m < KJ; ++m)
#pragma unroll
                        for (int j = 0; j < RJ; ++j) g[m][j] = fma(b[d][m], c[(l + d) * rows + j], g[m][j]);
        }
#pragma unroll
        for (int j = 0; j < RJ; ++j) {
            const int r = grp * RJ + j;
            if (r >= nr) break;
#pragma unroll
            for (int m = 0; m < KJ; ++m) init_store<R>(a, r0 + r, k + m * QK, f_n[r], f_u[r], f_T[r], g[m][j]);
        }
    }
}

// Conserved densities of every row of level 0 from the stored distributions plus reference
// (FP64 sums); those of the ghost rows, which all levels share, go to every level.
struct LevelU {
    double *U[3];
};

template <typename R>
__global__ void k_conserved_from_psi(const R *psi, const double *ref, LevelU lu, const double *p,
                                     int rows, int Q)
{
    int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= rows) return;
    const R *ph = psi + (size_t)r * 2 * Q;
    double n = 0, j = 0, e = 0;
    for (int k = 0; k < Q; ++k) {
        double v = (double)ph[k] + ref[k];
        n += v;
        j += p[k] * v;
        e += 0.5 * (p[k] * p[k] * v + (double)ph[Q + k] + ref[Q + k]);
    }
    auto put = [&](double *U) {
        U[3 * (size_t)r] = n;
        U[3 * (size_t)r + 1] = j;
        U[3 * (size_t)r + 2] = e;
    };
    put(lu.U[0]);
    if (r < NG || r >= rows - NG) {
        put(lu.U[1]);
        put(lu.U[2]);
    }
}

// --------------------------------------------------------------------------------------
// Whole distributions between the caller's planes phi, theta [nx][Q] (FP64) and level 0.  The
// planes lie in the interiors of levels 1 and 2, which hold nothing between steps.  Bound by
// the copies to and from the host; 10007 cells, Q = 40, FP32: storing 3.2 + 3.2 MB back took
// 470 to 1370 us with the conversion on the host (page faults of its buffer), restoring 1045.
//
// A launch must stay below 2^32 threads, and a plane of 2^32 values or more fits this card: one
// that large was launched with the remainder of its threads, and all other values were left as
// they were, without an error.  So the kernels over whole planes stride over them; 8192 blocks
// (eight rounds of four blocks per CU) keep the copy bandwidth-bound.
// --------------------------------------------------------------------------------------
constexpr int PLANE_THREADS = 256, PLANE_BLOCKS = 8192;

inline dim3 plane_grid(size_t values)
{
    const size_t blocks = (values + PLANE_THREADS - 1) / PLANE_THREADS;
    return dim3((unsigned)(blocks < (size_t)PLANE_BLOCKS ? blocks : (size_t)PLANE_BLOCKS));
}

__device__ inline size_t plane_first() { return (size_t)blockIdx.x * PLANE_THREADS + threadIdx.x; }
__device__ inline size_t plane_stride() { return (size_t)gridDim.x * PLANE_THREADS; }

template <typename R>
__global__ __launch_bounds__(PLANE_THREADS) void k_dist_planes(const R *psi, const double *ref, int nx, int Q, double *phi,
                                                               double *theta, const int *flag, int *flag_out)
{
    if (flag_out && plane_first() == 0) *flag_out = *flag;  // pinned memory: no copy of its own
    for (size_t t = plane_first(); t < (size_t)nx * Q; t += plane_stride()) {
        const size_t i = t / Q, o = (i + NG) * 2 * Q + (t - i * Q);
        const int k = (int)(t - i * Q);
        phi[t] = sizeof(R) == 8 ? (double)psi[o] : (double)psi[o] + ref[k];
        theta[t] = sizeof(R) == 8 ? (double)psi[o + Q] : (double)psi[o + Q] + ref[Q + k];
    }
}

// *bad = 1 when one of n values is not finite.
__global__ void k_all_finite(const double *v, size_t n, int *bad)
{
    bool b = false;
    for (size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (size_t)gridDim.x * blockDim.x)
        b |= !(fabs(v[t]) < HUGE_VAL);
    if (b) atomicOr(bad, 1);
}

// Density, velocity and temperature of every cell of the planes, one thread per cell, and the
// check for finite values.  The sums run over the nodes in order with every operation rounded
// (no fused multiply-add): the mean state they give is the reference of the FP32 storage, whose
// bits every later step follows.  Tiles of SUM_K nodes pass through LDS for coalesced reads.
constexpr int SUM_CELLS = 64, SUM_K = 8;

__global__ __launch_bounds__(SUM_CELLS) void k_dist_sums(const double *phi, const double *theta, const double *p, int nx,
                                                         int Q, double *fields, int *bad)
{
#pragma clang fp contract(off)
    __shared__ double f[2][SUM_CELLS][SUM_K + 1];
    const int i0 = blockIdx.x * SUM_CELLS, t = threadIdx.x, cells = min(SUM_CELLS, nx - i0);
    double n = 0, j = 0, e = 0;
    bool b = false;
    for (int k0 = 0; k0 < Q; k0 += SUM_K) {  // Q is a multiple of 4: the last tile may be half
        const int kn = min(SUM_K, Q - k0);
        for (int m = t; m < SUM_CELLS * SUM_K; m += SUM_CELLS) {
            const int c = m / SUM_K, k = m % SUM_K;
            if (c < cells && k < kn) {
                const size_t o = (size_t)(i0 + c) * Q + k0 + k;
                f[0][c][k] = phi[o];
                f[1][c][k] = theta[o];
            }
        }
        __syncthreads();
        if (t < cells)
            for (int k = 0; k < kn; ++k) {
                const double v = f[0][t][k], w = f[1][t][k], pk = p[k0 + k];
                b |= !(fabs(v) < HUGE_VAL) || !(fabs(w) < HUGE_VAL);
                n += v;
                j += pk * v;
                e += 0.5 * (pk * pk * v + w);
            }
        __syncthreads();
    }
    if (b) atomicOr(bad, 1);
    if (t < cells) {
        const double u = j / n;
        fields[i0 + t] = n;
        fields[(size_t)nx + i0 + t] = u;
        fields[2 * (size_t)nx + i0 + t] = (2.0 * e / n - u * u) / 3.0;
    }
}

// Level 0 from the planes; with old_ref != NULL (FP32) also the ghost rows of every level, moved
// from the old reference to the new one.  Clears the failure flag, which belongs to the state that
// these values replace.
template <typename R>
__global__ __launch_bounds__(PLANE_THREADS) void k_dist_pack(const double *phi, const double *theta, const double *ref,
                                                             const double *old_ref, int nx, int Q, R *psi0, R *psi1, R *psi2,
                                                             int *flag)
{
    if (plane_first() < 4) flag[plane_first()] = 0;
    const size_t interior = (size_t)nx * Q, all = old_ref ? interior + (size_t)2 * NG * Q : interior;
    for (size_t t = plane_first(); t < all; t += plane_stride()) {
        if (t < interior) {
            const size_t i = t / Q, o = (i + NG) * 2 * Q + (t - i * Q);
            const int k = (int)(t - i * Q);
            psi0[o] = sizeof(R) == 8 ? (R)phi[t] : (R)(phi[t] - ref[k]);
            psi0[o + Q] = sizeof(R) == 8 ? (R)theta[t] : (R)(theta[t] - ref[Q + k]);
        } else {
            const size_t g = t - interior, i = g / Q;  // ghost row 0..5
            const int k = (int)(g - i * Q);
            const size_t o = (i < NG ? i : i + nx) * 2 * Q + k;
            for (int h = 0; h < 2; ++h) {
                const int m = h * Q + k;
                const R v = (R)((double)psi0[o + h * Q] + old_ref[m] - ref[m]);
                psi0[o + h * Q] = v;
                psi1[o + h * Q] = v;
                psi2[o + h * Q] = v;
            }
        }
    }
}

// Per interior cell: n, u, T, q_x, P_xx (Sec. II.D) in FP64, two passes over the nodes, and
// the conserved densities (n, n u, E).  With U != NULL (bookkeeping) n, u, T and the
// conserved densities are the tracked ones; q_x and P_xx use that u.  `ref` is added to the
// stored values (deviation storage; zero for FP64).
//
// 16 lanes per cell (MOM_LANES), so a wave reads four rows as 64-byte segments: lane m
// takes the nodes m, m + 16, ... of phi and theta, and each pass ends with 4 exchange steps
// inside the 16-lane group.  The second pass re-reads the row from cache.  A launch takes the cells
// from `first` on, at most MOM_CELLS of them: one of 2^32 threads or more would run only the
// remainder.
constexpr int MOM_LANES = 16, MOM_CELLS = 1 << 24;
// Cells whose moments go straight to pinned memory.  us per readout, straight / by one copy: Q = 8
// 512 cells 15 / 24, 2048 17 / 26, 6144 24 / 33; Q = 200 2048 21 / 31, 6144 30 / 42.  The line is no
// crossing: to where the buffer ends (6553 cells) the copy is never the faster one.
constexpr size_t MOM_DIRECT = 2048;

__device__ inline double sum16(double v)
{
#pragma unroll
    for (int m = MOM_LANES / 2; m >= 1; m >>= 1) v += __shfl_xor(v, m, MOM_LANES);
    return v;
}

template <typename R>
__global__ void k_moments(const R *psi, const double *ref, const double *U, const double *p,
                          int nx, int Q, int first, double *out, const int *flag, double *out_cons)
{
    // out: n, u, T, q, Pxx [nx] each, and the failure flag behind them
    double *const out_n = out, *const out_u = out + nx, *const out_T = out + 2 * (size_t)nx,
           *const out_q = out + 3 * (size_t)nx, *const out_pxx = out + 4 * (size_t)nx;
    if (blockIdx.x == 0 && threadIdx.x == 0) *reinterpret_cast<int *>(out + 5 * (size_t)nx) = *flag;
    const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t i = first + gid / MOM_LANES;   // one cell per 16-lane group
    const int part = (int)(gid % MOM_LANES);
    // every lane of a group shares i, so a group is live or idle as a whole; idle groups
    // still run the exchanges (on zeros) and store nothing
    const bool live = i < (size_t)nx;
    const R *ph = psi + (live ? i + NG : (size_t)NG) * 2 * Q;
    const R *th = ph + Q;
    double n = 0, j = 0, e2 = 0;
    if (live)
        for (int k = part; k < Q; k += MOM_LANES) {
            const double v = (double)ph[k] + ref[k];
            n += v;
            j += p[k] * v;
            e2 += 0.5 * (p[k] * p[k] * v + (double)th[k] + ref[Q + k]);
        }
    n = sum16(n);
    j = sum16(j);
    e2 = sum16(e2);
    if (U && live) {
        const double *Ui = U + 3 * (i + NG);
        n = Ui[0];
        j = Ui[1];
        e2 = Ui[2];
    }
    const double u = live ? j / n : 0.0;
    double pxx = 0, e = 0, q = 0;
    if (live)
        for (int k = part; k < Q; k += MOM_LANES) {
            const double xi = p[k] - u;
            const double vp = (double)ph[k] + ref[k], vt = (double)th[k] + ref[Q + k];
            const double ek = 0.5 * xi * xi * vp + 0.5 * vt;
            pxx += xi * xi * vp;
            e += ek;
            q += xi * ek;
        }
    pxx = sum16(pxx);
    e = sum16(e);
    q = sum16(q);
    if (live && part == 0) {
        out_n[i] = n;
        out_u[i] = u;
        out_T[i] = U ? (2.0 * e2 / n - u * u) / 3.0 : e / (1.5 * n);
        out_q[i] = q;
        out_pxx[i] = pxx;
        if (out_cons) {
            out_cons[3 * i + 0] = n;
            out_cons[3 * i + 1] = j;
            out_cons[3 * i + 2] = e2;
        }
    }
}

}  // namespace elb
