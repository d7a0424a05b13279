// Readout kernels beyond the per-cell moments.
#pragma once

#include <hip/hip_runtime.h>

#include "state_kernels.h"

namespace elb {

constexpr int AMP_THREADS = 1024;
constexpr size_t AMP_DIRECT = 512;  // cells times 16-node groups (elb_get_amplitudes)

// Fourier amplitudes of the density over the cells (Sec. IV.A, the projection of the
// density perturbation): out[0] = (2/nx) sum_i n_i sin(k x_i), out[1] = (2/nx) sum_i n_i
// cos(k x_i), x_i = x0 + (i + 1/2) dx; out[2] is the failure flag, so that one copy brings
// all.  One block; FP64 sums in a fixed order (strided partial sums, then a tree over the
// threads), so repeated calls agree bit for bit.
//
// GIVEN: the density of cell i is dens[i stride] (the moment kernel's, or the tracked one).
// Otherwise it is summed here from the rows of psi, MOM_LANES lanes per cell in the order of
// k_moments, 64 cells at a time.  Bound by latency: 100 cells, Q = 8, 4.5 us
// and one copy, against 6.5 us in two kernels and two copies.
template <typename R, bool GIVEN>
__global__ __launch_bounds__(AMP_THREADS) void k_amplitudes(const R *psi, const double *ref, const double *dens, int stride,
                                                            int nx, int Q, double x0, double dx, double k, const int *flag,
                                                            double *out)
{
    __shared__ double ps[AMP_THREADS], pc[AMP_THREADS];
    const int tid = threadIdx.x;
    double s = 0.0, c = 0.0;
    for (int i0 = 0; i0 < nx; i0 += AMP_THREADS) {
        const int i = i0 + tid;
        double n = 0.0;
        if constexpr (GIVEN) {
            if (i < nx) n = dens[(size_t)i * stride];
        } else {
            // ps holds the densities of the next AMP_THREADS cells
            constexpr int CELLS = AMP_THREADS / MOM_LANES;
            const int part = tid % MOM_LANES;
            for (int j = tid / MOM_LANES; j < min(AMP_THREADS, (nx - i0 + CELLS - 1) / CELLS * CELLS); j += CELLS) {
                const bool live = i0 + j < nx;
                const R *ph = psi + (size_t)(live ? i0 + j + NG : NG) * 2 * Q;
                double v = 0.0;
                if (live)
                    for (int q = part; q < Q; q += MOM_LANES) v += (double)ph[q] + ref[q];
                v = sum16(v);
                if (part == 0) ps[j] = v;
            }
            __syncthreads();
            n = ps[tid];
            __syncthreads();
        }
        if (i < nx) {
            double sv, cv;
            sincos(k * (x0 + (i + 0.5) * dx), &sv, &cv);
            s = fma(n, sv, s);
            c = fma(n, cv, c);
        }
    }
    ps[tid] = s;
    pc[tid] = c;
    __syncthreads();
    for (int h = AMP_THREADS / 2; h > 0; h >>= 1) {
        if (tid < h) {
            ps[tid] += ps[tid + h];
            pc[tid] += pc[tid + h];
        }
        __syncthreads();
    }
    if (tid == 0) {
        out[0] = 2.0 * ps[0] / nx;
        out[1] = 2.0 * pc[0] / nx;
        out[2] = *flag ? 1.0 : 0.0;
    }
}

}  // namespace elb
