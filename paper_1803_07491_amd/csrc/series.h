// Tables of the Chebyshev expansion, built by a whole block in LDS; the caller
// synchronises.
#pragma once
#include "bop_internal.h"

namespace bop {

// Jackson kernel of length n_exp adapted to U polynomials: g_m = g^J_(m+1)/g^J_1
// (whole block)
__device__ inline void jackson_table(int n_exp, double *s_g)
{
    const double w = M_PI / (n_exp + 1.0);
    double sw, cw;
    sincos(w, &sw, &cw);
    const double cotw = cw / sw;
    const double g1 = ((double)n_exp * cw + sw * cotw) / (n_exp + 1.0);
    for (int m = threadIdx.x; m <= n_exp; m += blockDim.x) {
        int mm = m + 1;
        double sm, cm;
        sincos(w * mm, &sm, &cm);
        double gj = ((double)(n_exp - mm + 1) * cm + sm * cotw) / (n_exp + 1.0);
        s_g[m] = gj / g1;
    }
}

// p[m * M + n]: coefficient of x^n in U_m; c[n * M + l]: binomials; both M x M, M <= 64,
// by a lane per column of the block's first two waves (128 threads at least).  Every
// entry is an integer below 2^53 for M <= 41, so exact.
__device__ inline void series_tables(int M, double *p, double *c)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (wave == 0) {
        double v = lane == 0 ? 1.0 : 0.0;
        for (int n = 0; n < M; ++n) {
            if (lane < M) c[n * M + lane] = v;
            const double below = __shfl_up(v, 1);
            v += lane > 0 ? below : 0.0;
        }
    } else if (wave == 1) {
        double p0 = 0.0, p1 = lane == 0 ? 1.0 : 0.0;
        for (int m = 0; m < M; ++m) {
            if (lane < M) p[m * M + lane] = p1;
            const double below = __shfl_up(p1, 1);
            const double p2 = (lane > 0 ? 2.0 * below : 0.0) - p0;
            p0 = p1;
            p1 = p2;
        }
    }
}

}  // namespace bop
