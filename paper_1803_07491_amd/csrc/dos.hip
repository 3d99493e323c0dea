// FP64 tail of the energy path (App. B of arXiv:1803.07491):
//  * recursion coefficients from moments (App. B.3, Eqs. momtoa, momtob and the
//    c_j^n recursion) with the Gershgorin terminator (App. B.5, Eq. gershogorin);
//  * Chebyshev expansion coefficients sigma_m (Eq. sigma_i), extended beyond
//    n_max by the chain recursion of App. B.4 with the constant terminator, and
//    Jackson damping (Eq. Jackson);
//  * electron counts, bond energies and DOS at E (App. B.2), the Fermi level
//    by bisection and interpolation (Sec. II),
//    per-atom sums (App. A.1 Eq. TB-Ubond).
//
// The chain recursion is evaluated on the computed levels 0..L-1 plus one
// level L: beyond the computed coefficients the terminated chain is free
// (a^ = 0, b^ = 1/2), and a free semi-infinite chain started from rest only
// passes its input down with a delay of one step, so level L obeys
// zeta_L^(m+1) = 2 b^_L zeta_(L-1)^(m) exactly and the levels below it see the
// same values as with the infinite tail.  Each row's chain then fits in
// registers.
//
// Expansion coefficients are stored m-major ([n_exp+1][rows]) so that the
// per-orbital sums read coalesced columns.  Global sums (electron count,
// bracket, total energy) use per-block partials reduced in a fixed order by a
// one-block launch that follows, so results are deterministic and no block
// needs a device-scope fence (which would write back L2).
#include "bop_internal.h"
#include "series.h"

#include <cmath>
#include <mutex>

namespace bop {
namespace {

constexpr int MAX_NMAX = 40;
constexpr int DT = 256;        // threads per block in this file

__device__ inline int n_a_of(int n_max) { return n_max >= 1 ? (n_max - 1) / 2 + 1 : 0; }
__device__ inline int n_b_of(int n_max) { return n_max / 2; }

// ---------------------------------------------------------------------------
// recursion coefficients and band edges
// ---------------------------------------------------------------------------
// Centre and width of the terminator from a row's stored chain a[0..na-1],
// b[1..nb] for the estimates of App. B.5 other than Gershgorin and the global
// values: (i) lowest, (ii) highest computed levels, (iii) averages, (iv)
// average centre with the highest width, (v) extreme a with the largest b
// (Eq. findeminemax), and the weighted averages of Eq. (weighted) with
// w_m = 1 / (beta (M - m) + 1).  Only the levels the chain computed count: up
// to level L - 1 when it broke down at level L (flag level L).
__device__ inline void band_estimate(int mode, double beta, const double *ar, const double *br, int na, int nb,
                                     int fl, double &A, double &B)
{
    int nav = na, nbv = nb;
    if (fl & BOP_FLAG_BREAKDOWN) {
        const int L = fl >> 8;
        nav = min(nav, L);
        nbv = min(nbv, L - 1);
    }
    double asum = 0.0, amax = 0.0, amin = 0.0, b2sum = 0.0, bmax = 0.0;
    for (int n = 0; n < nav; ++n) {
        const double v = ar[n];
        asum += v;
        amax = n == 0 ? v : fmax(amax, v);
        amin = n == 0 ? v : fmin(amin, v);
    }
    for (int n = 1; n <= nbv; ++n) {
        const double v = br[n];
        b2sum += v * v;
        bmax = fmax(bmax, v);
    }
    const double amean = nav > 0 ? asum / nav : 0.0;
    const double blow = nbv >= 1 ? br[1] : 0.0, btop = nbv >= 1 ? br[nbv] : 0.0;
    switch (mode) {
    case BOP_BW_LOWEST: A = nav > 0 ? ar[0] : 0.0; B = blow; break;
    case BOP_BW_HIGHEST: A = nav > 0 ? ar[nav - 1] : 0.0; B = btop; break;
    case BOP_BW_AVERAGE: A = amean; B = nbv > 0 ? sqrt(b2sum / nbv) : 0.0; break;
    case BOP_BW_AVERAGE_HIGHEST: A = amean; B = btop; break;
    case BOP_BW_MINMAX: A = 0.5 * (amax + amin); B = 0.25 * (amax - amin + 4.0 * bmax); break;
    default: {
        double wa = 0.0, sa = 0.0, wb = 0.0, sb = 0.0;
        for (int m = 0; m < nav; ++m) {
            const double w = 1.0 / (beta * (double)(nav - 1 - m) + 1.0);
            wa += w;
            sa += w * ar[m];
        }
        for (int m = 1; m <= nbv; ++m) {
            const double w = 1.0 / (beta * (double)(nbv - m) + 1.0);
            wb += w;
            sb += w * br[m];
        }
        A = wa > 0.0 ? sa / wa : 0.0;
        B = wb > 0.0 ? sb / wb : 0.0;
    }
    }
}
__global__ void __launch_bounds__(DT)
k_recursion(int n_rows, int n_max, const double *__restrict__ mu, int bw_mode, double a_glob,
            double b_glob, double *__restrict__ a, double *__restrict__ b, double *__restrict__ a_inf,
            double *__restrict__ b_inf, int *__restrict__ flags)
{
    int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n_rows) return;
    const int na = n_a_of(n_max), nb = n_b_of(n_max);
    double *ar = a + (long)r * na, *br = b + (long)r * (nb + 1);
    int fl = 0;
    if (!mu) {
        // a, b given (Lanczos form); keep its breakdown and non-finite flags
        fl = flags[r];
        goto terminator;
    }
    {
    double m[MAX_NMAX + 1];
    const double *mr = mu + (long)r * (n_max + 1);
    const double m0 = mr[0];
    for (int t = 0; t <= n_max; ++t) {
        m[t] = mr[t] / m0;
        if (!isfinite(m[t])) fl |= BOP_FLAG_NONFINITE;
    }
    double cp[MAX_NMAX / 2 + 3], cc[MAX_NMAX / 2 + 3], d[MAX_NMAX / 2 + 3];
    for (int j = 0; j < MAX_NMAX / 2 + 3; ++j) { cp[j] = 0.0; cc[j] = 0.0; }
    cc[0] = 1.0;
    br[0] = 0.0;
    double bn = 0.0;                   // b_n of the current level
    const double var = (n_max >= 2) ? m[2] - m[1] * m[1] : 0.0;
    bool broke = false;
    for (int n = 0; n < na; ++n) {
        if (broke) { ar[n] = ar[n - 1]; continue; }
        double s = 0.0;
        for (int j = 0; j <= n; ++j)
            for (int l = 0; l <= n; ++l) s += cc[j] * cc[l] * m[j + l + 1];
        ar[n] = s;
        if (n + 1 > nb) break;
        for (int j = 0; j <= n + 1; ++j) d[j] = (j > 0 ? cc[j - 1] : 0.0) - s * cc[j] - bn * cp[j];
        double b2 = 0.0;
        for (int j = 0; j <= n + 1; ++j)
            for (int l = 0; l <= n + 1; ++l) b2 += d[j] * d[l] * m[j + l];
        if (!(b2 > 1e-14 * var)) {
            for (int t = n + 1; t <= nb; ++t) br[t] = 0.0;
            fl |= BOP_FLAG_BREAKDOWN | ((n + 1) << 8);
            broke = true;
            continue;
        }
        double bb = sqrt(b2);
        br[n + 1] = bb;
        for (int j = 0; j <= n + 1; ++j) { cp[j] = cc[j]; cc[j] = d[j] / bb; }
        bn = bb;
    }
    }
terminator:
    double ai, bi;
    if (bw_mode == BOP_BW_GLOBAL) { ai = a_glob; bi = b_glob; }
    else if (bw_mode != BOP_BW_GERSHGORIN) band_estimate(bw_mode, a_glob, ar, br, na, nb, fl, ai, bi);
    else {
        double lo = 0.0, hi = 0.0;
        for (int n = 0; n < na; ++n) {
            double bl = (n >= 1 && n <= nb) ? br[n] : 0.0;
            double bh = (n + 1 <= nb) ? br[n + 1] : 0.0;
            double e0 = ar[n] - bl - bh, e1 = ar[n] + bl + bh;
            if (n == 0 || e0 < lo) lo = e0;
            if (n == 0 || e1 > hi) hi = e1;
        }
        ai = 0.5 * (hi + lo);
        bi = 0.25 * (hi - lo);
    }
    if (!(bi >= 1e-6)) { bi = 1e-6; fl |= BOP_FLAG_NARROW; }
    a_inf[r] = ai;
    b_inf[r] = bi;
    flags[r] = fl;
}

// The same recursion with its arrays in registers, for moments up to NM: the
// loops over the levels and orbital indices are unrolled with compile-time
// bounds, so no array needs indexing at run time.  The additions are the
// generic kernel's, in the same order.
template <int NM>
__global__ void __launch_bounds__(DT)
k_recursion_reg(int n_rows, int n_max, const double *__restrict__ mu, int bw_mode, double a_glob,
                double b_glob, double *__restrict__ a, double *__restrict__ b, double *__restrict__ a_inf,
                double *__restrict__ b_inf, int *__restrict__ flags)
{
    constexpr int NA = (NM - 1) / 2 + 1;       // levels of a
    constexpr int NB = NM / 2;                  // levels of b
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n_rows) return;
    const int na = n_a_of(n_max), nb = n_b_of(n_max);
    double *ar = a + (long)r * na, *br = b + (long)r * (nb + 1);
    int fl = 0;
    double m[NM + 1];
    const double *mr = mu + (long)r * (n_max + 1);
    const double m0 = mr[0];
#pragma unroll
    for (int t = 0; t <= NM; ++t) {
        m[t] = (t <= n_max) ? mr[t] / m0 : 0.0;
        if (t <= n_max && !isfinite(m[t])) fl |= BOP_FLAG_NONFINITE;
    }
    double av[NA], bv[NB + 2];
    double cp[NB + 2], cc[NB + 2], d[NB + 2];
#pragma unroll
    for (int j = 0; j < NB + 2; ++j) { cp[j] = 0.0; cc[j] = 0.0; d[j] = 0.0; bv[j] = 0.0; }
    cc[0] = 1.0;
    double bn = 0.0;
    const double var = (n_max >= 2) ? m[2] - m[1] * m[1] : 0.0;
    bool broke = false, done = false;
#pragma unroll
    for (int n = 0; n < NA; ++n) {
        av[n] = 0.0;
        if (n >= na || done) continue;
        if (broke) { av[n] = av[n > 0 ? n - 1 : 0]; continue; }
        double s = 0.0;
#pragma unroll
        for (int j = 0; j <= n; ++j)
#pragma unroll
            for (int l = 0; l <= n; ++l) s += cc[j] * cc[l] * m[j + l + 1];
        av[n] = s;
        if (n + 1 > nb) { done = true; continue; }
#pragma unroll
        for (int j = 0; j <= n + 1; ++j) d[j] = (j > 0 ? cc[j - 1] : 0.0) - s * cc[j] - bn * cp[j];
        double b2 = 0.0;
#pragma unroll
        for (int j = 0; j <= n + 1; ++j)
#pragma unroll
            for (int l = 0; l <= n + 1; ++l) b2 += d[j] * d[l] * m[j + l];
        if (!(b2 > 1e-14 * var)) {
            fl |= BOP_FLAG_BREAKDOWN | ((n + 1) << 8);
            broke = true;
            continue;
        }
        const double bb = sqrt(b2);
        bv[n + 1] = bb;
#pragma unroll
        for (int j = 0; j <= n + 1; ++j) { cp[j] = cc[j]; cc[j] = d[j] / bb; }
        bn = bb;
    }
#pragma unroll
    for (int n = 0; n < NA; ++n)
        if (n < na) ar[n] = av[n];
#pragma unroll
    for (int n = 0; n <= NB; ++n)
        if (n <= nb) br[n] = bv[n];
    double ai, bi;
    if (bw_mode == 1) { ai = a_glob; bi = b_glob; }
    else {
        double lo = 0.0, hi = 0.0;
#pragma unroll
        for (int n = 0; n < NA; ++n) {
            if (n >= na) continue;
            const double bl = (n >= 1 && n <= nb) ? bv[n] : 0.0;
            const double bh = (n + 1 <= nb) ? bv[n + 1] : 0.0;
            const double e0 = av[n] - bl - bh, e1 = av[n] + bl + bh;
            if (n == 0 || e0 < lo) lo = e0;
            if (n == 0 || e1 > hi) hi = e1;
        }
        ai = 0.5 * (hi + lo);
        bi = 0.25 * (hi - lo);
    }
    if (!(bi >= 1e-6)) { bi = 1e-6; fl |= BOP_FLAG_NARROW; }
    a_inf[r] = ai;
    b_inf[r] = bi;
    flags[r] = fl;
}

// ---------------------------------------------------------------------------
// expansion coefficients g_m sigma_m, m-major
// ---------------------------------------------------------------------------
template <int LM>
__global__ void __launch_bounds__(DT)
k_dos_coeffs(int n_rows, int n_max, int n_exp, const double *__restrict__ mu,
             const double *__restrict__ a, const double *__restrict__ b,
             const double *__restrict__ a_inf, const double *__restrict__ b_inf,
             double *__restrict__ gs, int *__restrict__ flags)
{
    __shared__ double s_p[(MAX_NMAX + 1) * (MAX_NMAX + 1)];   // p_mn
    __shared__ double s_c[(MAX_NMAX + 1) * (MAX_NMAX + 1)];   // binomials
    __shared__ double s_g[1025];                              // Jackson g_m
    const int M = n_max + 1;
    series_tables(M, s_p, s_c);
    jackson_table(n_exp, s_g);
    __syncthreads();
    int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n_rows) return;
    const int na = n_a_of(n_max), nb = n_b_of(n_max);
    const double ai = a_inf[r], bi = b_inf[r];
    // Every sigma_m comes from the chain without moments (Lanczos form) and for
    // a band of zero width (b_inf at its floor), where the normalised moments
    // would divide rounding noise by (2 b_inf)^n.
    const int n_mom = (mu && bi > 1e-6) ? n_max : 0;
    double big = 0.0;          // |g sigma| of a proper DOS stays below m + 1
    if (n_mom == 0) {
        gs[r] = s_g[0];
    } else {
    const double *mr = mu + (long)r * M;
    // normalised moments mu^_n
    double mh[MAX_NMAX + 1];
    const double m0 = mr[0];
    for (int n = 0; n < M; ++n) {
        double s = 0.0, pa = 1.0;           // pa = (-a_inf)^l
        for (int l = 0; l <= n; ++l) {
            s += s_c[n * M + l] * pa * (mr[n - l] / m0);
            pa *= -ai;
        }
        mh[n] = s / pow(2.0 * bi, (double)n);
    }
    for (int m = 0; m < M && m <= n_exp; ++m) {
        double s = 0.0;
        for (int n = 0; n <= m; ++n) s += s_p[m * M + n] * mh[n];
        gs[(long)m * n_rows + r] = s_g[m] * s;
        big = fmax(big, fabs(s_g[m] * s));
    }
    }
    if (n_exp <= n_mom) {
        if (!(big <= 1e4)) flags[r] |= BOP_FLAG_DIVERGENT;
        return;
    }
    // chain on levels 0..L with the delay level L
    const int L = na > nb ? na : nb;
    double ah[LM + 1], bh[LM + 2], z0[LM + 1], z1[LM + 1];
#pragma unroll
    for (int k = 0; k <= LM; ++k) {
        ah[k] = (k < na) ? (a[(long)r * na + k] - ai) / (2.0 * bi) : 0.0;
        z0[k] = 0.0;
        z1[k] = 0.0;
    }
#pragma unroll
    for (int k = 0; k <= LM + 1; ++k)
        bh[k] = (k == 0) ? 0.0 : ((k <= nb) ? b[(long)r * (nb + 1) + k] / (2.0 * bi) : 0.5);
    z1[0] = 1.0;
    for (int m = 0; m < n_exp; ++m) {
        double zn[LM + 1];
#pragma unroll
        for (int k = 0; k <= LM; ++k) {
            double lower = (k > 0) ? z1[k > 0 ? k - 1 : 0] : 0.0;
            double upper = (k < LM) ? z1[k < LM ? k + 1 : LM] : 0.0;
            double full = 2.0 * (ah[k] * z1[k] + bh[k] * lower + bh[k + 1] * upper) - z0[k];
            double delay = 2.0 * bh[k] * lower;
            zn[k] = (k < L) ? full : ((k == L) ? delay : 0.0);
        }
#pragma unroll
        for (int k = 0; k <= LM; ++k) { z0[k] = z1[k]; z1[k] = zn[k]; }
        const int mm = m + 1;
        if (mm > n_mom) {
            double v = s_g[mm] * z1[0];
            gs[(long)mm * n_rows + r] = v;
            big = fmax(big, fabs(v));
        }
    }
    if (!(big <= 1e4)) flags[r] |= BOP_FLAG_DIVERGENT;
}


// value of the lane below / above in the row of 16 lanes, 0 at its ends; of its first lane
__device__ inline double row_below(double v) { return __builtin_amdgcn_update_dpp(0.0, v, 0x111, 0xf, 0xf, true); }
__device__ inline double row_above(double v) { return __builtin_amdgcn_update_dpp(0.0, v, 0x101, 0xf, 0xf, true); }
__device__ inline double row_first(double v) { return __builtin_amdgcn_update_dpp(0.0, v, 0x150, 0xf, 0xf, true); }

// The same with 16 lanes per row, lane k carrying the chain's level k: one step of
// the chain is then seven operations and two exchanges between neighbouring lanes
// instead of a dozen levels' operations one after the other, which is what a row takes
// while the rows are too few to fill the chip.  The tables are built by a lane per
// column.  The operations on every value, and their order, are those of k_dos_coeffs.
// 200 terms: 640 rows 109 -> 16 us, 5120 rows 123 -> 26, 40,960 rows 170 -> 90; at
// 138,240 rows 210 against 187, where a lane per row has the chip full: the line
// (CL_ROWS) lies between.
constexpr int CL = 16;                                       // lanes per row: up to 15 levels and the delay level
constexpr int CR = DT / CL;                                  // rows per block
constexpr int CL_NMAX = 20;
constexpr long CL_ROWS = 98304;

__global__ void __launch_bounds__(DT)
k_dos_coeffs_lanes(int n_rows, int n_max, int n_exp, const double *__restrict__ mu,
                   const double *__restrict__ a, const double *__restrict__ b,
                   const double *__restrict__ a_inf, const double *__restrict__ b_inf,
                   double *__restrict__ gs, int *__restrict__ flags)
{
    constexpr int MM = CL_NMAX + 1;
    __shared__ double s_p[MM * MM], s_c[MM * MM];            // p_mn, binomials
    __shared__ double s_g[1025];                              // Jackson g_m
    __shared__ double s_m[CR][MM], s_mh[CR][MM];              // mu_n / mu_0, normalised moments
    const int M = n_max + 1;
    const int k = threadIdx.x & (CL - 1), row = threadIdx.x / CL;
    const long r = (long)blockIdx.x * CR + row;
    const bool live = r < n_rows;
    const long rr = live ? r : n_rows - 1;
    const double ai = a_inf[rr], bi = b_inf[rr];
    const int na = n_a_of(n_max), nb = n_b_of(n_max);
    const double ak = k < na ? a[rr * na + k] : 0.0, bk = k <= nb ? b[rr * (nb + 1) + k] : 0.0;
    const double bk1 = k + 1 <= nb ? b[rr * (nb + 1) + k + 1] : 0.0;
    if (mu) {
        const double *mr = mu + rr * M;
        const double m0 = mr[0];
        for (int n = k; n < M; n += CL) s_m[row][n] = mr[n] / m0;
        series_tables(M, s_p, s_c);
    }
    jackson_table(n_exp, s_g);
    __syncthreads();
    const int n_mom = (mu && bi > 1e-6) ? n_max : 0;
    double big = 0.0;
    if (n_mom != 0) {
        for (int n = k; n < M; n += CL) {
            double s = 0.0, pa = 1.0;                         // pa = (-a_inf)^l
            for (int l = 0; l <= n; ++l) {
                s += s_c[n * M + l] * pa * s_m[row][n - l];
                pa *= -ai;
            }
            s_mh[row][n] = s / pow(2.0 * bi, (double)n);
        }
    }
    __syncthreads();
    if (n_mom == 0) {
        if (live && k == 0) gs[r] = s_g[0];
    } else {
        for (int m = k; m < M && m <= n_exp; m += CL) {
            double s = 0.0;
            for (int n = 0; n <= m; ++n) s += s_p[m * M + n] * s_mh[row][n];
            if (live) gs[(long)m * n_rows + r] = s_g[m] * s;
            big = fmax(big, fabs(s_g[m] * s));
        }
    }
    if (n_exp > n_mom) {
        const int L = na > nb ? na : nb;
        const double ah = k < na ? (ak - ai) / (2.0 * bi) : 0.0;
        const double bh = k == 0 || k > L ? 0.0 : (k <= nb ? bk / (2.0 * bi) : 0.5);
        const double bh1 = k + 1 <= nb ? bk1 / (2.0 * bi) : 0.5;
        double z0 = 0.0, z1 = k == 0 ? 1.0 : 0.0;
        // sixteen steps at a time, lane t keeping level 0 of the t-th, so that the
        // table reads and stores are not between the steps
        for (int m = 1; m <= n_exp; m += CL) {
            double top = 0.0;
#pragma unroll
            for (int t = 0; t < CL; ++t) {
                const double x = bh * row_below(z1);
                const double full = 2.0 * (ah * z1 + x + bh1 * row_above(z1)) - z0;
                z0 = z1;
                z1 = k < L ? full : x + x;                    // the delay level; 0 beyond it
                const double first = row_first(z1);
                top = k == t ? first : top;
            }
            const int mm = m + k;
            if (mm > n_mom && mm <= n_exp) {
                const double v = s_g[mm] * top;
                if (live) gs[(long)mm * n_rows + r] = v;
                big = fmax(big, fabs(v));
            }
        }
    }
    const bool bad = !(big <= 1e4);
    const unsigned long long any = __ballot(bad) >> (threadIdx.x & 48) & 0xffff;
    if (live && k == 0 && any) flags[r] |= BOP_FLAG_DIVERGENT;
}

// ---------------------------------------------------------------------------
// per-orbital sums at energy E
// ---------------------------------------------------------------------------
// Block sums of N values per thread at once: each wave folds its values with
// shuffles, one barrier, then thread p < N adds the waves' values in wave
// order.
// Result valid in thread p for value p.
template <int N>
__device__ inline double block_sum_n(double (&v)[N], double *s_red /* N x (DT / 64) */)
{
    constexpr int NW = DT / 64;
#pragma unroll
    for (int j = 0; j < N; ++j)
        for (int o = 32; o > 0; o >>= 1) v[j] += __shfl_xor(v[j], o);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) {
#pragma unroll
        for (int j = 0; j < N; ++j) s_red[j * NW + w] = v[j];
    }
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x < N)
        for (int q = 0; q < NW; ++q) t += s_red[threadIdx.x * NW + q];
    __syncthreads();
    return t;
}

// Fermi search state: bracket [lo, hi] with twice the counts at its ends, the expected
// level, whether the search is to bisect throughout, done flag, halvings taken so far.
struct FermiState { double lo, hi, nlo, nhi, x, plain, done, halvings; };

__global__ void __launch_bounds__(DT)
k_bracket(int n_rows, const double *__restrict__ a_inf, const double *__restrict__ b_inf,
          double *__restrict__ part)
{
    __shared__ double s_lo[DT / 64], s_hi[DT / 64];
    int r = blockIdx.x * blockDim.x + threadIdx.x;
    double lo = INFINITY, hi = -INFINITY;
    if (r < n_rows) { lo = a_inf[r] - 2.0 * b_inf[r]; hi = a_inf[r] + 2.0 * b_inf[r]; }
    for (int o = 32; o > 0; o >>= 1) { lo = fmin(lo, __shfl_xor(lo, o)); hi = fmax(hi, __shfl_xor(hi, o)); }
    if ((threadIdx.x & 63) == 0) { s_lo[threadIdx.x >> 6] = lo; s_hi[threadIdx.x >> 6] = hi; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 0; q < DT / 64; ++q) { lo = fmin(lo, s_lo[q]); hi = fmax(hi, s_hi[q]); }
        part[2 * blockIdx.x] = lo;
        part[2 * blockIdx.x + 1] = hi;
    }
}

// The bracket from the block partials (one block, fixed order).  Global sums
// and extrema are finished in a launch of their own: a last-block scheme
// would need a device-scope fence in every block, which writes back L2.
__global__ void __launch_bounds__(DT)
k_bracket_pick(int n_rows, unsigned n_blocks, const double *__restrict__ part, FermiState *st)
{
    __shared__ double s_red[DT / 64];
    const double L = partials_combine(part, n_blocks, 2, 0, 1, s_red);
    const double H = partials_combine(part, n_blocks, 2, 1, 2, s_red);
    if (threadIdx.x == 0) *st = FermiState{L, H, 0.0, 2.0 * n_rows, 0.0, 0.0, 0.0, 0.0};
}

// Fermi level (Sec. II): the root of the count by bisection, continued by interpolation.
// A pass evaluates the electron count at 15 energies (nodes) and the state moves on:
//  * bisecting passes (the first FT_TREE, and all after the closing ones): the nodes
//    are the midpoints that the next four halvings can visit, a binary tree in heap
//    order formed exactly as sequential bisection forms it, mid = (lo + hi)/2, and
//    the four decisions are replayed.  They are those of plain bisection;
//  * after FT_TREE passes the count is smooth on the bracket, a 4096th of the band (its
//    200 or so terms turn by a seventh of a radian over the pass's node spacing):
//    the polynomial through the eight nodes nearest to the sign change gives its root
//    to about 1e-12 of the band;
//  * closing passes (FT_CLOSE at most): nodes at growing distances on both sides
//    of the expected root, whose counts close the bracket around it.  Once it is
//    narrower than FT_TIGHT of the last one the root follows by linear interpolation
//    between the counts at its ends (its error is the bracket's square, below the
//    counts' own rounding);
//  * a count that is all but flat on the bracket (a gap, next to no or all electrons),
//    where the level depends on the counts' rounding, is bisected throughout, to
//    the last bit or FT_MAX_HALVINGS, and so is what the closing passes left open
//    (a band edge in the bracket);
//  * so is a count that the polynomial does not follow (rows whose band is a small
//    part of the others', diverging expansions), and one that a closing pass finds
//    above n_elec and below it again.  A closing pass that narrows the bracket by less
//    than a bisecting one is the last, so that the FT_PASSES passes of plain bisection do
//    for every search (one such pass in it, they reach a 2^60th of the band).  Where the count has several roots the level
//    is therefore plain bisection's, unless the count is smooth at its nodes and all of
//    a closing pass's nodes miss its turn.
// Four passes then do for what bisection alone takes 15 for.  Against it the level is
// within 1e-15 eV over 54 to 27,648 atoms and 1 to 1024 terms; whole tails, 200 terms: 128
// atoms 168 -> 124 us, 2000 atoms 326 -> 180, 8192 atoms 590 -> 289, 128,000 atoms 6.16 ->
// 2.10 ms; bisected throughout (a gap) 1000 rows take 208 us.
constexpr int FT_MAX_HALVINGS = 64;            // as many as plain bisection takes at most
constexpr int FT_LEVELS = 4, FT_NODES = (1 << FT_LEVELS) - 1;
constexpr int FT_TREE = 3, FT_CLOSE = 2;       // bisecting passes first, closing passes then
constexpr double FT_TIGHT = 1.0 / (1 << 24);
// Least change of the count over the bracket, per row, for the closing passes: the counts'
// rounding then moves the level by less than 1e-12 of the band.  (A count that is
// reached at the bracket's very end may be reached there without slope.)
constexpr double FT_SLOPE = 1e-7;
// Rounding of a count, relative to the rows or, where expansions diverge, to the counts
// at the bracket's ends: what a node past the root may lie below n_elec by.
constexpr double FT_ROUND = 1.0 / (1ull << 44);
constexpr int FP_ROWS = 32;                    // rows per row block (one per lane of half a wave)
constexpr int FP_GROUPS = DT / FP_ROWS;        // thread groups of a block, each with its own nodes
constexpr int FP_RUN = 26;                     // coefficients a thread stages
constexpr int FP_CH = 202;                     // terms held in LDS: what lets three blocks share a CU
static_assert(FP_CH <= FP_GROUPS * FP_RUN && FP_CH > (FP_GROUPS - 1) * FP_RUN, "the last group stages what is left");

__device__ inline bool closing(const FermiState &st, int pass)
{
    return pass >= FT_TREE && pass < FT_TREE + FT_CLOSE && st.plain == 0.0;
}

// energy of node p in a pass
__device__ inline double node_energy(const FermiState &st, int pass, int p)
{
    double l = st.lo, h = st.hi;
    if (closing(st, pass)) {
        const int j = p - FT_NODES / 2, d = j < 0 ? -j : j;
        // 2^-36, 2^-30, .. 2^-12, 2^-7, 2^-3 of the bracket
        const int e = d <= 5 ? -42 + 6 * d : (d == 6 ? -7 : -3);
        const double off = d ? ldexp(h - l, e) : 0.0, x = j < 0 ? st.x - off : st.x + off;
        return x < l ? l : (x > h ? h : x);
    }
    const int heap = p + 1;
    for (int bit = 30 - __clz(heap); bit >= 0; --bit) {
        const double m = 0.5 * (l + h);
        if (heap >> bit & 1) l = m; else h = m;
    }
    return 0.5 * (l + h);
}

// Root in [i, i + 1] of the polynomial through eight of the 17 equally spaced values
// v (Newton's form on forward differences, a few safeguarded Newton steps); -1 where the
// fourth to seventh differences do not fall below an eighth of the step from v[i] to
// v[i + 1].  The count is then not smooth at this spacing: most rows' bands lie in a
// few nodes' reach of a band that some rows stretch, or expansions diverge.  With that
// limit on the seventh alone, and at the step itself, 30% of the levels of 640 such rows
// were other roots than bisection's, and the closing passes took as long as it.
__device__ inline double root_between(const double *v, int i, double n_elec)
{
    const int j0 = min(max(i - 3, 0), FT_NODES + 1 - 7);
    double d[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) d[k] = v[j0 + k] - n_elec;
    const double fl = v[i] - n_elec, fh = v[i + 1] - n_elec;
#pragma unroll
    for (int k = 1; k < 8; ++k)
#pragma unroll
        for (int q = 7; q >= k; --q) d[q] -= d[q - 1];
    if (!(fabs(d[4]) + fabs(d[5]) + fabs(d[6]) + fabs(d[7]) <= 0.125 * (fh - fl))) return -1.0;
    const double a = i - j0;
    double u = a + fl / (fl - fh);
    for (int it = 0; it < 5; ++it) {
        double f = d[7], g = 0.0;
#pragma unroll
        for (int k = 6; k >= 0; --k) {
            const double r = 1.0 / (k + 1), m = (u - k) * r;
            g = fma(g, m, f * r);
            f = fma(m, f, d[k]);
        }
        u -= f / g;
        u = u < a ? a : (u > a + 1.0 ? a + 1.0 : u);
    }
    return u - a;
}

// The state after a pass from st, tot[p] the count at its node p (one thread; v:
// scratch of FT_NODES + 2).
__device__ inline FermiState fermi_advance(const FermiState &st, int pass, int n_rows, double n_elec, const double *tot,
                                           double *v)
{
    FermiState s = st;
    double frac = 0.5;                            // where in the new bracket the root is expected
    if (!closing(st, pass)) {
        int node = 1;
        for (int lev = 0; lev < FT_LEVELS; ++lev) {
            const double m = 0.5 * (s.lo + s.hi);
            if (s.halvings >= FT_MAX_HALVINGS || m <= s.lo || m >= s.hi) { s.done = 1.0; break; }
            const double c = 2.0 * tot[node - 1];
            if (c < n_elec) { s.lo = m; s.nlo = c; node = 2 * node + 1; }
            else { s.hi = m; s.nhi = c; node = 2 * node; }
            s.halvings += 1.0;
        }
        if (s.halvings >= FT_MAX_HALVINGS) s.done = 1.0;
        if (pass != FT_TREE - 1 || s.done != 0.0) return s;
        const double step = s.nhi - s.nlo, off = fmin(s.nhi - n_elec, n_elec - s.nlo);
        if (!(step >= FT_SLOPE * n_rows && off >= step / (1 << 16))) {
            s.plain = 1.0;
            return s;
        }
        v[0] = st.nlo;
        v[FT_NODES + 1] = st.nhi;
        for (int q = 1; q <= FT_NODES; ++q) {      // in order of energy: node of the tree's level by the trailing zeros
            const int z = __ffs(q) - 1;
            v[q] = 2.0 * tot[(1 << (FT_LEVELS - 1 - z)) + (q >> (z + 1)) - 1];
        }
        frac = root_between(v, node - (1 << FT_LEVELS), n_elec);
        if (frac < 0.0) {
            s.plain = 1.0;
            return s;
        }
    } else {
        int j = 0;
        while (j < FT_NODES && 2.0 * tot[j] < n_elec) ++j;
        const double slack = FT_ROUND * fmax((double)n_rows, fmax(fabs(st.nlo), fabs(st.nhi)));
        bool once = true;
        for (int q = j + 1; q < FT_NODES; ++q) once = once && 2.0 * tot[q] >= n_elec - slack;
        if (!once) {
            s.plain = 1.0;
            return s;
        }
        if (j < FT_NODES) { s.hi = node_energy(st, pass, j); s.nhi = 2.0 * tot[j]; }
        if (j > 0) { s.lo = node_energy(st, pass, j - 1); s.nlo = 2.0 * tot[j - 1]; }
        frac = (n_elec - s.nlo) / (s.nhi - s.nlo);
        if (s.hi - s.lo <= FT_TIGHT * (st.hi - st.lo)) s.done = 1.0;
        else if ((1 << FT_LEVELS) * (s.hi - s.lo) > st.hi - st.lo) s.plain = 1.0;
    }
    if (!(frac >= 0.0 && frac <= 1.0)) frac = 0.5;
    s.x = s.lo + frac * (s.hi - s.lo);
    if (s.done != 0.0) s.lo = s.hi = s.x;
    return s;
}

// A pass's 32-row partials: the row blocks of a node (a multiple of four of them) side
// by side, as the sums read them.
__host__ __device__ inline size_t ft_pitch(unsigned n_rb) { return (n_rb + 3) / 4 * 4; }

// Counts of every node in all threads' view (s_tot), from the 32-row partials of a
// pass, by one block.  The order of the additions is fixed: four row blocks in turn (128
// rows), then the tree over 64 such sums, then those trees in turn.
constexpr int FT_TREES = 2;
constexpr long FT_FUSED = FT_TREES * 128 * 64;

__device__ inline void node_totals(unsigned n_rb, const double *__restrict__ part, double *s_tot)
{
    constexpr int NW = DT / 64, PER = (FT_NODES + NW - 1) / NW;
    const unsigned lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    double sum[PER] = {};
    for (unsigned q0 = lane; 4 * (q0 - lane) < n_rb; q0 += 64) {
        double x[PER][4];
#pragma unroll
        for (int i = 0; i < PER; ++i)
#pragma unroll
            for (unsigned e = 0; e < 4; ++e)
                x[i][e] = part[min((int)(wv + i * NW), FT_NODES - 1) * ft_pitch(n_rb) + min(4 * q0 + e, n_rb - 1)];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            double t = 0.0;
#pragma unroll
            for (unsigned e = 0; e < 4; ++e) t += 4 * q0 + e < n_rb ? x[i][e] : 0.0;
            for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o);
            sum[i] += t;
        }
    }
#pragma unroll
    for (int i = 0; i < PER; ++i)
        if (lane == 0 && wv + i * NW < FT_NODES) s_tot[wv + i * NW] = sum[i];
    __syncthreads();
}

// State at the start of pass `pass` in every thread: the bracket of the block
// partials `prev` (pass 0), or the previous pass's state and partials.  s_tot: 96.
__device__ inline FermiState fermi_state(int pass, int n_rows, unsigned n_bracket, double n_elec,
                                         const double *__restrict__ prev, const FermiState *st, double *s_tot,
                                         FermiState *s_st)
{
    if (pass == 0) {
        const double L = partials_combine(prev, n_bracket, 2, 0, 1, s_tot);
        const double H = partials_combine(prev, n_bracket, 2, 1, 2, s_tot);
        if (threadIdx.x == 0) *s_st = FermiState{L, H, 0.0, 2.0 * n_rows, 0.0, 0.0, 0.0, 0.0};
    } else {
        const FermiState was = st[pass - 1];
        if (was.done != 0.0) return was;                     // the same in every thread
        node_totals((unsigned)((n_rows + FP_ROWS - 1) / FP_ROWS), prev, s_tot);
        if (threadIdx.x == 0) *s_st = fermi_advance(was, pass - 1, n_rows, n_elec, s_tot, s_tot + 64);
    }
    __syncthreads();
    return *s_st;
}

// One pass.  A row's count at an energy is Clenshaw's recurrence over its 200 or so
// coefficients, one multiply-add after the other, so a pass is as short as the
// loads before it and the nodes beside it allow:
//  * 32 rows' coefficients are staged in LDS, FP_CH terms at a time, every thread's
//    loads in flight at once (a recurrence that loads as it goes waited for memory
//    every few terms), as the terms w_k = (g_(k-2) - g_k) / k;
//  * the block's threads are 32 rows x 8 groups of nodes, so a wave reads each term
//    once per row from LDS, without conflicts;
//  * FUSED: the block first replays the previous pass's decisions itself, from its
//    partials, where those are few enough for every block to read; otherwise
//    k_fermi_pick does so in a launch between the passes.  (A last block that
//    did it at the end of the pass would need a device-scope fence in every block,
//    which writes back L2.)
template <bool FUSED>
__global__ void __launch_bounds__(DT)
k_fermi_pass(int n_rows, int n_exp, int pass, unsigned n_bracket, double n_elec, const double *__restrict__ gs,
             const double *__restrict__ a_inf, const double *__restrict__ b_inf, const double *__restrict__ prev,
             double *__restrict__ part, FermiState *st)
{
    constexpr int NPT = (FT_NODES + FP_GROUPS) / FP_GROUPS;  // nodes per thread
    __shared__ double s_w[FP_CH * FP_ROWS], s_inv[FP_CH], s_part[FP_GROUPS * NPT];
    __shared__ FermiState s_st;
    const unsigned n_rb = (unsigned)((n_rows + FP_ROWS - 1) / FP_ROWS);
    const int row = threadIdx.x & (FP_ROWS - 1), grp = threadIdx.x / FP_ROWS;
    const int r = min((int)blockIdx.x * FP_ROWS + row, n_rows - 1);
    const bool live = (int)blockIdx.x * FP_ROWS + row < n_rows;
    const int K = n_exp + 2, nch = (K + FP_CH - 1) / FP_CH;
    // g_(kb - 1 + FP_RUN grp + t), t = 0 .. FP_RUN + 1, of this thread's row, zero
    // outside 0 .. n_exp, where kb = K - (c + 1) FP_CH: chunk c holds the terms
    // k = kb + 1 .. kb + FP_CH, highest terms first
    double g[FP_RUN + 2];
    auto fetch = [&](int c) {
        const int k0 = K - (c + 1) * FP_CH - 1 + FP_RUN * grp;
        const double *q = gs + (long)k0 * n_rows + r;
#pragma unroll
        for (int t = 0; t < FP_RUN + 2; ++t, q += n_rows) {
            const bool in = k0 + t >= 0 && k0 + t <= n_exp;
            const double v = *(in ? q : gs);
            g[t] = in ? v : 0.0;
        }
    };
    FermiState now;
    if constexpr (FUSED) {
        fetch(0);                                            // comes while the decisions are replayed
        now = fermi_state(pass, n_rows, n_bracket, n_elec, prev, st, s_w, &s_st);
        if (blockIdx.x == 0 && threadIdx.x == 0) st[pass] = now;
        if (now.done != 0.0) return;
    } else {
        now = *st;
        if (now.done != 0.0) return;
        fetch(0);
    }
    const double ai = a_inf[r], bi = b_inf[r], g0 = gs[r];
    // the group's nodes; those past the last repeat it and are not kept
    const int p0 = grp * NPT;
    // sum_k w_k sin(k theta) = sin(theta) sum_k w_k U_(k-1)(cos theta), by
    // Clenshaw's recurrence from the highest term down
    double twoc[NPT], b1[NPT], b2[NPT];
#pragma unroll
    for (int j = 0; j < NPT; ++j) {
        const double eps = (node_energy(now, pass, min(p0 + j, FT_NODES - 1)) - ai) / (2.0 * bi);
        twoc[j] = 2.0 * (eps < -1.0 ? -1.0 : (eps > 1.0 ? 1.0 : eps));
        b1[j] = 0.0;
        b2[j] = 0.0;
    }
    for (int c = 0; c < nch; ++c) {
        const int kb = K - (c + 1) * FP_CH;
        __syncthreads();                                     // the previous terms (or counts) are used
        if (threadIdx.x < FP_CH) s_inv[threadIdx.x] = 1.0 / (double)max(kb + 1 + (int)threadIdx.x, 1);
        __syncthreads();
#pragma unroll
        for (int t = 0; t < FP_RUN; ++t) {
            const int i = FP_RUN * grp + t;
            if (i < FP_CH) s_w[i * FP_ROWS + row] = (g[t] - g[t + 2]) * s_inv[i];
        }
        __syncthreads();
        if (c + 1 < nch) fetch(c + 1);
        const int i0 = max(0, -kb);
#pragma unroll 8
        for (int i = FP_CH - 1; i >= i0; --i) {
            const double wk = s_w[i * FP_ROWS + row];
#pragma unroll
            for (int j = 0; j < NPT; ++j) {
                const double bn = fma(twoc[j], b1[j], wk - b2[j]);
                b2[j] = b1[j];
                b1[j] = bn;
            }
        }
    }
#pragma unroll
    for (int j = 0; j < NPT; ++j) {
        const double cc = 0.5 * twoc[j];
        const double sn = sqrt(fmax(0.0, 1.0 - cc * cc));
        double v = live ? g0 * (1.0 - acos(cc) / M_PI) + sn * b1[j] / M_PI : 0.0;
        for (int o = FP_ROWS / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
        if (row == 0) s_part[grp * NPT + j] = v;
    }
    __syncthreads();
    if (threadIdx.x < FT_NODES) part[threadIdx.x * ft_pitch(n_rb) + blockIdx.x] = s_part[threadIdx.x];
}

// The pass over so many rows that the chip is full: two lanes share an orbital row,
// lane h of the pair taking nodes 8h .. 8h+7 (the last lane 7 nodes), both reading
// the same coefficients as they go; no LDS copy and an eighth of the waves' starts
// and ends per row.  Partials of 128 rows.
constexpr int FT_HALF = (FT_NODES + 1) / 2;

__global__ void __launch_bounds__(DT)
k_fermi_tree(int n_rows, int n_exp, int pass, const double *__restrict__ gs, const double *__restrict__ a_inf,
             const double *__restrict__ b_inf, double *__restrict__ part, const FermiState *st)
{
    __shared__ double s_inv[1040], s_red[FT_NODES * (DT / 64)], s_mid[FT_NODES];
    if (st->done != 0.0) return;
    // by every lane for its own nodes: 44 against 40 us a pass, 320,000 rows, 10 terms
    if (threadIdx.x < FT_NODES) s_mid[threadIdx.x] = node_energy(*st, pass, threadIdx.x);
    for (int k = threadIdx.x; k <= n_exp + 2; k += blockDim.x) s_inv[k] = k ? 1.0 / k : 0.0;
    __syncthreads();
    const long gt = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const int r = (int)(gt >> 1), h = (int)(gt & 1);
    double cnt[FT_HALF];
    if (r < n_rows) {
        const double ai = a_inf[r], bi = b_inf[r];
        // only 2 cos(theta) and the two Clenshaw terms per node stay live in
        // the loop (the midpoints, sin(theta) and the arccos term are formed
        // before and after it), which keeps the kernel's registers low
        double twoc[FT_HALF], b1[FT_HALF], b2[FT_HALF];
        {
#pragma unroll
            for (int j = 0; j < FT_HALF; ++j) {
                const int p = h * FT_HALF + j < FT_NODES ? h * FT_HALF + j : FT_NODES - 1;
                double eps = (s_mid[p] - ai) / (2.0 * bi);
                twoc[j] = 2.0 * (eps < -1.0 ? -1.0 : (eps > 1.0 ? 1.0 : eps));
                b1[j] = 0.0;
                b2[j] = 0.0;
            }
        }
        // sum_k w_k sin(k theta) = sin(theta) sum_k w_k U_(k-1)(cos theta), by
        // Clenshaw's recurrence from the highest term down; w_k = (g_(k-2) - g_k) / k
        // (w_1 = -g_1), with g_k = 0 beyond n_exp
        double gk = 0.0, gkm1 = 0.0;
#pragma unroll 8
        for (int k = n_exp + 2; k >= 1; --k) {
            const double gkm2 = (k >= 2) ? gs[(long)(k - 2) * n_rows + r] : 0.0;
            const double wk = ((k >= 2) ? (gkm2 - gk) : -gk) * s_inv[k];
            gk = gkm1;
            gkm1 = gkm2;
#pragma unroll
            for (int j = 0; j < FT_HALF; ++j) {
                const double bn = fma(twoc[j], b1[j], wk - b2[j]);
                b2[j] = b1[j];
                b1[j] = bn;
            }
        }
        const double g0 = gs[r];
#pragma unroll
        for (int j = 0; j < FT_HALF; ++j) {
            const double c = 0.5 * twoc[j];
            const double sn = sqrt(fmax(0.0, 1.0 - c * c));
            cnt[j] = g0 * (1.0 - acos(c) / M_PI) + sn * b1[j] / M_PI;
        }
    } else {
#pragma unroll
        for (int j = 0; j < FT_HALF; ++j) cnt[j] = 0.0;
    }
    {
        double v[FT_NODES];
#pragma unroll
        for (int p = 0; p < FT_NODES; ++p) v[p] = (h == p / FT_HALF) ? cnt[p % FT_HALF] : 0.0;
        const double t = block_sum_n<FT_NODES>(v, s_red);
        if (threadIdx.x < FT_NODES) part[threadIdx.x * (size_t)gridDim.x + blockIdx.x] = t;
    }
}

// The decisions of a pass whose partials are many, in a launch of its own (one
// block): every node's sums (Q partials in turn) in a fixed order, thread t of DT
// taking sums t, t + DT, ..., then the fixed tree.  The nodes are dealt to FT_PICK such
// sets of threads, and a thread's loads are in flight together: one block waits for
// memory, not for its bandwidth.  AHEAD such loads: as many as there are sums for (eight
// where one will do took 6.3 us against 4.4, 50,000 rows).
constexpr int FT_PICK = 4;

template <int Q, int AHEAD>
__global__ void __launch_bounds__(FT_PICK * DT)
k_fermi_pick(unsigned n_rb, int pass, int n_rows, double n_elec, const double *__restrict__ part, FermiState *st)
{
    constexpr int NPT = (FT_NODES + FT_PICK - 1) / FT_PICK, NW = DT / 64;
    __shared__ double s_red[FT_PICK][NPT * NW], s_tot[FT_PICK * NPT], s_v[FT_NODES + 2];
    const FermiState was = *st;                              // comes while the partials do
    if (was.done != 0.0) return;
    const unsigned t = threadIdx.x % DT, set = threadIdx.x / DT, n = (n_rb + Q - 1) / Q;
    const size_t pitch = Q == 1 ? n_rb : ft_pitch(n_rb);
    double acc[NPT];
#pragma unroll
    for (int p = 0; p < NPT; ++p) acc[p] = 0.0;
    for (unsigned q0 = t; q0 < n; q0 += AHEAD * DT) {
        double x[AHEAD][NPT][Q];
#pragma unroll
        for (int i = 0; i < AHEAD; ++i)
#pragma unroll
            for (int p = 0; p < NPT; ++p)
#pragma unroll
                for (unsigned e = 0; e < Q; ++e)
                    x[i][p][e] = part[min((int)set * NPT + p, FT_NODES - 1) * pitch + min(Q * (q0 + i * DT) + e, n_rb - 1)];
#pragma unroll
        for (int i = 0; i < AHEAD; ++i)
#pragma unroll
            for (int p = 0; p < NPT; ++p) {
                double v = 0.0;
#pragma unroll
                for (unsigned e = 0; e < Q; ++e) v += Q * (q0 + i * DT) + e < n_rb ? x[i][p][e] : 0.0;
                acc[p] += v;
            }
    }
#pragma unroll
    for (int p = 0; p < NPT; ++p)
        for (int o = 32; o > 0; o >>= 1) acc[p] += __shfl_xor(acc[p], o);
    if ((t & 63) == 0) {
#pragma unroll
        for (int p = 0; p < NPT; ++p) s_red[set][p * NW + (t >> 6)] = acc[p];
    }
    __syncthreads();
    if (t < NPT) {
        double v = 0.0;
        for (int q = 0; q < NW; ++q) v += s_red[set][t * NW + q];
        s_tot[set * NPT + t] = v;
    }
    __syncthreads();
    if (threadIdx.x == 0) *st = fermi_advance(was, pass, n_rows, n_elec, s_tot, s_v);
}

// The level, by one block: where the blocks replay the decisions, after the last pass's
// (prev: its partials; else NULL).
__global__ void __launch_bounds__(DT)
k_fermi_finish(int n_rows, int pass, double n_elec, const double *__restrict__ prev, const FermiState *st, double *E_F)
{
    __shared__ double s_tot[96];
    __shared__ FermiState s_st;
    const FermiState now = prev ? fermi_state(pass, n_rows, 0, n_elec, prev, st, s_tot, &s_st) : *st;
    if (threadIdx.x == 0) E_F[0] = 0.5 * (now.lo + now.hi);
}

// Rows up to which k_fermi_pass makes the search's passes, k_fermi_tree beyond; fewer where
// the expansions are short: the pass stages 202 terms or none, three blocks to a CU, and
// a block's time passes for every 768 blocks or part of them (rounds).  Whole
// tails bisecting all the way, pass form and tree: 24,000 rows, 10 terms 233 and 226 us, 25
// terms 242 and 248; 41,000 rows, 50 terms 391 and 359, 75 terms 412 and 431; 57,000 rows, 75
// terms 471 and 447, 100 terms 516 and 518; 65,500 rows, 150 terms 654 and 628, 200 terms 745
// and 768.
constexpr long FT_SPREAD = 65536, FT_RESIDENT = 3 * 256 * FP_ROWS;

static bool pass_form(long n_rows, int n_exp)
{
    if (n_rows <= FT_FUSED) return true;
    const long rounds = (n_rows + FT_RESIDENT - 1) / FT_RESIDENT;
    return n_rows <= FT_SPREAD && n_exp >= (rounds <= 1 ? 20 : (rounds == 2 ? 64 : 128));
}
// Passes of a search: every halving of plain bisection.  Passes that find the bracket
// closed cost a small structure 35 us of its tail.  (One block doing what is left instead
// saves those, but takes 1.1 ms for 1000 rows with a gap, where they take 0.2 and
// bisecting all the way took 0.67.)
constexpr int FT_PASSES = FT_MAX_HALVINGS / FT_LEVELS;

// The search.  Up to FT_FUSED rows, two trees of sums per node, each block replays the
// previous decisions and `states` holds every pass's state.  `tree` holds the 32-row
// partials of two passes in turn; NULL where not pass_form and where the
// caller's workspace has no room for it.
static void fermi_search(int n_rows, int n_exp, double n_elec, const double *gs, const double *a_inf,
                         const double *b_inf, unsigned n_bracket, double *part, double *tree, FermiState *st,
                         FermiState *states, double *E_F, hipStream_t stream)
{
    const unsigned n_rb = (unsigned)((n_rows + FP_ROWS - 1) / FP_ROWS), n_tb = (unsigned)((2L * n_rows + DT - 1) / DT);
    if (tree && n_rows <= FT_FUSED) {
        double *buf[2] = {tree, tree + ft_pitch(n_rb) * (FT_NODES + 1)};
        for (int it = 0; it < FT_PASSES; ++it)
            k_fermi_pass<true><<<n_rb, DT, 0, stream>>>(n_rows, n_exp, it, n_bracket, n_elec, gs, a_inf, b_inf,
                                                        it ? buf[(it - 1) & 1] : part, buf[it & 1], states);
        k_fermi_finish<<<1, DT, 0, stream>>>(n_rows, FT_PASSES, n_elec, buf[(FT_PASSES - 1) & 1], states, E_F);
        return;
    }
    k_bracket_pick<<<1, DT, 0, stream>>>(n_rows, n_bracket, part, st);
    for (int it = 0; it < FT_PASSES; ++it) {
        if (tree) {
            k_fermi_pass<false><<<n_rb, DT, 0, stream>>>(n_rows, n_exp, it, 0, n_elec, gs, a_inf, b_inf, nullptr, tree,
                                                         st);
            auto *pick = n_rb <= 4 * DT ? k_fermi_pick<4, 1> : k_fermi_pick<4, 2>;
            pick<<<1, FT_PICK * DT, 0, stream>>>(n_rb, it, n_rows, n_elec, tree, st);
        } else {
            k_fermi_tree<<<n_tb, DT, 0, stream>>>(n_rows, n_exp, it, gs, a_inf, b_inf, part, st);
            auto *pick = n_tb <= DT ? k_fermi_pick<1, 1> : (n_tb <= 2 * DT ? k_fermi_pick<1, 2> : k_fermi_pick<1, 8>);
            pick<<<1, FT_PICK * DT, 0, stream>>>(n_tb, it, n_rows, n_elec, part, st);
        }
    }
    k_fermi_finish<<<1, DT, 0, stream>>>(n_rows, FT_PASSES, n_elec, nullptr, st, E_F);
}

// per-atom N, U, n(E_F) and block partials of U.  Where rows are few, a row's sums over
// its 200 or so terms are split over SEGS = 4 threads, each starting its run of terms from
// its own power of the rotation: a single thread per row waits for one memory access after
// another and for one rotation after another.  Where the rows fill the chip the runs'
// starts (square roots, arccosines, powers) are work on top, and a thread takes a row.
// Either way a run's coefficients are loaded EN_RUN at a time, all in flight, and summed
// among themselves first (N of 201 terms: 1.6e-16 from its value in the mean with one run or
// four, 4e-16 as one chain).  An atom's orbitals are then added in orbital order, as a per-atom loop would add them.
// 200 terms, four runs: 128 atoms 69 -> 8 us, 8192 atoms 75 -> 19 (one run: 27; eight: 28).
constexpr int EN_RUN = 13;                       // coefficients loaded at once
// Atoms per block: one run, 9 orbitals, 30,000 atoms, 75 terms 35 us with 64 (nine whole
// waves), 46 with 32; 5 orbitals, 40,000 atoms 37 with 64, 25 with 32.
__host__ __device__ constexpr int en_atoms(int no, int segs)
{
    return segs == 4 ? (no <= 2 ? 16 : 8) : (no > 4 && no < 9 ? 32 : 64);
}
constexpr int EN_FOUR = 8 * 9 * 4, EN_ONE = 32 * 8, EN_ONE9 = 64 * 9;     // most threads of a block
// One run from EN_FULL rows on, for long expansions from EN_MEMORY on.  Expansion and sums
// together, one against four runs: 9 orbitals, 270,000 rows, 25 terms 60 and 101 us, 75
// terms 130 and 176, 200 terms 349 and 382; 5 orbitals, 100,000 rows, 25 terms 38 and 44,
// 200 terms 155 and 154; 200,000 rows, 200 terms 301 and 289 (while the coefficients come
// from the cache, four runs' loads are worth their starts); 40,960 rows, 25 terms 26 and 29;
// 10,000 rows, 150 terms 40 and 33.
constexpr long EN_FULL = 32768, EN_MEMORY = 250000;
constexpr int EN_SHORT = 160;
constexpr int EN_TAB = 3 + 4 + EN_RUN;           // table entries past n_exp that the last run can reach

template <int SEGS, int MAXT>
__global__ void __launch_bounds__(MAXT)
k_energy(int n_atoms, int no, int n_exp, double wt, const double *__restrict__ gs, const double *__restrict__ a_inf,
         const double *__restrict__ b_inf, const double *__restrict__ H_on, const double *__restrict__ E_F,
         double *__restrict__ N_atom, double *__restrict__ U_atom, double *__restrict__ dos_atom,
         int *__restrict__ flags, double *__restrict__ part)
{
    __shared__ double s_inv[1024 + EN_TAB], s_s[3][MAXT];
    const int EA = en_atoms(no, SEGS), RB = EA * no;
    const int row = threadIdx.x % RB, seg = threadIdx.x / RB;
    const long n_rows = (long)n_atoms * no;
    const long r = (long)blockIdx.x * RB + row;
    const bool live = r < n_rows;
    const long rr = live ? r : n_rows - 1;
    const int T = (n_exp + SEGS) / SEGS;         // of the n_exp + 1 terms, per run
    const int m0 = seg * T, m1 = min(m0 + T, n_exp + 1);
    double g[EN_RUN];
    auto fetch = [&](int m) {
#pragma unroll
        for (int t = 0; t < EN_RUN; ++t) {
            const double v = gs[(long)min(m + t, n_exp) * n_rows + rr];
            g[t] = m + t < m1 ? v : 0.0;
        }
    };
    fetch(m0);
    const double E = E_F[0], ai = a_inf[rr], bi = b_inf[rr];
    for (int k = threadIdx.x; k < n_exp + EN_TAB; k += blockDim.x) s_inv[k] = k ? 1.0 / k : 0.0;
    const double eps = (E - ai) / (2.0 * bi);
    const double c = eps < -1.0 ? -1.0 : (eps > 1.0 ? 1.0 : eps);
    const double s = sqrt(fmax(0.0, 1.0 - c * c));
    const double c2 = c * c - s * s, s2 = 2.0 * c * s;
    // pi chi^_1, chi^_(m+2) = (sin((m+3) phi)/(m+3) - sin((m+1) phi)/(m+1)) / pi
    const double x1 = (M_PI - acos(c)) + 0.5 * s2;
    // (cos, sin)(m0 phi) by squarings
    double C = 1.0, S = 0.0;
    {
        double pc = c, ps = s;
        for (int e = m0; e; e >>= 1) {
            if (e & 1) {
                const double t = C * pc - S * ps;
                S = S * pc + C * ps;
                C = t;
            }
            const double t = pc * pc - ps * ps;
            ps = 2.0 * pc * ps;
            pc = t;
        }
    }
    __syncthreads();
    // sin((m+1) phi), sin((m+2) phi) and (cos, sin)((m+3) phi), advanced by
    // unit-modulus rotation; pi chi^_m, pi chi^_(m+1) carried along
    double w1 = S * c + C * s, w2 = S * c2 + C * s2;
    double c3 = (C * c2 - S * s2) * c - w2 * s, w3 = w2 * c + (C * c2 - S * s2) * s;
    double chi0 = m0 == 0 ? 0.0 : (m0 == 1 ? x1 : w1 * s_inv[m0 + 1] - (S * c - C * s) * s_inv[max(m0 - 1, 0)]);
    double chi1 = m0 == 0 ? x1 : w2 * s_inv[m0 + 2] - S * s_inv[m0];
    double N = 0.0, U = 0.0, D = 0.0;
    for (int mb = m0;;) {
        double n = 0.0, u = 0.0, d = 0.0;
#pragma unroll
        for (int t = 0; t < EN_RUN; ++t) {
            const int m = mb + t;
            const double chi2 = w3 * s_inv[m + 3] - w1 * s_inv[m + 1];
            n = fma(g[t], chi1, n);
            u = fma(g[t], chi2 + chi0, u);
            d = fma(g[t], w1, d);
            chi0 = chi1;
            chi1 = chi2;
            const double nc = c3 * c - w3 * s, ns = w3 * c + c3 * s;
            w1 = w2; w2 = w3; w3 = ns; c3 = nc;
        }
        N += n;
        U += u;
        D += d;
        mb += EN_RUN;
        if (mb - m0 >= T) break;                 // the same for every thread
        fetch(mb);
    }
    s_s[0][threadIdx.x] = N;
    s_s[1][threadIdx.x] = U;
    s_s[2][threadIdx.x] = D;
    __syncthreads();
    if (seg == 0) {
        for (int q = 1; q < SEGS; ++q) {
            N += s_s[0][q * RB + row];
            U += s_s[1][q * RB + row];
            D += s_s[2][q * RB + row];
        }
        N /= M_PI;
        U = bi * (U / M_PI) + (ai - H_on[rr]) * N;
        D = (eps > -1.0 && eps < 1.0) ? D / (M_PI * bi) : 0.0;
        if (live && !(eps > -1.0 && eps < 1.0)) flags[r] |= BOP_FLAG_OUTSIDE;
        s_s[0][row] = N;
        s_s[1][row] = U;
        s_s[2][row] = D;
    }
    __syncthreads();
    const int t = threadIdx.x;
    const long i = (long)blockIdx.x * EA + t;
    double Ui = 0.0;
    if (t < EA && i < n_atoms) {
        double sN = 0.0, sU = 0.0, sD = 0.0;
        for (int a = 0; a < no; ++a) {
            sN += s_s[0][t * no + a];
            sU += s_s[1][t * no + a];
            sD += s_s[2][t * no + a];
        }
        // both spins; wt orbitals per row in the atom-averaged mode
        N_atom[i] = 2.0 * wt * sN;
        U_atom[i] = 2.0 * wt * sU;
        dos_atom[i] = 2.0 * wt * sD;
        Ui = 2.0 * wt * sU;
    }
    // the block's atoms are in its first wave (a block may end in part of a wave, so
    // sums over its waves would need a slot for that one too)
    static_assert(en_atoms(1, SEGS) <= 64 && en_atoms(9, SEGS) <= 64, "one wave holds a block's atoms");
    for (int o = 32; o > 0; o >>= 1) Ui += __shfl_xor(Ui, o);
    if (t == 0) part[blockIdx.x] = Ui;
}

// total U from the block partials (one block, fixed order)
__global__ void __launch_bounds__(DT)
k_energy_total(unsigned n_blocks, const double *__restrict__ part, double *__restrict__ U_total)
{
    __shared__ double s_red[DT / 64];
    const double tot = partials_combine(part, n_blocks, 1, 0, 0, s_red);
    if (threadIdx.x == 0) U_total[0] = tot;
}

struct EnergyWs {
    double *gs, *part;
    FermiState *st;
    size_t bytes;           // what every call needs
    double *tree;           // the Fermi passes' 32-row partials (two passes in turn) and states, where n_rows <= FT_SPREAD
    FermiState *states;
    size_t bytes_tree;      // with these
};

EnergyWs carve(void *base, long n_rows, int n_exp)
{
    EnergyWs w{};
    char *p = (char *)base;
    auto take = [&](size_t b) { char *r = p; p += align_up(b, 256); return (void *)r; };
    w.gs = (double *)take(sizeof(double) * (size_t)(n_exp + 1) * (size_t)n_rows);
    long nblk = 2 * ((n_rows + DT - 1) / DT) + 1;       // 128-row sums of the 15 nodes of four halvings
    w.part = (double *)take(sizeof(double) * 15 * (size_t)nblk);
    w.st = (FermiState *)take(sizeof(FermiState));
    w.bytes = (size_t)(p - (char *)base);
    if (n_rows <= FT_SPREAD) {
        const size_t rb = ft_pitch((unsigned)((n_rows + FP_ROWS - 1) / FP_ROWS));
        w.tree = (double *)take(sizeof(double) * 2 * rb * (FT_NODES + 1));
        w.states = (FermiState *)take(sizeof(FermiState) * FT_PASSES);
    }
    w.bytes_tree = (size_t)(p - (char *)base);
    return w;
}

}  // namespace
}  // namespace bop

using namespace bop;

extern "C" int bop_recursion(int n_rows, int n_max, const double *mu, int bw_mode, double a_glob,
                             double b_glob, double *a, double *b, double *a_inf, double *b_inf,
                             int *flags, hipStream_t stream)
{
    BOP_REQUIRE(n_rows >= 0, BOP_E_ARG, "bop_recursion: n_rows < 0");
    BOP_REQUIRE(n_max >= 1 && n_max <= MAX_NMAX, BOP_E_UNSUPPORTED, "bop_recursion: n_max must be 1..%d", MAX_NMAX);
    BOP_REQUIRE(bw_mode >= BOP_BW_GERSHGORIN && bw_mode <= BOP_BW_WEIGHTED, BOP_E_ARG,
                "bop_recursion: bw_mode must be %d..%d", BOP_BW_GERSHGORIN, BOP_BW_WEIGHTED);
    BOP_REQUIRE(bw_mode != BOP_BW_WEIGHTED || a_glob >= 0.0, BOP_E_ARG, "bop_recursion: weighted beta must be >= 0");
    if (n_rows == 0) return BOP_OK;
    BOP_REQUIRE(a && b && a_inf && b_inf && flags, BOP_E_ARG, "bop_recursion: NULL array");
    // the register kernel covers Gershgorin and the global values; the other
    // estimates read the chain back from a and b in the generic kernel
    if (mu && n_max <= 20 && bw_mode <= BOP_BW_GLOBAL)
        k_recursion_reg<20><<<(n_rows + DT - 1) / DT, DT, 0, stream>>>(n_rows, n_max, mu, bw_mode, a_glob, b_glob,
                                                                       a, b, a_inf, b_inf, flags);
    else
    k_recursion<<<(n_rows + DT - 1) / DT, DT, 0, stream>>>(n_rows, n_max, mu, bw_mode, a_glob, b_glob, a, b,
                                                           a_inf, b_inf, flags);
    BOP_LAUNCHED();
    return BOP_OK;
}

extern "C" size_t bop_energy_workspace_size(int n_atoms, int n_orb, int n_exp)
{
    if (n_atoms < 0 || n_orb <= 0 || n_exp < 0) return 0;
    return carve(nullptr, (long)n_atoms * n_orb, n_exp).bytes_tree + 256;
}

// wt: orbitals each row stands for (1; n_orb in the atom-averaged mode, where
// a row is an atom's averaged chain): the Fermi search counts wt 2 N per row
// and the per-atom outputs are scaled by wt.
static int energy_impl(int n_atoms, int no, int n_max, int n_exp, const double *mu, const double *a,
                       const double *b, const double *a_inf, const double *b_inf, const double *H_on,
                       double n_elec, int ef_mode, double *E_F, double *N_atom, double *U_atom,
                       double *dos_atom, double *U_total, int *flags, void *ws, size_t ws_bytes,
                       hipStream_t stream, double wt = 1.0)
{
    BOP_REQUIRE(n_atoms > 0 && no > 0, BOP_E_ARG, "bop_energy: n_atoms and n_orb must be > 0");
    BOP_REQUIRE(no <= 9, BOP_E_UNSUPPORTED, "bop_energy: at most 9 orbitals per atom");
    BOP_REQUIRE(n_max >= 1 && n_max <= MAX_NMAX, BOP_E_UNSUPPORTED, "bop_energy: n_max must be 1..%d", MAX_NMAX);
    BOP_REQUIRE(n_exp >= 1 && n_exp <= 1024, BOP_E_UNSUPPORTED, "bop_energy: n_exp must be 1..1024");
    BOP_REQUIRE(ef_mode == 0 || ef_mode == 1, BOP_E_ARG, "bop_energy: ef_mode must be 0 or 1");
    BOP_REQUIRE(a && b && a_inf && b_inf && H_on && E_F && N_atom && U_atom && dos_atom && U_total && flags,
                BOP_E_ARG, "bop_energy: NULL array");
    const long R = (long)n_atoms * no;
    EnergyWs w = carve(ws, R, n_exp);
    BOP_REQUIRE(ws && ws_bytes >= w.bytes, BOP_E_CAPACITY, "bop_energy: workspace of %zu bytes needed", w.bytes);
    BOP_REQUIRE(ef_mode == 1 || (n_elec >= 0.0 && n_elec <= 2.0 * wt * (double)R), BOP_E_ARG,
                "bop_energy: n_elec outside [0, 2 n_rows]");
    const unsigned nblk = (unsigned)((R + DT - 1) / DT);
    const int L = (n_max - 1) / 2 + 1 > n_max / 2 ? (n_max - 1) / 2 + 1 : n_max / 2;
    if (n_max <= CL_NMAX && R <= CL_ROWS)
        k_dos_coeffs_lanes<<<(unsigned)((R + CR - 1) / CR), DT, 0, stream>>>((int)R, n_max, n_exp, mu, a, b, a_inf, b_inf,
                                                                             w.gs, flags);
    else if (L <= 11) k_dos_coeffs<11><<<nblk, DT, 0, stream>>>((int)R, n_max, n_exp, mu, a, b, a_inf, b_inf, w.gs, flags);
    else k_dos_coeffs<21><<<nblk, DT, 0, stream>>>((int)R, n_max, n_exp, mu, a, b, a_inf, b_inf, w.gs, flags);
    BOP_LAUNCHED();
    if (ef_mode == 0) {
        k_bracket<<<nblk, DT, 0, stream>>>((int)R, a_inf, b_inf, w.part);
        // a workspace without the tree's partials (of the size earlier versions asked
        // for, or the fixed array at its limit) takes the route of many rows
        const double ne = n_elec / wt;
        const bool tree = pass_form(R, n_exp) && ws_bytes >= w.bytes_tree;
        fermi_search((int)R, n_exp, ne, w.gs, a_inf, b_inf, nblk, w.part, tree ? w.tree : nullptr, w.st, w.states, E_F,
                     stream);
        BOP_LAUNCHED();
    }
    const int segs = R >= EN_FULL && (n_exp < EN_SHORT || R >= EN_MEMORY) ? 1 : 4, ea = en_atoms(no, segs);
    const unsigned ablk = (unsigned)((n_atoms + ea - 1) / ea);
    auto *energy = segs == 4 ? k_energy<4, EN_FOUR> : (no < 9 ? k_energy<1, EN_ONE> : k_energy<1, EN_ONE9>);
    energy<<<ablk, ea * no * segs, 0, stream>>>(n_atoms, no, n_exp, wt, w.gs, a_inf, b_inf, H_on, E_F, N_atom, U_atom,
                                                dos_atom, flags, w.part);
    k_energy_total<<<1, DT, 0, stream>>>(ablk, w.part, U_total);
    BOP_LAUNCHED();
    return BOP_OK;
}

extern "C" int bop_energy(int n_atoms, int no, int n_max, int n_exp, const double *mu, const double *a,
                          const double *b, const double *a_inf, const double *b_inf, const double *H_on,
                          double n_elec, int ef_mode, double *E_F, double *N_atom, double *U_atom,
                          double *dos_atom, double *U_total, int *flags, void *ws, size_t ws_bytes,
                          hipStream_t stream)
{
    return energy_impl(n_atoms, no, n_max, n_exp, mu, a, b, a_inf, b_inf, H_on, n_elec, ef_mode, E_F, N_atom,
                       U_atom, dos_atom, U_total, flags, ws, ws_bytes, stream);
}

// Atom-averaged mode: one chain per atom from mu_i / n_orb.
__global__ void __launch_bounds__(DT)
k_atom_average(int n_atoms, int no, int n_max, const double *__restrict__ mu, const double *__restrict__ H_on,
               double *__restrict__ mu_avg, double *__restrict__ H_avg)
{
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const int M = n_max + 1;
    if (e >= (long)n_atoms * M) return;
    const long i = e / M;
    const int n = (int)(e % M);
    double s = 0.0;
    for (int a = 0; a < no; ++a) s += mu[(i * no + a) * M + n];
    mu_avg[e] = s / no;
    if (n == 0) {
        double h = 0.0;
        for (int a = 0; a < no; ++a) h += H_on[i * no + a];
        H_avg[i] = h / no;
    }
}

extern "C" int bop_atom_average(int n_atoms, int n_orb, int n_max, const double *mu, const double *H_on,
                                double *mu_avg, double *H_avg, hipStream_t stream)
{
    BOP_REQUIRE(n_atoms >= 0 && n_orb > 0 && n_max >= 0 && n_max <= MAX_NMAX, BOP_E_ARG,
                "bop_atom_average: bad sizes");
    if (n_atoms == 0) return BOP_OK;
    BOP_REQUIRE(mu && H_on && mu_avg && H_avg, BOP_E_ARG, "bop_atom_average: NULL array");
    const long ne = (long)n_atoms * (n_max + 1);
    k_atom_average<<<(unsigned)((ne + DT - 1) / DT), DT, 0, stream>>>(n_atoms, n_orb, n_max, mu, H_on, mu_avg, H_avg);
    BOP_LAUNCHED();
    return BOP_OK;
}

extern "C" int bop_energy_atom_averaged(int n_atoms, int n_orb, int n_max, int n_exp, const double *mu_avg,
                                        const double *a, const double *b, const double *a_inf,
                                        const double *b_inf, const double *H_avg, double n_elec, int ef_mode,
                                        double *E_F, double *N_atom, double *U_atom, double *dos_atom,
                                        double *U_total, int *flags, void *ws, size_t ws_bytes, hipStream_t stream)
{
    BOP_REQUIRE(n_orb > 0, BOP_E_ARG, "bop_energy_atom_averaged: n_orb must be > 0");
    return energy_impl(n_atoms, 1, n_max, n_exp, mu_avg, a, b, a_inf, b_inf, H_avg, n_elec, ef_mode, E_F, N_atom,
                       U_atom, dos_atom, U_total, flags, ws, ws_bytes, stream, (double)n_orb);
}

// ---------------------------------------------------------------------------
// bop_energy without a caller workspace: the expansion coefficients, block
// partials and Fermi state live in a fixed device array of
// BOP_ENERGY_NOALLOC_BYTES, one copy per GPU the library runs on, held until
// the process ends.  Nothing in it must start at zero: every kernel writes the
// part of the workspace it reads before reading it.  Calls that overlap on one
// GPU (several streams or threads) share the array and race.
// ---------------------------------------------------------------------------
static __device__ __align__(256) char scratch[BOP_ENERGY_NOALLOC_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
std::mutex scratch_mu;
void *scratch_ptr[MAX_DEVICES];     // the array's device address on each GPU (NULL: not looked up yet)
}  // namespace

// The device address of `scratch` on the current GPU, looked up once per GPU
// with that GPU current.  The array's name in host code is only a host-side
// handle, never a device address.
static int scratch_address(void **out)
{
    int dev = -1;
    BOP_HIP(hipGetDevice(&dev));
    BOP_REQUIRE(dev >= 0 && dev < MAX_DEVICES, BOP_E_UNSUPPORTED, "bop_energy_noalloc: device %d out of range", dev);
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (!scratch_ptr[dev]) {
        void *p = nullptr;
        BOP_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        BOP_REQUIRE(p, BOP_E_HIP, "bop_energy_noalloc: no device address for the scratch array");
        scratch_ptr[dev] = p;
    }
    *out = scratch_ptr[dev];
    return BOP_OK;
}

extern "C" int bop_energy_noalloc(int n_atoms, int no, int n_max, int n_exp, const double *mu, const double *a,
                                  const double *b, const double *a_inf, const double *b_inf, const double *H_on,
                                  double n_elec, int ef_mode, double *E_F, double *N_atom, double *U_atom,
                                  double *dos_atom, double *U_total, int *flags, hipStream_t stream)
{
    BOP_REQUIRE(n_atoms > 0 && no > 0 && n_exp >= 0, BOP_E_ARG, "bop_energy_noalloc: n_atoms and n_orb must be > 0");
    const size_t need = carve(nullptr, (long)n_atoms * no, n_exp).bytes;
    BOP_REQUIRE(need <= BOP_ENERGY_NOALLOC_BYTES, BOP_E_CAPACITY,
                "bop_energy_noalloc: %d atoms x %d orbitals at n_exp %d need %zu bytes of scratch, more than its "
                "fixed %llu; use bop_energy with a caller workspace",
                n_atoms, no, n_exp, need, (unsigned long long)BOP_ENERGY_NOALLOC_BYTES);
    void *ws = nullptr;
    const int rc = scratch_address(&ws);
    if (rc != BOP_OK) return rc;
    return energy_impl(n_atoms, no, n_max, n_exp, mu, a, b, a_inf, b_inf, H_on, n_elec, ef_mode, E_F, N_atom,
                       U_atom, dos_atom, U_total, flags, ws, BOP_ENERGY_NOALLOC_BYTES, stream);
}

namespace bop {
double *energy_ws_scratch(void *ws, long n_rows, int n_exp)
{
    return carve(ws, n_rows, n_exp).part;
}
}  // namespace bop
