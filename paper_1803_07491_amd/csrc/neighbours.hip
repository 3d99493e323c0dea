// Periodic neighbour list on the GPU (Sec. II "Initialisation" of
// arXiv:1803.07491: pairs within the cutoff found through cell lists, the
// ghost cells of the paper expressed as explicit integer image shifts S).
//
// Atoms are binned into a grid of cells at least r_cut wide (in fractional
// coordinates along each reciprocal direction), cells numbered in 2x2x2
// blocks.  The atom order emitted for moment tiles follows a Hilbert curve
// over a grid three times finer (index order inside a grid cell): consecutive
// atoms then form compact groups, whose union of k-hop neighbourhoods is ~5%
// smaller than for groups taken in cell-list order.  Each atom then scans the 27 neighbouring
// cells; the image shift of a candidate follows from the cell wrap and the
// atoms' integer offsets.  If some axis has fewer than three cells, every atom
// scans all atoms and all image shifts that can reach the cutoff.
//
// The pair vector and the criterion are evaluated in one fixed operation
// order in FP64 with contraction disabled for this file, so the list is
// bit-exact; rows are sorted by (j, s1, s2, s3).
#include "bop_internal.h"

#include <cmath>

namespace bop {
namespace {

struct Geom {
    double A[9];      // rows a1, a2, a3
    double Ai[9];     // inverse: f = r . Ai
    double gn[3];     // |column k of Ai| = 1 / plane spacing
    int nc[3];        // cells per axis
    int nb[3];        // 2x2x2 blocks per axis
    int nt[3];        // tile-order grid per axis (Hilbert curve of tb bits per axis)
    int tb;
    double rc, rc2;
    int all_pairs;    // 1: brute-force over atoms and shifts
};

__host__ __device__ inline int bin_of_cell(const Geom &g, int c0, int c1, int c2)
{
    int blk = ((c0 >> 1) * g.nb[1] + (c1 >> 1)) * g.nb[2] + (c2 >> 1);
    return blk * 8 + ((c0 & 1) << 2) + ((c1 & 1) << 1) + (c2 & 1);
}

// d = (r_j - r_i) + ((s1 a1 + s2 a2) + s3 a3);  accepted when 0 < |d|^2 < rc^2
__device__ inline bool pair_vec(const Geom &g, const double *__restrict__ pos, int i, int j,
                                int s1, int s2, int s3, double d[3])
{
    for (int k = 0; k < 3; ++k) {
        double sv = ((double)s1 * g.A[k] + (double)s2 * g.A[3 + k]) + (double)s3 * g.A[6 + k];
        d[k] = (pos[3 * j + k] - pos[3 * i + k]) + sv;
    }
    double r2 = (d[0] * d[0] + d[1] * d[1]) + d[2] * d[2];
    return r2 > 0.0 && r2 < g.rc2;
}

__global__ void k_fill_int(int *p, long n, int v)
{
    long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// 3-D Hilbert index of (x0, x1, x2), b bits each (Skilling's transpose
// method: undo the excess work per bit plane, Gray-encode, interleave).
__device__ inline unsigned hilbert3(unsigned x0, unsigned x1, unsigned x2, int b)
{
    unsigned X[3] = {x0, x1, x2};
    const unsigned M = 1u << (b - 1);
    for (unsigned Q = M; Q > 1; Q >>= 1) {
        const unsigned P = Q - 1;
        for (int i = 0; i < 3; ++i) {
            if (X[i] & Q) X[0] ^= P;
            else {
                const unsigned t = (X[0] ^ X[i]) & P;
                X[0] ^= t;
                X[i] ^= t;
            }
        }
    }
    X[1] ^= X[0];
    X[2] ^= X[1];
    unsigned t = 0;
    for (unsigned Q = M; Q > 1; Q >>= 1)
        if (X[2] & Q) t ^= Q - 1;
    for (int i = 0; i < 3; ++i) X[i] ^= t;
    unsigned code = 0;
    for (int bit = b - 1; bit >= 0; --bit)
        for (int i = 0; i < 3; ++i) code = (code << 1) | ((X[i] >> bit) & 1u);
    return code;
}

// Cells and, with `key`, the tile-order keys (Hilbert index of the atom's cell in the
// fine grid) and how many atoms each holds.  Bins and keys are numbered in one
// sequence, bins first, so that one scan, one fill and one sort serve both: the list of
// a small structure costs its launches (19 -> 9, 152 -> 100 us for 128 atoms).
__global__ void k_bin_atoms(Geom g, int n, int nbins, const double *__restrict__ pos, double *__restrict__ f,
                            int *__restrict__ u, int *__restrict__ cellc, int *__restrict__ bin,
                            int *__restrict__ key, int *__restrict__ count)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int c[3];
    unsigned t[3];
    for (int k = 0; k < 3; ++k) {
        double fk = pos[3 * i] * g.Ai[k] + pos[3 * i + 1] * g.Ai[3 + k] + pos[3 * i + 2] * g.Ai[6 + k];
        double uk = floor(fk);
        double w = fk - uk;
        int ck = (int)(w * g.nc[k]);
        ck = ck < 0 ? 0 : (ck >= g.nc[k] ? g.nc[k] - 1 : ck);
        f[3 * i + k] = fk;
        u[3 * i + k] = (int)uk;
        c[k] = ck;
        const double wt = fk - (double)(int)uk;
        int tk = (int)(wt * g.nt[k]);
        t[k] = (unsigned)(tk < 0 ? 0 : (tk >= g.nt[k] ? g.nt[k] - 1 : tk));
    }
    cellc[i] = (c[0] << 20) | (c[1] << 10) | c[2];
    int b = bin_of_cell(g, c[0], c[1], c[2]);
    bin[i] = b;
    atomicAdd(&count[b], 1);
    if (key) {
        const int h = nbins + (int)hilbert3(t[0], t[1], t[2], g.tb);
        key[i] = h;
        atomicAdd(&count[h], 1);
    }
}

// the atoms of each bin, and of each key in the tile order
__global__ void k_fill_bins(int n, const int *__restrict__ bin, const int *__restrict__ key,
                            const int *__restrict__ start, int *__restrict__ cursor, int *__restrict__ bin_list,
                            int *__restrict__ order)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int b = bin[i];
    bin_list[start[b] + atomicAdd(&cursor[b], 1)] = i;
    if (key) {
        b = key[i];
        order[start[b] - n + atomicAdd(&cursor[b], 1)] = i;
    }
}

// sort each bin's and key's atoms by index (deterministic cell lists and atom order)
__global__ void k_sort_bins(int n, long nbins, long nkeys, const int *__restrict__ start, int *__restrict__ bin_list,
                            int *__restrict__ order)
{
    long b = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= nbins + nkeys) return;
    int *list = b < nbins ? bin_list : order - n;
    int lo = start[b], hi = start[b + 1];
    for (int t = lo + 1; t < hi; ++t) {
        int v = list[t], s = t - 1;
        while (s >= lo && list[s] > v) { list[s + 1] = list[s]; --s; }
        list[s + 1] = v;
    }
}

// Candidate enumeration shared by the count and fill passes, by LANES lanes of an
// atom (lane l takes candidates l, l + LANES, ...; cells l, l + LANES, ... of the 27).
// For each accepted (j, S) calls emit(j, s1, s2, s3, d).
template <int LANES, typename Emit>
__device__ inline void scan_atom(const Geom &g, int n, int i, int l, const double *__restrict__ pos,
                                 const double *__restrict__ f, const int *__restrict__ u,
                                 const int *__restrict__ cellc, const int *__restrict__ bin_start,
                                 const int *__restrict__ bin_list, Emit emit)
{
    if (g.all_pairs) {
        for (int j = l; j < n; j += LANES) {
            int lo[3], hi[3];
            for (int k = 0; k < 3; ++k) {
                double df = f[3 * j + k] - f[3 * i + k];
                lo[k] = (int)ceil(-g.rc * g.gn[k] - df) - 1;
                hi[k] = (int)floor(g.rc * g.gn[k] - df) + 1;
            }
            for (int s1 = lo[0]; s1 <= hi[0]; ++s1)
                for (int s2 = lo[1]; s2 <= hi[1]; ++s2)
                    for (int s3 = lo[2]; s3 <= hi[2]; ++s3) {
                        double d[3];
                        if (pair_vec(g, pos, i, j, s1, s2, s3, d)) emit(j, s1, s2, s3, d);
                    }
        }
        return;
    }
    int cc = cellc[i];
    int ci[3] = { cc >> 20, (cc >> 10) & 1023, cc & 1023 };
    int ui[3] = { u[3 * i], u[3 * i + 1], u[3 * i + 2] };
    for (int e = l; e < 27; e += LANES) {
        int c[3] = { ci[0] + e / 9 - 1, ci[1] + e / 3 % 3 - 1, ci[2] + e % 3 - 1 }, w[3];
        for (int k = 0; k < 3; ++k) {
            w[k] = 0;
            if (c[k] < 0) { c[k] += g.nc[k]; w[k] = -1; }
            else if (c[k] >= g.nc[k]) { c[k] -= g.nc[k]; w[k] = 1; }
        }
        int b = bin_of_cell(g, c[0], c[1], c[2]);
        for (int t = bin_start[b]; t < bin_start[b + 1]; ++t) {
            int j = bin_list[t];
            // the candidate sits at fractional f_j - u_j + w relative to
            // f_i - u_i, so S = w + u_i - u_j
            int s1 = w[0] + ui[0] - u[3 * j];
            int s2 = w[1] + ui[1] - u[3 * j + 1];
            int s3 = w[2] + ui[2] - u[3 * j + 2];
            double d[3];
            if (pair_vec(g, pos, i, j, s1, s2, s3, d)) emit(j, s1, s2, s3, d);
        }
    }
}

// The passes over the candidates: half a wave per atom, a lane per cell.  Both are
// chains of dependent loads (cell, atom, position), so a thread per atom took one such
// chain per candidate, and the fill pass a sorted insertion in global memory
// on top.  Counting and filling 128 atoms of 14 neighbours: 62 + 266 -> 7 + 9 us;
// the whole list with its launches 392 -> 100 us (128 atoms), 441 -> 110 (8192) and 717 ->
// 372 (128,000); 864 atoms of 47 neighbours 2282 -> 136.
constexpr int NL = 32;              // lanes per atom
constexpr int NT = 256;             // threads per block
constexpr int NA = NT / NL;         // atoms per block
constexpr int NROW = 256;           // pairs of a row sorted in LDS (the moment plan takes 64 at most)

__global__ void __launch_bounds__(NT)
k_count(Geom g, int n, const double *__restrict__ pos, const double *__restrict__ f, const int *__restrict__ u,
        const int *__restrict__ cellc, const int *__restrict__ bin_start, const int *__restrict__ bin_list,
        int *__restrict__ cnt)
{
    const int i = blockIdx.x * NA + threadIdx.x / NL, l = threadIdx.x % NL;
    int c = 0;
    if (i < n)
        scan_atom<NL>(g, n, i, l, pos, f, u, cellc, bin_start, bin_list,
                      [&](int, int, int, int, const double *) { ++c; });
    for (int o = NL / 2; o > 0; o >>= 1) c += __shfl_xor(c, o);
    if (i < n && l == 0) cnt[i] = c;
}

__device__ inline bool key_less(int ja, int a1, int a2, int a3, int jb, int b1, int b2, int b3)
{
    if (ja != jb) return ja < jb;
    if (a1 != b1) return a1 < b1;
    if (a2 != b2) return a2 < b2;
    return a3 < b3;
}

// The rows, sorted by (j, S).  The accepted candidates of a row are gathered in LDS in
// any order; a pair's place is the number of keys below its own (keys are
// unique), found by a lane per pair.  Rows longer than NROW are inserted one by one
// in the output by the first lane, which no plan takes (whole list against a thread per
// atom: 1,024 atoms of 258 pairs 8.2 -> 7.2 ms, 8,192 of 284 pairs 80 -> 26, 54 of 2,763 pairs
// 5.8 -> 4.3).
__global__ void __launch_bounds__(NT)
k_fill(Geom g, int n, const double *__restrict__ pos, const double *__restrict__ f, const int *__restrict__ u,
       const int *__restrict__ cellc, const int *__restrict__ bin_start, const int *__restrict__ bin_list,
       const int *__restrict__ row_ptr, int *__restrict__ nbr_j, int *__restrict__ nbr_shift,
       double *__restrict__ nbr_d)
{
    __shared__ int4 s_key[NA][NROW];
    __shared__ int s_n[NA];
    const int q = threadIdx.x / NL, i = blockIdx.x * NA + q, l = threadIdx.x % NL;
    const long base = i < n ? row_ptr[i] : 0;
    const int len = i < n ? (int)(row_ptr[i + 1] - base) : 0;
    if (l == 0) s_n[q] = 0;
    __syncthreads();
    if (len > NROW) {
        int c = 0;
        if (l == 0)
            scan_atom<1>(g, n, i, 0, pos, f, u, cellc, bin_start, bin_list,
                         [&](int j, int s1, int s2, int s3, const double *d) {
                             long t = base + c - 1;
                             while (t >= base && key_less(j, s1, s2, s3, nbr_j[t], nbr_shift[3 * t],
                                                          nbr_shift[3 * t + 1], nbr_shift[3 * t + 2])) {
                                 nbr_j[t + 1] = nbr_j[t];
                                 nbr_shift[3 * t + 3] = nbr_shift[3 * t];
                                 nbr_shift[3 * t + 4] = nbr_shift[3 * t + 1];
                                 nbr_shift[3 * t + 5] = nbr_shift[3 * t + 2];
                                 nbr_d[3 * t + 3] = nbr_d[3 * t];
                                 nbr_d[3 * t + 4] = nbr_d[3 * t + 1];
                                 nbr_d[3 * t + 5] = nbr_d[3 * t + 2];
                                 --t;
                             }
                             ++t;
                             nbr_j[t] = j;
                             nbr_shift[3 * t] = s1; nbr_shift[3 * t + 1] = s2; nbr_shift[3 * t + 2] = s3;
                             nbr_d[3 * t] = d[0]; nbr_d[3 * t + 1] = d[1]; nbr_d[3 * t + 2] = d[2];
                             ++c;
                         });
    } else if (len > 0) {
        scan_atom<NL>(g, n, i, l, pos, f, u, cellc, bin_start, bin_list,
                      [&](int j, int s1, int s2, int s3, const double *) {
                          const int t = atomicAdd(&s_n[q], 1);
                          if (t < NROW) s_key[q][t] = make_int4(j, s1, s2, s3);
                      });
    }
    __syncthreads();
    if (len > NROW) return;
    for (int e = l; e < len; e += NL) {
        const int4 k = s_key[q][e];
        int rank = 0;
        for (int t = 0; t < len; ++t) {
            const int4 o = s_key[q][t];
            rank += key_less(o.x, o.y, o.z, o.w, k.x, k.y, k.z, k.w);
        }
        double d[3];
        pair_vec(g, pos, i, k.x, k.y, k.z, k.w, d);
        const long t = base + rank;
        nbr_j[t] = k.x;
        nbr_shift[3 * t] = k.y; nbr_shift[3 * t + 1] = k.z; nbr_shift[3 * t + 2] = k.w;
        nbr_d[3 * t] = d[0]; nbr_d[3 * t + 1] = d[1]; nbr_d[3 * t + 2] = d[2];
    }
}

bool make_geom(const double *cell, double rc, Geom &g)
{
    for (int k = 0; k < 9; ++k) g.A[k] = cell[k];
    const double *A = cell;
    double det = A[0] * (A[4] * A[8] - A[5] * A[7]) - A[1] * (A[3] * A[8] - A[5] * A[6])
               + A[2] * (A[3] * A[7] - A[4] * A[6]);
    if (!(std::fabs(det) > 0.0) || !std::isfinite(det)) return false;
    double *B = g.Ai;
    B[0] = (A[4] * A[8] - A[5] * A[7]) / det;
    B[1] = (A[2] * A[7] - A[1] * A[8]) / det;
    B[2] = (A[1] * A[5] - A[2] * A[4]) / det;
    B[3] = (A[5] * A[6] - A[3] * A[8]) / det;
    B[4] = (A[0] * A[8] - A[2] * A[6]) / det;
    B[5] = (A[2] * A[3] - A[0] * A[5]) / det;
    B[6] = (A[3] * A[7] - A[4] * A[6]) / det;
    B[7] = (A[1] * A[6] - A[0] * A[7]) / det;
    B[8] = (A[0] * A[4] - A[1] * A[3]) / det;
    g.rc = rc;
    g.rc2 = rc * rc;
    g.all_pairs = 0;
    for (int k = 0; k < 3; ++k) {
        g.gn[k] = std::sqrt(B[k] * B[k] + B[3 + k] * B[3 + k] + B[6 + k] * B[6 + k]);
        double m = std::floor(1.0 / (rc * g.gn[k] * (1.0 + 1e-9)));
        g.nc[k] = m < 1.0 ? 1 : (m > 1023.0 ? 1023 : (int)m);
        if (g.nc[k] < 3) g.all_pairs = 1;
        g.nb[k] = (g.nc[k] + 1) / 2;
        g.nt[k] = g.nc[k] * 3 > 256 ? 256 : g.nc[k] * 3;
    }
    int m = g.nt[0] > g.nt[1] ? g.nt[0] : g.nt[1];
    m = m > g.nt[2] ? m : g.nt[2];
    g.tb = 1;
    while ((1 << g.tb) < m) ++g.tb;
    return true;
}

struct NbrWs {
    double *f; int *u, *cellc, *bin, *key, *count, *cursor, *start, *bin_list;
    void *scan;
    size_t bytes;
};

NbrWs carve(void *base, int n, long nbins, long nkeys)
{
    NbrWs w{};
    char *p = (char *)base;
    auto take = [&](size_t b) { char *r = p; p += align_up(b, 256); return (void *)r; };
    w.f = (double *)take(sizeof(double) * 3 * (size_t)n);
    w.u = (int *)take(sizeof(int) * 3 * (size_t)n);
    w.cellc = (int *)take(sizeof(int) * (size_t)n);
    w.bin = (int *)take(sizeof(int) * (size_t)n);
    w.bin_list = (int *)take(sizeof(int) * (size_t)n + 4);
    w.key = (int *)take(sizeof(int) * (size_t)n + 4);
    const long nb = nbins + nkeys;
    w.count = (int *)take(sizeof(int) * 2 * (size_t)nb);      // and the cursors: zeroed in one launch
    w.cursor = w.count + nb;
    w.start = (int *)take(sizeof(int) * (size_t)(nb + 1));
    w.scan = take(scan_scratch_bytes(nb > n ? nb : n));
    w.bytes = (size_t)(p - (char *)base);
    return w;
}

}  // namespace
}  // namespace bop

using namespace bop;

extern "C" size_t bop_neighbours_workspace_size(int n_atoms, const double *cell, double r_cut)
{
    Geom g;
    if (n_atoms < 0 || !cell || !(r_cut > 0) || !make_geom(cell, r_cut, g)) return 0;
    long nbins = (long)g.nb[0] * g.nb[1] * g.nb[2] * 8;
    return carve(nullptr, n_atoms, nbins, 1L << (3 * g.tb)).bytes + 256;
}

extern "C" int bop_build_neighbours(int n, const double *pos, const double *cell, double r_cut,
                                    long capacity, int *row_ptr, int *nbr_j, int *nbr_shift,
                                    double *nbr_d, int *order, long *n_pairs,
                                    void *ws, size_t ws_bytes, hipStream_t stream)
{
    BOP_REQUIRE(n >= 0 && cell && n_pairs && row_ptr && capacity >= 0, BOP_E_ARG,
                "bop_build_neighbours: bad arguments");
    BOP_REQUIRE(n == 0 || pos, BOP_E_ARG, "bop_build_neighbours: pos is NULL");
    BOP_REQUIRE(r_cut > 0 && std::isfinite(r_cut), BOP_E_ARG, "bop_build_neighbours: r_cut must be > 0");
    Geom g;
    BOP_REQUIRE(make_geom(cell, r_cut, g), BOP_E_ARG, "bop_build_neighbours: singular cell");
    long nbins = (long)g.nb[0] * g.nb[1] * g.nb[2] * 8;
    const long nkeys = 1L << (3 * g.tb);
    NbrWs w = carve(ws, n, nbins, order ? nkeys : 0);
    BOP_REQUIRE(ws && ws_bytes >= w.bytes, BOP_E_CAPACITY,
                "bop_build_neighbours: workspace of %zu bytes needed, %zu given", w.bytes, ws_bytes);
    *n_pairs = 0;
    const int T = 256;
    auto blocks = [&](long m) { return (unsigned)((m + T - 1) / T > 0 ? (m + T - 1) / T : 1); };

    const long nb = nbins + (order ? nkeys : 0);
    int rc = BOP_OK;
    if (n > 0) {
        int *key = order ? w.key : nullptr;
        k_fill_int<<<blocks(2 * nb), T, 0, stream>>>(w.count, 2 * nb, 0);
        k_bin_atoms<<<blocks(n), T, 0, stream>>>(g, n, (int)nbins, pos, w.f, w.u, w.cellc, w.bin, key, w.count);
        BOP_LAUNCHED();
        rc = exclusive_scan(w.count, w.start, nb, w.scan, stream);
        if (rc) return rc;
        k_fill_bins<<<blocks(n), T, 0, stream>>>(n, w.bin, key, w.start, w.cursor, w.bin_list, order);
        k_sort_bins<<<blocks(nb), T, 0, stream>>>(n, nbins, nb - nbins, w.start, w.bin_list, order);
        k_count<<<(unsigned)((n + NA - 1) / NA), NT, 0, stream>>>(g, n, pos, w.f, w.u, w.cellc, w.start, w.bin_list, row_ptr);
        BOP_LAUNCHED();
    }
    rc = exclusive_scan(row_ptr, row_ptr, n, w.scan, stream);
    if (rc) return rc;
    int total = 0;
    BOP_HIP(hipMemcpyAsync(&total, row_ptr + n, sizeof(int), hipMemcpyDeviceToHost, stream));
    BOP_HIP(hipStreamSynchronize(stream));
    *n_pairs = total;
    BOP_REQUIRE(total >= 0, BOP_E_CAPACITY, "bop_build_neighbours: more than 2^31 pairs");
    if (total > capacity) {
        set_error("bop_build_neighbours: %d pairs, capacity %ld", total, capacity);
        return BOP_E_CAPACITY;
    }
    if (n > 0 && total > 0) {
        BOP_REQUIRE(nbr_j && nbr_shift && nbr_d, BOP_E_ARG, "bop_build_neighbours: output arrays are NULL");
        k_fill<<<(unsigned)((n + NA - 1) / NA), NT, 0, stream>>>(g, n, pos, w.f, w.u, w.cellc, w.start, w.bin_list,
                                            row_ptr, nbr_j, nbr_shift, nbr_d);
        BOP_LAUNCHED();
    }
    return BOP_OK;
}
