// Tile plan and workspace layout shared by the moment passes and the force
// passes: per-tile support sizes, the tile records (support rows, layer and
// slot counts, neighbour slots, row masks) written by the prepare pass, and
// where the X buffers, chunk partials and Lanczos coefficients live in a
// bop_moments workspace.
#pragma once
#include "bop_internal.h"
#include <type_traits>

namespace bop {

constexpr int MAX_NMAX = 40;
constexpr int MAXK = MAX_NMAX / 2;
constexpr int HDR = 256;            // header ints: [0] queue, [1] error, [2] max rows, [3] max degree,
                                    // [8 + k] max rows of U^k (plan)
constexpr int LC_N = 8;             // Lanczos column coefficients per lane and tile
constexpr int SLOTS_HELD = 16;      // slots of a row whose words k_step32 holds in scalar registers from a row ahead

// Row assignment of the step kernels: a tile with nrow rows at this step uses
// nct = tile_chunks(..) of the launch's chunks, and chunk c < nct takes the
// wave-sized row groups c, c + nct, c + 2 nct, ...  nct depends on the tile
// alone, so the grouping of the partial sums (and the rounding of the moments)
// does not change with the other tiles of the plan.
__device__ inline int tile_chunks(int nrow, int chunk_rows, int nw)
{
    return min((nrow + chunk_rows - 1) / chunk_rows, (nrow + nw - 1) / nw);
}

// ---------------------------------------------------------------------------
// workspace layout
// ---------------------------------------------------------------------------
// Bytes of one row of X (all 64 columns): n_orb values per column in
// FP64/FP32 (planes of 16 bytes per column and one of the last orbital), or n_orb padded to the MFMA slot width in
// BF16 ([64][slot width] per row).
__host__ __device__ inline size_t x_row_bytes(int dtype, int n_orb)
{
    if (dtype == BOP_BF16) return 2ull * 64 * (n_orb <= 8 ? 8 : 16);
    return (dtype == BOP_F64 ? 8ull : (dtype == BOP_F16 ? 2ull : 4ull)) * n_orb * 64;
}

typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
constexpr int AUX_NT = 2;           // non-temporal bit of a buffer access

// Layout of a row of X (64 columns, one per lane): the orbitals are grouped into
// planes of V values per lane, so that a lane reads or writes its column's
// values of a row with one wide access per plane (16 bytes for FP64 and FP32)
// instead of one per orbital; the orbital left over has a plane of its own.
template <typename S, int NO> struct XRow {
    static constexpr int V = sizeof(S) >= 4 ? 16 / (int)sizeof(S) : NO - 1;
    static constexpr int NP = NO / V, TAIL = NP * V * 64;
    static_assert(NO - NP * V == 1, "one orbital is left over");
    typedef S vec __attribute__((ext_vector_type(V)));
    // element of orbital a, column c
    static __host__ __device__ int at(int a, int c) { return a < NP * V ? (a / V) * V * 64 + c * V + a % V : TAIL + c; }
    template <bool NT, typename T> static __device__ inline void load(const S *row, int lane, T (&x)[NO])
    {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const vec *q = (const vec *)(row + p * V * 64) + lane;
            const vec v = NT ? __builtin_nontemporal_load(q) : *q;
#pragma unroll
            for (int e = 0; e < V; ++e) x[p * V + e] = (T)v[e];
        }
        const S *q = row + TAIL + lane;
        x[NO - 1] = (T)(NT ? __builtin_nontemporal_load(q) : *q);
    }
    // non-temporal
    static __device__ inline void store(S *row, int lane, const S (&x)[NO])
    {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            vec v;
#pragma unroll
            for (int e = 0; e < V; ++e) v[e] = x[p * V + e];
            __builtin_nontemporal_store(v, (vec *)(row + p * V * 64) + lane);
        }
        __builtin_nontemporal_store(x[NO - 1], row + TAIL + lane);
    }
    // The same for FP32 and FP16 through a buffer descriptor of the row: its base is
    // wave-uniform, so that addresses cost no vector instruction, and one of no bytes (on
    // false) reads zeros and drops stores without a branch, which would hide the number
    // of accesses in flight from the waits that follow it.
    static __device__ inline __amdgpu_buffer_rsrc_t row_rsrc(const S *row, bool on)
    {
        return __builtin_amdgcn_make_buffer_rsrc((void *)row, 0, on ? NO * 64 * (int)sizeof(S) : 0, 0x00027000);
    }
    // Raw: a lane's values as stored.  A load held in flight keeps them so: converted
    // at once it would be waited for at once.
    struct Raw { vec v[NP]; S tail; };
    template <int AUX> static __device__ inline void load(__amdgpu_buffer_rsrc_t r, int lane, Raw &x)
    {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            if constexpr (sizeof(vec) == 16)
                x.v[p] = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b128(r, lane * 16 + p * 1024, 0, AUX));
            else x.v[p] = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b64(r, lane * 8 + p * 512, 0, AUX));
        }
        if constexpr (sizeof(S) == 4)
            x.tail = __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b32(r, (TAIL + lane) * (int)sizeof(S), 0, AUX));
        else x.tail = __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b16(r, (TAIL + lane) * (int)sizeof(S), 0, AUX));
    }
    template <typename T> static __device__ inline void values(const Raw &r, T (&x)[NO])
    {
#pragma unroll
        for (int a = 0; a < NO - 1; ++a) x[a] = (T)r.v[a / V][a % V];
        x[NO - 1] = (T)r.tail;
    }
    // Wide<T>: the values converted as they arrive.
    template <typename T> struct Wide { T x[NO]; };
    template <int AUX, typename T> static __device__ inline void load(__amdgpu_buffer_rsrc_t r, int lane, Wide<T> &x)
    {
        Raw v;
        load<AUX>(r, lane, v);
        values(v, x.x);
    }
    template <typename T> static __device__ inline void values(const Wide<T> &r, T (&x)[NO])
    {
#pragma unroll
        for (int a = 0; a < NO; ++a) x[a] = r.x[a];
    }
    // non-temporal
    static __device__ inline void store(__amdgpu_buffer_rsrc_t r, int lane, const S (&x)[NO])
    {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            vec v;
#pragma unroll
            for (int e = 0; e < V; ++e) v[e] = x[p * V + e];
            if constexpr (sizeof(vec) == 16)
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v), r, lane * 16 + p * 1024, 0, AUX_NT);
            else __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2_t, v), r, lane * 8 + p * 512, 0, AUX_NT);
        }
        if constexpr (sizeof(S) == 4)
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, x[NO - 1]), r, (TAIL + lane) * (int)sizeof(S), 0, AUX_NT);
        else __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, x[NO - 1]), r, (TAIL + lane) * (int)sizeof(S), 0, AUX_NT);
    }
};

// compile-time loop: f(integral_constant<int, I>) for I = 0 .. N-1
template <int N, int I = 0, typename F> __device__ inline void static_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<N, I + 1>(f);
    }
}

// acc += (lane K of every 16-lane row of h) * x.  A broadcasting operand costs
// no instruction of its own.  The operand may not be read within two waits of
// a VALU write; callers pass h as loaded, with dpp_guard() before the first use.
template <int K> __device__ inline void fma_bcast(float &acc, float h, float x)
{
    asm("v_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(h), "v"(x), "n"(K));
}
template <int K> __device__ inline void fma_bcast(double &acc, double h, double x)
{
    asm("v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(h), "v"(x), "n"(K));
}
template <typename T> __device__ inline void dpp_guard(T &h) { asm("s_nop 1" : "+v"(h)); }

struct Layout {
    size_t sizes;       // int [n_tiles][MAXK + 2]: rows of U^k per tile; [0] = -1 marks a failed tile
    size_t tiles;       // per tile: sup[rows_cap], rinfo[rows_cap], lnb[rows_cap * deg_max], rmask[rows_cap]
    size_t tile_stride;
    size_t x;           // X buffers: batch x 2 x rows_cap x n_orb x 64 (also prepare's maps)
    size_t x_stride;    // bytes of one X buffer
    size_t part;        // double [batch][chunks][2][64]
    size_t lc;          // double [batch][LC_N][64]: Lanczos column coefficients
    size_t bytes;
};

// Where each step's chunk partials start (doubles, for batch_tiles tiles) and
// how many chunks the step has.
struct StepParts {
    long off[MAXK + 2];
    int nch[MAXK + 2];
    size_t total_chunks;
};

__host__ __device__ inline StepParts step_parts(const bop_plan &p)
{
    StepParts sp{};
    const int K = p.n_max / 2, steps = K + (p.n_max & 1);
    size_t tot = 0;
    for (int k = 1; k <= steps && k <= MAXK + 1; ++k) {
        const int rows_k = k > K ? p.rows_k[K] : p.rows_k[k];
        sp.nch[k] = (rows_k + p.chunk_rows - 1) / p.chunk_rows;
        sp.off[k] = (long)(tot * 2 * 64 * (size_t)p.batch_tiles);
        tot += (size_t)sp.nch[k];
    }
    sp.total_chunks = tot;
    return sp;
}

__host__ __device__ inline Layout make_layout(const bop_plan &p, int n_prep_wg)
{
    Layout L;
    size_t o = HDR;
    auto take = [&](size_t b) { size_t r = o; o += (b + 255) / 256 * 256; return r; };
    L.sizes = take(4ull * p.n_tiles * (MAXK + 2));
    L.tile_stride = (4ull * p.rows_cap * (3 + p.deg_max) + 255) / 256 * 256;   // sup, rinfo, lnb, row masks
    L.tiles = take(L.tile_stride * p.n_tiles);
    // Keep something of SLOTS_HELD ints or more behind the tile records: k_step32 reads that
    // many words of every row's slot list, so past the last record where rows are few and
    // short (8 rows of 5 slots end 12 bytes short).  The X buffers take a row of 640 bytes
    // at least.
    L.x_stride = (x_row_bytes(p.dtype, p.n_orb) * p.rows_cap + 255) / 256 * 256;
    size_t xb = L.x_stride * (p.batch_tiles >= 2 ? 2 * (size_t)p.batch_tiles : 4);
    size_t maps = (size_t)n_prep_wg * ((4ull * p.n_atoms + 255) / 256 * 256);
    L.x = take(xb > maps ? xb : maps);
    // chunk partials: one step's worth for the Lanczos form (three per chunk at
    // its last level), every step's for the moment form (two per chunk,
    // reduced after the batch's last step)
    const size_t nch = (p.rows_cap + p.chunk_rows - 1) / p.chunk_rows;
    const size_t nch_all = step_parts(p).total_chunks;
    L.part = take(8ull * 64 * (3 * nch > 2 * nch_all ? 3 * nch : 2 * nch_all) * p.batch_tiles);
    L.lc = take(8ull * LC_N * 64 * p.batch_tiles);
    L.bytes = o;
    return L;
}

// Workgroups of the plan and prepare passes: two per CU, but at most about
// 1 GiB of per-workgroup global->local maps.
inline int map_workgroups(int n_atoms, int n_tiles)
{
    size_t per = align_up(4ull * n_atoms, 256) * 2;
    long cap = (long)((1ull << 30) / (per ? per : 1));
    long w = 2L * device_cus();
    if (w > cap) w = cap;
    if (w > n_tiles) w = n_tiles;
    return w < 1 ? 1 : (int)w;
}

}  // namespace bop
