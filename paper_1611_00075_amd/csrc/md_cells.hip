// Steps a1-a3: wrap + cell assignment, stable counting sort into
// Morton-ordered cells, permutation of per-atom arrays, scaled coordinates,
// and full Verlet neighbour lists from LDS-staged neighbour-cell tiles.
//
// Every floating-point decision here (wrap, cell index, r^2 < r_list^2) is
// taken in FP64 with the operation order of the plain definition and no FMA
// contraction (the library is built with -ffp-contract=off), so cell
// assignments and neighbour sets are reproducible bit for bit.
#include <algorithm>

#include "md_bin.h"
#include "md_pair.h"

namespace md {

// ---------------------------------------------------------------------------
// binning
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(kBlock) void k_bin_assign(int64_t n, double *x, GridArgs g, const int32_t *lin2rank,
                                                       int32_t *cell, int32_t *cnt, int32_t *slot)
{
    const int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (i >= n) return;
    int32_t c[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double w = wrap1(x[a * n + i], g.L[a]);
        x[a * n + i] = w;
        c[a] = cell1(w, g.inv_cell[a], g.nc[a]);
    }
    const int64_t lin = c[0] + int64_t(g.nc[0]) * (c[1] + int64_t(g.nc[1]) * c[2]);
    const int32_t r = lin2rank[lin];
    cell[i] = r;
    slot[i] = claim_slot(r, cnt);
}

__global__ __launch_bounds__(kBlock) void k_bin_scatter(int64_t n, const int32_t *__restrict__ cell,
                                                        const int32_t *__restrict__ slot,
                                                        const int32_t *__restrict__ cell_start,
                                                        int32_t *__restrict__ tmp)
{
    const int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (i >= n) return;
    tmp[cell_start[cell[i]] + slot[i]] = int32_t(i);
}

// The atomic slots give an arbitrary order inside each cell; restore input
// order (stability) by ranking each atom among the members of its cell.
__global__ __launch_bounds__(kBlock) void k_bin_stable(int64_t n, const int32_t *__restrict__ cell,
                                                       const int32_t *__restrict__ tmp,
                                                       const int32_t *__restrict__ cell_start,
                                                       int32_t *__restrict__ perm)
{
    const int64_t p = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (p >= n) return;
    const int32_t i = tmp[p];
    const int32_t c = cell[i];
    const int32_t s0 = cell_start[c], s1 = cell_start[c + 1];
    perm[s0 + stable_rank(tmp, s0, s1, i)] = i;
}

// ---------------------------------------------------------------------------
// permutation and scaled coordinates
// ---------------------------------------------------------------------------

template <typename T>
__global__ __launch_bounds__(kBlock) void k_permute(int64_t n, int32_t ncomp, const int32_t *perm, const T *src,
                                                    T *dst)
{
    const int64_t k = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (k >= n) return;
    const int64_t j = perm[k];
    for (int32_t c = 0; c < ncomp; ++c) dst[c * n + k] = src[c * n + j];
}

int permute(int64_t n, int32_t ncomp, const int32_t *perm, const void *src, void *dst, int32_t eb, hipStream_t s)
{
    if (n <= 0) return MD_OK;
    const uint32_t gb = uint32_t((n + kBlock - 1) / kBlock);
    switch (eb) {
    case 4:
        hipLaunchKernelGGL(k_permute<uint32_t>, dim3(gb), dim3(kBlock), 0, s, n, ncomp, perm,
                           static_cast<const uint32_t *>(src), static_cast<uint32_t *>(dst));
        break;
    case 8:
        hipLaunchKernelGGL(k_permute<uint64_t>, dim3(gb), dim3(kBlock), 0, s, n, ncomp, perm,
                           static_cast<const uint64_t *>(src), static_cast<uint64_t *>(dst));
        break;
    case 16:
        hipLaunchKernelGGL(k_permute<uint4>, dim3(gb), dim3(kBlock), 0, s, n, ncomp, perm,
                           static_cast<const uint4 *>(src), static_cast<uint4 *>(dst));
        break;
    default:
        return MD_ERR_ARG;
    }
    MD_HIP_TRY(hipGetLastError());
    return MD_OK;
}

// fixed-point fraction of the box, modulo 2^32 (negative and >= L positions
// wrap by the integer conversion)
__device__ __forceinline__ uint32_t scale1(double x, double k)
{
    return uint32_t(uint64_t(__double2ll_rn(x * k)));
}

__global__ __launch_bounds__(kBlock) void k_scale(int64_t n, const double *x, double k0, double k1, double k2,
                                                  uint4 *xs)
{
    const int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (i >= n) return;
    xs[i] = make_uint4(scale1(x[i], k0), scale1(x[n + i], k1), scale1(x[2 * n + i], k2), 0u);
}

int scale_positions(const md_box_t *box, int64_t n, const double *x, uint32_t *xs, hipStream_t s)
{
    if (n <= 0) return MD_OK;
    const double two32 = 4294967296.0;
    const uint32_t gb = uint32_t((n + kBlock - 1) / kBlock);
    hipLaunchKernelGGL(k_scale, dim3(gb), dim3(kBlock), 0, s, n, x, two32 / box->L[0], two32 / box->L[1],
                       two32 / box->L[2], reinterpret_cast<uint4 *>(xs));
    MD_HIP_TRY(hipGetLastError());
    return MD_OK;
}

// Positions, velocities and input indices into the sorted order in two
// passes: gather from the old order into xr (the new reference positions),
// vt and it; then copy vt, it and xr back into the state arrays and, with
// xs, write the scaled coordinates of the new positions.
__global__ __launch_bounds__(kBlock) void k_reorder_gather(int64_t n, const int32_t *__restrict__ perm,
                                                           const double *__restrict__ x,
                                                           const double *__restrict__ v,
                                                           const int32_t *__restrict__ ids, double *__restrict__ xr,
                                                           double *__restrict__ vt, int32_t *__restrict__ it)
{
    const int64_t k = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (k >= n) return;
    const int64_t j = perm[k];
    for (int c = 0; c < 3; ++c) {
        xr[c * n + k] = x[c * n + j];
        vt[c * n + k] = v[c * n + j];
    }
    it[k] = ids[j];
}

__global__ __launch_bounds__(kBlock) void k_reorder_put(int64_t n, const double *__restrict__ xr,
                                                        const double *__restrict__ vt,
                                                        const int32_t *__restrict__ it, double *__restrict__ x,
                                                        double *__restrict__ v, int32_t *__restrict__ ids, double k0,
                                                        double k1, double k2, uint4 *__restrict__ xs, int32_t *clear)
{
    const int64_t k = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (clear && k == 0) *clear = 0;
    if (k >= n) return;
    double p[3];
    for (int c = 0; c < 3; ++c) {
        p[c] = xr[c * n + k];
        x[c * n + k] = p[c];
        v[c * n + k] = vt[c * n + k];
    }
    ids[k] = it[k];
    if (xs) xs[k] = make_uint4(scale1(p[0], k0), scale1(p[1], k1), scale1(p[2], k2), 0u);
}

int reorder_state(int64_t n, const int32_t *perm, double *x, double *v, int32_t *ids, double *xref, double *vtmp,
                  int32_t *itmp, const md_box_t *box, uint32_t *xs, hipStream_t s, int32_t *clear)
{
    if (n <= 0) return MD_OK;
    const double two32 = 4294967296.0;
    const uint32_t gb = uint32_t((n + kBlock - 1) / kBlock);
    hipLaunchKernelGGL(k_reorder_gather, dim3(gb), dim3(kBlock), 0, s, n, perm, x, v, ids, xref, vtmp, itmp);
    hipLaunchKernelGGL(k_reorder_put, dim3(gb), dim3(kBlock), 0, s, n, xref, vtmp, itmp, x, v, ids,
                       two32 / box->L[0], two32 / box->L[1], two32 / box->L[2], reinterpret_cast<uint4 *>(xs), clear);
    MD_HIP_TRY(hipGetLastError());
    return MD_OK;
}

// ---------------------------------------------------------------------------
// sorting a small system in one launch
// ---------------------------------------------------------------------------

// What a build of the native driver reorders besides: state into the sorted order,
// the new reference positions and scaled coordinates (xs may be NULL).
struct SortState {
    double *v, *xref;
    int32_t *ids;
    double k[3];   // 2^32 / L
    uint4 *xs;
    int32_t *clear;   // a word set to 0
};

// Small systems: one block does the whole counting sort in LDS and, with STATE,
// the reordering: the same cells, order and permutation as the general path,
// whose five launches (seven with the reordering) of a few microseconds each
// are what such a sort costs there.  Each thread keeps its K atoms in registers
// from the wrap to their new places.  One CU does it all, so the work takes over
// from the launches at some size: with STATE beyond 4,096 atoms (a whole build in
// md_run, sort / general: 4,000 LJ atoms 46.8 / 54 us, 6,912 51.3 / 45), without
// beyond 8,192, and for both where cells are crowded (sorts_small).
constexpr int kSmallBlock = 1024;
constexpr int kSmallCells = 4096;
constexpr int64_t kSmallAtoms = 8192, kSmallState = 4096;
static_assert(kSmallCells % kSmallBlock == 0 && kSmallAtoms <= 65536, "a thread's run of cells; 16-bit indices");

template <bool STATE, int K>
__global__ __launch_bounds__(kSmallBlock) void k_sort_small(int32_t n, double *x, GridArgs g, int32_t n_cells,
                                                            const int32_t *lin2rank, int32_t *cell, int32_t *perm,
                                                            int32_t *cell_start, SortState st)
{
    __shared__ int32_t start[kSmallCells + 1];
    __shared__ uint16_t member[kSmallBlock * K];
    __shared__ int32_t wsum[kSmallBlock / kWave];
    const int t = threadIdx.x, lane = t % kWave, wave = t / kWave;
    constexpr int C = kSmallCells / kSmallBlock;
    for (int c = t; c <= kSmallCells; c += kSmallBlock) start[c] = 0;
    double p[K][3];
    int32_t rank[K], at[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int32_t i = t + k * kSmallBlock;
        if (i >= n) continue;
#pragma unroll
        for (int a = 0; a < 3; ++a) p[k][a] = x[a * n + i];
    }
    __syncthreads();
    // cell of each atom, a slot in it
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int32_t i = t + k * kSmallBlock;
        if (i >= n) continue;
        int32_t c[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            p[k][a] = wrap1(p[k][a], g.L[a]);
            if (!STATE) x[a * n + i] = p[k][a];
            c[a] = cell1(p[k][a], g.inv_cell[a], g.nc[a]);
        }
        rank[k] = lin2rank[c[0] + int64_t(g.nc[0]) * (c[1] + int64_t(g.nc[1]) * c[2])];
        cell[i] = rank[k];
        at[k] = atomicAdd(&start[rank[k]], 1);
    }
    __syncthreads();
    // first atom of each cell
    int32_t cnt[C], sum = 0;
#pragma unroll
    for (int q = 0; q < C; ++q) {
        cnt[q] = start[t * C + q];
        sum += cnt[q];
    }
    int32_t inc = sum;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int32_t u = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += u;
    }
    if (lane == kWave - 1) wsum[wave] = inc;
    __syncthreads();
    int32_t run = inc - sum;
    for (int w = 0; w < wave; ++w) run += wsum[w];
#pragma unroll
    for (int q = 0; q < C; ++q) {
        const int32_t c = t * C + q;
        start[c] = run;
        if (c <= n_cells) cell_start[c] = run;
        run += cnt[q];
    }
    if (t == kSmallBlock - 1) {
        start[kSmallCells] = run;
        if (n_cells == kSmallCells) cell_start[n_cells] = run;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (t + k * kSmallBlock < n) member[start[rank[k]] + at[k]] = uint16_t(t + k * kSmallBlock);
    __syncthreads();
    // stable order: the place among the members of the cell
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int32_t i = t + k * kSmallBlock;
        if (i >= n) continue;
        const int32_t s0 = start[rank[k]], s1 = start[rank[k] + 1];
        int32_t d = s0;
        for (int32_t q = s0; q < s1; q += 8) {   // eight reads in flight
            int32_t m[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) m[u] = member[min(q + u, s1 - 1)];
#pragma unroll
            for (int u = 0; u < 8; ++u) d += q + u < s1 && m[u] < i;
        }
        at[k] = d;
        perm[d] = i;
    }
    if constexpr (STATE) {
        // every thread has read its positions (before the first barrier)
        if (t == 0) *st.clear = 0;
        double v[K][3];
        int32_t id[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int32_t i = t + k * kSmallBlock;
            if (i >= n) continue;
            const int32_t d = at[k];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                x[a * n + d] = p[k][a];
                st.xref[a * n + d] = p[k][a];
                v[k][a] = st.v[a * n + i];
            }
            id[k] = st.ids[i];
            if (st.xs)
                st.xs[d] = make_uint4(scale1(p[k][0], st.k[0]), scale1(p[k][1], st.k[1]), scale1(p[k][2], st.k[2]), 0u);
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (t + k * kSmallBlock >= n) continue;
            const int32_t d = at[k];
#pragma unroll
            for (int a = 0; a < 3; ++a) st.v[a * n + d] = v[k][a];
            st.ids[d] = id[k];
        }
    }
}

// One CU handles each atom and compares it with the members of its cell: about
// n (n / n_cells + 22) comparisons' worth of work where atoms are spread evenly, which
// grows past the general path's launches where cells are crowded.  Us of calls in a row,
// one launch / general: 8,192 atoms 16 to a cell 24 / 19, 66 to a cell 46 / 20, 303 to a cell
// 138 / 26, 1,024 to a cell 416 / 52; 4,096 atoms 64 to a cell 22 / 19, 152 to a cell 43 / 21.
// Among other calls the host is behind and four launches less are worth more: rebuilds of
// 6,912 LJ atoms 20 to a cell 105 / 117, 55 to a cell 129 / 146, 108 to a cell 215 / 221, of
// 4,000 148 to a cell 263 / 277.  The line, at about 50 us of the one launch (8,192 atoms
// 74 to a cell, 4,096 170), lies where a call that is waited for takes the same.
static bool sorts_small(const md_grid_t *grid, int64_t n, int64_t most)
{
    return n > 0 && n <= most && grid->n_cells <= kSmallCells &&
           n * (n + 22 * grid->n_cells) <= (3 * grid->n_cells << 18);
}

int bin_cells(const md_grid_t *grid, int64_t n, double *x, int32_t *cell, int32_t *perm, int32_t *cell_start,
              void *ws, const WsLayout &w, hipStream_t s)
{
    const GridArgs g = grid_args(grid);
    if (sorts_small(grid, n, kSmallAtoms)) {
        hipLaunchKernelGGL((n <= 4 * kSmallBlock ? k_sort_small<false, 4> : k_sort_small<false, 8>), dim3(1), dim3(kSmallBlock), 0, s, int32_t(n), x, g,
                           int32_t(grid->n_cells), ws_ptr<int32_t>(ws, w.lin2rank), cell, perm, cell_start, SortState{});
        MD_HIP_TRY(hipGetLastError());
        return MD_OK;
    }
    int32_t *cnt = ws_ptr<int32_t>(ws, w.cell_cnt);
    int32_t *slot = ws_ptr<int32_t>(ws, w.slot);
    int32_t *tmp = ws_ptr<int32_t>(ws, w.tmp);
    int rc = launch_fill_i32(cnt, grid->n_cells + 1, 0, s);
    if (rc) return rc;
    if (n > 0) {
        const uint32_t gb = uint32_t((n + kBlock - 1) / kBlock);
        hipLaunchKernelGGL(k_bin_assign, dim3(gb), dim3(kBlock), 0, s, n, x, g, ws_ptr<int32_t>(ws, w.lin2rank), cell,
                           cnt, slot);
        MD_HIP_TRY(hipGetLastError());
    }
    rc = launch_scan_i32_to_i32(cnt, cell_start, grid->n_cells, ws_ptr<int64_t>(ws, w.scan), s);
    if (rc) return rc;
    if (n > 0) {
        const uint32_t gb = uint32_t((n + kBlock - 1) / kBlock);
        hipLaunchKernelGGL(k_bin_scatter, dim3(gb), dim3(kBlock), 0, s, n, cell, slot, cell_start, tmp);
        hipLaunchKernelGGL(k_bin_stable, dim3(gb), dim3(kBlock), 0, s, n, cell, tmp, cell_start, perm);
        MD_HIP_TRY(hipGetLastError());
    }
    return MD_OK;
}

// bin_cells and reorder_state of a build; sets *max_count to 0 for its lists (n > 0).
int sort_state(const md_grid_t *grid, int64_t n, double *x, int32_t *cell, int32_t *perm, int32_t *cell_start,
               void *ws, const WsLayout &w, double *v, int32_t *ids, double *xref, double *vtmp, int32_t *itmp,
               const md_box_t *box, uint32_t *xs, int32_t *max_count, hipStream_t s)
{
    if (sorts_small(grid, n, kSmallState)) {
        const double two32 = 4294967296.0;
        const SortState st{v, xref, ids, {two32 / box->L[0], two32 / box->L[1], two32 / box->L[2]},
                           reinterpret_cast<uint4 *>(xs), max_count};
        hipLaunchKernelGGL((k_sort_small<true, kSmallState / kSmallBlock>), dim3(1), dim3(kSmallBlock), 0, s, int32_t(n), x, grid_args(grid),
                           int32_t(grid->n_cells), ws_ptr<int32_t>(ws, w.lin2rank), cell, perm, cell_start, st);
        MD_HIP_TRY(hipGetLastError());
        return MD_OK;
    }
    if (int rc = bin_cells(grid, n, x, cell, perm, cell_start, ws, w, s)) return rc;
    return reorder_state(n, perm, x, v, ids, xref, vtmp, itmp, box, xs, s, max_count);
}

// The element of each atom (0 or 1; only bit 0 is used) into the fourth word
// of its scaled coordinates.
__global__ __launch_bounds__(kBlock) void k_set_elements(int64_t n, const int32_t *types, uint4 *xs)
{
    const int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (i < n) xs[i].w = uint32_t(types[i]) & 1u;
}

int set_elements(int64_t n, const int32_t *types, uint32_t *xs, hipStream_t s)
{
    if (n <= 0) return MD_OK;
    const uint32_t gb = uint32_t((n + kBlock - 1) / kBlock);
    hipLaunchKernelGGL(k_set_elements, dim3(gb), dim3(kBlock), 0, s, n, types, reinterpret_cast<uint4 *>(xs));
    MD_HIP_TRY(hipGetLastError());
    return MD_OK;
}

// ---------------------------------------------------------------------------
// neighbour lists
// ---------------------------------------------------------------------------

constexpr int kMaxStencil = 125;       // (2*reach+1)^3, reach <= 2

// Distinct values of (c + o) mod nc, o in [-reach, reach], in increasing o;
// img[k] = floor((c + o) / nc) of the value's first offset: the periodic
// image of that stencil cell (the only one when no value was de-duplicated).
__device__ __forceinline__ int stencil_axis(int32_t c, int32_t nc, int32_t reach, int32_t *out, int32_t *img)
{
    int m = 0;
    for (int o = -reach; o <= reach; ++o) {
        int32_t v = c + o, k = 0;
        while (v < 0) {
            v += nc;
            --k;
        }
        while (v >= nc) {
            v -= nc;
            ++k;
        }
        bool dup = false;
        for (int q = 0; q < m; ++q) dup |= (out[q] == v);
        if (!dup) {
            img[m] = k;
            out[m++] = v;
        }
    }
    return m;
}

// Wave-uniform copies of values the compiler cannot prove uniform.
__device__ __forceinline__ int32_t uni(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// The definition's minimum image without branches: subtracting 0, L or -L
// gives the same bits as leaving d alone, d - L or d + L.
__device__ __forceinline__ double minimg_sel(double d, double L, double hL)
{
    const double t = d > hL ? L : (d < -hL ? -L : 0.0);
    return d - t;
}

__device__ __forceinline__ double wave_min(double v)
{
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) v = fmin(v, __shfl_xor(v, o, kWave));
    return v;
}

__device__ __forceinline__ double wave_max(double v)
{
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) v = fmax(v, __shfl_xor(v, o, kWave));
    return v;
}

constexpr int kNbChunks = 4;                   // 64-candidate chunks held in registers at once
constexpr int kNbTile = kNbChunks * kWave;     // candidates per register tile
constexpr int kNbStage = 2 * kNbTile;          // staged candidates: a tile plus one raw tile's survivors
constexpr int kNbMap = 1024;                   // candidates whose stencil cell is tabulated in LDS
constexpr uint32_t kNbXcdChunk = 256;          // consecutive blocks (cells) an XCD takes at a time

// What the set-up of a cell found: its homes, its stencil cells, their atoms.
struct NbCell {
    int32_t h0, h1;      // sorted atoms of the cell
    int32_t m, total;    // stencil cells, candidates in them
    bool nodup;          // every stencil offset is a cell of its own
};

// The stencil of cell `rank` into L: per stencil cell (x fastest) the first
// atom, the candidates before it and its periodic image, and for up to kNbMap
// candidates the stencil cell of each.
template <class LDS>
__device__ __forceinline__ NbCell nb_stencil(LDS &L, int64_t rank, const GridArgs &g, const int32_t *cell_start,
                                             const int32_t *rank_xyz, const int32_t *lin2rank)
{
    const int lane = threadIdx.x % kWave;
    NbCell c;
    c.h0 = uni(cell_start[rank]);
    c.h1 = uni(cell_start[rank + 1]);
    c.m = c.total = 0;
    c.nodup = true;
    if (c.h0 == c.h1) return c;

    const int32_t pk = uni(rank_xyz[rank]);   // packed cell coordinates
    const int32_t c3[3] = {pk & 1023, (pk >> 10) & 1023, pk >> 20};
    for (int a = 0; a < 3; ++a) c.nodup &= g.nc[a] >= 2 * g.reach + 1;
    int32_t ax[5], ay[5], az[5], ix[5], iy[5], iz[5];
    const int mx = stencil_axis(c3[0], g.nc[0], g.reach, ax, ix);
    const int my = stencil_axis(c3[1], g.nc[1], g.reach, ay, iy);
    const int mz = stencil_axis(c3[2], g.nc[2], g.reach, az, iz);
    const int m = mx * my * mz;
    // stencil cells: lane t takes cells t and t + 64 (x-fastest order), reads
    // their ranges, and a shuffle scan forms the range prefix
    int32_t carry = 0;
    for (int t0 = 0; t0 < m; t0 += kWave) {
        const int t = t0 + lane;
        int32_t len = 0;
        if (t < m) {
            // t = a + mx (b + my c) for small mx, my: exact reciprocal multiplies
            const int q1 = (t * ((65536 + mx - 1) / mx)) >> 16;
            const int a = t - q1 * mx;
            const int cz = (q1 * ((65536 + my - 1) / my)) >> 16;
            const int b = q1 - cz * my;
            const int64_t l = ax[a] + int64_t(g.nc[0]) * (ay[b] + int64_t(g.nc[1]) * az[cz]);
            const int32_t r = lin2rank[l];
            const int32_t st = cell_start[r];
            len = cell_start[r + 1] - st;
            L.rstart[t] = st;
            L.rimg[t] = uint8_t((ix[a] + 1) | ((iy[b] + 1) << 2) | ((iz[cz] + 1) << 4));
        }
        int32_t v = len;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int32_t u = __shfl_up(v, o, kWave);
            if (lane >= o) v += u;
        }
        if (t < m) L.rbase[t + 1] = carry + v;
        carry += __builtin_amdgcn_readlane(v, kWave - 1);
    }
    if (lane == 0) L.rbase[0] = 0;
    wave_sync();
    if (carry <= kNbMap)   // tabulate the stencil cell of every candidate: lane t writes cell t's run
        for (int t = lane; t < m; t += kWave)
            for (int32_t q = L.rbase[t], e = L.rbase[t + 1]; q < e; ++q) L.cmap[q] = uint8_t(t);
    wave_sync();
    c.m = m;
    c.total = carry;
    return c;
}

// The stencil cell of candidate gq: tabulated, or the last range with
// rbase[k] <= gq (rbase[m] = total never is); top: highest power of two <= m.
template <class LDS>
__device__ __forceinline__ int nb_cell_of(const LDS &L, int32_t gq, int32_t m, int32_t total, int top)
{
    if (total <= kNbMap) return L.cmap[gq];
    int k = 0;
    for (int s = top; s > 0; s >>= 1) {
        const int t = min(k + s, m);
        k = L.rbase[t] <= gq ? t : k;
    }
    return k;
}

// *max_count only grows, so a wave whose longest row does not exceed a
// value already there has nothing to add: the check keeps the atomics on
// this one word (which the L2 serialises) to a few per launch.
__device__ __forceinline__ void nb_longest(int32_t longest, int32_t *max_count)
{
    for (int o = kWave / 2; o > 0; o >>= 1) longest = max(longest, __shfl_xor(longest, o, kWave));
    if (threadIdx.x % kWave == 0 &&
        longest > __hip_atomic_load(max_count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(max_count, longest);
}

// How a launch splits a cell's homes: `parts` wavefronts per cell, each
// taking every parts-th batch of `batch` homes.
struct NbSplit {
    int32_t parts, batch;
};

// Per-wave LDS state: the home atoms' positions (read back as broadcasts),
// the stencil's cell ranges with their periodic images, and the candidates
// that passed the bounding-box test, waiting for a register tile.
struct NbWaveLds {
    double hx[kWave], hy[kWave], hz[kWave];
    double box[6];                            // homes' bounding box: lo x, y, z, hi x, y, z
    int32_t rstart[kMaxStencil], rbase[kMaxStencil + 1];
    int32_t stage[kNbStage];
    uint8_t rimg[kMaxStencil];
    uint8_t cmap[kNbMap];                     // stencil cell of each candidate (up to kNbMap)
};

// A tile of candidates in registers: lane l holds candidates l, 64 + l, ...
struct NbTile {
    double x[kNbChunks], y[kNbChunks], z[kNbChunks];
    int32_t j[kNbChunks];
};

// Home atom i (position xi, yi, zi; r entries so far) against the first NC
// chunks of the tile: every hit is appended to the row at r in candidate
// order; returns the new row length.  All chunks are tested before any is
// stored, so the NC chains are independent; only lanes with a hit store,
// through a buffer whose range ends at the row capacity (stores past it are
// dropped).
template <int NC>
__device__ __forceinline__ uint32_t nb_home(const NbTile &T, double xi, double yi, double zi, int32_t i, uint32_t r,
                                            __amdgpu_buffer_rsrc_t row, double rl2, const GridArgs &g)
{
    uint64_t mk[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const double dx = minimg_sel(T.x[c] - xi, g.L[0], g.hL[0]);
        const double dy = minimg_sel(T.y[c] - yi, g.L[1], g.hL[1]);
        const double dz = minimg_sel(T.z[c] - zi, g.L[2], g.hL[2]);
        const double r2 = (dx * dx + dy * dy) + dz * dz;
        // the wave's hit mask straight from the two compares (r2 < rl2 as an
        // ordered less-than, so a +inf padding candidate never hits)
        mk[c] = __builtin_amdgcn_fcmp(r2, rl2, 4) & __builtin_amdgcn_ballot_w64(T.j[c] != i);
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        if (!mk[c]) continue;   // no hit in this chunk (wave-uniform)
        const uint32_t e = __builtin_amdgcn_mbcnt_hi(uint32_t(mk[c] >> 32),
                                                     __builtin_amdgcn_mbcnt_lo(uint32_t(mk[c]), r));
        // entry e of the row at byte (e / 8) * 256 + (e % 8) * 4
        if (__builtin_amdgcn_inverse_ballot_w64(mk[c]))   // this lane's bit of the mask
            __builtin_amdgcn_raw_buffer_store_b32(T.j[c], row, (e << 2) + __umul24(e >> 3, 224u), 0, 0);
        r += uint32_t(__popcll(mk[c]));
    }
    return r;
}

// The home batches of one cell against its stencil's candidates; returns the
// longest row of the cell.
//
// Candidates are streamed 256 at a time from the stencil's cell ranges.  With
// `filter`, a candidate is kept only if it lies within r_list of the
// bounding box of the batch's home atoms (in its periodic image of the
// stencil; with a margin of 1e-9 of r_list^2, far above the rounding of
// either test, so no candidate that the exact test accepts is dropped).
// Kept candidates are staged in LDS; every 256 of them fill a register
// tile, against which each home atom is tested with the exact FP64 test.
__device__ __forceinline__ int32_t nb_cell(NbWaveLds &L, int64_t n, const double *x, const GridArgs &g, double rl2,
                                           double keep2, const NbCell &cell, int32_t first, const NbSplit &sp,
                                           int32_t row_cap, int32_t *idx, int32_t *count)
{
    const int lane = threadIdx.x % kWave;
    const int32_t m = cell.m, total = cell.total;
    const bool filter = cell.nodup;
    int top = 1;                              // highest power of two <= m
    while (2 * top <= m) top *= 2;
    int32_t longest = 0;
    const double inf = __builtin_inf();
    // bytes of one row seen as a buffer: its last entry (row_cap - 1) ends there
    const uint32_t row_bytes = uint32_t(row_cap) * 32u - 224u;

    for (int32_t hb = cell.h0 + first; hb < cell.h1; hb += sp.parts * sp.batch) {
        const int32_t hn = min(sp.batch, cell.h1 - hb);
        const int32_t hl = hb + min(lane, hn - 1);
        const double xh = x[hl], yh = x[n + hl], zh = x[2 * n + hl];
        L.hx[lane] = xh;
        L.hy[lane] = yh;
        L.hz[lane] = zh;
        // bounding box of the batch's homes (lanes past hn repeat the last home)
        if (filter) {
            const double b0 = wave_min(xh), b1 = wave_min(yh), b2 = wave_min(zh);
            const double b3 = wave_max(xh), b4 = wave_max(yh), b5 = wave_max(zh);
            if (lane == 0) {
                L.box[0] = b0, L.box[1] = b1, L.box[2] = b2;
                L.box[3] = b3, L.box[4] = b4, L.box[5] = b5;
            }
        }
        // first int32 of the lane's home row (slice block + position in the slice)
        const int64_t row_l = int64_t(hl >> 3) * row_cap * 8 + (hl & 7) * 8;
        wave_sync();
        int32_t run_l = 0;                                // row length of home atom `lane`
        int32_t fill = 0;                                 // staged candidates (wave-uniform)
        for (int32_t t0 = 0; t0 < total; t0 += kNbTile) {
            // a raw tile of up to 256 candidates, four independent chunks
            bool keep[kNbChunks];
            int32_t jr[kNbChunks];
#pragma unroll
            for (int c = 0; c < kNbChunks; ++c) {
                const int32_t gq = t0 + c * kWave + lane;
                keep[c] = false;
                jr[c] = 0;
                if (gq < total) {
                    const int k = nb_cell_of(L, gq, m, total, top);
                    const int32_t j = L.rstart[k] + (gq - L.rbase[k]);
                    jr[c] = j;
                    keep[c] = true;
                    if (filter) {
                        double cx = x[j], cy = x[n + j], cz = x[2 * n + j];
                        const int32_t im = L.rimg[k];
                        cx += double((im & 3) - 1) * g.L[0];
                        cy += double(((im >> 2) & 3) - 1) * g.L[1];
                        cz += double(((im >> 4) & 3) - 1) * g.L[2];
                        const double dx = fmax(fmax(L.box[0] - cx, cx - L.box[3]), 0.0);
                        const double dy = fmax(fmax(L.box[1] - cy, cy - L.box[4]), 0.0);
                        const double dz = fmax(fmax(L.box[2] - cz, cz - L.box[5]), 0.0);
                        keep[c] = __builtin_fma(dz, dz, __builtin_fma(dy, dy, dx * dx)) < keep2;
                    }
                }
            }
#pragma unroll
            for (int c = 0; c < kNbChunks; ++c) {
                const uint64_t mk = __builtin_amdgcn_ballot_w64(keep[c]);
                if (keep[c])
                    L.stage[fill + int32_t(__builtin_amdgcn_mbcnt_hi(uint32_t(mk >> 32),
                                                                     __builtin_amdgcn_mbcnt_lo(uint32_t(mk), 0u)))] =
                        jr[c];
                fill += __popcll(mk);
            }
            const bool last = t0 + kNbTile >= total;
            while (fill >= kNbTile || (last && fill > 0)) {
                wave_sync();
                const int32_t nt = min(fill, kNbTile);
                const int nch = (nt + kWave - 1) / kWave;
                NbTile T;
#pragma unroll
                for (int c = 0; c < kNbChunks; ++c) {
                    const int32_t q = c * kWave + lane;
                    T.j[c] = -1;
                    T.x[c] = T.y[c] = T.z[c] = inf;
                    if (q < nt) {
                        const int32_t jj = L.stage[q];
                        T.j[c] = jj;
                        T.x[c] = x[jj];
                        T.y[c] = x[n + jj];
                        T.z[c] = x[2 * n + jj];
                    }
                }
                for (int32_t h = 0; h < hn; ++h) {
                    const int32_t i = hb + h;
                    const uint32_t r = uint32_t(__builtin_amdgcn_readlane(run_l, h));
                    const int64_t ro = int64_t(uint32_t(__builtin_amdgcn_readlane(int32_t(row_l), h))) |
                                       (int64_t(__builtin_amdgcn_readlane(int32_t(row_l >> 32), h)) << 32);
                    const auto row = make_rsrc(idx + ro, row_bytes);
                    const double xi = L.hx[h], yi = L.hy[h], zi = L.hz[h];
                    uint32_t rn;
                    switch (nch) {
                    case 4: rn = nb_home<4>(T, xi, yi, zi, i, r, row, rl2, g); break;
                    case 3: rn = nb_home<3>(T, xi, yi, zi, i, r, row, rl2, g); break;
                    case 2: rn = nb_home<2>(T, xi, yi, zi, i, r, row, rl2, g); break;
                    default: rn = nb_home<1>(T, xi, yi, zi, i, r, row, rl2, g); break;
                    }
                    if (lane == h) run_l = int32_t(rn);
                }
                // candidates staged past the tile move to the front
                const int32_t left = fill - nt;
                int32_t v[kNbChunks];
#pragma unroll
                for (int c = 0; c < kNbChunks; ++c)
                    if (c * kWave + lane < left) v[c] = L.stage[nt + c * kWave + lane];
                wave_sync();
#pragma unroll
                for (int c = 0; c < kNbChunks; ++c)
                    if (c * kWave + lane < left) L.stage[c * kWave + lane] = v[c];
                fill = left;
                wave_sync();
            }
        }
        if (lane < hn) count[hb + lane] = run_l;
        longest = max(longest, lane < hn ? run_l : 0);
        wave_sync();
    }
    return longest;
}

// ---- boxes of fewer than 2 reach + 2 cells on an axis, lengths past FP32 ----
// One wavefront per cell (Morton rank) and part in one-wave blocks, no
// block-wide barriers.  The atoms of the up to 27 (125) neighbouring cells are
// contiguous runs of the sorted arrays; the wave streams them, keeps those
// within reach of its homes' bounding box, and tests each home atom against
// 64 kept candidates at a time, compacting hits with a ballot straight into
// the sliced-ELL rows (entry e of atom i at
// idx[(i/8 * row_cap/8 + e/8) * 64 + (i%8) * 8 + e%8]).  Row order: stencil
// cell (x fastest), then sorted index.  Rows longer than row_cap are counted
// but truncated (the row is written through a buffer whose range ends at
// entry row_cap, so stores past it are dropped); the longest row length is
// folded into *max_count.  A padding candidate gives +inf, so it never
// passes r^2 < r_list^2.  The bounding-box filter runs when no stencil offset
// was de-duplicated on any axis (nc >= 2 reach + 1): each stencil cell is then
// one periodic image, the only one that can lie within r_list of a home.
__global__ __launch_bounds__(kWave)
void k_neighbors_small(int64_t n, const double *x, GridArgs g, double rl2, double keep2, NbSplit sp,
                       const int32_t *cell_start, const int32_t *rank_xyz, const int32_t *lin2rank, int32_t row_cap,
                       int32_t *idx, int32_t *count, int32_t *max_count)
{
    __shared__ NbWaveLds L;
    const uint32_t part = blockIdx.x % uint32_t(sp.parts);
    const NbCell c = nb_stencil(L, blockIdx.x / uint32_t(sp.parts), g, cell_start, rank_xyz, lin2rank);
    if (c.h0 == c.h1) return;
    nb_longest(nb_cell(L, n, x, g, rl2, keep2, c, int32_t(part) * sp.batch, sp, row_cap, idx, count), max_count);
}

// ---- the matrix-core build ----
typedef float nm_f32x4 __attribute__((ext_vector_type(4)));

template <int R, int D>
struct NmLds {
    static constexpr int kCells = (2 * R + 1) * (2 * R + 1) * (2 * R + 1);
    static constexpr int kStage = (D + 1) * kWave;   // staged candidates: a rest plus what D chunks of 64 keep
    float4 stage[kStage];          // kept candidates: position from the batch's centre, its square
    float4 home[kWave];              // homes: -2 x, -2 y, -2 z, 1
    float hom2[kWave];               // |home|^2 - r_list^2
    int32_t run[kWave], off[kWave];  // homes: row length so far, byte offset of the row in the batch's rows
    int32_t stage_j[kStage];
    int32_t shift[kCells];           // stencil cell: its first atom minus the candidates before it
    int32_t rbase[kCells + 1];       // candidates before it
    int8_t img[kCells][4];           // its periodic image
    uint8_t cmap[kNbMap];
};

template <bool MAX>
__device__ __forceinline__ float wave_extreme(float v)
{
    auto pick = [](float a, float b) { return MAX ? fmaxf(a, b) : fminf(a, b); };
#define MD_DPP(ctrl, rows) \
    v = pick(v, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), ctrl, rows, 0xf, false)))
    MD_DPP(0xb1, 0xf);    // lane ^ 1
    MD_DPP(0x4e, 0xf);    // lane ^ 2
    MD_DPP(0x141, 0xf);   // mirrored within 8
    MD_DPP(0x140, 0xf);   // mirrored within 16
    MD_DPP(0x142, 0xa);   // rows 1 and 3 take row 0's and 2's last lane
    MD_DPP(0x143, 0xc);   // rows 2 and 3 take lane 31
#undef MD_DPP
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), kWave - 1));
}

// Low (HI = 0) or high halves of two words side by side: one scalar
// instruction, which the compiler does not find from shifts and masks.
template <int HI>
__device__ __forceinline__ uint32_t pack16(uint32_t a, uint32_t b)
{
    uint32_t r;
    if (HI) asm("s_pack_hh_b32_b16 %0, %1, %2" : "=s"(r) : "s"(a), "s"(b));
    else asm("s_pack_ll_b32_b16 %0, %1, %2" : "=s"(r) : "s"(a), "s"(b));
    return r;
}

// v with `val` (wave-uniform) in lane LANE
template <int LANE>
__device__ __forceinline__ int32_t put_lane(int32_t v, uint32_t val)
{
    asm("v_writelane_b32 %0, %1, %2" : "+v"(v) : "s"(val), "n"(LANE));
    return v;
}

// Home H of a 16-home tile against 64 candidates: the hits of its mask
// (registers S, see nm_chunk) appended to its row in candidate order.  run,
// off: row length and row offset of home `lane` of the tile.
template <int H>
__device__ __forceinline__ void nm_home(const uint64_t (&S)[4][4], int32_t jj, __amdgpu_buffer_rsrc_t rows,
                                        int32_t off, uint32_t row_cap, int32_t &run)
{
    constexpr int r = H & 3, q = H >> 2;
    auto word = [&](int c) { return q < 2 ? uint32_t(S[c][r]) : uint32_t(S[c][r] >> 32); };
    const uint64_t mk = uint64_t(pack16<q & 1>(word(0), word(1))) | (uint64_t(pack16<q & 1>(word(2), word(3))) << 32);
    if (!mk) return;   // no hit (wave-uniform)
    const uint32_t r0 = uint32_t(__builtin_amdgcn_readlane(run, H));
    const uint32_t so = uint32_t(__builtin_amdgcn_readlane(off, H));
    const uint32_t r1 = r0 + uint32_t(__popcll(mk));
    const uint32_t e = __builtin_amdgcn_mbcnt_hi(uint32_t(mk >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(mk), r0));
    const uint32_t at = (e << 2) + __umul24(e >> 3, 224u);   // entry e of the row: byte (e / 8) * 256 + (e % 8) * 4
    uint64_t put = mk;
    if (__builtin_expect(r1 > row_cap, 0)) put &= __builtin_amdgcn_ballot_w64(e < row_cap);
    if (__builtin_amdgcn_inverse_ballot_w64(put)) __builtin_amdgcn_raw_buffer_store_b32(jj, rows, at, so, 0);
    run = put_lane<H>(run, r1);
}

// The rows of one batch of homes against 64 staged candidates at `base`.
//
// v_mfma_f32_16x16x4_f32 (A 16x4: lane = row + 16 k; B 4x16: lane = column +
// 16 k; D: lane = column + 16 (row / 4), register row % 4) gives
// |h|^2 - r_list^2 - 2 h.c + |c|^2 of 16 homes and 16 candidates at once.  A
// compare of one register is then the hit mask of four homes x 16
// candidates, and two 16-bit packs make it a home's mask over 64 candidates.
// Values within `eps` of zero (their rounding error is below that) are
// decided by the definition in FP64.
template <class LDS>
__device__ __forceinline__ void nm_chunk(LDS &L, int32_t base, int64_t n, const double *x, const GridArgs &g,
                                         double rl2, float eps, int32_t hb, int32_t hn, int32_t self,
                                         __amdgpu_buffer_rsrc_t rows, uint32_t row_cap)
{
    const int lane = threadIdx.x % kWave, li = lane & 15, gq = lane >> 4;
    const float *st = reinterpret_cast<const float *>(L.stage + base);
    float b[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) b[c] = st[(16 * c + li) * 4 + gq];
    const int32_t jj = L.stage_j[base + lane];
    const bool own = self < kWave && self + hn > 0;   // some home is among these candidates
    for (int32_t t = 0; t < hn; t += 16) {
        const float a = reinterpret_cast<const float *>(L.home + t + li)[gq];
        const nm_f32x4 c2 = *reinterpret_cast<const nm_f32x4 *>(L.hom2 + t + 4 * gq);
        int32_t run = L.run[t + li];
        const int32_t off = L.off[t + li];
        nm_f32x4 D[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) D[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b[c], c2, 0, 0, 0);
        if (own) {   // a home is no neighbour of its own
            const int32_t d = self + t + 4 * gq - li;
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r) D[c][r] = d + r == 16 * c ? 1e30f : D[c][r];
        }
        float near = __builtin_inff();
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            near = fminf(fminf(near, fabsf(D[c][0])), fabsf(D[c][1]));
            near = fminf(fminf(near, fabsf(D[c][2])), fabsf(D[c][3]));
        }
        if (__builtin_amdgcn_fcmpf(near, eps, 5)) {   // any lane: ordered less or equal
            uint32_t open = 0, hit = 0;   // bit 4 c + r: undecided values of this lane, those found to be hits
#pragma unroll
            for (int q = 0; q < 16; ++q) open |= fabsf(D[q >> 2][q & 3]) <= eps ? 1u << q : 0u;
            for (uint32_t m = open; __builtin_amdgcn_ballot_w64(m != 0); m &= m - 1) {
                const int q = m ? __builtin_ctz(m) : 0;
                const int32_t j = __shfl(jj, 4 * (q & 12) + li, kWave);
                if (m) {
                    const int32_t i = hb + t + 4 * gq + (q & 3);
                    const double dx = minimg_sel(x[j] - x[i], g.L[0], g.hL[0]);
                    const double dy = minimg_sel(x[n + j] - x[n + i], g.L[1], g.hL[1]);
                    const double dz = minimg_sel(x[2 * n + j] - x[2 * n + i], g.L[2], g.hL[2]);
                    hit |= (dx * dx + dy * dy) + dz * dz < rl2 ? 1u << q : 0u;
                }
            }
#pragma unroll
            for (int q = 0; q < 16; ++q)
                if (open & (1u << q)) D[q >> 2][q & 3] = hit & (1u << q) ? -1.f : 1.f;
        }
        uint64_t S[4][4];
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) S[c][r] = __builtin_amdgcn_fcmpf(D[c][r], 0.f, 4);   // ordered less-than
        // homes past hn have empty masks
#define NM_HOME(h) nm_home<h>(S, jj, rows, off, row_cap, run)
        NM_HOME(0); NM_HOME(1); NM_HOME(2); NM_HOME(3);
        if (t + 4 < hn) {
            NM_HOME(4); NM_HOME(5); NM_HOME(6); NM_HOME(7);
            if (t + 8 < hn) {
                NM_HOME(8); NM_HOME(9); NM_HOME(10); NM_HOME(11);
                if (t + 12 < hn) {
                    NM_HOME(12); NM_HOME(13); NM_HOME(14); NM_HOME(15);
                }
            }
        }
#undef NM_HOME
        if (lane < 16) L.run[t + lane] = run;
    }
}

// The homes of cell `rank` (those of `part`) against its stencil's
// candidates; returns the longest row.  Candidates are read D chunks of 64 at a
// time; one is kept if it lies within r_list of the bounding box of the batch's homes, in its periodic image of
// the stencil (FP32 positions from the box's centre, margin 1e-5 of r_list^2,
// far above their rounding), or is one of the homes itself, which keeps these
// consecutive in the stage.
template <int R, int D>
__device__ __forceinline__ int32_t nm_cell(NmLds<R, D> &L, int64_t rank, int32_t part, int64_t n, const double *x,
                                           const GridArgs &g, double rl2, const NbSplit &sp,
                                           const int32_t *cell_start, const int32_t *rank_xyz,
                                           const int32_t *lin2rank, int32_t row_cap, int32_t *idx, int32_t *count)
{
    constexpr int W = 2 * R + 1, kCells = W * W * W;
    const int lane = threadIdx.x % kWave;
    const int32_t pk = rank_xyz[rank];   // packed cell coordinates
    const int32_t h0 = uni(cell_start[rank]), h1 = uni(cell_start[rank + 1]);
    int32_t hb = h0 + part * sp.batch;
    if (hb >= h1) return 0;
    double xh, yh, zh;
    auto homes = [&](int32_t hn) {   // lanes past hn repeat the last home
        const int32_t hl = hb + min(lane, hn - 1);
        xh = x[hl], yh = x[n + hl], zh = x[2 * n + hl];
    };
    homes(min(sp.batch, h1 - hb));

    // the stencil (x fastest): lane t takes cells t and t + 64
    int32_t total = 0, centre = 0;
    bool interior = true;
#pragma unroll
    for (int t0 = 0; t0 < kCells; t0 += kWave) {
        const int t = t0 + lane;
        const int32_t cx = pk & 1023, cy = (pk >> 10) & 1023, cz = pk >> 20;
        int32_t vx = cx + t % W - R, vy = cy + (t / W) % W - R, vz = cz + t / (W * W) - R;
        const int32_t ix = vx < 0 ? -1 : (vx >= g.nc[0] ? 1 : 0), iy = vy < 0 ? -1 : (vy >= g.nc[1] ? 1 : 0),
                      iz = vz < 0 ? -1 : (vz >= g.nc[2] ? 1 : 0);
        int32_t st = 0, len = 0;
        if (t < kCells) {
            vx -= ix * g.nc[0], vy -= iy * g.nc[1], vz -= iz * g.nc[2];
            const int32_t r = lin2rank[vx + g.nc[0] * (vy + g.nc[1] * vz)];
            st = cell_start[r];
            len = cell_start[r + 1] - st;
        }
        interior &= !__builtin_amdgcn_ballot_w64(t < kCells && (ix | iy | iz));
        const int32_t end = total + wave_prefix(len), base = end - len;
        if (t < kCells) {
            L.shift[t] = st - base;
            L.rbase[t] = base;
            *reinterpret_cast<uint32_t *>(L.img[t]) = uint32_t(ix & 255) | uint32_t(iy & 255) << 8 | uint32_t(iz & 255) << 16;
        }
        if ((kCells - 1) / 2 >= t0 && (kCells - 1) / 2 < t0 + kWave)
            centre = __builtin_amdgcn_readlane(base, (kCells - 1) / 2 - t0);
        total = __builtin_amdgcn_readlane(end, kWave - 1);
    }
    if (lane == 0) L.rbase[kCells] = total;
    wave_sync();
    if (total <= kNbMap) {   // tabulate the stencil cell of every candidate
        constexpr int P = kCells <= kWave / 2 ? 2 : 1;   // lanes per stencil cell
        for (int t = lane / P; t < kCells; t += kWave / P)
            for (int32_t q = L.rbase[t] + lane % P, e = L.rbase[t + 1]; q < e; q += P) L.cmap[q] = uint8_t(t);
    }
    wave_sync();

    int32_t longest = 0;
    const float keep2 = float(rl2) * (1.f + 1e-5f), rl = __builtin_sqrtf(float(rl2));
    // sizes from four times the longest edge on (by the exponent: + 2)
    const uint32_t far = uint32_t(max(max(__double2hiint(g.L[0]), __double2hiint(g.L[1])), __double2hiint(g.L[2]))) + (2u << 20);
    while (hb < h1) {
        const int32_t hn = min(sp.batch, h1 - hb);
        // the slices of the batch as one buffer (at most 9 of them)
        const auto rows = make_rsrc(idx + int64_t(hb >> 3) * row_cap * 8, 9u * uint32_t(row_cap) * 32u);
        const int32_t hl = hb + min(lane, hn - 1);
        L.run[lane] = 0;
        L.off[lane] = int32_t(uint32_t((hl >> 3) - (hb >> 3)) * uint32_t(row_cap) * 32u + uint32_t(hl & 7) * 32u);
        // bounding box of the homes: its centre and half edges, through FP32
        // offsets from the first home.  Homes that are no number, or that FP64 could not
        // wrap into the box, take no part and have no hits: the others are as without
        // them, and the margins below stay in FP32 (with homes 1e18 apart `eps` passed the
        // 1e30 of the empty places, whose positions were then read past the last atom).
        // (Rows for such homes, of others as far out, by the definition: 340 -> 347 us.)
        const auto size = [](double v) { return uint32_t(__double2hiint(v)) & 0x7fffffffu; };   // of exponents first
        const bool near_box = max(max(size(xh), size(yh)), size(zh)) < far;
        const uint64_t in_box = __builtin_amdgcn_ballot_w64(near_box);
        const int src = in_box ? __builtin_ctzll(in_box) : 0;
        auto first = [&](double v) {
            return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), src),
                                    __builtin_amdgcn_readlane(__double2loint(v), src));
        };
        const double ox = first(xh), oy = first(yh), oz = first(zh);
        const float fx = near_box ? float(xh - ox) : 0.f, fy = near_box ? float(yh - oy) : 0.f,
                    fz = near_box ? float(zh - oz) : 0.f;
        const float lx = wave_extreme<false>(fx), ly = wave_extreme<false>(fy), lz = wave_extreme<false>(fz);
        const float ux = wave_extreme<true>(fx), uy = wave_extreme<true>(fy), uz = wave_extreme<true>(fz);
        const double mx = ox + double(0.5f * (lx + ux)), my = oy + double(0.5f * (ly + uy)),
                     mz = oz + double(0.5f * (lz + uz));
        const float bx = 0.5000004f * (ux - lx), by = 0.5000004f * (uy - ly), bz = 0.5000004f * (uz - lz);
        // rounding of the matrix-core squares: coordinates (2), |c|^2 (3),
        // |h|^2 - r_list^2 (1), four products and their sums (8), in units of
        // 2^-24 of (|h| + |c|)^2 + r_list^2 with |h| <= hd, |c| <= hd + r_list
        const float hd = __builtin_sqrtf(bx * bx + by * by + bz * bz) * 1.00001f;
        const float reach = 2.f * hd + rl * 1.00001f;
        const float eps = 16.f * 5.9604645e-8f * (reach * reach + keep2);
        const float px = float(xh - mx), py = float(yh - my), pz = float(zh - mz);
        const bool there = lane < hn && near_box;
        L.home[lane] = make_float4(there ? -2.f * px : 0.f, there ? -2.f * py : 0.f, there ? -2.f * pz : 0.f, 1.f);
        L.hom2[lane] = there ? float(double(px) * px + double(py) * py + double(pz) * pz - rl2) : 1e30f;
        const int32_t ts = centre + (hb - h0);   // candidate number of the first home
        int32_t self = 1 << 28;                  // its place in the stage, once staged

        int32_t j[D];
        uint32_t im[D];
        double cx[D], cy[D], cz[D];
        auto fetch = [&](int d, int32_t gq) {
            j[d] = 0, im[d] = 0, cx[d] = cy[d] = cz[d] = 0.0;
            if (gq >= total) return;
            int k = 0;
            if (total <= kNbMap) {
                k = L.cmap[gq];
            } else {   // the last cell with rbase <= gq
#pragma unroll
                for (int s = kCells > kWave ? 64 : 16; s > 0; s >>= 1) {
                    const int t = min(k + s, kCells);
                    k = L.rbase[t] <= gq ? t : k;
                }
            }
            j[d] = gq + L.shift[k];
            im[d] = *reinterpret_cast<const uint32_t *>(L.img[k]);
            cx[d] = x[j[d]], cy[d] = x[n + j[d]], cz[d] = x[2 * n + j[d]];
        };
        int32_t fill = 0;
        for (int32_t t0 = 0; t0 < total; t0 += D * kWave) {
#pragma unroll
            for (int d = 0; d < D; ++d) fetch(d, t0 + d * kWave + lane);
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const int32_t td = t0 + d * kWave;
                if (!interior) {
                    cx[d] += double(int8_t(im[d])) * g.L[0];
                    cy[d] += double(int8_t(im[d] >> 8)) * g.L[1];
                    cz[d] += double(int8_t(im[d] >> 16)) * g.L[2];
                }
                const float qx = float(cx[d] - mx), qy = float(cy[d] - my), qz = float(cz[d] - mz);
                const float dx = fmaxf(fabsf(qx) - bx, 0.f), dy = fmaxf(fabsf(qy) - by, 0.f),
                            dz = fmaxf(fabsf(qz) - bz, 0.f);
                const float d2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
                const bool keep = td + lane < total && (d2 < keep2 || uint32_t(j[d] - hb) < uint32_t(hn));
                const uint64_t mk = __builtin_amdgcn_ballot_w64(keep);
                const int32_t tl = ts - td;
                if (tl >= 0 && tl < kWave) self = fill + __popcll(mk & ((uint64_t(1) << tl) - 1));
                if (keep) {
                    const int32_t at = int32_t(__builtin_amdgcn_mbcnt_hi(
                        uint32_t(mk >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(mk), uint32_t(fill))));
                    L.stage[at] = make_float4(qx, qy, qz, __builtin_fmaf(qz, qz, __builtin_fmaf(qy, qy, qx * qx)));
                    L.stage_j[at] = j[d];
                }
                fill += __popcll(mk);
            }
            const bool last = t0 + D * kWave >= total;
            if (last && lane >= (fill & (kWave - 1)) && (fill & (kWave - 1))) {
                // candidates that no home hits fill the last chunk
                const int32_t at = (fill & ~(kWave - 1)) + lane;
                L.stage[at] = make_float4(0.f, 0.f, 0.f, 1e30f);
                L.stage_j[at] = 0;
            }
            wave_sync();
            int32_t done = 0;
            for (; fill - done >= kWave || (last && done < fill); done += kWave)
                nm_chunk(L, done, n, x, g, rl2, eps, hb, hn, self - done, rows, uint32_t(row_cap));
            if (!last && done > 0) {   // the rest moves to the front
                const int32_t left = fill - done;
                float4 p = make_float4(0.f, 0.f, 0.f, 0.f);
                int32_t q = 0;
                if (lane < left) {
                    p = L.stage[done + lane];
                    q = L.stage_j[done + lane];
                }
                wave_sync();
                if (lane < left) {
                    L.stage[lane] = p;
                    L.stage_j[lane] = q;
                }
                fill = left;
                self -= done;
            }
            wave_sync();
        }
        if (lane < hn) {
            const int32_t len = L.run[lane];
            count[hb + lane] = len;
            longest = max(longest, len);
        }
        hb += sp.parts * sp.batch;
        if (hb < h1) homes(min(sp.batch, h1 - hb));
        wave_sync();
    }
    return longest;
}

// One system, or the bricks of a decomposition (Bricks) in one launch: the cells of
// brick t follow those of brick t - 1, its atoms start at slot0[t] of the arrays, and
// it has an offsets array and a longest row of its own.
struct OneGrid {
    static constexpr bool many = false;
};
struct Bricks {
    static constexpr bool many = true;
    uint32_t n_cells;
    int32_t slot0[MD_DD_MAX_BRICKS];
};

template <int R, int D, class B>
__device__ __forceinline__ void nm_kernel(NmLds<R, D> &L, uint32_t blk, int64_t n, const double *x, const GridArgs &g,
                                          double rl2, const NbSplit &sp, const int32_t *cell_start,
                                          const int32_t *rank_xyz, const int32_t *lin2rank, int32_t row_cap,
                                          int32_t *idx, int32_t *count, int32_t *max_count, const B &bricks)
{
    uint32_t rank = blk / uint32_t(sp.parts);
    const uint32_t part = blk % uint32_t(sp.parts);
    if constexpr (B::many) {
        const uint32_t t = rank / bricks.n_cells;
        const int64_t s0 = bricks.slot0[t];
        rank -= t * bricks.n_cells;
        x += s0;
        cell_start += t * (bricks.n_cells + 1);
        idx += s0 * row_cap;
        count += s0;
        max_count += t;
    }
    nb_longest(nm_cell<R, D>(L, rank, int32_t(part), n, x, g, rl2, sp, cell_start, rank_xyz, lin2rank, row_cap, idx,
                             count),
               max_count);
}

// One wavefront per cell and part in one-wave blocks, as k_neighbors_small,
// for boxes of at least 2 reach + 2 cells on every axis: a stencil cell is
// then one periodic image and no home is further than half a box from a
// candidate in that image, so the minimum image of the definition is the
// image of the stencil (it differs only for pairs beyond half a box, which
// neither counts).  Same rows, same order, bit for bit.
//
// What bounds it: the addressers (busy 0.78 of the cycles on the porous system, 0.86 on
// copper) and the vector unit (issue 0.62, 0.68) together, neither of them full, and a
// chain of trips to memory per cell.  The FP64 test of every home against 64
// candidates took 8 FP64 operations, two compares and the broadcast of a home
// from LDS, ~27 vector instructions with the compaction; the squares now come
// from the matrix cores beside the vector unit (one compare per four homes
// and 16 candidates, a quarter of an instruction each for the check against
// rounding), ~10 vector and ~11 scalar instructions.  The build of 1.23 M
// atoms with voids went from 452 to 297 us (variants stripped at 315: set-up 40,
// reading and box test 75, squares and rows 195, of which stores 30), of 1 M
// copper atoms at 5.4 A from 334 to 223 us.
// Slower: 128 or 256 candidates read at once (LDS for fewer waves; 490 against
// 515 and 581 us for the whole rebuild of the void system), the next 64
// requested ahead (the registers cost more than the wait), 4, 5, 7 or 8 waves
// per SIMD.
template <int R, class B>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(6)))
void k_neighbors(int64_t n, const double *__restrict__ x, GridArgs g, double rl2, NbSplit sp,
                 const int32_t *__restrict__ cell_start, const int32_t *__restrict__ rank_xyz,
                 const int32_t *__restrict__ lin2rank, int32_t row_cap, int32_t *__restrict__ idx,
                 int32_t *__restrict__ count, int32_t *max_count, B bricks)
{
    __shared__ NmLds<R, 1> L;
    nm_kernel(L, xcd_chunked(blockIdx.x, gridDim.x, kNbXcdChunk), n, x, g, rl2, sp, cell_start, rank_xyz, lin2rank,
              row_cap, idx, count, max_count, bricks);
}

// The same with four chunks of candidates requested at once, for cells too few to
// fill the chip: a wavefront is then alone on its SIMD, and the trips to memory of
// its ~14 chunks, one after another, are a good part of its time (4,000 LJ atoms,
// 16 homes a wavefront: 34 us by single chunks, 31 by four; with 4 homes 23).
template <int R, class B>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(2)))
void k_neighbors_few(int64_t n, const double *__restrict__ x, GridArgs g, double rl2, NbSplit sp,
                     const int32_t *__restrict__ cell_start, const int32_t *__restrict__ rank_xyz,
                     const int32_t *__restrict__ lin2rank, int32_t row_cap, int32_t *__restrict__ idx,
                     int32_t *__restrict__ count, int32_t *max_count, B bricks)
{
    __shared__ NmLds<R, 4> L;
    nm_kernel(L, blockIdx.x, n, x, g, rl2, sp, cell_start, rank_xyz, lin2rank, row_cap, idx, count, max_count, bricks);
}

// Wavefronts per cell: one, unless the cells are too few to fill the chip
// (256 CUs x 4 SIMDs x 2); then batches of 16 homes (8 on the path without
// matrix cores), as many parts as an average cell has batches, and smaller
// batches, down to 4, while there is less than a wavefront a SIMD: the rows of
// a batch are written one after another (k_neighbors_few, 4,000 LJ atoms: 31 us with
// 16 homes a wavefront, 23 with 4).
constexpr int64_t kNbFew = 2048;   // cells

NbSplit nb_split(int64_t n, int64_t n_cells, bool small)
{
    if (n_cells >= kNbFew) return {1, kWave};
    int32_t batch = small ? 8 : 16;
    const auto parts = [&] { return (n + n_cells * batch - 1) / (n_cells * batch); };
    while (!small && batch > 4 && n_cells * parts() < kNbFew / 2) batch /= 2;
    return {int32_t(std::min<int64_t>(std::max<int64_t>(parts(), 1), 8)), batch};
}

// The matrix cores take squares of lengths in FP32, beside 1e30 for places that
// hold no atom: lengths between 1e-12 and 1e12 keep the squares below that and their
// rounding error, 1e-6 of r_list^2, above the smallest FP32 number.
static bool fp32_lengths(const md_grid_t *grid)
{
    bool ok = grid->r_list >= 1e-12;
    for (int a = 0; a < 3; ++a) ok = ok && grid->r_list <= 1e12 && grid->L[a] / grid->nc[a] <= 1e12;
    return ok;
}

int build_neighbors(const md_grid_t *grid, int64_t n, const double *x, const int32_t *cell_start, int32_t row_cap,
                    int32_t *idx, int32_t *count, int32_t *max_count, int32_t *needed, void *ws, const WsLayout &w,
                    hipStream_t s, bool cleared)
{
    const GridArgs g = grid_args(grid);
    const double rl2 = grid->r_list * grid->r_list;
    if (!cleared)
        if (int rc = launch_fill_i32(max_count, 1, 0, s)) return rc;
    if (n > 0) {
        const int32_t least = std::min(grid->nc[0], std::min(grid->nc[1], grid->nc[2]));
        // (rows of a million entries and more: nine slices of them pass a buffer's 32-bit range)
        const bool small = least < 2 * grid->reach + 2 || row_cap > (1 << 20) || !fp32_lengths(grid);
        const NbSplit sp = nb_split(n, grid->n_cells, small);
        const dim3 nb(uint32_t(grid->n_cells * sp.parts));
        const int32_t *xyz = ws_ptr<int32_t>(ws, w.rank2lin), *l2r = ws_ptr<int32_t>(ws, w.lin2rank);
        if (small)
            hipLaunchKernelGGL(k_neighbors_small, nb, dim3(kWave), 0, s, n, x, g, rl2, rl2 * (1.0 + 1e-9), sp,
                               cell_start, xyz, l2r, row_cap, idx, count, max_count);
        else {
            const bool few = grid->n_cells < kNbFew;
            const auto kernel = grid->reach == 1 ? (few ? k_neighbors_few<1, OneGrid> : k_neighbors<1, OneGrid>)
                                                 : (few ? k_neighbors_few<2, OneGrid> : k_neighbors<2, OneGrid>);
            hipLaunchKernelGGL(kernel, nb, dim3(kWave), 0, s, n, x, g, rl2, sp, cell_start, xyz, l2r, row_cap, idx,
                               count, max_count, OneGrid{});
        }
        MD_HIP_TRY(hipGetLastError());
    }
    if (needed) {
        int32_t mc = 0;
        MD_HIP_TRY(hipMemcpyAsync(&mc, max_count, sizeof(int32_t), hipMemcpyDeviceToHost, s));
        MD_HIP_TRY(hipStreamSynchronize(s));
        *needed = mc;
        if (mc > row_cap) return MD_ERR_CAPACITY;
    }
    return MD_OK;
}

// The lists of all bricks: sorted positions x of component stride `slots` and the
// bricks' slots in it, (n_cells + 1) offsets per brick, longest[t] cleared before.
int build_neighbors_bricks(const md_grid_t *grid, int n_bricks, const int64_t *slot0, int64_t slots, const double *x,
                           const int32_t *cell_start, int32_t row_cap, int32_t *idx, int32_t *count, int32_t *longest,
                           void *ws, const WsLayout &w, hipStream_t s)
{
    const int64_t cells = grid->n_cells * n_bricks;
    // one by one: what the kernel does not take, and more threads than a launch can have
    // (2^32, beyond which cells are dropped without an error; a wavefront per cell, parts
    // only where cells are few)
    if (row_cap > (1 << 20) || cells * kWave > int64_t(UINT32_MAX) || grid->reach != 1 || !fp32_lengths(grid)) {
        for (int t = 0; t < n_bricks; ++t)
            if (int rc = build_neighbors(grid, slots, x + slot0[t], cell_start + t * (grid->n_cells + 1), row_cap,
                                         idx + slot0[t] * row_cap, count + slot0[t], longest + t, nullptr, ws, w, s))
                return rc;
        return MD_OK;
    }
    Bricks b;
    b.n_cells = uint32_t(grid->n_cells);
    for (int t = 0; t < n_bricks; ++t) b.slot0[t] = int32_t(slot0[t]);
    const NbSplit sp = nb_split(slots, cells, false);
    const auto kernel = cells < kNbFew ? k_neighbors_few<1, Bricks> : k_neighbors<1, Bricks>;
    hipLaunchKernelGGL(kernel, dim3(uint32_t(cells * sp.parts)), dim3(kWave), 0, s, slots, x, grid_args(grid),
                       grid->r_list * grid->r_list, sp, cell_start, ws_ptr<int32_t>(ws, w.rank2lin),
                       ws_ptr<int32_t>(ws, w.lin2rank), row_cap, idx, count, longest, b);
    MD_HIP_TRY(hipGetLastError());
    return MD_OK;
}

}  // namespace md
