// Cells of a grid and the pieces of its counting sort that the binning of a
// whole system and of the bricks of a decomposition share.
#pragma once

#include "md_common.h"

namespace md {

struct GridArgs {
    double L[3], hL[3], inv_cell[3];
    int32_t nc[3], reach;
};

// Inside the box floor(x / L) is 0 (a quotient below 1 never rounds up to 1) and w
// is x (0 for -0), so the FP64 division is left out: most atoms at a build are
// where the last one put them.
__device__ __forceinline__ double wrap1(double x, double L)
{
    if (x >= 0.0 && x < L) return x + 0.0;
    double w = x - L * floor(x / L);
    if (w >= L) w -= L;
    if (w < 0.0) w += L;
    return w;
}

__device__ __forceinline__ int32_t cell1(double w, double inv, int32_t nc)
{
    int32_t c = int32_t(w * inv);
    c = c >= nc ? nc - 1 : c;
    return c < 0 ? 0 : c;
}

// A place among the atoms of cell r, counted in cnt[r] (any order; all active lanes
// of the wave call it).
__device__ __forceinline__ int32_t claim_slot(int32_t r, int32_t *cnt)
{
    // one atomic per distinct cell of the wave (atoms arrive nearly sorted):
    // the first lane of a cell claims a run of slots for all lanes of the cell,
    // which take consecutive slots in lane order.  The lanes are grouped first
    // and the claims of all groups made by one instruction: made one group after
    // another, their round trips to the L2 (~6 a wave) were the kernel's time.
    const int lane = threadIdx.x % kWave;
    int leader = lane;
    uint32_t before = 0;
    int32_t members = 0;
    uint64_t todo = __ballot(true);
    while (todo) {
        const int first = __builtin_ctzll(todo);
        const int32_t rc = __builtin_amdgcn_readlane(r, first);
        const uint64_t same = __ballot(r == rc) & todo;
        if (r == rc && ((todo >> lane) & 1u)) {
            leader = first;
            members = __popcll(same);
            before = __builtin_amdgcn_mbcnt_hi(uint32_t(same >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(same), 0u));
        }
        todo &= ~same;
    }
    int32_t base = 0;
    if (leader == lane) base = atomicAdd(&cnt[r], members);
    return __shfl(base, leader, kWave) + int32_t(before);
}

// How many of tmp[s0 .. s1) are below i: the place of atom i in input order among
// the atoms of its cell.
__device__ __forceinline__ int32_t stable_rank(const int32_t *tmp, int32_t s0, int32_t s1, int32_t i)
{
    int32_t rank = 0;
    for (int32_t q = s0; q < s1; q += 8) {   // eight loads in flight
        int32_t m[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) m[k] = tmp[min(q + k, s1 - 1)];
#pragma unroll
        for (int k = 0; k < 8; ++k) rank += q + k < s1 && m[k] < i;
    }
    return rank;
}

inline GridArgs grid_args(const md_grid_t *grid)
{
    GridArgs g;
    for (int a = 0; a < 3; ++a) {
        g.L[a] = grid->L[a];
        g.hL[a] = 0.5 * grid->L[a];
        g.inv_cell[a] = grid->inv_cell[a];
        g.nc[a] = grid->nc[a];
    }
    g.reach = grid->reach;
    return g;
}

}  // namespace md
