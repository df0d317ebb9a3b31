// Device-wide scans, fills and deterministic reductions.
//
// The scan turns per-cell atom counts into cell offsets (counting sort).
// Reductions combine per-block FP64 partials in one fixed order, so energies,
// virials and kinetic energies are bitwise reproducible run to run.
#include "md_common.h"

namespace md {

__global__ __launch_bounds__(kBlock) void k_fill_i32(int32_t *p, int64_t count, int32_t value)
{
    const int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (i < count) p[i] = value;
}

int launch_fill_i32(int32_t *p, int64_t count, int32_t value, hipStream_t s)
{
    if (count <= 0) return MD_OK;
    const int64_t g = (count + kBlock - 1) / kBlock;
    hipLaunchKernelGGL(k_fill_i32, dim3(uint32_t(g)), dim3(kBlock), 0, s, p, count, value);
    MD_HIP_TRY(hipGetLastError());
    return MD_OK;
}

// inclusive scan of one int64 per thread over the block (wave shuffles + LDS)
__device__ __forceinline__ int64_t block_incl_scan(int64_t v, int64_t *lds /* kBlock/kWave */)
{
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        int64_t t = __shfl_up(v, o, kWave);
        if (lane >= o) v += t;
    }
    if (lane == kWave - 1) lds[wave] = v;
    __syncthreads();
    int64_t pre = 0;
    for (int w = 0; w < wave; ++w) pre += lds[w];
    __syncthreads();
    return v + pre;
}

// phase 1: sum of each tile of kScanTile inputs
__global__ __launch_bounds__(kBlock) void k_scan_tile_sums(const int32_t *in, int64_t m, int64_t *bsum)
{
    __shared__ int64_t lds[kBlock / kWave];
    const int64_t base = int64_t(blockIdx.x) * kScanTile + int64_t(threadIdx.x) * kScanItems;
    int64_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t q = base + k;
        if (q < m) s += in[q];
    }
    s = block_incl_scan(s, lds);
    if (threadIdx.x == kBlock - 1) bsum[blockIdx.x] = s;
}

// phase 2: exclusive scan of the tile sums in place (one block, any count)
__global__ __launch_bounds__(kBlock) void k_scan_tile_offsets(int64_t *bsum, int64_t nb)
{
    __shared__ int64_t lds[kBlock / kWave];
    __shared__ int64_t carry;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int64_t b0 = 0; b0 < nb; b0 += kBlock) {
        const int64_t q = b0 + threadIdx.x;
        const int64_t v = q < nb ? bsum[q] : 0;
        const int64_t inc = block_incl_scan(v, lds);
        const int64_t c = carry;
        if (q < nb) bsum[q] = c + inc - v;
        __syncthreads();
        if (threadIdx.x == kBlock - 1) carry = c + inc;
        __syncthreads();
    }
}

// phase 3: rescan each tile and write out[q+1] = inclusive prefix (out[0] = 0).
// SUMS: bsum holds the tiles' sums, and the block adds those before its own itself.
template <bool SUMS>
__global__ __launch_bounds__(kBlock) void k_scan_write(const int32_t *in, int64_t m, const int64_t *bsum,
                                                       int32_t *out)
{
    __shared__ int64_t lds[kBlock / kWave];
    __shared__ int64_t before;
    const int64_t base = int64_t(blockIdx.x) * kScanTile + int64_t(threadIdx.x) * kScanItems;
    int32_t v[kScanItems];
    int64_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t q = base + k;
        v[k] = q < m ? in[q] : 0;
        s += v[k];
    }
    int64_t off;
    if (SUMS) {
        int64_t t = 0;
        for (uint32_t q = threadIdx.x; q < blockIdx.x; q += kBlock) t += bsum[q];
        t = block_incl_scan(t, lds);
        if (threadIdx.x == kBlock - 1) before = t;
        __syncthreads();
        off = before;
    } else {
        off = bsum[blockIdx.x];
    }
    const int64_t inc = block_incl_scan(s, lds);
    int64_t run = off + inc - s;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t q = base + k;
        run += v[k];
        if (q < m) out[q + 1] = int32_t(run);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) out[0] = 0;
}

// The whole scan by one block (of each of gridDim.x sets), in rows of 1,024 inputs:
// a wavefront's runs of 64 first, then the runs' sums, 16 of each row.
constexpr int kScanOneBlock = 1024, kScanOneRows = 16, kScanOne = kScanOneBlock * kScanOneRows;
__global__ __launch_bounds__(kScanOneBlock) void k_scan_one(const int32_t *in, int32_t m, int32_t *out, int64_t stride)
{
    constexpr int kWaves = kScanOneBlock / kWave, kRuns = kScanOneRows * kWaves;
    static_assert(kRuns == 4 * kWave, "four runs a lane of the first wavefront");
    __shared__ int32_t run[kRuns];
    in += blockIdx.x * stride;
    out += blockIdx.x * stride;
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    int32_t v[kScanOneRows];
#pragma unroll
    for (int k = 0; k < kScanOneRows; ++k) {
        const int32_t q = k * kScanOneBlock + int32_t(threadIdx.x);
        v[k] = q < m ? in[q] : 0;
    }
#pragma unroll
    for (int k = 0; k < kScanOneRows; ++k) {
        v[k] = wave_prefix(v[k]);
        if (lane == kWave - 1) run[k * kWaves + wave] = v[k];
    }
    __syncthreads();
    if (wave == 0) {
        int32_t r[4], s = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            r[q] = s;
            s += run[4 * lane + q];
        }
        const int32_t before = wave_prefix(s) - s;
#pragma unroll
        for (int q = 0; q < 4; ++q) run[4 * lane + q] = before + r[q];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kScanOneRows; ++k) {
        const int32_t q = k * kScanOneBlock + int32_t(threadIdx.x);
        if (q < m) out[q + 1] = run[k * kWaves + wave] + v[k];
    }
    if (threadIdx.x == 0) out[0] = 0;
}

// Launches are what a scan of cell counts costs (2 to 5 us each with the gap before
// it): one up to 16,384 values (3.8 us; three launches of 7.5 us before); two
// while a block can add the sums of the tiles before it in a few loads a thread
// (4 M values; 74,000 take 7.9 us, three launches took 10.5); else three.
constexpr int64_t kScanSelf = 2048;   // tiles

int launch_scan_i32_to_i32(const int32_t *in, int32_t *out, int64_t m, int64_t *bsum, hipStream_t s)
{
    return launch_scan_sets(in, out, m, 1, 0, bsum, s);
}

int launch_scan_sets(const int32_t *in, int32_t *out, int64_t m, int sets, int64_t stride, int64_t *bsum, hipStream_t s)
{
    if (m <= kScanOne) {
        hipLaunchKernelGGL(k_scan_one, dim3(uint32_t(sets)), dim3(kScanOneBlock), 0, s, in, int32_t(m > 0 ? m : 0), out,
                           stride);
        MD_HIP_TRY(hipGetLastError());
        return MD_OK;
    }
    const int64_t nb = (m + kScanTile - 1) / kScanTile;
    for (int k = 0; k < sets; ++k, in += stride, out += stride) {
        hipLaunchKernelGGL(k_scan_tile_sums, dim3(uint32_t(nb)), dim3(kBlock), 0, s, in, m, bsum);
        if (nb <= kScanSelf) {
            hipLaunchKernelGGL(k_scan_write<true>, dim3(uint32_t(nb)), dim3(kBlock), 0, s, in, m, bsum, out);
        } else {
            hipLaunchKernelGGL(k_scan_tile_offsets, dim3(1), dim3(kBlock), 0, s, bsum, nb);
            hipLaunchKernelGGL(k_scan_write<false>, dim3(uint32_t(nb)), dim3(kBlock), 0, s, in, m, bsum, out);
        }
        MD_HIP_TRY(hipGetLastError());
    }
    return MD_OK;
}

// Fixed-order sums of [rows][8] partials, `stride` rows apart.  Thread t adds
// column t % 8 of rows t / 8, t / 8 + T / 8, ... (a wavefront reads 8 whole
// rows at a time), then a fixed tree combines the T / 8 row classes; the
// totals end in lds[0 .. 7].
template <int T>
__device__ __forceinline__ void reduce_rows(const double *part, int64_t rows, int64_t stride, double *lds /* T / 8 */)
{
    const int col = threadIdx.x % 8, lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    double s = 0.0;
#pragma unroll 8
    for (int64_t r = threadIdx.x / 8; r < rows; r += T / 8) s += part[r * stride * 8 + col];
#pragma unroll
    for (int o = 8; o < kWave; o <<= 1) s += __shfl_xor(s, o, kWave);
    if (lane < 8) lds[wave * 8 + col] = s;
    __syncthreads();
    if (threadIdx.x < 8) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < T / kWave; ++w) t += lds[w * 8 + col];
        lds[col] = t;
    }
    __syncthreads();
}

// Rows [b C, (b + 1) C) of part1 (blockIdx.y = 0) or part2 (1) summed into
// row b C, in place: the block has read its rows before it writes.
__global__ __launch_bounds__(kBlock) void k_reduce_chunks(double *part1, int64_t nb1, double *part2, int64_t nb2,
                                                          int64_t C)
{
    __shared__ double lds[kBlock / 8];
    double *part = blockIdx.y ? part2 : part1;
    const int64_t r0 = int64_t(blockIdx.x) * C, left = (blockIdx.y ? nb2 : nb1) - r0;
    if (left <= 0) return;
    reduce_rows<kBlock>(part + r0 * 8, left < C ? left : C, 1, lds);
    if (threadIdx.x < 8) part[r0 * 8 + threadIdx.x] = lds[threadIdx.x];
}

// mode kReduceLJ : rows = [sum e, pair count, w0..w5] over a full list (every
//                  pair twice): out = [e/2, e/2 - count/2 * a0, w/2]; a0 = Phi(rc)
// mode kReduceEAM: part1 rows = [E_embed, ...], part2 rows = [sum V, 0, w0..w5]
//                  out = [E_embed + V/2, E_embed, w/2]
// mode kReduceKE : rows = [sum v^2, ...]; out[0] = a0 * sum / 2 (a0 = mass)
constexpr int kReduceBlock = 1024;
// Rows (every C-th of nb) that one block sums itself: 2,048 rows are 16 loads
// per thread, about one extra launch's time.
constexpr int64_t kReduceDirect = 2048;
constexpr int64_t kReduceBlocks = 1024;   // chunks at most above that

__global__ __launch_bounds__(kReduceBlock) void k_reduce_partials(const double *part1, int64_t rows1,
                                                                  const double *part2, int64_t rows2, int64_t stride,
                                                                  double *out, int mode, double a0)
{
    __shared__ double lds1[kReduceBlock / 8], lds2[kReduceBlock / 8];
    reduce_rows<kReduceBlock>(part1, rows1, stride, lds1);
    if (part2) reduce_rows<kReduceBlock>(part2, rows2, stride, lds2);
    if (threadIdx.x != 0) return;
    const double *r1 = lds1, *r2 = lds2;
    if (mode == kReduceLJ) {
        out[0] = 0.5 * r1[0];
        out[1] = 0.5 * r1[0] - 0.5 * r1[1] * a0;
        for (int c = 2; c < 8; ++c) out[c] = 0.5 * r1[c];
    } else if (mode == kReduceEAM) {
        out[0] = r1[0] + 0.5 * r2[0];
        out[1] = r1[0];
        for (int c = 2; c < 8; ++c) out[c] = 0.5 * r2[c];
    } else {
        out[0] = 0.5 * a0 * r1[0];
    }
}

// One block over all rows when they are few; otherwise chunks of C rows are
// summed first, on all CUs (the partials of 4 M atoms are 2 x 125,000 rows,
// 16 MB; half a million copper atoms: one block over 2 x 15,625 rows took
// 48 us of the 163 us of an energy evaluation, two launches take 9.4 of 120).
int launch_reduce_partials(double *part1, int64_t nb1, double *part2, int64_t nb2, double *out, int mode, double a0,
                           hipStream_t s)
{
    const int64_t nb = nb1 > nb2 ? nb1 : nb2;
    int64_t C = 1;
    if (nb > kReduceDirect) {
        C = (nb + kReduceBlocks - 1) / kReduceBlocks;
        if (C < 64) C = 64;
        hipLaunchKernelGGL(k_reduce_chunks, dim3(uint32_t((nb + C - 1) / C), part2 ? 2 : 1), dim3(kBlock), 0, s, part1,
                           nb1, part2, nb2, C);
    }
    hipLaunchKernelGGL(k_reduce_partials, dim3(1), dim3(kReduceBlock), 0, s, part1, (nb1 + C - 1) / C, part2,
                       (nb2 + C - 1) / C, C, out, mode, a0);
    MD_HIP_TRY(hipGetLastError());
    return MD_OK;
}

}  // namespace md
