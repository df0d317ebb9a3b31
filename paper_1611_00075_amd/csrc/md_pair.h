// Pair-loop building blocks shared by the force kernels: compensated
// accumulation, displacements from scaled coordinates, the sliced-ELL row
// walk and the cross-lane combine of an atom's 8 partial sums.
#pragma once

#include "md_common.h"

namespace md {

template <bool COMP>
__device__ __forceinline__ void acc_add(float &s, float &c, float a, float b)
{
    // s += a * b, with the running error of the sum compensated
    if (COMP) {
        const float y = __builtin_fmaf(a, b, -c);
        const float t = s + y;
        c = (t - s) - y;
        s = t;
    } else {
        s = __builtin_fmaf(a, b, s);
    }
}

// Displacement r_i - r_j from scaled coordinates.  CUBIC: in units of
// L/2^32 (no multiply); otherwise in physical units (ax = L_a / 2^32).
template <bool CUBIC>
__device__ __forceinline__ void disp(const uint4 &pi, const uint4 &pj, float ax, float ay, float az, float &dx,
                                     float &dy, float &dz)
{
    dx = float(int32_t(pi.x - pj.x));
    dy = float(int32_t(pi.y - pj.y));
    dz = float(int32_t(pi.z - pj.z));
    if (!CUBIC) {
        dx *= ax;
        dy *= ay;
        dz *= az;
    }
}

// Sliced-ELL row of atom i: entry e at row[(e / 8) * 64 + e % 8].
__device__ __forceinline__ const int32_t *ell_row(const int32_t *idx, int64_t i, int32_t cap)
{
    return idx + (int64_t(i / kSlice) * cap * kSlice + (i % kSlice) * kSlice);
}

__device__ __forceinline__ int64_t ell_pos(int32_t e) { return int64_t(e / kSlice) * (kSlice * kSlice) + e % kSlice; }

// s += v with the running error of the sum compensated (Kahan).
template <bool COMP>
__device__ __forceinline__ void acc_sum(float &s, float &c, float v)
{
    if (COMP) {
        const float y = v - c;
        const float t = s + y;
        c = (t - s) - y;
        s = t;
    } else {
        s += v;
    }
}

// Raw buffer resource over `bytes` bytes at `base` (gfx9 raw buffer
// semantics: a load at a byte offset >= bytes returns zero, so no load
// leaves the range).  base and bytes must be wave-uniform.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, int(bytes), 0x00020000);
}

// A list entry, read once a pass: with STREAM, past the caches (non-temporal).
// In a run's steps a list that the last-level cache (256 MB) cannot hold until the
// next step drives positions and velocities out of it; past it, these stay for
// the kick-drift and the gathers.  Us per step cached / streamed (bytes allocated
// for the rows): LJ of 666,000 atoms (264 MB) 87 / 91, of 864,000 (342 MB) 116 / 113, of
// 1.26 M (498 MB) 163 / 155, of 2 M 256 / 241; FS of 0.78 M Cu (190 MB) 129 / 149, of 1.15 M
// (280 MB) 211 / 210, of 2 M (500 MB) 365 / 355, of 4 M 692 / 693.  Evaluations alone gain
// nothing (FS of 4 M 650 / 651, LJ of 1.5 M 153 / 158) but the tabulated form's (2.9 M
// 579 / 556).
constexpr int64_t kStreamBytes = int64_t(300) << 20;
inline bool streams(int64_t n, int32_t cap) { return n * cap * 4 > kStreamBytes; }

template <bool STREAM>
__device__ __forceinline__ uint32_t load_entry(const __amdgpu_buffer_rsrc_t &row_r, uint32_t off)
{
    return __builtin_amdgcn_raw_buffer_load_b32(row_r, off, 0, STREAM ? 2 : 0);
}

// Compile-time flag handed to a row walk's body: whether slots of the
// batch may lie past the row's end (the body must then mask them).
template <bool M>
struct Masked {
    static constexpr bool value = M;
};

// Row walk through buffer loads.  The wavefront holds one slice of 8 atoms
// (lane = 8 * atom + sub); the slice's block of the list is one buffer
// (row_r, cap * 32 bytes), in which entry sub + 8 q of the lane's atom sits
// at byte q * 256 + 4 * lane: one lane offset plus an immediate per load.
// Per iteration each lane reads U entries, then their U positions (xs_r,
// 16 bytes per atom, WORDS = 3 or 4 words read), then calls
// body(pj, t, Masked<true>) with the U positions of entries t + 8 u.  For
// entries past the row end both loads are given an offset outside their
// buffer, so they move no data and return zero; the body masks them
// (t + 8 u >= cnt).
//
// MASKED = false drops the two per-slot selects: slots past the row end read
// whatever index the row holds there (or zero past the row's buffer), and
// the position load of any such index stays inside the positions' buffer
// or returns zero; the body masks those slots as before.  Fewer vector
// instructions for more gathered bytes: it pays for the forms whose pair
// terms are longest (the two-element tight-binding form).
template <int U, int WORDS, bool MASKED, bool STREAM, typename Body>
__device__ __forceinline__ void walk_buf(const __amdgpu_buffer_rsrc_t &xs_r, const __amdgpu_buffer_rsrc_t &row_r,
                                         int32_t cnt, int sub, Body &&body)
{
    constexpr uint32_t kOut = 0xfffffff0u;   // beyond any buffer here
    uint32_t off = (threadIdx.x % kWave) * 4u;
    for (int32_t t = sub; t < cnt; t += U * kSlice, off += U * 256u) {
        bool ok[U];
        uint32_t j[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            ok[u] = !MASKED || t + u * kSlice < cnt;
            j[u] = load_entry<STREAM>(row_r, ok[u] ? off + u * 256u : kOut);
        }
        uint4 pj[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t o = ok[u] ? j[u] << 4 : kOut;
            if (WORDS == 4) {
                const auto v = __builtin_amdgcn_raw_buffer_load_b128(xs_r, o, 0, 0);
                pj[u] = make_uint4(v[0], v[1], v[2], v[3]);
            } else {
                const auto v = __builtin_amdgcn_raw_buffer_load_b96(xs_r, o, 0, 0);
                pj[u] = make_uint4(v[0], v[1], v[2], 0u);
            }
        }
        body(pj, t, Masked<true>{});
    }
}

// Row walk in two parts.  Full batches: while all U entries t + 8 u of the
// lane are inside the row, body(pj, t, Masked<false>) gets U positions, all
// of them real neighbours, with no per-slot selects.  Tail (1 to U - 1
// entries left): one batch of U - 1 slots, body(pj, t, Masked<true>) with pj
// of length U - 1 and zeros in the slots past the end.  A lane thus evaluates
// fewer slots than U * ceil(cnt / 8U).
//
// Order of the loads: a batch's positions, then the next batch's list
// entries, then the arithmetic.  Loads return in the order of their issue, so
// with the entries (a miss to HBM) behind the positions (cache hits) the
// arithmetic waits for the positions alone and the entries travel meanwhile;
// entries first makes every batch wait for HBM, and entries only after the
// arithmetic leaves the list stream idle during it.  sched_barrier holds the
// compiler to this order.  Entries after the arithmetic against this order:
// LJ, 1.23 M atoms with voids, 114.3 -> 111.3 us; FS, 4 M Cu, both passes
// 602 -> 587 us; tabulated, 1 M Cu, 173.3 -> 166.5 us; same bits.
//
// Loads past the row's end are switched off in the execution mask: given an
// out-of-range offset instead, a lane still passes through the gather's
// address processing and issue (LJ 117 us).  (What bounds the pair kernels is
// the list stream, 4 bytes per entry read once, together with the pair
// arithmetic; entries in 16-byte loads, four consecutive ones per lane, ran
// LJ at 122-129 us: the lanes of a gather then spread over 32 entries of a
// row instead of 8 adjacent ones.)
template <int U, int WORDS, bool STREAM, typename Body>
__device__ __forceinline__ void walk_split(const __amdgpu_buffer_rsrc_t &xs_r, const __amdgpu_buffer_rsrc_t &row_r,
                                           int32_t cnt, int sub, Body &&body)
{
    static_assert(U > 1, "a tail batch holds U - 1 slots");
    auto pos = [&](uint32_t o) {
        if (WORDS == 4) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b128(xs_r, o, 0, 0);
            return make_uint4(v[0], v[1], v[2], v[3]);
        } else {
            const auto v = __builtin_amdgcn_raw_buffer_load_b96(xs_r, o, 0, 0);
            return make_uint4(v[0], v[1], v[2], 0u);
        }
    };
    uint32_t off = (threadIdx.x % kWave) * 4u;
    int32_t t = sub;
    uint32_t j[U];   // entries of the batch at t (zeros past the row's end)
    auto entries = [&]() {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            j[u] = 0u;
            if (t + u * kSlice < cnt) j[u] = load_entry<STREAM>(row_r, off + u * 256u);
        }
    };
    entries();
    while (t + (U - 1) * kSlice < cnt) {
        uint4 pj[U];
#pragma unroll
        for (int u = 0; u < U; ++u) pj[u] = pos(j[u] << 4);
        const int32_t t0 = t;
        t += U * kSlice;
        off += U * 256u;
        __builtin_amdgcn_sched_barrier(0);
        entries();
        __builtin_amdgcn_sched_barrier(0);
        body(pj, t0, Masked<false>{});
    }
    if (t < cnt) {
        constexpr int V = U - 1;
        uint4 pj[V];
#pragma unroll
        for (int u = 0; u < V; ++u) {
            pj[u] = make_uint4(0u, 0u, 0u, 0u);
            if (t + u * kSlice < cnt) pj[u] = pos(j[u] << 4);
        }
        body(pj, t, Masked<true>{});
    }
}

// The row walk of a pair form: split (SPLIT) or whole batches with no
// selects (walk_buf without masking).
template <bool SPLIT, int U, int WORDS, bool STREAM, typename Body>
__device__ __forceinline__ void walk_form(const __amdgpu_buffer_rsrc_t &xs_r, const __amdgpu_buffer_rsrc_t &row_r,
                                          int32_t cnt, int sub, Body &&body)
{
    if constexpr (SPLIT) walk_split<U, WORDS, STREAM>(xs_r, row_r, cnt, sub, body);
    else walk_buf<U, WORDS, false, STREAM>(xs_r, row_r, cnt, sub, body);
}

// The atoms a force launch covers: the slices from slice0 on, rows and
// outputs of atoms below n (the kernel's n argument); positions of the
// first n_xs atoms may be gathered (atoms from n to n_xs are ghost copies
// whose forces are not computed); force component c of atom i at
// f[c * fs + i].  Whole-system launches: n_xs = fs = n, slice0 = 0.
struct Span {
    int64_t n_xs;
    int64_t fs;
    uint32_t slice0;
};

__host__ __device__ inline Span whole(int64_t n) { return Span{n, n, 0u}; }

// Several bricks of a domain decomposition in one launch.  Logical block b
// belongs to brick e with blk0[e] <= b < blk0[e + 1]; for its blocks the
// kernel's position, list and count arrays start at the brick's first slot
// (slot0[e]) and its per-atom outputs at the brick's first atom (atom0[e]);
// its span is (n_xs[e], the launch's force stride, slice0[e]) over atoms
// below n_end[e] of the brick.
struct BrickTab {
    int32_t nb;
    int64_t blk0[MD_DD_MAX_BRICKS + 1];
    int64_t slot0[MD_DD_MAX_BRICKS], atom0[MD_DD_MAX_BRICKS], n_end[MD_DD_MAX_BRICKS], n_xs[MD_DD_MAX_BRICKS];
    uint32_t slice0[MD_DD_MAX_BRICKS];
};

struct BrickSel {
    uint32_t blk;                    // block within the brick's range
    int64_t slot0, atom0, n_end, n_xs;
    uint32_t slice0;
};

__device__ __forceinline__ BrickSel brick_select(const BrickTab *t, uint32_t b)
{
    int lo = 0, hi = t->nb;   // blk0[lo] <= b < blk0[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) / 2;
        if (t->blk0[mid] <= b) lo = mid;
        else hi = mid;
    }
    return {uint32_t(b - t->blk0[lo]), t->slot0[lo], t->atom0[lo], t->n_end[lo], t->n_xs[lo], t->slice0[lo]};
}

// Buffers of a force kernel's wavefront: the positions (n_xs < 2^28 atoms)
// and its slice's block of the list.
struct SliceBufs {
    __amdgpu_buffer_rsrc_t xs, row;
};

__device__ __forceinline__ SliceBufs slice_bufs(const void *xs, int64_t n_xs, const int32_t *idx, int32_t cap,
                                                uint32_t blk, uint32_t slice0 = 0)
{
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t slice = int64_t(slice0) + int64_t(blk) * (kBlock / kWave) + wave;
    return {make_rsrc(xs, uint32_t(n_xs) * 16u), make_rsrc(idx + slice * cap * kSlice, uint32_t(cap) * 32u)};
}

// A double from the lane that data-parallel-primitive control CTRL names
// (row and bank masks full): quad_perm 0xB1 = lane ^ 1, 0x4E = lane ^ 2,
// row_half_mirror 0x141 = 7 - lane within each group of 8, row_ror:8 0x128 =
// lane ^ 8, quad_perm 0x00, 0x55, 0xaa = lane 0, 1, 2 of the quad.
template <int CTRL>
__device__ __forceinline__ double dpp_double(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

// The sum over the 8 lanes of an atom in every one of them, the pairwise order
// ((g0 + g1) + (g2 + g3)) + ((g4 + g5) + (g6 + g7)).  All lanes of the wave must
// be active.
__device__ __forceinline__ double sum8(double g)
{
    g += dpp_double<0xb1>(g);
    g += dpp_double<0x4e>(g);
    g += dpp_double<0x141>(g);
    return g;
}

// The same of a compensated sum.
__device__ __forceinline__ double combine(float s, float c) { return sum8(double(s) - double(c)); }

// Sums of 8 doubles over a block of WAVES wavefronts, written to out[0..8) in a
// fixed order.  A wave adds its lanes by halving the values instead of by eight
// butterflies: lanes that differ in a bit of their number exchange one half of the
// values and keep the other, so three exchanges inside 8 lanes (4 + 2 + 1 doubles,
// on the vector unit) leave lane c with value c, and three more doubles finish
// it.  (Eight butterflies are 96 passes through the LDS crossbar a wave, which
// for a wave of 8 atoms is a good part of its life: force pass with MD_ENERGY of
// 500,000 Cu atoms 80.4 us, now 64.5.)
template <int WAVES>
__device__ __forceinline__ void block_sum8(const double (&v)[8], double *lds /* 8 * WAVES */, double *out)
{
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const bool h4 = lane & 4, h2 = lane & 2, h1 = lane & 1;
    double a[4], b[2];
#pragma unroll
    for (int k = 0; k < 4; ++k) a[k] = (h4 ? v[k + 4] : v[k]) + dpp_double<0x141>(h4 ? v[k] : v[k + 4]);
#pragma unroll
    for (int k = 0; k < 2; ++k) b[k] = (h2 ? a[k + 2] : a[k]) + dpp_double<0x4e>(h2 ? a[k] : a[k + 2]);
    double t = (h1 ? b[1] : b[0]) + dpp_double<0xb1>(h1 ? b[0] : b[1]);
    t += dpp_double<0x128>(t);   // row_ror:8 = lane ^ 8
    t += __shfl_xor(t, 16, kWave);
    t += __shfl_xor(t, 32, kWave);
    if (lane < 8) lds[wave * 8 + lane] = t;
    __syncthreads();
    if (threadIdx.x < 8) {
        double s = 0.0;
        for (int w = 0; w < WAVES; ++w) s += lds[w * 8 + threadIdx.x];
        out[threadIdx.x] = s;
    }
}

// A lane's FP64 sum of the virials g d_a d_b of its pairs (order xx, yy, zz, xy,
// xz, yz).  The products are FP64, which takes fewer conversions (4) and operations
// than six FP32 products converted one by one, and there is no branch: pairs not
// counted have g = 0 and a finite d.  (That form: 64.5 us where this takes 63.0,
// force pass with MD_ENERGY of 500,000 Cu atoms.)
__device__ __forceinline__ void add_virial(double (&w)[6], float g, float dx, float dy, float dz)
{
    const double x = double(dx), y = double(dy), z = double(dz);
    const double gx = double(g) * x, gy = double(g) * y, gz = double(g) * z;
    w[0] = __builtin_fma(gx, x, w[0]);
    w[1] = __builtin_fma(gy, y, w[1]);
    w[2] = __builtin_fma(gz, z, w[2]);
    w[3] = __builtin_fma(gx, y, w[3]);
    w[4] = __builtin_fma(gx, z, w[4]);
    w[5] = __builtin_fma(gy, z, w[5]);
}

// Atom and lane-in-atom of this thread: a wave holds one slice of kSlice
// atoms, lane = kSlice * a + sub.
struct SliceLane {
    int64_t i;
    int sub;
};

__device__ __forceinline__ SliceLane slice_lane(uint32_t blk, uint32_t slice0 = 0)
{
    return {int64_t(slice0) * kSlice + int64_t(blk) * (kBlock / kSlice) + threadIdx.x / kSlice,
            int(threadIdx.x % kSlice)};
}

// ---- velocity update behind the forces (Advance) ---------------------------
template <class A>
__device__ __forceinline__ bool writes_f(const A &adv)
{
    if constexpr (A::on) return adv.write_f;
    else return true;
}

// The launch's first thread posts the flag of the step whose forces these are, or
// the longest row of the build before it (before the gate: the host waits for
// either in any case).
template <class A>
__device__ __forceinline__ void post_flag(const A &adv)
{
    if constexpr (A::on) {
        if (adv.a.post.word && blockIdx.x == 0 && threadIdx.x == 0) {
            const bool stop = adv.status[0] == adv.a.post.tag;
            post_flag_word(adv.a.post.word, adv.a.post.tag, stop, stop && adv.status[1] != 0);
        }
        if (adv.longest_host && blockIdx.x == 0 && threadIdx.x == 0)
            __hip_atomic_store(adv.longest_host, *adv.longest, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// Kick and, with drift, move of the wave's 8 atoms from their forces (gx, gy, gz
// in every lane of an atom), operation by operation as k_kick_drift and k_kick do
// it: lane sub = c < 3 of an atom takes component c.  keep: the fourth word of the
// new scaled coordinates.  All lanes of the wave call it.  (The state read before
// the row walk instead: the same to 0.3 us a step slower below 50,000 atoms.)
__device__ __forceinline__ void advance_atoms(const Advance &adv, int64_t n, int64_t i, int sub, double gx, double gy,
                                              double gz, uint32_t keep)
{
    const DriftArgs &a = adv.a;
    const bool mine = i < n && sub < 3;
    const int64_t at = sub * n + i;
    double v = 0.0, x = 0.0, ref = 0.0;
    if (mine) {
        v = adv.v[at];
        if (adv.drift) {
            x = adv.x[at];
            if (adv.xref) ref = adv.xref[at];
        }
    }
    const double fc = sub == 0 ? gx : (sub == 1 ? gy : gz);
    const double vc = v + a.hk * fc;
    if (mine) adv.v[at] = vc;
    if (!adv.drift) return;
    const double p = x + a.dt * vc;
    if (mine) adv.x_out[at] = p;
    const bool bad = mine && !isfinite(p);
    const double L = sub == 0 ? a.L[0] : (sub == 1 ? a.L[1] : a.L[2]);
    const double hL = sub == 0 ? a.hL[0] : (sub == 1 ? a.hL[1] : a.hL[2]);
    double d = p - ref;
    if (d > hL)
        d -= L;
    else if (d < -hL)
        d += L;
    const double d2 = d * d;
    const double x2 = dpp_double<0x00>(d2), y2 = dpp_double<0x55>(d2), z2 = dpp_double<0xaa>(d2);
    bool moved = adv.xref && sub == 0 && i < n && ((x2 + y2) + z2) > a.half_skin_sq;
    if (adv.xs_out) {
        const double k = sub == 0 ? a.k[0] : (sub == 1 ? a.k[1] : a.k[2]);
        const uint32_t u = sub == 3 ? keep : uint32_t(uint64_t(__double2ll_rn(p * k)));
        if (i < n && sub < 4) adv.xs_out[4 * i + sub] = u;
    }
    moved |= bad || (a.post.first && i == 0 && sub == 0 && adv.status[1] != 0);
    if (__ballot(moved) && (threadIdx.x % kWave) == 0) adv.status[0] = a.tag;
    if (__ballot(bad) && (threadIdx.x % kWave) == 0) atomicOr(&adv.status[1], 1);
}

}  // namespace md
