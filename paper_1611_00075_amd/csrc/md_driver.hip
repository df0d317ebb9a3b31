// Native velocity-Verlet driver (Sec. 3.3): runs whole steps of the path
// without returning to the caller, so no interpreter sits between kernels.
//
// Per step: the force evaluation of the current positions, whose last kernel
// also applies the kick (the closing half of this step and the opening half of
// the next) and the drift to the next positions with the rebuild check.  The new
// scaled coordinates (FP64: positions) go to a second buffer, md_system_t.scratch,
// as other blocks still read the old ones; the two buffers swap each step, and the
// first drift of a run chooses its side so that the run ends in the caller's.
// Evaluations are queued two ahead of the host: that of step k + 2 does nothing if
// the flag of step k, k + 1 or k + 2 asks for a build.  Each posts its step's
// flag to pinned host memory; when some atom has moved more than half the skin the
// host rebuilds the lists, evaluates step k again and queues the next steps anew.  A
// step is one launch (two with two-pass forces) and the GPU does not wait for the
// host.  (One ahead, a step waited for the host's round trip: LJ of 4,000 atoms
// 7.9 us a step, now 6.3; FS of 2,048 10.9, now 9.5.)
//
// In large systems (kFuseAtoms), with timing (a force evaluation then has to be a
// launch of its own), with plain FP32 sums or with a scratch buffer that is not aligned to 16 bytes, a kick-drift kernel
// before each evaluation does the update in place, and posts the flag of the
// step before it; the host is then one step behind.
#include <chrono>
#include <thread>

#include "md_common.h"

namespace md {

// The flag of step `tag`, the last of a run (the earlier ones are posted by
// the kick-drift that follows).
__global__ void k_publish(const int32_t *status, uint32_t *word, int32_t tag)
{
    const bool stop = status[0] == tag;
    post_flag_word(word, tag, stop, stop && status[1] != 0);
}

// The longest row of the list just built, into host word 3 (which the host
// set negative before queueing this kernel).
__global__ void k_publish_longest(const int32_t *max_count, int32_t *host)
{
    volatile int32_t *h = host;
    h[3] = *max_count;
    __threadfence_system();
}

namespace {

constexpr int kNoAnswer = 1;   // a wait for the device given up: MD_ERR_HIP, with no other wait behind it

// Host word of a step's flag: three words in turn, as the flags of steps k + 1 and
// k + 2 can be posted before the host has read that of step k.  `host_dev` is the
// device's address of md_system_t.host_status.
inline uint32_t *flag_slot(int32_t *base, int32_t tag) { return reinterpret_cast<uint32_t *>(base) + uint32_t(tag) % 3u; }

// Clears the word before the kernel that posts `tag` is queued.
void expect_flag(md_system_t *sys, int32_t tag)
{
    *static_cast<volatile uint32_t *>(flag_slot(sys->host_status, tag)) = ~flag_word(tag, false, false);
}

// Waits for the flag of step `tag`; sets *moved (which a non-finite position
// sets too), *bad.  Without pinned memory: a copy and a stream
// synchronisation.
int read_flag(md_system_t *sys, int32_t *host_dev, int32_t tag, hipStream_t s, bool *moved, bool *bad)
{
    if (host_dev) {
        const volatile uint32_t *h = flag_slot(sys->host_status, tag);
        const uint32_t want = flag_word(tag, false, false);
        const auto t0 = std::chrono::steady_clock::now();
        uint32_t got = *h;
        for (uint64_t spin = 0; (got & ~3u) != want; ++spin, got = *h) {
            if ((spin & 4095) == 4095) {
                const hipError_t e = hipStreamQuery(s);
                if (e != hipSuccess && e != hipErrorNotReady) return kNoAnswer;
                if (std::chrono::steady_clock::now() - t0 > std::chrono::seconds(120)) return kNoAnswer;
                std::this_thread::yield();
            }
        }
        __atomic_thread_fence(__ATOMIC_ACQUIRE);
        *moved = got & 1u;
        *bad = got & 2u;
        return MD_OK;
    }
    int32_t st[2];
    MD_HIP_TRY(hipMemcpyAsync(st, sys->status, sizeof(st), hipMemcpyDeviceToHost, s));
    MD_HIP_TRY(hipStreamSynchronize(s));
    *moved = st[0] == tag;
    *bad = *moved && st[1] != 0;
    return MD_OK;
}

// Bins, sorts and builds the lists without waiting for the longest row:
// check_build reads it once the force evaluation (gated on the device by the
// same row length) is queued behind the build.
int rebuild(md_system_t *sys, const WsLayout &w, hipStream_t s)
{
    const int64_t n = sys->n;
    // state into the sorted order; xref = the sorted positions
    uint32_t *xs = (sys->flags & MD_PAIR_FP64) ? nullptr : sys->xs;
    int rc = sort_state(&sys->grid, n, sys->x, sys->cell, sys->perm, sys->cell_start, sys->ws, w, sys->v, sys->ids,
                        sys->xref, sys->scratch, sys->ids_scratch, &sys->box, xs, sys->max_count, s);
    if (rc) return rc;
    if (n > 0) {
        if (sys->potential == MD_POT_TBM) {
            // elements follow their atoms into the new order and into the scaled coordinates
            MD_HIP_TRY(hipMemcpyAsync(sys->types_scratch, sys->types, size_t(n) * 4, hipMemcpyDeviceToDevice, s));
            if ((rc = permute(n, 1, sys->perm, sys->types_scratch, sys->types, 4, s))) return rc;
            if ((rc = set_elements(n, sys->types, sys->xs, s))) return rc;
        }
    }
    return build_neighbors(&sys->grid, n, sys->x, sys->cell_start, sys->row_cap, sys->idx, sys->count, sys->max_count,
                           nullptr, sys->ws, w, s, n > 0);
}

// The host word of the longest row, before the kernel that posts it is queued.
void expect_longest(md_system_t *sys) { reinterpret_cast<volatile int32_t *>(sys->host_status)[3] = -1; }

// Posts the longest row where the evaluation behind the build does not.
int publish_longest(md_system_t *sys, hipStream_t s, int32_t *host_dev)
{
    if (!host_dev) return MD_OK;
    expect_longest(sys);
    hipLaunchKernelGGL(k_publish_longest, dim3(1), dim3(1), 0, s, sys->max_count, host_dev);
    MD_HIP_TRY(hipGetLastError());
    return MD_OK;
}

// Waits for the longest row of the last build: MD_ERR_CAPACITY (with
// row_cap_needed) when it exceeds row_cap.
int check_build(md_system_t *sys, int32_t *host_dev, hipStream_t s)
{
    int32_t longest = 0;
    if (host_dev) {
        volatile int32_t *h = sys->host_status;
        const auto t0 = std::chrono::steady_clock::now();
        for (uint64_t spin = 0; h[3] < 0; ++spin) {
            if ((spin & 4095) == 4095) {
                const hipError_t e = hipStreamQuery(s);
                if (e != hipSuccess && e != hipErrorNotReady) return kNoAnswer;
                if (std::chrono::steady_clock::now() - t0 > std::chrono::seconds(120)) return kNoAnswer;
                std::this_thread::yield();
            }
        }
        __atomic_thread_fence(__ATOMIC_ACQUIRE);
        longest = h[3];
    } else {
        MD_HIP_TRY(hipMemcpyAsync(&longest, sys->max_count, sizeof(longest), hipMemcpyDeviceToHost, s));
        MD_HIP_TRY(hipStreamSynchronize(s));
    }
    if (longest > sys->row_cap) {
        sys->row_cap_needed = longest;
        return MD_ERR_CAPACITY;
    }
    ++sys->builds;
    return MD_OK;
}

// Where a step's positions are: what the force kernels read (x in the FP64 path,
// xs in the other; the FP32 path updates x in place).
struct Positions {
    double *x;
    uint32_t *xs;
};

// The force evaluation of the positions `at`; with a gate, the kernels
// do nothing when the gate's flag is set on the device.
int forces(md_system_t *sys, const WsLayout &w, hipStream_t s, const Positions &at, Gate gate = {},
           const Advance *adv = nullptr)
{
    if (sys->potential == MD_POT_LJ)
        return forces_lj(&sys->box, sys->n, at.x, at.xs, sys->row_cap, sys->idx, sys->count, &sys->lj, sys->f,
                         nullptr, sys->flags & (MD_PAIR_FP64 | MD_NO_COMPENSATE), sys->ws, w, s, gate, adv);
    if (sys->potential == MD_POT_TBM)
        return forces_tbm(&sys->box, sys->n, at.xs, sys->row_cap, sys->idx, sys->count, &sys->tbm, sys->rho,
                          sys->fprime, static_cast<float *>(sys->f), nullptr, nullptr, sys->flags & MD_NO_COMPENSATE,
                          sys->ws, w, s, gate, adv);
    if (sys->potential == MD_POT_TAB)
        return forces_tab(&sys->box, sys->n, at.xs, sys->row_cap, sys->idx, sys->count, &sys->tab, sys->tab_table,
                          sys->rho, sys->fprime, static_cast<float *>(sys->f), nullptr, nullptr,
                          sys->flags & MD_NO_COMPENSATE, sys->ws, w, s, gate, adv);
    if (sys->potential == MD_POT_TB)
        return forces_tb(&sys->box, sys->n, at.xs, sys->row_cap, sys->idx, sys->count, &sys->tb, sys->rho,
                         sys->fprime, static_cast<float *>(sys->f), nullptr, nullptr, sys->flags & MD_NO_COMPENSATE,
                         sys->ws, w, s, gate, adv);
    if (sys->potential == MD_POT_MLP)
        return forces_mlp(&sys->box, sys->n, at.xs, sys->row_cap, sys->idx, sys->count, &sys->mlp, sys->mlp_w,
                          sys->dEdG, sys->idx_in, sys->cnt_in, nullptr, static_cast<float *>(sys->f), nullptr,
                          sys->flags & MD_NO_COMPENSATE, sys->ws, w, s, gate, adv);
    return forces_eam(&sys->box, sys->n, at.xs, sys->row_cap, sys->idx, sys->count, &sys->fs, sys->rho,
                      sys->fprime, static_cast<float *>(sys->f), nullptr, nullptr, sys->flags & MD_NO_COMPENSATE,
                      sys->ws, w, s, gate, adv);
}

// Optional timing of the force evaluations: one event pair per evaluation,
// kept in recording order and read back once the stream has passed it.  A
// speculative evaluation that the device skipped is dropped unread.
struct ForceTimer {
    static constexpr int kSlots = 4;
    bool on = false;
    hipEvent_t ev[kSlots][2] = {};
    int queue[kSlots] = {};   // recorded, unread pairs, oldest first
    int queued = 0;
    int next = 0;
    bool init(bool want)
    {
        if (!want) return true;
        for (auto &p : ev)
            for (auto &e : p)
                if (hipEventCreate(&e) != hipSuccess) return false;
        on = true;
        return true;
    }
    ~ForceTimer()
    {
        if (on)
            for (auto &p : ev)
                for (auto &e : p) (void)hipEventDestroy(e);
    }
    void start(hipStream_t s)
    {
        if (on) (void)hipEventRecord(ev[next][0], s);
    }
    void stop(md_system_t *sys, hipStream_t s)
    {
        if (!on) return;
        if (queued == kSlots) collect(sys, true, 0);   // keep a free slot
        (void)hipEventRecord(ev[next][1], s);
        queue[queued++] = next;
        next = (next + 1) % kSlots;
    }
    void drop_last()
    {
        if (on && queued > 0) --queued;
    }
    // Reads back all but the `keep` most recent pairs (waiting for them when
    // `wait`; otherwise the caller knows the stream has passed them).
    void collect(md_system_t *sys, bool wait, int keep)
    {
        if (!on) return;
        int k = 0;
        for (; k < queued - keep; ++k) {
            const int p = queue[k];
            if (wait) (void)hipEventSynchronize(ev[p][1]);
            float ms = 0.f;
            if (hipEventElapsedTime(&ms, ev[p][0], ev[p][1]) == hipSuccess) {
                sys->force_ms += ms;
                ++sys->force_calls;
            }
        }
        for (int j = k; j < queued; ++j) queue[j - k] = queue[j];
        queued -= k;
    }
};

}  // namespace

// Largest system whose force kernels apply the kick and drift.  A launch less per
// step is what small systems gain; but the update's reads and writes, 64 bytes at
// a time behind a row walk, run at half the rate of the kick-drift kernel's, and
// from about 100,000 atoms on that costs more.  us per step without builds,
// separate / fused: LJ of 4,000 atoms 13.9 / 8.6, of 42,592 14.9 / 12.6, of 70,304
// 17.4 / 16.9, of 108,000 21.5 / 21.5, of 1.26 M 156 / 182; FS of 2,048 14.3 / 10.8, of 55,296
// 19.7 / 19.2, of 108,000 29.4 / 29.4, of 500,000 79.8 / 89.0; FP64 LJ of 4,000 14.4 / 9.0.
constexpr int64_t kFuseAtoms = 65536;

static int run_steps(md_system_t *sys, int64_t steps, hipStream_t s)
{
    const WsLayout w = ws_layout(sys->grid.n_cells, sys->n);
    const int64_t n = sys->n;
    const bool f64 = sys->flags & MD_PAIR_FP64;
    const double hk = 0.5 * sys->dt * sys->accel;
    int32_t *host_dev = nullptr;
    if (sys->host_status && n > 0) {   // (with no atoms no kernel runs to post a flag)
        void *p = nullptr;
        if (hipHostGetDevicePointer(&p, sys->host_status, 0) == hipSuccess) host_dev = static_cast<int32_t *>(p);
        else (void)hipGetLastError();
    }
    int rc = MD_OK;
    bool moved = false, bad = false;
    ForceTimer timer;
    if (!timer.init(sys->timing != 0)) return MD_ERR_HIP;
    // the caller's buffers and the second one (side 0 and side 1)
    const bool fuse = n > 0 && n <= kFuseAtoms && !sys->timing && !(sys->flags & MD_NO_COMPENSATE) && sys->scratch &&
                      (f64 || (reinterpret_cast<uintptr_t>(sys->scratch) & 15u) == 0);
    const Positions side[2] = {{sys->x, f64 ? nullptr : sys->xs},
                               {f64 ? sys->scratch : sys->x,
                                f64 ? nullptr : reinterpret_cast<uint32_t *>(sys->scratch)}};
    // a step's positions back on side 0 (before a build, which reads x, and on an error)
    const auto settle = [&](int b) -> int {
        if (b == 0) return MD_OK;
        if (f64)
            MD_HIP_TRY(hipMemcpyAsync(sys->x, side[1].x, size_t(n) * 24, hipMemcpyDeviceToDevice, s));
        else
            MD_HIP_TRY(hipMemcpyAsync(sys->xs, side[1].xs, size_t(n) * 16, hipMemcpyDeviceToDevice, s));
        return MD_OK;
    };
    // forces of a fresh build, skipped on the device when a row overflowed
    const Gate fits{nullptr, 0, 0, sys->max_count, sys->row_cap};
    if (sys->phase == 0 && sys->need_build) {
        if ((rc = rebuild(sys, w, s))) return rc;
        if ((rc = publish_longest(sys, s, host_dev))) return rc;
        if ((rc = forces(sys, w, s, side[0], fits))) return rc;
        if ((rc = check_build(sys, host_dev, s))) return rc;
        sys->need_build = 0;
    }
    int64_t done = 0;
    const int64_t last = sys->step + steps;
    // What the evaluation of step k with its positions on side b does besides:
    // the closing kick of the run; kick and drift to the other side, when as many
    // drifts as are left end on side 0; else nothing, and a kick-drift in place
    // follows.
    enum { kNothing, kDrift, kClose };
    const auto besides = [&](int64_t k, int b) -> int {
        if (!fuse) return kNothing;
        if (k == last) return kClose;
        return ((last - k) & 1) == b ? kDrift : kNothing;
    };
    bool first = true;   // no drift queued in this run yet
    // Queues the evaluation of step k (positions on side b).  post: it posts the
    // flag of step k; where it cannot and no kick-drift follows, a kernel does.
    // built: behind a build, whose longest row is posted likewise.
    const auto queue_forces = [&](int64_t k, int b, Gate gate, bool post, bool built = false) -> int {
        const int what = besides(k, b);
        const int32_t tag = int32_t(k);
        Advance adv{};
        if (what != kNothing) {
            adv.a = drift_args(&sys->box, what == kClose ? hk : 2.0 * hk, sys->dt, sys->half_skin_sq, tag + 1);
            adv.drift = what == kDrift;
            if (adv.drift) {
                adv.a.post.first = first;
                first = false;
            }
            adv.write_f = what == kClose;
            adv.x = side[b].x;
            adv.x_out = side[what == kDrift ? !b : b].x;
            adv.v = sys->v;
            adv.xref = sys->xref;
            adv.status = sys->status;
            adv.xs_out = what == kDrift ? side[!b].xs : nullptr;
        }
        if (post && host_dev && (what != kNothing || k == last)) {
            expect_flag(sys, tag);
            if (what != kNothing) {
                adv.a.post.word = flag_slot(host_dev, tag);
                adv.a.post.tag = tag;
            } else {
                hipLaunchKernelGGL(k_publish, dim3(1), dim3(1), 0, s, sys->status, flag_slot(host_dev, tag), tag);
                MD_HIP_TRY(hipGetLastError());
            }
        }
        if (built && host_dev) {
            if (what != kNothing) {
                expect_longest(sys);
                adv.longest = sys->max_count;
                adv.longest_host = host_dev + 3;
            } else if (int r = publish_longest(sys, s, host_dev)) {
                return r;
            }
        }
        timer.start(s);
        if (int r = forces(sys, w, s, side[b], gate, what != kNothing ? &adv : nullptr)) return r;
        timer.stop(sys, s);
        return MD_OK;
    };
    // Queues the kick (h) and drift of step k from side b to side to, for FP32
    // from whatever scaled coordinates to those of side to.  ahead: the flag of
    // step k - 1 is not read yet; the kernel posts it and is gated by it.
    const auto queue_drift = [&](double h, int64_t k, int b, int to, bool ahead) -> int {
        const int32_t tag = int32_t(k);
        FlagPost post;
        post.driven = true;
        post.first = first;
        first = false;
        if (ahead) {
            expect_flag(sys, tag - 1);
            post.word = flag_slot(host_dev, tag - 1);
            post.tag = tag - 1;
        }
        return kick_drift(&sys->box, n, side[b].x, sys->v, sys->f, f64, h, sys->dt, sys->xref, sys->half_skin_sq,
                          sys->status, tag, side[to].xs, s, sys->potential == MD_POT_TBM, post, side[to].x);
    };
    const int64_t depth = fuse ? 2 : 1;   // steps queued behind the one in flight
    int b = 0;                    // side of the positions of the step in flight
    int64_t known = sys->step;    // flags up to this step's are read
    int64_t queued = sys->step;   // evaluations up to this step's are queued (none beyond `step`: none in flight)
    int qb = 0;                   // side of the positions of the last queued one
    // Queues the step after the last queued one: its kick and drift unless that
    // one's evaluation makes them, and its evaluation.
    const auto queue_after = [&]() -> int {
        int to = qb;
        if (besides(queued, qb) == kDrift) to = !qb;
        else if (int r = queue_drift(2.0 * hk, queued + 1, qb, qb, queued > known)) return r;
        if (int r = queue_forces(queued + 1, to, Gate{sys->status, int32_t(queued + 1), int32_t(known + 1)}, true))
            return r;
        ++queued;
        qb = to;
        return MD_OK;
    };
    for (;;) {
        const int64_t k = sys->step + 1;
        const int32_t tag = int32_t(k);
        if (sys->phase == 0) {
            if (done >= steps) break;
            b = fuse && sys->potential != MD_POT_TBM ? int((last - k) & 1) : 0;   // (elements stay in the caller's xs)
            if ((rc = queue_drift(hk, k, 0, b, false))) return rc;
            sys->phase = 1;
            if ((rc = queue_forces(k, b, Gate{sys->status, tag, tag}, true))) return rc;
            queued = k;
            qb = b;
        }
        // a step is in flight: positions drifted, forces stale unless queued
        bool ready = false;
        if (queued >= k) {
            // (a kick-drift kernel is gated by the flag of the step before it alone)
            while (host_dev && queued < last && queued - k < depth && (queued == k || besides(queued, qb) == kDrift))
                if ((rc = queue_after())) return rc;
            if ((rc = read_flag(sys, host_dev, tag, s, &moved, &bad))) return rc;
            if (bad) {
                if ((rc = settle(b))) return rc;
                return MD_ERR_NONFINITE;
            }
            ready = !moved;
            if (!ready)   // the device skipped this step's forces and the steps queued ahead
                for (; queued >= k; --queued) timer.drop_last();
            // the flag was posted behind every evaluation but the newest one
            timer.collect(sys, false, ready ? 1 : 0);
            sys->need_build |= moved ? 1 : 0;
        }
        const bool built = sys->need_build != 0;
        if (built) {
            ready = false;
            if (f64 && (rc = settle(b))) return rc;
            b = 0;
            if ((rc = rebuild(sys, w, s))) return rc;
        }
        if (!ready) {
            if ((rc = queue_forces(k, b, built ? fits : Gate{}, false, built))) return rc;
            queued = k;
            qb = b;
        }
        if (built) {
            if ((rc = check_build(sys, host_dev, s))) {
                timer.drop_last();
                return rc;
            }
            sys->need_build = 0;
        }
        known = k;
        ++sys->step;
        ++done;
        const int what = besides(k, b);
        if (done < steps) {
            if (queued == k && (rc = queue_after())) return rc;
            if (what == kDrift) b = !b;
        } else {
            if (what != kClose &&
                (rc = integrate(MD_KICK, &sys->box, n, sys->x, sys->v, sys->f, sys->dt, sys->accel, 1.0, nullptr, 0.0,
                                nullptr, 0, nullptr, nullptr, sys->flags & MD_PAIR_FP64, sys->ws, w, s)))
                return rc;
            sys->phase = 0;
        }
    }
    timer.collect(sys, true, 0);
    return MD_OK;
}

// The evaluations queued ahead post their steps' flags to host_status whatever
// became of the step in flight, so a run that ends early waits for them: once it
// has returned nothing writes to the caller's words.  (MD_ERR_CAPACITY needs no
// wait: the longest row was posted behind all of them.)
int run(md_system_t *sys, int64_t steps, hipStream_t s)
{
    const int rc = run_steps(sys, steps, s);
    if (rc == kNoAnswer) return MD_ERR_HIP;
    if (rc != MD_OK && rc != MD_ERR_CAPACITY) (void)hipStreamSynchronize(s);
    return rc;
}

}  // namespace md
