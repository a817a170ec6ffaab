// flow.hpp -- the flow engine: one persistent launch runs every observation
// interval of a batch of filters.
//
// The per-interval engine advances all filters together: a launch per
// interval, so every filter waits at each observation time for the slowest
// wavefront of that interval, and the compute units idle through each
// launch's tail.  Here a filter advances as soon as its own particles are
// weighed.  Wavefronts take work items -- pools of particles of one filter
// over one interval, exactly those of the per-interval engine -- from a
// ring in arrival order, one item each.  The wavefront
// that finishes a filter's last item of an interval weighs that filter
// (log-weights, log-sum-exp, systematic resampling; the same arithmetic in
// the same order as k_weigh, so results are bit-identical) and writes the
// items of its next interval to the ring.  Wavefronts left without an item
// leave once every filter is done.
//
// Ring protocol (bounded multi-producer multi-consumer queues with one
// sequence word per slot): a producer reserves position p from a ring's
// tail counter, waits until slot p & mask holds sequence p (free for p) and
// writes (p + 1, entry); a consumer takes p from the head counter, waits
// until the slot holds p + 1, takes the entry and marks the slot free for
// position p + capacity.  Every wavefront claims its item with one
// fetch-and-add, so thousands of waiting wavefronts never contend on a
// compare-and-swap.
//
// Priority without a second claim path: first come, first served would let
// a filter wait at every interval behind a whole generation of other
// filters' items, and the filters with the longest chains (many intervals
// left times long items) would set the end of the run.  So the item ring is
// kept short: a filter that is not urgent and finds `backlog` items already
// waiting is parked (its id goes to a second ring) instead of appending its
// items; every wavefront that finishes an interval takes parked filters and
// appends their items while fewer than `backlog` wait.  Urgent filters always
// append, and so wait only behind a short ring.  No deadlock: a filter is
// parked only while items wait, and the last of them to finish un-parks.
// At most one interval of items per filter is outstanding: its groups of 64,
// and split items beyond them counted in kCtlExtra, so at most
// sum(groups of 64) + split_waves <= capacity entries sit in a ring and a
// producer never waits for a slot that no wavefront has claimed.
//
// Hand-offs between wavefronts (item results before the weighing, the
// weighing's state before the next items): everything a later wavefront reads
// is stored at agent scope, through the L2 cache of the storing XCD; the giver
// waits for its stores (stores_done) and then makes the hand-off known with an
// atomic operation; the taker acquires at agent scope.  No store of this
// kernel stays dirty in an L2 while another XCD may write or read its address
// (the weights' scratch included), so every store of it has to go through
// store_global or an agent-scope atomic.  Releasing plain stores instead wrote the
// XCD's whole L2 back, three times per item: 326 -> 322 ms for 1024 telegraph
// rate vectors in FP64, 213 -> 166 ms for 512 in FP32-mixed without.
#pragma once
#ifndef __HIPCC_RTC__
#include <hip/hip_runtime.h>
#include <stdint.h>
#endif

#include "propagate.hpp"
#include "weigh.hpp"

namespace lik {

__device__ __forceinline__ uint32_t ctl_load(const FlowArgs &fa, int w) {
    return __hip_atomic_load(&fa.ctl[w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Progress of the launch that a waiting wavefront polls: items of finished
// intervals and items claimed (a wavefront that finishes its item leaves, and
// the next one claims).
__device__ __forceinline__ uint32_t flow_progress(const FlowArgs &fa) {
    return ctl_load(fa, kCtlProgress) + ctl_load(fa, kCtlHead + 64 * kRingItems);
}

// What a wait has seen of the progress, and when.
struct StallWatch {
    uint32_t seen = 0;
    uint64_t since = 0;
    bool counted = false;  // `left` was taken at `since`
    uint64_t left = 0;     // items not finished, over every filter's interval
};

__device__ __forceinline__ void watch_start(const FlowArgs &fa, StallWatch &w) {
    w.since = wall_clock64();
    w.seen = flow_progress(fa);
}

// Gives up (sets the abort word, which every waiting wavefront then sees) once
// no item has finished for stall_ticks.  Where every wavefront left already
// holds its item, no claim shows that items of a long interval finish one after
// another: after stall_ticks without polled progress the filters' items left
// are counted, and only a second count, stall_ticks later, with the same result
// ends the flow (so it comes between one and two limits after the last item).
__device__ __forceinline__ bool flow_stalled(const FlowArgs &fa, StallWatch &w) {
    if (ctl_load(fa, kCtlAbort) != 0u) return true;
    const uint32_t prog = flow_progress(fa);
    const uint64_t now = wall_clock64();
    if (prog != w.seen) {
        w.seen = prog;
        w.since = now;
        w.counted = false;
    } else if (now - w.since > fa.stall_ticks) {
        uint64_t left = 0;
#pragma unroll 4
        for (int f = 0; f < fa.n_slots; ++f)
            left += __hip_atomic_load(&fa.remaining[f], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (w.counted && left == w.left) {
            __hip_atomic_store(&fa.ctl[kCtlAbort], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return true;
        }
        w.left = left;
        w.counted = true;
        w.since = now;
    }
    return false;
}

__device__ __forceinline__ uint64_t *ring_slot(const FlowArgs &fa, int r, uint32_t pos) {
    return fa.ring + (size_t)r * (fa.mask + 1) + (pos & fa.mask);
}

// Waits until slot `pos` of ring r holds sequence `want` (its entry in
// *entry); false if the flow has given up, or (when `until_done`) once
// every filter is done.
__device__ __forceinline__ bool ring_wait(const FlowArgs &fa, int r, uint32_t pos, uint32_t want,
                                          uint64_t *entry, bool until_done) {
    StallWatch watch;
    for (bool first = true;; first = false) {
        const uint64_t v =
            __hip_atomic_load(ring_slot(fa, r, pos), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((uint32_t)(v >> 32) == want) {
            *entry = v;
            return true;
        }
        if (first) watch_start(fa, watch);
        if (until_done && (int)ctl_load(fa, kCtlFinished) >= fa.n_slots) return false;
        if (flow_stalled(fa, watch)) return false;
        __builtin_amdgcn_s_sleep(8);
    }
}

// Reserves n positions of ring r and writes entry first + k step at the k-th of
// them (a lane waits until its slot is free for the position).  The caller has
// released what the entries' readers need.
__device__ __forceinline__ void ring_put(const FlowArgs &fa, int r, int n, uint32_t first,
                                         uint32_t step, int lane) {
    uint32_t base = 0;
    if (lane == 0)
        base = __hip_atomic_fetch_add(&fa.ctl[kCtlTail + 64 * r], (uint32_t)n, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
    base = __builtin_amdgcn_readfirstlane(base);  // lane 0's: every lane is active
    for (int k = lane; k < n; k += 64) {
        const uint32_t pos = base + (uint32_t)k;
        uint64_t ent;
        if (ring_wait(fa, r, pos, pos, &ent, false))
            __hip_atomic_store(ring_slot(fa, r, pos),
                               ((uint64_t)(pos + 1u) << 32) | (first + (uint32_t)k * step),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Takes the slot's entry of position pos and frees the slot for its next lap.
__device__ __forceinline__ void ring_take(const FlowArgs &fa, int r, uint32_t pos) {
    __hip_atomic_store(ring_slot(fa, r, pos), (uint64_t)(pos + fa.mask + 1u) << 32,
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A filter is urgent (its items never wait in the parked ring) when its
// intervals left times the expected events per lane of its items (events
// per particle times the G particles a lane takes) reach urgent_events.
__device__ __forceinline__ bool flow_urgent(const EngineArgs &e, const FlowArgs &fa, int f,
                                            uint32_t cost, int G) {
    if (fa.urgent_events == 0u) return true;  // no parking: first come, first served
    const FilterDesc &d = e.desc[f];
    const uint64_t per_lane = (uint64_t)(cost / (uint32_t)d.H) * (uint64_t)G;
    const uint64_t left = (uint64_t)(d.T - e.tcur[f]);
    return per_lane * left >= (uint64_t)fa.urgent_events;
}

// Items waiting in the item ring; negative when wavefronts wait for items
// (they take positions ahead of the tail).
__device__ __forceinline__ int32_t item_backlog(const FlowArgs &fa) {
    return (int32_t)(ctl_load(fa, kCtlTail + 64 * kRingItems) -
                     ctl_load(fa, kCtlHead + 64 * kRingItems));
}

// Writes the work items of filter f (item code `code`, state already released)
// to the item ring.
__device__ __forceinline__ void emit_items(const EngineArgs &e, const FlowArgs &fa, int f,
                                           int code, int lane) {
    ring_put(fa, kRingItems, code_items(code, e.desc[f].H), (uint32_t)f << e.item_shift,
             (uint32_t)code_step(code), lane);
}

// A filter's part of what is left of the batch: the expected events of one of
// its particles (c: of its whole next interval) times its intervals left, from
// interval t on -- the length of its chain.
__device__ __forceinline__ uint64_t flow_weight(const FilterDesc &d, uint32_t c, int t) {
    return min((uint64_t)(c / (uint32_t)d.H) * (uint64_t)(d.T - t), (uint64_t)1 << 30);
}
// Adds to one of the two sums over the unfinished filters; returns the sum.
__device__ __forceinline__ uint64_t add_weight(const FlowArgs &fa, int word, uint64_t by) {
    return by + __hip_atomic_fetch_add(reinterpret_cast<uint64_t *>(&fa.ctl[word]), by,
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A filter is critical when its chain of events alone takes about as long as
// everything left, spread over the GPU's wavefronts (waves: one per SIMD):
// the launch then ends with it, whatever the others do.
__device__ __forceinline__ bool flow_critical(const FlowArgs &fa, uint64_t w, uint64_t work) {
    return (uint64_t)fa.split_waves * w >= work;
}
__device__ __forceinline__ uint32_t ctl_add(const FlowArgs &fa, int w, uint32_t by) {
    return __hip_atomic_fetch_add(&fa.ctl[w], by, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Items the next interval of a filter of weight w should be cut into: its
// share, by weight, of split_waves, as far as the items running now leave
// room (none while items wait).  A batch that keeps the GPU busy is not split:
// an item of 32 particles issues 1.3 times the instructions of its half of 64.
// A critical filter is, into items of 16, from the start on: 512 uneven requests
// 218 -> 208 ms, 256 Lac-Gfp rate vectors 598 -> 569 ms (means of three seeds).
__device__ __forceinline__ int flow_goal(const FlowArgs &fa, uint64_t w, uint64_t sum,
                                         int nchunk, bool critical) {
    const int least = critical ? 4 * nchunk : 0;
    const uint32_t head = ctl_load(fa, kCtlHead + 64 * kRingItems);
    const uint32_t tail = ctl_load(fa, kCtlTail + 64 * kRingItems);
    const uint32_t done = ctl_load(fa, kCtlProgress);
    if ((int32_t)(tail - head) > 0 || sum == 0) return least;
    const int room = (int)fa.split_waves - (int)(tail - done);
    if (room <= 0) return least;
    return max(least, min((int)((double)fa.split_waves * ((double)w / (double)sum)), nchunk + room));
}

// The launch has one wavefront per group of 64 particles of every interval
// and fa.spare more; kCtlSpare counts those that no item needs.  A filter
// whose interval takes fewer items than groups gives the rest; one that is
// split takes the difference, or is not split when too few are left (an item
// always finds a wavefront) or when the split items outstanding would exceed
// split_waves (a ring slot is always free).  One lane only.
__device__ __forceinline__ int settle_spare(const FlowArgs &fa, int code, int H, int nchunk) {
    const int need = code_items(code, H) - nchunk;
    if (need < 0) ctl_add(fa, kCtlSpare, (uint32_t)-need);
    if (need <= 0) return code;
    if ((int)ctl_add(fa, kCtlExtra, (uint32_t)need) + need <= (int)fa.split_waves) {
        if ((int)ctl_add(fa, kCtlSpare, (uint32_t)-need) >= need) return code;
        ctl_add(fa, kCtlSpare, (uint32_t)need);
    }
    ctl_add(fa, kCtlExtra, (uint32_t)-need);
    return 0;
}

// A filter's interval (item code `code`, expected events c, interval t) is
// over: its items (counted here once, not one by one: every finished item
// adding to one word held 512 telegraph rate vectors in FP32-mixed to 12,500
// items per ms), its share of the split ones and of the weights.  One lane only.
__device__ __forceinline__ uint64_t leave_interval(const FlowArgs &fa, const FilterDesc &d,
                                                   int code, uint32_t c, int t) {
    const int n_items = code_items(code, d.H), extra = n_items - (d.Hp >> 6);
    if (extra > 0) ctl_add(fa, kCtlExtra, (uint32_t)-extra);
    ctl_add(fa, kCtlProgress, (uint32_t)n_items);
    return flow_weight(d, c, t);
}

// While the item ring is short and filters are parked, takes one parked
// filter and writes its items; false if it took none.  Called by every
// wavefront that finishes an interval, and by the wavefront first in line for
// the next item while it waits, so that parked filters move as soon as
// there is room.
__device__ __forceinline__ bool flow_unpark(const EngineArgs &e, const FlowArgs &fa, int lane) {
    int f = -1;
    if (lane == 0 && item_backlog(fa) < (int32_t)fa.backlog) {
        uint32_t h = ctl_load(fa, kCtlHead + 64 * kRingParked);
        const uint32_t tl = ctl_load(fa, kCtlTail + 64 * kRingParked);
        if ((int32_t)(tl - h) > 0 &&
            __hip_atomic_compare_exchange_strong(&fa.ctl[kCtlHead + 64 * kRingParked], &h, h + 1u,
                                                 __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT)) {
            uint64_t ent;
            if (ring_wait(fa, kRingParked, h, h + 1u, &ent, false)) {
                ring_take(fa, kRingParked, h);
                f = (int)(uint32_t)ent;
            }
        }
    }
    f = __builtin_amdgcn_readfirstlane(f);
    if (f < 0) return false;
    // acquire the parked filter's state (its items' takers acquire it themselves)
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    emit_items(e, fa, f, (int)e.pool[f] & 63, lane);
    return true;
}

// After an interval: takes parked filters (at most kUnparkPerItem) while the
// item ring is short.
constexpr int kUnparkPerItem = 4;
__device__ __forceinline__ void flow_unpark_some(const EngineArgs &e, const FlowArgs &fa,
                                                 int lane) {
    for (int k = 0; k < kUnparkPerItem; ++k)
        if (!flow_unpark(e, fa, lane)) break;
}

// Waits (lane 0) for the item of position pos of the item ring: 1 with the
// entry in *entry; 2 when this wavefront is first in line (no producer has
// reserved pos yet) and filters are parked -- the caller un-parks one and
// waits again; 0 once every filter is done or the flow has given up.
// Thousands of wavefronts may wait here while a few work, and the control
// words they would read are the ones every hand-off goes through: a waiting
// wavefront reads its own ring slot, and the control words every eighth time;
// one far from its turn sleeps longer and reads one of them.
__device__ __forceinline__ int item_wait(const FlowArgs &fa, uint32_t pos, uint64_t *entry) {
    constexpr uint32_t kFar = 256;  // positions beyond the last item written
    StallWatch watch;
    bool far = false;
    for (uint32_t n = 0;; ++n) {
        const uint64_t v = __hip_atomic_load(ring_slot(fa, kRingItems, pos), __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
        if ((uint32_t)(v >> 32) == pos + 1u) {
            *entry = v;
            return 1;
        }
        if (n == 0) watch_start(fa, watch);
        if ((n & 7u) == 0u || far) {
            if ((int)ctl_load(fa, kCtlFinished) >= fa.n_slots) return 0;
        }
        if ((n & 7u) == 0u) {
            const uint32_t tail = ctl_load(fa, kCtlTail + 64 * kRingItems);
            if (tail == pos && (int32_t)(ctl_load(fa, kCtlTail + 64 * kRingParked) -
                                         ctl_load(fa, kCtlHead + 64 * kRingParked)) > 0)
                return 2;
            if (flow_stalled(fa, watch)) return 0;
            far = (int32_t)(pos - tail) > (int32_t)kFar;
        }
        if (far)
            __builtin_amdgcn_s_sleep(100);
        else
            __builtin_amdgcn_s_sleep(32);
    }
}

// Number of resampling points j*Q + rho (j = 0, 1, ...) below x, at most H:
// ceil((x - rho) / Q) for x > rho.  The quotient (at most H) is estimated in
// binary64 (inv_Q: the nearest to 1 / Q) and then made exact with integer
// products (x < 2^57, Q < 2^45).
__device__ __forceinline__ uint32_t points_below(uint64_t x, uint64_t rho, uint64_t Q,
                                                 double inv_Q, uint32_t H) {
    if (x <= rho) return 0;
    const uint64_t y = x - rho - 1;  // n = floor(y / Q) + 1
    uint32_t m = (uint32_t)((double)y * inv_Q);
    while (m > 0 && m * Q > y) --m;
    while ((m + 1) * Q <= y) ++m;
    return min(m + 1, H);
}

// Weighing of filter f after its interval tcur[f], by one wavefront, with
// k_weigh's results bit for bit.  Per-particle steps (log-weights, e_j, q_j)
// run over particles lane-strided, so every lane's loads are independent.
// The one order-dependent sum, S = sum e_j, follows k_weigh's order: each
// lane adds its particles j = lane + 64 k in increasing k, then one
// butterfly over the lanes.  The slot's lw array holds l_j, then e_j.
// Resampling is taken from the particles' side: with
// J(x) = #{j >= 0 : j Q + rho < x}, particle i is the ancestor of exactly
// the j in [J(H C_i), J(H C_{i+1})) -- the same a_j = min{i : H C_{i+1} >
// j Q + rho} as the search over j, found without dependent loads.  Every
// particle with offspring marks its first output in LDS (`lds`, the item's
// buffer), and a running maximum over the outputs fills the rest, so a
// filter whose weight sits on one particle takes no longer than another.
//
// On a filter's chain of intervals nothing hides this step: it is bound by
// the latency of its loads (the counts come from other wavefronts through the
// last-level cache), so each pass takes kB groups of 64 particles at a time,
// their loads issued together, and scans run on DPP adds, not through LDS.
// A near-eventless interval of one filter (hand-offs included) went from 75 to
// 48 us at 1000 particles and from 250 to 125 us at 4096.
// Returns true when the filter goes on to another interval; *cost receives
// its expected events.
__device__ __forceinline__ bool flow_weigh(const EngineArgs &e, int f, double *logy,
                                           uint32_t *lds, uint32_t *cost) {
    const FilterDesc &d = e.desc[f];
    const int lane = lane_id();
    const int t = e.tcur[f];
    const int H = d.H;
    const int status = e.fstatus[f];
    auto stop_filter = [&](double ll) {
        store_global(e.tcur, (uint32_t)f, t + 1);
        store_global(e.fll, (uint32_t)f, ll);
        store_global(e.fflags, (uint32_t)f, e.fflags[f] | kFlagStopped);
    };
    {
        uint64_t evs = 0;
        constexpr int kE = 16;
        for (int base = lane; base < H; base += 64 * kE) {
            uint32_t v[kE];
#pragma unroll
            for (int k = 0; k < kE; ++k) v[k] = base + 64 * k < H ? d.pev[base + 64 * k] : 0u;
#pragma unroll
            for (int k = 0; k < kE; ++k) evs += v[k];
        }
        evs = wave_sum_u64(evs, lane);
        if (lane == 0) store_global(e.fevents, (uint32_t)f, e.fevents[f] + evs);
    }
    if (status != LIK_STATUS_OK) {
        if (lane == 0) stop_filter(__builtin_nan(""));
        return false;
    }
    const int32_t *xs = (t & 1) ? d.xa : d.xb;  // counts at the observation time
    const double *yt = d.y + (size_t)t * d.P;
    if (lane < d.P) logy[lane] = d.obs_kind == LIK_OBS_LOGNORMAL ? dlog(yt[lane]) : 0.0;
    __syncthreads();
    double *w = d.lw;
    const ObsParams op = obs_params(d);

    // kB particles per lane at a time, their loads issued together.
    constexpr int kB = 4;
    // log-weights and their maximum
    double mx = -__builtin_inf();
    if (op.kind == LIK_OBS_FLUORESCENCE) {
        // one particle at a time: its count-dependent variance makes the term
        // longer, and groups would raise the kernel's register count
        for (int j = lane; j < H; j += 64) {
            const double l = obs_logweight(d, op, xs, j, logy, yt);
            store_global(w, (uint32_t)j, l);
            mx = fmax(mx, l);
        }
    } else {
        for (int base = lane; base < H; base += 64 * kB) {
            double l[kB];
            bool on[kB];
#pragma unroll
            for (int k = 0; k < kB; ++k) {
                l[k] = 0.0;
                on[k] = base + 64 * k < H;
            }
            for (int o = 0; o < d.P; ++o) {
                const int32_t *xo = xs + (size_t)d.obs_species[o] * d.Hp;
                int cnt[kB];
#pragma unroll
                for (int k = 0; k < kB; ++k) cnt[k] = base + 64 * k < H ? xo[base + 64 * k] : 0;
#pragma unroll
                for (int k = 0; k < kB; ++k)
                    if (on[k]) on[k] = obs_term<false>(op, o, cnt[k], logy, yt, l[k]);
            }
#pragma unroll
            for (int k = 0; k < kB; ++k)
                if (base + 64 * k < H) {
                    store_global(w, (uint32_t)(base + 64 * k), l[k]);
                    mx = fmax(mx, l[k]);
                }
        }
    }
    mx = wave_max(mx, lane);
    if (mx == -__builtin_inf()) {
        if (lane == 0) stop_filter(-__builtin_inf());
        return false;
    }
    // e_j = exp(l_j - mx) in place, S = sum e_j in k_weigh's order (each
    // lane's particles in increasing j, then one butterfly), and the total Q of
    // q_j = floor(e_j 2^32); the next batch is loaded before this one's stores
    double s = 0.0;
    uint64_t Q = 0;
    double v[kB];
#pragma unroll
    for (int k = 0; k < kB; ++k) v[k] = lane + 64 * k < H ? w[lane + 64 * k] : 0.0;
    for (int base = lane; base < H; base += 64 * kB) {
        double nx[kB];
#pragma unroll
        for (int k = 0; k < kB; ++k) {
            const int jn = base + 64 * (kB + k);
            nx[k] = jn < H ? w[jn] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < kB; ++k)
            if (base + 64 * k < H) {
                const double ej = dexp_nonpos(v[k] - mx);
                store_global(w, (uint32_t)(base + 64 * k), ej);
                s += ej;
                Q += (uint64_t)(ej * 4294967296.0);
            }
#pragma unroll
        for (int k = 0; k < kB; ++k) v[k] = nx[k];
    }
    const double S = wave_sum(s, lane);
    if (lane == 0) {
        store_global(e.fll, (uint32_t)f, e.fll[f] + loglik_increment(d, mx, S, yt));
        store_global(e.tcur, (uint32_t)f, t + 1);
    }
    if (t + 1 >= d.T) return false;

    Q = wave_sum_u64(Q, lane);
    const double inv_Q = 1.0 / (double)Q;
    const uint64_t rho = __umul64hi(resample_word(d, t), Q);
    const uint64_t Hu = (uint64_t)H;
    // kG groups of 64 particles at a time: prefix sums C_{i+1} (carried over
    // groups) and outputs [J(H C_i), J(H C_{i+1})), the first of them marked
    // (index + 1, 16 bits) in the window of outputs [w0, w1) that LDS holds;
    // a full window is filled and written, and the next one begun
    constexpr int kG = 4;
    constexpr int kWin = 2 * kPoolLdsWords;  // 3072 outputs
    uint16_t *mark = reinterpret_cast<uint16_t *>(lds);
    float pred = 0.0f;     // sum of the ancestors' total propensities
    uint64_t carry = 0;    // C at the batch's first particle
    uint32_t carry_j = 0;  // J(H C) there
    uint32_t last = 0;     // mark carried into the window
    int w0 = 0, w1 = min(H, kWin);
    auto clear = [&]() {
        for (int q = lane; q < (w1 - w0 + 1) / 2; q += 64) lds[q] = 0u;
        __syncthreads();  // the workgroup is this one wavefront
    };
    clear();
    static_assert(kG == kB, "v holds a batch");
    float a0[kG];
#pragma unroll
    for (int k = 0; k < kG; ++k) {
        const int i = 64 * k + lane;
        v[k] = i < H ? w[i] : 0.0;
        a0[k] = i < H ? d.pa0[i] : 0.0f;
    }
    for (int b0 = 0; b0 < H; b0 += 64 * kG) {
        // the next batch's weights, loaded before this one's stores
        double nv[kG];
        float na[kG];
#pragma unroll
        for (int k = 0; k < kG; ++k) {
            const int i = b0 + 64 * (kG + k) + lane;
            nv[k] = i < H ? w[i] : 0.0;
            na[k] = i < H ? d.pa0[i] : 0.0f;
        }
        uint64_t incl[kG];
#pragma unroll
        for (int k = 0; k < kG; ++k)
            incl[k] = wave_incl_scan_u64((uint64_t)(v[k] * 4294967296.0));
        uint32_t j_lo[kG], j_hi[kG];
#pragma unroll
        for (int k = 0; k < kG; ++k) {
            incl[k] += carry;  // C_{i+1}
            carry = lane_last(incl[k]);
        }
#pragma unroll
        for (int k = 0; k < kG; ++k) {
            // J(H C_{i+1}); J(H C_i) is the previous particle's
            j_hi[k] = b0 + 64 * k + lane < H
                          ? points_below(Hu * incl[k], rho, Q, inv_Q, (uint32_t)H)
                          : (uint32_t)H;
            j_lo[k] = lane_prev(j_hi[k], carry_j);
            carry_j = lane_last(j_hi[k]);
            if (b0 + 64 * k + lane < H) pred += (float)(j_hi[k] - j_lo[k]) * a0[k];
        }
        for (;;) {
#pragma unroll
            for (int k = 0; k < kG; ++k)
                if (j_lo[k] < j_hi[k] && (int)j_lo[k] >= w0 && (int)j_lo[k] < w1)
                    mark[j_lo[k] - (uint32_t)w0] = (uint16_t)(b0 + 64 * k + lane + 1);
            if ((int)carry_j < w1) break;
            // every mark below w1 is set: fill the window
            __syncthreads();
            for (int q0 = 0; q0 < w1 - w0; q0 += 64 * kG) {
                uint32_t m[kG];
#pragma unroll
                for (int k = 0; k < kG; ++k) {
                    const int q = q0 + 64 * k + lane;
                    m[k] = wave_incl_max_u32(q < w1 - w0 ? mark[q] : 0u);
                }
#pragma unroll
                for (int k = 0; k < kG; ++k) {
                    const int q = q0 + 64 * k + lane;
                    m[k] = max(m[k], last);
                    last = lane_last(m[k]);
                    if (q < w1 - w0) store_global(d.anc, (uint32_t)(w0 + q), (int32_t)m[k] - 1);
                }
            }
            __syncthreads();
            if (w1 >= H) {
                w1 = 1 << 30;  // every output is written: the particles left have none
                break;
            }
            w0 = w1;
            w1 = min(H, w0 + kWin);
            clear();
        }
#pragma unroll
        for (int k = 0; k < kG; ++k) {
            v[k] = nv[k];
            a0[k] = na[k];
        }
    }
    pred = wave_sum_f32(pred, lane);
    *cost = cost_estimate(d, t, (double)pred);
    return true;
}

// Sets up filter f's next interval and writes its items to the item ring,
// or parks the filter when the ring already holds `backlog` items and the
// filter is not urgent.
__device__ __forceinline__ void flow_push(const EngineArgs &e, const FlowArgs &fa, int f,
                                          uint32_t cost) {
    const int lane = lane_id();
    __syncthreads();  // the weighing's state (tcur, ancestors) from every lane
    // lane 0 wrote tcur: its reading decides, for every lane
    const int H = e.desc[f].H;
    int code = 0, prio = 0, critical = 0;
    if (lane == 0) {
        const FilterDesc &d = e.desc[f];
        const int t = e.tcur[f], nchunk = d.Hp >> 6;
        const uint64_t was = leave_interval(fa, d, e.pool[f] & 63, e.cost[f], t - 1);
        const uint64_t w = flow_weight(d, cost, t);
        const uint64_t sum = add_weight(fa, kCtlWeight, w - was);
        const uint64_t work = add_weight(fa, kCtlWork, (w - was) * (uint64_t)nchunk);
        critical = flow_critical(fa, w, work);
        code = settle_spare(
            fa, item_code(e, f, cost, fa.g_par, flow_goal(fa, w, sum, nchunk, critical != 0)), H,
            nchunk);
        // wavefront priority for the longest chains left (2 and 4 times the
        // average; tuning.priority is the per-interval schedule's): 256 Lac-Gfp
        // rate vectors 635 -> 565 ms (means of three seeds)
        const double chain = (double)w * (double)(fa.n_slots - (int)ctl_load(fa, kCtlFinished));
        prio = critical || chain >= 4.0 * (double)sum ? 3 : chain >= 2.0 * (double)sum ? 1 : 0;
    }
    code = __builtin_amdgcn_readfirstlane(code);
    const int n_items = code_items(code, H);
    const int park = __builtin_amdgcn_readfirstlane(
        (int)(!critical && !flow_urgent(e, fa, f, cost, code < kSplitCode ? code + 1 : 1) &&
              item_backlog(fa) >= (int32_t)fa.backlog));
    if (lane == 0) {
        store_global(e.cost, (uint32_t)f, cost);
        store_global(e.pool, (uint32_t)f, (uint8_t)((prio << 6) | code));
        __hip_atomic_store(&fa.remaining[f], (uint32_t)n_items, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    // everything above (agent-scope stores) before the items or the parked
    // entry are visible
    stores_done();
    __syncthreads();
    if (park)
        ring_put(fa, kRingParked, 1, (uint32_t)f, 0u, lane);
    else
        emit_items(e, fa, f, code, lane);
}

// One work item per wavefront (a grid of at least as many wavefronts as the
// batch has work items, settle_spare; the hardware starts each as a slot frees): claim the
// next ring position, run its item, and if it was its filter's last of the
// interval, weigh the filter and write its next items.  A wavefront whose
// position is never filled leaves when every filter is done.  One item per
// wavefront, rather than a loop over items, keeps the event loop's register
// allocation that of the per-interval kernel.
// The kernel's first argument, its EngineArgs, read from the kernel-argument
// segment (constant memory: scalar loads) behind an empty asm statement, so
// the compiler issues new loads at the uses instead of keeping the values
// loaded at the kernel's start.  Every kernel that calls flow_run takes its
// EngineArgs by value as its first argument (offset 0 of the segment).
__device__ __forceinline__ const EngineArgs &reload_engine_args() {
    auto p = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const EngineArgs *)p;
}

// run(item) runs one work item (the propagation of its pool); a launch over
// several networks picks the item's network inside it.
// lds: the item's buffer, at least kPoolLdsWords words (the weighing uses it
// after the item).
template <class RunItem>
__device__ __forceinline__ void flow_run_with(const EngineArgs &e, const FlowArgs &fa,
                                              uint32_t *lds, RunItem &&run) {
    __shared__ double logy[LIK_MAX_OBSERVED];
    // the wavefronts beyond the batch's last item start after it is done (a
    // cached reading: one that is out of date waits for an item and finds out)
    if ((int)__builtin_amdgcn_readfirstlane(
            __hip_atomic_load(&fa.ctl[kCtlFinished], __ATOMIC_RELAXED,
                              __HIP_MEMORY_SCOPE_WORKGROUP)) >= fa.n_slots)
        return;
    uint64_t ent = 0;
    uint32_t pos = 0;
    if (lane_id() == 0)
        pos = __hip_atomic_fetch_add(&fa.ctl[kCtlHead + 64 * kRingItems], 1u, __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
    int ok = 0;
    for (;;) {
        int st = 0;
        if (lane_id() == 0) st = item_wait(fa, pos, &ent);
        st = __builtin_amdgcn_readfirstlane(st);  // lane 0's: every lane is active
        if (st != 2) {
            ok = st;
            break;
        }
        flow_unpark(e, fa, lane_id());
    }
    if (ok && lane_id() == 0) ring_take(fa, kRingItems, pos);
    if (!ok) return;  // every filter is done (or the flow gave up)
    // acquire: the filter's state written before the item was published
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    const uint32_t item = __builtin_amdgcn_readfirstlane((uint32_t)ent);
    const int f = (int)(item >> e.item_shift);
    run(item);

    // this item's results (agent-scope stores) before the filter's count goes
    // down
    stores_done();
    __syncthreads();
    // From here on the engine's arguments are read again from the kernel's
    // argument segment, where used (the fields loaded at the kernel's start
    // would otherwise stay in scalar registers through the event loop).
    const EngineArgs &ec = reload_engine_args();
    uint32_t left = 0;
    if (lane_id() == 0)
        left = __hip_atomic_fetch_sub(&fa.remaining[f], 1u, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
    left = __builtin_amdgcn_readfirstlane(left);
    if (left != 1u) return;
    // the last item of the interval: weigh the filter with every item's results
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    uint32_t cost = 0;
    if (flow_weigh(ec, f, logy, lds, &cost)) {
        flow_push(ec, fa, f, cost);
        flow_unpark_some(ec, fa, lane_id());
    } else {
        if (lane_id() == 0) {
            const uint64_t was = leave_interval(fa, ec.desc[f], ec.pool[f] & 63, ec.cost[f],
                                                ec.tcur[f] - 1);
            add_weight(fa, kCtlWeight, 0 - was);
            add_weight(fa, kCtlWork, 0 - was * (uint64_t)(ec.desc[f].Hp >> 6));
            if (ec.fdone) store_global(ec.fdone, (uint32_t)f, (uint64_t)wall_clock64());
            __hip_atomic_fetch_add(&fa.ctl[kCtlFinished], 1u, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        }
        flow_unpark_some(ec, fa, lane_id());
    }
}

template <class NetT, int UMAX, int RMAX, int W, int PREC>
__device__ __forceinline__ void flow_run(const EngineArgs &e, const FlowArgs &fa,
                                         const NetT &net) {
    __shared__ __attribute__((aligned(16))) uint32_t lds[item_lds_words<UMAX, RMAX, PREC>()];
    flow_run_with(e, fa, lds,
                  [&](uint32_t item) { run_item<NetT, UMAX, RMAX, W, PREC>(e, net, item, lds); });
}

}  // namespace lik
