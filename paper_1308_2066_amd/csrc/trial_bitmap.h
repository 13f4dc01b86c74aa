// Device code of the YLT path with an occurrence filter in LDS and the values in HBM/L2,
// for catalogs whose dense table does not fit in LDS (internal; used by the plain trial
// kernel and the batched kernel).
//
// Computes, per trial (Section II-B, steps 1-4),
//   ylt = min(max(P - AggR, 0), AggL),  P = sum over the trial's occurrences of the
//   occurrence-net loss of their event,
// which equals the basic algorithm's sum of per-occurrence ceded losses: the
// cumulative sum is non-decreasing and the aggregate clamp is non-decreasing with
// value 0 at 0, so the differences telescope.
//
// The filter has 2^20 bits (128 KB).  In a larger catalog an event passes when any event
// whose ID agrees with its own in the low 20 bits is in the layer: it is folded; the value
// of an event that should not have passed is zero.  Values come from the catalog's table
// (zero outside the layer).  That table is larger than the layer's values on their own, but
// these need ranks in LDS, 25 instructions for each queued row and two more launches per
// change of the layer: 200,000 trials of 250 events in an 800,000-event catalog took 95 us
// and 12 us for the ranks, now 97; 2000 trials of 300 54 us with everything, now 41.
// Catalogs past 2^20 events were read without a filter, bound by fetching a line of the
// table for each event (8 10^10 a second): 1.5 10^6 events, 200,000 trials of 250 717 -> 97
// us, of 700 1580 -> 213.
//
// A wave walks its trials in segments of 1024 events (four non-temporal loads per
// lane: 16 bytes of int32 IDs, or 12 bytes of the YET's packed 3-byte copy, which
// cuts the dominant stream by a quarter).  Per segment:
//   filter  each lane tests the LDS bit of its events, up to 16 (one LDS read each, all
//           issued together): events whose occurrence-net loss is nonzero pass, and in a
//           folded filter those that share a bit with one;
//   queue   passing events are appended to the wave's LDS queue in slot-then-lane
//           order (mbcnt positions), so they end up dense;
//   rows    the queue is resolved 64 events at a time, their values from the table;
//   sum     values are added per lane in queue order, then reduced over the wave
//           at the trial's end (deterministic for a given YET layout).
// Software pipeline: the ID loads of segment i+2 are issued after the value reads of
// segment i, and the values of segment i are added one segment later.  Vector-memory
// operations complete in issue order, so waiting for values never waits for the
// newest ID loads: each ID load has two segments of time to arrive.
#pragma once

#include "trial_common.h"

namespace ara {

constexpr int kRows = kQueueCapMax / kQueueRow;                  // value reads per segment
constexpr int kFoldWords = 1 << (kFoldBits - 5);                 // static LDS for the filter
static_assert((kFoldWords + kQueueWords) * 4 <= kLdsMaxBytes, "filter and queues");

// Copies the layer's filter into LDS, folded to 2^20 bits (whole workgroup; ends with a
// barrier).
__device__ __forceinline__ void stage_fold(const TrialArgs &a, uint32_t *tab) {
    const u32x4 *g4 = reinterpret_cast<const u32x4 *>(a.bitmap);
    for (int i = threadIdx.x; i < kFoldWords / 4; i += blockDim.x) {
        u32x4 w = i < a.nblk ? g4[i] : u32x4{0u, 0u, 0u, 0u};
        for (int k = i + kFoldWords / 4; k < a.nblk; k += kFoldWords / 4) w |= g4[k];
        reinterpret_cast<u32x4 *>(tab)[i] = w;
    }
    __syncthreads();
}

// Wave-uniform position: trial t (relative to t_begin; t >= n when done), segment
// start sbase (multiple of 4), trial end o1, and lo = leading events before the
// trial's first event in its first segment (0..3).
struct BCur {
    uint32_t t;
    uint32_t lo;
    int64_t sbase;
    int64_t o1;
};

__device__ __forceinline__ BCur bcur_open(const TrialArgs &a, uint32_t t, uint32_t n, uint32_t &bad) {
    BCur c;
    c.t = t;
    c.lo = 0;
    c.sbase = 0;
    c.o1 = 0;
    if (t < n) {
        const int64_t r0 = uniform64(offset_at(a.offs, a.t_begin + t));
        const int64_t r1 = uniform64(offset_at(a.offs, a.t_begin + t + 1));
        const bool ok = r0 >= 0 && r0 <= r1 && r1 <= a.n_events;   // else: an empty trial, reported
        bad |= ok ? 0u : uint32_t(ERR_OFFSETS);
        const int64_t o0 = ok ? r0 : 0, o1 = ok ? r1 : 0;
        c.sbase = o0 & ~int64_t(3);
        c.lo = uint32_t(o0 - c.sbase);
        c.o1 = o1;
    }
    return c;
}

__device__ __forceinline__ bool bcur_last(const BCur &c) { return c.sbase + kSeg >= c.o1; }

// Loop-carried cursors are wave-uniform; this keeps them in scalar registers.
__device__ __forceinline__ BCur bcur_uniform(const BCur &c) {
    BCur u;
    u.t = __builtin_amdgcn_readfirstlane(c.t);
    u.lo = __builtin_amdgcn_readfirstlane(c.lo);
    u.sbase = uniform64(c.sbase);
    u.o1 = uniform64(c.o1);
    return u;
}

__device__ __forceinline__ BCur bcur_next(const TrialArgs &a, const BCur &c, uint32_t stride, uint32_t n,
                                          uint32_t &bad) {
    if (c.t >= n) return c;
    if (!bcur_last(c)) {
        BCur d = c;
        d.sbase += kSeg;
        d.lo = 0;
        return d;
    }
    return bcur_open(a, c.t + stride, n, bad);
}

// Event IDs of one segment in registers: int32 (four 16-byte loads per lane) or the
// packed copy (four 12-byte loads per lane).
template <bool P24> struct IdRegs;
template <> struct IdRegs<false> { u32x4 r[kNch]; };
template <> struct IdRegs<true> { u32x3 r[kNch]; };

template <bool P24>
__device__ __forceinline__ void bcur_load(const TrialArgs &a, const BCur &c, uint32_t n, int lane, IdRegs<P24> &g) {
    const bool live = c.t < n;
    if constexpr (P24)
        load_ids24(a.ids24, live ? c.sbase : 0, live ? seg_avail24(c.sbase, c.o1) : 0, lane, g.r);
    else
        load_ids(a.ids, live ? c.sbase : 0, live ? seg_avail(c.sbase, c.o1, a.n_events) : 0, lane, g.r);
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t vals_rsrc(const TrialArgs &a) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)a.occ, 0, int(uint32_t(a.catalog) * 8u), kBufWord3);
}

__device__ __forceinline__ double load_val(__amdgpu_buffer_rsrc_t vr, uint32_t byte_off) {
    const uint2 q = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(vr, byte_off, 0, 0));
    return __builtin_bit_cast(double, q);
}

// MAX: each trial's largest value instead of the sum (values are >= +0.0).
template <bool MAX>
__device__ __forceinline__ double join(double x, double y) { return MAX ? (y > x ? y : x) : x + y; }

template <bool MAX>
__device__ __forceinline__ double wave_join(double x) {
    if (!MAX) return wave_total(x);
    x = join<true>(x, dpp_f64<0xB1>(x));    // the steps of wave_total
    x = join<true>(x, dpp_f64<0x4E>(x));
    x = join<true>(x, dpp_f64<0x141>(x));
    x = join<true>(x, dpp_f64<0x140>(x));
    return join<true>(join<true>(readlane_f64(x, 0), readlane_f64(x, 16)),
                      join<true>(readlane_f64(x, 32), readlane_f64(x, 48)));
}

// Resolve queue entries [0, qn) now (queue overflow: many flagged events).
template <bool MAX>
__device__ __forceinline__ void drain_queue(const TrialArgs &a, const uint32_t *q, uint32_t qn, int lane, double &acc) {
    const __amdgpu_buffer_rsrc_t vr = vals_rsrc(a);
    for (uint32_t r0 = 0; r0 < qn; r0 += kQueueRow) {
        double v = 0.0;
        if (r0 + lane < qn) v = load_val(vr, q[r0 + lane] * 8u);
        acc = join<MAX>(acc, v);
    }
}

// Filter + queue of one segment held in r; returns the queue length.  Slot s of a
// lane holds the event at position k*256 + 4*lane + j (s = 4k + j) of the segment;
// it counts if that position lies in [lo, hi) and the event's filter bit is set.
// lo < 4, so only lane 0 of the first load can hold events before the trial.
// The int32 IDs are range-checked here (mx); the packed copy was checked when built.
// NC: the 256-event chunks looked at (hi <= 256 NC).
template <bool P24, bool MAX, int NC>
__device__ __forceinline__ uint32_t seg_queue(const TrialArgs &a, const uint32_t *tab, uint32_t *q,
                                              const IdRegs<P24> &g, int lane, int lo, int hi, uint32_t &mx,
                                              double &dacc) {
    const uint32_t cmax = uint32_t(a.catalog) - 1u;
    constexpr int kS = 4 * NC;
    uint32_t id[kS], e[kS], w[kS];
#pragma unroll
    for (int k = 0; k < NC; ++k) {
        if constexpr (P24) {
            unpack_ids24(g.r[k], id + 4 * k);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) id[4 * k + j] = g.r[k][j];
            mx = max(mx, max(max(id[4 * k], id[4 * k + 1]), max(id[4 * k + 2], id[4 * k + 3])));
        }
    }
#pragma unroll
    for (int s = 0; s < kS; ++s) {
        // the packed copy was checked against the catalog when it was built
        e[s] = P24 ? id[s] : min(id[s], cmax);
        w[s] = tab[(e[s] >> 5) & uint32_t(kFoldWords - 1)];
    }
    const int l4 = lane * 4;
    bool f[kS];
    uint32_t total = 0;
#pragma unroll
    for (int s = 0; s < kS; ++s) {
        const int base = (s >> 2) * kChunk + (s & 3);
        f[s] = (__builtin_amdgcn_ubfe(w[s], e[s], 1) != 0u) & (l4 < hi - base);
        if (s < 4) f[s] = f[s] & (l4 + base >= lo);
        total += uint32_t(__popcll(__builtin_amdgcn_ballot_w64(f[s])));
    }
    uint32_t qn = 0;
    if (total <= uint32_t(a.qcap)) {
        // common case: the whole segment fits the queue
#pragma unroll
        for (int s = 0; s < kS; ++s) {
            const uint64_t m = __builtin_amdgcn_ballot_w64(f[s]);
            uint32_t *qs = q + qn;
            if (f[s]) qs[__builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0u))] = e[s];
            qn += uint32_t(__popcll(m));
        }
        return qn;
    }
    // many flagged events: resolve the queue whenever the next slot would overflow it
#pragma unroll
    for (int s = 0; s < kS; ++s) {
        const uint64_t m = __builtin_amdgcn_ballot_w64(f[s]);
        const uint32_t cnt = uint32_t(__popcll(m));
        if (qn + cnt > uint32_t(a.qcap)) {
            drain_queue<MAX>(a, q, qn, lane, dacc);
            qn = 0;
        }
        if (f[s]) q[__builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), qn))] = e[s];
        qn += cnt;
    }
    return qn;
}

// Value reads of the queued events: always kRows 64-lane reads (lanes past the queue
// read outside the buffer record: 0, no memory access), so the number of
// outstanding vector-memory operations per segment is fixed.
__device__ __forceinline__ void seg_rows(const TrialArgs &a, const uint32_t *q, uint32_t qn, int lane,
                                         double (&v)[kRows]) {
    const __amdgpu_buffer_rsrc_t vr = vals_rsrc(a);
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
        const uint32_t r0 = uint32_t(k) * kQueueRow;
        uint32_t off = 0xFFFFFFF8u;
        if (r0 < qn) {
            const uint32_t slot = r0 + uint32_t(lane);
            off = slot < qn ? q[slot] * 8u : 0xFFFFFFF8u;
        }
        v[k] = load_val(vr, off);
    }
}

struct Pending {
    uint32_t t;      // trial of the segment whose values are in flight (>= n: none)
    uint32_t last;   // that segment ends its trial
    double dacc;     // its values already resolved on the overflow path
};

template <bool P24, bool MAX>
__device__ __forceinline__ void issue(const TrialArgs &a, const uint32_t *tab, uint32_t *q, IdRegs<P24> &r,
                                      const BCur &cur, const BCur &nxt, uint32_t n, int lane, uint32_t &mx,
                                      double (&v)[kRows], Pending &p) {
    const int64_t h = cur.o1 - cur.sbase;
    const int hi = int(h > kSeg ? kSeg : h);
    p.t = cur.t;
    p.last = bcur_last(cur) ? 1u : 0u;
    p.dacc = 0.0;
    // Chunks past the trial's end are not looked at (wave-uniform).  The kernel is bound by
    // its instructions (vector units 62% busy; with all four chunks of every segment
    // looked at 265 of them per trial of 250 events, now 160): 200,000 trials of 250 events
    // 145 -> 95 us, of 450 154 -> 126, of 50 142 -> 84.  (A wave's trials next to each other,
    // their offsets in its lanes, instead of a grid apart: 102.)
    const int lo = int(cur.lo);
    const uint32_t qn = hi <= kChunk       ? seg_queue<P24, MAX, 1>(a, tab, q, r, lane, lo, hi, mx, p.dacc)
                        : hi <= 2 * kChunk ? seg_queue<P24, MAX, 2>(a, tab, q, r, lane, lo, hi, mx, p.dacc)
                                           : seg_queue<P24, MAX, kNch>(a, tab, q, r, lane, lo, hi, mx, p.dacc);
    seg_rows(a, q, qn, lane, v);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    bcur_load<P24>(a, nxt, n, lane, r);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

template <bool MAX>
__device__ __forceinline__ void retire(const TrialArgs &a, const Pending &p, const double (&v)[kRows], uint32_t n,
                                       int lane, double &acc) {
    if (p.t >= n) return;
    double s = p.dacc;
#pragma unroll
    for (int k = 0; k < kRows; ++k) s = join<MAX>(s, v[k]);
    acc = join<MAX>(acc, s);
    if (p.last) {
        const double P = wave_join<MAX>(acc);
        if (lane == 0) a.ylt[p.t] = MAX ? P : excess(P, a.agg_r, a.agg_l);
        acc = 0.0;
    }
}

// The waves of a workgroup walk trials first, first + stride, ... of [0, t_end -
// t_begin) (relative to a.t_begin) with the filter already in tab; q is this wave's
// queue of a.qcap entries.
template <bool P24, bool MAX>
__device__ __forceinline__ void bitmap_wave_run(const TrialArgs &a, const uint32_t *tab, uint32_t *q, uint32_t first,
                                                uint32_t stride, int lane) {
    const uint32_t n = uint32_t(a.t_end - a.t_begin);
    uint32_t bad = 0, mx = 0;

    BCur c0 = bcur_uniform(bcur_open(a, first, n, bad));
    BCur c1 = bcur_uniform(bcur_next(a, c0, stride, n, bad));
    // The prologue issues what a loop iteration leaves in flight (IDs, value reads of
    // an empty segment, IDs), so the waits at the loop's top are the same on entry.
    IdRegs<P24> A, B;
    double vA[kRows], vB[kRows];
    bcur_load<P24>(a, c0, n, lane, A);
    seg_rows(a, q, 0u, lane, vB);
    bcur_load<P24>(a, c1, n, lane, B);

    Pending pA, pB;
    pB.t = n;
    pB.last = 0;
    pB.dacc = 0.0;
    double acc = 0.0;
    // One exit, at the top: a segment past the last trial is issued as an empty one
    // (no IDs, no queued events) rather than leaving the loop in the middle, so the
    // compiler's wait counts at the top do not assume an empty pipeline.
    while (c0.t < n) {
        pB.t = __builtin_amdgcn_readfirstlane(pB.t);
        pB.last = __builtin_amdgcn_readfirstlane(pB.last);
        const BCur c2 = bcur_uniform(bcur_next(a, c1, stride, n, bad));
        issue<P24, MAX>(a, tab, q, A, c0, c2, n, lane, mx, vA, pA);
        retire<MAX>(a, pB, vB, n, lane, acc);
        const BCur c3 = bcur_uniform(bcur_next(a, c2, stride, n, bad));
        issue<P24, MAX>(a, tab, q, B, c1, c3, n, lane, mx, vB, pB);
        retire<MAX>(a, pA, vA, n, lane, acc);
        c0 = c2;
        c1 = c3;
    }
    retire<MAX>(a, pB, vB, n, lane, acc);
    if (mx > uint32_t(a.catalog) - 1u) bad |= ERR_ID_RANGE;
    if (bad) atomicOr(a.err, bad);
}

}  // namespace ara
