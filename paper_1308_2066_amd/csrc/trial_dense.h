// Device code of the YLT path for a dense occurrence-net table (in LDS, or in HBM/L2
// for catalogs too large for LDS), shared by the plain trial kernels and the
// batched kernel (internal).
#pragma once

#include <type_traits>

#include "trial_common.h"

namespace ara {

// Wave-uniform position in a wave's sequence of (trial, segment).
struct Cursor {
    int64_t t;       // trial; >= t_end when the wave is done
    int64_t o0, o1;  // trial's events [o0, o1)
    int64_t sbase;   // first event of the segment, a multiple of 4
};

__device__ __forceinline__ void open_trial(const TrialArgs &a, int64_t t, Cursor &c, uint32_t &bad) {
    c.t = t;
    c.o0 = c.o1 = c.sbase = 0;
    if (t < a.t_end) {
        int64_t o0 = offset_at(a.offs, t), o1 = offset_at(a.offs, t + 1);
        if (!(o0 >= 0 && o0 <= o1 && o1 <= a.n_events)) {
            bad |= ERR_OFFSETS;
            o0 = o1 = 0;
        }
        c.o0 = o0;
        c.o1 = o1;
        c.sbase = o0 & ~int64_t(3);
    }
}

__device__ __forceinline__ bool seg_last(const Cursor &c) { return c.sbase + kSeg >= c.o1; }

// Re-asserts that a cursor is wave-uniform (keeps it in scalar registers across
// loop back-edges that the compiler cannot prove uniform).
__device__ __forceinline__ Cursor uniform_cursor(const Cursor &c) {
    Cursor u;
    u.t = uniform64(c.t);
    u.o0 = uniform64(c.o0);
    u.o1 = uniform64(c.o1);
    u.sbase = uniform64(c.sbase);
    return u;
}

__device__ __forceinline__ Cursor seg_next(const TrialArgs &a, const Cursor &c, int64_t stride, uint32_t &bad) {
    Cursor n = c;
    if (c.t >= a.t_end) return n;
    if (!seg_last(c)) {
        n.sbase = c.sbase + kSeg;
        return n;
    }
    open_trial(a, c.t + stride, n, bad);
    return n;
}

__device__ __forceinline__ void load_seg(const TrialArgs &a, const Cursor &c, int lane, u32x4 (&r)[kNch]) {
    const bool live = c.t < a.t_end;
    load_ids(a.ids, live ? c.sbase : 0, live ? seg_avail(c.sbase, c.o1, a.n_events) : 0, lane, r);
}

// Stage the layer's table into LDS (whole workgroup; ends with a barrier).
template <int PL>
__device__ __forceinline__ void stage_lds(const TrialArgs &a, uint32_t *lds, bool zero = false) {
    if (PL == ARA_PLACE_LDS_BITMAP) {
        stage_bitmap(a, lds);
        return;
    } else if (PL == ARA_PLACE_LDS_DENSE) {
        // occurrence-net table, catalog doubles = 2*catalog words; eight loads of a thread in
        // flight (one at a time, the 20 loads of a 256-thread workgroup for a 10,000-event
        // catalog took most of the 20 us of a small launch)
        const uint32_t *g = reinterpret_cast<const uint32_t *>(a.occ);
        const int n = 2 * a.catalog, n4 = n >> 2, bd = int(blockDim.x);
        u32x4 *l4 = reinterpret_cast<u32x4 *>(lds);
        const u32x4 *g4 = reinterpret_cast<const u32x4 *>(g);
        for (int i0 = threadIdx.x; i0 < n4; i0 += 8 * bd) {
            u32x4 v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = g4[min(i0 + k * bd, n4 - 1)];
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (i0 + k * bd < n4) l4[i0 + k * bd] = v[k];
        }
        for (int i = (n4 << 2) + threadIdx.x; i < n; i += blockDim.x) lds[i] = g[i];
        if (zero) {   // an entry of +0.0 after the table, and the row masks (see row_add)
            uint32_t *m = lds + lane_masks_at(a.catalog) / 4;
            if (threadIdx.x < 2) lds[n + threadIdx.x] = 0u;
            if (threadIdx.x < kRowMaskBytes / 4) {
                const int r = int(threadIdx.x >> 2), j = 2 * int(threadIdx.x & 3);   // IDs j, j + 1 of a piece that holds r
                m[threadIdx.x] = (j < r ? 0u : 0xFFFFu) | (j + 1 < r ? 0u : 0xFFFF0000u);
            }
        }
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------------
// Look up the 16 IDs a lane holds for one segment: v[s] = occurrence-net loss of
// the event in slot s, 0 for slots outside the trial.  For the bitmap placement the
// L2 reads are issued here and consumed later (after the next prefetch is issued).
template <int PL>
__device__ __forceinline__ void seg_lookup(const TrialArgs &a, const uint32_t *lds, const u32x4 (&r)[kNch],
                                           int lane, int lo, int hi, double (&v)[kSlots], uint32_t &bad) {
    const uint32_t C = uint32_t(a.catalog);
    if (PL == ARA_PLACE_LDS_BITMAP) {
        // handled by seg_bitmap_filter / seg_bitmap_rows
    } else if (PL == ARA_PLACE_LDS_DENSE) {
        const double *tab = reinterpret_cast<const double *>(lds);
#pragma unroll
        for (int s = 0; s < kSlots; ++s) {
            const int rel = (s >> 2) * kChunk + lane * 4 + (s & 3);
            const uint32_t id = r[s >> 2][s & 3];
            const bool valid = rel >= lo && rel < hi;
            const bool inr = id < C;
            if (valid && !inr) bad |= ERR_ID_RANGE;
            v[s] = 0.0;
            if (valid && inr) v[s] = tab[id];
        }
    } else {
        const __amdgpu_buffer_rsrc_t vr =
            __builtin_amdgcn_make_buffer_rsrc((void *)a.occ, 0, int(C < 0x1FFFFFFFu ? C * 8u : 0xFFFFFFF8u), kBufWord3);
#pragma unroll
        for (int s = 0; s < kSlots; ++s) {
            const int rel = (s >> 2) * kChunk + lane * 4 + (s & 3);
            const uint32_t id = r[s >> 2][s & 3];
            const bool valid = rel >= lo && rel < hi;
            const bool inr = id < C;
            if (valid && !inr) bad |= ERR_ID_RANGE;
            // always issued (slots outside the trial read past the record: 0, no
            // memory access), so the count of loads in flight is the same on every path
            const uint32_t off = valid && inr ? id * 8u : 0xFFFFFFF8u;
            const uint2 q = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(vr, off, 0, 0));
            v[s] = __builtin_bit_cast(double, q);
        }
    }
}

__device__ __forceinline__ void seg_bounds(const Cursor &c, int &lo, int &hi) {
    const int64_t l = c.o0 - c.sbase, h = c.o1 - c.sbase;
    lo = int(l < 0 ? 0 : l);
    hi = int(h > kSeg ? kSeg : h);
}

__device__ __forceinline__ void finish_trial(const TrialArgs &a, int64_t t, double acc, int lane) {
    const double P = wave_total(acc);
    if (lane == 0) a.ylt[t - a.t_begin] = excess(P, a.agg_r, a.agg_l);
}

// One segment: look up its events (the L2 reads of the global placement are left
// in flight in v), then issue the loads of segment `nxt` into the register buffer
// just consumed, then add the values.
template <int PL>
__device__ __forceinline__ void seg_step(const TrialArgs &a, uint32_t *lds, uint32_t *q, u32x4 (&r)[kNch],
                                         const Cursor &cur, const Cursor &nxt, int lane, uint32_t &bad, double &acc) {
    int lo, hi;
    seg_bounds(cur, lo, hi);
    {
        double v[kSlots];
        seg_lookup<PL>(a, lds, r, lane, lo, hi, v, bad);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        load_seg(a, nxt, lane, r);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < kSlots; ++s) acc += v[s];
    }
}

// Wave per trial: the waves of a workgroup walk trials first, first + stride, ...
// (absolute trial indices, < a.t_end), two segments in flight per wave.
template <int PL>
__device__ __forceinline__ void dense_wave_run(const TrialArgs &a, uint32_t *lds, int64_t first, int64_t stride,
                                               int lane) {
    uint32_t *q = nullptr;   // no queue outside the bitmap placement
    uint32_t bad = 0;

    Cursor c0, c1;
    open_trial(a, first, c0, bad);
    c0 = uniform_cursor(c0);
    u32x4 A[kNch], B[kNch];
    load_seg(a, c0, lane, A);
    c1 = uniform_cursor(seg_next(a, c0, stride, bad));
    load_seg(a, c1, lane, B);

    double acc = 0.0;
    // One exit, at the top: a segment past the wave's last trial is stepped as an
    // empty one (no events) rather than leaving the loop in the middle, so the
    // compiler's wait counts at the top do not assume an empty pipeline.
    while (c0.t < a.t_end) {
        // segment c0 (in A) while c1 (in B) is in flight; A then receives c2
        const Cursor c2 = uniform_cursor(seg_next(a, c1, stride, bad));
        seg_step<PL>(a, lds, q, A, c0, c2, lane, bad, acc);
        if (seg_last(c0)) {
            finish_trial(a, c0.t, acc, lane);
            acc = 0.0;
        }
        const Cursor c3 = uniform_cursor(seg_next(a, c2, stride, bad));
        seg_step<PL>(a, lds, q, B, c1, c3, lane, bad, acc);
        if (c1.t < a.t_end && seg_last(c1)) {
            finish_trial(a, c1.t, acc, lane);
            acc = 0.0;
        }
        c0 = c2;
        c1 = c3;
    }
    if (bad) atomicOr(a.err, bad);
}

// Lane per trial, for short trials: lane i of the workgroup's wave w takes trial
// first + i, first + i + stride, ... and adds its occurrences' values in time order
// (the same sequence of additions as a sequential loop over the trial, so P is
// exactly the oracle's cumulative total).  The occurrence-net values come from the dense
// table.
//   A lane reads its trial 16 IDs (64 bytes) at a time from the trial's first ID, two such
// chunks ahead, through a buffer record that starts at the wave's first trial and ends
// with the YET (a 16-byte load gives 0 for its words past the end).
//   What bounds it: VALU instructions per ID.  With 64-bit position tests for each ID,
// about 20 a lookup, and each chunk's loads waited for before the next one's were issued,
// 8.3x10^8 occurrences took 1.58 ms; here the lanes of a chunk that lies inside every
// lane's trial test nothing.
constexpr int kLaneIds = 16;

__device__ __forceinline__ void lane_load(__amdgpu_buffer_rsrc_t r, uint32_t at, bool live, u32x4 (&q)[4]) {
    const uint32_t off = live ? at * 4u : 0xFFFFFF00u;   // outside any record: no memory access
#pragma unroll
    for (int u = 0; u < 4; ++u) q[u] = __builtin_amdgcn_raw_buffer_load_b128(r, int(off + 16u * u), 0, 0);
}

// Values of the first `left` IDs of q (all 16 when ALL); the others' are +0.0.
template <int PL, bool ALL>
__device__ __forceinline__ void lane_lookup(const double *tab, __amdgpu_buffer_rsrc_t vr, uint32_t C, const u32x4 (&q)[4],
                                            int32_t left, double (&v)[kLaneIds], uint32_t &mx) {
#pragma unroll
    for (int j = 0; j < kLaneIds; ++j) {
        const bool in = ALL || j < left;
        const uint32_t id = in ? q[j >> 2][j & 3] : 0u;
        mx = max(mx, id);
        if constexpr (PL == ARA_PLACE_LDS_DENSE) {
            const double x = tab[min(id, C - 1u)];
            v[j] = in ? x : 0.0;   // adding +0.0 leaves P's bits unchanged
        } else {
            const uint32_t off = in ? id * 8u : 0xFFFFFFF8u;   // past the record: 0
            v[j] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(vr, int(off), 0, 0));
        }
    }
}

template <int PL>
__device__ __forceinline__ void lane_step(const double *tab, __amdgpu_buffer_rsrc_t vr, uint32_t C,
                                          __amdgpu_buffer_rsrc_t rs, u32x4 (&q)[4], uint32_t at, int32_t left, double &P,
                                          uint32_t &mx) {
    double v[kLaneIds];
    if (PL == ARA_PLACE_LDS_DENSE && __builtin_amdgcn_ballot_w64(left < kLaneIds) == 0)
        lane_lookup<PL, true>(tab, vr, C, q, left, v, mx);
    else
        lane_lookup<PL, false>(tab, vr, C, q, left, v, mx);
    lane_load(rs, at + 2 * kLaneIds, left > 2 * kLaneIds, q);   // the chunk after the next
#pragma unroll
    for (int j = 0; j < kLaneIds; ++j) P += v[j];
}

template <int PL>
__device__ __forceinline__ void dense_lane_run(const TrialArgs &a, const uint32_t *lds, int64_t first, int64_t stride) {
    const uint32_t C = uint32_t(a.catalog);
    const double *tab = reinterpret_cast<const double *>(lds);
    const __amdgpu_buffer_rsrc_t vr = __builtin_amdgcn_make_buffer_rsrc((void *)a.occ, 0, int(C * 8u), kBufWord3);
    uint32_t bad = 0, mx = 0;
    // the wave's trials are consecutive; lanes past the last trial go along with none
    for (int64_t t = first; __builtin_amdgcn_ballot_w64(t < a.t_end) != 0; t += stride) {
        const bool live = t < a.t_end;
        int64_t o0 = 0, o1 = 0;
        if (live) o0 = a.offs[t], o1 = a.offs[t + 1];
        const bool ok = o0 >= 0 && o0 <= o1 && o1 <= a.n_events;
        if (!ok) {
            bad |= ERR_OFFSETS;
            o0 = o1 = 0;
        }
        const int64_t base = uniform64(o0);
        constexpr int64_t kSpan = int64_t(1) << 28;
        double P = 0.0;
        if (__builtin_amdgcn_ballot_w64(o1 > o0 && (o0 < base || o1 - base > kSpan)) != 0) {
            // trials too long for one record (or bad offsets among them): one ID at a time
            for (int64_t p = o0; p < o1; ++p) {
                const uint32_t id = uint32_t(a.ids[p]);
                mx = max(mx, id);
                P += PL == ARA_PLACE_LDS_DENSE ? tab[min(id, C - 1u)] : a.occ[min(id, C - 1u)];
            }
        } else {
            const int64_t n = min(a.n_events - base, kSpan);
            const __amdgpu_buffer_rsrc_t rs =
                __builtin_amdgcn_make_buffer_rsrc((void *)(a.ids + base), 0, int(uint32_t(n) * 4u), kBufWord3);
            uint32_t at = o1 > o0 ? uint32_t(o0 - base) : 0u;
            int32_t left = int32_t(o1 - o0);
            u32x4 A[4], B[4];
            lane_load(rs, at, left > 0, A);
            lane_load(rs, at + kLaneIds, left > kLaneIds, B);
            while (__builtin_amdgcn_ballot_w64(left > 0) != 0) {
                lane_step<PL>(tab, vr, C, rs, A, at, left, P, mx);
                at += kLaneIds;
                left -= kLaneIds;
                lane_step<PL>(tab, vr, C, rs, B, at, left, P, mx);
                at += kLaneIds;
                left -= kLaneIds;
            }
        }
        if (live) a.ylt[t - a.t_begin] = excess(P, a.agg_r, a.agg_l);
    }
    if (mx >= C) bad |= ERR_ID_RANGE;
    if (bad) atomicOr(a.err, bad);
}

// The same with the IDs staged through LDS, for tables that leave a wave 4 KB
// (lane_staged_fits).  A lane that reads its own trial touches lines no other lane of the
// load does, and the vector-memory path takes about two clocks for each of those (2.65x10^11
// lane requests a second over the chip: 0.9 ms of the 1.19 ms that 8.3x10^8 occurrences took
// above).  Here eight lanes read 32 consecutive IDs of one trial, so a load instruction
// covers eight 128-byte (packed: 96-byte) stretches instead of 64 lines; the IDs go to LDS as
// 16-bit numbers, a row of 64 bytes per trial, and each lane reads its own row.
//   Window w of a wave's 64 trials: IDs [32 w, 32 w + 32) of each, counted from the trial's
// first group of four.  Window w + 1, or the first of the wave's next 64 trials, is loaded
// while window w is added.
//   IDs of the catalog size or more are clamped to it and read the zero entry after the
// table; so do the positions outside the trial.  The packed copy was checked when it was
// built, so its IDs take no test or clamp, and two bytes of each go to LDS as they are.
//   What it measured: 7.2x10^8 occurrences of 13 requests in a batch 715 us; with the masks,
// the packed IDs as they are, and no address kept over the loop that two instructions form
// (ten of them were spilled, and a reload goes the way of the loads) 657; 64 jobs over
// 10,000 trials 49 -> 39.  2.4 GB of IDs come from HBM (390 us at 6.1 TB/s); the LDS is busy
// 40% of the time, the path that returns loads 70%.
constexpr int kRowBytes = 64;   // 32 IDs of one trial
static_assert(64 * kRowBytes == kStageBytes, "a row per lane");
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pk_min(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ uint32_t pk_max(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}

// Adds the 8 IDs of a row's piece q in order: all of them, or those before the r-th (TAIL,
// any r) and from the lead-th on (FIRST: the trial's first piece, lead < 4).  The others
// become 0xFFFF, which the clamp turns into the zero entry's: by a row of masks in LDS for
// each r (two comparisons and selections for each ID took twice the instructions).
// CHECKED: the IDs are known to be in the catalog.
template <bool FIRST, bool TAIL, bool CHECKED>
__device__ __forceinline__ void row_add(const char *tab, const char *masks, const u32x4 &q, int32_t lead, int32_t r,
                                        uint32_t c2, double &P, uint32_t &mx) {
    u32x4 w = q, out{0u, 0u, 0u, 0u};   // out: what is not to be added
    if (TAIL) out = *reinterpret_cast<const u32x4 *>(masks + 16 * max(0, min(r, 8)));
    if (FIRST) {
        out[0] |= lead >= 2 ? ~0u : lead == 1 ? 0xFFFFu : 0u;
        out[1] |= lead == 3 ? 0xFFFFu : 0u;
    }
    double v[8];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        if (!CHECKED) mx = pk_max(mx, FIRST || TAIL ? w[d] & ~out[d] : w[d]);
        if (FIRST || TAIL) w[d] |= out[d];
        if (FIRST || TAIL || !CHECKED) w[d] = pk_min(w[d], c2);
        v[2 * d] = *reinterpret_cast<const double *>(tab + value_lo(w[d]));
        v[2 * d + 1] = *reinterpret_cast<const double *>(tab + value_hi(w[d]));
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) P += v[j];
}

// tab: the table in LDS (occ, then a zero entry at index catalog); stage: this wave's rows.
template <bool P24>
__device__ __forceinline__ void dense_lane_staged(const TrialArgs &a, const char *tab, char *stage, int64_t first,
                                                  int64_t stride) {
    typedef typename std::conditional<P24, u32x3, u32x4>::type Ids;   // four IDs
    constexpr int kBytes = P24 ? 3 : 4;
    constexpr int64_t kSpan = int64_t(1) << 28;
    const uint32_t C = uint32_t(a.catalog), c2 = C | (C << 16);
    const int lane = threadIdx.x & 63, row8 = lane >> 3, col = lane & 7;
    const char *masks = tab + lane_masks_at(a.catalog);
    const char *src = P24 ? reinterpret_cast<const char *>(a.ids24) : reinterpret_cast<const char *>(a.ids);
    // IDs that can be read: the packed copy is padded to whole groups
    const int64_t n_ids = P24 ? (a.n_events + 3) & ~int64_t(3) : a.n_events;
    uint32_t bad = 0, mx = 0, big = 0;
    // the trials being loaded, of trial 8 i + row8 for column col of its windows: the byte
    // offset in window 0, and the IDs from there to the trial's end
    uint32_t st[8];
    int32_t left[8];
    __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)src, 0, 0, kBufWord3);
    Ids R[8];
    auto load = [&](uint32_t w) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t off = int32_t(32u * w) < left[i] ? st[i] : 0xF0000000u;   // outside any record
            const int window = int(32u * w * uint32_t(kBytes));
            if constexpr (P24) R[i] = __builtin_amdgcn_raw_buffer_load_b96(rs, int(off), window, 0);
            else R[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, int(off), window, 0);
        }
    };
    // the trial's positions [lead, len) from its first group on, and its sum so far
    struct Trial {
        int32_t lead, len;
        double P;
    };
    int64_t o0 = 0, o1 = 0;   // offsets of the trial to open next
    auto fetch = [&](int64_t t) {
        o0 = o1 = 0;
        if (t < a.t_end) o0 = a.offs[t], o1 = a.offs[t + 1];
    };
    auto open = [&]() {
        Trial x{0, 0, 0.0};
        if (!(o0 >= 0 && o0 <= o1 && o1 <= a.n_events)) {
            bad |= ERR_OFFSETS;
            o0 = o1 = 0;
        }
        const int64_t base = uniform64(o0) & ~int64_t(3);
        if (__builtin_amdgcn_ballot_w64(o1 > o0 && (o0 < base || o1 - base > kSpan)) != 0) {
            // trials too long for one record (or bad offsets among them): one ID at a time
            for (int64_t p = o0; p < o1; ++p) {
                const uint32_t id = uint32_t(a.ids[p]);
                big |= id >= C ? 1u : 0u;
                x.P += *reinterpret_cast<const double *>(tab + 8u * min(id, C));
            }
            o0 = o1 = 0;
        }
        uint32_t s = 0;
        if (o1 > o0) {
            s = uint32_t((o0 & ~int64_t(3)) - base);
            x.lead = int32_t(o0 & 3);
            x.len = int32_t(o1 - (o0 & ~int64_t(3)));
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            st[i] = (uint32_t(__shfl(int(s), 8 * i + row8, 64)) + 4u * uint32_t(col)) * uint32_t(kBytes);
            left[i] = __shfl(x.len, 8 * i + row8, 64) - 4 * col;
        }
        const int64_t n = min(n_ids - base, kSpan + 4);
        rs = __builtin_amdgcn_make_buffer_rsrc((void *)(src + base * kBytes), 0, int(uint32_t(n) * uint32_t(kBytes)), kBufWord3);
        return x;
    };
    int64_t t = first;
    if (__builtin_amdgcn_ballot_w64(t < a.t_end) == 0) return;
    fetch(t);
    Trial cur = open();
    fetch(t + stride);
    load(0);
    uint32_t w = 0;
    for (;;) {
        // this window's IDs to LDS; a row's 16-byte pieces are rotated by its number / 4 so that
        // the lanes' reads below fall on different banks
        uint32_t to = uint32_t(row8 * kRowBytes + ((col >> 1) ^ (row8 >> 2)) * 16 + (col & 1) * 8);
        asm volatile("" : "+v"(to));   // formed here, not kept over the loop (as turn below)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
            u32x2 p;
            if constexpr (P24) {   // the low two bytes of each three (the IDs are below the catalog, it below 2^16)
                p.x = __builtin_amdgcn_perm(R[i].y, R[i].x, 0x04030100u);
                p.y = __builtin_amdgcn_perm(R[i].z, R[i].y, 0x06050302u);
            } else {
                p.x = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pk_u16(R[i].x, R[i].y));   // saturated
                p.y = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pk_u16(R[i].z, R[i].w));
            }
            *reinterpret_cast<u32x2 *>(stage + (to ^ (i & 1 ? 32u : 0u)) + 8 * i * kRowBytes) = p;
        }
        const bool more = __builtin_amdgcn_ballot_w64(cur.len > int32_t(32u * w + 32u)) != 0;
        Trial nxt = cur;
        const int64_t tn = t + stride;
        const bool last = !more && __builtin_amdgcn_ballot_w64(tn < a.t_end) == 0;
        if (!more && !last) {
            nxt = open();
            fetch(tn + stride);
        }
        if (!last) load(more ? w + 1u : 0u);
        __builtin_amdgcn_wave_barrier();
        const int32_t hi = cur.len - int32_t(32u * w);
        const char *row = stage + lane * kRowBytes;
        uint32_t turn = uint32_t((lane >> 2) & 3) * 16u;
        asm volatile("" : "+v"(turn));   // four addresses formed here, not kept over the loop
        u32x4 q[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) q[p] = *reinterpret_cast<const u32x4 *>(row + (turn ^ uint32_t(16 * p)));
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            if (p == 0 && w == 0)
                row_add<true, true, P24>(tab, masks, q[0], cur.lead, hi, c2, cur.P, mx);
            else if (__builtin_amdgcn_ballot_w64(hi < 8 * p + 8) == 0)
                row_add<false, false, P24>(tab, masks, q[p], 0, 0, c2, cur.P, mx);
            else if (__builtin_amdgcn_ballot_w64(hi > 8 * p) != 0)
                row_add<false, true, P24>(tab, masks, q[p], 0, hi - 8 * p, c2, cur.P, mx);
        }
        __builtin_amdgcn_wave_barrier();
        if (more) {
            ++w;
            continue;
        }
        if (t < a.t_end) a.ylt[t - a.t_begin] = excess(cur.P, a.agg_r, a.agg_l);
        if (last) break;
        t = tn;
        cur = nxt;
        w = 0;
    }
    if (max(mx & 0xFFFFu, mx >> 16) >= C || big) bad |= ERR_ID_RANGE;
    if (bad) atomicOr(a.err, bad);
}

// Lane per trial from a table in LDS: staged when the table leaves the workgroup's waves the
// room, from the packed IDs if there are any.  lds: the table, staged with its zero entry in
// that case; the rows follow it.
__device__ __forceinline__ void dense_lane_lds(const TrialArgs &a, uint32_t *lds, int64_t first, int64_t stride) {
    if (!a.staged) {
        dense_lane_run<ARA_PLACE_LDS_DENSE>(a, lds, first, stride);
        return;
    }
    char *tab = reinterpret_cast<char *>(lds);
    char *stage = tab + lane_table_bytes(a.catalog) + (threadIdx.x >> 6) * kStageBytes;
    if (a.ids24) dense_lane_staged<true>(a, tab, stage, first, stride);
    else dense_lane_staged<false>(a, tab, stage, first, stride);
}

}  // namespace ara
