// Tiled trial kernel: the YLT path for catalogs whose occurrence-net table does not fit
// in LDS as a whole.
//
// Per trial it computes what the bitmap kernel computes (Section II-B, steps 1-4):
//   ylt = min(max(P - AggR, 0), AggL),  P = sum over the trial's occurrences of the
//   occurrence-net loss of their event,
// which telescopes from the basic algorithm's per-occurrence ceded losses.  P is a sum
// of non-negative terms, so they may be taken in any grouping; here they are grouped
// by catalog bin.  The YET's catalog-binned copy (k_bin.hip) holds, bin after bin, the
// occurrences of each bin's 2^14 events as 2-byte bin-local IDs, trial after trial.
// A persistent workgroup owns up to kTiledPassTrials trials per pass.  For each bin it
// stages the bin's 2^14 occurrence-net values in LDS (binary64, the layer's `occ`
// table: zero for events outside the layer), then each lane adds the values of its own
// trial's run in the bin: one LDS read per occurrence, and no filter, queue, search or
// atomic.
//   Lane l of wave w, group g (< 4) holds trial T0(w) + 64 g + l.  A group's 64 runs are
//   one span of the bin; a lane reads its run 8 IDs (16 bytes) at a time from the run's
//   first even position.  An odd-starting run's first ID slot is the previous run's
//   last ID: it is redirected to a zero slot after the table.
//   Four such loads (runs of up to 32 occurrences) are issued one group before the
//   group is added (the groups take turns in two register slots); the rest of a longer
//   run is read 32 IDs at a time when reached.  Each bin's values are loaded into registers
//   while the previous bin is added, and written to LDS between two barriers.
//   (Three slots, two groups ahead, need an unrolled loop over three bins and more
//   registers than a wave has: 30 KB of code and 15 spilled registers.  Two take 18 KB and
//   none, and are faster everywhere: 10^6 trials of 1000 occurrences over 62 bins 0.483 ->
//   0.470 ms, 50,000 of 600 over 19 bins 36 -> 30 us.  With runs of 36 to 88 occurrences
//   per bin the rest of the run, read 8 IDs at a time with a wait each, took another 5% of
//   eight uneven analyses: 638 -> 602 -> 575 us.)
// A trial's P is added in a fixed order (bin groups, bins, positions) that depends on the
// catalog alone: the same bits on every run, in every launch and in every YET that holds the
// trial.  A group's sums are in registers (a lane's four trials), the totals in LDS (one
// binary64 per trial of the wave).
#include <algorithm>

#include <hip/hip_ext.h>

#include "trial_common.h"

namespace ara {

constexpr int kGroups = 4;                                       // groups of 64 trials per wave and pass
constexpr int kOct = 4;                                          // 8-ID loads issued ahead per run
constexpr uint32_t kZeroAddr = uint32_t(kBinEvents) * 8u;        // LDS byte address of the zero slot
constexpr uint32_t kZeroId = uint32_t(kBinEvents);               // bin-local ID that reads the zero slot
constexpr int kStageVecs = kBinEvents / (2 * kTiledWaves * 64);  // 16-byte value loads per thread per bin
static_assert(kTiledWaveTrials <= 64 * kGroups && kStageVecs * 2 * kTiledWaves * 64 == kBinEvents, "shapes");
static_assert(kTiledPassTrials == kTiledWaveTrials * kTiledWaves, "a pass fills every wave's sums");

typedef double f64x2 __attribute__((ext_vector_type(2)));

// Wave-uniform reads of tables the kernel never writes, through the scalar data path.
template <typename V>
__device__ __forceinline__ V sload(const V *p) {
    typedef const __attribute__((address_space(4))) V *cptr;
    return *(cptr)p;
}

__device__ __forceinline__ double lds_f64(const double *tab, uint32_t byte_addr) {
    return *reinterpret_cast<const double *>(reinterpret_cast<const char *>(tab) + byte_addr);
}

template <bool MAX>
__device__ __forceinline__ void fold(double &acc, double v) {
    if (MAX) acc = v > acc ? v : acc;   // occurrence-net losses are >= +0.0
    else acc += v;
}

// Bin b's span of the binned copy as a buffer (reads past it return zero).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t bin_rsrc(const TiledArgs &a, int32_t b) {
    const int64_t r0 = offset_at(a.region, b), r1 = offset_at(a.region, b + 1);
    return __builtin_amdgcn_make_buffer_rsrc((void *)(a.ids16 + r0), 0, int(uint32_t((r1 - r0) * 2)), kBufWord3);
}

// The same record as four words, for inline assembly.
__device__ __forceinline__ i32x4 bin_words(const TiledArgs &a, int32_t b) {
    const int64_t r0 = offset_at(a.region, b), r1 = offset_at(a.region, b + 1);
    const uint64_t base = reinterpret_cast<uint64_t>(a.ids16 + r0);
    return i32x4{int32_t(uint32_t(base)), int32_t(uint32_t(base >> 32) & 0xFFFFu), int32_t(uint32_t((r1 - r0) * 2)), kBufWord3};
}

// Bin b's values into registers: occ[2^14 b + i] (zero past the catalog).
__device__ __forceinline__ void stage_load(const TiledArgs &a, int32_t b, f64x2 (&st)[kStageVecs]) {
    const int64_t e0 = int64_t(b) * kBinEvents;
    const int64_t n = min(int64_t(kBinEvents), int64_t(a.catalog) - e0);
    const __amdgpu_buffer_rsrc_t r =
        __builtin_amdgcn_make_buffer_rsrc((void *)(a.occ + e0), 0, int(max(n, int64_t(0)) * 8), kBufWord3);
#pragma unroll
    for (int u = 0; u < kStageVecs; ++u)
        st[u] = __builtin_bit_cast(f64x2, __builtin_amdgcn_raw_buffer_load_b128(
                                              r, int((threadIdx.x + u * kTiledWaves * 64) * 16), 0, 0));
}

// One lane's run in one bin.
struct Unit {
    uint32_t s;       // first position of the run, in the bin's span
    u32x4 q[kOct];    // IDs at positions (s & ~1) + 8 k .. + 7
};

// Loads with the default cache policy: a lane's four loads overlap the next lanes'
// runs, so the same lines are read several times within a group (a non-temporal hint
// made the kernel 30% slower).
__device__ __forceinline__ void unit_issue(__amdgpu_buffer_rsrc_t r, Unit &u) {
    const uint32_t s1 = u.s & ~1u;
#pragma unroll
    for (int k = 0; k < kOct; ++k) u.q[k] = __builtin_amdgcn_raw_buffer_load_b128(r, int((s1 + 8u * k) * 2u), 0, 0);
}

// The 32 IDs from byte offset `at` of the span on, for the part of a run past the loads
// issued ahead.  The loads wait for themselves inside the asm block, so the compiler's
// count of the outstanding prefetch loads (which it uses to wait for exactly the group it
// adds next) stays exact (as builtins they cost runs without such a part 2%).  s_nop: a
// scalar register of the record that a vector instruction wrote is ready.
__device__ __forceinline__ void load_ids_now(const i32x4 &span, uint32_t at, u32x4 (&q)[kOct]) {
    static_assert(kOct == 4, "four loads");
    asm volatile("s_nop 4\n\t"
                 "buffer_load_dwordx4 %0, %4, %5, 0 offen\n\t"
                 "buffer_load_dwordx4 %1, %4, %5, 0 offen offset:16\n\t"
                 "buffer_load_dwordx4 %2, %4, %5, 0 offen offset:32\n\t"
                 "buffer_load_dwordx4 %3, %4, %5, 0 offen offset:48\n\t"
                 "s_waitcnt vmcnt(0)"
                 : "=&v"(q[0]), "=&v"(q[1]), "=&v"(q[2]), "=&v"(q[3]) : "v"(at), "s"(span) : "memory");
}

// Four IDs (words w0, w1) at positions p .. p + 3 of a run of `len`; those past the run
// read the zero slot.  One test per ID everywhere costs two instructions each, but a wave
// takes its longest run's words once (28 of 64 lanes' 16.4 on average): whole words under a
// lane mask and then a tail of up to 7 apart took 0.500 ms for 10^6 trials of 1000
// occurrences over 62 bins, this 0.483 (both with three slots).  (What bounds it: the LDS is busy 60% of the time,
// half of that with bank conflicts of the random reads, and the vector units 47%; twice as
// many reads in flight per wave, or an untested path for full words, were slower: 0.500 and
// 0.490.)
template <bool MAX>
__device__ __forceinline__ void add4(const double *tab, uint32_t w0, uint32_t w1, uint32_t p, uint32_t len, double &acc) {
    uint32_t at[4] = {value_lo(w0), value_hi(w0), value_lo(w1), value_hi(w1)};
    double v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = lds_f64(tab, p + uint32_t(j) < len ? at[j] : kZeroAddr);
#pragma unroll
    for (int j = 0; j < 4; ++j) fold<MAX>(acc, v[j]);
}

// The 8 IDs of q at positions p .. p + 7, as far as any lane's run reaches.
template <bool MAX>
__device__ __forceinline__ void add8(const double *tab, const u32x4 &q, uint32_t p, uint32_t len, double &acc) {
    add4<MAX>(tab, q[0], q[1], p, len, acc);
    if (__builtin_amdgcn_ballot_w64(len > p + 4u) != 0) add4<MAX>(tab, q[2], q[3], p + 4u, len, acc);
}

// Adds the run [u.s, e) into acc, positions in order.  span: the bin's record.
constexpr uint32_t kPastSpan = 0xFFFFFF00u;   // no access (with the loads' offsets too)
template <bool MAX>
__device__ __forceinline__ void unit_run(const double *tab, const i32x4 &span, Unit &u, uint32_t e, double &acc) {
    const uint32_t s1 = u.s & ~1u;
    const uint32_t len = e > s1 ? e - s1 : 0u;
    if (u.s & 1u) u.q[0].x = (u.q[0].x & 0xFFFF0000u) | kZeroId;
#pragma unroll
    for (int k = 0; k < kOct; ++k) {
        if (__builtin_amdgcn_ballot_w64(len > 8u * k) == 0) return;
        add8<MAX>(tab, u.q[k], 8u * k, len, acc);
    }
#pragma unroll 1
    for (uint32_t p = 8u * kOct; __builtin_amdgcn_ballot_w64(len > p) != 0; p += 8u * kOct) {
        load_ids_now(span, len > p ? (s1 + p) * 2u : kPastSpan, u.q);
#pragma unroll
        for (int k = 0; k < kOct; ++k) {
            if (__builtin_amdgcn_ballot_w64(len > p + 8u * k) == 0) return;
            add8<MAX>(tab, u.q[k], p + 8u * k, len, acc);
        }
    }
}

// One pass of a workgroup over trials [T0, T1) of each wave (at most kTiledWaveTrials) and bin
// groups [g0, g1) of analysis a: every bin staged once, each lane's trials added bin by bin
// in registers; where a group ends its sums join the total so far in ws[64 g + lane] (groups
// up to a.first_row, all of them without a.part), or go to the group's row of a.part.
// MAX = false: sums of the occurrence-net losses; MAX = true: each trial's largest.
// Units u = 4 b + g (bin b, group g of 64 trials) take turns in two register slots (slot
// u % 2): unit u + 2 is issued once unit u is added.  No load is issued under a condition, so
// that every wait counts only the loads issued after the one it waits for: past the last
// bin, the last one's loads are issued again and its runs are empty.
// B24: run starts in 3 bytes each, read as an unaligned 4-byte word (its top byte,
// the next entry's first, masked off where the value is taken).
// rare: the same arguments in memory, for what a group's end needs (kept in registers over the
// loop, they spilled others: 0.52 ms with 3-byte run starts, now 0.48).
typedef const __attribute__((address_space(4))) TiledArgs *ArgsInMemory;
template <bool MAX, bool B24>
__device__ __forceinline__ void tiled_pass(const TiledArgs &a, ArgsInMemory rare, int64_t T0, int64_t T1, int32_t g0,
                                           int32_t g1, double *tab, double *ws, int lane) {
    const int32_t bin0 = g0 * a.group_bins, bin1 = min(g1 * a.group_bins, a.n_bins);
    int32_t bg = g0, bg_end = min(bin0 + a.group_bins, bin1);   // the bin group and its last bin + 1
    double acc[kGroups] = {};
    // start of the run of trial T0 + 64 g + lane (the wave's span end past T1), and
    // the end of the group's last run (scalar)
    constexpr uint32_t kRunMask = B24 ? 0xFFFFFFu : 0xFFFFFFFFu;
    auto run_start = [&](int32_t b, int g) -> uint32_t {   // the word before masking
        const int64_t i = int64_t(b) * a.stride + min(T0 + 64 * g + lane, T1);
        if (!B24) return a.boff[i];
        uint32_t w;
        __builtin_memcpy(&w, a.boff24 + 3 * i, 4);
        return w;
    };
    auto group_end = [&](int32_t b, int g) -> uint32_t {
        const int64_t i = int64_t(b) * a.stride + min(T0 + 64 * g + 64, T1);
        if (!B24) return sload(a.boff + i);
        // the two aligned words holding bytes 3 i .. 3 i + 2
        const uint32_t *p = reinterpret_cast<const uint32_t *>(a.boff24 + ((3 * i) & ~int64_t(3)));
        const uint64_t w = uint64_t(sload(p)) | (uint64_t(sload(p + 1)) << 32);
        return uint32_t(w >> (8 * ((3 * i) & 3))) & kRunMask;
    };
    f64x2 st[kStageVecs];
    stage_load(a, bin0, st);
    __amdgpu_buffer_rsrc_t rc = bin_rsrc(a, bin0);
    i32x4 pc = bin_words(a, bin0);
    Unit U[2];
    uint32_t sc[kGroups], ge[kGroups];   // this bin's run starts and group ends
#pragma unroll
    for (int g = 0; g < kGroups; ++g) sc[g] = run_start(bin0, g) & kRunMask;
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        U[g].s = sc[g];
        unit_issue(rc, U[g]);
    }
#pragma unroll
    for (int g = 0; g < kGroups; ++g) ge[g] = group_end(bin0, g);
#pragma unroll 1
    for (int32_t b = bin0; b < bin1; ++b) {
        const bool more = b + 1 < bin1;
        const int32_t bn = more ? b + 1 : bin1 - 1;
        const __amdgpu_buffer_rsrc_t rn = bin_rsrc(a, bn);
        const i32x4 pn = bin_words(a, bn);
        uint32_t sn[kGroups], gn[kGroups];
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            const uint32_t x = run_start(bn, g), y = group_end(bn, g);
            sn[g] = more ? x & kRunMask : 0u;
            gn[g] = more ? y : 0u;
        }
        __syncthreads();   // every wave is done with the previous bin
        f64x2 *dst = reinterpret_cast<f64x2 *>(tab);
#pragma unroll
        for (int u = 0; u < kStageVecs; ++u) dst[threadIdx.x + u * kTiledWaves * 64] = st[u];
        __syncthreads();
        stage_load(a, bn, st);
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            const int slot = g & 1;
            // a run ends where the next lane's starts; lane 63's at the group end
            const uint32_t nx = uint32_t(__builtin_amdgcn_ds_bpermute(((lane + 1) & 63) * 4, int(U[slot].s)));
            const uint32_t e = lane == 63 ? ge[g] : nx;
            unit_run<MAX>(tab, pc, U[slot], e, acc[g]);   // lanes past T1: empty runs
            U[slot].s = g < 2 ? sc[g + 2] : sn[g - 2];
            unit_issue(g < 2 ? rc : rn, U[slot]);
        }
#pragma unroll
        for (int g = 0; g < kGroups; ++g) sc[g] = sn[g], ge[g] = gn[g];
        rc = rn;
        pc = pn;
        if (b + 1 != bg_end) continue;
        ArgsInMemory m = rare;
        asm volatile("" : "+s"(m));   // read here, not before the loop
        double *part = m->part && bg > m->first_row ? m->part + (bg * m->part_stride - m->t_begin) : nullptr;
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            const int64_t t = T0 + 64 * g + lane;
            if (t < T1) {
                if (part) {
                    part[t] = acc[g];
                } else {
                    double x = ws[64 * g + lane];   // group 0: an earlier pass's
                    x = bg > 0 ? x : 0.0;
                    fold<MAX>(x, acc[g]);
                    ws[64 * g + lane] = x;
                }
            }
            acc[g] = 0.0;
        }
        ++bg;
        bg_end = min(bg_end + m->group_bins, bin1);
    }
}

// Trials [t0, t1) (at most one pass) over bin groups [g0, g1) of analysis a.  A trial's
// total is ((s_0 + s_1) + s_2) + ..., s_g its sum over group g's bins, taken here (every
// group) or, with a.part, by k_tiled_combine in the same order: row first_row of a.part holds
// the total up to its group, each later row its own group's sum.  The groups depend on the
// catalog alone, so a trial's YLT does not depend on how they are spread over workgroups,
// nor on the other trials of its YET.
template <bool MAX, bool B24>
__device__ __forceinline__ void tiled_groups(const TiledArgs &a, ArgsInMemory rare, int64_t t0, int64_t t1, int32_t g0, int32_t g1,
                                             double *tab, double *ws, int lane, uint32_t wave) {
    const int64_t per_wave = (t1 - t0 + kTiledWaves - 1) / kTiledWaves;
    const int64_t T0 = min(t0 + int64_t(wave) * per_wave, t1);
    const int64_t T1 = min(T0 + per_wave, t1);
    tiled_pass<MAX, B24>(a, rare, T0, T1, g0, g1, tab, ws, lane);
    asm volatile("" : "+s"(rare));
    const bool whole = rare->part == nullptr;
    if (!whole && g0 > rare->first_row) return;
    double *out = whole ? rare->ylt : rare->part + rare->first_row * rare->part_stride;
    const double r = whole ? rare->agg_r : 0.0, l = whole ? rare->agg_l : __builtin_inf();
#pragma unroll 1
    for (int g = 0; g < kGroups; ++g) {
        const int64_t t = T0 + 64 * g + lane;
        if (t < T1) out[t - rare->t_begin] = MAX ? ws[64 * g + lane] : excess(ws[64 * g + lane], r, l);
    }
}

// One analysis.  Whole (part null): workgroup w owns trials [t_begin + w
// per_wg, + per_wg), in passes, over every bin group.  Split: item i = (span of span_groups bin
// groups, chunk of per_wg trials), a workgroup each, chunks of a span in a row; XCD x
// (workgroups x, x + 8, ...) takes a contiguous eighth of the items, so its L2 holds the
// values of its own spans' bins only.
template <bool MAX, bool B24>
__global__ __launch_bounds__(1024) void k_trial_tiled(TiledArgs a) {
    __shared__ __attribute__((aligned(16))) double tab[kBinEvents + 2];   // a bin's values, the zero slot
    __shared__ double sums[kTiledWaves * kTiledWaveTrials];
    const int lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (threadIdx.x == 0) tab[kBinEvents] = 0.0;
    int32_t g0 = 0, g1 = a.n_groups;
    int64_t wg0 = a.t_begin + int64_t(blockIdx.x) * a.per_wg;
    if (a.part) {
        const int32_t items = a.chunks * tiled_spans(a.n_groups, a.span_groups), each = (items + kXcds - 1) / kXcds;
        const int32_t i = int32_t(blockIdx.x % kXcds) * each + int32_t(blockIdx.x / kXcds);
        if (i >= items || int32_t(blockIdx.x / kXcds) >= each) return;
        g0 = i / a.chunks * a.span_groups;
        g1 = min(g0 + a.span_groups, a.n_groups);
        wg0 = a.t_begin + int64_t(i % a.chunks) * a.per_wg;
    }
    const int64_t wg1 = min(wg0 + a.per_wg, a.t_end);
#pragma unroll 1
    for (int64_t pass = wg0; pass < wg1; pass += kTiledPassTrials)
        tiled_groups<MAX, B24>(a, (ArgsInMemory)__builtin_amdgcn_kernarg_segment_ptr(), pass,   // its only argument
                               min(pass + int64_t(kTiledPassTrials), wg1), g0, g1, tab, sums + wave * kTiledWaveTrials, lane,
                               wave);
}

// The totals of split analyses from their bin groups' sums (grid.y: the analysis), two
// trials per thread.
template <bool MAX>
__device__ __forceinline__ void combine_groups(const TiledArgs &a) {
    const int64_t n = a.t_end - a.t_begin;
    for (int64_t i = (int64_t(blockIdx.x) * 256 + threadIdx.x) * 2; i < n; i += int64_t(gridDim.x) * 512) {
        // part rows are 16-byte aligned and padded
        f64x2 s = *reinterpret_cast<const f64x2 *>(a.part + a.first_row * a.part_stride + i);
#pragma unroll 4
        for (int32_t g = a.first_row + 1; g < a.n_groups; ++g) {
            const f64x2 x = *reinterpret_cast<const f64x2 *>(a.part + g * a.part_stride + i);
#pragma unroll
            for (int k = 0; k < 2; ++k) s[k] = MAX ? (x[k] > s[k] ? x[k] : s[k]) : s[k] + x[k];
        }
#pragma unroll
        for (int k = 0; k < 2; ++k)
            if (i + k < n) a.ylt[i + k] = MAX ? s[k] : excess(s[k], a.agg_r, a.agg_l);
    }
}

template <bool MAX>
__global__ __launch_bounds__(256) void k_tiled_combine(TiledArgs a) {
    combine_groups<MAX>(a);
}

// Analysis j's arguments from device memory, through the scalar data path.
__device__ __forceinline__ TiledArgs load_args(const TiledArgs *jobs, int32_t j) {
    static_assert(sizeof(TiledArgs) % 4 == 0, "whole words");
    TiledArgs a;
    const uint32_t *src = reinterpret_cast<const uint32_t *>(jobs + j);
    uint32_t w[sizeof(TiledArgs) / 4];
#pragma unroll
    for (int i = 0; i < int(sizeof(TiledArgs) / 4); ++i) w[i] = sload(src + i);
    __builtin_memcpy(&a, w, sizeof(TiledArgs));
    return a;
}

// Many analyses in one launch (YLTs): each item is a pass over up to kTiledPassTrials
// trials of one analysis, over every bin group or (split analyses) some of them, taken in
// list order from a counter by whichever workgroup is free; a workgroup stops once the
// counter passes the list.  A trial's YLT does not depend on the pass that holds it, so
// these give the bits of k_trial_tiled.
__global__ __launch_bounds__(1024) void k_trial_tiled_items(const TiledArgs *__restrict__ jobs,
                                                            const TiledItem *__restrict__ items, int32_t n_items,
                                                            uint32_t *__restrict__ next) {
    __shared__ __attribute__((aligned(16))) double tab[kBinEvents + 2];
    __shared__ double sums[kTiledWaves * kTiledWaveTrials];
    __shared__ uint32_t took;
    const int lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (threadIdx.x == 0) tab[kBinEvents] = 0.0;
    for (;;) {
        if (threadIdx.x == 0) took = atomicAdd(next, 1u);
        __syncthreads();
        const uint32_t it = __builtin_amdgcn_readfirstlane(took);
        __syncthreads();   // every wave has read `took` before it is taken again
        if (it >= uint32_t(n_items)) return;
        const uint32_t *iw = reinterpret_cast<const uint32_t *>(items + it);
        const int32_t job = int32_t(sload(iw + 0));
        const uint32_t groups = sload(iw + 1);
        const int64_t t0 = int64_t(uint64_t(sload(iw + 2)) | (uint64_t(sload(iw + 3)) << 32));
        const int64_t t1 = int64_t(uint64_t(sload(iw + 4)) | (uint64_t(sload(iw + 5)) << 32));
        const TiledArgs a = load_args(jobs, job);
        const int32_t g0 = int32_t(groups & 0xFFFFu), g1 = int32_t(groups >> 16);
        double *ws = sums + wave * kTiledWaveTrials;
        const ArgsInMemory rare = (ArgsInMemory)(jobs + job);
        if (a.boff24) tiled_groups<false, true>(a, rare, t0, t1, g0, g1, tab, ws, lane, wave);
        else tiled_groups<false, false>(a, rare, t0, t1, g0, g1, tab, ws, lane, wave);
    }
}

__global__ __launch_bounds__(256) void k_tiled_combine_items(const TiledArgs *__restrict__ jobs,
                                                             const int32_t *__restrict__ split) {
    const TiledArgs a = load_args(jobs, int32_t(sload(split + blockIdx.y)));
    combine_groups<false>(a);
}

static unsigned combine_blocks(int64_t n) {
    return unsigned(std::max<int64_t>(1, std::min<int64_t>((n + 511) / 512, 1024)));
}

hipError_t launch_tiled_combine_items(const TiledArgs *jobs, const int32_t *split, int32_t n_split, int64_t n_max,
                                      hipStream_t s) {
    if (n_split <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_tiled_combine_items, dim3(combine_blocks(n_max), unsigned(n_split)), dim3(256), 0, s, jobs, split);
    return hipGetLastError();
}

hipError_t launch_trial_tiled_items(const TiledArgs *jobs, const TiledItem *items, int32_t n_items, uint32_t *next,
                                    int grid, hipStream_t s) {
    if (n_items <= 0) return hipSuccess;
    const hipError_t e = launch_fill_u32(next, 1, 0u, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_trial_tiled_items, dim3(grid), dim3(kTiledWaves * 64), 0, s, jobs, items, n_items, next);
    return hipGetLastError();
}

hipError_t launch_trial_tiled(const TiledArgs &a, int grid, hipStream_t s, bool occ_max, hipEvent_t start,
                              hipEvent_t stop) {
    const int items = a.part ? (a.chunks * tiled_spans(a.n_groups, a.span_groups) + kXcds - 1) / kXcds * kXcds : grid;
    const dim3 g(items), b(kTiledWaves * 64);
    hipEvent_t end = a.part ? nullptr : stop;
    if (a.boff24) {
        if (occ_max) hipExtLaunchKernelGGL((k_trial_tiled<true, true>), g, b, 0, s, start, end, 0, a);
        else hipExtLaunchKernelGGL((k_trial_tiled<false, true>), g, b, 0, s, start, end, 0, a);
    } else {
        if (occ_max) hipExtLaunchKernelGGL((k_trial_tiled<true, false>), g, b, 0, s, start, end, 0, a);
        else hipExtLaunchKernelGGL((k_trial_tiled<false, false>), g, b, 0, s, start, end, 0, a);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !a.part) return e;
    const dim3 cg(combine_blocks(a.t_end - a.t_begin));
    if (occ_max) hipExtLaunchKernelGGL((k_tiled_combine<true>), cg, dim3(256), 0, s, nullptr, stop, 0, a);
    else hipExtLaunchKernelGGL((k_tiled_combine<false>), cg, dim3(256), 0, s, nullptr, stop, 0, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// Splitting.  Every workgroup stages the bins it goes through, so a launch of few trials
// spread over all CUs was bound by the staging: 10^5 trials of 1000 occurrences over 62 bins
// took 330 us on 256 workgroups of 391 trials, 50,000 of 600 over 19 bins 122 us.  Instead a
// workgroup takes a chunk of up to a full pass of trials and a span of the bin groups: 64 and
// 28 us with the adding up.  Costs in us: 6 per workgroup (start, first bin's load, sums
// written); a bin's staging, and for each 64 trials of a wave, however many of them it has,
// what a run of `run` occurrences takes (325,634 trials of 19.4 per bin: 2 spans of 128 chunks,
// three 64s per wave, 7.4 us a bin; 3 of 85, four, 8.6: 167 and 146 us in all; 250,000 of 13.5:
// 5.7 and 7.0).
static double bin_us(int64_t trials, double run) {
    const int64_t groups = ((trials + kTiledWaves - 1) / kTiledWaves + 63) / 64;
    return 2.0 + double(groups) * (0.55 + 0.055 * run);
}

static double whole_us(int64_t n, int32_t n_bins, double run, int n_cu) {
    const int64_t wgs = std::max<int64_t>(1, std::min<int64_t>(n_cu, (n + 63) / 64));
    const int64_t per = (n + wgs - 1) / wgs, passes = (per + kTiledPassTrials - 1) / kTiledPassTrials;
    return double(passes) * (6.0 + n_bins * bin_us((per + passes - 1) / passes, run));
}

// The split of n trials over n_bins bins that costs least, or chunks = 0: whole.  Sums are
// taken by bin groups; maxima, which are the same in any order, by spans of bins.
TiledSplit tiled_split(int64_t n, int32_t n_bins, double run, int n_cu, bool occ_max) {
    const int32_t gb = occ_max ? (n_bins + 63) / 64 : tiled_group_bins(n_bins), groups = (n_bins + gb - 1) / gb;
    const int64_t least = (n + kTiledPassTrials - 1) / kTiledPassTrials;
    TiledSplit best{0, 0, 0, 0};
    double cost = whole_us(n, n_bins, run, n_cu);
    for (int32_t span = 1; span < groups; ++span) {
        const int32_t spans = tiled_spans(groups, span);
        if (span > 1 && tiled_spans(groups, span - 1) == spans) continue;
        const int32_t bins = std::min(span * gb, n_bins), parts = occ_max ? spans : groups - span + 1;
        // the parts written and read at 4 TB/s, and the combining launch
        const double sums = 5.7 + double(n) * parts * 16.0 / 4e6;
        // as many chunks as fill so many rounds of the CUs, of at least a group of 64 trials
        const int64_t first = (least * spans + n_cu - 1) / n_cu;
        for (int64_t rounds = first; rounds < first + 3; ++rounds) {
            const int64_t chunks = std::max(least, std::min(rounds * n_cu / spans, n / 64));
            const double c = double((chunks * spans + n_cu - 1) / n_cu) * (6.0 + bins * bin_us((n + chunks - 1) / chunks, run)) +
                             sums;
            if (c < cost) {
                cost = c;
                best = occ_max ? TiledSplit{chunks, bins, spans, 1} : TiledSplit{chunks, gb, groups, span};
            }
        }
    }
    return best;
}

}  // namespace ara
