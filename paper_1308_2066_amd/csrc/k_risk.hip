// Risk measures (the PML and TVaR filters of Section I over the YLT of Section II-C)
// by selection.  PML(rp) = the k-th largest loss, TVaR(rp) = the mean of the k largest,
// k = ara_return_period_rank(n, rp).  In descending-order keys PML is the k-th smallest
// key K; the k largest losses are the losses whose key is below K plus (k - their
// number) copies of PML, so
//   TVaR = (sum of the losses whose key is below K + copies * PML) / k.
// That sum is taken in a fixed order: per tile of 2048 losses in index order, 256 slots
// (slot t adds the tile's losses t, t + 256, ..., t + 1792 in turn; the others add
// +0.0) and a fixed tree over the slots; then the tile sums, slot t adding tiles t,
// t + 256, ... in turn, and the same tree.  So every path below gives the same bits.
//
// K is found from a sample of 1024 losses (4096 past 2^22), one pass that counts bins and one that copies a
// few keys out.  The sample gives the smallest sampled key L and a key T that the largest
// rank asked for lies below (five standard deviations beyond its place in the sample).
// The pass counts the keys below L, the keys equal to L (years capped at the aggregate
// limit share it) and 4096 equal bins of [L, T]; keys past T, nine in ten when the
// shortest return period is 10, are not counted at all.  In a YLT without negative losses
// zeros (quiet years) come last: they are counted on their own and do not stretch the
// bins.  The few keys of each rank's bin are then copied out and sorted out.
//
//   up to kRiskOneWg losses: one workgroup (k_risk_one); a rank that the counts do not reach
//   (the sample misled), or whose bin is large, is found by refine(), in more passes.
//   longer: k_risk_sample (one workgroup; clears the counts), k_risk_bins, k_risk_collect
//   (the last workgroup to finish picks K), k_risk_sum (tile sums; the last workgroup to
//   finish forms PML and TVaR).  Where a rank's range holds more than kRiskCollect keys of more
//   than one value, the YLT stays open: the host, which waits for the results anyway, then
//   launches rounds of k_risk_narrow (1024 to 4096 bins of the range's smallest to largest key, by
//   the whole grid), k_risk_collect and k_risk_sum until none is.  A round narrows a range at
//   least 512 times.  (One workgroup went through the YLT alone for such a rank: 2.6 ms for 10^6 losses
//   half of which are close, 18 ms for the 1000-year loss of 10^7, 134 ms of 5 10^7.)
// Both take many YLTs at once (one descriptor each), so a batch pays for the launches
// once.
//
// What bounds it: launches, and the chain of round trips within each.  A launch of
// dependent kernels takes 4.5-5 us whatever it does (8 MB of losses are 1.3 us of HBM), so
// the passes that replaced one 8-bit digit each (12 launches, 105 us for 10^6 distinct
// losses and 135 us when a rank fell among capped years, whose bucket never became small)
// are now four (34 us for 10^6 losses, 24 us for 50,000).  Within a launch, code that runs
// once costs its fetch: with every loop over a thread's 16 keys unrolled for each rank (31 KB
// of code) k_risk_one took 21 us for 1000 losses (11 now).  Counting every key in bins of the
// whole range took 26 us for 10^6 losses: most years fall in a few of those bins, and LDS
// atomics on one word go one after another.
//
// The last workgroup of a launch reads what the others wrote in the same launch: those
// words are stored and loaded with agent-scope atomics (write-through past the XCDs' L2s,
// which do not snoop each other), each workgroup waits for its stores to complete, then
// counts itself; the one that completes the count continues.  No workgroup waits for
// another, and no fence writes an L2 back (one per workgroup cost 50 us a pass).
#include <algorithm>

#include "order_keys.h"

namespace ara {

constexpr int kRiskThreads = 1024;
constexpr int kRiskWaves = kRiskThreads / 64;
constexpr int kRiskBins = 4096;
constexpr int kNarrowBins = 16384;     // bins of k_risk_narrow's ranges together
constexpr int kRiskTile = 2048;        // losses per tile of the TVaR sum
constexpr int kRiskBlocks = 128;       // most workgroups of a pass over one YLT
constexpr int kRiskRow = 4096;         // fewest losses per workgroup
constexpr int kRiskLoads = 8;          // losses a thread reads at a time
constexpr int kRiskCollect = 8192;     // largest bin whose keys are copied out
constexpr uint32_t kFewKeys = 1024;    // a bin that one wave sorts out
constexpr int kWaveKeys = int(kFewKeys) / 64;
static_assert(kRiskGroup <= kRiskWaves, "one wave per rank");
static_assert(kRiskTile == 8 * 256, "a tile is 8 losses for each of 256 slots");

constexpr uint64_t kZeroKey = 0x7FFFFFFFFFFFFFFFull;   // desc_key(0.0): keys above it are negative losses

// (min and max of mixed 64-bit integer types would go through binary64)
__device__ __forceinline__ uint64_t umin(uint64_t a, uint64_t b) { return a < b ? a : b; }
__device__ __forceinline__ uint64_t umax(uint64_t a, uint64_t b) { return a > b ? a : b; }

template <typename T>
__device__ __forceinline__ T agent_load(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void agent_store(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Whether this workgroup is the last of n to come here (whole workgroup).  Its earlier
// agent-scope stores and atomics have completed before it is counted.
__device__ __forceinline__ bool last_to_finish(uint32_t *done, uint32_t n, uint32_t *lds) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0)
        *lds = __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    return *lds == n - 1;
}

__device__ __forceinline__ uint64_t readlane64(uint64_t x, int l) {
    return uint64_t(uint32_t(__builtin_amdgcn_readlane(int(uint32_t(x)), l))) |
           uint64_t(uint32_t(__builtin_amdgcn_readlane(int(uint32_t(x >> 32)), l))) << 32;
}

__host__ __device__ inline int64_t risk_tiles(int64_t n) { return (n + kRiskTile - 1) / kRiskTile; }

// Descriptor i's fields (uniform: scalar loads), and its rank r.
struct JobView {
    const double *y;
    int64_t n;
    double *out;
    unsigned char *ws;
    int m;
    int64_t k_max;
};
typedef const __attribute__((address_space(4))) RiskJob *ConstJob;
__device__ __forceinline__ JobView job_view(const RiskArgs &a, int i) {
    if (!a.jobs) return JobView{a.one.y, a.one.n, a.one.out, a.one.ws, int(a.one.m), a.one.k_max};
    const ConstJob j = (ConstJob)(a.jobs + i);
    return JobView{j->y, j->n, j->out, j->ws, int(j->m), j->k_max};
}
__device__ __forceinline__ int64_t job_rank(const RiskArgs &a, int i, int r) {
    return a.jobs ? ((ConstJob)(a.jobs + i))->k[r] : a.one.k[r];
}

// ------------------------------------------------------------------ sample and bins
// What the passes count, from the sample: keys below lo, keys equal to lo, and bins
// (key - lo) >> shift of the keys in (lo, hi]; with zeros_last, zeros on their own (every
// key in the bins is a positive loss's, and hi is below zero's key).
struct Binning {
    uint64_t lo, hi;
    uint32_t shift;
    uint32_t zeros_last;
};
struct Counts {          // beside the bins
    uint32_t below, equal, zero;
};

// The right shift that maps keys 0 .. range (>= 1) to 2^log bins.
__device__ __forceinline__ uint32_t bin_shift(uint64_t range, int log = __builtin_ctz(kRiskBins)) {
    const int bits = 64 - __builtin_clzll(range);
    return bits > log ? uint32_t(bits - log) : 0u;
}

__device__ __forceinline__ bool in_bins(const Binning &b, uint64_t k) { return k > b.lo && k <= b.hi; }
// The bin of a key in the bins; one far past the sampled keys (in 64 bits: its place may not
// fit in 32) is in the last.
__device__ __forceinline__ uint32_t bin_of(const Binning &b, uint64_t k) {
    return uint32_t(umin((k - b.lo) >> b.shift, uint64_t(kRiskBins - 1)));
}

// Reductions and scans over a wave by DPP lane moves: within rows of 16 lanes, then the
// four rows (a cross-lane permute through the LDS unit takes three times as long).
template <int Ctrl>
__device__ __forceinline__ uint64_t dpp64(uint64_t x) {
    return uint64_t(uint32_t(__builtin_amdgcn_update_dpp(0, int(uint32_t(x)), Ctrl, 0xF, 0xF, false))) |
           uint64_t(uint32_t(__builtin_amdgcn_update_dpp(0, int(uint32_t(x >> 32)), Ctrl, 0xF, 0xF, false))) << 32;
}
template <typename Op>
__device__ __forceinline__ uint64_t wave_reduce(uint64_t x, Op op) {
    x = op(x, dpp64<0xB1>(x));    // quad_perm [1,0,3,2]
    x = op(x, dpp64<0x4E>(x));    // quad_perm [2,3,0,1]
    x = op(x, dpp64<0x141>(x));   // row_half_mirror
    x = op(x, dpp64<0x140>(x));   // row_mirror
    return op(op(readlane64(x, 0), readlane64(x, 16)), op(readlane64(x, 32), readlane64(x, 48)));
}
__device__ __forceinline__ uint64_t wave_min(uint64_t x) {
    return wave_reduce(x, [](uint64_t p, uint64_t q) { return umin(p, q); });
}
__device__ __forceinline__ uint64_t wave_max(uint64_t x) {
    return wave_reduce(x, [](uint64_t p, uint64_t q) { return umax(p, q); });
}
__device__ __forceinline__ uint32_t wave_scan(uint32_t x) {   // inclusive
    x += uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x111, 0xF, 0xF, true));    // row_shr 1
    x += uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x112, 0xF, 0xF, true));    // row_shr 2
    x += uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x114, 0xF, 0xF, true));    // row_shr 4
    x += uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x118, 0xF, 0xF, true));    // row_shr 8
    x += uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x142, 0xA, 0xF, false));   // row_bcast 15 into rows 1, 3
    x += uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x143, 0xC, 0xF, false));   // row_bcast 31 into rows 2, 3
    return x;
}

// ------------------------------------------------------------------ picking
// The state of one rank: its keys are those of [lo, lo + span], `count` of them, and
// the rank is the left-th smallest of these; or it is solved: K, and the copies of K
// among the k largest.
struct RankState {
    uint64_t lo, span, K;
    int64_t left, copies;
    uint32_t count;
    bool solved;
};

// The rank's bin in a row of 64 PER counts (whole wave): the state within it (bins of
// 2^width keys from lo on), or false when the rank lies past the row's last key (total).
// The lanes' shares first, then the PER bins of the lane whose share holds the rank.  Each
// lane starts its share at another place: from the same one, 64 lanes read the same four
// LDS banks.
template <int PER>
__device__ __forceinline__ bool wave_pick(const uint32_t *row, uint64_t lo, uint32_t width, int64_t left, RankState &out,
                                          uint32_t &total) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    static_assert(PER % 4 == 0 && PER <= 64 && (PER & (PER - 1)) == 0, "16-byte reads; one lane per bin of a share");
    const int lane = threadIdx.x & 63;
    uint32_t own = 0;
#pragma unroll 8
    for (int i = 0; i < PER / 4; ++i) {
        const u32x4 q = reinterpret_cast<const u32x4 *>(row + PER * lane)[(i + lane) & (PER / 4 - 1)];
        own += q[0] + q[1] + q[2] + q[3];
    }
    const uint32_t inc = wave_scan(own);
    total = uint32_t(__builtin_amdgcn_readlane(int(inc), 63));
    if (left > int64_t(total)) return false;
    const int l = __ffsll(static_cast<unsigned long long>(__ballot(left <= int64_t(inc)))) - 1;
    const uint32_t before = uint32_t(__builtin_amdgcn_readlane(int(inc - own), l));
    const uint32_t c = lane < PER ? row[PER * l + lane] : 0u;
    const uint32_t run = before + wave_scan(c);
    const int at = __ffsll(static_cast<unsigned long long>(__ballot(left <= int64_t(run)))) - 1;
    out.count = uint32_t(__builtin_amdgcn_readlane(int(c), at));
    out.lo = lo + (uint64_t(PER * l + at) << width);
    out.span = (1ull << width) - 1ull;
    out.left = left - int64_t(uint32_t(__builtin_amdgcn_readlane(int(run - c), at)));
    out.solved = false;
    return true;
}

// The last key of [lo, lo + span] up to hi >= lo.  lo + span itself may lie past the last key
// there is (bins 2^52 wide from a positive loss's key on, the rank among negative NaNs): taken
// modulo 2^64, the range went on among the smallest keys, more of them than were counted.
__device__ __forceinline__ uint64_t range_end(uint64_t lo, uint64_t span, uint64_t hi) {
    return span < hi - lo ? lo + span : hi;
}

// Rank k of `losses` after the counting pass (a wave on its own).  Keys come in the order:
// below lo, equal to lo, bins, with zeros_last zeros, and the rest (`past` is set: they were
// not counted one by one).  A bin's first key is kept out of [lo, ..] when it is b.lo itself,
// and its last one ends at b.hi.
__device__ __forceinline__ RankState pick_bin(const uint32_t *row, const Binning &b, const Counts &n, int64_t k,
                                              int64_t losses, bool &past) {
    RankState s;
    past = false;
    s.solved = false;
    s.K = b.lo;
    s.lo = 0;
    s.left = k, s.copies = 0;
    if (k <= int64_t(n.below)) {
        s.span = b.lo - 1ull;
        s.count = n.below;
        return s;
    }
    const int64_t before = int64_t(n.below) + int64_t(n.equal);
    if (k <= before) {
        s.copies = k - int64_t(n.below);
        s.solved = true;
        return s;
    }
    uint32_t total;
    if (wave_pick<kRiskBins / 64>(row, b.lo, b.shift, k - before, s, total)) {
        const bool last = s.lo == b.lo + (uint64_t(kRiskBins - 1) << b.shift);   // holds the keys up to b.hi
        const uint64_t end = last ? b.hi : range_end(s.lo, s.span, b.hi);
        s.lo = umax(s.lo, b.lo + 1ull);
        s.span = end - s.lo;
        return s;
    }
    // past the bins: a zero, if the bins held every positive loss, or one of the rest
    int64_t counted = before + int64_t(total);
    s.lo = b.hi + 1ull;   // b.hi is not the last key there is: the bins would hold the rank
    if (b.zeros_last && b.hi == kZeroKey - 1ull) {
        if (k <= counted + int64_t(n.zero)) {
            s.K = kZeroKey;
            s.copies = k - counted;
            s.solved = true;
            return s;
        }
        counted += int64_t(n.zero);
        s.lo = kZeroKey + 1ull;
    }
    s.span = ~0ull - s.lo;
    s.left = k - counted;
    s.count = uint32_t(losses - counted);
    past = true;
    return s;
}

// The first rank whose bin is rank r's too (r itself if none before it); a wave on its own.
__device__ __forceinline__ int first_of_bin(const RankState *st, int r) {
    const int q = threadIdx.x & 63;
    const bool same = q <= r && !st[q].solved && st[q].lo == st[r].lo && st[q].span == st[r].span;
    return __ffsll(static_cast<unsigned long long>(__ballot(same))) - 1;
}

// The left-th smallest of the c <= 64 keys the lanes hold.
__device__ __forceinline__ void wave_select(uint64_t key, int c, int64_t left, uint64_t &K, int64_t &copies) {
    const int lane = threadIdx.x & 63;
    int less = 0, eq = 0;
#pragma unroll 1
    for (int j = 0; j < c; ++j) {
        const uint64_t o = readlane64(key, j);
        less += o < key ? 1 : 0;
        eq += o == key ? 1 : 0;
    }
    const bool hit = lane < c && int64_t(less) < left && left <= int64_t(less + eq);
    const int l = __ffsll(static_cast<unsigned long long>(__ballot(hit))) - 1;
    K = readlane64(key, l);
    copies = left - int64_t(__builtin_amdgcn_readlane(less, l));
}

// The left-th smallest of the c <= kFewKeys keys key(i), by one wave: up to 64 at once; more
// by halving the range of the keys still in question, which ends at once when they are all
// one loss (losses that come from few events are shared by many years).  Each rank has its
// own wave; refine() takes the workgroup through them one after another, and k_risk_collect
// took 25 us for the three ranks of 10^5 trials' largest occurrences, now 13.
template <typename Key>
__device__ __forceinline__ void wave_select_any(int count, int64_t left, uint64_t &K, int64_t &copies, Key key) {
    const int lane = threadIdx.x & 63;
    const int c = __builtin_amdgcn_readfirstlane(count);
    if (c <= 64) {
        wave_select(lane < c ? key(lane) : ~0ull, c, left, K, copies);
        return;
    }
    uint64_t x[kWaveKeys];
    uint32_t in = 0;   // the keys still in question, a bit each
#pragma unroll
    for (int u = 0; u < kWaveKeys; ++u) {
        if (64 * u >= c) continue;
        const bool have = lane + 64 * u < c;
        x[u] = have ? key(lane + 64 * u) : 0ull;
        in |= have ? 1u << u : 0u;
    }
#pragma unroll 1
    for (;;) {
        uint64_t lo = ~0ull, hi = 0ull;
#pragma unroll
        for (int u = 0; u < kWaveKeys; ++u)
            if (64 * u < c && (in >> u & 1u)) lo = umin(lo, x[u]), hi = umax(hi, x[u]);
        lo = wave_min(lo);
        hi = wave_max(hi);
        if (lo == hi) {
            K = lo;
            copies = left;
            return;
        }
        const uint64_t mid = lo + (hi - lo) / 2;
        uint32_t low = 0;
#pragma unroll
        for (int u = 0; u < kWaveKeys; ++u) low |= 64 * u < c && x[u] <= mid ? 1u << u : 0u;
        uint32_t n = uint32_t(__popc(in & low));
        n = wave_scan(n);
        const int64_t below = int64_t(uint32_t(__builtin_amdgcn_readlane(int(n), 63)));
        if (left <= below) in &= low;
        else in &= ~low, left -= below;
    }
}

// ------------------------------------------------------------------ one workgroup on its own
struct RefineLds {
    __attribute__((aligned(16))) uint32_t bins[kRiskBins];
    uint64_t lo[kRiskWaves], hi[kRiskWaves];
    RankState st;
};

// Smallest and largest of the workgroup's keys, in every thread.
__device__ __forceinline__ void wg_range(uint64_t &lo, uint64_t &hi, RefineLds &lds) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    lo = wave_min(lo);
    hi = wave_max(hi);
    if (lane == 0) lds.lo[wave] = lo, lds.hi[wave] = hi;
    __syncthreads();
    lo = wave_min(lds.lo[lane & (kRiskWaves - 1)]);
    hi = wave_max(lds.hi[lane & (kRiskWaves - 1)]);
}

// The left-th smallest of the keys in [lo, lo + span] that each() visits (every key of the
// workgroup once, each call): their range, bins of that range, the rank's bin, and so on;
// every round narrows the range at least 2048 times.  Whole workgroup.
template <typename Each>
__device__ __forceinline__ void refine(Each each, RankState s, uint64_t &K, int64_t &copies, RefineLds &lds) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#pragma unroll 1
    for (;;) {
        const uint64_t lo0 = s.lo, span = s.span;
        uint64_t lo = ~0ull, hi = 0ull;
        each([&](uint64_t k) {
            if (k - lo0 <= span) lo = umin(lo, k), hi = umax(hi, k);
        });
        __syncthreads();   // the previous round's (or caller's) use of lds is over
        for (int i = tid; i < kRiskBins; i += kRiskThreads) lds.bins[i] = 0u;
        wg_range(lo, hi, lds);
        if (lo >= hi) {   // one key value
            K = lo;
            copies = s.left;
            return;
        }
        const uint32_t width = bin_shift(hi - lo);
        each([&](uint64_t k) {
            if (k >= lo && k <= hi) atomicAdd(&lds.bins[(k - lo) >> width], 1u);
        });
        __syncthreads();
        if (wave == 0) {
            uint32_t total;
            RankState n = s;
            (void)wave_pick<kRiskBins / 64>(lds.bins, lo, width, s.left, n, total);
            n.span = range_end(n.lo, n.span, hi) - n.lo;
            if (lane == 0) lds.st = n;
        }
        __syncthreads();
        s = lds.st;
        if (s.span == 0) {   // one key per bin
            K = s.lo;
            copies = s.left;
            return;
        }
    }
}

// What to count for ranks up to k_max of y[0, n), from a sample of PER losses per thread
// (whole workgroup; lds.bins cleared on return).  Sample j is a loss of the j-th of as many
// equal stretches of the YLT, at a place within it that varies from stretch to stretch.
template <int PER>
struct Sampled {
    double loss[PER];
    bool have[PER];
};
template <int PER>
__device__ __forceinline__ Sampled<PER> sample_losses(const double *__restrict__ y, int64_t n) {
    Sampled<PER> s;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const uint32_t j = uint32_t(threadIdx.x) + uint32_t(u) * kRiskThreads;
        const int64_t a = int64_t(j) * n / (PER * kRiskThreads), e = int64_t(j + 1) * n / (PER * kRiskThreads);
        s.have[u] = e > a;
        s.loss[u] = 0.0;
        if (s.have[u]) s.loss[u] = y[a + __umulhi(j * 2654435761u, uint32_t(e - a))];
    }
    return s;
}
template <int PER>
__device__ __forceinline__ Binning sample_binning(const Sampled<PER> &own, int64_t n, int64_t k_max, RefineLds &lds) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint64_t key[PER];
    uint64_t lo = ~0ull, hi = 0ull;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        key[u] = own.have[u] ? desc_key(own.loss[u]) : ~0ull;
        lo = umin(lo, key[u]);
        if (own.have[u]) hi = umax(hi, key[u]);
    }
    for (int i = tid; i < kRiskBins; i += kRiskThreads) lds.bins[i] = 0u;
    // no negative loss sampled: zeros are taken to come last
    wg_range(lo, hi, lds);
    Binning b;
    b.lo = lo;
    b.zeros_last = hi <= kZeroKey && lo < kZeroKey ? 1u : 0u;
    const uint64_t last = b.zeros_last ? kZeroKey - 1ull : ~0ull;   // the bins' last key unless the sample ends them before
    __syncthreads();
    uint64_t top = 0ull, none = ~0ull;
#pragma unroll
    for (int u = 0; u < PER; ++u)
        if (own.have[u] && key[u] <= last) top = umax(top, key[u]);
    wg_range(none, top, lds);
    const int64_t ns = min(n, int64_t(PER * kRiskThreads));
    const double q = double(k_max) / double(n), at = q * double(ns);
    const int64_t place = int64_t(at + 5.0 * __builtin_sqrt(at * (1.0 - q)) + 6.0);
    const uint32_t width = top > lo ? bin_shift(top - lo) : 0u;
#pragma unroll
    for (int u = 0; u < PER; ++u)
        if (own.have[u] && key[u] <= top) atomicAdd(&lds.bins[(key[u] - lo) >> width], 1u);
    __syncthreads();
    if (wave == 0) {
        uint32_t total;
        RankState s;
        s.span = last;
        if (wave_pick<kRiskBins / 64>(lds.bins, lo, width, place, s, total)) s.span = range_end(s.lo, s.span, last);
        if (lane == 0) lds.st.span = s.span;
    }
    __syncthreads();
    b.hi = lds.st.span;
    // the bins cover the sampled keys; those past the last one sampled share the last bin
    const uint64_t end = b.hi == last ? umax(top, lo) : b.hi;
    b.shift = end > lo ? bin_shift(end - lo) : 0u;
    for (int i = tid; i < kRiskBins; i += kRiskThreads) lds.bins[i] = 0u;
    __syncthreads();
    return b;
}

// The losses from y[i0] (i0 wave-uniform) on as a buffer record, at most 2^28 of them:
// reads past the YLT's end give +0.0 without a branch.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t losses_from(const double *y, int64_t n, int64_t i0) {
    const int64_t left = max(int64_t(0), min(n - i0, int64_t(1) << 28));
    return __builtin_amdgcn_make_buffer_rsrc((void *)(y + (left ? i0 : 0)), 0, int(uint32_t(left) * 8u), kBufWord3);
}
__device__ __forceinline__ double loss_at(__amdgpu_buffer_rsrc_t r, uint32_t i) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, int(i * 8u), 0, 0));
}

// A workgroup's share of a YLT's keys, kRiskLoads per thread at a time: f(keys, which of
// them are losses of the YLT, a bit each).  The workgroup takes 1024 consecutive losses
// from `first` on, then from first + step on, ... (step at most 2^20).
template <typename F>
__device__ __forceinline__ void each_keys(const double *__restrict__ y, int64_t n, int64_t first, uint32_t step, F f) {
    const uint32_t tid = threadIdx.x;
#pragma unroll 1
    for (int64_t i0 = first; i0 < n; i0 += int64_t(step) * kRiskLoads) {
        const __amdgpu_buffer_rsrc_t r = losses_from(y, n, i0);
        const uint32_t left = uint32_t(min(n - i0, int64_t(1) << 28));
        double v[kRiskLoads];
#pragma unroll
        for (int u = 0; u < kRiskLoads; ++u) v[u] = loss_at(r, tid + u * step);
        uint64_t k[kRiskLoads];
        uint32_t in = 0;
#pragma unroll
        for (int u = 0; u < kRiskLoads; ++u) {
            k[u] = desc_key(v[u]);
            in |= tid + uint32_t(u) * step < left ? 1u << u : 0u;
        }
        f(k, in);
    }
}

// Counts the keys of f's calls: the bins in LDS, the other three as the wave's totals.
__device__ __forceinline__ void count_keys(const uint64_t (&k)[kRiskLoads], uint32_t in, const Binning &b, uint32_t *bins,
                                           Counts &n) {
#pragma unroll
    for (int u = 0; u < kRiskLoads; ++u) {
        const bool ok = (in >> u & 1u) != 0;
        if (ok && in_bins(b, k[u])) atomicAdd(&bins[bin_of(b, k[u])], 1u);
        n.below += uint32_t(__popcll(__ballot(ok && k[u] < b.lo)));
        n.equal += uint32_t(__popcll(__ballot(ok && k[u] == b.lo)));
        n.zero += uint32_t(__popcll(__ballot(ok && b.zeros_last && k[u] == kZeroKey)));
    }
}
__device__ __forceinline__ void add_counts(const Counts &n, Counts *to) {   // lane 0 of each wave
    if ((threadIdx.x & 63) != 0) return;
    if (n.below) atomicAdd(&to->below, n.below);
    if (n.equal) atomicAdd(&to->equal, n.equal);
    if (n.zero) atomicAdd(&to->zero, n.zero);
}

// Bins of up to kRiskCollect keys together: where each rank's lie among the copied keys
// (ranks of one bin share the first one's), at off[kRiskGroup] the number of copied keys, and in
// *large a bit for the first rank of each larger bin, which is not copied.  st[0, m) set; first
// (-1: solved), off and *large written; whole workgroup, with barriers on both sides.
__device__ __forceinline__ void place_bins(const RankState *st, int m, int wave, int *first, uint32_t *off, uint32_t *large) {
    const int lane = threadIdx.x & 63;
    if (wave < m) {
        const int f = st[wave].solved ? -1 : first_of_bin(st, wave);
        if (lane == 0) first[wave] = f;
    }
    __syncthreads();
    if (wave == 0) {
        const bool own = lane < m && first[lane] == lane, copied = own && st[lane].count <= uint32_t(kRiskCollect);
        const uint32_t c = copied ? st[lane].count : 0u;
        const uint32_t inc = wave_scan(c);
        const uint64_t rest = __ballot(own && !copied);
        if (lane < m) off[lane] = inc - c;
        if (lane == 63) off[kRiskGroup] = inc, *large = uint32_t(rest);
    }
    __syncthreads();
}

// Copies the keys of each rank's bin (the first ranks' of them), a whole wave together:
// reserve(r, c) by one lane gives the wave room for its c keys of rank r, put(r, place, key)
// stores one.  One returning atomic per rank, not one per key register (with wave_pick's banks
// k_risk_collect went from 15 to 14.3 us for the largest occurrences of 10^5 trials).
template <typename Reserve, typename Put>
__device__ __forceinline__ void copy_bins(const uint64_t (&k)[kRiskLoads], uint32_t in, const RankState *st,
                                          const int *first, int m, Reserve reserve, Put put) {
    const int lane = threadIdx.x & 63;
#pragma unroll 1
    for (int r = 0; r < m; ++r) {
        if (first[r] != r || st[r].count > uint32_t(kRiskCollect)) continue;
        const uint64_t lo = st[r].lo, span = st[r].span;
        uint32_t hit = 0, c = 0;
#pragma unroll
        for (int u = 0; u < kRiskLoads; ++u) {
            const bool h = (in >> u & 1u) && k[u] - lo <= span;
            hit |= h ? 1u << u : 0u;
            c += uint32_t(__popcll(__ballot(h)));
        }
        if (c == 0) continue;
        uint32_t at = 0;
        if (lane == 0) at = reserve(r, c);
        at = uint32_t(__builtin_amdgcn_readfirstlane(int(at)));
#pragma unroll
        for (int u = 0; u < kRiskLoads; ++u) {
            const bool h = (hit >> u & 1u) != 0;
            const uint64_t all = __ballot(h);
            if (h) put(r, at + __builtin_amdgcn_mbcnt_hi(uint32_t(all >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(all), 0u)), k[u]);
            at += uint32_t(__popcll(all));
        }
    }
}

// The same where the bins' counts are in LDS: a bin marked kTaken holds the place of its next
// key, so that a key takes one lookup however many ranks there are.  (With a pass over the keys
// per rank the copying took 4.3 of k_risk_one's 21.3 us for 10,000 losses of 74 values, now 1.9
// of 18.6.)
constexpr uint32_t kTaken = 0x80000000u;
template <typename Put>
__device__ __forceinline__ void copy_taken(const uint64_t (&k)[kRiskLoads], uint32_t in, const Binning &b, uint32_t *bins,
                                           uint32_t *to_below, Put put) {
    uint32_t at[kRiskLoads], to[kRiskLoads];
#pragma unroll
    for (int u = 0; u < kRiskLoads; ++u) {
        at[u] = in_bins(b, k[u]) ? bin_of(b, k[u]) : 0u;
        to[u] = bins[at[u]];
    }
    if (*to_below & kTaken) {
#pragma unroll
        for (int u = 0; u < kRiskLoads; ++u)
            if ((in >> u & 1u) && k[u] < b.lo) put(atomicAdd(to_below, 1u) & ~kTaken, k[u]);
    }
    uint32_t hit = 0;
#pragma unroll
    for (int u = 0; u < kRiskLoads; ++u) hit |= (to[u] & kTaken) && in_bins(b, k[u]) ? 1u << u : 0u;
    hit &= in;
    if (hit == 0u) return;
#pragma unroll
    for (int u = 0; u < kRiskLoads; ++u)   // all on their way before the first is waited for
        if (hit >> u & 1u) to[u] = atomicAdd(&bins[at[u]], 1u);
#pragma unroll
    for (int u = 0; u < kRiskLoads; ++u)
        if (hit >> u & 1u) put(to[u] & ~kTaken, k[u]);
}

// Lane t + o into lane t, o = 32, 16, ..., 1; the result in lane 0.
template <int Ctrl>
__device__ __forceinline__ double add_row_shl(double x) {
    return x + __builtin_bit_cast(double, dpp64<Ctrl>(__builtin_bit_cast(uint64_t, x)));
}
__device__ __forceinline__ double wave_tree(double x) {
    x += __shfl_down(x, 32, 64);
    x += __shfl_down(x, 16, 64);
    x = add_row_shl<0x108>(x);
    x = add_row_shl<0x104>(x);
    x = add_row_shl<0x102>(x);
    return add_row_shl<0x101>(x);
}

// A quarter of a tile: the losses of the tile's slots 64 q .. 64 q + 63, a slot per lane.
// (A wave per tile had four times the losses and formed their keys again for each rank:
// the sums of 50,000 losses took 9.4 us, now 6.2, of 10^6 10.5 and 8.1.)
struct Quarter {
    double v[8];
    uint64_t key[8];
};
__device__ __forceinline__ void quarter_losses(const double *__restrict__ y, int64_t n, int64_t tile, int q, Quarter &x) {
    const __amdgpu_buffer_rsrc_t rs = losses_from(y, n, tile * kRiskTile);
#pragma unroll
    for (int u = 0; u < 8; ++u) x.v[u] = loss_at(rs, uint32_t(threadIdx.x & 63) + 64u * uint32_t(q) + 256u * uint32_t(u));
}
__device__ __forceinline__ void quarter_keys(Quarter &x) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        x.v[u] += 0.0;
        x.key[u] = desc_key(x.v[u]);
    }
}
// Which of them are losses of the YLT, a bit each.
__device__ __forceinline__ uint32_t quarter_in(int64_t n, int64_t tile, int q) {
    const int64_t left = n - tile * kRiskTile - 64 * q - (threadIdx.x & 63);   // slot's losses: every 256th of these
    const int64_t c = (left + 255) >> 8;
    return c >= 8 ? 0xFFu : c <= 0 ? 0u : (1u << int(c)) - 1u;
}
// The slot's sum of the losses below K.
__device__ __forceinline__ double quarter_sum(const Quarter &x, uint64_t K) {
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) s += x.key[u] < K ? x.v[u] : 0.0;
    return s;
}
// The tree over a tile's 256 slots (quarter q's at s + 64 q) by one wave: slot t + o into
// slot t, o = 128, 64, ..., 1; the result in lane 0.
__device__ __forceinline__ double tile_tree(const double *s) {
    const int lane = threadIdx.x & 63;
    return wave_tree((s[lane] + s[128 + lane]) + (s[64 + lane] + s[192 + lane]));
}
constexpr int kSumRanks = 4;   // ranks whose slots are in LDS together

// The tile sums of one rank in the same order (slot t adds tiles t, t + 256, ...), by one
// wave; the result in lane 0.  Eight of a lane's loads are in flight together.
template <typename At>
__device__ __forceinline__ double wave_sum_tiles(int64_t tiles, At at) {
    const int lane = threadIdx.x & 63;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
    for (int64_t t0 = lane; t0 - lane < tiles; t0 += 512) {
        double v[2][4];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t t = t0 + 256 * i + 64 * q;
                v[i][q] = t < tiles ? at(t) : 0.0;
            }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) s[q] += v[i][q];
    }
    return wave_tree((s[0] + s[2]) + (s[1] + s[3]));
}

__device__ __forceinline__ void write_measures(double *out, int m, int r, uint64_t K, int64_t copies, double s, int64_t k) {
    const double pml = key_value(K);
    out[r] = pml;
    out[m + r] = (s + double(copies) * pml) / double(k);
}

// A YLT of at most kRiskOneWg losses per workgroup (blockIdx.x), in its registers from the
// start: quarter tiles wave and wave + 16, for the bins, the few keys of each rank's bin and
// the tile sums.  Its instructions bound it: 16 losses per lane, four waves per SIMD (of 20 us
// forming the keys and counting them take 3, sampling 5.6 with its round trips).  Reading the
// YLT anew for each of the three it took 16.9 us for 10,000 losses, now 13.7, and 12.8 and 11.2
// for 1000.
constexpr int kOneTiles = kRiskOneWg / kRiskTile;
__global__ __launch_bounds__(kRiskThreads) void k_risk_one(RiskArgs a) {
    __shared__ RefineLds ref;
    __shared__ Counts cnt;
    __shared__ RankState st[64];
    __shared__ int first[kRiskGroup];
    __shared__ uint32_t off[kRiskGroup + 1], large, to_below;
    __shared__ uint64_t K[kRiskGroup];
    __shared__ uint64_t cand[kRiskCollect];
    __shared__ double tile_s[kRiskGroup][kOneTiles];
    const JobView j = job_view(a, blockIdx.x);
    const double *y = j.y;
    const int64_t n = j.n;
    const int m = j.m;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid == 0) cnt = Counts{0u, 0u, 0u}, to_below = 0u;
    const int nt = int(risk_tiles(n)), i0 = wave, i1 = wave + kRiskWaves;
    static_assert(4 * kOneTiles <= 2 * kRiskWaves, "two quarters per wave");
    const Sampled<1> own = sample_losses<1>(y, n);
    Quarter x0, x1;   // past the last tile: zeros
    quarter_losses(y, n, i0 >> 2, i0 & 3, x0);
    quarter_losses(y, n, i1 >> 2, i1 & 3, x1);
    const Binning b = sample_binning(own, n, j.k_max, ref);
    quarter_keys(x0);
    quarter_keys(x1);
    Counts c{0u, 0u, 0u};
    const uint32_t in0 = quarter_in(n, i0 >> 2, i0 & 3), in1 = quarter_in(n, i1 >> 2, i1 & 3);
    if (i0 < 4 * nt) count_keys(x0.key, in0, b, ref.bins, c);
    if (i1 < 4 * nt) count_keys(x1.key, in1, b, ref.bins, c);
    add_counts(c, &cnt);
    __syncthreads();
    if (wave < m) {   // wave r picks rank r's bin
        bool past;
        RankState s = pick_bin(ref.bins, b, cnt, job_rank(a, blockIdx.x, wave), n, past);
        if (past) s.count = ~0u;   // their bins have no place for copies
        if (lane == 0) st[wave] = s;
    }
    __syncthreads();
    place_bins(st, m, wave, first, off, &large);
    const bool fits = off[kRiskGroup] <= uint32_t(kRiskCollect);   // the copied keys fit in LDS
    if (fits && off[kRiskGroup] > 0u) {
        // the count of a rank's bin becomes where its next key goes (the keys below b.lo: to_below)
        if (tid < m && first[tid] == tid && st[tid].count <= uint32_t(kRiskCollect)) {
            const uint64_t at = st[tid].lo;
            (at < b.lo ? to_below : ref.bins[bin_of(b, at)]) = kTaken | off[tid];
        }
        __syncthreads();
        auto put = [&](uint32_t i, uint64_t k) { cand[i] = k; };
        if (i0 < 4 * nt) copy_taken(x0.key, in0, b, ref.bins, &to_below, put);
        if (i1 < 4 * nt) copy_taken(x1.key, in1, b, ref.bins, &to_below, put);
    }
    __syncthreads();
    if (wave < m && lane == 0) K[wave] = st[wave].K;
    if (fits && wave < m && !st[wave].solved && st[wave].count <= kFewKeys) {
        const int nc = int(st[wave].count);
        uint64_t x;
        int64_t copies;
        const uint64_t *from = cand + off[first[wave]];
        wave_select_any(nc, st[wave].left, x, copies, [&](int i) { return from[i]; });
        if (lane == 0) K[wave] = x, st[wave].copies = copies, st[wave].solved = true;
    }
    __syncthreads();
    const uint64_t open = __ballot(lane < m && !st[lane].solved);
#pragma unroll 1
    for (int q = 0; __builtin_expect(open >> q != 0, 0); ++q) {   // larger bins, one after another
        if (!(open >> q & 1)) continue;
        uint64_t x;
        int64_t copies;
        if (fits && st[q].count <= uint32_t(kRiskCollect)) {
            const uint64_t *from = cand + off[first[q]];
            const int nc = int(st[q].count);
            refine([&](auto f) { for (int i = tid; i < nc; i += kRiskThreads) f(from[i]); }, st[q], x, copies, ref);
        } else {
            refine([&](auto f) { for (int64_t i = tid; i < n; i += kRiskThreads) f(desc_key(y[i])); }, st[q], x, copies, ref);
        }
        __syncthreads();
        if (tid == 0) K[q] = x, st[q].copies = copies;
    }
    __syncthreads();
    // the quarters' slots go where the candidates were
    static_assert(kSumRanks * 4 * kOneTiles * 64 <= kRiskCollect, "slots");
    double *slots = reinterpret_cast<double *>(cand);   // [rank][tile][256]
#pragma unroll 1
    for (int r0 = 0; r0 < m; r0 += kSumRanks) {
#pragma unroll 1
        for (int r = r0; r < min(r0 + kSumRanks, m); ++r) {
            double *to = slots + ((r - r0) * kOneTiles) * 256 + lane;
            if (i0 < 4 * nt) to[64 * i0] = quarter_sum(x0, K[r]);
            if (i1 < 4 * nt) to[64 * i1] = quarter_sum(x1, K[r]);
        }
        __syncthreads();
#pragma unroll 1
        for (int i = wave; i < kSumRanks * nt; i += kRiskWaves) {
            const int r = r0 + (i & (kSumRanks - 1)), t = i / kSumRanks;
            if (r >= m) continue;
            const double s = tile_tree(slots + ((r - r0) * kOneTiles + t) * 256);
            if (lane == 0) tile_s[r][t] = s;
        }
        __syncthreads();
    }
    if (wave < m) {
        const double s = wave_sum_tiles(nt, [&](int64_t t) { return tile_s[wave][t]; });
        if (lane == 0) write_measures(j.out, m, wave, K[wave], st[wave].copies, s, job_rank(a, blockIdx.x, wave));
    }
    if (tid == 0 && a.err_out) *a.err_out = *a.err;
}

// ------------------------------------------------------------------ longer YLTs
// Workspace of one YLT and group of ranks (risk_workspace_bytes), 256-byte aligned.
enum : uint32_t { kRiskDone = 0, kRiskOpen = 1, kRiskPicked = 2 };   // picked: every K is known, not the sums
struct RiskWs {
    uint32_t *done;      // [2]: workgroups that finished k_risk_collect, k_risk_sum
    uint32_t *open;      // kRiskDone ...
    uint32_t *ranges;    // of an open YLT: a bit for the first rank of each range to narrow
    Counts *counts;
    Binning *binning;
    uint32_t *n_cand;    // [kRiskGroup] keys copied out per bin
    uint64_t *b_lo, *b_hi;   // [2][kRiskGroup] smallest and largest key of a range too large to copy out:
                             // of k_risk_collect's round r in the half r & 1
    uint64_t *K;         // [kRiskGroup]
    int64_t *copies;     // [kRiskGroup]
    RankState *state;    // [kRiskGroup], of an open YLT
    uint32_t *bins;      // [kRiskBins]
    uint32_t *narrow;    // [kNarrowBins], of the ranges too large to copy out, one after another
    double *tile_sum;    // [m][tiles]
    uint64_t *cand;      // the copied bins, one after another: at most min(n, m kRiskCollect) keys
};

__host__ __device__ inline size_t risk_align(size_t x) { return (x + 255) & ~size_t(255); }
__host__ __device__ inline int risk_blocks(int64_t n) {
    const int64_t b = (n + kRiskRow - 1) / kRiskRow;
    return int(b < kRiskBlocks ? b : kRiskBlocks);
}
constexpr size_t kRiskCtrlBytes = 2048;

__device__ __forceinline__ RiskWs risk_ws(const JobView &j) {
    RiskWs w;
    unsigned char *p = j.ws;
    w.done = reinterpret_cast<uint32_t *>(p);
    w.open = w.done + 2;
    w.ranges = w.done + 3;
    w.counts = reinterpret_cast<Counts *>(p + 16);
    w.binning = reinterpret_cast<Binning *>(p + 32);
    w.n_cand = reinterpret_cast<uint32_t *>(p + 64);
    w.b_lo = reinterpret_cast<uint64_t *>(p + 128);
    w.b_hi = w.b_lo + 2 * kRiskGroup;
    w.K = w.b_hi + 2 * kRiskGroup;
    w.copies = reinterpret_cast<int64_t *>(w.K + kRiskGroup);
    w.state = reinterpret_cast<RankState *>(w.copies + kRiskGroup);
    static_assert(sizeof(Counts) <= 16 && sizeof(Binning) <= 32 && 4 * kRiskGroup <= 64 &&
                  128 + kRiskGroup * (6 * 8 + sizeof(RankState)) <= kRiskCtrlBytes, "control block");
    p += kRiskCtrlBytes;
    w.bins = reinterpret_cast<uint32_t *>(p);
    p += kRiskBins * 4;
    w.narrow = reinterpret_cast<uint32_t *>(p);
    p += kNarrowBins * 4;
    w.tile_sum = reinterpret_cast<double *>(p);
    p += risk_align(size_t(j.m) * size_t(risk_tiles(j.n)) * 8);
    w.cand = reinterpret_cast<uint64_t *>(p);
    return w;
}

size_t risk_workspace_bytes(int64_t n, int m) {
    if (n <= kRiskOneWg) return 0;
    return kRiskCtrlBytes + size_t(kRiskBins + kNarrowBins) * 4 +
           risk_align(size_t(m) * size_t(risk_tiles(n)) * 8) +
           risk_align(size_t(std::min<int64_t>(n, int64_t(m) * kRiskCollect)) * 8);
}

// log2 of the bins of each of n ranges in k_risk_narrow.
__device__ __forceinline__ int narrow_log(int n) { return n <= 4 ? 12 : n <= 8 ? 11 : 10; }
static_assert(4 << 12 <= kNarrowBins && 8 << 11 <= kNarrowBins && kRiskGroup << 10 <= kNarrowBins, "bins of all ranges");

template <typename F>
__device__ __forceinline__ void each_keys_of_grid(const JobView &j, int nb, F f) {
    each_keys(j.y, j.n, int64_t(blockIdx.x) * kRiskThreads, uint32_t(nb) * kRiskThreads, f);
}

// The binning from the sample; clears the counts.  The keys below the smallest one sampled are
// a range of their own, of n / (1024 PER) keys or so, which a rank of a long return period
// lies in: with one loss per thread it is too large to copy out from about 5 10^6 losses on.
constexpr int64_t kRiskSampleMore = int64_t(1) << 22;   // longer YLTs: PER = 4
template <int PER>
__global__ __launch_bounds__(kRiskThreads) void k_risk_sample(RiskArgs a) {
    __shared__ RefineLds ref;
    const JobView j = job_view(a, blockIdx.x);
    if ((j.n > kRiskSampleMore) != (PER > 1)) return;
    const RiskWs w = risk_ws(j);
    const int tid = threadIdx.x;
    for (int i = tid; i < kRiskBins; i += kRiskThreads) w.bins[i] = 0u;
    if (tid < 2) w.done[tid] = 0u;
    if (tid < kRiskGroup) w.n_cand[tid] = 0u, w.b_lo[tid] = ~0ull, w.b_hi[tid] = 0ull;
    const Binning b = sample_binning(sample_losses<PER>(j.y, j.n), j.n, j.k_max, ref);
    if (tid == 0) {
        *w.counts = Counts{0u, 0u, 0u};
        *w.binning = b;
    }
}

__global__ __launch_bounds__(kRiskThreads) void k_risk_bins(RiskArgs a) {
    __shared__ uint32_t bins[kRiskBins];
    __shared__ Counts cnt;
    const JobView j = job_view(a, blockIdx.y);
    const int nb = min(risk_blocks(j.n), int(gridDim.x));
    if (int(blockIdx.x) >= nb) return;
    const RiskWs w = risk_ws(j);
    const int tid = threadIdx.x;
    for (int i = tid; i < kRiskBins; i += kRiskThreads) bins[i] = 0u;
    if (tid == 0) cnt = Counts{0u, 0u, 0u};
    const Binning b = *w.binning;
    __syncthreads();
    Counts c{0u, 0u, 0u};
    each_keys_of_grid(j, nb, [&](const uint64_t (&k)[kRiskLoads], uint32_t in) { count_keys(k, in, b, bins, c); });
    add_counts(c, &cnt);
    __syncthreads();
    // one addition per workgroup: one per wave, all on the same three words, took 20 us
    if (tid == 0) add_counts(cnt, w.counts);
    for (int i = tid; i < kRiskBins; i += kRiskThreads)
        if (bins[i]) atomicAdd(&w.bins[i], bins[i]);
}

// The keys of each open rank's range, copied out; the last workgroup picks each rank's K
// among them.  Of a range of more than kRiskCollect keys the smallest and largest are kept
// instead: equal for a loss that occurs that often, else the YLT stays open.  FIRST: the
// ranges are bins that k_risk_bins counted, in later rounds k_risk_narrow's.  (One kernel for
// both took 22 us for 10^6 losses, this 14.)
constexpr int kRangesAtOnce = 4;   // large ranges per pass over the keys
template <bool FIRST>
__global__ __launch_bounds__(kRiskThreads) void k_risk_collect(RiskArgs a) {
    __shared__ RefineLds ref;
    __shared__ RankState st[64];
    __shared__ int first[kRiskGroup];
    __shared__ uint32_t off[kRiskGroup + 1], large;
    __shared__ uint32_t last;
    __shared__ uint64_t ends[2][kRangesAtOnce][kRiskWaves];
    const JobView j = job_view(a, blockIdx.y);
    const int nb = min(risk_blocks(j.n), int(gridDim.x)), m = j.m, half = FIRST ? 0 : a.round & 1;
    if (int(blockIdx.x) >= nb) return;
    const RiskWs w = risk_ws(j);
    if (!FIRST && *w.open != kRiskOpen) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    RankState s;
    if (FIRST) {
        bool past;
        if (wave < m) s = pick_bin(w.bins, *w.binning, *w.counts, job_rank(a, blockIdx.y, wave), j.n, past);
    } else {
        if (tid < m) st[tid] = w.state[tid];
        __syncthreads();
        if (wave < m) {
            s = st[wave];
            if (!s.solved) {
                const int f = first_of_bin(st, wave), at = (half ^ 1) * kRiskGroup + f;
                const uint64_t lo = w.b_lo[at], hi = w.b_hi[at];
                const int log = narrow_log(__popc(*w.ranges));
                const uint32_t *row = w.narrow + (__popc(*w.ranges & ((1u << f) - 1u)) << log), width = bin_shift(hi - lo, log);
                uint32_t total;
                if (log == 12) (void)wave_pick<64>(row, lo, width, s.left, s, total);
                else if (log == 11) (void)wave_pick<32>(row, lo, width, s.left, s, total);
                else (void)wave_pick<16>(row, lo, width, s.left, s, total);
                s.span = range_end(s.lo, s.span, hi) - s.lo;
            }
        }
        __syncthreads();
    }
    if (wave < m && lane == 0) st[wave] = s;
    __syncthreads();
    place_bins(st, m, wave, first, off, &large);
    if (off[kRiskGroup] > 0u)
        each_keys_of_grid(j, nb, [&](const uint64_t (&k)[kRiskLoads], uint32_t in) {
            copy_bins(k, in, st, first, m, [&](int r, uint32_t c) { return atomicAdd(&w.n_cand[r], c); },
                      [&](int r, uint32_t i, uint64_t x) { agent_store(&w.cand[off[r] + i], x); });
        });
#pragma unroll 1
    for (uint32_t left = large; __builtin_expect(left != 0u, 0);) {
        int r[kRangesAtOnce];   // -1: none
        uint64_t lo[kRangesAtOnce], span[kRangesAtOnce], mn[kRangesAtOnce], mx[kRangesAtOnce];
#pragma unroll
        for (int q = 0; q < kRangesAtOnce; ++q) {
            r[q] = left ? __builtin_ctz(left) : -1;
            left &= left - 1u;
            lo[q] = st[max(r[q], 0)].lo, span[q] = st[max(r[q], 0)].span, mn[q] = ~0ull, mx[q] = 0ull;
        }
        each_keys_of_grid(j, nb, [&](const uint64_t (&k)[kRiskLoads], uint32_t in) {
#pragma unroll
            for (int q = 0; q < kRangesAtOnce; ++q) {
                if (r[q] < 0) continue;
#pragma unroll
                for (int u = 0; u < kRiskLoads; ++u)
                    if ((in >> u & 1u) && k[u] - lo[q] <= span[q]) mn[q] = umin(mn[q], k[u]), mx[q] = umax(mx[q], k[u]);
            }
        });
        // one addition per workgroup: one per wave, all on the same two words, took 20 us
#pragma unroll
        for (int q = 0; q < kRangesAtOnce; ++q) {
            if (r[q] < 0) continue;
            mn[q] = wave_min(mn[q]);
            mx[q] = wave_max(mx[q]);
            if (lane == 0) ends[0][q][wave] = mn[q], ends[1][q][wave] = mx[q];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kRangesAtOnce; ++q) {
            if (r[q] < 0 || wave != q) continue;
            const uint64_t l = wave_min(ends[0][q][lane & (kRiskWaves - 1)]), h = wave_max(ends[1][q][lane & (kRiskWaves - 1)]);
            if (lane == 0 && l <= h) {
                const int at = half * kRiskGroup + r[q];
                atomicMin(reinterpret_cast<unsigned long long *>(&w.b_lo[at]), static_cast<unsigned long long>(l));
                atomicMax(reinterpret_cast<unsigned long long *>(&w.b_hi[at]), static_cast<unsigned long long>(h));
            }
        }
        __syncthreads();
    }
    if (!last_to_finish(&w.done[0], uint32_t(nb), &last)) return;
    if (wave < m) {
        const int f = first[wave];
        if (!s.solved && s.count <= kFewKeys) {
            const uint64_t *from = w.cand + off[f];
            wave_select_any(int(s.count), s.left, s.K, s.copies, [&](int i) { return agent_load(&from[i]); });
            s.solved = true;
        } else if (!s.solved && s.count > uint32_t(kRiskCollect)) {
            const int at = half * kRiskGroup + f;
            const uint64_t lo = agent_load(&w.b_lo[at]), hi = agent_load(&w.b_hi[at]);
            if (lo == hi) s.K = lo, s.copies = s.left, s.solved = true;
        }
        if (lane == 0) st[wave] = s;
    }
    __syncthreads();
    const uint64_t unsolved = __ballot(lane < m && !st[lane].solved);
    uint64_t open = 0;
#pragma unroll 1
    for (int r = 0; __builtin_expect(unsolved >> r != 0, 0); ++r) {
        if (!(unsolved >> r & 1)) continue;
        if (st[r].count > uint32_t(kRiskCollect)) {
            open |= 1ull << r;
            continue;
        }
        uint64_t K;
        int64_t copies;
        const uint64_t *c = w.cand + off[first[r]];
        const int nc = int(st[r].count);
        refine([&](auto f) { for (int i = tid; i < nc; i += kRiskThreads) f(agent_load(&c[i])); }, st[r], K, copies, ref);
        __syncthreads();
        if (tid == 0) st[r].K = K, st[r].copies = copies, st[r].solved = true;
    }
    __syncthreads();
    if (tid < m) {
        w.K[tid] = st[tid].K;
        w.copies[tid] = st[tid].copies;
    }
    if (tid == 0) *w.open = open ? kRiskOpen : kRiskPicked;
    if (__builtin_expect(open == 0, 1)) return;
    // for the next round
    if (tid < m) w.state[tid] = st[tid];
    for (int i = tid; i < kNarrowBins; i += kRiskThreads) w.narrow[i] = 0u;
    if (tid == 0) w.done[0] = 0u, *w.ranges = large & uint32_t(open);
    if (tid < kRiskGroup) {
        w.n_cand[tid] = 0u;
        w.b_lo[(half ^ 1) * kRiskGroup + tid] = ~0ull, w.b_hi[(half ^ 1) * kRiskGroup + tid] = 0ull;
    }
}

// Counts the keys of the open ranks' ranges, each in 2^narrow_log bins from its smallest key to
// its largest (one addition where a wave's keys fall in one bin: a loss that many years share
// would otherwise be added one after another).
__global__ __launch_bounds__(kRiskThreads) void k_risk_narrow(RiskArgs a) {
    __shared__ uint32_t bins[kNarrowBins];
    const JobView j = job_view(a, blockIdx.y);
    const int nb = min(risk_blocks(j.n), int(gridDim.x));
    if (int(blockIdx.x) >= nb) return;
    const RiskWs w = risk_ws(j);
    if (*w.open != kRiskOpen) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t ranges = *w.ranges;
    const int log = narrow_log(__popc(ranges)), n_bins = __popc(ranges) << log;
    for (int i = tid; i < n_bins; i += kRiskThreads) bins[i] = 0u;
    __syncthreads();
    const uint64_t *b_lo = w.b_lo + ((a.round & 1) ^ 1) * kRiskGroup, *b_hi = w.b_hi + ((a.round & 1) ^ 1) * kRiskGroup;
    int done = 0;
#pragma unroll 1
    for (uint32_t left = ranges; left != 0u; done += kRangesAtOnce) {
        int r[kRangesAtOnce];
        uint64_t lo[kRangesAtOnce], span[kRangesAtOnce];
        uint32_t width[kRangesAtOnce];
#pragma unroll
        for (int q = 0; q < kRangesAtOnce; ++q) {
            r[q] = left ? __builtin_ctz(left) : -1;
            left &= left - 1u;
            lo[q] = b_lo[max(r[q], 0)], span[q] = b_hi[max(r[q], 0)] - lo[q];
            width[q] = r[q] < 0 ? 0u : bin_shift(span[q], log);
        }
        each_keys_of_grid(j, nb, [&](const uint64_t (&k)[kRiskLoads], uint32_t in) {
#pragma unroll
            for (int q = 0; q < kRangesAtOnce; ++q) {
                if (r[q] < 0) continue;
                uint32_t *row = bins + ((done + q) << log);
#pragma unroll
                for (int u = 0; u < kRiskLoads; ++u) {
                    const bool own = (in >> u & 1u) && k[u] - lo[q] <= span[q];
                    const uint64_t all = __ballot(own);
                    if (all == 0) continue;
                    const uint32_t at = own ? uint32_t((k[u] - lo[q]) >> width[q]) : 0u;
                    const int lead = __ffsll(static_cast<unsigned long long>(all)) - 1;
                    const uint32_t at0 = uint32_t(__builtin_amdgcn_readlane(int(at), lead));
                    if (__ballot(own && at != at0) == 0) {
                        if (lane == lead) atomicAdd(&row[at], uint32_t(__popcll(all)));
                    } else if (own) {
                        atomicAdd(&row[at], 1u);
                    }
                }
            }
        });
    }
    __syncthreads();
    for (int i = tid; i < n_bins; i += kRiskThreads)
        if (bins[i]) atomicAdd(&w.narrow[i], bins[i]);
}

// Each tile's sum of the losses below each rank's K, four waves per tile; the last
// workgroup adds the tile sums up.  (Four tiles per workgroup: with one, the workgroups'
// counting themselves, one atomic each on one word, took 7 us of the 13 us for 489 tiles.)
constexpr int kSumTiles = 4;
constexpr int kSumWaves = 4 * kSumTiles;
__global__ __launch_bounds__(kSumWaves * 64) void k_risk_sum(RiskArgs a) {
    __shared__ double slots[kSumRanks][kSumTiles][256];
    __shared__ uint32_t last;
    const JobView j = job_view(a, blockIdx.y);
    const int64_t tiles = risk_tiles(j.n), wgs = (tiles + kSumTiles - 1) / kSumTiles;
    if (int64_t(blockIdx.x) >= wgs) return;
    const RiskWs w = risk_ws(j);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), m = j.m;
    const int t = wave >> 2, q = wave & 3;
    const int64_t tile = int64_t(blockIdx.x) * kSumTiles + t;
    Quarter x;
    quarter_losses(j.y, j.n, tile, q, x);   // past the last tile: zeros
    if (const uint32_t open = *w.open; open != kRiskPicked) {   // summed in an earlier round, or open
        if (open == kRiskOpen && blockIdx.x == 0 && tid == 0) {
            *a.open_out = 1u;
            if (a.err_out) *a.err_out = *a.err;
        }
        return;
    }
    quarter_keys(x);
#pragma unroll 1
    for (int r0 = 0; r0 < m; r0 += kSumRanks) {
#pragma unroll 1
        for (int r = r0; r < min(r0 + kSumRanks, m); ++r) slots[r - r0][t][64 * q + lane] = quarter_sum(x, w.K[r]);
        __syncthreads();
        if (r0 + q < m && tile < tiles) {
            const double s = tile_tree(slots[q][t]);
            if (lane == 0) agent_store(&w.tile_sum[(r0 + q) * tiles + tile], s);
        }
        __syncthreads();
    }
    if (!last_to_finish(&w.done[1], uint32_t(wgs), &last)) return;
#pragma unroll 1
    for (int r = wave; r < m; r += kSumWaves) {
        const double s = wave_sum_tiles(tiles, [&](int64_t t) { return agent_load(&w.tile_sum[r * tiles + t]); });
        if (lane == 0) write_measures(j.out, m, r, w.K[r], w.copies[r], s, job_rank(a, blockIdx.y, r));
    }
    if (tid != 0) return;
    *w.open = kRiskDone;
    if (a.err_out) *a.err_out = *a.err;
}

// Workgroups per YLT of a pass over several: no more together than are resident at once, where
// that can be had, since each has a fixed part (clearing and adding its bins; in the collection,
// picking the ranks' bins and being counted) however few losses it takes.  A workgroup of
// k_risk_bins leaves room for another on its CU, one of k_risk_collect does not.  15 YLTs of
// 10^5 to 10^6 losses with 128 workgroups each: bins 32 us, collection 65; now 25 and 39.
constexpr int kResidentBins = 512, kResidentCollect = 256;
static int blocks_each(const RiskJob *jobs, int n_jobs, int resident) {
    auto total = [&](int most) {
        int64_t t = 0;
        for (int i = 0; i < n_jobs; ++i) t += std::min(risk_blocks(jobs[i].n), most);
        return t;
    };
    if (total(kRiskBlocks) <= resident) return kRiskBlocks;
    int fits = 1, over = kRiskBlocks;   // total(over) > resident
    while (over - fits > 1) {
        const int mid = (fits + over) / 2;
        (total(mid) <= resident ? fits : over) = mid;
    }
    return fits;
}

// Grids of the passes over jobs[0, n): (workgroups of the counting, of the collection, of the
// sums) per YLT.
struct RiskGrids {
    dim3 bins, collect, sum;
};
static hipError_t risk_grids(const RiskJob *jobs, int n_long, RiskGrids &g) {
    int64_t n = 0;
    for (int i = 0; i < n_long; ++i) n = std::max(n, jobs[i].n);
    const int64_t tiles = risk_tiles(n);
    if (tiles > int64_t(INT32_MAX) || n_long > 65535) return hipErrorInvalidValue;
    g.bins = dim3(unsigned(std::min(risk_blocks(n), blocks_each(jobs, n_long, kResidentBins))), unsigned(n_long));
    g.collect = dim3(unsigned(std::min(risk_blocks(n), blocks_each(jobs, n_long, kResidentCollect))), unsigned(n_long));
    g.sum = dim3(unsigned((tiles + kSumTiles - 1) / kSumTiles), unsigned(n_long));
    return hipSuccess;
}

static RiskArgs risk_args(const RiskJob *host, const RiskJob *dev, const RiskOut &out, int round) {
    RiskArgs a{};
    a.jobs = dev;
    if (!dev) a.one = host[0];
    a.err = out.err;
    a.err_out = out.err_out;
    a.open_out = out.open_out;
    a.round = round;
    return a;
}

hipError_t launch_risk(const RiskJob *host, const RiskJob *dev, int n_short, int n_long, const RiskOut &out, hipStream_t s) {
    const dim3 block(kRiskThreads);
    if (n_short > 0) {
        hipLaunchKernelGGL(k_risk_one, dim3(unsigned(n_short)), block, 0, s, risk_args(host, dev, out, 0));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (n_long <= 0) return hipSuccess;
    host += n_short;
    const RiskArgs a = risk_args(host, dev ? dev + n_short : nullptr, out, 0);
    RiskGrids g;
    const hipError_t e = risk_grids(host, n_long, g);
    if (e != hipSuccess) return e;
    bool some = false, more = false;
    for (int i = 0; i < n_long; ++i) (host[i].n > kRiskSampleMore ? more : some) = true;
    if (some) hipLaunchKernelGGL(k_risk_sample<1>, dim3(unsigned(n_long)), block, 0, s, a);
    if (more) hipLaunchKernelGGL(k_risk_sample<4>, dim3(unsigned(n_long)), block, 0, s, a);
    hipLaunchKernelGGL(k_risk_bins, g.bins, block, 0, s, a);
    hipLaunchKernelGGL(k_risk_collect<true>, g.collect, block, 0, s, a);
    hipLaunchKernelGGL(k_risk_sum, g.sum, dim3(kSumWaves * 64), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_risk_round(const RiskJob *host, const RiskJob *dev, int n_long, int round, const RiskOut &out,
                             hipStream_t s) {
    const RiskArgs a = risk_args(host, dev, out, round);
    RiskGrids g;
    const hipError_t e = risk_grids(host, n_long, g);
    if (e != hipSuccess) return e;
    const dim3 block(kRiskThreads);
    hipLaunchKernelGGL(k_risk_narrow, g.bins, block, 0, s, a);
    hipLaunchKernelGGL(k_risk_collect<false>, g.collect, block, 0, s, a);
    hipLaunchKernelGGL(k_risk_sum, g.sum, dim3(kSumWaves * 64), 0, s, a);
    return hipGetLastError();
}

}  // namespace ara
