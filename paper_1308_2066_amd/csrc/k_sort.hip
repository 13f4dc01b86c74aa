// The YLT sorted in descending order (ara_sort_desc).  PML and TVaR need no sort: see
// k_risk.hip.
//
// A binary64 value maps to an unsigned key whose order is the value order (sign flip for
// non-negatives, complement for negatives, -0.0 canonicalised to +0.0); descending order
// sorts the complemented key ascending.  What bounds it up to about 10^6 losses is the
// number of dependent launches, 4.5-5 us each (10^5 losses are 0.2 us of HBM), so the path
// goes by the size (times with the wait, for distinct losses):
//   up to 1024: one workgroup (27 us for 1000 losses; 26 radix launches 121 us);
//   up to 2^20: buckets by sampled splitters, four launches (32 us for 4000 losses, 47 for
//     10^5, 87 for 5 10^5, 131 for 10^6; radix 120, 127, 147, 173).  One workgroup takes 38 us for
//     2000;
//   more: the radix passes (2 10^6 losses 247 us; a bucket would no longer fit the registers
//     of its workgroup).
//
// The radix sort: LSD, 64-bit keys, 8-bit digits, 8 passes.  The encoding pass also finds the digits in which
// keys differ; a pass in which every key has the same digit is skipped on the device
// (capped YLTs often hold one value many times).  Each other pass: per-tile digit
// counts, exclusive offsets per (digit, tile), and a stable scatter in which every
// wave ranks its keys by matching digits across lanes with 8 ballots; the tile's keys
// are placed in LDS in output order first, so a store instruction writes runs of
// consecutive output positions.
#include "order_keys.h"

namespace ara {

constexpr int kSortThreads = 1024;
constexpr int kSortPerThread = 2;
constexpr int kSortTile = kSortThreads * kSortPerThread;   // 2048 keys
constexpr int kWavesPerTile = kSortThreads / 64;            // 16
constexpr int kWaveKeys = 64 * kSortPerThread;              // consecutive keys a wave owns
constexpr int kPasses = 8;
static_assert(kSortThreads >= 256 && kSortThreads % 64 == 0, "the first 256 threads take one digit each");

static inline int64_t sort_tiles(int64_t n) { return (n + kSortTile - 1) / kSortTile; }

// Workspace: two key buffers, per-(digit, tile) counts, the encoding's digit
// differences (one 64-bit word per workgroup), and the pass plan (which buffer holds
// the keys before each pass, and which passes leave the order unchanged because
// every key has the same digit).
struct SortWs {
    uint64_t *a, *b;
    uint32_t *counts;   // [256][tiles]
    uint32_t *hist;     // 8 KB: the encoding's per-workgroup digit differences (uint64)
    uint32_t *dtotal;   // [256] keys per digit in the current pass (in the second half of hist)
    uint32_t *plan;     // plan[p]: keys before pass p are in b (1) or a (0), p = 0..8;
                        // plan[16 + p]: pass p is skipped
};

constexpr size_t kSortSpareBytes = 128 * 1024;   // room for the splitters and counts of the sort by buckets

static size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

size_t sort_workspace_bytes(int64_t n) {
    return 2 * align256(size_t(n) * 8) + align256(size_t(sort_tiles(n)) * 256 * 4) + align256(8 * 256 * 4) + 256 +
           kSortSpareBytes;
}

static SortWs sort_ws(void *ws, int64_t n) {
    char *p = reinterpret_cast<char *>(ws);
    const size_t keys = align256(size_t(n) * 8);
    const size_t counts = align256(size_t(sort_tiles(n)) * 256 * 4);
    SortWs w;
    w.a = reinterpret_cast<uint64_t *>(p);
    w.b = reinterpret_cast<uint64_t *>(p + keys);
    w.counts = reinterpret_cast<uint32_t *>(p + 2 * keys);
    w.hist = reinterpret_cast<uint32_t *>(p + 2 * keys + counts);
    w.dtotal = w.hist + 1024;   // after 512 64-bit slots of encoding differences
    w.plan = reinterpret_cast<uint32_t *>(p + 2 * keys + counts + align256(8 * 256 * 4));
    return w;
}

__device__ __forceinline__ const uint64_t *cur_keys(const SortWs &w, int pass) {
    return w.plan[pass] ? w.b : w.a;
}

// Encode values into descending-order keys.  A pass leaves the order unchanged when
// every key has the same digit in it; so each workgroup also ORs key ^ (the first
// key) over its keys, and a pass is skipped when that digit of the OR over all
// workgroups is zero.  A wave reads 8 rows of 64 values at a time.
constexpr int kEncodeBlocks = 256;   // workgroups of k_sort_encode (one OR slot each)
static_assert(kEncodeBlocks <= 512, "the OR slots end where the digit totals start");

__global__ __launch_bounds__(1024) void k_sort_encode(const double *__restrict__ in, int64_t n,
                                                     uint64_t *__restrict__ keys, uint64_t *__restrict__ diff) {
    constexpr int kRows = 8;
    __shared__ uint64_t wdiff[16];
    const uint64_t k0 = desc_key(in[0]);
    const int64_t stride = int64_t(gridDim.x) * blockDim.x;
    uint64_t d = 0;
    for (int64_t i0 = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i0 < n; i0 += kRows * stride) {
        uint64_t k[kRows];
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const int64_t i = i0 + r * stride;
            k[r] = i < n ? desc_key(in[i]) : k0;
        }
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const int64_t i = i0 + r * stride;
            if (i < n) keys[i] = k[r];
            d |= k[r] ^ k0;
        }
    }
    for (int o = 32; o >= 1; o >>= 1) d |= __shfl_xor(d, o, 64);
    if ((threadIdx.x & 63) == 0) wdiff[threadIdx.x >> 6] = d;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t o = 0;
        for (int k = 0; k < 16; ++k) o |= wdiff[k];
        diff[blockIdx.x] = o;
    }
}

// The plan: which buffer holds the keys before each pass, and which passes are skipped.
__global__ __launch_bounds__(64) void k_sort_plan(const uint64_t *__restrict__ diff, int n_slots,
                                                  uint32_t *__restrict__ plan) {
    uint64_t d = 0;
    for (int i = threadIdx.x; i < n_slots; i += 64) d |= diff[i];
    for (int o = 32; o >= 1; o >>= 1) d |= __shfl_xor(d, o, 64);
    if (threadIdx.x != 0) return;
    uint32_t sel = 0;
    plan[0] = 0;
    for (int p = 0; p < kPasses; ++p) {
        const uint32_t triv = ((d >> (8 * p)) & 255u) == 0 ? 1u : 0u;
        plan[16 + p] = triv;
        sel = triv ? sel : 1u - sel;
        plan[p + 1] = sel;
    }
}

// Lanes whose digit equals this lane's digit (among lanes with `valid`).
__device__ __forceinline__ uint64_t match_digit(uint32_t d, bool valid) {
    uint64_t m = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const uint64_t bb = __ballot((d >> b) & 1u);
        m &= ((d >> b) & 1u) ? bb : ~bb;
    }
    return m;
}

__device__ __forceinline__ uint64_t lanes_below(int lane) { return lane ? (~0ull >> (64 - lane)) : 0ull; }

// counts[d * tiles + tile] = number of keys of the tile with digit d
__global__ __launch_bounds__(kSortThreads) void k_sort_count(SortWs w, int64_t n, int pass, int64_t tiles) {
    if (w.plan[16 + pass]) return;
    __shared__ uint32_t hist[256];
    const uint64_t *keys = cur_keys(w, pass);
    const int shift = 8 * pass;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (threadIdx.x < 256) hist[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = int64_t(blockIdx.x) * kSortTile + wv * kWaveKeys;
    uint32_t d[kSortPerThread];
#pragma unroll
    for (int r = 0; r < kSortPerThread; ++r) {
        const int64_t i = base + r * 64 + lane;
        d[r] = i < n ? uint32_t(keys[i] >> shift) & 255u : 0u;
    }
#pragma unroll
    for (int r = 0; r < kSortPerThread; ++r) {
        if (base + r * 64 + lane < n) atomicAdd(&hist[d[r]], 1u);
    }
    __syncthreads();
    if (threadIdx.x < 256) w.counts[int64_t(threadIdx.x) * tiles + blockIdx.x] = hist[threadIdx.x];
}

// Exclusive offsets within each digit's row of tile counts: one workgroup per digit
// scans its row in place, in chunks of 1024 (four consecutive counts per thread), and
// stores the row's total in w.dtotal.  The scatter adds the prefix of the totals over
// the smaller digits, so the offset of (d, t) is that of the flat digit-major array.
__global__ __launch_bounds__(256) void k_sort_rowscan(SortWs w, int pass, int64_t tiles) {
    if (w.plan[16 + pass]) return;
    __shared__ uint32_t wsum[4];
    uint32_t *c = w.counts + int64_t(blockIdx.x) * tiles;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    uint32_t carry = 0;
    for (int64_t base = 0; base < tiles; base += 1024) {
        uint32_t v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t i = base + 4 * tid + j;
            v[j] = i < tiles ? c[i] : 0u;
        }
        const uint32_t t = v[0] + v[1] + v[2] + v[3];
        uint32_t inc = t;   // inclusive wave scan of the threads' sums
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(inc, o, 64);
            if (lane >= o) inc += y;
        }
        if (lane == 63) wsum[wv] = inc;
        __syncthreads();
        uint32_t before = 0;
        for (int k = 0; k < wv; ++k) before += wsum[k];
        const uint32_t total = wsum[0] + wsum[1] + wsum[2] + wsum[3];
        uint32_t run = carry + before + inc - t;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t i = base + 4 * tid + j;
            if (i < tiles) c[i] = run;
            run += v[j];
        }
        carry += total;
        __syncthreads();
    }
    if (tid == 0) w.dtotal[blockIdx.x] = carry;
}

__global__ __launch_bounds__(kSortThreads) void k_sort_scatter(SortWs w, int64_t n, int pass, int64_t tiles) {
    if (w.plan[16 + pass]) return;
    __shared__ uint32_t whist[kWavesPerTile][256];
    __shared__ uint32_t woff[kWavesPerTile][256];   // tile-local start of (wave, digit)
    __shared__ uint32_t lstart[256];                // tile-local start of each digit
    __shared__ uint32_t gstart[256];                // output index of the tile's first key of each digit
    __shared__ uint64_t stage[kSortTile];           // the tile's keys in output order
    __shared__ uint32_t wtot[4], ltot[4];
    const uint64_t *in = cur_keys(w, pass);
    uint64_t *out = w.plan[pass] ? w.a : w.b;
    const int shift = 8 * pass;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int i = threadIdx.x; i < kWavesPerTile * 256; i += kSortThreads) whist[i >> 8][i & 255] = 0;
    // keys in the smaller digits: exclusive scan of the digit totals (first four waves)
    uint32_t dt = 0, dinc = 0;
    if (threadIdx.x < 256) {
        dt = w.dtotal[threadIdx.x];
        dinc = dt;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(dinc, o, 64);
            if (lane >= o) dinc += y;
        }
        if (lane == 63) wtot[wv] = dinc;
    }
    __syncthreads();
    uint32_t dbase = dinc - dt;
    for (int k = 0; k < wv && k < 4; ++k) dbase += wtot[k];
    const int64_t tile0 = int64_t(blockIdx.x) * kSortTile;
    const int64_t base = tile0 + wv * kWaveKeys;
    uint64_t key[kSortPerThread];
    uint32_t rank[kSortPerThread];
#pragma unroll
    for (int r = 0; r < kSortPerThread; ++r) {
        const int64_t i = base + r * 64 + lane;
        key[r] = i < n ? in[i] : 0ull;
    }
#pragma unroll
    for (int r = 0; r < kSortPerThread; ++r) {
        const bool valid = base + r * 64 + lane < n;
        const uint32_t d = uint32_t(key[r] >> shift) & 255u;
        const uint64_t m = match_digit(d, valid);
        const uint64_t below = m & lanes_below(lane);
        rank[r] = whist[wv][d] + uint32_t(__popcll(below));   // read before this round's update
        if (valid && below == 0) whist[wv][d] += uint32_t(__popcll(m));
    }
    __syncthreads();
    // tile-local start of each digit: exclusive scan of the tile's digit counts
    uint32_t tt = 0, tinc = 0;
    if (threadIdx.x < 256) {
        for (int k = 0; k < kWavesPerTile; ++k) tt += whist[k][threadIdx.x];
        tinc = tt;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(tinc, o, 64);
            if (lane >= o) tinc += y;
        }
        if (lane == 63) ltot[wv] = tinc;
    }
    __syncthreads();
    if (threadIdx.x < 256) {
        const int d = threadIdx.x;
        uint32_t run = tinc - tt;
        for (int k = 0; k < wv; ++k) run += ltot[k];
        lstart[d] = run;
        gstart[d] = dbase + w.counts[int64_t(d) * tiles + blockIdx.x];
        for (int k = 0; k < kWavesPerTile; ++k) {
            woff[k][d] = run;
            run += whist[k][d];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortPerThread; ++r) {
        if (base + r * 64 + lane < n) {
            const uint32_t d = uint32_t(key[r] >> shift) & 255u;
            stage[woff[wv][d] + rank[r]] = key[r];
        }
    }
    __syncthreads();
    // consecutive threads write consecutive keys of a digit's run
    const int tile_n = int(std::min<int64_t>(kSortTile, n - tile0));
    for (int i = threadIdx.x; i < tile_n; i += kSortThreads) {
        const uint64_t k = stage[i];
        const uint32_t d = uint32_t(k >> shift) & 255u;
        out[gstart[d] + uint32_t(i) - lstart[d]] = k;
    }
}

__global__ __launch_bounds__(256) void k_sort_decode(SortWs w, int64_t n, double *__restrict__ out) {
    const uint64_t *keys = cur_keys(w, kPasses);
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x)
        out[i] = key_value(keys[i]);
}

// Every pass is launched (the caller must not block); trivial ones return at once.
static hipError_t launch_radix(const double *in, int64_t n, const SortWs &w, double *out, hipStream_t s) {
    const int64_t tiles = sort_tiles(n);
    const unsigned eb = unsigned(std::min<int64_t>((n + 255) / 256, kEncodeBlocks));
    uint64_t *diff = reinterpret_cast<uint64_t *>(w.hist);
    hipLaunchKernelGGL(k_sort_encode, dim3(eb), dim3(1024), 0, s, in, n, w.a, diff);
    hipLaunchKernelGGL(k_sort_plan, dim3(1), dim3(64), 0, s, diff, int(eb), w.plan);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    for (int pass = 0; pass < kPasses; ++pass) {
        hipLaunchKernelGGL(k_sort_count, dim3(unsigned(tiles)), dim3(kSortThreads), 0, s, w, n, pass, tiles);
        hipLaunchKernelGGL(k_sort_rowscan, dim3(256), dim3(256), 0, s, w, pass, tiles);
        hipLaunchKernelGGL(k_sort_scatter, dim3(unsigned(tiles)), dim3(kSortThreads), 0, s, w, n, pass, tiles);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const unsigned db = unsigned(std::min<int64_t>((n + 255) / 256, 4096));
    hipLaunchKernelGGL(k_sort_decode, dim3(db), dim3(256), 0, s, w, n, out);
    return hipGetLastError();
}

// ------------------------------------------------------------------ by sampled buckets
// Splitters: every fourth of 4 `buckets` sampled keys in order.  Bucket 2 i holds the keys
// between splitters i - 1 and i, bucket 2 i + 1 those equal to splitter i (the first of
// equal splitters), so a value that many losses share is a bucket that needs no sorting.
// Four launches: the sample ranked and the splitters taken (7 us for 10^5 losses, 2048
// samples, 512 buckets), each key's bucket and place in it (8 us), the keys moved (5 us), the
// buckets sorted and decoded (12 us: 256 keys in a wave's registers at a time; a bitonic
// network in LDS with the workgroup's barriers took 22 us).
constexpr int kOverSample = 4;
constexpr int kMaxBuckets = 1024;                         // splitter buckets (strict ones)
constexpr int kMaxSample = kOverSample * kMaxBuckets;
constexpr int kRankShare = 16;                            // samples ranked by a workgroup of 256
constexpr int kBucketKeys = 4;                            // keys per thread of the counting pass
constexpr int kBucketLds = 8192;                          // largest bucket sorted in LDS
constexpr int kOneWgSort = 1024;                          // losses sorted by one workgroup
constexpr int64_t kBucketMaxN = int64_t(1) << 20;         // a key's bucket and place share 32 bits
static_assert(2 * kMaxBuckets <= 1 << 11, "bucket in 11 bits, place in 21");

struct BucketWs {
    uint64_t *split;    // [buckets] (the last: all ones)
    uint32_t *counts;   // [2 buckets]
    uint32_t *starts;   // [2 buckets + 1]
    uint32_t *place;    // [n] bucket << 21 | place in it; its memory is the radix fallback's afterwards
    uint64_t *tmp;      // [n] the same memory
    uint64_t *keys;     // [n] the strict buckets' keys, bucket after bucket
    int buckets;        // a power of two
    int log_sample;     // log2(kOverSample * buckets)
};

static int bucket_count(int64_t n) {
    int b = 128;
    while (b < kMaxBuckets && b * int64_t(256) < n) b *= 2;
    return b;
}

static BucketWs bucket_ws(const SortWs &w, int64_t n) {
    BucketWs k;
    char *p = reinterpret_cast<char *>(w.plan) + 256;   // the spare bytes at the workspace's end
    k.split = reinterpret_cast<uint64_t *>(p);
    k.counts = reinterpret_cast<uint32_t *>(p + kMaxBuckets * 8);
    k.starts = k.counts + 2 * kMaxBuckets;
    k.place = reinterpret_cast<uint32_t *>(w.a);
    k.tmp = w.a;
    k.keys = w.b;
    k.buckets = bucket_count(n);
    k.log_sample = __builtin_ctz(unsigned(kOverSample * k.buckets));
    static_assert(kMaxBuckets * 8 + 4 * kMaxBuckets * 4 + 4 <= kSortSpareBytes, "spare bytes");
    return k;
}

// Sample j is a loss of the j-th of S equal stretches, at a place within it that varies.
// Each workgroup reads the whole sample and ranks 16 of its keys, by the keys before them
// (equal ones in sample order): 16 threads per key count a sixteenth of the sample each.
// The counts of the next kernel are cleared on the way.
__global__ __launch_bounds__(256) void k_bucket_split(const double *__restrict__ y, int64_t n, BucketWs w) {
    __shared__ uint64_t key[kMaxSample];
    __shared__ uint32_t rank[kRankShare];
    const int tid = threadIdx.x, S = kOverSample * w.buckets;
#pragma unroll 4
    for (int j = tid; j < S; j += 256) {
        const int64_t a = (int64_t(j) * n) >> w.log_sample, e = (int64_t(j + 1) * n) >> w.log_sample;
        const uint64_t k = desc_key(y[a + __umulhi(uint32_t(j) * 2654435761u, uint32_t(e - a))]);
        key[j] = k == ~0ull ? ~0ull - 1ull : k;   // splitters need not be losses; key + 1 must exist
    }
    if (tid < kRankShare) rank[tid] = 0u;
    const int g = int(blockIdx.x) * 256 + tid;
    if (g < 2 * w.buckets) w.counts[g] = 0u;
    if (g == 0) w.split[w.buckets - 1] = ~0ull;
    __syncthreads();
    const int len = S / 16, seg = tid >> 4, me = int(blockIdx.x) * kRankShare + (tid & 15);
    const uint64_t k = key[me];
    uint32_t c = 0;
#pragma unroll 8
    for (int x = 0; x < len; ++x) {
        const int j = seg * len + ((x + seg) & (len - 1));   // a wave's four segments in different banks
        c += key[j] < (j < me ? k + 1ull : k) ? 1u : 0u;
    }
    c += __shfl_xor(c, 16, 64);
    c += __shfl_xor(c, 32, 64);
    if ((tid & 48) == 0) atomicAdd(&rank[tid & 15], c);
    __syncthreads();
    if (tid >= kRankShare) return;
    const int r = int(rank[tid]) + 1;
    if (r % kOverSample == 0 && r < S) w.split[r / kOverSample - 1] = k;
}

// The keys' buckets: their places among the buckets - 1 splitters (binary searches side by side).
__device__ __forceinline__ void buckets_of(const uint64_t *split, int buckets, const uint64_t (&k)[kBucketKeys],
                                           uint32_t (&b)[kBucketKeys]) {
#pragma unroll
    for (int r = 0; r < kBucketKeys; ++r) b[r] = 0u;
#pragma unroll 1
    for (uint32_t step = uint32_t(buckets) >> 1; step >= 1u; step >>= 1) {
        uint64_t s[kBucketKeys];
#pragma unroll
        for (int r = 0; r < kBucketKeys; ++r) s[r] = split[b[r] + step - 1u];
#pragma unroll
        for (int r = 0; r < kBucketKeys; ++r) b[r] += s[r] < k[r] ? step : 0u;
    }
#pragma unroll
    for (int r = 0; r < kBucketKeys; ++r)
        b[r] = 2u * b[r] + (split[b[r]] == k[r] && b[r] < uint32_t(buckets) - 1u ? 1u : 0u);
}

// Every key's bucket and place in it: places within the workgroup from LDS counters, the
// workgroup's first place from the bucket's counter (the order in a bucket is free).
__global__ __launch_bounds__(1024) void k_bucket_place(const double *__restrict__ y, int64_t n, BucketWs w) {
    __shared__ uint64_t split[kMaxBuckets];
    __shared__ uint32_t hist[2 * kMaxBuckets];
    const int64_t i0 = int64_t(blockIdx.x) * blockDim.x * kBucketKeys + threadIdx.x;
    double v[kBucketKeys];
#pragma unroll
    for (int r = 0; r < kBucketKeys; ++r) {
        const int64_t i = i0 + r * int64_t(blockDim.x);
        v[r] = i < n ? y[i] : 0.0;
    }
    for (int i = threadIdx.x; i < w.buckets; i += blockDim.x) split[i] = w.split[i];
    for (int i = threadIdx.x; i < 2 * w.buckets; i += blockDim.x) hist[i] = 0u;
    __syncthreads();
    uint64_t k[kBucketKeys];
    uint32_t b[kBucketKeys], at[kBucketKeys];
#pragma unroll
    for (int r = 0; r < kBucketKeys; ++r) k[r] = desc_key(v[r]);
    buckets_of(split, w.buckets, k, b);
#pragma unroll
    for (int r = 0; r < kBucketKeys; ++r)
        if (i0 + r * int64_t(blockDim.x) < n) at[r] = atomicAdd(&hist[b[r]], 1u);
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * w.buckets; i += blockDim.x)
        if (hist[i]) hist[i] = atomicAdd(&w.counts[i], hist[i]);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kBucketKeys; ++r) {
        const int64_t i = i0 + r * int64_t(blockDim.x);
        if (i < n) w.place[i] = b[r] << 21 | (hist[b[r]] + at[r]);
    }
}

// The keys of the strict buckets to their buckets.  Every workgroup forms the buckets'
// starts (an exclusive scan of the counts); the first one keeps them for the next kernel.
__global__ __launch_bounds__(1024) void k_bucket_scatter(const double *__restrict__ y, int64_t n, BucketWs w) {
    __shared__ uint32_t start[2 * kMaxBuckets + 1];
    __shared__ uint32_t wsum[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, total = 2 * w.buckets;
    const int64_t i0 = int64_t(blockIdx.x) * blockDim.x * kBucketKeys + tid;
    double v[kBucketKeys];
    uint32_t q[kBucketKeys];
#pragma unroll
    for (int r = 0; r < kBucketKeys; ++r) {
        const int64_t i = i0 + r * int64_t(blockDim.x);
        v[r] = i < n ? y[i] : 0.0;
        q[r] = i < n ? w.place[i] : 1u << 21;   // an equal bucket's key stays
    }
    for (int i = tid; i < total; i += blockDim.x) start[i] = w.counts[i];
    __syncthreads();
    const int per = (total + int(blockDim.x) - 1) / int(blockDim.x), c0 = min(tid * per, total), c1 = min(c0 + per, total);
    uint32_t own = 0;
    for (int i = c0; i < c1; ++i) own += start[i];
    uint32_t inc = own;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t x = __shfl_up(inc, o, 64);
        if (lane >= o) inc += x;
    }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    uint32_t run = inc - own;
    for (int k = 0; k < wave; ++k) run += wsum[k];
    for (int i = c0; i < c1; ++i) {
        const uint32_t c = start[i];
        start[i] = run;
        run += c;
    }
    if (tid == 0) start[total] = uint32_t(n);
    __syncthreads();
    if (blockIdx.x == 0)
        for (int i = tid; i <= total; i += blockDim.x) w.starts[i] = start[i];
#pragma unroll
    for (int r = 0; r < kBucketKeys; ++r) {
        const uint32_t b = q[r] >> 21;
        if (!(b & 1u)) w.keys[start[b] + (q[r] & 0x1FFFFFu)] = desc_key(v[r]);
    }
}

// keys[0, M) ascending, M a power of two (whole workgroup; keys written before).  Steps of
// distance at most 64 stay within a wave's own 128 keys and need no barrier.
__device__ __forceinline__ void bitonic_sort(uint64_t *keys, int M) {
    __syncthreads();
#pragma unroll 1
    for (int k = 2; k <= M; k <<= 1) {
#pragma unroll 1
        for (int j = k >> 1; j >= 1; j >>= 1) {
#pragma unroll 1
            for (int p = threadIdx.x; p < M / 2; p += blockDim.x) {
                const int i = 2 * p - (p & (j - 1));
                const uint64_t x = keys[i], z = keys[i + j];
                if ((x > z) == ((i & k) == 0)) keys[i] = z, keys[i + j] = x;
            }
            // the next step's distance: j / 2, or k at the start of the next k
            const int next = j > 1 ? j >> 1 : k;
            if (j > 64 || next > 64) __syncthreads();
            else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"), __builtin_amdgcn_wave_barrier();
        }
    }
    __syncthreads();
}

__device__ __forceinline__ void order(uint64_t &a, uint64_t &b, bool up) {
    const bool swap = (a > b) == up;
    const uint64_t t = swap ? b : a;
    b = swap ? a : b;
    a = t;
}

// 256 keys ascending in a wave's registers (key 4 lane + r in x[r]): a bitonic network
// whose steps of distance 1 and 2 stay in a lane and whose others go across lanes.
__device__ __forceinline__ void wave_sort(uint64_t (&x)[4], int lane) {
    order(x[0], x[1], true);
    order(x[2], x[3], false);
#pragma unroll 1
    for (int k = 1; k <= 64; k <<= 1) {
        const bool up = (lane & k) == 0;
#pragma unroll 1
        for (int l = k >> 1; l >= 1; l >>= 1) {
            const bool low = ((lane & l) == 0) == up;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint64_t o = uint64_t(__shfl_xor((unsigned long long)x[r], l, 64));
                x[r] = (x[r] < o) == low ? x[r] : o;
            }
        }
        order(x[0], x[2], up);
        order(x[1], x[3], up);
        order(x[0], x[1], up);
        order(x[2], x[3], up);
    }
}

constexpr int kWaveSort = 256;   // keys a wave sorts

// The m keys of in() (in(i), i < m; at most 4 per thread) in order, to out(place, key): each
// wave sorts 256, then every key finds its place among the other waves' (equal keys in wave
// order).  Whole workgroup; lds holds kWaveSort keys per wave.
template <typename In, typename Out>
__device__ __forceinline__ void wave_merge_sort(int m, uint64_t *lds, In in, Out out) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int runs = (m + kWaveSort - 1) / kWaveSort;
    uint64_t x[4];
    if (wave < runs) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = wave * kWaveSort + 64 * r + lane;
            x[r] = i < m ? in(i) : ~0ull;
        }
        wave_sort(x, lane);
    }
    uint32_t at[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) at[r] = uint32_t(4 * lane + r);
    if (runs > 1) {
        if (wave < runs) {
#pragma unroll
            for (int r = 0; r < 4; ++r) lds[wave * kWaveSort + 4 * lane + r] = x[r];
        }
        __syncthreads();
        if (wave < runs) {
#pragma unroll 1
            for (int c = 0; c < runs; ++c) {
                if (c == wave) continue;
                const uint64_t *run = lds + c * kWaveSort;
                const bool before = c < wave;   // its equal keys come first
                uint32_t p[4] = {};
                auto step = [&](uint32_t w) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const uint64_t o = run[p[r] + w - 1u];
                        p[r] += (before ? o <= x[r] : o < x[r]) ? w : 0u;
                    }
                };
#pragma unroll 1
                for (uint32_t w = kWaveSort / 2; w >= 1u; w >>= 1) step(w);
                step(1u);
#pragma unroll
                for (int r = 0; r < 4; ++r) at[r] += p[r];
            }
        }
    }
    if (wave < runs) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (at[r] < uint32_t(m)) out(at[r], x[r]);
    }
}

// A bucket too large for LDS (the sample missed most of its keys): LSD radix passes by the
// first 256 threads of a workgroup, between src and dst; returns where the sorted keys are.
__device__ __forceinline__ uint64_t *bucket_radix(uint64_t *src, uint64_t *dst, int m, uint32_t *lds) {
    uint32_t *offs = lds, *hist = lds + 256;   // hist: [4][256]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool on = tid < 256;                 // every thread meets the barriers
#pragma unroll 1
    for (int shift = 0; shift < 64; shift += 8) {
        __syncthreads();
        if (on) offs[tid] = 0u;
        __syncthreads();
        for (int i = tid; i < m; i += blockDim.x) atomicAdd(&offs[(src[i] >> shift) & 255u], 1u);
        __syncthreads();
        uint32_t before = 0;
        if (on)
            for (int d = 0; d < tid; ++d) before += offs[d];
        __syncthreads();
        if (on) offs[tid] = before;
#pragma unroll 1
        for (int t0 = 0; t0 < m; t0 += 256) {
            if (on)
                for (int q = 0; q < 4; ++q) hist[256 * q + tid] = 0u;
            __syncthreads();
            const bool valid = on && t0 + tid < m;
            const uint64_t k = valid ? src[t0 + tid] : 0ull;
            const uint32_t d = uint32_t(k >> shift) & 255u;
            const uint64_t same = match_digit(d, valid), below = same & lanes_below(lane);
            if (valid && below == 0) hist[256 * wave + d] = uint32_t(__popcll(same));
            __syncthreads();
            if (valid) {
                uint32_t at = offs[d] + uint32_t(__popcll(below));
                for (int q = 0; q < wave; ++q) at += hist[256 * q + d];
                dst[at] = k;
            }
            __syncthreads();
            if (on) offs[tid] += hist[tid] + hist[256 + tid] + hist[512 + tid] + hist[768 + tid];
        }
        uint64_t *x = src;
        src = dst;
        dst = x;
    }
    __syncthreads();
    return src;
}

// Workgroup g sorts strict bucket g, and writes the equal buckets' values in its share of
// the output positions.
__global__ __launch_bounds__(512) void k_bucket_sort(int64_t n, BucketWs w, double *__restrict__ out) {
    __shared__ uint64_t keys[kBucketLds];
    __shared__ uint32_t start[2 * kMaxBuckets + 1];
    const int tid = threadIdx.x, threads = blockDim.x, g = blockIdx.x, total = 2 * w.buckets;
    const uint32_t s0 = w.starts[2 * g];
    const int m = int(w.starts[2 * g + 1] - s0);
    const uint64_t *src = w.keys + s0;
    double *dst = out + s0;
    for (int i = tid; i <= total; i += threads) start[i] = w.starts[i];
    if (m <= 4 * threads) {
        wave_merge_sort(m, keys, [&](int i) { return src[i]; }, [&](uint32_t at, uint64_t k) { dst[at] = key_value(k); });
    } else {
        const uint64_t *sorted = keys;
        if (m <= kBucketLds) {
            int M = 2;
            while (M < m) M <<= 1;
            for (int i = tid; i < M; i += threads) keys[i] = i < m ? src[i] : ~0ull;
            bitonic_sort(keys, M);
        } else {
            sorted = bucket_radix(w.keys + s0, w.tmp + s0, m, reinterpret_cast<uint32_t *>(keys));
        }
        for (int i = tid; i < m; i += threads) dst[i] = key_value(sorted[i]);
    }
    __syncthreads();
    const int64_t share = (n + w.buckets - 1) / w.buckets;
    const uint32_t p1 = uint32_t(min(n, (g + 1) * share));
    for (uint32_t p = uint32_t(g * share) + tid; p < p1; p += threads) {
        uint32_t b = 0;   // the last bucket that starts at or before p
        for (uint32_t step = uint32_t(total) >> 1; step >= 1u; step >>= 1)
            if (start[b + step] <= p) b += step;
        if (b & 1u) out[p] = key_value(w.split[b >> 1]);
    }
}

// Up to kOneWgSort losses, in one workgroup.
__global__ __launch_bounds__(512) void k_sort_one(const double *in, int n, double *out) {
    __shared__ uint64_t keys[kOneWgSort];
    wave_merge_sort(n, keys, [&](int i) { return desc_key(in[i]); }, [&](uint32_t at, uint64_t k) { out[at] = key_value(k); });
}

hipError_t launch_sort_desc(const double *in, int64_t n, double *out, void *ws, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    if (n <= kOneWgSort) {
        hipLaunchKernelGGL(k_sort_one, dim3(1), dim3(unsigned((n + 255) / 256) * 64u), 0, s, in, int(n), out);
        return hipGetLastError();
    }
    const SortWs w = sort_ws(ws, n);
    if (n > kBucketMaxN) return launch_radix(in, n, w, out, s);
    const BucketWs k = bucket_ws(w, n);
    const unsigned threads = n > 1 << 18 ? 1024u : 256u, tile = threads * kBucketKeys;
    const unsigned blocks = unsigned((n + tile - 1) / tile);
    hipLaunchKernelGGL(k_bucket_split, dim3(unsigned(kOverSample * k.buckets / kRankShare)), dim3(256), 0, s, in, n, k);
    hipLaunchKernelGGL(k_bucket_place, dim3(blocks), dim3(threads), 0, s, in, n, k);
    hipLaunchKernelGGL(k_bucket_scatter, dim3(blocks), dim3(threads), 0, s, in, n, k);
    hipLaunchKernelGGL(k_bucket_sort, dim3(unsigned(k.buckets)), dim3(n > 1 << 18 ? 512u : 256u), 0, s, n, k, out);
    return hipGetLastError();
}

}  // namespace ara
