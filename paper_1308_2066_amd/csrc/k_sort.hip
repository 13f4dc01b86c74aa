// The YLT sorted in descending order (ara_sort_desc).  PML and TVaR need no sort: see
// k_risk.hip.
//
// LSD radix sort of 64-bit keys, 8-bit digits, 8 passes.  A binary64 value maps to
// an unsigned key whose order is the value order (sign flip for non-negatives,
// complement for negatives, -0.0 canonicalised to +0.0); descending order sorts the
// complemented key ascending.  The encoding pass also finds the digits in which
// keys differ; a pass in which every key has the same digit is skipped on the device
// (capped YLTs often hold one value many times).  Each other pass: per-tile digit
// counts, exclusive offsets per (digit, tile), and a stable scatter in which every
// wave ranks its keys by matching digits across lanes with 8 ballots; the tile's keys
// are placed in LDS in output order first, so a store instruction writes runs of
// consecutive output positions.
#include "ara_internal.h"

namespace ara {

constexpr int kSortThreads = 1024;
constexpr int kSortPerThread = 2;
constexpr int kSortTile = kSortThreads * kSortPerThread;   // 2048 keys
constexpr int kWavesPerTile = kSortThreads / 64;            // 16
constexpr int kWaveKeys = 64 * kSortPerThread;              // consecutive keys a wave owns
constexpr int kPasses = 8;
static_assert(kSortThreads >= 256 && kSortThreads % 64 == 0, "the first 256 threads take one digit each");

__device__ __forceinline__ uint64_t desc_key(double d) {
    uint64_t u = __builtin_bit_cast(uint64_t, d + 0.0);   // -0.0 + 0.0 == +0.0
    u = (u >> 63) ? ~u : (u | 0x8000000000000000ull);       // ascending order key
    return ~u;                                             // descending
}

__device__ __forceinline__ double key_value(uint64_t k) {
    uint64_t u = ~k;
    u = (u >> 63) ? (u & 0x7FFFFFFFFFFFFFFFull) : ~u;
    return __builtin_bit_cast(double, u);
}

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

constexpr size_t kSortSpareBytes = 128 * 1024;   // room for the risk measures' counts (k_risk.hip uses the
                                                 // same workspace)

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

// Sorted descending keys of `in` end in the workspace key buffer the plan names.
// host_plan: pinned host memory of 32 words, or null.  With it, the host reads the
// pass plan (one small copy and a wait) and launches only the passes that reorder
// keys; without it every pass is launched and trivial ones return at once (for
// callers that must not block).
hipError_t launch_sort_desc_keys(const double *in, int64_t n, void *ws, hipStream_t s, uint32_t *host_plan) {
    if (n <= 0) return hipSuccess;
    SortWs w = sort_ws(ws, n);
    const int64_t tiles = sort_tiles(n);
    const unsigned eb = unsigned(std::min<int64_t>((n + 255) / 256, kEncodeBlocks));
    uint64_t *diff = reinterpret_cast<uint64_t *>(w.hist);
    hipLaunchKernelGGL(k_sort_encode, dim3(eb), dim3(1024), 0, s, in, n, w.a, diff);
    hipLaunchKernelGGL(k_sort_plan, dim3(1), dim3(64), 0, s, diff, int(eb), w.plan);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    bool skip[kPasses] = {};
    if (host_plan) {
        e = hipMemcpyAsync(host_plan, w.plan, 32 * sizeof(uint32_t), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) return e;
        for (int p = 0; p < kPasses; ++p) skip[p] = host_plan[16 + p] != 0;
    }
    for (int pass = 0; pass < kPasses; ++pass) {
        if (skip[pass]) continue;
        hipLaunchKernelGGL(k_sort_count, dim3(unsigned(tiles)), dim3(kSortThreads), 0, s, w, n, pass, tiles);
        hipLaunchKernelGGL(k_sort_rowscan, dim3(256), dim3(256), 0, s, w, pass, tiles);
        hipLaunchKernelGGL(k_sort_scatter, dim3(unsigned(tiles)), dim3(kSortThreads), 0, s, w, n, pass, tiles);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_sort_decode(const void *ws, int64_t n, double *out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    SortWs w = sort_ws(const_cast<void *>(ws), n);
    const unsigned eb = unsigned(std::min<int64_t>((n + 255) / 256, 4096));
    hipLaunchKernelGGL(k_sort_decode, dim3(eb), dim3(256), 0, s, w, n, out);
    return hipGetLastError();
}

}  // namespace ara
