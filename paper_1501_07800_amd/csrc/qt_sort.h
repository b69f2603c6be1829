// Stable device sorts by an integer key (matrix build, copy-out, truncation).
//
// A sort takes its keys from a source, src(i) = key of entry i (computed from
// arrays that stay in place), and hands its result to a sink,
// sink(rank, i, key): only the permutation moves between passes. Entries of
// equal keys keep their order (ascending i).
//
//  * Up to RANK_SORT_MAX entries: one launch. Every workgroup holds all keys
//    in LDS and ranks 64 entries by counting the keys before each, a quarter
//    of the keys per wave. n = 374: 2 launches (with the copy that follows)
//    where a bitonic network took one launch per stage, 47.
//  * Beyond: least-significant-digit radix passes over the key's bits, three
//    launches a pass: digit counts per tile; an exclusive scan of every
//    digit's counts over the tiles; the scatter. A digit has up to 11 bits
//    (2048 LDS counters per wave), so the row of a block, all that a
//    row-major copy-out sorts by, takes one pass up to 2048 block rows. What
//    bounds a pass are its three dependent launches of 3-6 us each, at any
//    size below a million entries.
#pragma once
#include "qt_internal.h"

#include <algorithm>

namespace qt {

constexpr int RANK_SORT_MAX = 4096;      // 32 KiB of keys in LDS; above, a radix pass is as fast
constexpr int RADIX_DIGIT_MAX = 11;
constexpr int RADIX_THREADS = 256, RADIX_WAVES = RADIX_THREADS / 64;
constexpr int64_t RADIX_TILE_MIN = 1024;  // entries per workgroup: 133 workgroups at 136 k entries
constexpr int64_t RADIX_TILES_MAX = 448;  // the counts stay below 4 MiB at any n

struct RadixPlan {
    int passes = 1, digit = 1;
    int64_t tile = RADIX_TILE_MIN, tiles = 1;
    int bins() const { return 1 << digit; }
};

inline RadixPlan radix_plan(int64_t n, int key_bits) {
    RadixPlan p;
    key_bits = std::max(key_bits, 1);
    p.passes = (key_bits + RADIX_DIGIT_MAX - 1) / RADIX_DIGIT_MAX;
    p.digit = (key_bits + p.passes - 1) / p.passes;
    while (n > RADIX_TILES_MAX * p.tile) p.tile *= 2;
    p.tiles = std::max<int64_t>((n + p.tile - 1) / p.tile, 1);
    return p;
}

// Words (int32) of scratch a sort of n entries takes beside the permutation
// array that the caller lends it: the counts and digit totals, and a second
// permutation when there is more than one pass.
inline size_t sort_tmp_words(int64_t n, int key_bits) {
    if (n <= RANK_SORT_MAX) return 0;
    const RadixPlan p = radix_plan(n, key_bits);
    return (size_t)p.bins() * (p.tiles + 1) + (p.passes > 1 ? (size_t)n : 0);
}

// The same for any number of entries up to n (beyond the smallest tiles, fewer
// entries can mean more tiles).
inline size_t sort_tmp_bound(int64_t n, int key_bits) {
    if (n <= RANK_SORT_MAX) return 0;
    const RadixPlan p = radix_plan(n, key_bits);
    const int64_t tiles = p.tile == RADIX_TILE_MIN ? p.tiles : RADIX_TILES_MAX;
    return (size_t)p.bins() * (tiles + 1) + (p.passes > 1 ? (size_t)n : 0);
}

// Entries 64 blockIdx.x .. + 63 to their places (256 threads; sort_keys: n words of LDS).
template <class Src, class Sink>
__device__ __forceinline__ void rank_sort(const Src& src, const Sink& sink, int n, uint64_t* sort_keys) {
    __shared__ int part[4][64];
    for (int t = threadIdx.x; t < n; t += 256) sort_keys[t] = src(t);
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int item = (int)blockIdx.x * 64 + lane;
    const uint64_t k = item < n ? sort_keys[item] : 0;
    const int q = (n + 3) / 4, lo = wave * q, hi = min(n, lo + q);
    int before = 0;
#pragma unroll 8
    for (int u = lo; u < hi; ++u) {
        const uint64_t x = sort_keys[u];
        before += (x < k || (x == k && u < item)) ? 1 : 0;
    }
    part[wave][lane] = before;
    __syncthreads();
    if (wave == 0 && item < n) sink(part[0][lane] + part[1][lane] + part[2][lane] + part[3][lane], item, k);
}

template <class Src, class Sink>
__global__ __launch_bounds__(256) void k_rank_sort(Src src, Sink sink, int n) {
    extern __shared__ uint64_t sort_keys[];
    rank_sort(src, sink, n, sort_keys);
}

// Several sorts of up to RANK_SORT_MAX entries in one launch: the job is the
// workgroup's y index.
template <class Src, class Sink>
struct RankJob {
    Src src;
    Sink sink;
    int32_t n;
};

template <class Src, class Sink>
__global__ __launch_bounds__(256) void k_rank_sort_many(const RankJob<Src, Sink>* __restrict__ jobs) {
    extern __shared__ uint64_t sort_keys[];
    const RankJob<Src, Sink> j = jobs[blockIdx.y];
    if ((int)blockIdx.x * 64 < j.n) rank_sort(j.src, j.sink, j.n, sort_keys);
}

// counts[tile * bins + d]: entries of the tile whose digit is d
template <class Src>
__global__ __launch_bounds__(RADIX_THREADS) void k_radix_count(Src src, const int32_t* __restrict__ perm, int64_t n,
                                                               int64_t tile, int shift, int digit,
                                                               int32_t* __restrict__ counts) {
    extern __shared__ int32_t radix_lds[];
    const int bins = 1 << digit;
    for (int d = threadIdx.x; d < bins; d += RADIX_THREADS) radix_lds[d] = 0;
    __syncthreads();
    const int64_t t0 = (int64_t)blockIdx.x * tile, t1 = min(n, t0 + tile);
    for (int64_t t = t0 + threadIdx.x; t < t1; t += RADIX_THREADS) {
        const int32_t i = perm ? perm[t] : (int32_t)t;
        atomicAdd(&radix_lds[(int)(src(i) >> shift) & (bins - 1)], 1);
    }
    __syncthreads();
    int32_t* out = counts + (int64_t)blockIdx.x * bins;
    for (int d = threadIdx.x; d < bins; d += RADIX_THREADS) out[d] = radix_lds[d];
}

// Lane = one digit, the tiles split over the workgroup's waves: counts become
// their exclusive prefix over the tiles, totals[d] the digit's entries.
static __global__ __launch_bounds__(1024) void k_radix_scan(int32_t* __restrict__ counts,
                                                            int32_t* __restrict__ totals, int bins, int tiles) {
    __shared__ int32_t sums[16][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int d = (int)blockIdx.x * 64 + lane;
    const int per = (tiles + 15) / 16, a = min(tiles, wave * per), b = min(tiles, a + per);
    int32_t s = 0;
    if (d < bins) {
#pragma unroll 8
        for (int t = a; t < b; ++t) s += counts[(int64_t)t * bins + d];
    }
    sums[wave][lane] = s;
    __syncthreads();
    if (d >= bins) return;
    int32_t run = 0, all = 0;
    for (int w = 0; w < 16; ++w) {
        if (w < wave) run += sums[w][lane];
        all += sums[w][lane];
    }
    if (wave == 0) totals[d] = all;
#pragma unroll 8
    for (int t = a; t < b; ++t) {
        const int32_t c = counts[(int64_t)t * bins + d];
        counts[(int64_t)t * bins + d] = run;
        run += c;
    }
}

// A wave takes a contiguous quarter of the tile, 64 entries at a time: lanes
// of one digit find each other with a ballot per bit, the lowest claims their
// places from the wave's counter, so equal digits keep their order.
template <class Src, class Sink>
__global__ __launch_bounds__(RADIX_THREADS) void k_radix_scatter(Src src, Sink sink, const int32_t* __restrict__ perm,
                                                                 int32_t* __restrict__ perm_out, int64_t n,
                                                                 int64_t tile, int shift, int digit,
                                                                 const int32_t* __restrict__ counts,
                                                                 const int32_t* __restrict__ totals) {
    extern __shared__ int32_t radix_lds[];   // RADIX_WAVES x bins: each wave's next place per digit; two rows of
    __shared__ int32_t wsum[RADIX_WAVES];    // bins: the digits' totals and their entries in the tiles before
    const int bins = 1 << digit;
    int32_t* tot = radix_lds + RADIX_WAVES * bins;
    int32_t* prior = tot + bins;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t t0 = (int64_t)blockIdx.x * tile, quarter = tile / RADIX_WAVES;
    const int64_t w0 = min(n, t0 + wave * quarter), w1 = min(n, w0 + quarter);
    for (int d = threadIdx.x; d < RADIX_WAVES * bins; d += RADIX_THREADS) radix_lds[d] = 0;
    for (int d = threadIdx.x; d < bins; d += RADIX_THREADS) {
        tot[d] = totals[d];
        prior[d] = counts[(int64_t)blockIdx.x * bins + d];
    }
    __syncthreads();
    int32_t* mine = radix_lds + wave * bins;
    for (int64_t t = w0 + lane; t < w1; t += 64) {
        const int32_t i = perm ? perm[t] : (int32_t)t;
        atomicAdd(&mine[(int)(src(i) >> shift) & (bins - 1)], 1);
    }
    __syncthreads();
    // first place of every digit: the exclusive scan of the totals (each
    // thread a run of digits), the tiles before, the waves before
    const int per = (bins + RADIX_THREADS - 1) / RADIX_THREADS;
    const int d0 = min(bins, (int)threadIdx.x * per), d1 = min(bins, d0 + per);
    int32_t sum = 0;
    for (int d = d0; d < d1; ++d) sum += tot[d];
    int32_t x = sum;
#pragma unroll
    for (int k = 1; k < 64; k <<= 1) {
        const int32_t y = __shfl_up(x, k, 64);
        if (lane >= k) x += y;
    }
    if (lane == 63) wsum[wave] = x;
    __syncthreads();
    int32_t run = x - sum;
    for (int w = 0; w < wave; ++w) run += wsum[w];
    for (int d = d0; d < d1; ++d) {
        int32_t at = run + prior[d];
#pragma unroll
        for (int w = 0; w < RADIX_WAVES; ++w) {
            const int32_t c = radix_lds[w * bins + d];
            radix_lds[w * bins + d] = at;
            at += c;
        }
        run += tot[d];
    }
    __syncthreads();
    for (int64_t base = w0; base < w1; base += 64) {
        const int64_t t = base + lane;
        const bool in = t < w1;
        const int32_t i = in ? (perm ? perm[t] : (int32_t)t) : 0;
        const uint64_t k = in ? src(i) : 0;
        const int d = (int)(k >> shift) & (bins - 1);
        uint64_t same = __ballot(in);
        for (int b = 0; b < digit; ++b) {
            const bool bit = (d >> b) & 1;
            const uint64_t m = __ballot(in && bit);
            same &= bit ? m : ~m;
        }
        const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
        const int leader = in ? __ffsll((unsigned long long)same) - 1 : lane;
        int32_t first = 0;
        if (in && lane == leader) first = atomicAdd(&mine[d], (int32_t)__popcll(same));
        first = __shfl(first, leader, 64);
        const int32_t to = first + (int32_t)__popcll(same & below);
        if (!in) continue;
        if (perm_out)
            perm_out[to] = i;
        else
            sink(to, i, k);
    }
}

// Sorts entries 0 .. n-1 (n < 2^31) by the low key_bits bits of src, stably.
// tmp: sort_tmp_words(n, key_bits) words; perm: n words, overwritten (the sink
// may write them in turn: the last pass does not read them).
template <class Src, class Sink>
void stable_sort(const Src& src, const Sink& sink, int64_t n, int key_bits, int32_t* tmp, int32_t* perm,
                 hipStream_t s) {
    if (n <= 0) return;
    if (n <= RANK_SORT_MAX) {
        k_rank_sort<Src, Sink><<<(unsigned)((n + 63) / 64), 256, n * sizeof(uint64_t), s>>>(src, sink, (int)n);
        QT_LAUNCH("k_rank_sort");
        return;
    }
    const RadixPlan p = radix_plan(n, key_bits);
    const int bins = p.bins();
    int32_t* counts = tmp;
    int32_t* totals = counts + (size_t)bins * p.tiles;
    int32_t* other = totals + bins;
    const int32_t* in = nullptr;
    for (int pass = 0; pass < p.passes; ++pass) {
        const int shift = pass * p.digit;
        // alternating so that the last pass reads `other`
        int32_t* out = pass + 1 == p.passes ? nullptr : ((p.passes - pass) & 1) ? perm : other;
        k_radix_count<Src><<<(unsigned)p.tiles, RADIX_THREADS, bins * sizeof(int32_t), s>>>(src, in, n, p.tile, shift,
                                                                                          p.digit, counts);
        QT_LAUNCH("k_radix_count");
        k_radix_scan<<<(unsigned)((bins + 63) / 64), 1024, 0, s>>>(counts, totals, bins, (int)p.tiles);
        QT_LAUNCH("k_radix_scan");
        k_radix_scatter<Src, Sink><<<(unsigned)p.tiles, RADIX_THREADS, (RADIX_WAVES + 2) * bins * sizeof(int32_t), s>>>(
            src, sink, in, out, n, p.tile, shift, p.digit, counts, totals);
        QT_LAUNCH("k_radix_scatter");
        in = out;
    }
}

}  // namespace qt
