// Building a quadtree matrix from a block list, copying it back out, and the
// derived operand forms (fp32 copy, bf16 hi/lo split) and count histograms.
//
// Representation (Sec. 3.1 and 4.1 of the paper): blocks sorted by Morton
// key, so every quadtree node covers a contiguous run; leaves are lb x lb
// block grids stored as three 64-bit occupancy masks plus the index of their
// first block; every level above holds a 4-entry child table per node, -1
// marking a NIL child. Nodes carry no global offsets, only their Morton key.
#include "qt_internal.h"
#include "qt_morton.h"
#include "qt_readback.h"
#include "qt_sort.h"

#include <algorithm>
#include <map>
#include <mutex>
#include <atomic>
#include <set>

namespace qt {

// ------------------------------------------------------------ allocation

static std::mutex g_pool_mu;
static std::set<int> g_pool_ready;

static void ensure_pool() {
    int dev = 0;
    QT_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_pool_mu);
    if (g_pool_ready.count(dev)) return;
    hipMemPool_t pool;
    QT_HIP(hipDeviceGetDefaultMemPool(&pool, dev));
    uint64_t thr = ~0ull;
    QT_HIP(hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &thr));
    // The pool takes any wait of stream X for an event of stream A, however old the
    // event, as leave to hand X what was freed on A since, work on A or not.
    int no = 0;
    QT_HIP(hipMemPoolSetAttribute(pool, hipMemPoolReuseFollowEventDependencies, &no));
    g_pool_ready.insert(dev);
}

static std::atomic<const Allocator*> g_allocator{nullptr};

const Allocator* current_allocator() { return g_allocator.load(std::memory_order_acquire); }

void set_allocator(const Allocator* a) { g_allocator.store(a, std::memory_order_release); }

// Memory made on one stream and released on another. The pool hands memory freed
// on a stream to the stream it was made on at once, whatever still runs on the
// first: the next traversal would write its lists where the numeric kernel reads
// them. So it goes back to the pool once an event recorded at its release has
// been passed: looked at with every allocation, and on that allocation's stream,
// as the one that it was made on may be a caller's that is gone by then.
struct Parked {
    void* p;
    hipEvent_t passed;
};
static std::mutex g_park_mu;
static std::map<int, std::vector<Parked>> g_parked;       // per device
static std::map<int, std::vector<hipEvent_t>> g_park_ev;  // for reuse

static bool capturing(hipStream_t s) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) == hipSuccess) return st != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

// wait: until all of it is passed. Not while s is captured: it would go back at
// every replay.
static void unpark(int dev, hipStream_t s, bool wait) {
    std::lock_guard<std::mutex> lk(g_park_mu);
    auto& list = g_parked[dev];
    if (list.empty() || capturing(s)) return;
    size_t kept = 0;
    for (const Parked& k : list) {
        if ((wait ? hipEventSynchronize(k.passed) : hipEventQuery(k.passed)) == hipSuccess) {
            (void)hipFreeAsync(k.p, s);
            g_park_ev[dev].push_back(k.passed);
        } else {
            (void)hipGetLastError();
            list[kept++] = k;
        }
    }
    list.resize(kept);
}

// Called by destructors: whatever cannot be had, the memory is waited for here.
// An event of a stream that is captured never reads as passed: a release in the
// capture is the graph's.
static void park(void* p, hipStream_t s) noexcept {
    hipEvent_t e = nullptr;
    if (capturing(s)) {
        (void)hipFreeAsync(p, s);
        return;
    }
    try {
        int dev = 0;
        QT_HIP(hipGetDevice(&dev));
        {
            std::lock_guard<std::mutex> lk(g_park_mu);
            auto& events = g_park_ev[dev];
            if (!events.empty()) {
                e = events.back();
                events.pop_back();
            }
        }
        if (!e) QT_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
        QT_HIP(hipEventRecord(e, s));
        std::lock_guard<std::mutex> lk(g_park_mu);
        g_parked[dev].push_back(Parked{p, e});
    } catch (...) {
        (void)hipGetLastError();
        (void)hipDeviceSynchronize();
        (void)hipFreeAsync(p, s);
        if (e) (void)hipEventDestroy(e);
    }
}

void* dev_alloc(size_t bytes, hipStream_t s, const Allocator** who) {
    const Allocator* a = current_allocator();
    *who = a;
    void* p = nullptr;
    if (a) {
        p = a->alloc(bytes, (void*)s, a->ctx);
        if (!p) fail(QT_ERR_OOM, "the installed allocator returned no memory");
        if (reinterpret_cast<uintptr_t>(p) & 255) {
            a->free_(p, (void*)s, a->ctx);
            fail(QT_ERR_DEVICE, "the installed allocator returned memory not aligned to 256 bytes");
        }
        return p;
    }
    ensure_pool();
    int dev = 0;
    QT_HIP(hipGetDevice(&dev));
    unpark(dev, s, false);
    hipError_t e = hipMallocAsync(&p, bytes, s);
    if (e == hipErrorOutOfMemory) {   // what is parked may be what is missing
        (void)hipGetLastError();
        unpark(dev, s, true);
        e = hipMallocAsync(&p, bytes, s);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        hip_check(e, "hipMallocAsync");
    }
    return p;
}

void dev_free(void* p, hipStream_t s, hipStream_t made, const Allocator* who) {
    if (!p) return;
    if (who)
        who->free_(p, (void*)s, who->ctx);
    else if (s == made)
        (void)hipFreeAsync(p, s);
    else
        park(p, s);
}

// --------------------------------------------------------------- kernels

__global__ void k_fill_i32(int32_t* p, int64_t n, int32_t v) {
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step) p[i] = v;
}

// fn(first, count) over 0 .. n-1 in runs of at most 2^30 threads, `each` an item
// (a grid of 2^32 threads or more is launched in part, without an error).
template <class F>
static void in_launches(int64_t n, int64_t each, const F& fn) {
    const int64_t most = (int64_t(1) << 30) / each;
    for (int64_t at = 0; at < n; at += most) fn(at, std::min(n - at, most));
}

// Sort sources and sinks (see qt_sort.h). A block list's entry t sorts by the
// Morton key of (I[t], J[t]); one out of range sets the error flag.
struct ListKeys {
    const int32_t* I;
    const int32_t* J;
    int64_t nbr, nbc;
    int32_t* err;
    __device__ uint64_t operator()(int32_t t) const {
        const int32_t i = I[t], j = J[t];
        if (i < 0 || j < 0 || i >= nbr || j >= nbc) {
            atomicOr(err, 1);
            return 0;   // a position of any grid build() accepts: the tree is formed before the flag is read
        }
        return morton_key((uint32_t)i, (uint32_t)j);
    }
};

struct KeyPermSink {
    uint64_t* keys;
    int32_t* perm;
    __device__ void operator()(int32_t at, int32_t t, uint64_t k) const {
        keys[at] = k;
        perm[at] = t;
    }
};

// Blocks in Morton order come out row-major when sorted by row alone: the
// sort is stable, and Morton order lists the blocks of one row by column.
struct RowKeys {
    const uint64_t* bkey;
    __device__ uint64_t operator()(int32_t t) const { return morton_row(bkey[t]); }
};

// Row-major copy-out: source block of every output position.
struct PermSink {
    int32_t* perm;
    __device__ void operator()(int32_t at, int32_t t, uint64_t) const { perm[at] = t; }
};

struct GatherF64Sink {
    const double* src;
    double* dst;
    __device__ void operator()(int32_t at, int32_t t, uint64_t) const { dst[at] = src[t]; }
};

// Squared norms by their bit pattern (non-negative doubles order like it).
struct NormKeys {
    const double* norm2;
    __device__ uint64_t operator()(int32_t t) const { return (uint64_t)__double_as_longlong(norm2[t]); }
};

struct NormSink {
    double* sorted;
    int32_t* idx;
    __device__ void operator()(int32_t at, int32_t t, uint64_t k) const {
        sorted[at] = __longlong_as_double((long long)k);
        idx[at] = t;
    }
};

// Blocks copied in permuted order: dst block t = src block perm[t], converted
// (fp64 to fp32 rounds to nearest even). A wave moves COPY_PIECES pieces of
// 64 x VE consecutive entries, all of its loads issued before its stores, VE
// entries (16 bytes of the wider type or more) per lane. Bound by HBM; what it
// needs is bytes in flight: with one entry per lane and load, a workgroup per
// block, the 440 k fp32 blocks of a random 48000 product moved at 3.6 TB/s
// (read + written, beside the next traversal) where this reaches 5.1, 890 k
// fp64 blocks of b = 16 at 3.1 where this reaches 6.1. VE = 1 is for a caller's array that
// is not aligned to 16 bytes.
constexpr int COPY_PIECES = 4, COPY_WAVES = 4;

// VE entries as a copy reads and writes them: 16 bytes at an address that is
// aligned to that, also where the vector itself is longer (four doubles).
constexpr size_t COPY_ALIGN = 16;
template <class T, int VE>
struct CopyVec {
    static constexpr size_t align = sizeof(T) * VE < COPY_ALIGN ? sizeof(T) * VE : COPY_ALIGN;
    typedef T type __attribute__((ext_vector_type(VE), aligned(align)));
    static_assert(alignof(type) == align, "the alignment that copy_aligned checks");
};

static bool copy_aligned(const void* src, const void* dst) {
    return ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & (COPY_ALIGN - 1)) == 0;
}

// Where a copy-out writes its blocks' coordinates (I NULL: nowhere), and the
// blocks' keys.
struct Coords {
    const uint64_t* bkey;
    int32_t* I;
    int32_t* J;
    __device__ void operator()(int64_t at, int32_t t) const {
        const uint64_t key = bkey[t];
        I[at] = (int32_t)morton_row(key);
        J[at] = (int32_t)morton_col(key);
    }
};

template <class S, class D, int VE>
__global__ __launch_bounds__(64 * COPY_WAVES) void k_copy_blocks(const S* __restrict__ src,
                                                                 const int32_t* __restrict__ perm, int64_t pieces,
                                                                 int ppb_log, D* __restrict__ dst, Coords coords) {
    typedef typename CopyVec<S, VE>::type svec;
    typedef typename CopyVec<D, VE>::type dvec;
    const int lane = threadIdx.x & 63;
    const int64_t p0 = ((int64_t)blockIdx.x * COPY_WAVES + (threadIdx.x >> 6)) * COPY_PIECES;
    svec v[COPY_PIECES];
#pragma unroll
    for (int r = 0; r < COPY_PIECES; ++r) {
        const int64_t p = p0 + r;
        if (p >= pieces) break;
        const int64_t at = ((int64_t)perm[p >> ppb_log] << ppb_log) + (p & ((int64_t(1) << ppb_log) - 1));
        v[r] = __builtin_nontemporal_load(reinterpret_cast<const svec*>(src) + at * 64 + lane);
    }
#pragma unroll
    for (int r = 0; r < COPY_PIECES; ++r) {
        const int64_t p = p0 + r;
        if (p >= pieces) break;
        __builtin_nontemporal_store(__builtin_convertvector(v[r], dvec), reinterpret_cast<dvec*>(dst) + p * 64 + lane);
    }
    if (coords.I && lane < COPY_PIECES) {
        const int64_t p = p0 + lane;
        if (p < pieces && (p & ((int64_t(1) << ppb_log) - 1)) == 0) coords(p >> ppb_log, perm[p >> ppb_log]);
    }
}

__global__ void k_coords(const int32_t* __restrict__ perm, int64_t n, Coords coords) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) coords(t, perm[t]);
}

template <class S, class D, int VE>
static void launch_copy_blocks(const S* src, const int32_t* perm, int64_t n, int bb, D* dst, hipStream_t s,
                               const Coords& coords) {
    int ppb_log = 0;   // b is 16, 32 or 64: a power of two of pieces per block
    while (((64 * VE) << ppb_log) < bb) ++ppb_log;
    // 16 threads per piece: 69 GB of fp32, an entry per lane, are 2^32
    constexpr int64_t per = COPY_WAVES * COPY_PIECES;
    in_launches(n, (64 * COPY_WAVES / per) << ppb_log, [&](int64_t at, int64_t m) {
        const Coords here{coords.bkey, coords.I ? coords.I + at : nullptr, coords.J ? coords.J + at : nullptr};
        const int64_t pieces = m << ppb_log;
        k_copy_blocks<S, D, VE><<<(unsigned)((pieces + per - 1) / per), 64 * COPY_WAVES, 0, s>>>(
            src, perm + at, pieces, ppb_log, dst + at * bb, here);
        QT_LAUNCH("k_copy_blocks");
    });
}

// src and dst: device arrays of n blocks of bb entries; perm: n entries.
template <class S, class D>
static void copy_blocks(const S* src, const int32_t* perm, int64_t n, int bb, D* dst, hipStream_t s,
                        const Coords& coords = Coords{}) {
    constexpr int VE = (sizeof(S) == 8 && sizeof(D) == 8) ? 2 : 4;
    if (copy_aligned(src, dst))
        launch_copy_blocks<S, D, VE>(src, perm, n, bb, dst, s, coords);
    else
        launch_copy_blocks<S, D, 1>(src, perm, n, bb, dst, s, coords);
}

// Row-major copy-out of few blocks in one launch, without a permutation: a
// workgroup per block finds the block's place itself, the number of blocks in
// rows above and before it in its own (in Morton order a row's blocks lie by
// column), and copies it there. Bound by latency and, towards RANKED_MAX, by the
// n^2 keys read from the caches. Copies in a loop, sort and copy against this, in
// us: b = 16, 9 to 374 blocks 11.6 and 7.9, 2000 20 and 7.7, 4000 37 and 18; b = 32,
// 2000 24 and 8.7; b = 64, 2000 40 and 25, 4000 77 and 53. Beyond, the radix sort
// is ahead: b = 16, 4500 17.6 and 21.9, 8000 20 and 61; b = 64, 4500 63 and 61,
// 6000 79 and 87.
constexpr int64_t RANKED_MAX = 4096;

template <class S, class D, int VE>
__global__ __launch_bounds__(256) void k_copy_ranked(const uint64_t* __restrict__ bkey, int32_t n,
                                                     const S* __restrict__ src, int bb, int32_t* __restrict__ I,
                                                     int32_t* __restrict__ J, D* __restrict__ dst) {
    typedef typename CopyVec<S, VE>::type svec;
    typedef typename CopyVec<D, VE>::type dvec;
    constexpr int U = 4;
    __shared__ int before[4];
    const int tid = threadIdx.x, wave = tid >> 6;
    const int32_t t = (int32_t)blockIdx.x;
    const uint64_t key = bkey[t];
    const int32_t row = (int32_t)morton_row(key);
    const svec* from = reinterpret_cast<const svec*>(src + (size_t)t * bb);
    const int m = dst ? bb / VE : 0;
    svec v[U];                       // the first vectors, on their way while the place is found
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (tid + 256 * u < m) v[u] = __builtin_nontemporal_load(from + tid + 256 * u);
    int c = 0;
    for (int32_t i = tid; i < n; i += 256) {
        const int32_t r = (int32_t)morton_row(bkey[i]);
        c += r < row || (r == row && i < t);
    }
    for (int d = 32; d > 0; d >>= 1) c += __shfl_xor(c, d, 64);
    if ((tid & 63) == 0) before[wave] = c;
    __syncthreads();
    const int64_t at = before[0] + before[1] + before[2] + before[3];
    if (tid == 0) {
        I[at] = row;
        J[at] = (int32_t)morton_col(key);
    }
    dvec* to = reinterpret_cast<dvec*>(dst + at * bb);
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (tid + 256 * u < m) __builtin_nontemporal_store(__builtin_convertvector(v[u], dvec), to + tid + 256 * u);
    for (int e = tid + 256 * U; e < m; e += 256)
        __builtin_nontemporal_store(__builtin_convertvector(__builtin_nontemporal_load(from + e), dvec), to + e);
}

// src and dst: device arrays of n blocks of bb entries in C's order and in
// row-major order (dst may be NULL).
template <class S, class D>
static void copy_ranked(const uint64_t* bkey, const S* src, int64_t n, int bb, int32_t* I, int32_t* J, D* dst,
                        hipStream_t s) {
    constexpr int VE = (sizeof(S) == 8 && sizeof(D) == 8) ? 2 : 4;
    if (copy_aligned(src, dst))
        k_copy_ranked<S, D, VE><<<(unsigned)n, 256, 0, s>>>(bkey, (int32_t)n, src, bb, I, J, dst);
    else
        k_copy_ranked<S, D, 1><<<(unsigned)n, 256, 0, s>>>(bkey, (int32_t)n, src, bb, I, J, dst);
    QT_LAUNCH("k_copy_ranked");
}

// The quadtree over n blocks from their ascending Morton keys. A block starts
// a node of level l when its key's prefix above that level differs from the
// block's before it, so it starts nodes of every level from some first one
// down (L: the leaves); node numbers are ranks of those starts.
//   init:  clears the read-back words and the histograms, and marks every
//          child NIL;
//   tiles: the starts of every level per tile of blocks (and equal
//          neighbours: the same block twice);
//   scan:  k_radix_scan over the tiles, a lane per level, whose totals are the
//          levels' node counts;
//   fill:  ranks within the tile from ballots, then every level's keys and
//          child links, the leaves' masks, and the node and block counts per
//          row and column.
// The tables are placed by bounds on the levels' node counts, so the host
// waits once, for the counts and histograms together. Bound by that chain of
// dependent launches: with the counts read back first, a flag per block and
// level, a scan of them all and a histogram launch per level, three waits and
// 25 launches, build and copy-out of 29300 blocks took 437 us, now 278.
constexpr int MAX_TREE_LEVELS = 32;
constexpr int TREE_THREADS = 256, TREE_WAVES = TREE_THREADS / 64;
constexpr int64_t TREE_TILES_MAX = 2048;

struct TreeBuild {
    const uint64_t* keys;
    const int32_t* n;                      // number of blocks (device)
    int L, lb_log;
    int64_t tile;                          // blocks per workgroup
    int32_t* starts;                       // per tile and level
    int32_t* err;
    int32_t* child[MAX_TREE_LEVELS];       // levels 0 .. L-1: 4 per node
    uint64_t* key[MAX_TREE_LEVELS];
    int32_t* base;                         // leaves
    uint64_t* lkey;
    uint64_t* mo;
    uint64_t* rm;
    uint64_t* cm;
    int32_t* hist;                         // levels 0 .. L, then blocks: counts per row, per column
};

// words[at] = n, the others 0; nil[..] = -1
__global__ void k_tree_init(int32_t* words, int64_t nwords, int64_t at, int32_t n, int32_t* nil, int64_t nnil) {
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t i = i0; i < nwords; i += step) words[i] = i == at ? n : 0;
    for (int64_t i = i0; i < nnil; i += step) nil[i] = -1;
}

// First level of which block t (key k, kp the key before it) starts a node;
// L + 1: none.
__device__ __forceinline__ int first_level(int64_t t, uint64_t k, uint64_t kp, int L, int lb_log) {
    if (t == 0) return 0;
    const uint64_t d = k ^ kp;
    if ((d >> (2 * lb_log)) == 0) return L + 1;
    const int depth = (63 - __clzll((long long)d) - 2 * lb_log) >> 1;   // levels above the leaves
    return depth >= L ? 0 : L - depth;
}

__global__ __launch_bounds__(TREE_THREADS) void k_tree_tiles(TreeBuild b) {
    __shared__ int32_t cnt[MAX_TREE_LEVELS + 1];
    const int64_t n = *b.n, t0 = (int64_t)blockIdx.x * b.tile;
    if ((int)threadIdx.x <= b.L) cnt[threadIdx.x] = 0;
    __syncthreads();
    bool dup = false;
    for (int64_t base = t0; base < t0 + b.tile; base += TREE_THREADS) {
        const int64_t t = base + threadIdx.x;
        int f = b.L + 1;
        if (t < n) {
            const uint64_t k = b.keys[t], kp = t > 0 ? b.keys[t - 1] : 0;
            dup = dup || (t > 0 && k == kp);
            f = first_level(t, k, kp, b.L, b.lb_log);
        }
        for (int l = 0; l <= b.L; ++l) {
            const uint64_t m = __ballot(f <= l);
            if ((threadIdx.x & 63) == 0 && m) atomicAdd(&cnt[l], (int32_t)__popcll(m));
        }
    }
    if (dup) atomicOr(b.err, 2);
    __syncthreads();
    if ((int)threadIdx.x <= b.L) b.starts[(int64_t)blockIdx.x * (b.L + 1) + threadIdx.x] = cnt[threadIdx.x];
}

__global__ __launch_bounds__(TREE_THREADS) void k_tree_tables(TreeBuild b) {
    __shared__ int32_t before[MAX_TREE_LEVELS + 1];                 // starts before this round of blocks
    __shared__ int32_t wcnt[TREE_WAVES][MAX_TREE_LEVELS + 1];
    const int64_t n = *b.n, t0 = (int64_t)blockIdx.x * b.tile;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int L = b.L, leaf_shift = 2 * b.lb_log;
    if ((int)threadIdx.x <= L) before[threadIdx.x] = b.starts[(int64_t)blockIdx.x * (L + 1) + threadIdx.x];
    const uint64_t upto = ~0ull >> (63 - lane);
    for (int64_t base = t0; base < t0 + b.tile && base < n; base += TREE_THREADS) {
        const int64_t t = base + threadIdx.x;
        uint64_t k = 0;
        int f = L + 1;
        if (t < n) {
            k = b.keys[t];
            f = first_level(t, k, t > 0 ? b.keys[t - 1] : 0, L, b.lb_log);
        }
        for (int l = 0; l <= L; ++l) {
            const uint64_t m = __ballot(f <= l);
            if (lane == 0) wcnt[wave][l] = (int32_t)__popcll(m);
        }
        __syncthreads();
        int32_t up = 0;              // this block's node one level up
        int32_t* hist = b.hist;
        for (int l = 0; l <= L; ++l) {
            int32_t r = before[l] + (int32_t)__popcll(__ballot(f <= l) & upto) - 1;
            for (int w = 0; w < wave; ++w) r += wcnt[w][l];
            const int64_t side = int64_t(1) << l;
            if (f <= l) {
                const uint64_t nk = k >> (leaf_shift + 2 * (L - l));
                (l < L ? b.key[l] : b.lkey)[r] = nk;
                if (l > 0) b.child[l - 1][4 * (int64_t)up + (int)(nk & 3)] = r;
                atomicAdd(hist + morton_row(nk), 1);
                atomicAdd(hist + side + morton_col(nk), 1);
                if (l == L) {
                    // the leaf's blocks: eight keys at a time, so that their loads overlap;
                    // no further than a leaf can hold, as a list that is about to be
                    // refused may repeat one key (300 k times: 20.7 ms a call, now 4.0)
                    const int64_t full = t + (int64_t(1) << leaf_shift);
                    uint64_t mo = 0;
                    bool more = true;
                    for (int64_t u = t; more && u < full; u += 8) {
                        uint64_t x[8];
#pragma unroll
                        for (int e = 0; e < 8; ++e) x[e] = u + e < n ? b.keys[u + e] : ~nk << leaf_shift;
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            more = more && (x[e] >> leaf_shift) == nk;
                            if (more) mo |= 1ull << (x[e] & ((1ull << leaf_shift) - 1));
                        }
                    }
                    const uint64_t rm = morton_to_rowmajor(mo, b.lb_log);
                    b.base[r] = (int32_t)t;
                    b.mo[r] = mo;
                    b.rm[r] = rm;
                    b.cm[r] = rowmajor_to_colmajor(rm, b.lb_log);
                }
            }
            up = r;
            hist += 2 * side;
        }
        if (t < n) {
            atomicAdd(hist + morton_row(k), 1);
            atomicAdd(hist + ((int64_t)(1 << b.lb_log) << L) + morton_col(k), 1);
        }
        __syncthreads();
        if ((int)threadIdx.x <= L)
            for (int w = 0; w < TREE_WAVES; ++w) before[threadIdx.x] += wcnt[w][threadIdx.x];
        __syncthreads();
    }
}

__global__ void k_hist(const uint64_t* __restrict__ keys, int64_t n, int32_t* __restrict__ rowcnt,
                       int32_t* __restrict__ colcnt) {
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    uint64_t k = keys[t];
    atomicAdd(rowcnt + morton_row(k), 1);
    atomicAdd(colcnt + morton_col(k), 1);
}

__global__ void k_f64_to_f32(const double* __restrict__ s, int64_t n, float* __restrict__ d) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) d[i] = __double2float_rn(s[i]);
}

__global__ void k_f32_to_f64(const float* __restrict__ s, int64_t n, double* __restrict__ d) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) d[i] = (double)s[i];
}

// Round a binary32 value to bfloat16, nearest even, on the bit pattern.
__device__ inline uint16_t bf16_round(float x) {
    uint32_t u = __float_as_uint(x);
    if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu)) return (uint16_t)((u >> 16) | 0x40);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ inline float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// hi = bf16(a32), lo = bf16(a32 - hi) per entry, row-major and transposed.
template <class T>
__global__ void k_bf16_split(const T* __restrict__ src, int64_t nblk, int b, uint16_t* __restrict__ hi,
                             uint16_t* __restrict__ lo, uint16_t* __restrict__ hi_t, uint16_t* __restrict__ lo_t) {
    const int64_t bb = (int64_t)b * b;
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nblk * bb) return;
    float a = (float)src[i];   // fp64 -> fp32 rounds to nearest even
    uint16_t h = bf16_round(a);
    uint16_t l = bf16_round(a - bf16_to_f32(h));
    int64_t t = i / bb;
    int e = (int)(i - t * bb);
    int r = e / b, c = e - r * b;
    hi[i] = h;
    lo[i] = l;
    hi_t[t * bb + (int64_t)c * b + r] = h;
    lo_t[t * bb + (int64_t)c * b + r] = l;
}

// One workgroup per requested block: binary search of its Morton key, then
// a copy (or zeros when the block is not stored).
template <class S, class D>
__global__ void k_get_blocks(const uint64_t* __restrict__ bkey, int64_t nblocks, int64_t nbr, int64_t nbc,
                             const S* __restrict__ vals, const int32_t* __restrict__ I,
                             const int32_t* __restrict__ J, int64_t count, int bb, D* __restrict__ out,
                             int32_t* __restrict__ found) {
    __shared__ int64_t pos;
    for (int64_t t = blockIdx.x; t < count; t += gridDim.x) {
        if (threadIdx.x == 0) {
            int64_t at = -1;
            const int32_t i = I[t], j = J[t];
            if (i >= 0 && j >= 0 && i < nbr && j < nbc) {
                const uint64_t k = morton_key((uint32_t)i, (uint32_t)j);
                int64_t lo = 0, hi = nblocks;           // first index with bkey >= k
                while (lo < hi) {
                    const int64_t mid = (lo + hi) >> 1;
                    if (bkey[mid] < k) lo = mid + 1; else hi = mid;
                }
                if (lo < nblocks && bkey[lo] == k) at = lo;
            }
            pos = at;
            found[t] = at >= 0 ? 1 : 0;
        }
        __syncthreads();
        const int64_t at = pos;
        D* d = out + (size_t)t * bb;
        if (at >= 0) {
            const S* src = vals + (size_t)at * bb;
            for (int e = threadIdx.x; e < bb; e += blockDim.x) d[e] = (D)src[e];
        } else {
            for (int e = threadIdx.x; e < bb; e += blockDim.x) d[e] = (D)0;
        }
        __syncthreads();
    }
}

template <>
__global__ void k_get_blocks<double, float>(const uint64_t* __restrict__ bkey, int64_t nblocks, int64_t nbr,
                                            int64_t nbc, const double* __restrict__ vals,
                                            const int32_t* __restrict__ I, const int32_t* __restrict__ J,
                                            int64_t count, int bb, float* __restrict__ out,
                                            int32_t* __restrict__ found) {
    __shared__ int64_t pos;
    for (int64_t t = blockIdx.x; t < count; t += gridDim.x) {
        if (threadIdx.x == 0) {
            int64_t at = -1;
            const int32_t i = I[t], j = J[t];
            if (i >= 0 && j >= 0 && i < nbr && j < nbc) {
                const uint64_t k = morton_key((uint32_t)i, (uint32_t)j);
                int64_t lo = 0, hi = nblocks;
                while (lo < hi) {
                    const int64_t mid = (lo + hi) >> 1;
                    if (bkey[mid] < k) lo = mid + 1; else hi = mid;
                }
                if (lo < nblocks && bkey[lo] == k) at = lo;
            }
            pos = at;
            found[t] = at >= 0 ? 1 : 0;
        }
        __syncthreads();
        const int64_t at = pos;
        float* d = out + (size_t)t * bb;
        if (at >= 0) {
            const double* src = vals + (size_t)at * bb;
            for (int e = threadIdx.x; e < bb; e += blockDim.x) d[e] = __double2float_rn(src[e]);
        } else {
            for (int e = threadIdx.x; e < bb; e += blockDim.x) d[e] = 0.f;
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------- helpers

static inline unsigned grid_for(int64_t n, int T = 256) {
    int64_t g = (n + T - 1) / T;
    return (unsigned)std::max<int64_t>(g, 1);
}

static inline unsigned block_grid(int64_t n) {
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(n, 1 << 20));
}

static int ilog2(int64_t x) {
    int l = 0;
    while ((int64_t(1) << l) < x) ++l;
    return l;
}

// ------------------------------------------------------------ histograms

// The counts of M as the device makes them: per level 0 .. L the nodes per row
// and per column, then the blocks per row and per column of the padded grid.
static int64_t histogram_words(const qt_matrix* M) {
    int64_t total = 2 * ((int64_t)M->lb << M->L);
    for (int l = 0; l <= M->L; ++l) total += 2 * (int64_t(1) << l);
    return total;
}

static void adopt_histograms(qt_matrix* M, const int32_t* w) {
    Histograms h;
    h.rowcnt.resize(M->L + 1);
    h.colcnt.resize(M->L + 1);
    auto take = [&](std::vector<int32_t>& v, int64_t side) {
        v.assign(w, w + side);
        w += side;
    };
    for (int l = 0; l <= M->L; ++l) {
        take(h.rowcnt[l], int64_t(1) << l);
        take(h.colcnt[l], int64_t(1) << l);
    }
    take(h.blk_row, (int64_t)M->lb << M->L);
    take(h.blk_col, (int64_t)M->lb << M->L);
    h.ready = true;
    M->hist = std::move(h);
}

void build_histograms(qt_matrix* M, hipStream_t s) {
    std::lock_guard<std::mutex> lk(M->mu);
    if (M->hist.ready || M->nblocks == 0) return;   // (nothing counts an empty matrix's pairs)
    const int64_t nb_pad = (int64_t)M->lb << M->L;
    const int64_t total = histogram_words(M);
    DBuf<int32_t> d(total, s);
    k_fill_i32<<<std::min(grid_for(total), 4096u), 256, 0, s>>>(d.p, total, 0);
    QT_LAUNCH("k_fill_i32");
    int64_t off = 0;
    for (int l = 0; l <= M->L; ++l) {
        const int64_t side = int64_t(1) << l;
        const uint64_t* keys = (l < M->L) ? M->levels[l].key.p : M->leaves.key.p;
        const int64_t n = (l < M->L) ? M->levels[l].n : M->leaves.n;
        if (n > 0) {
            k_hist<<<grid_for(n), 256, 0, s>>>(keys, n, d.p + off, d.p + off + side);
            QT_LAUNCH("k_hist");
        }
        off += 2 * side;
    }
    k_hist<<<grid_for(M->nblocks), 256, 0, s>>>(M->bkey.p, M->nblocks, d.p + off, d.p + off + nb_pad);
    QT_LAUNCH("k_hist");
    ReadBack words(total);
    words.publish(d.p, s);
    adopt_histograms(M, words.wait(s));
}

// ----------------------------------------------------- operand forms

// A derived form was just queued on s: record its event there.
static void form_mark(hipEvent_t& ev, hipStream_t s) {
    if (!ev) QT_HIP(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
    QT_HIP(hipEventRecord(ev, s));
}

// Work queued on s from here on must see the form: wait for its event unless
// it has completed already (then the event is dropped, so later calls skip
// even the query). Called with M->mu held.
static void form_ready(hipEvent_t& ev, hipStream_t s) {
    if (!ev) return;
    const hipError_t q = hipEventQuery(ev);
    if (q == hipSuccess) {
        (void)hipEventDestroy(ev);
        ev = nullptr;
        return;
    }
    if (q != hipErrorNotReady) hip_check(q, "hipEventQuery");
    QT_HIP(hipStreamWaitEvent(s, ev, 0));
}

const double* operand_f64(qt_matrix* M, hipStream_t s) {
    if (M->vtype == QT_F64) return M->v64.p;
    std::lock_guard<std::mutex> lk(M->mu);
    if (!M->v64_cache.p && M->nblocks > 0) {
        const int64_t n = M->nblocks * (int64_t)M->b * M->b;
        M->v64_cache.alloc(n, s);
        in_launches(n, 1, [&](int64_t at, int64_t m) {
            k_f32_to_f64<<<grid_for(m), 256, 0, s>>>(M->v32.p + at, m, M->v64_cache.p + at);
            QT_LAUNCH("k_f32_to_f64");
        });
        form_mark(M->ev_v64, s);
    }
    form_ready(M->ev_v64, s);
    return M->v64_cache.p;
}

const float* operand_f32(qt_matrix* M, hipStream_t s) {
    std::lock_guard<std::mutex> lk(M->mu);
    if (!M->v32.p && M->nblocks > 0) {
        const int64_t n = M->nblocks * (int64_t)M->b * M->b;
        M->v32.alloc(n, s);
        in_launches(n, 1, [&](int64_t at, int64_t m) {
            k_f64_to_f32<<<grid_for(m), 256, 0, s>>>(M->v64.p + at, m, M->v32.p + at);
            QT_LAUNCH("k_f64_to_f32");
        });
        form_mark(M->ev_v32, s);
    }
    form_ready(M->ev_v32, s);
    return M->v32.p;
}

void operand_bf16(qt_matrix* M, hipStream_t s) {
    std::lock_guard<std::mutex> lk(M->mu);
    if (!M->bf_hi.p && M->nblocks > 0) {
        // all four parts are obtained before any is attached to the handle,
        // so a failed allocation leaves no partial form behind
        const int64_t n = M->nblocks * (int64_t)M->b * M->b;
        DBuf<uint16_t> hi(n, s), lo(n, s), hi_t(n, s), lo_t(n, s);
        const int64_t bb = (int64_t)M->b * M->b;
        in_launches(M->nblocks, bb, [&](int64_t at, int64_t m) {
            const unsigned g = grid_for(m * bb);
            const int64_t e = at * bb;
            if (M->vtype == QT_F64)
                k_bf16_split<double><<<g, 256, 0, s>>>(M->v64.p + e, m, M->b, hi.p + e, lo.p + e, hi_t.p + e, lo_t.p + e);
            else
                k_bf16_split<float><<<g, 256, 0, s>>>(M->v32.p + e, m, M->b, hi.p + e, lo.p + e, hi_t.p + e, lo_t.p + e);
            QT_LAUNCH("k_bf16_split");
        });
        form_mark(M->ev_bf16, s);
        M->bf_hi = std::move(hi);
        M->bf_lo = std::move(lo);
        M->bf_hi_t = std::move(hi_t);
        M->bf_lo_t = std::move(lo_t);
    }
    form_ready(M->ev_bf16, s);
}

// ----------------------------------------------------------------- build

// A tree under construction: its arrays, placed by bounds, and the words the
// host reads when they are done: kErr, kCount, two for a caller's double
// (kSum), the node counts of levels 0 .. L, the histograms.
struct TreeJob {
    enum { kErr = 0, kCount = 1, kSum = 2, kLevels = 4 };
    qt_matrix* M;
    int64_t bound;                 // at most this many blocks
    DBuf<int32_t> words, starts;
    std::vector<size_t> child_at, key_at;
    size_t base_at = 0, lkey_at = 0, mo_at = 0, rm_at = 0, cm_at = 0;
    int64_t nwords = 0;
    TreeBuild b{};
    int32_t* err() { return words.p + kErr; }
    int32_t* count() { return words.p + kCount; }
    double* sum() { return reinterpret_cast<double*>(words.p + kSum); }
};

// Allocates and clears everything (n: the number of blocks, where the device
// does not write it to count() before tree_fill).
static void tree_begin(TreeJob& j, qt_matrix* M, int64_t bound, int64_t n, hipStream_t s) {
    const int L = M->L;
    if (L >= MAX_TREE_LEVELS) fail(QT_ERR_UNSUPPORTED, "quadtree too deep");
    j.M = M;
    j.bound = bound;
    ArenaPlan plan;
    std::vector<int64_t> cap(L + 1);
    for (int l = 0; l <= L; ++l) {   // node positions of M's shape at level l
        const int64_t side = (int64_t)M->leaf << (L - l);
        const int64_t positions = ((M->n_rows + side - 1) / side) * ((M->n_cols + side - 1) / side);
        cap[l] = std::max<int64_t>(std::min(bound, positions), 1);   // a list's first entry starts a node whatever it is
        j.child_at.push_back(0);
        j.key_at.push_back(0);
    }
    for (int l = 0; l < L; ++l) j.child_at[l] = plan.take(4 * (size_t)cap[l] * sizeof(int32_t));
    const size_t child_end = plan.bytes;   // the child tables come first: one clear covers them
    for (int l = 0; l < L; ++l) j.key_at[l] = plan.take((size_t)cap[l] * sizeof(uint64_t));
    j.base_at = plan.take((size_t)cap[L] * sizeof(int32_t));
    j.lkey_at = plan.take((size_t)cap[L] * sizeof(uint64_t));
    j.mo_at = plan.take((size_t)cap[L] * sizeof(uint64_t));
    j.rm_at = plan.take((size_t)cap[L] * sizeof(uint64_t));
    j.cm_at = plan.take((size_t)cap[L] * sizeof(uint64_t));
    M->arena.alloc(plan.bytes, s);
    j.nwords = TreeJob::kLevels + (L + 1) + histogram_words(M);
    j.words.alloc(j.nwords, s);
    TreeBuild& b = j.b;
    b.tile = TREE_THREADS;
    while (bound > TREE_TILES_MAX * b.tile) b.tile *= 2;
    const int64_t tiles = (bound + b.tile - 1) / b.tile;
    j.starts.alloc(tiles * (L + 1), s);
    char* at = M->arena.p;
    for (int l = 0; l < L; ++l) {
        b.child[l] = (int32_t*)(at + j.child_at[l]);
        b.key[l] = (uint64_t*)(at + j.key_at[l]);
    }
    b.base = (int32_t*)(at + j.base_at);
    b.lkey = (uint64_t*)(at + j.lkey_at);
    b.mo = (uint64_t*)(at + j.mo_at);
    b.rm = (uint64_t*)(at + j.rm_at);
    b.cm = (uint64_t*)(at + j.cm_at);
    b.n = j.count();
    b.L = L;
    b.lb_log = M->lb_log;
    b.starts = j.starts.p;
    b.err = j.err();
    b.hist = j.words.p + TreeJob::kLevels + (L + 1);
    const int64_t nnil = (int64_t)(child_end / sizeof(int32_t));
    const unsigned g = (unsigned)std::min<int64_t>(grid_for(std::max(nnil, j.nwords)), 4096);
    k_tree_init<<<g, 256, 0, s>>>(j.words.p, j.nwords, TreeJob::kCount, (int32_t)n, (int32_t*)at, nnil);
    QT_LAUNCH("k_tree_init");
}

// Forms the tree over the ascending keys (j.bound of them at most).
static void tree_fill(TreeJob& j, const uint64_t* keys, hipStream_t s) {
    TreeBuild& b = j.b;
    b.keys = keys;
    const unsigned tiles = (unsigned)((j.bound + b.tile - 1) / b.tile);
    k_tree_tiles<<<tiles, TREE_THREADS, 0, s>>>(b);
    QT_LAUNCH("k_tree_tiles");
    k_radix_scan<<<1, 1024, 0, s>>>(b.starts, j.words.p + TreeJob::kLevels, b.L + 1, (int)tiles);
    QT_LAUNCH("k_radix_scan");
    k_tree_tables<<<tiles, TREE_THREADS, 0, s>>>(b);
    QT_LAUNCH("k_tree_tables");
}

// Parts of a buffer moved to another one.
constexpr int MAX_PARTS = 2 * MAX_TREE_LEVELS + 6;
struct Parts {
    int n;
    const int32_t* from[MAX_PARTS];
    int32_t* to[MAX_PARTS];
    int64_t words[MAX_PARTS];
};

__global__ void k_copy_parts(Parts a) {
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    for (int p = 0; p < a.n; ++p)
        for (int64_t i = i0; i < a.words[p]; i += step) a.to[p][i] = a.from[p][i];
}

// The tree and keys of M in buffers of their size, where those made by bounds
// hold much more: over 1 MiB and a 16th of what the values take (a truncation to
// few blocks, many blocks in few leaves: 100 k blocks over 2048 block rows
// truncated to three held 3.7 MB). A move takes a call some 15 us. True: it is
// queued on s and has to be waited for before the handle is given out, as products
// on any stream read a handle's structure without waiting for its own.
static bool tree_shrink(TreeJob& j, const int32_t* cnt, hipStream_t s) {
    qt_matrix* M = j.M;
    const int L = M->L;
    const int64_t n = M->nblocks;
    ArenaPlan plan;
    std::vector<size_t> child_at, key_at;
    for (int l = 0; l < L; ++l) child_at.push_back(plan.take(4 * (size_t)cnt[l] * sizeof(int32_t)));
    for (int l = 0; l < L; ++l) key_at.push_back(plan.take((size_t)cnt[l] * sizeof(uint64_t)));
    const size_t nl = cnt[L];
    const size_t base_at = plan.take(nl * sizeof(int32_t)), lkey_at = plan.take(nl * sizeof(uint64_t));
    const size_t mo_at = plan.take(nl * sizeof(uint64_t)), rm_at = plan.take(nl * sizeof(uint64_t));
    const size_t cm_at = plan.take(nl * sizeof(uint64_t)), bkey_at = plan.take(n * sizeof(uint64_t));
    const int64_t held = (int64_t)(M->arena.n + M->bkey.n * sizeof(uint64_t));
    const int64_t values = M->vsrc ? 0 : n * M->b * M->b * (int64_t)sizeof(double);
    if (held - (int64_t)plan.bytes <= std::max(int64_t(1) << 20, values / 16)) return false;
    if (n == 0) {
        M->arena.release();
        M->bkey.release();
        return false;
    }
    DBuf<char> arena;
    try {
        arena.alloc(plan.bytes, s);
    } catch (const Error& e) {
        if (e.status != QT_ERR_OOM) throw;
        return false;   // the call has all that it needs
    }
    Parts parts{};
    auto move = [&](size_t& at, size_t to, size_t bytes) {
        if (bytes) {
            parts.from[parts.n] = (const int32_t*)(M->arena.p + at);
            parts.to[parts.n] = (int32_t*)(arena.p + to);
            parts.words[parts.n++] = (int64_t)(bytes / sizeof(int32_t));
        }
        at = to;
    };
    for (int l = 0; l < L; ++l) {
        move(j.child_at[l], child_at[l], 4 * (size_t)cnt[l] * sizeof(int32_t));
        move(j.key_at[l], key_at[l], (size_t)cnt[l] * sizeof(uint64_t));
    }
    move(j.base_at, base_at, nl * sizeof(int32_t));
    move(j.lkey_at, lkey_at, nl * sizeof(uint64_t));
    move(j.mo_at, mo_at, nl * sizeof(uint64_t));
    move(j.rm_at, rm_at, nl * sizeof(uint64_t));
    move(j.cm_at, cm_at, nl * sizeof(uint64_t));
    parts.from[parts.n] = (const int32_t*)M->bkey.p;
    parts.to[parts.n] = (int32_t*)(arena.p + bkey_at);
    parts.words[parts.n++] = 2 * n;
    k_copy_parts<<<(unsigned)std::min<int64_t>(grid_for((int64_t)plan.bytes / 16), 1024), 256, 0, s>>>(parts);
    QT_LAUNCH("k_copy_parts");
    M->arena = std::move(arena);   // the old buffers go in order, after the move
    M->bkey.view(M->arena.p + bkey_at, n);
    return true;
}

// Reads the words back and sets M's tree, block count and histograms; throws
// what the error flags say. out (may be nullptr): the caller's double. True: s is
// to be waited for (see tree_shrink).
static bool tree_finish(TreeJob& j, hipStream_t s, double* out = nullptr) {
    ReadBack back(j.nwords);
    back.publish(j.words.p, s);
    const int32_t* w = back.wait(s);
    if (w[TreeJob::kErr] & 1) fail(QT_ERR_ARG, "block index out of range");
    if (w[TreeJob::kErr] & 2) fail(QT_ERR_DUPLICATE, "the same (I, J) block is listed twice");
    qt_matrix* M = j.M;
    const int L = M->L;
    const int32_t* cnt = w + TreeJob::kLevels;
    M->nblocks = w[TreeJob::kCount];
    const bool moved = tree_shrink(j, cnt, s);
    char* at = M->arena.p;
    for (int l = 0; l < L; ++l) {
        M->levels[l].n = cnt[l];
        M->levels[l].child.view(at + j.child_at[l], 4 * (size_t)cnt[l]);
        M->levels[l].key.view(at + j.key_at[l], cnt[l]);
    }
    LeafLevel& lv = M->leaves;
    lv.n = cnt[L];
    lv.base.view(at + j.base_at, cnt[L]);
    lv.key.view(at + j.lkey_at, cnt[L]);
    lv.mask_mo.view(at + j.mo_at, cnt[L]);
    lv.mask_rm.view(at + j.rm_at, cnt[L]);
    lv.mask_cm.view(at + j.cm_at, cnt[L]);
    if (out) std::memcpy(out, w + TreeJob::kSum, sizeof(double));
    adopt_histograms(M, cnt + (L + 1));
    return moved;
}

// Block keys in Morton order and the quadtree of M (shape fields set) from a
// device block list; perm[t] receives the list position of the block at sorted
// position t. Queued on s; tree_finish completes it and rejects out-of-range
// and repeated (I, J).
static void begin_structure(TreeJob& j, qt_matrix* M, const int32_t* pI, const int32_t* pJ, int64_t nblocks,
                            int64_t nbr, int64_t nbc, DBuf<int32_t>& perm, hipStream_t s) {
    const int key_bits = 2 * ilog2(std::max(nbr, nbc));
    M->bkey.alloc(nblocks, s);
    perm.alloc(nblocks, s);
    DBuf<int32_t> tmp(sort_tmp_words(nblocks, key_bits), s);
    tree_begin(j, M, nblocks, nblocks, s);
    stable_sort(ListKeys{pI, pJ, nbr, nbc, j.err()}, KeyPermSink{M->bkey.p, perm.p}, nblocks, key_bits, tmp.p, perm.p,
                s);
    tree_fill(j, M->bkey.p, s);
}

qt_matrix* build(int64_t n_rows, int64_t n_cols, int32_t b, int32_t leaf, int64_t nblocks, const int32_t* I,
                 const int32_t* J, const double* values, qt_mem where, hipStream_t s) {
    if (n_rows < 0 || n_cols < 0 || nblocks < 0) fail(QT_ERR_ARG, "negative size");
    if (where != QT_MEM_HOST && where != QT_MEM_DEVICE) fail(QT_ERR_ARG, "bad memory kind");
    if (nblocks > 0 && (!I || !J || !values)) fail(QT_ERR_ARG, "NULL block list");
    if (b != 16 && b != 32 && b != 64) fail(QT_ERR_SHAPE, "block size must be 16, 32 or 64");
    if (leaf <= 0 || leaf % b) fail(QT_ERR_SHAPE, "leaf size must be a positive multiple of the block size");
    const int lb = leaf / b;
    if (lb & (lb - 1)) fail(QT_ERR_SHAPE, "leaf size / block size must be a power of two");
    if (lb > 8) fail(QT_ERR_SHAPE, "leaf size / block size must be at most 8");
    if (n_rows % b || n_cols % b) fail(QT_ERR_SHAPE, "dimensions must be multiples of the block size");
    const int64_t nbr = n_rows / b, nbc = n_cols / b;
    if (nbr > (int64_t(1) << 30) || nbc > (int64_t(1) << 30)) fail(QT_ERR_UNSUPPORTED, "too many blocks per side");
    if (nblocks > (int64_t(1) << 31) - 2) fail(QT_ERR_UNSUPPORTED, "too many blocks");
    // a grid without positions: no index is in range, and the tree, formed before
    // the device's error flag is read, would have no place for a node
    if (nblocks > 0 && (nbr == 0 || nbc == 0)) fail(QT_ERR_ARG, "block index out of range");

    std::unique_ptr<qt_matrix> M(new qt_matrix);
    M->n_rows = n_rows;
    M->n_cols = n_cols;
    M->b = b;
    M->leaf = leaf;
    M->lb = lb;
    M->lb_log = ilog2(lb);
    int64_t side = lb;
    int L = 0;
    while (side < std::max<int64_t>(std::max<int64_t>(nbr, nbc), 1)) {
        side *= 2;
        ++L;
    }
    M->L = L;
    M->vtype = QT_F64;
    M->nblocks = nblocks;
    M->stream = s;
    QT_HIP(hipGetDevice(&M->device));
    M->levels.resize(L);
    const int bb = b * b;

    if (nblocks == 0) return M.release();

    // operands on the device
    DBuf<int32_t> dI, dJ;
    DBuf<double> dV;
    const int32_t* pI = I;
    const int32_t* pJ = J;
    const double* pV = values;
    if (where == QT_MEM_HOST) {
        dI.alloc(nblocks, s);
        dJ.alloc(nblocks, s);
        dV.alloc((size_t)nblocks * bb, s);
        QT_HIP(hipMemcpyAsync(dI.p, I, nblocks * sizeof(int32_t), hipMemcpyHostToDevice, s));
        QT_HIP(hipMemcpyAsync(dJ.p, J, nblocks * sizeof(int32_t), hipMemcpyHostToDevice, s));
        QT_HIP(hipMemcpyAsync(dV.p, values, (size_t)nblocks * bb * sizeof(double), hipMemcpyHostToDevice, s));
        pI = dI.p;
        pJ = dJ.p;
        pV = dV.p;
    }

    DBuf<int32_t> perm;
    TreeJob job;
    M->v64.alloc((size_t)nblocks * bb, s);
    begin_structure(job, M.get(), pI, pJ, nblocks, nbr, nbc, perm, s);
    copy_blocks(pV, perm.p, nblocks, bb, M->v64.p, s);
    // the last thing queued, but for a moved tree: the caller's arrays have been read
    if (tree_finish(job, s)) QT_HIP(hipStreamSynchronize(s));
    return M.release();
}

// ------------------------------------------------------------ copy out

// Words of scratch of a row-major copy-out: the permutation and the sort's.
static size_t rowmajor_words(const qt_matrix* M) {
    if (M->nblocks <= RANKED_MAX) return 0;
    return (size_t)M->nblocks + sort_tmp_words(M->nblocks, ilog2(M->n_rows / M->b));
}

// A stream of the library's own for the sort of a copy-out, which needs only the
// blocks' keys, there since the call that made the matrix returned: beside
// whatever is queued on the caller's stream, usually the kernel that computes
// the values. The caller's arrays are written on the caller's stream alone. One
// per device, of default priority. For copies of ASIDE_BYTES and more: the event
// between the streams costs host and GPU some 15 us, which a product of 27 MB
// lost (13 k blocks of 16, 140 and 156 us a pass with its copy-out), while the
// sort's 25 to 70 us show from some 200 MB on: build and copy-out of 240 MB 282 and
// 274 us, sysq with 360 MB 734 and 722, an R-MAT product with 1.7 GB 1546 and 1493.
constexpr size_t ASIDE_BYTES = size_t(128) << 20;

// The stream is lent to one call at a time, and not while another caller's sort
// may still run on it: nobody waits for the sort of a stream that is not its own.
// Such a call, rare as a sort takes tens of us, sorts on its own stream.
struct SortStream {
    std::mutex mu;                // held from the loan until the sort is queued
    hipStream_t st = nullptr;
    hipEvent_t done = nullptr;    // recorded behind the latest sort
    hipStream_t user = nullptr;   // the stream it was for
    bool used = false;
};
static std::mutex g_sort_mu;
static std::map<int, SortStream> g_sort_stream;   // per device; entries stay where they are

// nullptr: none to be had (the lock says for how long it is).
static SortStream* borrow_sort_stream(hipStream_t s, std::unique_lock<std::mutex>& lock) {
    int dev = 0;
    QT_HIP(hipGetDevice(&dev));
    SortStream* b;
    {
        std::lock_guard<std::mutex> lk(g_sort_mu);
        b = &g_sort_stream[dev];
    }
    std::unique_lock<std::mutex> mine(b->mu, std::try_to_lock);
    if (!mine.owns_lock()) return nullptr;
    if (!b->st) QT_HIP(hipStreamCreateWithFlags(&b->st, hipStreamNonBlocking));
    if (!b->done) QT_HIP(hipEventCreateWithFlags(&b->done, hipEventDisableTiming));
    if (b->used && b->user != s && hipEventQuery(b->done) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    lock = std::move(mine);
    return b;
}

// Whether work is queued on s that the sort need not wait for; not while s is
// captured, where all of a call's work belongs to s.
static bool stream_behind(hipStream_t s) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) != hipSuccess || st != hipStreamCaptureStatusNone) {
        (void)hipGetLastError();
        return false;
    }
    const bool behind = hipStreamQuery(s) == hipErrorNotReady;
    (void)hipGetLastError();
    return behind;
}

// Row-major order of more than RANKED_MAX blocks, on `sorts`: tmp, of
// rowmajor_words(M), begins with the source block of every output position.
static void rowmajor_sort(const qt_matrix* M, int32_t* tmp, hipStream_t sorts) {
    const int64_t n = M->nblocks;
    if (n > RANKED_MAX)
        stable_sort(RowKeys{M->bkey.p}, PermSink{tmp}, n, ilog2(M->n_rows / M->b), tmp + n, tmp, sorts);
}

// Copy-out into device arrays I, J, values (values may be NULL) on s, in the
// order that rowmajor_sort left in perm.
static void rowmajor_copy(const qt_matrix* M, const int32_t* perm, int32_t* I, int32_t* J, void* values,
                          qt_prec out_type, hipStream_t s) {
    const int64_t n = M->nblocks;
    const int bb = M->b * M->b;
    if (n <= RANKED_MAX) {
        if (M->vtype == QT_F64 && (out_type == QT_F64 || !values))
            copy_ranked(M->bkey.p, M->v64.p, n, bb, I, J, (double*)values, s);
        else if (M->vtype == QT_F64)
            copy_ranked(M->bkey.p, M->v64.p, n, bb, I, J, (float*)values, s);
        else if (out_type == QT_F64 && values)
            copy_ranked(M->bkey.p, M->v32.p, n, bb, I, J, (double*)values, s);
        else
            copy_ranked(M->bkey.p, M->v32.p, n, bb, I, J, (float*)values, s);
        return;
    }
    const Coords coords{M->bkey.p, I, J};
    if (!values) {   // pattern only
        k_coords<<<grid_for(n), 256, 0, s>>>(perm, n, coords);
        QT_LAUNCH("k_coords");
    } else if (M->vtype == QT_F64 && out_type == QT_F64)
        copy_blocks(M->v64.p, perm, n, bb, (double*)values, s, coords);
    else if (M->vtype == QT_F64)
        copy_blocks(M->v64.p, perm, n, bb, (float*)values, s, coords);
    else if (out_type == QT_F64)
        copy_blocks(M->v32.p, perm, n, bb, (double*)values, s, coords);
    else
        copy_blocks(M->v32.p, perm, n, bb, (float*)values, s, coords);
}

// The sort on the borrowed stream: the caller's s runs after it, and takes its
// scratch over, once that order is known to stand; after an error the sort has
// ended before the scratch and M's keys can go.
static void rowmajor_sort_aside(const qt_matrix* M, DBuf<int32_t>& tmp, SortStream& aside, hipStream_t s) {
    struct Drain {
        hipStream_t st;
        ~Drain() {
            if (st) (void)hipStreamSynchronize(st);
        }
    } drain{aside.st};
    rowmajor_sort(M, tmp.p, aside.st);
    QT_HIP(hipEventRecord(aside.done, aside.st));
    QT_HIP(hipStreamWaitEvent(s, aside.done, 0));
    aside.user = s;
    aside.used = true;
    tmp.s = s;
    drain.st = nullptr;
}

void to_blocks(const qt_matrix* M, int32_t* I, int32_t* J, void* values, qt_prec out_type, qt_mem where,
               hipStream_t s) {
    if (out_type != QT_F64 && out_type != QT_F32) fail(QT_ERR_UNSUPPORTED, "output type must be F64 or F32");
    if (where != QT_MEM_HOST && where != QT_MEM_DEVICE) fail(QT_ERR_ARG, "bad memory kind");
    const int64_t n = M->nblocks;
    if (n == 0) return;
    if (!I || !J) fail(QT_ERR_ARG, "NULL output array");
    const int bb = M->b * M->b;
    const size_t words = rowmajor_words(M);
    const size_t vbytes = values ? (size_t)n * bb * (out_type == QT_F64 ? sizeof(double) : sizeof(float)) : 0;
    std::unique_lock<std::mutex> loan;
    SortStream* aside = nullptr;
    if (words > 0 && vbytes >= ASIDE_BYTES && stream_behind(s)) aside = borrow_sort_stream(s, loan);
    DBuf<int32_t> tmp(words, aside ? aside->st : s);
    DBuf<int32_t> tI, tJ;
    DBuf<char> tV;
    int32_t* oI = I;
    int32_t* oJ = J;
    void* oV = values;
    if (where == QT_MEM_HOST) {
        tI.alloc(n, s);
        tJ.alloc(n, s);
        if (values) tV.alloc(vbytes, s);
        oI = tI.p;
        oJ = tJ.p;
        oV = values ? (void*)tV.p : nullptr;
    }
    if (aside) {
        rowmajor_sort_aside(M, tmp, *aside, s);
        loan.unlock();
    } else {
        rowmajor_sort(M, tmp.p, s);
    }
    rowmajor_copy(M, tmp.p, oI, oJ, oV, out_type, s);
    if (where == QT_MEM_HOST) {
        QT_HIP(hipMemcpyAsync(I, oI, n * sizeof(int32_t), hipMemcpyDeviceToHost, s));
        QT_HIP(hipMemcpyAsync(J, oJ, n * sizeof(int32_t), hipMemcpyDeviceToHost, s));
        if (values) QT_HIP(hipMemcpyAsync(values, oV, vbytes, hipMemcpyDeviceToHost, s));
        QT_HIP(hipStreamSynchronize(s));
    }
}

// -------------------------------------------- copy-out without allocation

// Scratch of the allocation-free copy-out of up to QT_NOALLOC_MAX_BLOCKS
// blocks: the permutation, and the sort's counts and permutations, 12 MiB in
// all, one copy per device for the life of the process. Host code never passes `scratch` itself (on the host it names
// a stand-in, not device memory): it takes the array's device address once
// per device with hipGetSymbolAddress and uses that address only.
constexpr int64_t kNoAllocEntries = QT_NOALLOC_MAX_BLOCKS;
constexpr int64_t kNoAllocWords = 3 * kNoAllocEntries;
static __device__ __align__(256) int32_t scratch[kNoAllocWords];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_addr[kMaxDevices] = {};

// Device address of `scratch` on the current device (taken on the first call
// made with that device current).
static void* scratch_address(int dev) {
    if (dev < 0 || dev >= kMaxDevices) fail(QT_ERR_UNSUPPORTED, "device ordinal beyond the library's table");
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_addr[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            (void)hipGetLastError();
            fail(QT_ERR_DEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        }
        g_scratch_addr[dev] = p;
    }
    return g_scratch_addr[dev];
}

void to_blocks_noalloc(const qt_matrix* M, int32_t* I, int32_t* J, void* values, qt_prec out_type, hipStream_t s) {
    if (out_type != QT_F64 && out_type != QT_F32) fail(QT_ERR_UNSUPPORTED, "output type must be F64 or F32");
    const int64_t n = M->nblocks;
    if (n > QT_NOALLOC_MAX_BLOCKS)
        fail(QT_ERR_UNSUPPORTED, "matrix has " + std::to_string(n) + " blocks; the allocation-free copy-out takes at most " +
                                     std::to_string((long long)QT_NOALLOC_MAX_BLOCKS));
    int dev = 0;
    QT_HIP(hipGetDevice(&dev));
    if (dev != M->device) fail(QT_ERR_ARG, "the matrix lives on another device than the current one");
    int32_t* tmp = static_cast<int32_t*>(scratch_address(dev));
    if (n == 0) return;
    if (!I || !J) fail(QT_ERR_ARG, "NULL output array");
    // every word is written before it is read, so nothing left by an earlier
    // call is seen and nothing needs clearing
    if (rowmajor_words(M) > (size_t)kNoAllocWords) fail(QT_ERR_DEVICE, "copy-out scratch exceeded");
    rowmajor_sort(M, tmp, s);
    rowmajor_copy(M, tmp, I, J, values, out_type, s);
}

// ------------------------------------------------------------ norms
//
// Squared Frobenius norms of a matrix and of every submatrix in its
// quadtree (the paper's conclusions name such per-submatrix norms as an
// addition to the library, after Bock and Challacombe): of every block, one
// wave per block; of every leaf, the sum over its blocks; of every node
// above, the sum over its present children. A node's squared norm is at
// least each block's below it, whatever the order of the sums (every term is
// non-negative and rounding is monotone), which is what lets a product be
// dropped by its norm at any level.

// One wave per block, 16 bytes per lane and load, the loads ahead of the sums.
// Bound by HBM.
template <class T>
__global__ __launch_bounds__(256) void k_block_norm2(const T* __restrict__ v, int64_t n, int bb,
                                                    double* __restrict__ out) {
    constexpr int VE = 16 / sizeof(T), U = 4;
    typedef T vec __attribute__((ext_vector_type(VE)));
    const int lane = threadIdx.x & 63;
    const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t >= n) return;
    const vec* x = reinterpret_cast<const vec*>(v + (size_t)t * bb);
    const int m = bb / VE;   // 64 (fp32, b = 16) to 2048 vectors
    double s = 0.0;
    for (int e = lane; e < m; e += 64 * U) {
        vec y[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (e + 64 * u < m) y[u] = x[e + 64 * u];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (e + 64 * u < m) {
#pragma unroll
                for (int c = 0; c < VE; ++c) {
                    const double d = (double)y[u][c];
                    s += d * d;
                }
            }
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d, 64);
    if (lane == 0) out[t] = s;
}

static void launch_block_norm2(const qt_matrix* M, double* out, hipStream_t s) {
    const int bb = M->b * M->b;
    in_launches(M->nblocks, 64, [&](int64_t at, int64_t n) {
        const unsigned g = (unsigned)((n + 3) / 4);
        if (M->vtype == QT_F64)
            k_block_norm2<double><<<g, 256, 0, s>>>(M->v64.p + at * bb, n, bb, out + at);
        else
            k_block_norm2<float><<<g, 256, 0, s>>>(M->v32.p + at * bb, n, bb, out + at);
        QT_LAUNCH("k_block_norm2");
    });
}

// The leaf's norms are added in block order, eight loads at a time.
__global__ void k_leaf_norm2(const int32_t* __restrict__ base, const uint64_t* __restrict__ mo, int64_t n,
                             const double* __restrict__ bn2, double* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t b0 = base[i], cnt = __popcll(mo[i]);
    double s = 0.0;
    for (int32_t k = 0; k < cnt; k += 8) {
        double x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = k + e < cnt ? bn2[b0 + k + e] : 0.0;
#pragma unroll
        for (int e = 0; e < 8; ++e) s += x[e];
    }
    out[i] = s;
}

__device__ __forceinline__ double node_norm2(const int32_t* __restrict__ child, int64_t i, const double* below) {
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int32_t c = child[4 * i + q];
        if (c >= 0) s += below[c];
    }
    return s;
}

__global__ void k_node_norm2(const int32_t* __restrict__ child, int64_t n, const double* __restrict__ below,
                             double* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = node_norm2(child, i, below);
}

// The small levels at the top in one launch: a workgroup goes up the tree,
// level by level.
constexpr int64_t TOP_NODES = 4096;
struct TopNorms {
    int levels;
    const int32_t* child[MAX_TREE_LEVELS];   // from the lowest up
    int32_t n[MAX_TREE_LEVELS];
    double* out[MAX_TREE_LEVELS];
    const double* below;
};

__global__ __launch_bounds__(1024) void k_top_norm2(TopNorms a) {
    const double* below = a.below;
    for (int l = 0; l < a.levels; ++l) {
        for (int i = threadIdx.x; i < a.n[l]; i += 1024) a.out[l][i] = node_norm2(a.child[l], i, below);
        below = a.out[l];
        __threadfence_block();
        __syncthreads();
    }
}

void build_norms(qt_matrix* M, hipStream_t s, hipStream_t reader) {
    std::lock_guard<std::mutex> lk(M->mu);
    if (M->vsrc) fail(QT_ERR_UNSUPPORTED, "norms of a structure-only matrix");
    if (!M->bn2) {
        const int L = M->L;
        int64_t total = std::max<int64_t>(M->nblocks, 1) + M->leaves.n;
        for (int l = 0; l < L; ++l) total += M->levels[l].n;
        M->norms.alloc(total, s);
        double* p = M->norms.p;
        double* bn2 = p;
        p += std::max<int64_t>(M->nblocks, 1);
        if (M->nblocks > 0) launch_block_norm2(M, bn2, s);
        std::vector<const double*> nn2(L + 1, nullptr);
        double* below = p;
        p += M->leaves.n;
        if (M->leaves.n > 0) {
            k_leaf_norm2<<<grid_for(M->leaves.n), 256, 0, s>>>(M->leaves.base.p, M->leaves.mask_mo.p, M->leaves.n,
                                                              bn2, below);
            QT_LAUNCH("k_leaf_norm2");
        }
        nn2[L] = below;
        TopNorms top{};
        for (int l = L - 1; l >= 0; --l) {
            double* here = p;
            const int64_t nl = M->levels[l].n;
            p += nl;
            if (nl > TOP_NODES) {
                k_node_norm2<<<grid_for(nl), 256, 0, s>>>(M->levels[l].child.p, nl, below, here);
                QT_LAUNCH("k_node_norm2");
            } else {   // and no level above has more nodes
                if (top.levels == 0) top.below = below;
                top.child[top.levels] = M->levels[l].child.p;
                top.n[top.levels] = (int32_t)nl;
                top.out[top.levels++] = here;
            }
            nn2[l] = here;
            below = here;
        }
        if (top.levels > 0 && top.n[0] > 0) {
            k_top_norm2<<<1, 1024, 0, s>>>(top);
            QT_LAUNCH("k_top_norm2");
        }
        M->nn2 = nn2;
        M->bn2 = bn2;
        form_mark(M->ev_norms, s);
    }
    form_ready(M->ev_norms, reader);
}

// The squared norms of M's blocks in (I, J) row-major order, and of M.
void norms_out(qt_matrix* M, double* block_norm2, double* total_norm2, qt_mem where, hipStream_t s) {
    build_norms(M, s, s);
    const int64_t n = M->nblocks;
    if (block_norm2 && n > 0) {
        const int row_bits = ilog2(M->n_rows / M->b);
        DBuf<int32_t> stmp(sort_tmp_words(n, row_bits), s), perm(n, s);
        DBuf<double> tmp;
        double* out = block_norm2;
        if (where == QT_MEM_HOST) {
            tmp.alloc(n, s);
            out = tmp.p;
        }
        stable_sort(RowKeys{M->bkey.p}, GatherF64Sink{M->bn2, out}, n, row_bits, stmp.p, perm.p, s);
        if (where == QT_MEM_HOST) QT_HIP(hipMemcpyAsync(block_norm2, tmp.p, n * sizeof(double), hipMemcpyDeviceToHost, s));
    }
    if (total_norm2) {
        // the root's squared norm (0 for an all-NIL matrix)
        const bool any = M->L == 0 ? M->leaves.n > 0 : M->levels[0].n > 0;
        if (!any) {
            if (where == QT_MEM_HOST)
                *total_norm2 = 0.0;
            else
                QT_HIP(hipMemsetAsync(total_norm2, 0, sizeof(double), s));
        } else if (where == QT_MEM_HOST) {
            ReadBack back(2);
            back.publish(reinterpret_cast<const int32_t*>(M->nn2[0]), s);
            std::memcpy(total_norm2, back.wait(s), sizeof(double));
            if (!block_norm2) return;   // everything queued here is done
        } else {
            QT_HIP(hipMemcpyAsync(total_norm2, M->nn2[0], sizeof(double), hipMemcpyDeviceToDevice, s));
        }
    }
    if (where == QT_MEM_HOST) QT_HIP(hipStreamSynchronize(s));
}

// The full symmetric matrix S from its upper block triangle A, as structure
// only: block (I, J), I <= J, of A is block (I, J) of S, and for I < J also
// block (J, I) of S, read transposed. S holds no values; its block map points
// every block of S at the block of A that holds it (top bit: transposed).
__global__ void k_mirror_flags(const uint64_t* __restrict__ bkey, int64_t n, int32_t* __restrict__ upper,
                               int32_t* __restrict__ err) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    const uint32_t i = morton_row(bkey[t]), j = morton_col(bkey[t]);
    upper[t] = i < j ? 1 : 0;
    if (i > j) atomicOr(err, 1);
}

// entries t < n: A's blocks; entry n + rank[t]: the mirror of strictly upper block t
__global__ void k_mirror_list(const uint64_t* __restrict__ bkey, int64_t n, const int32_t* __restrict__ upper,
                              const int32_t* __restrict__ rank, int32_t* __restrict__ I, int32_t* __restrict__ J,
                              int32_t* __restrict__ src) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    const int32_t i = (int32_t)morton_row(bkey[t]), j = (int32_t)morton_col(bkey[t]);
    I[t] = i;
    J[t] = j;
    src[t] = (int32_t)t;
    if (upper[t]) {
        const int64_t m = n + rank[t];
        I[m] = j;
        J[m] = i;
        src[m] = (int32_t)((uint32_t)t | PROD_TRANS);
    }
}

__global__ void k_gather_i32(const int32_t* __restrict__ src, const int32_t* __restrict__ perm, int64_t n,
                             int32_t* __restrict__ dst) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) dst[t] = src[perm[t]];
}

qt_matrix* symmetric_full(qt_matrix* A, hipStream_t s) {
    std::lock_guard<std::mutex> lk(A->mu);
    if (A->sym_full) return A->sym_full.get();
    if (A->n_rows != A->n_cols) fail(QT_ERR_SHAPE, "a symmetric matrix must be square");
    const int64_t n = A->nblocks;
    std::unique_ptr<qt_matrix> S(new qt_matrix);
    S->n_rows = A->n_rows;
    S->n_cols = A->n_cols;
    S->b = A->b;
    S->leaf = A->leaf;
    S->lb = A->lb;
    S->lb_log = A->lb_log;
    S->L = A->L;
    S->vtype = A->vtype;
    S->stream = s;
    S->device = A->device;
    S->levels.resize(S->L);
    S->vsrc = A;
    if (n > 0) {
        DBuf<int32_t> up(n, s), rank(n + 1, s), tmp(scan_tmp_elems(n) + 1, s), err(1, s);
        k_fill_i32<<<1, 64, 0, s>>>(err.p, 1, 0);
        QT_LAUNCH("k_fill_i32");
        k_mirror_flags<<<grid_for(n), 256, 0, s>>>(A->bkey.p, n, up.p, err.p);
        QT_LAUNCH("k_mirror_flags");
        exclusive_scan(up.p, rank.p, n, tmp.p, s);
        int32_t h[2] = {0, 0};
        QT_HIP(hipMemcpyAsync(&h[0], rank.p + n, sizeof(int32_t), hipMemcpyDeviceToHost, s));
        QT_HIP(hipMemcpyAsync(&h[1], err.p, sizeof(int32_t), hipMemcpyDeviceToHost, s));
        QT_HIP(hipStreamSynchronize(s));
        if (h[1]) fail(QT_ERR_ARG, "upper-triangular storage holds a block below the diagonal");
        const int64_t total = n + h[0];
        if (total > (int64_t(1) << 31) - 2) fail(QT_ERR_UNSUPPORTED, "too many blocks");
        DBuf<int32_t> I(total, s), J(total, s), src(total, s);
        k_mirror_list<<<grid_for(n), 256, 0, s>>>(A->bkey.p, n, up.p, rank.p, I.p, J.p, src.p);
        QT_LAUNCH("k_mirror_list");
        S->nblocks = total;
        DBuf<int32_t> perm;
        TreeJob job;
        S->bmap.alloc(total, s);
        begin_structure(job, S.get(), I.p, J.p, total, A->n_rows / A->b, A->n_cols / A->b, perm, s);
        k_gather_i32<<<grid_for(total), 256, 0, s>>>(src.p, perm.p, total, S->bmap.p);
        QT_LAUNCH("k_gather_i32");
        if (tree_finish(job, s)) QT_HIP(hipStreamSynchronize(s));
    }
    A->sym_full = std::move(S);
    return A->sym_full.get();
}

// ------------------------------------------------------------- C = A + B

// An empty matrix shaped like `like` (L levels above the leaves).
static qt_matrix* shaped_like(const qt_matrix* like, int L, hipStream_t s) {
    std::unique_ptr<qt_matrix> C(new qt_matrix);
    C->n_rows = like->n_rows;
    C->n_cols = like->n_cols;
    C->b = like->b;
    C->leaf = like->leaf;
    C->lb = like->lb;
    C->lb_log = like->lb_log;
    C->L = L;
    C->vtype = QT_F64;
    C->stream = s;
    QT_HIP(hipGetDevice(&C->device));
    C->levels.resize(L);
    return C.release();
}

// Merge of two ascending key lists without a sort: A's key i comes after i
// keys of A and #{B keys < it} of B, less the keys in both lists before it;
// B's key j, where A does not hold it too, likewise. The common keys are
// counted per tile of 256 of A's (and kept as a bit per key), so the result's
// keys and its tree are formed without the host knowing their number: one
// wait for the tree, one for the values, where a merge, a scan and a tree took
// five (square, truncate, add and norms of a 16384 matrix: 1617 us with those,
// 1467 with this and the truncation below, which waits as often).
__device__ __forceinline__ int64_t count_below(const uint64_t* __restrict__ k, int64_t n, uint64_t x, bool le) {
    int64_t lo = 0, hi = n;   // first position whose key is >= x (le: > x)
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        const bool left = le ? (k[mid] <= x) : (k[mid] < x);
        if (left)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

constexpr int MERGE_TILE = 256;

__global__ __launch_bounds__(MERGE_TILE) void k_merge_common(const uint64_t* __restrict__ ka, int64_t na,
                                                             const uint64_t* __restrict__ kb, int64_t nb,
                                                             int32_t* __restrict__ below_b,
                                                             uint64_t* __restrict__ common,
                                                             int32_t* __restrict__ tiles) {
    __shared__ int32_t cnt;
    if (threadIdx.x == 0) cnt = 0;
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * MERGE_TILE + threadIdx.x;
    bool both = false;
    if (i < na) {
        const int64_t p = count_below(kb, nb, ka[i], false);
        below_b[i] = (int32_t)p;
        both = p < nb && kb[p] == ka[i];
    }
    const uint64_t m = __ballot(both);
    if ((threadIdx.x & 63) == 0) {
        common[i >> 6] = m;
        if (m) atomicAdd(&cnt, (int32_t)__popcll(m));
    }
    __syncthreads();
    if (threadIdx.x == 0) tiles[blockIdx.x] = cnt;
}

// common keys among A's first i (i <= na; tiles: scanned)
__device__ __forceinline__ int64_t common_before(const uint64_t* __restrict__ common,
                                                 const int32_t* __restrict__ tiles, int64_t i) {
    int64_t c = tiles[i / MERGE_TILE];
    for (int64_t w = i / MERGE_TILE * (MERGE_TILE / 64); w < (i >> 6); ++w) c += __popcll(common[w]);
    if (i & 63) c += __popcll(common[i >> 6] & (~0ull >> (64 - (i & 63))));
    return c;
}

// Output block o: A's block sa[o] (-1: none) plus B's block sb[o] (-1: none).
__global__ void k_merge_write(const uint64_t* __restrict__ ka, int64_t na, const uint64_t* __restrict__ kb, int64_t nb,
                              const int32_t* __restrict__ below_b, const uint64_t* __restrict__ common,
                              const int32_t* __restrict__ tiles, const int32_t* __restrict__ total,
                              uint64_t* __restrict__ key, int32_t* __restrict__ sa, int32_t* __restrict__ sb,
                              int32_t* __restrict__ count) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t == 0) *count = (int32_t)(na + nb - *total);
    if (t >= na + nb) return;
    int64_t o;
    if (t < na) {
        o = t + below_b[t] - common_before(common, tiles, t);
        key[o] = ka[t];
        sa[o] = (int32_t)t;
        sb[o] = (common[t >> 6] >> (t & 63)) & 1 ? below_b[t] : -1;
    } else {
        const int64_t j = t - na, p = count_below(ka, na, kb[j], false);
        if (p < na && ka[p] == kb[j]) return;   // written with A's block
        o = j + p - common_before(common, tiles, p);
        key[o] = kb[j];
        sa[o] = -1;
        sb[o] = (int32_t)j;
    }
}

// Values of the sum, in pieces of 64 two-entry vectors (see k_copy_blocks).
__global__ __launch_bounds__(64 * COPY_WAVES) void k_add_blocks(const int32_t* __restrict__ sa,
                                                                const int32_t* __restrict__ sb, int64_t pieces,
                                                                int ppb_log, const double* __restrict__ va,
                                                                const double* __restrict__ vb,
                                                                double* __restrict__ vc) {
    typedef double vec __attribute__((ext_vector_type(2)));
    const int lane = threadIdx.x & 63;
    const int64_t p0 = ((int64_t)blockIdx.x * COPY_WAVES + (threadIdx.x >> 6)) * COPY_PIECES;
    const int64_t in_block = (int64_t(1) << ppb_log) - 1;
    vec x[COPY_PIECES], y[COPY_PIECES];
    int32_t a[COPY_PIECES], b[COPY_PIECES];
#pragma unroll
    for (int r = 0; r < COPY_PIECES; ++r) {
        const int64_t p = p0 + r;
        if (p >= pieces) break;
        a[r] = sa[p >> ppb_log];
        b[r] = sb[p >> ppb_log];
        const int64_t e = (p & in_block) * 64 + lane;
        if (a[r] >= 0) x[r] = __builtin_nontemporal_load(reinterpret_cast<const vec*>(va) + ((int64_t)a[r] << ppb_log) * 64 + e);
        if (b[r] >= 0) y[r] = __builtin_nontemporal_load(reinterpret_cast<const vec*>(vb) + ((int64_t)b[r] << ppb_log) * 64 + e);
    }
#pragma unroll
    for (int r = 0; r < COPY_PIECES; ++r) {
        const int64_t p = p0 + r;
        if (p >= pieces) break;
        const vec v = a[r] < 0 ? y[r] : b[r] < 0 ? x[r] : x[r] + y[r];
        __builtin_nontemporal_store(v, reinterpret_cast<vec*>(vc) + p * 64 + lane);
    }
}

qt_matrix* add(qt_matrix* A, qt_matrix* B, hipStream_t s) {
    if (A->b != B->b || A->leaf != B->leaf) fail(QT_ERR_SHAPE, "operands differ in block or leaf size");
    if (A->n_rows != B->n_rows || A->n_cols != B->n_cols) fail(QT_ERR_SHAPE, "operands differ in dimensions");
    const double* va = operand_f64(A, s);
    const double* vb = operand_f64(B, s);
    const int64_t na = A->nblocks, nb = B->nblocks, n = na + nb;
    if (n > (int64_t(1) << 31) - 2) fail(QT_ERR_UNSUPPORTED, "too many blocks");
    if (n == 0) return build(A->n_rows, A->n_cols, A->b, A->leaf, 0, nullptr, nullptr, nullptr, QT_MEM_DEVICE, s);
    const int bb = A->b * A->b;
    std::unique_ptr<qt_matrix> C(shaped_like(A, std::max(A->L, B->L), s));
    const int64_t tiles = na / MERGE_TILE + 1;   // the last one may be empty: common_before(na) reads it
    DBuf<int32_t> below(std::max<int64_t>(na, 1), s), tcnt(tiles + 1, s), sa(n, s), sb(n, s);
    DBuf<uint64_t> common(tiles * (MERGE_TILE / 64), s);
    C->bkey.alloc(n, s);
    TreeJob job;
    tree_begin(job, C.get(), n, 0, s);
    k_merge_common<<<(unsigned)tiles, MERGE_TILE, 0, s>>>(A->bkey.p, na, B->bkey.p, nb, below.p, common.p, tcnt.p);
    QT_LAUNCH("k_merge_common");
    k_radix_scan<<<1, 1024, 0, s>>>(tcnt.p, tcnt.p + tiles, 1, (int)tiles);
    QT_LAUNCH("k_radix_scan");
    k_merge_write<<<grid_for(n), 256, 0, s>>>(A->bkey.p, na, B->bkey.p, nb, below.p, common.p, tcnt.p, tcnt.p + tiles,
                                              C->bkey.p, sa.p, sb.p, job.count());
    QT_LAUNCH("k_merge_write");
    tree_fill(job, C->bkey.p, s);
    tree_finish(job, s);
    const int64_t nc = C->nblocks;
    C->v64.alloc((size_t)nc * bb, s);
    int ppb_log = 0;
    while ((128 << ppb_log) < bb) ++ppb_log;
    const int64_t pieces = nc << ppb_log, per = COPY_WAVES * COPY_PIECES;
    k_add_blocks<<<(unsigned)((pieces + per - 1) / per), 64 * COPY_WAVES, 0, s>>>(sa.p, sb.p, pieces, ppb_log, va, vb,
                                                                                 C->v64.p);
    QT_LAUNCH("k_add_blocks");
    QT_HIP(hipStreamSynchronize(s));
    return C.release();
}

// --------------------------------------------------- value truncation

// Sorted position p is removed while the running sum of squared norms up to
// and including p stays below eps^2; the survivors are flagged by block.
__global__ void k_trunc_flags(const double* __restrict__ excl, const double* __restrict__ sorted, int64_t n,
                              double eps2, const int32_t* __restrict__ idx, int32_t* __restrict__ keep) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n) keep[idx[p]] = (excl[p] + sorted[p] < eps2) ? 0 : 1;
}

constexpr int KEEP_TILE = 256;

__global__ __launch_bounds__(KEEP_TILE) void k_keep_tiles(const int32_t* __restrict__ keep, int64_t n,
                                                         int32_t* __restrict__ tiles) {
    __shared__ int32_t cnt;
    if (threadIdx.x == 0) cnt = 0;
    __syncthreads();
    const int64_t t = (int64_t)blockIdx.x * KEEP_TILE + threadIdx.x;
    const uint64_t m = __ballot(t < n && keep[t] != 0);
    if ((threadIdx.x & 63) == 0 && m) atomicAdd(&cnt, (int32_t)__popcll(m));
    __syncthreads();
    if (threadIdx.x == 0) tiles[blockIdx.x] = cnt;
}

// Kept blocks, in their (Morton) order: keys and source blocks of the result,
// their number, and the squared norm of the k = n - kept smallest (excl:
// exclusive scan of the sorted norms).
__global__ __launch_bounds__(KEEP_TILE) void k_keep_write(const int32_t* __restrict__ keep, int64_t n,
                                                         const int32_t* __restrict__ tiles,
                                                         const int32_t* __restrict__ total,
                                                         const uint64_t* __restrict__ bkey,
                                                         const double* __restrict__ excl,
                                                         const double* __restrict__ sorted,
                                                         uint64_t* __restrict__ okey, int32_t* __restrict__ src,
                                                         int32_t* __restrict__ count, double* __restrict__ removed2) {
    __shared__ int32_t wcnt[KEEP_TILE / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t t = (int64_t)blockIdx.x * KEEP_TILE + threadIdx.x;
    const bool k = t < n && keep[t] != 0;
    const uint64_t m = __ballot(k);
    if (lane == 0) wcnt[wave] = (int32_t)__popcll(m);
    __syncthreads();
    if (k) {
        int64_t o = tiles[blockIdx.x] + __popcll(m & (lane ? ~0ull >> (64 - lane) : 0ull));
        for (int w = 0; w < wave; ++w) o += wcnt[w];
        okey[o] = bkey[t];
        src[o] = (int32_t)t;
    }
    if (t == 0) {
        const int64_t gone = n - *total;
        *count = *total;
        *removed2 = gone > 0 ? excl[gone - 1] + sorted[gone - 1] : 0.0;
    }
}

qt_matrix* truncate(qt_matrix* M, double eps, hipStream_t s, int64_t* removed, double* removed_norm2) {
    if (!(eps >= 0.0)) fail(QT_ERR_ARG, "eps must be a non-negative number");
    const double* v = operand_f64(M, s);
    const int64_t n = M->nblocks;
    const int bb = M->b * M->b;
    if (removed) *removed = 0;
    if (removed_norm2) *removed_norm2 = 0.0;
    if (n == 0) return build(M->n_rows, M->n_cols, M->b, M->leaf, 0, nullptr, nullptr, nullptr, QT_MEM_DEVICE, s);
    std::unique_ptr<qt_matrix> T(shaped_like(M, M->L, s));
    const int64_t tiles = (n + KEEP_TILE - 1) / KEEP_TILE;
    DBuf<double> norm2(n, s), sorted(n, s), excl(n + 1, s), dtmp(scan_tmp_elems(n) + 1, s);
    DBuf<int32_t> idx(n, s), keep(n, s), tcnt(tiles + 1, s), stmp(sort_tmp_words(n, 64), s), src(n, s);
    T->bkey.alloc(n, s);
    TreeJob job;
    tree_begin(job, T.get(), n, 0, s);
    launch_block_norm2(M, norm2.p, s);
    stable_sort(NormKeys{norm2.p}, NormSink{sorted.p, idx.p}, n, 64, stmp.p, idx.p, s);
    exclusive_scan(sorted.p, excl.p, n, dtmp.p, s);
    k_trunc_flags<<<grid_for(n), 256, 0, s>>>(excl.p, sorted.p, n, eps * eps, idx.p, keep.p);
    QT_LAUNCH("k_trunc_flags");
    k_keep_tiles<<<(unsigned)tiles, KEEP_TILE, 0, s>>>(keep.p, n, tcnt.p);
    QT_LAUNCH("k_keep_tiles");
    k_radix_scan<<<1, 1024, 0, s>>>(tcnt.p, tcnt.p + tiles, 1, (int)tiles);
    QT_LAUNCH("k_radix_scan");
    k_keep_write<<<(unsigned)tiles, KEEP_TILE, 0, s>>>(keep.p, n, tcnt.p, tcnt.p + tiles, M->bkey.p, excl.p, sorted.p,
                                                       T->bkey.p, src.p, job.count(), job.sum());
    QT_LAUNCH("k_keep_write");
    tree_fill(job, T->bkey.p, s);
    double gone2 = 0.0;
    tree_finish(job, s, &gone2);
    const int64_t nk = T->nblocks;
    if (removed) *removed = n - nk;
    if (removed_norm2) *removed_norm2 = gone2;
    T->v64.alloc((size_t)nk * bb, s);
    if (nk > 0) copy_blocks(v, src.p, nk, bb, T->v64.p, s);
    QT_HIP(hipStreamSynchronize(s));
    return T.release();
}

void get_blocks(const qt_matrix* M, int64_t count, const int32_t* I, const int32_t* J, void* values,
                int32_t* found, qt_prec out_type, qt_mem where, hipStream_t s) {
    if (out_type != QT_F64 && out_type != QT_F32) fail(QT_ERR_UNSUPPORTED, "output type must be F64 or F32");
    if (where != QT_MEM_HOST && where != QT_MEM_DEVICE) fail(QT_ERR_ARG, "bad memory kind");
    if (count < 0) fail(QT_ERR_ARG, "negative count");
    if (count == 0) return;
    if (!I || !J || !values || !found) fail(QT_ERR_ARG, "NULL array");
    const int bb = M->b * M->b;
    const size_t esz = out_type == QT_F64 ? sizeof(double) : sizeof(float);
    DBuf<int32_t> dI, dJ, dF;
    DBuf<char> dV;
    const int32_t* pI = I;
    const int32_t* pJ = J;
    int32_t* pF = found;
    void* pV = values;
    if (where == QT_MEM_HOST) {
        dI.alloc(count, s);
        dJ.alloc(count, s);
        dF.alloc(count, s);
        dV.alloc((size_t)count * bb * esz, s);
        QT_HIP(hipMemcpyAsync(dI.p, I, count * sizeof(int32_t), hipMemcpyHostToDevice, s));
        QT_HIP(hipMemcpyAsync(dJ.p, J, count * sizeof(int32_t), hipMemcpyHostToDevice, s));
        pI = dI.p;
        pJ = dJ.p;
        pF = dF.p;
        pV = dV.p;
    }
    const int64_t nbr = M->n_rows / M->b, nbc = M->n_cols / M->b;
    const unsigned g = block_grid(count);
    const bool src64 = M->vtype == QT_F64;
    if (src64 && out_type == QT_F64)
        k_get_blocks<double, double><<<g, 256, 0, s>>>(M->bkey.p, M->nblocks, nbr, nbc, M->v64.p, pI, pJ, count, bb,
                                                      (double*)pV, pF);
    else if (src64)
        k_get_blocks<double, float><<<g, 256, 0, s>>>(M->bkey.p, M->nblocks, nbr, nbc, M->v64.p, pI, pJ, count, bb,
                                                     (float*)pV, pF);
    else if (out_type == QT_F64)
        k_get_blocks<float, double><<<g, 256, 0, s>>>(M->bkey.p, M->nblocks, nbr, nbc, M->v32.p, pI, pJ, count, bb,
                                                     (double*)pV, pF);
    else
        k_get_blocks<float, float><<<g, 256, 0, s>>>(M->bkey.p, M->nblocks, nbr, nbc, M->v32.p, pI, pJ, count, bb,
                                                    (float*)pV, pF);
    QT_LAUNCH("k_get_blocks");
    if (where == QT_MEM_HOST) {
        QT_HIP(hipMemcpyAsync(found, pF, count * sizeof(int32_t), hipMemcpyDeviceToHost, s));
        QT_HIP(hipMemcpyAsync(values, pV, (size_t)count * bb * esz, hipMemcpyDeviceToHost, s));
        QT_HIP(hipStreamSynchronize(s));
    }
}

}  // namespace qt
