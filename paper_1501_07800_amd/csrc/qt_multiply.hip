// C = A*B: symbolic traversal of both quadtrees, then the numeric kernel.
//
// Algorithm 1 of the paper recurses from the roots: a pair of present nodes
// (A_mk, B_kn) spawns the eight child pairs (A_m'k', B_k'n'), pairs with a
// NIL operand are dropped, and at the leaves the block-sparse leaf multiply
// runs; Algorithm 2 then sums the products landing on the same C node.
//
// On the GPU the recursion runs breadth-first, one level per step, with the
// frontier of pairs grouped by the C node they contribute to and, inside a
// group, in ascending inner index k. One wavefront owns one C node:
//   count: it counts, for each of the four child quadrants (m, n), the child
//          pairs present(A_m0) & present(B_0n) + present(A_m1) & present(B_1n)
//          over its pairs, giving (child pairs, child C nodes) packed in an
//          int64;
//   offsets: an exclusive prefix sum of those packed counts gives every C
//          node the place of its child pairs and child C nodes in the next
//          level (from per-workgroup aggregates, or a scan for large levels);
//   fill:  it writes its child pairs, quadrant by quadrant, pairs in order and
//          k' = 0 before k' = 1 (child k = 2k + k'), so the new frontier is
//          again grouped by C node with k ascending; quadrants without pairs
//          are NIL children and get no node.
// A level takes one launch (its counts are made by the fill before it) or two
// (count, fill), plus a scan on the largest. Three kinds of product go other
// ways to the same lists: levels of few pairs per node and leaves of few
// products give a lane, not a wave, to a pair; a small product runs in one
// launch; the problems of a batch share launches (each below, where it says
// why).
//
// The leaf step gives a C leaf one wavefront whose lanes are the lb x lb
// blocks of the leaf: lane (i, j) counts popcount(rowmask_A(i) & colmask_B(j))
// over the leaf pairs of the C leaf, then lists its products, pair by pair,
// k ascending. The result is the product list of every C block with C blocks
// in Morton order -- which is also C's block order, so no sort is needed, and
// since the order of products inside a C block does not depend on the leaf
// size, neither does the result.
//
// The number of pairs at every level and the number of block products are
// known on the host before any launch (from per-level row/column counts of
// both operands), so all buffers are sized up front in two allocations (the
// result's tree, and scratch); the single synchronization reads back how many
// C blocks there are before C's values are allocated. A level's per-node
// arrays and its grids are sized by a bound on its C nodes: the smaller of its
// pair count and the number of node positions C's shape has at that level.
// Once the C block count is known, a launch order of C's blocks may also be
// built: strips of block rows, or a grouping by inner index (see "launch
// order" below).
// The whole phase runs on a stream of the library, beside the caller's (see
// side_stream below).
#include "qt_internal.h"
#include "qt_morton.h"
#include "qt_readback.h"
#include "qt_sort.h"

#include <algorithm>
#include <deque>
#include <map>
#include <string>

namespace qt {

// ------------------------------------------------------------- helpers

__device__ __forceinline__ int64_t pack2(int32_t lo, int32_t hi) {
    return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}
__device__ __forceinline__ int32_t lo32(int64_t v) { return (int32_t)(uint32_t)((uint64_t)v & 0xffffffffu); }
__device__ __forceinline__ int32_t hi32(int64_t v) { return (int32_t)((uint64_t)v >> 32); }

__device__ __forceinline__ uint64_t lanes_below(int lane) { return lane ? (~0ull >> (64 - lane)) : 0ull; }

// Inclusive prefix sum over the wave with data-parallel row moves: one add
// each, where a general shuffle goes through the LDS crossbar (the leaf
// kernels are bound by instructions and these chains).
__device__ __forceinline__ int wave_incl_scan(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // from 1 lane below, within a row of 16
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);   // 2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);   // 4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);   // 8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // a row's last lane into the next: rows 1, 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // lane 31 into rows 2 and 3
    return x;
}

__device__ __forceinline__ int wave_sum(int x) { return __builtin_amdgcn_readlane(wave_incl_scan(x), 63); }

__device__ __forceinline__ int wave_excl_scan(int x) { return wave_incl_scan(x) - x; }

// bits k of row r of an lb x lb occupancy mask stored row-major
__device__ __forceinline__ uint32_t mask_row(uint64_t m, int r, int lb) {
    return (uint32_t)((m >> (r * lb)) & ((1ull << lb) - 1));
}

// the OR of all lb rows of such a mask: bit k set iff column k holds a block
// (for a column-major mask: bit k set iff row k does)
__device__ __forceinline__ uint32_t mask_fold(uint64_t m, int lb) {
    for (int sh = lb * lb / 2; sh >= lb; sh >>= 1) m |= m >> sh;
    return (uint32_t)(m & ((1ull << lb) - 1));
}

// ------------------------------------------------- one level of the tree

struct TreeStep {
    // this level
    const int32_t* fa;        // A node of each pair
    const int32_t* fb;        // B node of each pair
    const int32_t* cseg;      // pairs of C node c: cseg[c] .. cseg[c+1]-1
    const uint64_t* ckey;     // Morton key of C node c
    const int32_t* ncount;    // number of C nodes (device)
    const int32_t* Ach;       // child tables of A and B at this level
    const int32_t* Bch;
    int64_t* cnt;             // per C node: (child pairs, child C nodes)
    int4* tot4;               // per C node: child pairs per quadrant
    int64_t* off;             // exclusive scan of cnt; off[ncap] = totals (scan path)
                              // or each node's offset inside its workgroup (aggregate path)
    int64_t* wagg;            // aggregate path: per count workgroup, the sum of its nodes' cnt
    int64_t* gsum;            // aggregate path: per group of 64 count workgroups, their sum (zeroed first)
    int use_agg;              // offsets from workgroup aggregates instead of a scan
    int32_t ncap;             // bound on C nodes at this level
    int32_t group;            // levels of few pairs per node: C nodes per wave
    // next level
    int32_t* nfa;
    int32_t* nfb;
    int32_t* ncseg;
    uint64_t* nckey;
    int32_t* cchild;          // C's child table at this level (4 per node), before NIL normalisation
    int32_t* nparent;         // parent (C node at this level) of every C node of the next level
    int32_t* ncount_next;
    int32_t np_next;          // bound on pairs at the next level (exact unless `upper`)
    int32_t nc_next;          // bound on C nodes at the next level
    int32_t* check;           // device total of child pairs, for the host check
    int ta, tb;               // operand used transposed: child (m, k) of op(A) is child (k, m) of A
    int upper;                // keep only C nodes on or above the block diagonal
    const double* An2;        // squared norms of the operands' next-level nodes (nullptr: no
    const double* Bn2;        // norm threshold): a child pair is dropped when An2 Bn2 < tau2
    double tau2;
    // The next level's counts, made by this level's fill when ncnt is set (a
    // single-wave next level): the fill holds every pair of each child node it
    // creates, so it counts their child pairs too, and the next level needs no
    // count kernel of its own.
    const int32_t* nAch;      // child tables of A and B at the next level
    const int32_t* nBch;
    const double* nAn2;       // norms of the nodes two levels down (norm threshold)
    const double* nBn2;
    int64_t* ncnt;            // the next level's cnt, tot4, off, wagg, gsum
    int4* ntot4;
    int64_t* noff;
    int64_t* nwagg;
    int64_t* ngsum;
};

// The norm threshold's one comparison, of squared norms: nodes and blocks, counts
// and lists alike. A product that is not a number (a NaN block, an infinite one
// times a zero one) is not kept; a count and a list that judged it differently
// would write over each other's places.
__device__ __forceinline__ bool norms_kept(double a2, double b2, double tau2) { return a2 * b2 >= tau2; }

// Child a of op(A) and child b of op(B) form a pair: both present and, with
// a norm threshold (PRUNE), the product of their norms not below it. PRUNE is
// a template argument of every traversal kernel: tested at run time, the
// norm loads sat behind 80 branches of k_tree_fill, 36 KB of code of which a
// level of a few nodes runs each line once, from a cold instruction cache.
template <bool PRUNE>
__device__ __forceinline__ bool pair_kept(const double* An2, const double* Bn2, double tau2, int32_t a, int32_t b) {
    if constexpr (PRUNE)
        return a >= 0 && b >= 0 && norms_kept(An2[a], Bn2[b], tau2);
    else
        return (a | b) >= 0;
}

// Children of an operand node in the orientation of op(X): for a transposed
// operand the off-diagonal children swap (quadrant (m, k) of X^T is (k, m) of X).
__device__ __forceinline__ int4 op_swap(int4 c, int transposed) {
    if (transposed) {
        const int t = c.y;
        c.y = c.z;
        c.z = t;
    }
    return c;
}

// The child tables of A node a and B node b, both loads issued before either
// is used (left alone, the compiler waits for the first before it issues
// the second).
__device__ __forceinline__ void op_children2(const int32_t* atab, int32_t a, int ta, const int32_t* btab, int32_t b,
                                             int tb, int4& x, int4& y) {
    const int4 ra = *reinterpret_cast<const int4*>(atab + 4 * (int64_t)a);
    const int4 rb = *reinterpret_cast<const int4*>(btab + 4 * (int64_t)b);
    __builtin_amdgcn_sched_barrier(0);
    x = op_swap(ra, ta);
    y = op_swap(rb, tb);
}

// Quadrant mn of C node `key` is dropped when only the upper triangle is
// wanted and the node lies on the diagonal (its lower-left child is strictly
// below it); nodes off the diagonal are entirely above it.
__device__ __forceinline__ bool quadrant_dropped(int upper, uint64_t key, int mn) {
    return upper && mn == 2 && morton_row(key) == morton_col(key);
}

template <bool PRUNE>
__device__ __forceinline__ int64_t tree_count_node(const TreeStep& st, int32_t c, int lane) {
    if (c >= *st.ncount) {
        if (lane == 0) st.cnt[c] = 0;
        return 0;
    }
    const int32_t s0 = st.cseg[c], len = st.cseg[c + 1] - s0;
    int t0 = 0, t1 = 0, t2 = 0, t3 = 0;
    for (int32_t base = 0; base < len; base += 64) {
        if (base + lane < len) {
            const int32_t p = s0 + base + lane;
            int4 a, b;   // A child (m, k) at 2m + k, B child (k, n) at 2k + n
            op_children2(st.Ach, st.fa[p], st.ta, st.Bch, st.fb[p], st.tb, a, b);
            auto kept = [&](int32_t x, int32_t y) { return pair_kept<PRUNE>(st.An2, st.Bn2, st.tau2, x, y); };
            t0 += kept(a.x, b.x) + kept(a.y, b.z);
            t1 += kept(a.x, b.y) + kept(a.y, b.w);
            t2 += kept(a.z, b.x) + kept(a.w, b.z);
            t3 += kept(a.z, b.y) + kept(a.w, b.w);
        }
    }
    if (quadrant_dropped(st.upper, st.ckey[c], 2)) t2 = 0;
    t0 = wave_sum(t0);
    t1 = wave_sum(t1);
    t2 = wave_sum(t2);
    t3 = wave_sum(t3);
    const int64_t v = pack2(t0 + t1 + t2 + t3, (t0 > 0) + (t1 > 0) + (t2 > 0) + (t3 > 0));
    if (lane == 0) {
        st.cnt[c] = v;
        st.tot4[c] = make_int4(t0, t1, t2, t3);
    }
    return v;
}

// Totals T = (child pairs, child C nodes) of a whole level.
__device__ void tree_level_totals(const TreeStep& st, int64_t T) {
    const int32_t nc_next = hi32(T);
    *st.ncount_next = nc_next;
    if (nc_next <= st.nc_next) st.ncseg[nc_next] = lo32(T);
    *st.check = lo32(T);
}

// Workgroup aggregates of a level are summed in groups of 64 (aggregate path, below).
constexpr int AGG_GROUP_LOG = 6;

// Counting the next level's child pairs (the rule of tree_count_node one
// level down). A pair of child tables x, y gives quadrant q = 2m + n the pairs
// k' = 0 and 1 for which x(m, k') and y(k', n) are both present: with the
// presence bits spread over the bytes of a word per k', byte q, two ANDs and
// an add count all four quadrants at once. A lane adds up its own pairs that
// way; the lanes are summed once per node. (Counted with a ballot per
// quadrant and k', 64 of them per 64 pairs into 16 scalar counters, the
// compiler ran out of scalar registers: 800 of k_tree_fill's 3400 instructions
// moved spilled ones, 36 KB of code. With this and the template arguments
// above, 12 KB, the traversal of decay32768 went from 0.162 to 0.130 ms alone,
// of a random 48000 product from 0.386 to 0.334.)
struct QuadBytes {
    uint32_t k0, k1;
};

__device__ __forceinline__ uint32_t present(int32_t node) { return (uint32_t)~node >> 31; }

__device__ __forceinline__ QuadBytes a_bytes(int4 x, uint32_t has) {
    return {(present(x.x) * 0x00000101u + present(x.z) * 0x01010000u) * has,
            (present(x.y) * 0x00000101u + present(x.w) * 0x01010000u) * has};
}
__device__ __forceinline__ QuadBytes b_bytes(int4 y, uint32_t has) {
    return {(present(y.x) * 0x00010001u + present(y.y) * 0x01000100u) * has,
            (present(y.z) * 0x00010001u + present(y.w) * 0x01000100u) * has};
}

// Byte q: the child pairs of quadrant q that a norm threshold keeps.
__device__ __forceinline__ uint32_t pruned_bytes(const double* An2, const double* Bn2, double tau2, int4 x, int4 y) {
    const int xa[4] = {x.x, x.y, x.z, x.w}, yb[4] = {y.x, y.y, y.z, y.w};
    uint32_t u = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int k = 0; k < 2; ++k)
            u += (uint32_t)pair_kept<true>(An2, Bn2, tau2, xa[(q & 2) + k], yb[2 * k + (q & 1)]) << (8 * q);
    return u;
}

// The child table of one child of a pair: a NIL child reads node 0 (every
// level of a non-empty operand has one) and its value is dropped, so the loads
// need no branch.
__device__ __forceinline__ int4 next_table(const int32_t* tab, int32_t node) {
    return *reinterpret_cast<const int4*>(tab + 4 * (int64_t)(node >= 0 ? node : 0));
}

constexpr int QUAD_FLUSH = 60;   // chunks of 64 pairs after which a byte (at most 4 per chunk) is added up

// Lanes with bit 8 h set keep the upper h of 2 h words, the others the lower.
template <int H>
__device__ __forceinline__ void halve(uint32_t (&w)[8], int lane) {
    const bool up = lane & (8 * H);
#pragma unroll
    for (int i = 0; i < H; ++i) {
        const uint32_t keep = up ? w[i + H] : w[i], give = up ? w[i] : w[i + H];
        w[i] = keep + __shfl_xor(give, 8 * H, 64);
    }
}

// Sums u[mn] over the wave; lane mn adds its quadrants' totals to mine[0..3].
__device__ __forceinline__ void quad_flush(uint32_t (&u)[4], int lane, int (&mine)[4]) {
    uint32_t w[8];   // 16-bit sums: quadrants 0 and 2, 1 and 3 of child mn
#pragma unroll
    for (int mn = 0; mn < 4; ++mn) {
        w[2 * mn] = u[mn] & 0x00ff00ffu;
        w[2 * mn + 1] = (u[mn] >> 8) & 0x00ff00ffu;
        u[mn] = 0;
    }
    // halving exchanges: lanes 8 i .. 8 i + 7 end up with word i
    halve<4>(w, lane);
    halve<2>(w, lane);
    halve<1>(w, lane);
#pragma unroll
    for (int d = 4; d >= 1; d >>= 1) w[0] += __shfl_xor(w[0], d, 64);
    const uint32_t even = __shfl(w[0], (16 * lane) & 63, 64), odd = __shfl(w[0], (16 * lane + 8) & 63, 64);
    mine[0] += even & 0xffffu;
    mine[1] += odd & 0xffffu;
    mine[2] += even >> 16;
    mine[3] += odd >> 16;
}

// The counts of c's children, as the next level's count kernel would write
// them for single-wave workgroups (node c2 is workgroup c2, its offset inside
// the workgroup 0); lane mn writes those of child quadrant mn: node c2 (-1:
// none) with child pairs mine[0..3].
__device__ __forceinline__ void next_level_write(const TreeStep& st, int32_t c, int lane, int c2, int (&mine)[4]) {
    if (lane >= 4 || c2 < 0 || c2 >= st.nc_next) return;
    if (quadrant_dropped(st.upper, st.ckey[c] * 4 + (uint64_t)lane, 2)) mine[2] = 0;
    const int64_t v = pack2(mine[0] + mine[1] + mine[2] + mine[3],
                            (mine[0] > 0) + (mine[1] > 0) + (mine[2] > 0) + (mine[3] > 0));
    st.ncnt[c2] = v;
    st.ntot4[c2] = make_int4(mine[0], mine[1], mine[2], mine[3]);
    st.noff[c2] = 0;
    st.nwagg[c2] = v;
    if (v) atomicAdd((unsigned long long*)(st.ngsum + (c2 >> AGG_GROUP_LOG)), (unsigned long long)v);
}

// o: (first child pair, first child C node) of node c in the next level.
template <bool PRUNE, bool COUNTS>
__device__ __forceinline__ void tree_fill_node(const TreeStep& st, int32_t c, int lane, int64_t o) {
    if (c >= *st.ncount) return;
    const int4 t4 = st.tot4[c];
    const int t[4] = {t4.x, t4.y, t4.z, t4.w};
    int run[4], my_c = -1;
    {
        int pr = lo32(o), ci = hi32(o), my_run = 0;
#pragma unroll
        for (int mn = 0; mn < 4; ++mn) {
            run[mn] = pr;
            if (lane == mn && t[mn] > 0) {
                my_c = ci;
                my_run = pr;
            }
            pr += t[mn];
            ci += t[mn] > 0 ? 1 : 0;
        }
        if (lane < 4) {
            st.cchild[4 * (int64_t)c + lane] = my_c;
            if (my_c >= 0 && my_c < st.nc_next) {
                st.nckey[my_c] = st.ckey[c] * 4 + (uint64_t)lane;
                st.ncseg[my_c] = my_run;
                st.nparent[my_c] = c;
            }
        }
    }
    const int32_t s0 = st.cseg[c], len = st.cseg[c + 1] - s0;
    const uint64_t below = lanes_below(lane);
    const bool drop_lower = quadrant_dropped(st.upper, st.ckey[c], 2);
    uint32_t u[4] = {0, 0, 0, 0};      // per child quadrant mn of c: bytes of its child pairs, this lane's
    int mine[4] = {0, 0, 0, 0}, chunks = 0;
    for (int32_t base = 0; base < len; base += 64) {
        const bool act = base + lane < len;
        int4 a = make_int4(-1, -1, -1, -1), b = make_int4(-1, -1, -1, -1);
        if (act) {
            const int32_t p = s0 + base + lane;
            op_children2(st.Ach, st.fa[p], st.ta, st.Bch, st.fb[p], st.tb, a, b);
        }
        const int av[4] = {a.x, a.y, a.z, a.w};
        const int bv[4] = {b.x, b.y, b.z, b.w};
        // this lane's pair k' of child quadrant mn
        auto kept = [&](int mn, int k) {
            const int x = av[(mn & 2) + k], y = bv[2 * k + (mn & 1)];
            return !(mn == 2 && drop_lower) && pair_kept<PRUNE>(st.An2, st.Bn2, st.tau2, x, y);
        };
        // the next level's counts first, the chunk's pair stores after them: a
        // wait for loads issued after stores would wait for the stores too
        if constexpr (COUNTS) {
            int4 x[4], y[4];   // the eight children's tables: each serves two quadrants
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                x[q] = next_table(st.nAch, av[q]);
                y[q] = next_table(st.nBch, bv[q]);
            }
            __builtin_amdgcn_sched_barrier(0);   // all eight loads before the first use
            if constexpr (PRUNE) {
#pragma unroll
                for (int mn = 0; mn < 4; ++mn)
#pragma unroll
                    for (int k = 0; k < 2; ++k)
                        if (kept(mn, k))
                            u[mn] += pruned_bytes(st.nAn2, st.nBn2, st.tau2, x[(mn & 2) + k], y[2 * k + (mn & 1)]);
            } else {
                QuadBytes xa[4], yb[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    xa[q] = a_bytes(op_swap(x[q], st.ta), present(av[q]));
                    yb[q] = b_bytes(op_swap(y[q], st.tb), present(bv[q]));
                }
#pragma unroll
                for (int mn = 0; mn < 4; ++mn) {
                    uint32_t v = 0;
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const QuadBytes &xk = xa[(mn & 2) + k], &yk = yb[2 * k + (mn & 1)];
                        v += (xk.k0 & yk.k0) + (xk.k1 & yk.k1);
                    }
                    u[mn] += (mn == 2 && drop_lower) ? 0u : v;
                }
            }
            if (++chunks == QUAD_FLUSH) {
                quad_flush(u, lane, mine);
                chunks = 0;
            }
        }
#pragma unroll
        for (int mn = 0; mn < 4; ++mn) {
            const int m = mn >> 1, n = mn & 1;
            const bool e0 = kept(mn, 0), e1 = kept(mn, 1);
            const uint64_t m0 = __ballot(e0), m1 = __ballot(e1);
            int w = run[mn] + __popcll(m0 & below) + __popcll(m1 & below);
            run[mn] += __popcll(m0) + __popcll(m1);
            if (e0) {
                if (w < st.np_next) {
                    st.nfa[w] = av[2 * m];
                    st.nfb[w] = bv[n];
                }
                ++w;
            }
            if (e1 && w < st.np_next) {
                st.nfa[w] = av[2 * m + 1];
                st.nfb[w] = bv[2 + n];
            }
        }
    }
    if constexpr (COUNTS) {
        quad_flush(u, lane, mine);
        next_level_write(st, c, lane, my_c, mine);
    }
}

// The per-level kernels run W waves (one C node each) per workgroup: W = 1
// for levels of up to WIDE_LEVEL nodes, so that while a previous numeric
// kernel still fills the GPU with single-wave workgroups the traversal's
// workgroups find room as soon as any wave ends (a wider workgroup waits for
// several free slots on one CU); W = 4 above that, where the number of
// workgroups itself costs.
constexpr int64_t WIDE_LEVEL = 65536;
static inline int level_waves(int64_t n) { return n <= WIDE_LEVEL ? 1 : 4; }

constexpr int32_t AGG_MAX = 65536;   // workgroups per level on the aggregate path

// Sum over the wave of packed pairs of counts (neither half overflows).
__device__ __forceinline__ int64_t wave_sum_pack2(int64_t x) { return pack2(wave_sum(lo32(x)), wave_sum(hi32(x))); }

// Aggregate path, count side: node offsets inside the workgroup and the
// workgroup's aggregate, from each wave's packed count v.
template <int W>
__device__ __forceinline__ void level_local_offsets(int64_t v, int32_t c, int32_t ncap, int64_t* off,
                                                    int64_t* wagg, int64_t* gsum, int64_t* lds) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) lds[wave] = v;
    __syncthreads();
    if (lane == 0 && c < ncap) {
        int64_t pre = 0;
        for (int w = 0; w < wave; ++w) pre += lds[w];
        off[c] = pre;
    }
    if (threadIdx.x == 0) {
        int64_t tot = 0;
        for (int w = 0; w < W; ++w) tot += lds[w];
        wagg[blockIdx.x] = tot;
        if (tot) atomicAdd((unsigned long long*)(gsum + (blockIdx.x >> AGG_GROUP_LOG)), (unsigned long long)tot);
    }
}

// Aggregate path, fill side: the sum of the aggregates of all earlier
// workgroups (every thread gets it).
template <int W>
__device__ __forceinline__ int64_t level_base(const int64_t* wagg, const int64_t* gsum, int64_t* lds,
                                              int32_t b = (int32_t)blockIdx.x) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t g = b >> AGG_GROUP_LOG, first = g << AGG_GROUP_LOG;
    int64_t part = 0;
    for (int32_t i = threadIdx.x; i < g; i += 64 * W) part += gsum[i];
    for (int32_t i = first + threadIdx.x; i < b; i += 64 * W) part += wagg[i];
    part = wave_sum_pack2(part);
    if (lane == 0) lds[wave] = part;
    __syncthreads();
    int64_t base = 0;
    for (int w = 0; w < W; ++w) base += lds[w];
    return base;
}

// Only the first ncount of the ncap node slots hold C nodes: on the aggregate
// path a workgroup whose slots are all past ncount has a zero aggregate and
// nothing to fill, and only the last workgroup (which writes the level's
// totals) still runs.
template <int W>
__device__ __forceinline__ bool level_wg_empty(const int32_t* ncount) {
    return (int64_t)blockIdx.x * W >= *ncount;
}

// The last workgroup of a level of ncap >= 1 node slots.
template <int W>
__device__ __forceinline__ bool level_wg_last(int32_t ncap) {
    return (int32_t)blockIdx.x == (ncap - 1) / W;
}

template <int W, bool PRUNE>
__device__ __forceinline__ void tree_count_level(const TreeStep& st) {
    __shared__ int64_t lds[W];
    if (st.use_agg && level_wg_empty<W>(st.ncount)) {
        if (threadIdx.x == 0) st.wagg[blockIdx.x] = 0;
        return;
    }
    const int32_t c = (int32_t)(blockIdx.x * W + (threadIdx.x >> 6));
    int64_t v = 0;
    if (c < st.ncap) v = tree_count_node<PRUNE>(st, c, threadIdx.x & 63);
    if (st.use_agg) level_local_offsets<W>(v, c, st.ncap, st.off, st.wagg, st.gsum, lds);
}

template <int W, bool PRUNE>
__global__ __launch_bounds__(64 * W) void k_tree_count(TreeStep st) {
    tree_count_level<W, PRUNE>(st);
}

// COUNTS: the fill also makes the next level's counts (st.ncnt is set).
template <int W, bool PRUNE, bool COUNTS>
__device__ __forceinline__ void tree_fill_level(const TreeStep& st) {
    __shared__ int64_t lds[W];
    const int32_t c = (int32_t)(blockIdx.x * W + (threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    if (st.use_agg) {
        const bool last = level_wg_last<W>(st.ncap);
        if (level_wg_empty<W>(st.ncount) && !last) return;
        const int64_t base = level_base<W>(st.wagg, st.gsum, lds);
        if (last && threadIdx.x == 0) tree_level_totals(st, base + st.wagg[blockIdx.x]);
        if (c < st.ncap) tree_fill_node<PRUNE, COUNTS>(st, c, lane, base + st.off[c]);
    } else {
        if (c == 0 && lane == 0) tree_level_totals(st, st.off[st.ncap]);
        if (c < st.ncap) tree_fill_node<PRUNE, COUNTS>(st, c, lane, st.off[c]);
    }
}

template <int W, bool PRUNE, bool COUNTS>
__global__ __launch_bounds__(64 * W) void k_tree_fill(TreeStep st) {
    tree_fill_level<W, PRUNE, COUNTS>(st);
}

// ------------------------------------------ levels of few pairs per node
//
// The deep levels of an unstructured product have many C nodes of a few pairs
// (an R-MAT product of 39634 blocks of 16 has 2.2 M pairs in 475 k nodes on its
// last level), where a wave per node is mostly idle lanes and its own chain of
// loads. Here a lane takes a pair, and a wave the pairs of
// `group` nodes, 64 at a time. The count adds a pair's four quadrant counts (0
// to 2 each) to its node's in LDS. The fill scans them over the lanes, a byte
// per quadrant (at most 128 in 64 lanes): a child pair's place is its node's
// quadrant's first, plus the scan here less the scan at the node's first lane.
// Pairs, nodes and their order are the same as with a wave per node.
// On that product's two widest tree levels 271 -> 133 us, counts, scan and fills
// together. Left are the chain of loads of each 64 pairs, about 3 us, and the
// scattered child tables.
// Chosen from TREE_MIN positions (below, the counts that the wave-per-node fill
// makes for the next level save a launch) and up to TREE_PAIRS pairs per position.
// The symbolic phase, node per wave and pair per lane, in us: R-MAT of 8192, 2
// edges a row: 422 and 290, 5 edges: 650 and 503; of 2048: 185 and 180; with no
// bound on the pairs per position: random of 1500 block rows 234 and 246, R-MAT
// of 4096 with 10 edges 450 and 479. With TREE_MIN a quarter or four times as
// large: within 3 us.
constexpr int TREE_GROUP_MAX = 64;     // C nodes per wave
constexpr int64_t TREE_MIN = 8192;     // C node positions of a level
constexpr int64_t TREE_PAIRS = 24;     // pairs per position

// Of the pairs base .. base + 63, the C node (lane of the wave) that this
// lane's pair belongs to, and the first lane of that node's pairs; seg: the
// first pair of the node of each lane (INT32_MAX past the last). Every C node
// has a pair. mark: 64 words of LDS.
__device__ __forceinline__ int pair_node(int32_t seg, int32_t base, int lane, int32_t* mark, int& head) {
    mark[lane] = 0;
    __syncthreads();
    const bool here = seg >= base && seg - base < 64;
    if (here) mark[seg - base] = 1;
    __syncthreads();
    const uint64_t heads = __ballot(mark[lane] != 0) & (lanes_below(lane) | (1ull << lane));
    const int before = __popcll(__ballot(seg < base));
    __syncthreads();
    head = heads ? 63 - __clzll((long long)heads) : 0;
    return before + __popcll(heads) - 1;
}

// Byte q: the child pairs of quadrant q of a pair with child tables a, b.
__device__ __forceinline__ uint32_t quad_counts(int4 a, int4 b) {
    const QuadBytes x = a_bytes(a, 1), y = b_bytes(b, 1);
    return (x.k0 & y.k0) + (x.k1 & y.k1);
}

__global__ __launch_bounds__(64) void k_tree_count_sparse(TreeStep st) {
    __shared__ int32_t mark[64];
    __shared__ unsigned long long quads[64];   // 16 bits each: quadrants 0, 2, 1, 3
    const int lane = threadIdx.x;
    const int32_t n = *st.ncount, c0 = (int32_t)blockIdx.x * st.group;
    if (c0 >= n) {
        if (lane == 0) st.wagg[blockIdx.x] = 0;
        return;
    }
    const int32_t nl = min(st.group, n - c0), c = c0 + lane;
    const int32_t seg = lane < nl ? st.cseg[c] : INT32_MAX;
    const int32_t end = st.cseg[c0 + nl];
    quads[lane] = 0;
    for (int32_t base = __builtin_amdgcn_readfirstlane(seg); base < end; base += 64) {
        uint32_t v = 0;
        if (base + lane < end) {
            int4 a, b;
            op_children2(st.Ach, st.fa[base + lane], st.ta, st.Bch, st.fb[base + lane], st.tb, a, b);
            v = quad_counts(a, b);
        }
        int head;
        const int q = pair_node(seg, base, lane, mark, head);
        if (v)
            atomicAdd(&quads[q], (unsigned long long)(v & 0x00ff00ffu) |
                                     ((unsigned long long)((v >> 8) & 0x00ff00ffu) << 32));
    }
    __syncthreads();
    const unsigned long long u = quads[lane];
    const int t0 = (int)(u & 0xffffu), t2 = (int)((u >> 16) & 0xffffu), t1 = (int)((u >> 32) & 0xffffu),
              t3 = (int)(u >> 48);
    const int np = t0 + t1 + t2 + t3, nn = (t0 > 0) + (t1 > 0) + (t2 > 0) + (t3 > 0);
    const int s_np = wave_incl_scan(np), s_nn = wave_incl_scan(nn);
    if (lane < nl) {
        st.off[c] = pack2(s_np - np, s_nn - nn);
        st.tot4[c] = make_int4(t0, t1, t2, t3);
    }
    if (lane == 63) {
        const int64_t tot = pack2(s_np, s_nn);
        st.wagg[blockIdx.x] = tot;
        if (tot) atomicAdd((unsigned long long*)(st.gsum + (blockIdx.x >> AGG_GROUP_LOG)), (unsigned long long)tot);
    }
}

__global__ __launch_bounds__(64) void k_tree_fill_sparse(TreeStep st) {
    __shared__ int64_t lds[1];
    __shared__ int32_t mark[64];
    __shared__ int32_t run[64][4];             // next place of each node's quadrants' child pairs
    const int lane = threadIdx.x;
    const int32_t n = *st.ncount, c0 = (int32_t)blockIdx.x * st.group;
    const bool last = (int32_t)blockIdx.x == (st.ncap - 1) / st.group;
    if (c0 >= n && !last) return;
    const int64_t base0 = level_base<1>(st.wagg, st.gsum, lds);
    if (last && lane == 0) tree_level_totals(st, base0 + st.wagg[blockIdx.x]);
    if (c0 >= n) return;
    const int32_t nl = min(st.group, n - c0), c = c0 + lane;
    const int32_t seg = lane < nl ? st.cseg[c] : INT32_MAX;
    const int32_t end = st.cseg[c0 + nl];
    if (lane < nl) {
        const int4 t4 = st.tot4[c];
        const int t[4] = {t4.x, t4.y, t4.z, t4.w};
        const int64_t o = base0 + st.off[c];
        const uint64_t key = st.ckey[c] * 4;
        int pr = lo32(o), ci = hi32(o), child[4];
#pragma unroll
        for (int mn = 0; mn < 4; ++mn) {
            run[lane][mn] = pr;
            child[mn] = t[mn] > 0 ? ci : -1;
            if (t[mn] > 0 && ci < st.nc_next) {
                st.nckey[ci] = key + (uint64_t)mn;
                st.ncseg[ci] = pr;
                st.nparent[ci] = c;
            }
            pr += t[mn];
            ci += t[mn] > 0 ? 1 : 0;
        }
        *reinterpret_cast<int4*>(st.cchild + 4 * (int64_t)c) = make_int4(child[0], child[1], child[2], child[3]);
    }
    for (int32_t base = __builtin_amdgcn_readfirstlane(seg); base < end; base += 64) {
        int4 a = make_int4(-1, -1, -1, -1), b = make_int4(-1, -1, -1, -1);
        if (base + lane < end)
            op_children2(st.Ach, st.fa[base + lane], st.ta, st.Bch, st.fb[base + lane], st.tb, a, b);
        int head;
        const int q = pair_node(seg, base, lane, mark, head);
        const uint32_t v = quad_counts(a, b), s = (uint32_t)wave_incl_scan((int)v);
        const uint32_t before = s - v - (uint32_t)__shfl((int)(s - v), head);   // of this node, in this chunk
        const int av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
        for (int mn = 0; mn < 4; ++mn) {
            int w = run[q][mn] + (int)((before >> (8 * mn)) & 255u);
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int x = av[(mn & 2) + k], y = bv[2 * k + (mn & 1)];
                if ((x | y) < 0) continue;
                if (w < st.np_next) {
                    st.nfa[w] = x;
                    st.nfb[w] = y;
                }
                ++w;
            }
        }
        __syncthreads();
        if (lane == 63)   // its node may go on in the next chunk
#pragma unroll
            for (int mn = 0; mn < 4; ++mn) run[q][mn] += (int)(((before + v) >> (8 * mn)) & 255u);
        __syncthreads();
    }
}

// Level-0 frontier: the pair of roots, one C node.
struct RootInit {
    int32_t* fa;
    int32_t* fb;
    int32_t* cseg;
    uint64_t* ckey;
    int32_t* ncount;
    int32_t* clear;           // NIL flags, group sums, workgroup aggregates (as words)
    int64_t nclear;
};

// The first kernel of the traversal: every workgroup clears its part of the
// scratch that later kernels accumulate into; the first writes the roots.
__device__ void root_init(const RootInit& r) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < r.nclear) r.clear[i] = 0;
    if (blockIdx.x != 0) return;
    if (threadIdx.x == 0) {
        r.fa[0] = 0;
        r.fb[0] = 0;
        r.cseg[0] = 0;
        r.cseg[1] = 1;
        r.ckey[0] = 0;
        r.ncount[0] = 1;
    }
}

__global__ __launch_bounds__(64) void k_root_init(RootInit r) { root_init(r); }

// ------------------------------------------------------ the leaf step

// NIL normalisation of C (see below): the leaf step's count flags every C leaf
// that receives a block, and its ancestors; its fill counts the flags per tile.
constexpr int NIL_MAX_LEVELS = 32;
constexpr int NIL_TILE = 256;   // four flags per lane

struct NilMark {
    int L;
    int64_t foff[NIL_MAX_LEVELS + 2];              // flags of level l at foff[l] .. foff[l+1]-1
    const int32_t* uparent[NIL_MAX_LEVELS + 1];    // parent of every C node, levels 1 .. L
    int32_t* flags;                                // foff[L+1] entries (whole tiles), cleared before the traversal
    int32_t* tcnt;                                 // flags set per tile
    int64_t tiles;                                 // foff[L+1] / NIL_TILE + 1
};

// C leaf c holds a block: it and its ancestors are kept. A walk stops at the
// first ancestor flagged already: whoever flagged it walks on from there. Two
// waves may both find an ancestor unflagged and walk on; they store the same
// value, so no atomics are needed.
__device__ __forceinline__ void nil_mark_up(const NilMark& m, int32_t c) {
    int32_t p = c;
    m.flags[m.foff[m.L] + p] = 1;
    for (int l = m.L; l > 0; --l) {
        p = m.uparent[l][p];
        int32_t* f = m.flags + m.foff[l - 1] + p;
        if (__hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != 0) return;
        __hip_atomic_store(f, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
}

// The flags set in every tile of NIL_TILE, by the waves of the leaf fill (the
// marks are the leaf count's): wave w of nw.
__device__ __forceinline__ void nil_tile_counts(const NilMark& m, int64_t w, int64_t nw) {
    const int lane = threadIdx.x & 63;
    for (int64_t t = w; t < m.tiles; t += nw) {
        const int4 f = reinterpret_cast<const int4*>(m.flags)[t * 64 + lane];
        const int c = wave_sum(f.x + f.y + f.z + f.w);
        if (lane == 0) m.tcnt[t] = c;
    }
}

struct LeafStep {
    const int32_t* fa;        // A leaf of each leaf pair
    const int32_t* fb;        // B leaf of each leaf pair
    const int32_t* cseg;
    const uint64_t* ckey;
    const int32_t* ncount;
    int32_t ncap;
    int lb_log;
    const uint64_t* Arm;      // A leaves: row-major masks
    const uint64_t* Bcm;      // B leaves: column-major masks
    const uint64_t* Brm;      // B leaves: row-major masks (leaves of few products)
    int32_t group;            // leaves of few products: C leaves per wave
    int32_t* heavy;           // and the leaves among them of many: their number (zeroed first), then the leaves
    int32_t heavy_max;
    const uint64_t* Amo;      // Morton-order masks (rank of a block in its leaf)
    const uint64_t* Bmo;
    const int32_t* Abase;
    const int32_t* Bbase;
    int64_t* cnt;             // per C leaf: (products, C blocks)
    int32_t* lane_cnt;        // per C leaf, 64 entries: the block products of each block position
    int64_t* off;             // scan path: exclusive scan of cnt; aggregate path: offset inside the workgroup
    int64_t* wagg;            // aggregate path: per count workgroup, the sum of its leaves' cnt
    int64_t* gsum;            // aggregate path: per group of 64 count workgroups, their sum (zeroed first)
    int use_agg;
    int32_t* prodA;
    int32_t* prodB;
    int32_t P;
    uint64_t* cbkey;          // C block keys, Morton order
    int32_t* cbseg;           // first product of each C block
    int32_t cap;              // bound on C blocks
    int32_t* lbase;           // C leaves: first block, masks
    uint64_t* lmo;
    uint64_t* lrm;
    uint64_t* lcm;
    int32_t* nblocks_out;
    int32_t* check;
    int ta, tb;               // op(A) = A^T / op(B) = B^T (masks already swapped by the host)
    int upper;                // keep only blocks on or above the diagonal
    const int32_t* amap;      // structure-only A: its block t is held by its value source as amap[t]
    const int32_t* bmap;
    const double* Abn2;       // squared block norms (nullptr: no norm threshold): a block product
    const double* Bbn2;       // is dropped when Abn2 Bbn2 < tau2
    double tau2;
};

// Lane t's value in every lane, for a t that is the same in every lane: a
// read of one lane into a scalar register, with no LDS round trip (a general
// shuffle goes through the LDS crossbar).
__device__ __forceinline__ uint32_t lane_value(uint32_t v, int t) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, t);
}
__device__ __forceinline__ uint64_t lane_value(uint64_t v, int t) {
    return (uint64_t)lane_value((uint32_t)v, t) | ((uint64_t)lane_value((uint32_t)(v >> 32), t) << 32);
}

// Block q of a C leaf is kept unless only the upper triangle is wanted and
// it lies below the diagonal of a diagonal leaf.
__device__ __forceinline__ bool leaf_block_kept(const LeafStep& st, uint64_t leafkey, int i, int j) {
    return !(st.upper && i > j && morton_row(leafkey) == morton_col(leafkey));
}

// Lane q (a block of the C leaf, local Morton index) counts its products.
// The leaf pairs are taken 64 at a time, one per lane, and only those that
// can add a block product at all are walked: some inner index k with column
// k of the op(A) leaf and row k of the op(B) leaf both occupied. In an
// unstructured product most leaf pairs have none (random65536: four in five).
__device__ __forceinline__ int leaf_lane_count(const LeafStep& st, int32_t s0, int32_t len, int lane, int i, int j,
                                               int lb, bool on) {
    int cnt = 0;
    for (int32_t base = 0; base < len; base += 64) {
        const int32_t nb = min(64, len - base);
        uint64_t ra = 0, cb = 0;
        if (lane < nb) {
            ra = st.Arm[st.fa[s0 + base + lane]];
            cb = st.Bcm[st.fb[s0 + base + lane]];
        }
        for (uint64_t live = __ballot((mask_fold(ra, lb) & mask_fold(cb, lb)) != 0); live; live &= live - 1) {
            const int t = __ffsll((unsigned long long)live) - 1;
            const uint64_t rat = lane_value(ra, t);
            const uint64_t cbt = lane_value(cb, t);
            if (on) cnt += __popc(mask_row(rat, i, lb) & mask_row(cbt, j, lb));
        }
    }
    return cnt;
}

// Local Morton positions of A(i,k) and B(k,j) in the stored (untransposed) leaves.
__device__ __forceinline__ void leaf_positions(const LeafStep& st, int i, int k, int j, uint32_t& qa, uint32_t& qb) {
    qa = st.ta ? (uint32_t)morton_key((uint32_t)k, (uint32_t)i) : (uint32_t)morton_key((uint32_t)i, (uint32_t)k);
    qb = st.tb ? (uint32_t)morton_key((uint32_t)j, (uint32_t)k) : (uint32_t)morton_key((uint32_t)k, (uint32_t)j);
}

// leaf_lane_count with a norm threshold: every candidate product A(i,k)
// B(k,j) is looked at on its own, kept when its blocks' squared norms
// multiply to at least tau2.
__device__ __forceinline__ int leaf_lane_count_norms(const LeafStep& st, int32_t s0, int32_t len, int lane, int i,
                                                     int j, int lb, bool on) {
    int cnt = 0;
    for (int32_t base = 0; base < len; base += 64) {
        const int32_t nb = min(64, len - base);
        uint64_t ra = 0, cb = 0, amo = 0, bmo = 0;
        int32_t ab = 0, bb = 0;
        if (lane < nb) {
            const int32_t a = st.fa[s0 + base + lane], b = st.fb[s0 + base + lane];
            ra = st.Arm[a];
            cb = st.Bcm[b];
            amo = st.Amo[a];
            bmo = st.Bmo[b];
            ab = st.Abase[a];
            bb = st.Bbase[b];
        }
        for (uint64_t live = __ballot((mask_fold(ra, lb) & mask_fold(cb, lb)) != 0); live; live &= live - 1) {
            const int t = __ffsll((unsigned long long)live) - 1;
            uint32_t m = on ? (mask_row(lane_value(ra, t), i, lb) & mask_row(lane_value(cb, t), j, lb)) : 0u;
            if (__ballot(m != 0) == 0) continue;
            const uint64_t amot = lane_value(amo, t), bmot = lane_value(bmo, t);
            const int32_t abt = (int32_t)lane_value((uint32_t)ab, t), bbt = (int32_t)lane_value((uint32_t)bb, t);
            while (m) {
                const int k = __ffs(m) - 1;
                m &= m - 1;
                uint32_t qa, qb;
                leaf_positions(st, i, k, j, qa, qb);
                const int32_t ia = abt + __popcll(amot & ((1ull << qa) - 1));
                const int32_t ib = bbt + __popcll(bmot & ((1ull << qb) - 1));
                cnt += norms_kept(st.Abn2[ia], st.Bbn2[ib], st.tau2);
            }
        }
    }
    return cnt;
}

template <bool PRUNE>
__device__ __forceinline__ int64_t leaf_count_node(const LeafStep& st, const NilMark& nil, int32_t c, int lane) {
    if (c >= *st.ncount) {
        if (lane == 0) st.cnt[c] = 0;
        return 0;
    }
    const int lb = 1 << st.lb_log;
    const int i = (int)morton_row((uint64_t)lane), j = (int)morton_col((uint64_t)lane);
    const bool on = lane < lb * lb && leaf_block_kept(st, st.ckey[c], i, j);
    const int32_t s0 = st.cseg[c], len = st.cseg[c + 1] - s0;
    const int cnt = PRUNE ? leaf_lane_count_norms(st, s0, len, lane, i, j, lb, on)
                          : leaf_lane_count(st, s0, len, lane, i, j, lb, on);
    st.lane_cnt[(int64_t)c * 64 + lane] = cnt;   // the fill reads it instead of walking the pairs twice
    const uint64_t em = __ballot(cnt > 0);
    const int tot = wave_sum(cnt);
    const int64_t v = pack2(tot, __popcll(em));
    if (lane == 0) {
        st.cnt[c] = v;
        if (em) nil_mark_up(nil, c);
    }
    return v;
}

// Totals T = (block products, C blocks) of the leaf level.
__device__ void leaf_level_totals(const LeafStep& st, int64_t T) {
    const int32_t nb = hi32(T);
    *st.nblocks_out = nb;
    if (nb <= st.cap) st.cbseg[nb] = lo32(T);
    *st.check = lo32(T);
}

// Lists the products of every block of a C leaf (lane: one block), pair by
// pair of the leaf pairs s0 .. s0 + len - 1, k ascending, from place `out` on.
// PLAIN: stored operands (no block maps) and no norm threshold.
template <bool PLAIN>
__device__ __forceinline__ void leaf_fill_products(const LeafStep& st, int32_t s0, int32_t len, int lane, int i, int j,
                                                   int lb, bool on, int32_t out) {
    for (int32_t base = 0; base < len; base += 64) {
        const int32_t nb = min(64, len - base);
        uint64_t ra = 0, cb = 0, amo = 0, bmo = 0;
        int32_t ab = 0, bb = 0;
        if (lane < nb) {
            const int32_t a = st.fa[s0 + base + lane], b = st.fb[s0 + base + lane];
            ra = st.Arm[a];
            cb = st.Bcm[b];
            amo = st.Amo[a];
            bmo = st.Bmo[b];
            ab = st.Abase[a];
            bb = st.Bbase[b];
        }
        for (uint64_t live = __ballot((mask_fold(ra, lb) & mask_fold(cb, lb)) != 0); live; live &= live - 1) {
            const int t = __ffsll((unsigned long long)live) - 1;
            const uint64_t rat = lane_value(ra, t);
            const uint64_t cbt = lane_value(cb, t);
            uint32_t m = on ? (mask_row(rat, i, lb) & mask_row(cbt, j, lb)) : 0u;
            // most leaf pairs of an unstructured product add no block product
            // to any block of this C leaf: skip their block positions
            if (__ballot(m != 0) == 0) continue;
            const uint64_t amot = lane_value(amo, t);
            const uint64_t bmot = lane_value(bmo, t);
            const int32_t abt = (int32_t)lane_value((uint32_t)ab, t);
            const int32_t bbt = (int32_t)lane_value((uint32_t)bb, t);
            if constexpr (PLAIN) {
                // stored operands, no norm threshold: no loads in this loop, so
                // no wait on memory (a wait here would also wait for the stores
                // of the products before)
                const uint32_t tra = st.ta ? PROD_TRANS : 0u, trb = st.tb ? PROD_TRANS : 0u;
                while (m) {
                    const int k = __ffs(m) - 1;
                    m &= m - 1;
                    uint32_t qa, qb;   // local Morton positions of A(i,k) / B(k,j) in the stored leaves
                    leaf_positions(st, i, k, j, qa, qb);
                    const int32_t ia = abt + __popcll(amot & ((1ull << qa) - 1));
                    const int32_t ib = bbt + __popcll(bmot & ((1ull << qb) - 1));
                    if (out < st.P) {
                        st.prodA[out] = (int32_t)((uint32_t)ia | tra);
                        st.prodB[out] = (int32_t)((uint32_t)ib | trb);
                    }
                    ++out;
                }
            } else while (m) {
                const int k = __ffs(m) - 1;
                m &= m - 1;
                uint32_t qa, qb;   // local Morton positions of A(i,k) / B(k,j) in the stored leaves
                leaf_positions(st, i, k, j, qa, qb);
                const int32_t ia = abt + __popcll(amot & ((1ull << qa) - 1));
                const int32_t ib = bbt + __popcll(bmot & ((1ull << qb) - 1));
                if (st.Abn2 && !norms_kept(st.Abn2[ia], st.Bbn2[ib], st.tau2)) continue;
                if (out < st.P) {
                    // the block of the value source, with the transposition bit
                    st.prodA[out] = st.amap ? st.amap[ia] : (int32_t)((uint32_t)ia | (st.ta ? PROD_TRANS : 0u));
                    st.prodB[out] = st.bmap ? st.bmap[ib] : (int32_t)((uint32_t)ib | (st.tb ? PROD_TRANS : 0u));
                }
                ++out;
            }
        }
    }
}

// o: (first product, first C block) of leaf c.
template <bool PLAIN>
__device__ __forceinline__ void leaf_fill_node(const LeafStep& st, int32_t c, int lane, int64_t o) {
    if (c >= *st.ncount) return;
    const int lb = 1 << st.lb_log;
    const int i = (int)morton_row((uint64_t)lane), j = (int)morton_col((uint64_t)lane);
    const bool on = lane < lb * lb && leaf_block_kept(st, st.ckey[c], i, j);
    const int32_t s0 = st.cseg[c], len = st.cseg[c + 1] - s0;
    const int cnt = st.lane_cnt[(int64_t)c * 64 + lane];   // from the count kernel
    const bool exists = cnt > 0;
    const uint64_t em = __ballot(exists);
    const int32_t bidx = hi32(o) + __popcll(em & lanes_below(lane));
    int32_t out = lo32(o) + wave_excl_scan(cnt);
    if (exists && bidx < st.cap) {
        st.cbkey[bidx] = (st.ckey[c] << (2 * st.lb_log)) | (uint64_t)lane;
        st.cbseg[bidx] = out;
    }
    leaf_fill_products<PLAIN>(st, s0, len, lane, i, j, lb, on, out);
    if (lane == 0) {
        const uint64_t rm = morton_to_rowmajor(em, st.lb_log);
        st.lbase[c] = hi32(o);
        st.lmo[c] = em;
        st.lrm[c] = rm;
        st.lcm[c] = rowmajor_to_colmajor(rm, st.lb_log);
    }
}

template <int W, bool PRUNE>
__device__ __forceinline__ void leaf_count_level(const LeafStep& st, const NilMark& nil) {
    __shared__ int64_t lds[W];
    if (st.use_agg && level_wg_empty<W>(st.ncount)) {
        if (threadIdx.x == 0) st.wagg[blockIdx.x] = 0;
        return;
    }
    const int32_t c = (int32_t)(blockIdx.x * W + (threadIdx.x >> 6));
    int64_t v = 0;
    if (c < st.ncap) v = leaf_count_node<PRUNE>(st, nil, c, threadIdx.x & 63);
    if (st.use_agg) level_local_offsets<W>(v, c, st.ncap, st.off, st.wagg, st.gsum, lds);
}

template <int W, bool PRUNE>
__global__ __launch_bounds__(64 * W) void k_leaf_count(LeafStep st, NilMark nil) {
    leaf_count_level<W, PRUNE>(st, nil);
}

template <int W, bool PLAIN>
__device__ __forceinline__ void leaf_fill_level(const LeafStep& st, const NilMark& nil) {
    __shared__ int64_t lds[W];
    const int32_t c = (int32_t)(blockIdx.x * W + (threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    nil_tile_counts(nil, c, (int64_t)((st.ncap - 1) / W + 1) * W);
    if (st.use_agg) {
        const bool last = level_wg_last<W>(st.ncap);
        if (level_wg_empty<W>(st.ncount) && !last) return;
        const int64_t base = level_base<W>(st.wagg, st.gsum, lds);
        if (last && threadIdx.x == 0) leaf_level_totals(st, base + st.wagg[blockIdx.x]);
        if (c < st.ncap) leaf_fill_node<PLAIN>(st, c, lane, base + st.off[c]);
    } else {
        if (c == 0 && lane == 0) leaf_level_totals(st, st.off[st.ncap]);
        if (c < st.ncap) leaf_fill_node<PLAIN>(st, c, lane, st.off[c]);
    }
}

template <int W, bool PLAIN>
__global__ __launch_bounds__(64 * W) void k_leaf_fill(LeafStep st, NilMark nil) {
    leaf_fill_level<W, PLAIN>(st, nil);
}

// ------------------------------------------- C leaves of few block products
//
// The kernels above give a C leaf to a wave and a block position to a lane, and
// walk its leaf pairs one by one: right where a leaf has hundreds of products.
// In an unstructured product it has a few (an R-MAT product of 39634 blocks of
// 16: 475 k leaves, 4.6 leaf pairs and 2.4 products each; random48000 at b =
// 32: 55 pairs, 14 products), and each then costs a wave's fixed part and, per
// leaf pair, instructions for 64 lanes of which one or two have a product. Here
// a lane takes a leaf pair instead, and a wave the pairs of `group` leaves, 64
// at a time:
//   count: a lane forms its pair's boolean product, eight outer products of
//          bytes, and adds the number of block products and the C blocks to
//          its leaf's in LDS;
//   fill:  leaves are taken together while their products are at most 64.
//          Every lane lists the products of its pairs in LDS, one per step; each
//          gets a key (leaf, block position, pair, k), the order of the product
//          list, and its place is the number of smaller keys. The list goes out
//          with one product per lane.
// A leaf of more than 64 products goes through the walk above, in a wave of its
// own: the count lists these leaves, and the fill's first workgroups take them
// (sixteen of them in one wave, next to R-MAT's hubs, took as long as all other
// waves together). Products, their order and C's tree are the same either way.
// Count and fill alone: that R-MAT product 253 + 373 -> 51 + 97 us, random48000
// 47 + 76 -> 46 + 44. What is left of them are the gathers of the leaves' masks
// and bases and the LDS round trips of one wave.
constexpr int SPARSE_MAX = 64;                 // products listed together
// Chosen up to 40 products per C leaf position that the host's bounds allow. The
// symbolic phase, wave per leaf and lane per pair, in us: random of 1500 block
// rows with 1.5 products per leaf 175 and 134, 14: 269 and 230, 38: 374 and 288,
// 55: 431 and 344, 86 (most leaves above SPARSE_MAX): 599 and 867; R-MAT of
// 8192 with 1.1: 1163 and 646; of 1024 with 0.9 (4517 leaves): 113 and 121, with
// 34 (hubs): 158 and 149.
constexpr int SPARSE_LEAF = 40;

// x: a flag in the lowest bit of each byte; y: a byte. y in every flagged byte.
__device__ __forceinline__ uint64_t bytes_where(uint64_t x, uint32_t y) {
    return (uint64_t)((uint32_t)x * y) | ((uint64_t)((uint32_t)(x >> 32) * y) << 32);
}

// Column k of a row-major 8 x 8 mask, as flags of the rows.
__device__ __forceinline__ uint64_t mask_column(uint64_t m, int k) { return (m >> k) & 0x0101010101010101ull; }

__device__ __forceinline__ uint64_t rowmajor_to_morton8(uint64_t m) {
    m = swap_index_bits(m, 3, 2, 0x00F000F000F000F0ull);
    m = swap_index_bits(m, 2, 1, 0x0C0C0C0C0C0C0C0Cull);
    return swap_index_bits(m, 4, 3, 0x0000FF000000FF00ull);
}

__global__ __launch_bounds__(64) void k_leaf_count_sparse(LeafStep st, NilMark nil) {
    __shared__ int32_t mark[64];
    __shared__ int32_t lcnt[64];
    __shared__ unsigned long long lem[64];
    const int lane = threadIdx.x;
    const int32_t n = *st.ncount, c0 = (int32_t)blockIdx.x * st.group;
    if (c0 >= n) {
        if (lane == 0) st.wagg[blockIdx.x] = 0;
        return;
    }
    const int32_t nl = min(st.group, n - c0), c = c0 + lane;
    const int32_t seg = lane < nl ? st.cseg[c] : INT32_MAX;
    const int32_t end = st.cseg[c0 + nl];
    lcnt[lane] = 0;
    lem[lane] = 0;
    for (int32_t base = __builtin_amdgcn_readfirstlane(seg); base < end; base += 64) {
        uint64_t ra = 0, rb = 0;
        if (base + lane < end) {
            const int32_t a = st.fa[base + lane], b = st.fb[base + lane];
            ra = st.Arm[a];
            rb = st.Brm[b];
        }
        int head;
        const int q = pair_node(seg, base, lane, mark, head);
        uint64_t e = 0;
        int cnt = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint64_t x = mask_column(ra, k);
            const uint32_t y = (uint32_t)(rb >> (8 * k)) & 255u;
            e |= bytes_where(x, y);
            cnt += __popcll(x) * __popc(y);
        }
        if (cnt) {
            atomicAdd(&lcnt[q], cnt);
            atomicOr(&lem[q], (unsigned long long)e);
        }
    }
    __syncthreads();
    const int cnt = lcnt[lane];
    const uint64_t em = lem[lane];
    const int nb = __popcll(em);
    const int s_cnt = wave_incl_scan(cnt), s_nb = wave_incl_scan(nb);
    if (lane < nl) {
        st.off[c] = pack2(s_cnt - cnt, s_nb - nb);
        st.lrm[c] = em;
        st.lcm[c] = rowmajor_to_colmajor(em, 3);
        st.lmo[c] = rowmajor_to_morton8(em);
        if (em) nil_mark_up(nil, c);
        if (cnt > SPARSE_MAX) {
            const int32_t h = atomicAdd(st.heavy, 1);
            if (h < st.heavy_max) st.heavy[1 + h] = c;
        }
    }
    if (lane == 63) {
        const int64_t tot = pack2(s_cnt, s_nb);
        st.wagg[blockIdx.x] = tot;
        if (tot) atomicAdd((unsigned long long*)(st.gsum + (blockIdx.x >> AGG_GROUP_LOG)), (unsigned long long)tot);
    }
}

// The block products of C leaf c, one of more than SPARSE_MAX.
__device__ __forceinline__ void leaf_fill_heavy(const LeafStep& st, int32_t c, int64_t* lds) {
    const int lane = threadIdx.x;
    const int64_t o = level_base<1>(st.wagg, st.gsum, lds, c / st.group) + st.off[c];
    const int i = (int)morton_row((uint64_t)lane), j = (int)morton_col((uint64_t)lane);
    const int32_t s0 = st.cseg[c], len = st.cseg[c + 1] - s0;
    const int cnt = leaf_lane_count(st, s0, len, lane, i, j, 8, true);
    const uint64_t em = __ballot(cnt > 0);
    const int32_t bidx = hi32(o) + __popcll(em & lanes_below(lane));
    const int32_t out = lo32(o) + wave_excl_scan(cnt);
    if (cnt > 0 && bidx < st.cap) {
        st.cbkey[bidx] = (st.ckey[c] << 6) | (uint64_t)lane;
        st.cbseg[bidx] = out;
    }
    leaf_fill_products<true>(st, s0, len, lane, i, j, 8, true, out);
}

// The first heavy_max workgroups take the leaves of many products.
__global__ __launch_bounds__(64) void k_leaf_fill_sparse(LeafStep st, NilMark nil) {
    __shared__ int64_t lds[1];
    __shared__ int32_t mark[64];
    __shared__ uint32_t skey[64];                  // leaf << 26 | block position << 20 | pair << 3 | k
    __shared__ int32_t sa[64], sb[64];
    __shared__ uint64_t lkey[64];
    const int lane = threadIdx.x;
    if ((int32_t)blockIdx.x < st.heavy_max) {
        if ((int32_t)blockIdx.x < *st.heavy) leaf_fill_heavy(st, st.heavy[1 + blockIdx.x], lds);
        return;
    }
    const int32_t wg = (int32_t)blockIdx.x - st.heavy_max;
    nil_tile_counts(nil, wg, (int64_t)(st.ncap - 1) / st.group + 1);
    const int32_t n = *st.ncount, c0 = wg * st.group;
    const bool last = wg == (st.ncap - 1) / st.group;
    if (c0 >= n && !last) return;
    const int64_t base0 = level_base<1>(st.wagg, st.gsum, lds, wg);
    const int64_t agg = st.wagg[wg];
    if (last && lane == 0) leaf_level_totals(st, base0 + agg);
    if (c0 >= n) return;
    const int32_t nl = min(st.group, n - c0), c = c0 + lane;
    int32_t seg = INT32_MAX, lo = 0, hi = 0, lo_end = 0;   // the leaf's first pair, product and C block; the products' end
    if (lane < nl) {
        seg = st.cseg[c];
        const int64_t o = st.off[c], oe = lane + 1 < nl ? st.off[c + 1] : agg;
        lo = lo32(o);
        hi = hi32(o);
        lo_end = lo32(oe);
        st.lbase[c] = hi32(base0) + hi;
        lkey[lane] = st.ckey[c];
    }
    const int32_t end = st.cseg[c0 + nl];
    __syncthreads();
    const uint32_t tra = st.ta ? PROD_TRANS : 0u, trb = st.tb ? PROD_TRANS : 0u;
    for (int q = 0; q < nl;) {
        const int32_t plo = (int32_t)lane_value((uint32_t)lo, q), s0 = (int32_t)lane_value((uint32_t)seg, q);
        // the leaves from q on whose products are together at most 64
        const int take = __popcll(__ballot(lane >= q && lane < nl && lo_end - plo <= SPARSE_MAX));
        if (take == 0) {   // taken by a workgroup of its own
            ++q;
            continue;
        }
        const int qe = q + take;
        const int32_t np = (int32_t)lane_value((uint32_t)lo_end, qe - 1) - plo;
        const int32_t hi_q = (int32_t)lane_value((uint32_t)hi, q);
        const int32_t s1 = qe < nl ? (int32_t)lane_value((uint32_t)seg, qe) : end;
        q = qe;
        if (np == 0) continue;
        // the list, in any order
        int listed = 0;
        for (int32_t base = s0; base < s1; base += 64) {
            uint64_t ra = 0, rb = 0, amo = 0, bmo = 0;
            int32_t ab = 0, bb = 0;
            if (base + lane < s1) {
                const int32_t a = st.fa[base + lane], b = st.fb[base + lane];
                ra = st.Arm[a];
                rb = st.Brm[b];
                amo = st.Amo[a];
                bmo = st.Bmo[b];
                ab = st.Abase[a];
                bb = st.Bbase[b];
            }
            int head;
            const int leaf = pair_node(seg, base, lane, mark, head);
            // inner indices with a block on either side
            uint32_t km = mask_fold(ra, 8);
            {
                uint64_t y = rb | (rb >> 4);       // bit 8 k: row k is occupied
                y |= y >> 2;
                y |= y >> 1;
                y &= 0x0101010101010101ull;
                km &= (uint32_t)((y * 0x0102040810204080ull) >> 56);
            }
            uint64_t e = 0;
            int k = 0;
            while (true) {
                if (e == 0 && km != 0) {
                    k = __ffs(km) - 1;
                    km &= km - 1;
                    e = bytes_where(mask_column(ra, k), (uint32_t)(rb >> (8 * k)) & 255u);
                }
                const uint64_t live = __ballot(e != 0);
                if (live == 0) break;
                const int slot = listed + __popcll(live & lanes_below(lane));
                if (e != 0 && slot < 64) {
                    const int pos = __ffsll((unsigned long long)e) - 1, i = pos >> 3, j = pos & 7;
                    uint32_t qa, qb;
                    leaf_positions(st, i, k, j, qa, qb);
                    skey[slot] = ((uint32_t)leaf << 26) | ((uint32_t)morton_key((uint32_t)i, (uint32_t)j) << 20) |
                                 ((uint32_t)(base + lane - s0) << 3) | (uint32_t)k;
                    sa[slot] = (int32_t)((uint32_t)(ab + __popcll(amo & ((1ull << qa) - 1))) | tra);
                    sb[slot] = (int32_t)((uint32_t)(bb + __popcll(bmo & ((1ull << qb) - 1))) | trb);
                }
                e &= e - 1;
                listed += __popcll(live);
            }
        }
        // its order: the place of a product is the number of smaller keys
        __syncthreads();
        const int m = min(np, 64);
        const bool on = lane < m;
        const uint32_t key = on ? skey[lane] : 0xffffffffu;
        const int32_t ia = on ? sa[lane] : 0, ib = on ? sb[lane] : 0;
        int rank = 0;
        for (int t = 0; t < m; ++t) rank += lane_value(key, t) < key;
        __syncthreads();
        if (on && rank < 64) {
            skey[rank] = key;
            sa[rank] = ia;
            sb[rank] = ib;
        }
        __syncthreads();
        const uint32_t sk = skey[lane] >> 20, prev = lane ? skey[lane - 1] >> 20 : 0xffffffffu;
        const bool head = on && sk != prev;
        const uint64_t heads = __ballot(head);
        const int32_t out = lo32(base0) + plo + lane;
        if (on && out < st.P) {
            st.prodA[out] = sa[lane];
            st.prodB[out] = sb[lane];
        }
        const int32_t bidx = hi32(base0) + hi_q + __popcll(heads & lanes_below(lane));
        if (head && bidx < st.cap) {
            st.cbkey[bidx] = (lkey[sk >> 6] << 6) | (uint64_t)(sk & 63u);
            st.cbseg[bidx] = out;
        }
        __syncthreads();
    }
}

// ---------------------------------------------- NIL normalisation of C
//
// The traversal creates a C node for every quadrant that receives a pair, and
// a C leaf for every leaf pair group, before it knows whether any block
// product lands there: a leaf whose pairs all miss (no k with A(i,k) and
// B(k,j) both present) holds no block, and so does a node above only such
// leaves. Zero submatrices are NIL at every level of the quadtree (Sec. 3.1),
// so C's tree keeps exactly the nodes with a stored block below them:
//   mark:    the leaf count flags every leaf that receives a block, and its
//            ancestors (parents were recorded by the traversal); the leaf
//            fill's waves count the flags per tile (nil_mark_up,
//            nil_tile_counts);
//   offsets: one wave per tile adds up the counts of the tiles before it and
//            ranks its own flags: the exclusive scan of the flags of all
//            levels, concatenated, which gives every kept node its index among
//            the kept nodes of its level (one launch, where a general scan
//            takes three);
//   compact: kept nodes are copied into C's tree, child tables remapped
//            (a child that is not kept becomes NIL), and the kept counts of
//            every level are written for the read-back.
// C's blocks, their order and the product lists do not change: an empty leaf
// owns none of them. The traversal runs beside the previous multiply's
// numeric kernel, where each launch waits tens of microseconds for wave
// slots; folding the marks and the tile counts into the leaf step and the scan
// into one launch leaves two launches of the five a separate pass would take.
// (Marked with an atomic exchange per flag and an atomic count per tile, in
// the leaf fill, that kernel took 460 instead of 373 us on an R-MAT product
// of 0.6 M leaves, 110 instead of 75 us on a random 48000 one.)

struct NilTree {
    int L;
    int64_t foff[NIL_MAX_LEVELS + 2];        // flags of level l at foff[l] .. foff[l+1]-1
    const int32_t* uchild[NIL_MAX_LEVELS];   // levels 0 .. L-1 (4 per node)
    const uint64_t* ukey[NIL_MAX_LEVELS + 1];
    const int32_t* ubase;                    // leaves
    const uint64_t* umo;
    const uint64_t* urm;
    const uint64_t* ucm;
    const int32_t* flags;                    // foff[L+1] entries, set by the leaf count
    const int32_t* tcnt;                     // flags set per tile
    int64_t tiles;
    int32_t* ex;                             // exclusive scan of flags (foff[L+1] + 1 entries)
    int32_t* child[NIL_MAX_LEVELS];          // the kept tree
    uint64_t* key[NIL_MAX_LEVELS + 1];
    int32_t* base;
    uint64_t* mo;
    uint64_t* rm;
    uint64_t* cm;
    int32_t* kept;                           // kept nodes per level, levels 0 .. L
};

// ex[i] = number of flags set before i, for every i of the tiles (n among
// them: the total); one wave per tile, which adds up the counts of the tiles
// before its own. (With tiles of 64 and 4-byte loads the waves of an R-MAT
// product with 1.4 M nodes read 1 GB of counts, 90 us; 6 us now.)
__device__ __forceinline__ void nil_offsets_tile(const int32_t* __restrict__ flags, const int32_t* __restrict__ tcnt,
                                                 int32_t* __restrict__ ex) {
    const int lane = threadIdx.x;
    const int64_t t = blockIdx.x;
    const int4 f = reinterpret_cast<const int4*>(flags)[t * 64 + lane];
    int before = 0;
#pragma unroll 4
    for (int64_t u = lane; u < t / 4; u += 64) {
        const int4 c = reinterpret_cast<const int4*>(tcnt)[u];
        before += c.x + c.y + c.z + c.w;
    }
    if (lane < (t & 3)) before += tcnt[(t & ~int64_t(3)) + lane];
    before = wave_sum(before) + wave_excl_scan(f.x + f.y + f.z + f.w);
    reinterpret_cast<int4*>(ex)[t * 64 + lane] =
        make_int4(before, before + f.x, before + f.x + f.y, before + f.x + f.y + f.z);
}

__global__ __launch_bounds__(64) void k_nil_offsets(const int32_t* flags, const int32_t* tcnt, int32_t* ex) {
    nil_offsets_tile(flags, tcnt, ex);
}

__device__ __forceinline__ int32_t nil_rank(const NilTree& t, int l, int64_t c) {
    return t.ex[t.foff[l] + c] - t.ex[t.foff[l]];
}

__device__ __forceinline__ void nil_compact(const NilTree& t) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int L = t.L;
    if (i == 0)
        for (int l = 0; l <= L; ++l) t.kept[l] = t.ex[t.foff[l + 1]] - t.ex[t.foff[l]];
    if (i >= t.foff[L + 1] || !t.flags[i]) return;
    int l = 0;
    while (i >= t.foff[l + 1]) ++l;
    const int64_t c = i - t.foff[l];
    const int32_t n = nil_rank(t, l, c);
    t.key[l][n] = t.ukey[l][c];
    if (l < L) {
        const int4 u = *reinterpret_cast<const int4*>(t.uchild[l] + 4 * c);
        const int32_t uc[4] = {u.x, u.y, u.z, u.w};
        int32_t out[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            out[q] = (uc[q] >= 0 && t.flags[t.foff[l + 1] + uc[q]]) ? nil_rank(t, l + 1, uc[q]) : -1;
        *reinterpret_cast<int4*>(t.child[l] + 4 * (int64_t)n) = make_int4(out[0], out[1], out[2], out[3]);
    } else {
        t.base[n] = t.ubase[c];
        t.mo[n] = t.umo[c];
        t.rm[n] = t.urm[c];
        t.cm[n] = t.ucm[c];
    }
}

__global__ __launch_bounds__(64) void k_nil_compact(NilTree t) { nil_compact(t); }

// ------------------------------------------------ launch order of C's blocks
//
// The numeric kernels give each XCD runs of consecutive launch slots. In
// Morton order such a run is a square patch of C, whose operands, a patch of
// A's rows and one of B's columns, are far more than an XCD's 4 MB of L2 holds
// (a 64-block row of A at b = 64 in FP64 is 2 MB): 72% of the operand reads of
// a 32768 decay product at b = 64 missed it, and those misses, 98 GB at about
// 5 TB/s, bounded the kernel. Taken in strips instead, 2^s block rows high and
// column by column, a run stays within rows whose blocks of A fit (STRIP_BYTES)
// while B streams past, shared by the strip's rows. Measured at b = 64 with 58
// blocks a row, Morton -> strips of 1, 2, 4, 8 rows: FP64 18.8 -> 17.2, 19.1,
// 18.8, 20.2 ms, FP32 9.55 -> 8.77, 9.41, 9.48, 10.6, BF16X3 6.10 -> 5.09,
// 5.20, 5.18, 6.12; A^T A of 20 k blocks in FP32 5.22 -> 4.90 ms. So a strip
// holds about STRIP_BYTES of A, at most a leaf's height. At b = 32 the operands
// of a run nearly fit as they are: FP64 2.5% faster, FP32 1.5%, but the order
// costs 25 us of the next traversal, which shorter products (sysq of a 24576
// matrix 0.594 -> 0.628 ms, a tau product 0.494 -> 0.524) do not win back; so
// the rule is b = 64 and several products per C block.
// Morton order lists the blocks of an aligned strip by column, so a stable
// sort by row >> s of C's Morton-ordered keys gives the order, three launches
// up to 2048 strips.
constexpr int64_t STRIP_BYTES = 1 << 20;
constexpr int STRIP_MAX_LOG = 3;
constexpr int64_t STRIP_MIN_BLOCKS = 8192;   // fewer: under a millisecond of work

struct StripKeys {
    const uint64_t* bkey;
    int log;
    __device__ uint64_t operator()(int32_t t) const { return morton_row(bkey[t]) >> log; }
};
struct OrderSink {
    int32_t* order;
    __device__ void operator()(int32_t at, int32_t t, uint64_t) const { order[at] = t; }
};

// Where C blocks average fewer than two block products (an unstructured
// pattern such as random65536), neighbouring C blocks in Morton order share
// no operand, and nearly every block product fetches its A and B blocks from
// beyond L2. Taking the C blocks grouped by the inner index k of their first
// product instead puts C(i,j) = A(i,k) B(k,j) for all i and j of one k into
// consecutive launch slots: the run an XCD receives reads block column k of
// A and block row k of B, both small enough to stay in its L2, and the
// blocks of each are fetched about once (random65536 fp64: 2.3 GB fetched
// instead of 11.8 GB). The order is a stable sort by k, three launches up to
// 2048 inner blocks, six beyond. (A counting sort of its own, five launches
// with tables of every k per workgroup, took a lone traversal of 437 k C blocks
// 40 us more, one of 890 k with 8192 inner blocks 92 us.)
// Small operands stay cached in any order, and then the sort only costs its
// 35 us: lone calls, Morton and by k, with the operand bytes the products read:
// FP32 b = 32, 0.42 GB 225 and 248 us, 0.82 GB 311 and 312, 4.0 GB 944 and 818;
// FP64 b = 32, 0.35 GB 203 and 209, 0.84 GB 302 and 272, 8.0 GB 1663 and 1070;
// FP64 b = 16, 0.41 GB 240 and 247, 2.0 GB 565 and 492.
// A plan sorts once and runs many times: its problems are sorted at any size, the
// smaller ones when it first runs again (a plan that runs once would lose what the
// sorts take, 16 problems made, run and read out 1156 and 1228 us). Replays, Morton
// and by k, in us: b = 16 FP64, one problem of 64 k blocks 54.8 and 36.5, 16 of 4 k 53.5
// and 44.0, 64 of 1 k 50.2 and 42.7; b = 32, 8 of 4.5 k FP64 113.8 and 86.2, one of 61 k
// BF16X3 130 and 103; b = 64, 4 of 2.6 k FP32 74.9 and 68.9. Slower, by 2 to 6 %: b = 32 FP32,
// 64 of 2.1 k 199 and 211, 8 of 25 k 323 and 335 (qt_plan_tune tries both).
constexpr int64_t KORDER_MIN_BYTES = int64_t(700) << 20;
// Up to 16384 inner blocks: beyond, the two passes take 45 to 130 us and what they
// give depends on the pattern. Lone calls, Morton and by k: bands of two or three
// blocks b = 16 FP64, 20000 block rows 285 and 331 us, 40000 464 and 515, b = 32 589
// and 640; random within 4 % of 20000 block rows 544 and 598; random b = 16 17000
// 2765 and 2806; random b = 32 FP64 17000 1394 and 1336.
constexpr int KORDER_MAX_BITS = 14;

struct FirstKeys {
    const uint64_t* akey;      // keys of the blocks the products name
    const int32_t* prodA;
    const int32_t* seg;
    __device__ uint64_t operator()(int32_t t) const {
        // a product whose A block is read transposed (top bit set) has its
        // inner index in the stored block's row
        const int32_t pa = prodA[seg[t]];
        const uint64_t key = akey[pa & PROD_INDEX];
        return pa < 0 ? morton_row(key) : morton_col(key);   // column of op(A)
    }
};

// ------------------------------------------------- small products: one launch
//
// A product with few node pairs spends its symbolic phase on launches and on
// chains of dependent loads, not on work: banded1024 (1 + 8 + 26 pairs) took
// eleven launches and 37 us. Where every level fits, one workgroup runs the
// whole phase in one launch: the frontier, C's tree before NIL normalisation
// and every count stay in LDS, a barrier takes the place of a launch, and the
// counts go to the host's slot from the same kernel. It lists the same
// products in the same order and forms the same tree. What bounds it is its
// own chain, a few us per level, on one compute unit, so the line lies where
// the level by level launches with all of the GPU come out ahead. The phase
// alone, levels and small, in us (b = 32; pairs of the widest level, products):
// banded1024 (26, 1428) 54 and 25, decay 512 (8, 2228) 50 and 22, decay 1536
// (216, 19048) 56 and 50, decay 2048 (396, 28610) 55 and 73, random 2048 (480,
// 622) 54 and 44, random 3072 (1680, 2200) 56 and 99. Loops of banded1024 with
// the numeric kernel 77 and 51 us a product.
constexpr int SMALL_LEVELS = 8;
constexpr int SMALL_PAIRS = 512;            // node pairs of one level
constexpr int SMALL_NODES = 256;            // C nodes of all levels together
constexpr int64_t SMALL_PRODUCTS = 20000;
constexpr int SMALL_THREADS = 1024, SMALL_WAVES = SMALL_THREADS / 64;

struct SmallStep {
    int L;
    const int32_t* Ach[SMALL_LEVELS];          // child tables, levels 0 .. L-1
    const int32_t* Bch[SMALL_LEVELS];
    const double* An2[SMALL_LEVELS + 1];       // squared norms of the nodes (norm threshold)
    const double* Bn2[SMALL_LEVELS + 1];
    LeafStep leaf;                             // operands' leaves, product lists, C blocks
    int32_t* child[SMALL_LEVELS];              // C's tree
    uint64_t* key[SMALL_LEVELS + 1];
    int32_t* base;
    uint64_t* mo;
    uint64_t* rm;
    uint64_t* cm;
    HostSlot* slot;                            // the counts go there
    uint32_t seq;
    int32_t* counts;                           // or (slot NULL) here, published with other problems'
};

template <bool PRUNE, bool PLAIN>
__device__ __forceinline__ void small_symbolic(const SmallStep& a) {
    __shared__ int32_t fa[2][SMALL_PAIRS], fb[2][SMALL_PAIRS];   // the frontier, this level's and the next
    __shared__ int32_t cseg[2][SMALL_NODES + 1];
    __shared__ uint64_t ukey[SMALL_NODES];                       // all levels' nodes, concatenated
    __shared__ int32_t uchild[4 * SMALL_NODES];                  // index within the next level, or -1
    __shared__ int4 tot[SMALL_NODES];                            // this level: child pairs per quadrant
    __shared__ int32_t cnt_lo[SMALL_NODES], cnt_hi[SMALL_NODES]; // this level: (pairs, nodes) or (products,
                                                                 // blocks) per node, then their scan
    __shared__ uint64_t lmo[SMALL_NODES];
    __shared__ int32_t lbase[SMALL_NODES], kept[SMALL_NODES], rank[SMALL_NODES];
    __shared__ int32_t total_lo, total_hi;
    __shared__ int32_t counts[3 * SMALL_LEVELS + 4], first[SMALL_LEVELS + 2];
    const LeafStep& lf = a.leaf;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, L = a.L;
    const uint64_t below = lanes_below(lane);
    if (tid == 0) {
        fa[0][0] = 0;
        fb[0][0] = 0;
        cseg[0][0] = 0;
        cseg[0][1] = 1;
        ukey[0] = 0;
        counts[0] = 1;
        first[0] = 0;
        first[1] = 1;
    }
    __syncthreads();
    // exclusive scans of cnt_lo and cnt_hi [0 .. n), by two waves
    auto scan = [&](int n) {
        __syncthreads();
        if (wave < 2) {
            int32_t* cnt = wave ? cnt_hi : cnt_lo;
            int run = 0;
            for (int b = 0; b < n; b += 64) {
                const int v = b + lane < n ? cnt[b + lane] : 0;
                const int x = wave_incl_scan(v);
                if (b + lane < n) cnt[b + lane] = run + x - v;
                run += __builtin_amdgcn_readlane(x, 63);
            }
            if (lane == 0) (wave ? total_hi : total_lo) = run;
        }
        __syncthreads();
    };
    int nodes = 1;
    for (int l = 0; l < L; ++l) {
        const int cur = l & 1, at = first[l];
        const double* an2 = a.An2[l + 1];
        const double* bn2 = a.Bn2[l + 1];
        int4 hx = make_int4(-1, -1, -1, -1), hy = hx;   // a wave's child tables, kept from pass 0 where it
                                                        // has one node of at most 64 pairs
        // pass 0 counts the child pairs of every node, pass 1 writes them
#pragma unroll 1
        for (int pass = 0; pass < 2; ++pass) {
#pragma unroll 1
            for (int c = wave; c < nodes; c += SMALL_WAVES) {
                const int s0 = cseg[cur][c], len = cseg[cur][c + 1] - s0;
                const uint64_t key = ukey[at + c];
                const bool drop_lower = quadrant_dropped(lf.upper, key, 2);
                int run[4] = {0, 0, 0, 0};
                if (pass == 1) {
                    const int4 t4 = tot[c];
                    const int t[4] = {t4.x, t4.y, t4.z, t4.w};
                    int pr = cnt_lo[c], ci = cnt_hi[c], mine = -1, my_run = 0;
#pragma unroll
                    for (int mn = 0; mn < 4; ++mn) {
                        run[mn] = pr;
                        if (lane == mn && t[mn] > 0) {
                            mine = ci;
                            my_run = pr;
                        }
                        pr += t[mn];
                        ci += t[mn] > 0;
                    }
                    if (lane < 4) {
                        uchild[4 * (at + c) + lane] = mine;
                        if (mine >= 0 && at + nodes + mine < SMALL_NODES) {
                            ukey[at + nodes + mine] = key * 4 + (uint64_t)lane;
                            cseg[1 - cur][mine] = my_run;
                        }
                    }
                }
#pragma unroll 1
                for (int b = 0; b < len; b += 64) {
                    if (pass == 0 || nodes > SMALL_WAVES || len > 64) {
                        hx = hy = make_int4(-1, -1, -1, -1);
                        if (b + lane < len)
                            op_children2(a.Ach[l], fa[cur][s0 + b + lane], lf.ta, a.Bch[l], fb[cur][s0 + b + lane],
                                         lf.tb, hx, hy);
                    }
                    const int av[4] = {hx.x, hx.y, hx.z, hx.w}, bv[4] = {hy.x, hy.y, hy.z, hy.w};
#pragma unroll
                    for (int mn = 0; mn < 4; ++mn) {
                        const int m = mn >> 1, n = mn & 1;
                        const bool keep = !(mn == 2 && drop_lower);
                        const bool e0 = keep && pair_kept<PRUNE>(an2, bn2, lf.tau2, av[2 * m], bv[n]);
                        const bool e1 = keep && pair_kept<PRUNE>(an2, bn2, lf.tau2, av[2 * m + 1], bv[2 + n]);
                        const uint64_t m0 = __ballot(e0), m1 = __ballot(e1);
                        int w = run[mn] + __popcll(m0 & below) + __popcll(m1 & below);
                        run[mn] += __popcll(m0) + __popcll(m1);
                        if (pass == 0) continue;
                        if (e0 && w < SMALL_PAIRS) {
                            fa[1 - cur][w] = av[2 * m];
                            fb[1 - cur][w] = bv[n];
                        }
                        w += e0;
                        if (e1 && w < SMALL_PAIRS) {
                            fa[1 - cur][w] = av[2 * m + 1];
                            fb[1 - cur][w] = bv[2 + n];
                        }
                    }
                }
                if (pass == 0 && lane == 0) {
                    tot[c] = make_int4(run[0], run[1], run[2], run[3]);
                    cnt_lo[c] = run[0] + run[1] + run[2] + run[3];
                    cnt_hi[c] = (run[0] > 0) + (run[1] > 0) + (run[2] > 0) + (run[3] > 0);
                }
            }
            if (pass == 0) scan(nodes);
        }
        // (the host's bounds make everything fit; the limits keep every access inside)
        const int fits = min(total_hi, SMALL_NODES - (at + nodes));
        if (tid == 0) {
            counts[l + 1] = total_hi;
            counts[L + 2 + l] = total_lo;
            first[l + 2] = at + nodes + fits;
            cseg[1 - cur][fits] = min(total_lo, SMALL_PAIRS);
        }
        nodes = fits;
        __syncthreads();
    }
    // leaf step over the frontier's leaf pairs
    LeafStep st = lf;
    st.fa = fa[L & 1];
    st.fb = fb[L & 1];
    const int at = first[L], lb = 1 << lf.lb_log;
    const int i = (int)morton_row((uint64_t)lane), j = (int)morton_col((uint64_t)lane);
    int n = 0;
#pragma unroll 1
    for (int pass = 0; pass < 2; ++pass) {
#pragma unroll 1
        for (int c = wave; c < nodes; c += SMALL_WAVES) {
            const int s0 = cseg[L & 1][c], len = cseg[L & 1][c + 1] - s0;
            const uint64_t key = ukey[at + c];
            const bool on = lane < lb * lb && leaf_block_kept(st, key, i, j);
            if (pass == 0 || nodes > SMALL_WAVES)
                n = PRUNE ? leaf_lane_count_norms(st, s0, len, lane, i, j, lb, on)
                          : leaf_lane_count(st, s0, len, lane, i, j, lb, on);
            const uint64_t em = __ballot(n > 0);
            const int incl = wave_incl_scan(n);
            if (pass == 0) {
                if (lane == 63) cnt_lo[c] = incl;
                if (lane == 0) cnt_hi[c] = __popcll(em);
                continue;
            }
            const int32_t bidx = cnt_hi[c] + __popcll(em & below), out = cnt_lo[c] + incl - n;
            if (n > 0 && bidx < lf.cap) {
                lf.cbkey[bidx] = (key << (2 * lf.lb_log)) | (uint64_t)lane;
                lf.cbseg[bidx] = out;
            }
            leaf_fill_products<PLAIN>(st, s0, len, lane, i, j, lb, on, out);
            if (lane == 0) {
                lbase[c] = cnt_hi[c];
                lmo[c] = em;
                kept[at + c] = em != 0;
            }
        }
        if (pass == 0) scan(nodes);
    }
    if (tid == 0) {
        counts[L + 1] = total_hi;
        counts[2 * L + 2] = total_lo;
        if (total_hi <= lf.cap) lf.cbseg[total_hi] = total_lo;
    }
    // NIL normalisation: a node is kept when one of its children is
    for (int l = L - 1; l >= 0; --l) {
        __syncthreads();
        for (int c = first[l] + tid; c < first[l + 1]; c += SMALL_THREADS) {
            int k = 0;
            for (int q = 0; q < 4; ++q) k |= uchild[4 * c + q] >= 0 && kept[first[l + 1] + uchild[4 * c + q]];
            kept[c] = k;
        }
    }
    __syncthreads();
    for (int l = wave; l <= L; l += SMALL_WAVES) {   // ranks among a level's kept nodes
        int run = 0;
        for (int b = first[l]; b < first[l + 1]; b += 64) {
            const bool k = b + lane < first[l + 1] && kept[b + lane];
            const uint64_t m = __ballot(k);
            if (k) rank[b + lane] = run + __popcll(m & below);
            run += __popcll(m);
        }
        if (lane == 0) counts[2 * L + 3 + l] = run;
    }
    __syncthreads();
    int l = 0;
    for (int c = tid; c < first[L + 1]; c += SMALL_THREADS) {
        while (c >= first[l + 1]) ++l;
        if (!kept[c]) continue;
        const int to = rank[c];
        a.key[l][to] = ukey[c];
        if (l < L) {
            int out[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int u = uchild[4 * c + q];
                out[q] = u >= 0 && kept[first[l + 1] + u] ? rank[first[l + 1] + u] : -1;
            }
            *reinterpret_cast<int4*>(a.child[l] + 4 * (int64_t)to) = make_int4(out[0], out[1], out[2], out[3]);
        } else {
            const int f = c - first[L];
            const uint64_t rm = morton_to_rowmajor(lmo[f], lf.lb_log);
            a.base[to] = lbase[f];
            a.mo[to] = lmo[f];
            a.rm[to] = rm;
            a.cm[to] = rowmajor_to_colmajor(rm, lf.lb_log);
        }
    }
    if (a.slot)
        publish_words(counts, 3 * L + 4, a.slot, a.seq);
    else if (tid < 3 * L + 4)   // written by this thread's wave or before the last barrier
        a.counts[tid] = counts[tid];
}

template <bool PRUNE, bool PLAIN>
__global__ __launch_bounds__(SMALL_THREADS) void k_small_symbolic(SmallStep a) {
    small_symbolic<PRUNE, PLAIN>(a);
}

// ------------------------------------------ the problems of a batch together
//
// A plan of many products ran their symbolic phases one after another, each a
// dozen launches of few workgroups and a wait of the host for its counts: 16
// products of up to 384 block rows took 1.2 ms so, on a GPU mostly idle.
// Together they share the launches: the problem is the workgroup's y index
// (x, for the small ones, a workgroup each) and its step record is read from
// memory, in place of the kernel's arguments; trees of different depth are
// aligned at their leaves. One kernel publishes all problems' counts. Those 16
// products, their plan made and run and the results read out: 2299 us one by
// one, 1413 together; what is left of the symbolic phase is its chain of a
// dozen launches and the host's part, allocations and launch orders.
struct ManyStep {
    int first;        // the problem's first level among the launches: its root
    RootInit root;
    LeafStep leaf;
    NilMark mark;
    NilTree nil;
};

__global__ __launch_bounds__(64) void k_root_init_many(const ManyStep* __restrict__ many) {
    root_init(many[blockIdx.y].root);
}

// steps: [level among the launches][problem]; no nodes where the problem has
// no such level.
__global__ __launch_bounds__(64) void k_tree_count_many(const ManyStep* __restrict__ many,
                                                        const TreeStep* __restrict__ steps) {
    const TreeStep st = steps[many[blockIdx.y].first * gridDim.y + blockIdx.y];
    tree_count_level<1, false>(st);
}

template <bool COUNTS>
__global__ __launch_bounds__(64) void k_tree_fill_many(const TreeStep* __restrict__ steps) {
    const TreeStep st = steps[blockIdx.y];
    if ((int32_t)blockIdx.x >= st.ncap) return;
    tree_fill_level<1, false, COUNTS>(st);
}

__global__ __launch_bounds__(64) void k_leaf_count_many(const ManyStep* __restrict__ many) {
    const LeafStep st = many[blockIdx.y].leaf;
    if ((int32_t)blockIdx.x >= st.ncap) return;
    leaf_count_level<1, false>(st, many[blockIdx.y].mark);
}

__global__ __launch_bounds__(64) void k_leaf_fill_many(const ManyStep* __restrict__ many) {
    const LeafStep st = many[blockIdx.y].leaf;
    if ((int32_t)blockIdx.x >= st.ncap) return;
    leaf_fill_level<1, true>(st, many[blockIdx.y].mark);
}

__global__ __launch_bounds__(64) void k_nil_offsets_many(const ManyStep* __restrict__ many) {
    const NilTree& t = many[blockIdx.y].nil;
    if ((int64_t)blockIdx.x < t.tiles) nil_offsets_tile(t.flags, t.tcnt, t.ex);
}

__global__ __launch_bounds__(64) void k_nil_compact_many(const ManyStep* __restrict__ many) {
    nil_compact(many[blockIdx.y].nil);
}

__global__ __launch_bounds__(SMALL_THREADS) void k_small_symbolic_many(const SmallStep* __restrict__ steps) {
    small_symbolic<false, true>(steps[blockIdx.x]);
}

// ----------------------------------------------------------- host side

// Events that order one stream after another (record on one, wait on the
// other), kept for reuse per device: a wait already queued keeps the
// recording it was queued after, so an event can be recorded again as soon as
// the wait is queued.
static std::mutex g_order_ev_mu;
static std::map<int, std::vector<hipEvent_t>> g_order_ev;

// Work queued on `waiter` from here on runs after what is queued on `first`.
static hipError_t stream_after(hipStream_t waiter, hipStream_t first) {
    int dev = 0;
    hipError_t r = hipGetDevice(&dev);
    if (r != hipSuccess) return r;
    hipEvent_t e = nullptr;
    {
        std::lock_guard<std::mutex> lk(g_order_ev_mu);
        auto& pool = g_order_ev[dev];
        if (!pool.empty()) {
            e = pool.back();
            pool.pop_back();
        }
    }
    if (!e) {
        r = hipEventCreateWithFlags(&e, hipEventDisableTiming);
        if (r != hipSuccess) return r;
    }
    r = hipEventRecord(e, first);
    if (r == hipSuccess) r = hipStreamWaitEvent(waiter, e, 0);
    {
        std::lock_guard<std::mutex> lk(g_order_ev_mu);
        g_order_ev[dev].push_back(e);
    }
    return r;
}

// Workgroups of the per-level kernels for n C nodes (one wave each).
static inline int64_t level_wgs(int64_t n) {
    const int w = level_waves(n);
    return std::max<int64_t>((n + w - 1) / w, 1);
}

// Launch kernel template K (count or fill) with the level's workgroup width
// and the template arguments that follow its own.
#define QT_ARGS(...) __VA_ARGS__
#define QT_LEVEL_LAUNCH(K, n, wgs, stream, arg, ...)                             \
    do {                                                                          \
        if (level_waves(n) == 1)                                                  \
            K<1, __VA_ARGS__><<<(unsigned)(wgs), 64, 0, (stream)>>>(arg);         \
        else                                                                      \
            K<4, __VA_ARGS__><<<(unsigned)(wgs), 256, 0, (stream)>>>(arg);        \
        QT_LAUNCH(#K);                                                            \
    } while (0)

// The symbolic phase reads only the operands' structure (child tables, keys,
// masks), which every handle has complete when the call that made it returns
// (build and multiply both wait for it). So it runs on a library stream of its
// own and overlaps whatever is still queued on the caller's stream -- in a
// loop of multiplies, the previous numeric kernel. The numeric launch on the
// caller's stream then waits for the symbolic phase through an event. The
// stream has the default priority.
static std::mutex g_side_mu;
static std::map<int, hipStream_t> g_side;

static hipStream_t side_stream() {
    int dev = 0;
    QT_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_side_mu);
    auto it = g_side.find(dev);
    if (it != g_side.end()) return it->second;
    hipStream_t st = nullptr;
    QT_HIP(hipStreamCreateWithFlags(&st, hipStreamNonBlocking));
    g_side[dev] = st;
    return st;
}

// A device-resident child table {0, -1, -1, -1}: the single node of a level
// added above a shallower operand so both trees have the same depth (the
// shallower matrix sits in the top-left quadrant at every added level).
static std::mutex g_lift_mu;
static std::map<int, int32_t*> g_lift;

static const int32_t* lift_table() {
    int dev = 0;
    QT_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_lift_mu);
    auto it = g_lift.find(dev);
    if (it != g_lift.end()) return it->second;
    int32_t* p = nullptr;
    QT_HIP(hipMalloc(&p, 4 * sizeof(int32_t)));
    const int32_t h[4] = {0, -1, -1, -1};
    QT_HIP(hipMemcpy(p, h, sizeof(h), hipMemcpyHostToDevice));
    g_lift[dev] = p;
    return p;
}

static const std::vector<int32_t>& unit_hist() {
    static const std::vector<int32_t> one(1, 1);
    return one;
}

static int64_t dot_counts(const std::vector<int32_t>& a, const std::vector<int32_t>& b) {
    const size_t n = std::min(a.size(), b.size());
    int64_t s = 0;
    for (size_t k = 0; k < n; ++k) s += (int64_t)a[k] * b[k];
    return s;
}

static const int64_t kMaxI32 = (int64_t(1) << 31) - 2;

static qt_matrix* new_result(const qt_matrix* A, const qt_matrix* B, int L, qt_prec prec, hipStream_t s,
                             const MulOp& op) {
    std::unique_ptr<qt_matrix> C(new qt_matrix);
    C->n_rows = op.ta ? A->n_cols : A->n_rows;
    C->n_cols = op.tb ? B->n_rows : B->n_cols;
    C->b = A->b;
    C->leaf = A->leaf;
    C->lb = A->lb;
    C->lb_log = A->lb_log;
    C->L = L;
    C->vtype = (prec == QT_F32) ? QT_F32 : QT_F64;
    C->nblocks = 0;
    C->stream = s;
    QT_HIP(hipGetDevice(&C->device));
    C->levels.resize(L);
    return C.release();
}

static qt_matrix* empty_result(const qt_matrix* A, const qt_matrix* B, int L, qt_prec prec, hipStream_t s,
                               const MulOp& op) {
    qt_matrix* C = new_result(A, B, L, prec, s, op);
    C->pairs.assign(L + 1, 0);
    return C;
}

// Symbolic phase of C = A*B: C's tree, block keys and (uninitialised) value
// array, plus the product lists the numeric phase reads (kept in
// out.scratch). out.na.nseg == 0 means C has no blocks. In three steps, so that
// the problems of a batch can share launches and one wait:
//   plan:    checks, counts, operand forms, the two allocations;
//   launch:  the kernels, on the traversal's stream, and the read-back;
//   finish:  waits for the counts (the one synchronization), forms C.
struct Symbolic {
    qt_matrix* A;
    qt_matrix* B;
    qt_prec prec;
    hipStream_t s;
    SymbolicOut& out;
    MulOp op;
    bool batched = false;   // one of many: its launches may be shared, and are not timed

    // plan
    bool done = false;      // C is empty, known without a traversal
    bool prune = false, bounds = false, small = false, sparse = false, may_strip = false, may_korder = false, prof = false;
    int L = 0, liftA = 0, liftB = 0, lb_log = 0, strip_log = 0, strip_bits = 1, kbits = 1;
    hipStream_t ss = nullptr;                 // the traversal's stream
    std::vector<int64_t> pairs, ncap, foff, gsum_at;
    std::vector<int32_t> group;               // levels taken a pair per lane: C nodes per wave, else 0
    int64_t P = 0, cap = 0, nil_tiles = 0, nclear = 0, read_bytes = 0;
    qt_matrix* Av = nullptr;
    NumericArgs na{};
    std::vector<size_t> o_child, o_key, u_child, u_key, u_parent, o_fa, o_fb, o_cseg, o_cnt, o_off, o_tot, o_wagg;
    size_t o_lbase = 0, o_lmo = 0, o_lrm = 0, o_lcm = 0, o_bkey = 0;
    size_t o_prodA = 0, o_prodB = 0, o_cbseg = 0, u_lbase = 0, u_lmo = 0, u_lrm = 0, u_lcm = 0, o_nflags = 0,
           o_ntcnt = 0, o_nex = 0, o_gsum = 0, o_scan = 0, o_lcnt = 0, o_heavy = 0, o_sort = 0, o_order = 0, o_count = 0;
    size_t keep_bytes = 0, work_bytes = 0;
    char* K = nullptr;
    char* W = nullptr;
    const int32_t* lift = nullptr;
    int32_t* dcount = nullptr;                // the counts (see plan)
    int32_t* nflags = nullptr;
    LeafStep ls{};

    // launch
    std::unique_ptr<ReadBack> counts;         // unless shared with other problems
    hipError_t traced = hipSuccess;
    bool running = false;                     // launched, not known to have ended
    bool strips = false, korder = false;      // the launch order, known once C's blocks are counted
    bool later = false;                       // by inner index, left to the plan

    Symbolic(qt_matrix* a, qt_matrix* b, qt_prec p, hipStream_t stream, SymbolicOut& o, const MulOp& which)
        : A(a), B(b), prec(p), s(stream), out(o), op(which) {}
    Symbolic(const Symbolic&) = delete;
    Symbolic& operator=(const Symbolic&) = delete;
    // after an error between launch and finish: the kernels use the scratch
    // and the slot
    ~Symbolic() {
        if (running) (void)hipStreamSynchronize(ss);
    }

    static void* at(char* base, size_t off) { return (void*)(base + off); }
    int ncounts() const { return 3 * L + 4; }
    int64_t wgs(int l) const { return group[l] ? (ncap[l] + group[l] - 1) / group[l] : level_wgs(ncap[l]); }
    int32_t pick_group(int l) const;
    int32_t heavy_max() const { return (int32_t)(P / (SPARSE_MAX + 1)); }   // leaves of more than SPARSE_MAX products
    bool single_waves() const;                // every level in single-wave workgroups
    void plan();
    void bind(char* tree, char* work);
    TreeStep tree_step(int l) const;
    TreeStep fill_step(int l) const;          // with the next level's counts, where the fill makes them
    bool fill_counts(int l) const;
    bool together() const;                    // its launches may be shared with other problems
    RootInit root_step() const;
    LeafStep leaf_step() const;
    NilMark nil_mark() const;
    NilTree nil_tree() const;
    SmallStep small_step() const;
    void launch();
    const int32_t* wait();                    // the counts, by the problem's own read-back
    void finish(const int32_t* hc);           // of a batch, the launch orders are sorted after it
    int32_t* order() const { return (int32_t*)at(W, o_order); }
    void sort_order(int32_t nnzC);
    size_t value_bytes() const { return (size_t)na.nseg * A->b * A->b * (prec == QT_F32 ? sizeof(float) : sizeof(double)); }
    void bind_values(char* values);
};

void Symbolic::plan() {
    if (prec != QT_F64 && prec != QT_F32 && prec != QT_BF16X3) fail(QT_ERR_ARG, "unknown precision");
    if (A->b != B->b || A->leaf != B->leaf) fail(QT_ERR_SHAPE, "operands differ in block or leaf size");
    const int64_t a_cols = op.ta ? A->n_rows : A->n_cols;   // op(A) = A or A^T
    const int64_t b_rows = op.tb ? B->n_cols : B->n_rows;
    if (a_cols != b_rows) fail(QT_ERR_SHAPE, "inner dimensions differ");
    if (op.upper && (op.ta ? A->n_cols : A->n_rows) != (op.tb ? B->n_rows : B->n_cols))
        fail(QT_ERR_SHAPE, "an upper-triangular product must be square");
    if (prec == QT_BF16X3 && A->b == 16) fail(QT_ERR_UNSUPPORTED, "split-bf16 path needs b = 32 or 64");
    prune = op.tau2 > 0;   // a norm threshold
    if (prune && (op.ta || op.tb || op.upper || A->vsrc || B->vsrc))
        fail(QT_ERR_UNSUPPORTED, "a norm threshold needs C = A * B of stored operands");
    // with a norm threshold (or only the upper triangle) the counts known
    // beforehand are bounds, not exact
    bounds = op.upper || prune;
    L = std::max(A->L, B->L);
    liftA = L - A->L;
    liftB = L - B->L;
    out.na = NumericArgs{};
    out.prof = false;
    if (A->nblocks == 0 || B->nblocks == 0) {
        out.C.reset(empty_result(A, B, L, prec, s, op));
        done = true;
        return;
    }

    ss = side_stream();
    build_histograms(A, ss);
    build_histograms(B, ss);
    if (prune) {
        // the norms read the operands' values, ready in order on the caller's
        // stream: made there, and the traversal waits for them, not for what
        // else is queued on that stream: in a loop of products with a threshold
        // and their copy-outs it runs beside the copy-out before it (a decay32768
        // product in FP32 597 -> 499 us)
        build_norms(A, s, ss);
        build_norms(B, s, ss);
    }

    // pair counts per level and block products: exact, or upper bounds when
    // only the upper triangle of C is formed. Columns of op(A) are rows of A
    // when A is used transposed, and likewise for B.
    const auto& a_col = op.ta ? A->hist.rowcnt : A->hist.colcnt;
    const auto& b_row = op.tb ? B->hist.colcnt : B->hist.rowcnt;
    pairs.resize(L + 1);
    for (int l = 0; l <= L; ++l) {
        const auto& ca = (l < liftA) ? unit_hist() : a_col[l - liftA];
        const auto& rb = (l < liftB) ? unit_hist() : b_row[l - liftB];
        pairs[l] = dot_counts(ca, rb);
    }
    P = dot_counts(op.ta ? A->hist.blk_row : A->hist.blk_col,
                   op.tb ? B->hist.blk_col : B->hist.blk_row);
    lb_log = A->lb_log;
    const int64_t lb2 = int64_t(1) << (2 * lb_log);
    for (int l = 0; l <= L; ++l)
        if (4 * pairs[l] > kMaxI32) fail(QT_ERR_UNSUPPORTED, "too many node pairs at one level");
    // bound on C nodes per level: every C node has at least one pair, and
    // there are only so many node positions in C's shape at that level (the
    // per-node arrays and the level kernels' grids are sized by this; at the
    // deep levels of an unstructured product it is far below the pair count)
    ncap.resize(L + 1);
    {
        const int64_t c_rows = op.ta ? A->n_cols : A->n_rows, c_cols = op.tb ? B->n_rows : B->n_cols;
        for (int l = 0; l <= L; ++l) {
            const int64_t side = (int64_t)A->leaf << (L - l);
            const int64_t pos = ((c_rows + side - 1) / side) * ((c_cols + side - 1) / side);
            ncap[l] = std::max<int64_t>(std::min(pairs[l], pos), 1);
        }
    }
    if (P > kMaxI32) fail(QT_ERR_UNSUPPORTED, "too many block products");
    if (P == 0) {
        out.C.reset(empty_result(A, B, L, prec, s, op));
        out.C->pairs = pairs;
        done = true;
        return;
    }

    // operand forms for this precision, from the matrices that hold the values
    // (a structure-only operand reads its value source's blocks). A block read
    // transposed is marked in the product lists and transposed as it is
    // loaded: no transposed copy of any operand is made.
    Av = A->vsrc ? A->vsrc : A;
    qt_matrix* Bv = B->vsrc ? B->vsrc : B;
    na.b = A->b;
    na.prec = prec;
    na.dyn = (op.ta || op.tb || A->vsrc || B->vsrc) ? 1 : 0;
    if (prec == QT_F64) {
        na.A = operand_f64(Av, s);
        na.B = operand_f64(Bv, s);
    } else if (prec == QT_F32) {
        na.A = operand_f32(Av, s);
        na.B = operand_f32(Bv, s);
    } else {
        operand_bf16(Av, s);
        operand_bf16(Bv, s);
        na.Ahi = Av->bf_hi.p;
        na.Alo = Av->bf_lo.p;
        na.Ahi_t = Av->bf_hi_t.p;
        na.Alo_t = Av->bf_lo_t.p;
        na.Bhi = Bv->bf_hi.p;
        na.Blo = Bv->bf_lo.p;
        na.Bhi_t = Bv->bf_hi_t.p;
        na.Blo_t = Bv->bf_lo_t.p;
    }

    // ---- plan the two allocations
    cap = std::min<int64_t>(P, lb2 * ncap[L]);   // bound on C blocks
    // one launch for the whole phase when every level fits one workgroup
    small = L <= SMALL_LEVELS && P <= SMALL_PRODUCTS;
    int64_t all_nodes = 0;
    for (int l = 0; l <= L; ++l) {
        small = small && pairs[l] <= SMALL_PAIRS;
        all_nodes += ncap[l];
    }
    small = small && all_nodes <= SMALL_NODES;
    // levels of few pairs per node, leaves of few products: a pair per lane
    group.assign(L + 1, 0);
    if (!small && !bounds && !(batched && single_waves())) {
        for (int l = 0; l < L; ++l)
            if (ncap[l] >= TREE_MIN && pairs[l] <= TREE_PAIRS * ncap[l]) group[l] = pick_group(l);
        if (!A->vsrc && !B->vsrc && lb_log == 3 && P <= SPARSE_LEAF * ncap[L]) group[L] = pick_group(L);
    }
    sparse = group[L] != 0;
    // a wave per node is 64 threads, of which a grid has fewer than 2^32 (a larger
    // one is launched in part, without an error)
    for (int l = 0; l <= L; ++l)
        if (!group[l] && ncap[l] >= (int64_t(1) << 26) - 4) fail(QT_ERR_UNSUPPORTED, "too many C nodes at one level");
    // the launch order in strips, of the block rows of C (see above)
    const int64_t c_rows_blk = (op.ta ? A->n_cols : A->n_rows) / A->b;
    const int64_t row_bytes = A->nblocks * (int64_t)A->b * A->b * (prec == QT_F64 ? 8 : 4) / std::max<int64_t>(c_rows_blk, 1);
    while (strip_log < STRIP_MAX_LOG && (row_bytes << (strip_log + 1)) <= STRIP_BYTES) ++strip_log;
    while ((int64_t(1) << (strip_bits + strip_log)) < c_rows_blk) ++strip_bits;
    may_strip = !small && A->b == 64 && cap >= STRIP_MIN_BLOCKS && P >= 2 * STRIP_MIN_BLOCKS;
    // the order by inner index is built once C's block count is known, if
    // the products are then fewer than twice the C blocks (cap bounds those)
    const int64_t kdim = (op.ta ? A->n_rows : A->n_cols) / A->b;
    while ((int64_t(1) << kbits) < kdim) ++kbits;
    read_bytes = 2 * P * A->b * A->b * (prec == QT_F64 ? 8 : 4);
    may_korder = P < 2 * cap && kbits <= KORDER_MAX_BITS && (batched || (!small && read_bytes >= KORDER_MIN_BYTES));
    ArenaPlan keep, tmp;   // keep: C's tree; tmp: scratch freed after the call
    o_child.resize(L);
    o_key.resize(L + 1);
    for (int l = 0; l < L; ++l) o_child[l] = keep.take(4 * ncap[l] * sizeof(int32_t));
    for (int l = 0; l <= L; ++l) o_key[l] = keep.take(ncap[l] * sizeof(uint64_t));
    o_lbase = keep.take(ncap[L] * sizeof(int32_t));
    o_lmo = keep.take(ncap[L] * sizeof(uint64_t));
    o_lrm = keep.take(ncap[L] * sizeof(uint64_t));
    o_lcm = keep.take(ncap[L] * sizeof(uint64_t));
    o_bkey = keep.take(cap * sizeof(uint64_t));
    if (L + 1 > NIL_MAX_LEVELS) fail(QT_ERR_UNSUPPORTED, "quadtree too deep");
    o_prodA = tmp.take(P * sizeof(int32_t));
    o_prodB = tmp.take(P * sizeof(int32_t));
    o_cbseg = tmp.take((cap + 1) * sizeof(int32_t));
    if (may_strip || may_korder) {   // one order is built at most
        o_sort = tmp.take(std::max(may_strip ? sort_tmp_bound(cap, strip_bits) : 0,
                                   may_korder ? sort_tmp_bound(cap, kbits) : 0) * sizeof(int32_t));
        o_order = tmp.take(cap * sizeof(int32_t));
    }
    // The scratch of the level by level traversal from here on (a small
    // product's stays in LDS): first the tree before NIL normalisation.
    const size_t small_bytes = tmp.bytes;
    u_child.resize(L);
    u_key.resize(L + 1);
    u_parent.resize(L + 1);
    for (int l = 0; l < L; ++l) u_child[l] = tmp.take(4 * ncap[l] * sizeof(int32_t));
    for (int l = 0; l <= L; ++l) u_key[l] = tmp.take(ncap[l] * sizeof(uint64_t));
    for (int l = 1; l <= L; ++l) u_parent[l] = tmp.take(ncap[l] * sizeof(int32_t));
    u_lbase = tmp.take(ncap[L] * sizeof(int32_t));
    u_lmo = tmp.take(ncap[L] * sizeof(uint64_t));
    u_lrm = tmp.take(ncap[L] * sizeof(uint64_t));
    u_lcm = tmp.take(ncap[L] * sizeof(uint64_t));
    foff.assign(L + 2, 0);
    for (int l = 0; l <= L; ++l) foff[l + 1] = foff[l] + ncap[l];
    if (foff[L + 1] > kMaxI32) fail(QT_ERR_UNSUPPORTED, "too many C nodes");
    // Cleared by the traversal's first kernel, in one run: the NIL flags of all
    // levels, the group sums of every level's
    // workgroup aggregates, and the aggregates themselves (the levels whose
    // counts the previous level's fill makes have no count kernel to write
    // the aggregates of workgroups without a node).
    nil_tiles = foff[L + 1] / NIL_TILE + 1;
    o_ntcnt = tmp.take(nil_tiles * sizeof(int32_t));
    o_nflags = tmp.take(nil_tiles * NIL_TILE * sizeof(int32_t));
    gsum_at.resize(L + 1);
    int64_t gsum_total = 0;
    for (int l = 0; l <= L; ++l) {
        gsum_at[l] = gsum_total;
        gsum_total += (wgs(l) + (1 << AGG_GROUP_LOG) - 1) >> AGG_GROUP_LOG;
    }
    o_gsum = tmp.take(std::max<int64_t>(gsum_total, 1) * sizeof(int64_t));
    for (auto* v : {&o_fa, &o_fb, &o_cseg, &o_cnt, &o_off, &o_tot, &o_wagg}) v->resize(L + 1);
    for (int l = 0; l <= L; ++l) o_wagg[l] = tmp.take(wgs(l) * sizeof(int64_t));
    if (sparse) o_heavy = tmp.take(sizeof(int32_t));   // its number is cleared, too; the list lies behind
    nclear = (int64_t)(tmp.bytes - o_nflags) / (int64_t)sizeof(int32_t);
    if (sparse) (void)tmp.take(heavy_max() * sizeof(int32_t));
    o_nex = tmp.take(nil_tiles * NIL_TILE * sizeof(int32_t));
    size_t scan_elems = 0;
    for (int l = 0; l <= L; ++l) {
        o_fa[l] = tmp.take(pairs[l] * sizeof(int32_t));
        o_fb[l] = tmp.take(pairs[l] * sizeof(int32_t));
        o_cseg[l] = tmp.take((ncap[l] + 1) * sizeof(int32_t));
        o_cnt[l] = tmp.take(ncap[l] * sizeof(int64_t));
        o_off[l] = tmp.take((ncap[l] + 1) * sizeof(int64_t));
        o_tot[l] = tmp.take(ncap[l] * sizeof(int4));
        scan_elems = std::max(scan_elems, scan_tmp_elems(ncap[l]));
    }
    o_scan = tmp.take((scan_elems + 1) * sizeof(int64_t));
    o_lcnt = sparse ? 0 : tmp.take(ncap[L] * 64 * sizeof(int32_t));   // leaf step: products per block position
    o_count = tmp.take(ncounts() * sizeof(int32_t));

    out.C.reset(new_result(A, B, L, prec, s, op));
    qt_matrix* C = out.C.get();
    C->pairs = pairs;
    C->products = P;
    keep_bytes = keep.bytes;
    work_bytes = small ? small_bytes : tmp.bytes;
    if (!batched) bind(nullptr, nullptr);
}

// The two buffers: its own (NULL), or parts of buffers shared by the problems of
// a batch.
void Symbolic::bind(char* tree, char* work) {
    qt_matrix* C = out.C.get();
    if (tree) {
        C->arena.view(tree, keep_bytes);
        out.scratch.view(work, work_bytes);
    } else {
        // both live on past this call and are released on the caller's stream,
        // after the numeric kernel that reads them
        C->arena.alloc(keep_bytes, ss);
        C->arena.s = s;
        out.scratch.alloc(work_bytes, ss);
        out.scratch.s = s;
    }
    K = C->arena.p;
    W = out.scratch.p;
    // [0..L] C nodes per level as traversed, [L+1] C blocks, [L+2..2L+2] checks,
    // [2L+3..3L+3] C nodes per level after NIL normalisation
    dcount = (int32_t*)at(W, o_count);
    nflags = (int32_t*)at(W, o_nflags);

    prof = out.prof = !batched && profiling_on();
    lift = (liftA > 0 || liftB > 0) ? lift_table() : nullptr;
    // the leaf step's operands and outputs
    ls.lb_log = lb_log;
    // rows of op(A) are columns of A when transposed; columns of op(B) rows of B
    ls.Arm = op.ta ? A->leaves.mask_cm.p : A->leaves.mask_rm.p;
    ls.Bcm = op.tb ? B->leaves.mask_rm.p : B->leaves.mask_cm.p;
    ls.Brm = op.tb ? B->leaves.mask_cm.p : B->leaves.mask_rm.p;
    ls.group = group[L];
    ls.ta = op.ta;
    ls.tb = op.tb;
    ls.upper = op.upper;
    ls.amap = A->vsrc ? A->bmap.p : nullptr;
    ls.bmap = B->vsrc ? B->bmap.p : nullptr;
    if (prune) {
        ls.Abn2 = A->bn2;
        ls.Bbn2 = B->bn2;
        ls.tau2 = op.tau2;
    }
    ls.Amo = A->leaves.mask_mo.p;
    ls.Bmo = B->leaves.mask_mo.p;
    ls.Abase = A->leaves.base.p;
    ls.Bbase = B->leaves.base.p;
    ls.prodA = (int32_t*)at(W, o_prodA);
    ls.prodB = (int32_t*)at(W, o_prodB);
    ls.P = (int32_t)P;
    ls.cbkey = (uint64_t*)at(K, o_bkey);
    ls.cbseg = (int32_t*)at(W, o_cbseg);
    ls.cap = (int32_t)cap;
    if (ncounts() > kSlotWords) fail(QT_ERR_UNSUPPORTED, "tree too deep for the count read-back");
}

TreeStep Symbolic::tree_step(int l) const {
    TreeStep st{};
    st.fa = (const int32_t*)at(W, o_fa[l]);
    st.fb = (const int32_t*)at(W, o_fb[l]);
    st.cseg = (const int32_t*)at(W, o_cseg[l]);
    st.ckey = (const uint64_t*)at(W, u_key[l]);
    st.ncount = dcount + l;
    st.Ach = (l < liftA) ? lift : A->levels[l - liftA].child.p;
    st.Bch = (l < liftB) ? lift : B->levels[l - liftB].child.p;
    st.cnt = (int64_t*)at(W, o_cnt[l]);
    st.tot4 = (int4*)at(W, o_tot[l]);
    st.wagg = (int64_t*)at(W, o_wagg[l]);
    st.gsum = (int64_t*)at(W, o_gsum) + gsum_at[l];
    st.group = group[l];
    st.use_agg = wgs(l) <= AGG_MAX;
    st.off = (int64_t*)at(W, o_off[l]);
    st.ncap = (int32_t)ncap[l];
    st.nfa = (int32_t*)at(W, o_fa[l + 1]);
    st.nfb = (int32_t*)at(W, o_fb[l + 1]);
    st.ncseg = (int32_t*)at(W, o_cseg[l + 1]);
    st.nckey = (uint64_t*)at(W, u_key[l + 1]);
    st.cchild = (int32_t*)at(W, u_child[l]);
    st.nparent = (int32_t*)at(W, u_parent[l + 1]);
    st.ncount_next = dcount + l + 1;
    st.np_next = (int32_t)pairs[l + 1];
    st.nc_next = (int32_t)ncap[l + 1];
    st.check = dcount + L + 2 + l;
    st.ta = op.ta;
    st.tb = op.tb;
    st.upper = op.upper;
    if (prune) {
        // norms of the next level's nodes; above a shallower operand's root
        // (the lifted levels) every child is its root
        st.An2 = (l + 1 <= liftA) ? A->nn2[0] : A->nn2[l + 1 - liftA];
        st.Bn2 = (l + 1 <= liftB) ? B->nn2[0] : B->nn2[l + 1 - liftB];
        st.tau2 = op.tau2;
    }
    return st;
}

// a single-wave next tree level gets its counts from this level's fill
bool Symbolic::fill_counts(int l) const {
    return l + 1 < L && level_waves(ncap[l + 1]) == 1 && !group[l] && !group[l + 1];
}

TreeStep Symbolic::fill_step(int l) const {
    TreeStep st = tree_step(l);
    if (fill_counts(l)) {
        const TreeStep nx = tree_step(l + 1);
        st.nAch = nx.Ach;
        st.nBch = nx.Bch;
        st.nAn2 = nx.An2;
        st.nBn2 = nx.Bn2;
        st.ncnt = nx.cnt;
        st.ntot4 = nx.tot4;
        st.noff = nx.off;
        st.nwagg = nx.wagg;
        st.ngsum = nx.gsum;
    }
    return st;
}

// C nodes per wave at level l: as many as fill it with pairs, while the waves
// still fill the GPU; 0: the kernels that take a pair per lane don't apply.
int32_t Symbolic::pick_group(int l) const {
    int64_t g = 1;
    while (g < 16 && 2 * g * pairs[l] <= 64 * ncap[l] && ncap[l] / (2 * g) >= 4096) g *= 2;
    while (g < TREE_GROUP_MAX && (ncap[l] + g - 1) / g > AGG_MAX) g *= 2;
    // a C node has at most as many pairs as there are inner node positions: the
    // tree count's 16-bit sums and the product keys' 17 bits hold that
    const int64_t side = (int64_t)A->leaf << (L - l), inner = ((op.ta ? A->n_rows : A->n_cols) + side - 1) / side;
    const bool fits = l < L ? 2 * inner < (1 << 16) : inner * g <= (1 << 17);
    return fits && (ncap[l] + g - 1) / g <= AGG_MAX ? (int32_t)g : 0;
}

// What the shared kernels are compiled for: no norms and no block maps, and
// one node per workgroup (so every fill makes the next level's counts).
bool Symbolic::together() const {
    if (prof || prune || ls.amap || ls.bmap) return false;
    return small || (L > 0 && single_waves());
}

bool Symbolic::single_waves() const {
    for (int l = 0; l <= L; ++l)
        if (level_waves(ncap[l]) != 1) return false;
    return true;
}

RootInit Symbolic::root_step() const {
    return RootInit{(int32_t*)at(W, o_fa[0]), (int32_t*)at(W, o_fb[0]), (int32_t*)at(W, o_cseg[0]),
                    (uint64_t*)at(W, u_key[0]), dcount, nflags, nclear};
}

LeafStep Symbolic::leaf_step() const {
    LeafStep st = ls;
    st.fa = (const int32_t*)at(W, o_fa[L]);
    st.fb = (const int32_t*)at(W, o_fb[L]);
    st.cseg = (const int32_t*)at(W, o_cseg[L]);
    st.ckey = (const uint64_t*)at(W, u_key[L]);
    st.ncount = dcount + L;
    st.ncap = (int32_t)ncap[L];
    st.cnt = (int64_t*)at(W, o_cnt[L]);
    st.lane_cnt = (int32_t*)at(W, o_lcnt);
    st.off = (int64_t*)at(W, o_off[L]);
    st.wagg = (int64_t*)at(W, o_wagg[L]);
    st.gsum = (int64_t*)at(W, o_gsum) + gsum_at[L];
    st.use_agg = wgs(L) <= AGG_MAX;
    if (sparse) {
        st.heavy = (int32_t*)at(W, o_heavy);
        st.heavy_max = heavy_max();
    }
    st.lbase = (int32_t*)at(W, u_lbase);
    st.lmo = (uint64_t*)at(W, u_lmo);
    st.lrm = (uint64_t*)at(W, u_lrm);
    st.lcm = (uint64_t*)at(W, u_lcm);
    st.nblocks_out = dcount + L + 1;
    st.check = dcount + 2 * L + 2;
    return st;
}

NilMark Symbolic::nil_mark() const {
    NilMark m{};
    m.L = L;
    for (int l = 0; l <= L + 1; ++l) m.foff[l] = foff[l];
    for (int l = 1; l <= L; ++l) m.uparent[l] = (const int32_t*)at(W, u_parent[l]);
    m.flags = nflags;
    m.tcnt = (int32_t*)at(W, o_ntcnt);
    m.tiles = nil_tiles;
    return m;
}

// NIL normalisation: C keeps only the nodes with a block below them
NilTree Symbolic::nil_tree() const {
    NilTree nt{};
    nt.L = L;
    for (int l = 0; l <= L + 1; ++l) nt.foff[l] = foff[l];
    for (int l = 0; l < L; ++l) {
        nt.uchild[l] = (const int32_t*)at(W, u_child[l]);
        nt.child[l] = (int32_t*)at(K, o_child[l]);
    }
    for (int l = 0; l <= L; ++l) {
        nt.ukey[l] = (const uint64_t*)at(W, u_key[l]);
        nt.key[l] = (uint64_t*)at(K, o_key[l]);
    }
    nt.ubase = (const int32_t*)at(W, u_lbase);
    nt.umo = (const uint64_t*)at(W, u_lmo);
    nt.urm = (const uint64_t*)at(W, u_lrm);
    nt.ucm = (const uint64_t*)at(W, u_lcm);
    nt.flags = nflags;
    nt.tcnt = (const int32_t*)at(W, o_ntcnt);
    nt.tiles = nil_tiles;
    nt.ex = (int32_t*)at(W, o_nex);
    nt.base = (int32_t*)at(K, o_lbase);
    nt.mo = (uint64_t*)at(K, o_lmo);
    nt.rm = (uint64_t*)at(K, o_lrm);
    nt.cm = (uint64_t*)at(K, o_lcm);
    nt.kept = dcount + 2 * L + 3;
    return nt;
}

SmallStep Symbolic::small_step() const {
    SmallStep sm{};
    sm.L = L;
    for (int l = 0; l < L; ++l) {
        sm.Ach[l] = (l < liftA) ? lift : A->levels[l - liftA].child.p;
        sm.Bch[l] = (l < liftB) ? lift : B->levels[l - liftB].child.p;
        sm.child[l] = (int32_t*)at(K, o_child[l]);
    }
    for (int l = 0; l <= L; ++l) {
        if (prune) {
            sm.An2[l] = A->nn2[std::max(l - liftA, 0)];
            sm.Bn2[l] = B->nn2[std::max(l - liftB, 0)];
        }
        sm.key[l] = (uint64_t*)at(K, o_key[l]);
    }
    sm.leaf = ls;
    sm.base = (int32_t*)at(K, o_lbase);
    sm.mo = (uint64_t*)at(K, o_lmo);
    sm.rm = (uint64_t*)at(K, o_lrm);
    sm.cm = (uint64_t*)at(K, o_lcm);
    if (counts) {
        sm.slot = counts->device_slot();
        sm.seq = counts->seq();
    } else {
        sm.counts = dcount;
    }
    return sm;
}

void Symbolic::launch() {
    PhaseEvents& ev = out.ev;
    if (prof) {
        timing_event(&ev.e0);
        timing_event(&ev.e1);
        timing_event(&ev.e2);
        timing_event(&ev.e3);
        QT_HIP(hipEventRecord(ev.e0, ss));
    }
    counts.reset(new ReadBack(ncounts()));
    running = true;
    if (small) {
        const SmallStep sm = small_step();
        if (prune)
            k_small_symbolic<true, false><<<1, SMALL_THREADS, 0, ss>>>(sm);
        else if (ls.amap || ls.bmap)
            k_small_symbolic<false, false><<<1, SMALL_THREADS, 0, ss>>>(sm);
        else
            k_small_symbolic<false, true><<<1, SMALL_THREADS, 0, ss>>>(sm);
        QT_LAUNCH("k_small_symbolic");
    } else {
        k_root_init<<<(unsigned)((nclear + 63) / 64), 64, 0, ss>>>(root_step());
        QT_LAUNCH("k_root_init");
        int64_t* scan_tmp = (int64_t*)at(W, o_scan);
        bool counted = false;   // this level's counts were made by the previous level's fill
        for (int l = 0; l < L; ++l) {
            const TreeStep sl = fill_step(l);
            const int64_t wgs = this->wgs(l);
            if (group[l]) {
                k_tree_count_sparse<<<(unsigned)wgs, 64, 0, ss>>>(sl);
                QT_LAUNCH("k_tree_count_sparse");
                k_tree_fill_sparse<<<(unsigned)wgs, 64, 0, ss>>>(sl);
                QT_LAUNCH("k_tree_fill_sparse");
                counted = false;
                continue;
            }
            if (!counted) {
                if (prune)
                    QT_LEVEL_LAUNCH(k_tree_count, ncap[l], wgs, ss, sl, true);
                else
                    QT_LEVEL_LAUNCH(k_tree_count, ncap[l], wgs, ss, sl, false);
                if (!sl.use_agg) exclusive_scan(sl.cnt, sl.off, ncap[l], scan_tmp, ss);
            }
            counted = fill_counts(l);
            if (prune && counted)
                QT_LEVEL_LAUNCH(k_tree_fill, ncap[l], wgs, ss, sl, true, true);
            else if (prune)
                QT_LEVEL_LAUNCH(k_tree_fill, ncap[l], wgs, ss, sl, true, false);
            else if (counted)
                QT_LEVEL_LAUNCH(k_tree_fill, ncap[l], wgs, ss, sl, false, true);
            else
                QT_LEVEL_LAUNCH(k_tree_fill, ncap[l], wgs, ss, sl, false, false);
        }
        const LeafStep st = leaf_step();
        const NilMark mark = nil_mark();
        if (sparse) {
            k_leaf_count_sparse<<<(unsigned)wgs(L), 64, 0, ss>>>(st, mark);
            QT_LAUNCH("k_leaf_count_sparse");
            k_leaf_fill_sparse<<<(unsigned)(st.heavy_max + wgs(L)), 64, 0, ss>>>(st, mark);
            QT_LAUNCH("k_leaf_fill_sparse");
        } else {
            if (prune)
                QT_LEVEL_LAUNCH(k_leaf_count, ncap[L], wgs(L), ss, QT_ARGS(st, mark), true);
            else
                QT_LEVEL_LAUNCH(k_leaf_count, ncap[L], wgs(L), ss, QT_ARGS(st, mark), false);
            if (!st.use_agg) exclusive_scan(st.cnt, st.off, ncap[L], scan_tmp, ss);
            if (prune || st.amap || st.bmap)
                QT_LEVEL_LAUNCH(k_leaf_fill, ncap[L], wgs(L), ss, QT_ARGS(st, mark), false);
            else
                QT_LEVEL_LAUNCH(k_leaf_fill, ncap[L], wgs(L), ss, QT_ARGS(st, mark), true);
        }
        const NilTree nt = nil_tree();
        k_nil_offsets<<<(unsigned)nil_tiles, 64, 0, ss>>>(nt.flags, nt.tcnt, nt.ex);
        QT_LAUNCH("k_nil_offsets");
        k_nil_compact<<<(unsigned)((foff[L + 1] + 63) / 64), 64, 0, ss>>>(nt);
        QT_LAUNCH("k_nil_compact");
        counts->publish(dcount, ss);
    }
    traced = prof ? hipEventRecord(ev.e1, ss) : hipSuccess;
}

const int32_t* Symbolic::wait() {
    const int32_t* hc = counts->wait(ss);
    QT_HIP(traced);
    return hc;
}

// hc: the counts, published after all of the problem's kernels
void Symbolic::finish(const int32_t* hc) {
    running = false;
    qt_matrix* C = out.C.get();
    PhaseEvents& ev = out.ev;
    for (int l = 0; l <= L; ++l) {
        if (hc[l] < 0 || hc[l] > ncap[l]) fail(QT_ERR_DEVICE, "symbolic phase: C node count out of range");
        if (hc[2 * L + 3 + l] < 0 || hc[2 * L + 3 + l] > hc[l])
            fail(QT_ERR_DEVICE, "symbolic phase: kept C node count out of range");
        const int64_t expect = (l < L) ? pairs[l + 1] : P;
        const bool bad = bounds ? (hc[L + 2 + l] < 0 || hc[L + 2 + l] > expect) : (hc[L + 2 + l] != expect);
        if (bad) fail(QT_ERR_DEVICE, "symbolic phase: pair count mismatch");
        if (l < L) C->pairs[l + 1] = hc[L + 2 + l];   // pairs actually formed
    }
    C->products = hc[2 * L + 2];
    const int32_t nnzC = hc[L + 1];
    if (nnzC < 0 || nnzC > cap || (nnzC == 0 && !bounds)) fail(QT_ERR_DEVICE, "symbolic phase: C block count out of range");

    strips = may_strip && nnzC >= STRIP_MIN_BLOCKS && C->products >= 2 * (int64_t)nnzC;
    korder = may_korder && nnzC > 0 && C->products < 2 * (int64_t)nnzC;
    later = korder && batched && read_bytes < KORDER_MIN_BYTES;
    if (later)
        out.later = LaterOrder{Av->bkey.p, ls.prodA, ls.cbseg, order(), (int32_t*)at(W, o_sort), nnzC, kbits};
    if ((strips || korder) && !batched) {
        running = true;   // until s runs after the sort, which uses the scratch
        sort_order(nnzC);
        if (prof) QT_HIP(hipEventRecord(ev.e1, ss));   // the symbolic phase ends here then
        QT_HIP(stream_after(s, ss));
        running = false;
    }

    // C's tree (NIL-normalised): views into its arena
    const int32_t* kept = hc + 2 * L + 3;
    for (int l = 0; l < L; ++l) {
        C->levels[l].n = kept[l];
        C->levels[l].child.view(at(K, o_child[l]), 4 * (size_t)kept[l]);
        C->levels[l].key.view(at(K, o_key[l]), kept[l]);
    }
    LeafLevel& CL = C->leaves;
    CL.n = kept[L];
    CL.key.view(at(K, o_key[L]), kept[L]);
    CL.base.view(at(K, o_lbase), kept[L]);
    CL.mask_mo.view(at(K, o_lmo), kept[L]);
    CL.mask_rm.view(at(K, o_lrm), kept[L]);
    CL.mask_cm.view(at(K, o_lcm), kept[L]);
    if ((nnzC > 0) != (kept[L] > 0)) fail(QT_ERR_DEVICE, "symbolic phase: C leaves and blocks disagree");
    C->bkey.view(at(K, o_bkey), nnzC);
    C->nblocks = nnzC;

    na.prodA = ls.prodA;
    na.prodB = ls.prodB;
    na.seg = ls.cbseg;
    na.order = (strips || (korder && !later)) ? order() : nullptr;
    na.by_k = korder && !later ? 1 : 0;
    na.nseg = nnzC;
    ev.products = C->products;
    ev.cblocks = nnzC;
    if (!batched) bind_values(nullptr);
}

// The launch order that finish() chose, sorted on ss.
void Symbolic::sort_order(int32_t nnzC) {
    int32_t* tmp = (int32_t*)at(W, o_sort);
    if (strips)
        stable_sort(StripKeys{ls.cbkey, strip_log}, OrderSink{order()}, nnzC, strip_bits, tmp, order(), ss);
    else
        stable_sort(FirstKeys{Av->bkey.p, ls.prodA, ls.cbseg}, OrderSink{order()}, nnzC, kbits, tmp, order(), ss);
}

// C's values: a buffer of its own (NULL), or part of a shared one.
void Symbolic::bind_values(char* values) {
    qt_matrix* C = out.C.get();
    const size_t n = (size_t)na.nseg * C->b * C->b;
    if (prec == QT_F32) {
        if (values)
            C->v32.view(values, n);
        else
            C->v32.alloc(n, s);
        na.C = C->v32.p;
    } else {
        if (values)
            C->v64.view(values, n);
        else
            C->v64.alloc(n, s);
        na.C = C->v64.p;
    }
    out.na = na;
}

static void symbolic(qt_matrix* A, qt_matrix* B, qt_prec prec, hipStream_t s, SymbolicOut& out, const MulOp& op) {
    Symbolic sym(A, B, prec, s, out, op);
    sym.plan();
    if (sym.done) return;
    sym.launch();
    // the caller's stream follows the traversal from here on (the numeric
    // kernel first), ordered while the counts are on their way; a launch order
    // built by finish() adds a second wait
    const hipError_t ordered = stream_after(s, sym.ss);
    const int32_t* hc = sym.wait();
    QT_HIP(ordered);
    sym.finish(hc);
}

// The problems of `who` level by level, one launch per step for all of them;
// their counts go to dcount. The step records are made in `host`, which lives
// until the copy from it is known to have ended.
static void launch_levels(const std::vector<Symbolic*>& who, std::vector<char>& host, DBuf<char>& dev, hipStream_t ss) {
    const size_t np = who.size();
    int depth = 0;
    for (const Symbolic* p : who) depth = std::max(depth, p->L);
    ArenaPlan ap;
    const size_t o_many = ap.take(np * sizeof(ManyStep)), o_steps = ap.take(np * depth * sizeof(TreeStep));
    host.assign(ap.bytes, 0);
    ManyStep* many = (ManyStep*)(host.data() + o_many);
    TreeStep* steps = (TreeStep*)(host.data() + o_steps);
    int64_t clear = 1, leaves = 1, tiles = 1, nodes = 1;
    std::vector<int64_t> widest(depth, 1);
    for (size_t i = 0; i < np; ++i) {
        Symbolic& p = *who[i];
        many[i].first = depth - p.L;
        many[i].root = p.root_step();
        many[i].leaf = p.leaf_step();
        many[i].mark = p.nil_mark();
        many[i].nil = p.nil_tree();
        for (int l = 0; l < p.L; ++l) {
            steps[(many[i].first + l) * np + i] = p.fill_step(l);
            widest[many[i].first + l] = std::max(widest[many[i].first + l], p.ncap[l]);
        }
        clear = std::max(clear, p.nclear);
        leaves = std::max(leaves, p.ncap[p.L]);
        tiles = std::max(tiles, p.nil_tiles);
        nodes = std::max(nodes, p.foff[p.L + 1]);
        p.running = true;
    }
    dev.alloc(ap.bytes, ss);
    QT_HIP(hipMemcpyAsync(dev.p, host.data(), ap.bytes, hipMemcpyHostToDevice, ss));
    const ManyStep* dm = (const ManyStep*)(dev.p + o_many);
    const TreeStep* ds = (const TreeStep*)(dev.p + o_steps);
    const unsigned y = (unsigned)np;
    k_root_init_many<<<dim3((unsigned)((clear + 63) / 64), y), 64, 0, ss>>>(dm);
    QT_LAUNCH("k_root_init_many");
    k_tree_count_many<<<dim3(1, y), 64, 0, ss>>>(dm, ds);
    QT_LAUNCH("k_tree_count_many");
    for (int r = 0; r < depth; ++r) {
        const dim3 grid((unsigned)widest[r], y);
        if (r + 1 < depth)
            k_tree_fill_many<true><<<grid, 64, 0, ss>>>(ds + r * np);
        else
            k_tree_fill_many<false><<<grid, 64, 0, ss>>>(ds + r * np);
        QT_LAUNCH("k_tree_fill_many");
    }
    k_leaf_count_many<<<dim3((unsigned)leaves, y), 64, 0, ss>>>(dm);
    QT_LAUNCH("k_leaf_count_many");
    k_leaf_fill_many<<<dim3((unsigned)leaves, y), 64, 0, ss>>>(dm);
    QT_LAUNCH("k_leaf_fill_many");
    k_nil_offsets_many<<<dim3((unsigned)tiles, y), 64, 0, ss>>>(dm);
    QT_LAUNCH("k_nil_offsets_many");
    k_nil_compact_many<<<dim3((unsigned)((nodes + 63) / 64), y), 64, 0, ss>>>(dm);
    QT_LAUNCH("k_nil_compact_many");
}

// The small problems of `who`, one workgroup each.
static void launch_small(const std::vector<Symbolic*>& who, std::vector<char>& host, DBuf<char>& dev, hipStream_t ss) {
    if (who.empty()) return;
    host.assign(who.size() * sizeof(SmallStep), 0);
    SmallStep* steps = (SmallStep*)host.data();
    for (size_t i = 0; i < who.size(); ++i) {
        steps[i] = who[i]->small_step();
        who[i]->running = true;
    }
    dev.alloc(host.size(), ss);
    QT_HIP(hipMemcpyAsync(dev.p, host.data(), host.size(), hipMemcpyHostToDevice, ss));
    k_small_symbolic_many<<<(unsigned)who.size(), SMALL_THREADS, 0, ss>>>((const SmallStep*)dev.p);
    QT_LAUNCH("k_small_symbolic_many");
}

// Problems whose launches are shared: at most MANY_MAX (their records, counts
// and read-back slots are bounded by it), and level by level only while the
// workgroups of a launch that find no node of their problem stay few: the grid
// is the widest problem's times the number of problems, at most MANY_GRID or
// MANY_WASTE times what the problems need (an idle workgroup costs about a
// nanosecond: below MANY_GRID less than the twelve launches that a group of
// its own takes).
constexpr int32_t MANY_MAX = 256;
constexpr int64_t MANY_GRID = 65536, MANY_WASTE = 4;

// Parts of shared buffers for the problems of a batch: an allocation takes the
// host 5 us and its release 3, of which three a problem were a third of the time
// of a plan of 16. A buffer holds parts of up to SHARED_MAX together (a part
// beyond it has one of its own), allocated on `ready`, released on `s`.
constexpr size_t SHARED_MAX = size_t(256) << 20;

static std::vector<char*> shared_parts(const std::vector<size_t>& bytes, hipStream_t ready, hipStream_t s,
                                       std::vector<DBuf<char>>& pool) {
    std::vector<char*> at(bytes.size(), nullptr);
    for (size_t i = 0; i < bytes.size();) {
        ArenaPlan ap;
        std::vector<size_t> off;
        for (size_t j = i; j < bytes.size() && (off.empty() || ap.bytes + bytes[j] <= SHARED_MAX); ++j)
            off.push_back(ap.take(bytes[j]));
        pool.emplace_back();
        pool.back().alloc(ap.bytes, ready);
        pool.back().s = s;
        for (size_t o : off) at[i++] = pool.back().p + o;
    }
    return at;
}

// The launch orders of the problems of `who`, but those left to the plan; s runs
// after them.
static void sort_orders(const std::vector<Symbolic*>& who, hipStream_t s, hipStream_t ss) {
    struct Drain {   // the sorts use the problems' scratch: after an error they have ended before it goes
        hipStream_t st;
        bool on;
        ~Drain() {
            if (on) (void)hipStreamSynchronize(st);
        }
    } drain{ss, false};
    for (Symbolic* p : who) {
        if (!p->strips && (!p->korder || p->later)) continue;
        drain.on = true;
        p->sort_order(p->na.nseg);
    }
    if (!drain.on) return;
    QT_HIP(stream_after(s, ss));
    drain.on = false;
}

// A plan's orders by inner index, sorted when it first runs again. Those of up to
// RANK_SORT_MAX blocks share a launch: one, with an event and a wait, for each took 17 us
// a problem (64 small ones 1.1 ms).
typedef RankJob<FirstKeys, OrderSink> LaterJob;

size_t later_job_bytes() { return sizeof(LaterJob); }
bool later_shares(const LaterOrder& o) { return o.n <= RANK_SORT_MAX; }
void later_job(const LaterOrder& o, void* job) {
    const LaterJob j{FirstKeys{o.akey, o.prodA, o.seg}, OrderSink{o.order}, o.n};
    std::memcpy(job, &j, sizeof(j));
}

void sort_later(const std::vector<LaterOrder>& who, const void* jobs, hipStream_t s) {
    int32_t most = 0;
    unsigned shared = 0;
    for (const LaterOrder& o : who) {
        if (later_shares(o)) {
            most = std::max(most, o.n);
            ++shared;
        } else {
            stable_sort(FirstKeys{o.akey, o.prodA, o.seg}, OrderSink{o.order}, o.n, o.kbits, o.tmp, o.order, s);
        }
    }
    for (unsigned at = 0; at < shared; at += 32768) {   // of the 65535 a grid may have in y
        const dim3 grid((unsigned)((most + 63) / 64), std::min(shared - at, 32768u));
        k_rank_sort_many<FirstKeys, OrderSink>
            <<<grid, 256, most * sizeof(uint64_t), s>>>((const LaterJob*)jobs + at);
        QT_LAUNCH("k_rank_sort_many");
    }
}

void symbolic_batch(int32_t count, qt_matrix* const* A, qt_matrix* const* B, qt_prec prec, hipStream_t s,
                    SymbolicOut* out, std::vector<DBuf<char>>& pool) {
    for (int32_t at = 0; at < count; at += MANY_MAX) {
        const int32_t n = std::min(MANY_MAX, count - at);
        // declared before the problems, whose destructors wait for the kernels
        std::deque<std::vector<char>> host;
        std::deque<DBuf<char>> dev;
        DBuf<int32_t> words;
        std::unique_ptr<ReadBack> shared;
        std::vector<std::unique_ptr<Symbolic>> all;
        std::vector<Symbolic*> work, alone, small, levels, order;   // order: as their counts lie in words
        std::vector<size_t> bytes;
        for (int32_t i = at; i < at + n; ++i) {
            all.emplace_back(new Symbolic(A[i], B[i], prec, s, out[i], MulOp{}));
            Symbolic* p = all.back().get();
            p->batched = true;
            p->plan();
            if (p->done) continue;
            work.push_back(p);
            bytes.push_back(p->keep_bytes);
            bytes.push_back(p->work_bytes);
        }
        if (work.empty()) continue;
        const hipStream_t ss = work[0]->ss;
        const std::vector<char*> parts = shared_parts(bytes, ss, s, pool);
        for (size_t i = 0; i < work.size(); ++i) {
            Symbolic* p = work[i];
            p->bind(parts[2 * i], parts[2 * i + 1]);
            if (!p->together())
                alone.push_back(p);
            else
                (p->small ? small : levels).push_back(p);
        }
        order = small;
        order.insert(order.end(), levels.begin(), levels.end());
        for (Symbolic* p : alone) p->launch();
        int stride = 0;
        for (Symbolic* p : order) stride = std::max(stride, p->ncounts());
        if (!order.empty()) {
            words.alloc(stride * order.size(), ss);
            for (size_t i = 0; i < order.size(); ++i) order[i]->dcount = words.p + i * stride;
            launch_small(small, host.emplace_back(), dev.emplace_back(), ss);
            // widest first, so that problems of about one size share launches
            std::stable_sort(levels.begin(), levels.end(),
                             [](const Symbolic* x, const Symbolic* y) { return x->foff[x->L + 1] > y->foff[y->L + 1]; });
            for (size_t i = 0; i < levels.size();) {
                std::vector<Symbolic*> group;
                int64_t need = 0;
                const int64_t widest = levels[i]->foff[levels[i]->L + 1];
                for (; i < levels.size(); ++i) {
                    need += levels[i]->foff[levels[i]->L + 1];
                    if (widest * (int64_t)(group.size() + 1) > std::max(MANY_GRID, MANY_WASTE * need)) break;
                    group.push_back(levels[i]);
                }
                launch_levels(group, host.emplace_back(), dev.emplace_back(), ss);
            }
            shared.reset(new ReadBack(stride * order.size()));
            shared->publish(words.p, ss);
        }
        const hipError_t ordered = stream_after(s, ss);
        const int32_t* hc = order.empty() ? nullptr : shared->wait(ss);
        QT_HIP(ordered);
        for (size_t i = 0; i < order.size(); ++i) order[i]->finish(hc + i * stride);
        for (Symbolic* p : alone) p->finish(p->wait());
        sort_orders(work, s, ss);
        bytes.clear();
        for (Symbolic* p : work) bytes.push_back(p->value_bytes());
        const std::vector<char*> values = shared_parts(bytes, s, s, pool);
        for (size_t i = 0; i < work.size(); ++i) work[i]->bind_values(values[i]);
    }
}

qt_matrix* multiply(qt_matrix* A, qt_matrix* B, qt_prec prec, hipStream_t s, const MulOp& op) {
    SymbolicOut sym;
    symbolic(A, B, prec, s, sym, op);
    if (sym.prof) QT_HIP(hipEventRecord(sym.ev.e3, s));
    if (sym.na.nseg > 0) launch_numeric(sym.na, s);
    if (sym.prof) {
        QT_HIP(hipEventRecord(sym.ev.e2, s));
        profile_push(sym.ev);
    }
    return sym.C.release();   // sym.scratch is released in stream order
}

}  // namespace qt
