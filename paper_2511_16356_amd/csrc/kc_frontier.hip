// kc_frontier.hip -- the frontier sampler: uniform spanning trees by bulk cycle
// popping, one workgroup per sample, and the kernels built on it.
//
// Cycle popping (section 2.2 by its equivalent of Propp and Wilson, J. Algorithms
// 27, 1998): every vertex but the root holds the arrow of its k-th draw; while
// the arrows have a cycle, any cycle is popped, i.e. its vertices draw again.
// The tree and the draw counts do not depend on the order of the pops, so all
// cycles of the current arrows that are found in a round are popped together:
//
//   walk    each vertex that drew in the round before (the frontier) follows the
//           arrows; it is back at itself (a cycle), at a vertex known to reach the
//           root, or at a frontier vertex with a smaller index, which will find
//           any cycle through both (so exactly one vertex finds a cycle)
//   pop     the finder lists the cycle's vertices: the next frontier
//   draw    they draw again
//
// with a barrier between the three.  The frontier is all vertices at first.
// On graphs with short walks that leaves a few dozen rounds per tree, which
// stream the arrows and touch no per-vertex state beyond one word and the draw
// count; on small graphs the arrows are held in LDS, where a step of a walk is
// one LDS read (large graphs with long walks keep the chain sampler of
// kc_device.hip: there the longest walk of each round would be paid in L2 round
// trips; so do calls with many samples where the words leave a CU one or two
// workgroups.  kc_host::route_of has the rule and both sides' times).

#include <algorithm>
#include <type_traits>

#include "kc_tree.h"

namespace kc {
namespace {

// Threads per sample.  Words in LDS: the frontier is a few dozen vertices, 256 threads
// cover it, the draws ahead and the streaming passes (2,000 trees of the 32 x 32 grid:
// 12.1 / 12.6 / 16.8 ms with 128 / 256 / 512; 256 of a road-like graph of 8,609 vertices:
// 250 / 226 / 212 ms).  Words in memory: a tree has enough work for 512, and fewer trees
// in flight share the caches better (2,048 of a power-law graph of 481,994 vertices:
// 321 / 294 / 281 ms; one tree: 36 / 22 / 15.6 ms).
constexpr int LT = 256, GT = 512;
constexpr int FT_WAVES = 4;  // wavefronts per SIMD the kernels are built to fit (128 VGPRs)
// Trees the caller holds: as above (1,024 vertices and 2,000 trees: 1.7 against 2.6 ms
// with 512; 481,994 vertices and 256 trees: 29.0 against 25.4 ms).  Small trees, in more
// slots than 256 threads each let be in flight (four on a CU), are evaluated by one
// wavefront each: their phases are too short for the barriers (20,000 trees, 256 threads
// against 64: grid of 1,024 10.1 / 6.7 ms, of 64 1.38 / 0.63 ms, power-law graph of 497
// vertices 1.46 / 0.54 ms; 4,096 trees of a grid of 4,096 7.4 / 6.9 ms; from there on, and
// with fewer slots, 256 are as fast or faster: road-like graph of 5,749, 1,024 trees 2.25 /
// 2.99 ms).
int tree_threads(int64_t n, int traversal, int mode, int64_t slots) {
    if (traversal != 2 && n > LDS_MAX_N) return GT;
    return mode == RUN_EVALUATE && slots > 1024 && n <= (traversal == 2 ? 4096 : 512) ? WAVE : LT;
}

// Entries of the frontier, of the found cycles and of the due walks' table kept
// in LDS; frontier and cycles beyond (early rounds only) go to the slot's block.
constexpr int F_LDS = 512, O_LDS = 256, D_LDS = 512;

// The limit of rounds (iter_cap) counts the chain sampler's: two of these are one.  Bulk pops
// take a fraction of the chains' rounds on most graphs, but as many and up to 9% more where
// walks are longest (paths of 700 vertices 87.9k against 85.1k, caterpillars of 1,000 88.7k
// against 81.2k), and what is within the limit there has to be within it here.

// A walk that is not over after this many steps stays due until no shorter
// cycle is left, so that a round is not as long as the longest walk.
constexpr int WALK_CAP = 12;

struct FrontierShared {
    int32_t front[F_LDS];
    int2 found[O_LDS];      // {finder, first position of its cycle in the next frontier}
    uint64_t n_cycles[2];   // a round's cycles: vertices << 32 | cycles (even and odd rounds)
    int32_t n_list, n_long; // walkers listed, long walks
    int32_t err;
    // the due walks (sample_lds): vertex, its word, the next due vertex's place, steps to it
    uint16_t due_v[D_LDS];
    int16_t due_next[D_LDS];
    uint16_t due_len[D_LDS];
    uint32_t due_word[D_LDS];
};

template <int T>
struct FrontierLds {
    FrontierShared samp;
    TreeShared<T> tree;
};

// Where a sampler keeps its lists in a slot's state block (20 bytes per vertex).
struct FrontierWS {
    uint32_t *word;   // sample_global: the words
    uint32_t *cnt;    // how often each vertex drew
    int2 *found;      // n / 2 entries
    int32_t *front, *longs;
};
__device__ __forceinline__ FrontierWS frontier_ws(const SlotPtrs &sp) {
    unsigned char *st = sp.state;
    const size_t n = sp.stride;
    return {reinterpret_cast<uint32_t *>(st), reinterpret_cast<uint32_t *>(st + 4 * n),
            reinterpret_cast<int2 *>(st + 8 * n), reinterpret_cast<int32_t *>(st + 12 * n),
            reinterpret_cast<int32_t *>(st + 16 * n)};
}
__device__ __forceinline__ int get_front(const FrontierShared &sh, const FrontierWS &ws, int i) {
    return i < F_LDS ? sh.front[i] : aload(&ws.front[i]);
}
__device__ __forceinline__ void put_front(FrontierShared &sh, const FrontierWS &ws, int i, int v) {
    if (i < F_LDS) sh.front[i] = v;
    else astore(&ws.front[i], (int32_t)v);
}
__device__ __forceinline__ int2 get_found(const FrontierShared &sh, const FrontierWS &ws, int i) {
    return i < O_LDS ? sh.found[i] : ws.found[i];
}
// f found a cycle of len vertices (cycles are disjoint, so there are at most n / 2).
__device__ __forceinline__ void put_found(FrontierShared &sh, const FrontierWS &ws, int parity, int n, int f, int len) {
    const uint64_t c = afetch_add(&sh.n_cycles[parity], (uint64_t)len << 32 | 1);
    const int pos = (int)(c >> 32), at = (int)(uint32_t)c;
    if (at < O_LDS) sh.found[at] = make_int2(f, pos);
    else if (at < n / 2) ws.found[at] = make_int2(f, pos);
}

// A vertex's graph record, and the neighbour it holds or the row does at slot j.
struct VRec {
    int4 a, b;
};
__device__ __forceinline__ VRec load_rec(const GraphDev &g, int v) {
    return {g.vrec[2 * (size_t)v], g.vrec[2 * (size_t)v + 1]};
}
__device__ __forceinline__ int32_t neighbour(const GraphDev &g, const VRec &r, uint32_t j) {
    if (j >= (uint32_t)VREC_INLINE) return g.adj[(size_t)r.a.x + j];
    // select in registers (an indexed read would place the record in scratch memory)
    const bool odd = (j & 1u) != 0u;
    int p01 = odd ? r.a.w : r.a.z, p23 = odd ? r.b.y : r.b.x, p45 = odd ? r.b.w : r.b.z;
    asm volatile("" : "+v"(p01), "+v"(p23), "+v"(p45));
    return j < 2u ? p01 : (j < 4u ? p23 : p45);
}

// The words of sample_lds: the arrow's target, the target of the vertex's next
// draw (drawn ahead), SET: known to reach the root (the roots from the start),
// FLAG: the walk since its last draw is still due.  Both flags: a place in the
// table of the due walks, while those are taken.
constexpr uint32_t L_MASK = (1u << 15) - 1, L_SET = 1u << 30, L_FLAG = 1u << 31;
static_assert(LDS_MAX_N <= (int64_t)L_MASK, "vertices fit a word's fields");

// One sample's tree, its words in LDS.
//
// All vertices start with a walk due; they enter as walkers in the threads the
// frontier leaves free.  While some wavefronts walk, others draw ahead for the
// vertices that have just drawn, so that a pop needs no memory but LDS: the
// finder of a cycle steps along it and turns each vertex's arrow to the target
// drawn ahead.  A round is bound by the latency of its longest walk and pop.
//
// When no cycle within WALK_CAP steps of a frontier vertex is left, the vertices
// whose walks were cut get places in a table.  Each walks to the next of them
// (every cycle holds one, and no walk goes further than that), and the cycles
// are those of the table's links.
//
// Trees of the chain sampler (a wavefront each, its words in L2) and these: the
// 32 x 32 grid, 2,000 trees 50.9 -> 10.9 ms, one tree 3.8 -> 0.86 ms; a road-like
// graph of 8,609 vertices, 256 trees 519 -> 198 ms.
// Returns the total number of draws, or -1 (error recorded in ctl).
template <int T>
__device__ __forceinline__ int64_t sample_lds(const GraphDev &g, const FrontierWS &ws, uint32_t *words,
                                              FrontierShared &sh, uint64_t seed, uint64_t s, int64_t iter_cap,
                                              int32_t *ctl, int idx, int64_t *iters_used, int32_t root_u,
                                              int32_t root_v) {
    const int tid = threadIdx.x;
    const int n = g.n;
    const bool two_roots = root_u >= 0;  // start from {u, v} instead of {root}
    const int top = two_roots ? root_u : g.root;
    auto load = [&](int v) __attribute__((always_inline)) { return *(const volatile uint32_t *)(words + v); };
    if (tid == 0) {
        sh.n_cycles[0] = sh.n_cycles[1] = 0;
        sh.n_list = sh.err = 0;
    }
    // every vertex's first arrow, and the next
    constexpr int U = 4;
    for (int b = 0; b < n; b += T * U) {
        int64_t o[U];
        uint32_t d[U];
        int32_t t0[U], t1[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int v = b + k * T + tid;
            o[k] = v < n ? g.off[v] : 0;
            d[k] = v < n ? (uint32_t)(g.off[v + 1] - o[k]) : 0;
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int v = b + k * T + tid;
            t0[k] = t1[k] = 0;
            if (v < n) {
                t0[k] = g.adj[o[k] + arrow_slot(seed, s, (uint32_t)v, 0u, d[k])];
                t1[k] = g.adj[o[k] + arrow_slot(seed, s, (uint32_t)v, 1u, d[k])];
            }
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int v = b + k * T + tid;
            if (v >= n) continue;
            const bool in_tree = two_roots ? (v == root_u || v == root_v) : v == g.root;
            words[v] = in_tree ? ((uint32_t)v | L_SET) : ((uint32_t)t0[k] | (uint32_t)t1[k] << 15 | L_FLAG);
            astore(&ws.cnt[v], in_tree ? 0u : 1u);
        }
    }
    __syncthreads();

    int64_t steps = n - (two_roots ? 2 : 1), iters = 0;
    int n_front = 0, next = 0;
    while (true) {
        const int parity = (int)(iters & 1);
        const int take = min(max(T - n_front, 0), n - next), walkers = n_front + take;
        if (walkers != 0) {
            // ---- walk (thread i: walker i), and draw ahead (thread i + T/2 mod T: frontier vertex i)
            const int r = (tid + T / 2) & (T - 1);
            int av = -1;
            uint32_t ak = 0;
            VRec ar{};
            if (r < n_front) {
                av = get_front(sh, ws, r);
                ak = aload(&ws.cnt[av]) + 1;
                ar = load_rec(g, av);
            }
            for (int b = 0; b < walkers; b += T) {
                const int i = b + tid;
                int f = -1;
                if (i < n_front) {
                    f = get_front(sh, ws, i);
                    if (f >= next) f = -1;  // its first walk is still to come
                } else if (i < walkers) {
                    f = next + i - n_front;
                }
                const uint32_t w = load(f >= 0 ? f : top);
                if (w & L_SET) f = -1;
                int x = f >= 0 ? (int)(w & L_MASK) : top, len = 1, left = WALK_CAP;
                uint32_t wx;
                bool go;
                // a step leaves a walk that is over where it is: no branch per lane
                do {
                    wx = load(x);
                    go = !((wx & L_SET) || ((wx & L_FLAG) && x <= f));
                    x = go ? (int)(wx & L_MASK) : x;
                    len += go ? 1 : 0;
                } while (--left && __builtin_amdgcn_ballot_w64(go) != 0ull);
                if (f >= 0 && !go) {
                    if (x == f) put_found(sh, ws, parity, n, f, len);
                    else (void)afetch_xor(&words[f], wx & L_SET ? L_SET | L_FLAG : L_FLAG);
                }
            }
            for (int i = r; i < n_front; i += T) {
                if (i != r) {
                    av = get_front(sh, ws, i);
                    ak = aload(&ws.cnt[av]) + 1;
                    ar = load_rec(g, av);
                }
                const int32_t t = neighbour(g, ar, arrow_slot(seed, s, (uint32_t)av, ak, (uint32_t)ar.a.y));
                astore(&ws.cnt[av], ak);
                (void)afetch_or(&words[av], (uint32_t)t << 15);
            }
            next += take;
        } else {
            // ---- the due walks (four words per thread at a time: most hold none)
            for (int b = 0; b < n; b += 4 * T) {
                const int v0 = b + 4 * tid;
                uint4 q = make_uint4(0, 0, 0, 0);
                if (v0 < n) q = *reinterpret_cast<const uint4 *>(words + v0);  // (padded to 16 bytes)
                const uint32_t w[4] = {q.x, q.y, q.z, q.w};
                uint32_t due = 0;
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (v0 + k < n && (w[k] & (L_FLAG | L_SET)) == L_FLAG) due |= 1u << k;
                if (__ballot(due != 0) == 0ull) continue;
                int c = 0;
#pragma unroll
                for (int k = 0; k < 4; ++k) c += __popcll(__ballot(due >> k & 1u));
                int at = take_shared(&sh.n_list, c);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint64_t m = __ballot(due >> k & 1u);
                    const int i = at + rank_in(m);
                    if ((due >> k & 1u) && i < D_LDS) {
                        sh.due_v[i] = (uint16_t)(v0 + k);
                        sh.due_word[i] = w[k];
                        words[v0 + k] = (uint32_t)i | L_FLAG | L_SET;
                    }
                    at += __popcll(m);
                }
            }
            __syncthreads();
            const int n_list = sh.n_list, n_due = min(n_list, D_LDS);  // (the others: next time)
            if (n_due == 0) break;
            for (int b = 0; b < n_due; b += T) {
                const int i = b + tid;
                int x = i < n_due ? (int)(sh.due_word[i] & L_MASK) : top, len = 1, mark = -1;
                uint32_t wx, step = 1;
                bool go;
                do {  // (as above; Brent's marks only where the table is too small, so that a cycle
                      // may have no place in it)
                    wx = load(x);
                    go = !(wx & L_SET) && x != mark;
                    if (n_list > D_LDS && (step & (step - 1)) == 0) mark = go ? x : mark;
                    x = go ? (int)(wx & L_MASK) : x;
                    len += go ? 1 : 0;
                    ++step;
                } while (__builtin_amdgcn_ballot_w64(go) != 0ull);
                if (i < n_due) {
                    sh.due_next[i] = (int16_t)(!(wx & L_SET) ? -2 : (wx & L_FLAG ? (int)(wx & L_MASK) : -1));
                    sh.due_len[i] = (uint16_t)len;
                }
            }
            __syncthreads();
            for (int i = tid; i < n_due; i += T) {
                int y = sh.due_next[i], len = sh.due_len[i], mark = -1, at = 1;
                while (y > i && y != mark) {
                    if ((at & (at - 1)) == 0) mark = y;
                    ++at;
                    len += sh.due_len[y];
                    y = sh.due_next[y];
                }
                const int f = sh.due_v[i];
                const uint32_t w = sh.due_word[i];
                if (y == i) put_found(sh, ws, parity, n, f, len);
                words[f] = y == i ? w : (y == -1 ? w ^ (L_FLAG | L_SET) : w ^ L_FLAG);
            }
        }
        if (++iters >> 1 > iter_cap) {
            if (tid == 0) report_error(ctl, DEV_LIMIT, idx);
            return -1;
        }
        __syncthreads();
        // ---- pop: the found cycles' vertices draw, and are the next frontier
        const uint64_t cycles = sh.n_cycles[parity];
        const int n_found = (int)(uint32_t)cycles;
        n_front = (int)(cycles >> 32);
        if (n_front > n || n_found > n / 2) {  // never
            if (tid == 0) report_error(ctl, DEV_PROTOCOL, idx);
            return -1;
        }
        steps += n_front;
        for (int i = tid; i < n_found; i += T) {
            const int2 e = get_found(sh, ws, i);
            int y = e.x, pos = e.y;
            do {
                const uint32_t w = load(y);
                words[y] = (w >> 15 & L_MASK) | L_FLAG;
                put_front(sh, ws, pos++, y);
                y = (int)(w & L_MASK);
            } while (y != e.x && pos < n_front);
        }
        if (tid == 0) {
            sh.n_cycles[parity ^ 1] = 0;
            sh.n_list = 0;
        }
        __syncthreads();
    }
    *iters_used = iters;
    return steps;
}

// The words of sample_global: the arrow's target and the two flags.
constexpr uint32_t G_MASK = (1u << 30) - 1, G_SET = 1u << 30, G_FLAG = 1u << 31;

// One sample's tree, its words in the slot's block.  The first round walks from
// every vertex (there the smallest index on a cycle finds it, without flags),
// the later ones from the frontier.
//
// Bound by the random lines of the words and graph records: about two per draw
// where the chain sampler has a claim, an arrow and a record.  A power-law graph of
// 481,994 vertices, 2,048 trees 174 -> 91 ms, one tree 65 -> 6.5 ms; a dense one of
// 150,001 vertices, 2,560 trees 90 -> 30 ms.
template <int T>
__device__ __forceinline__ int64_t sample_global(const GraphDev &g, const FrontierWS &ws, FrontierShared &sh,
                                                 TreeShared<T> &tree, uint64_t seed, uint64_t s, int64_t iter_cap,
                                                 int32_t *ctl, int idx, int64_t *iters_used, int32_t root_u,
                                                 int32_t root_v) {
    constexpr uint32_t FLAG = G_FLAG, SET = G_SET, MASK = G_MASK;
    const int tid = threadIdx.x;
    const int n = g.n;
    const bool two_roots = root_u >= 0;  // start from {u, v} instead of {root}
    const int top = two_roots ? root_u : g.root;
    uint32_t *words = ws.word;
    auto wload = [](const uint32_t *w, int v) __attribute__((always_inline)) { return aload(w + v); };
    auto wstore = [](uint32_t *w, int v, uint32_t x) __attribute__((always_inline)) { astore(w + v, x); };
    auto front = [&](int i) { return get_front(sh, ws, i); };
    if (tid == 0) {
        sh.n_cycles[0] = sh.n_cycles[1] = 0;
        sh.n_list = sh.n_long = sh.err = 0;
    }

    // every vertex's first arrow
    constexpr int U = 4;
    int64_t steps = 0;
    for (int b = 0; b < n; b += T * U) {
        int64_t o[U];
        uint32_t d[U];
        int32_t t[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int v = b + k * T + tid;
            o[k] = 0;
            d[k] = 0;
            if (v < n) {
                o[k] = g.off[v];
                d[k] = (uint32_t)(g.off[v + 1] - o[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int v = b + k * T + tid;
            t[k] = v;
            if (v < n) t[k] = g.adj[o[k] + arrow_slot(seed, s, (uint32_t)v, 0u, d[k])];
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int v = b + k * T + tid;
            if (v >= n) continue;
            const bool in_tree = two_roots ? (v == root_u || v == root_v) : v == g.root;
            wstore(words, v, in_tree ? ((uint32_t)v | SET) : (uint32_t)t[k]);
            astore(&ws.cnt[v], in_tree ? 0u : 1u);
            steps += in_tree ? 0 : 1;
        }
    }
    __syncthreads();

    int n_front = 0;
    bool first = true;
    int64_t iters = 0;
    while (true) {
        int walkers = first ? n : n_front;
        if (walkers == 0) break;
        const int parity = (int)(iters & 1);
        if (++iters >> 1 > iter_cap) {
            if (tid == 0) report_error(ctl, DEV_LIMIT, idx);
            return -1;
        }
        // ---- walk
        // the end of f's walk at x (f's word w, x's word wx) after len steps
        auto ended = [&](int f, uint32_t w, int x, uint32_t wx, int len) __attribute__((always_inline)) {
            if (x == f) {
                put_found(sh, ws, parity, n, f, len);
            } else if (wx & SET) {
                wstore(words, f, (w & MASK) | SET);
            } else if (!first) {
                wstore(words, f, w & MASK);
            }
        };
        // WU walks per thread, of the walkers at + k T (count in all).  A step leaves a walk
        // that is over where it is, so a wavefront steps without a branch per lane until none
        // of its walks goes on, or (CAPPED) for WALK_CAP steps: long(f) for those
        auto walk = [&](auto wu, auto is_capped, int at, int count, auto walker, auto long_walk)
            __attribute__((always_inline)) {
            constexpr int WU = decltype(wu)::value;
            constexpr bool CAPPED = decltype(is_capped)::value;
            int f[WU], x[WU], len[WU], mark[WU];
            uint32_t w[WU], wx[WU];
            bool go[WU];
#pragma unroll
            for (int k = 0; k < WU; ++k) {
                const int i = at + k * T;
                f[k] = i < count ? walker(i) : -1;
                len[k] = 1;
                mark[k] = -1;  // Brent's cycle finding: a cycle without f
                go[k] = false;
            }
#pragma unroll
            for (int k = 0; k < WU; ++k) w[k] = wload(words, f[k] >= 0 ? f[k] : top);
#pragma unroll
            for (int k = 0; k < WU; ++k) {
                if (w[k] & SET) f[k] = -1;
                x[k] = f[k] >= 0 ? (int)(w[k] & MASK) : top;
            }
            uint32_t step = 1;
            const uint32_t most = CAPPED ? WALK_CAP + 1 : 8u * (uint32_t)n + 64;  // no walk is longer
            uint64_t any;
            do {
                any = 0;
#pragma unroll
                for (int k = 0; k < WU; ++k) wx[k] = wload(words, x[k]);
#pragma unroll
                for (int k = 0; k < WU; ++k) {
                    go[k] = !((wx[k] & SET) || ((first || (wx[k] & FLAG)) && x[k] <= f[k]) ||
                              (!CAPPED && x[k] == mark[k]));
                    if (!CAPPED && (step & (step - 1)) == 0) mark[k] = go[k] ? x[k] : mark[k];
                    x[k] = go[k] ? (int)(wx[k] & MASK) : x[k];
                    len[k] += go[k] ? 1 : 0;
                    any |= __builtin_amdgcn_ballot_w64(go[k]);
                }
            } while (++step < most && any != 0ull);
#pragma unroll
            for (int k = 0; k < WU; ++k) {
                if (f[k] < 0) continue;
                if (go[k]) long_walk(f[k]);
                else ended(f[k], w[k], x[k], wx[k], len[k]);
            }
        };
        constexpr auto one = std::integral_constant<int, 1>{};
        constexpr auto four = std::integral_constant<int, 4>{};
        auto never = [&](int) { sh.err = 1; };
        if (first) {
            // the first round walks from every vertex.  Most walks end at their first step:
            // those are streamed, several per thread, and the others listed
            for (int b = 0; b < n; b += T * U) {
                uint32_t w[U], wx[U];
#pragma unroll
                for (int k = 0; k < U; ++k) {
                    const int v = b + k * T + tid;
                    w[k] = v < n ? wload(words, v) : SET;
                }
#pragma unroll
                for (int k = 0; k < U; ++k) wx[k] = w[k] & SET ? SET : wload(words, (int)(w[k] & MASK));
                int c = 0;
                uint32_t more = 0;
#pragma unroll
                for (int k = 0; k < U; ++k) {
                    const int v = b + k * T + tid;
                    if (!(wx[k] & SET) && (int)(w[k] & MASK) > v) more |= 1u << k;
                    c += __popcll(__ballot(more >> k & 1u));
                }
                int at = take_shared(&sh.n_list, c);
#pragma unroll
                for (int k = 0; k < U; ++k) {
                    const uint64_t m = __ballot(more >> k & 1u);
                    if (more >> k & 1u) put_front(sh, ws, at + rank_in(m), b + k * T + tid);
                    at += __popcll(m);
                }
            }
            __syncthreads();
            walkers = sh.n_list;
        }
        if (walkers <= T) {
            walk(one, std::false_type{}, tid, walkers, front, never);
        } else {
            // many: in short steps first, so that a wavefront rarely waits for a long walk
            for (int at = tid; at - tid < walkers; at += 4 * T)
                walk(four, std::true_type{}, at, walkers, front,
                     [&](int f) { astore(&ws.longs[afetch_add(&sh.n_long, 1)], (int32_t)f); });
            __syncthreads();
            const int n_long = sh.n_long;
            for (int at = tid; at - tid < n_long; at += T)
                walk(one, std::false_type{}, at, n_long, [&](int i) { return (int)aload(&ws.longs[i]); }, never);
        }
        __syncthreads();
        // ---- pop: the found cycles' vertices are the next frontier
        const uint64_t cycles = sh.n_cycles[parity];
        const int n_found = (int)(uint32_t)cycles;
        n_front = (int)(cycles >> 32);
        if (n_front > n || n_found > n / 2 || sh.err != 0) {  // (cycles are disjoint) never
            if (tid == 0) report_error(ctl, DEV_PROTOCOL, idx);
            return -1;
        }
        for (int i = tid; i < n_found; i += T) {
            const int2 e = get_found(sh, ws, i);
            int y = e.x, pos = e.y;
            do {
                put_front(sh, ws, pos++, y);
                y = (int)(wload(words, y) & MASK);
            } while (y != e.x && pos < n_front);
        }
        first = false;
        __syncthreads();
        // ---- draw
        for (int i = tid; i < n_front; i += T) {
            const int v = front(i);
            const uint32_t k = aload(&ws.cnt[v]);
            const VRec r = load_rec(g, v);
            const int32_t t = neighbour(g, r, arrow_slot(seed, s, (uint32_t)v, k, (uint32_t)r.a.y));
            wstore(words, v, (uint32_t)t | FLAG);
            astore(&ws.cnt[v], k + 1);
            ++steps;
        }
        if (tid == 0) {
            sh.n_cycles[parity] = 0;
            sh.n_list = sh.n_long = 0;
        }
        __syncthreads();
    }
    *iters_used = iters;
    return block_sum<T>(steps, tree);
}

extern __shared__ __align__(16) uint32_t dyn_words[];

// One sample through the whole path, as process_one of the chain sampler.
// (ROUTES: the routes compiled in, one bit each; a launch over one graph has one.
// TREES: the trees go to the caller, else they are evaluated here; kernels of their own,
// so that the evaluation's registers do not weigh on a launch that has none.)
template <int T, int ROUTES, bool TREES>
__device__ __forceinline__ bool process_frontier(const GraphDev &g, const SlotPtrs &sp, FrontierLds<T> &lds,
                                                 uint32_t *dyn, const RunParams &rp, int route, int64_t fen_len,
                                                 int idx, uint64_t s) {
    const FrontierWS ws = frontier_ws(sp);
    const bool in_lds = (ROUTES >> ROUTE_LDS & 1) && (!(ROUTES >> ROUTE_GLOBAL & 1) || route == ROUTE_LDS);
    int64_t steps = 0, iters = 0;
    if (in_lds)
        steps = sample_lds<T>(g, ws, dyn, lds.samp, rp.seed, s, rp.iter_cap, rp.ctl, idx, &iters, rp.root_u,
                              rp.root_v);
    else
        steps = sample_global<T>(g, ws, lds.samp, lds.tree, rp.seed, s, rp.iter_cap, rp.ctl, idx, &iters, rp.root_u,
                                 rp.root_v);
    if (steps < 0) return false;
    auto parent_of = [&](int v) __attribute__((always_inline)) {
        return (int32_t)(in_lds ? dyn[v] & L_MASK : aload(&ws.word[v]) & G_MASK);
    };
    if constexpr (TREES) {
        const size_t n = (size_t)g.n;
        int32_t *po = rp.parents_out + (size_t)idx * n;
        uint32_t *co = rp.cnt_out ? rp.cnt_out + (size_t)idx * n : nullptr;
        for (int v = threadIdx.x; v < g.n; v += T) {
            const bool top = rp.root_u >= 0 ? (v == rp.root_u || v == rp.root_v) : v == g.root;
            po[v] = top ? -1 : parent_of(v);
            if (co) co[v] = aload(&ws.cnt[v]);
        }
    } else {
        evaluate_tree<T>(g, sp, lds.tree, dyn, path_bits(g.n), rp, fen_len, idx, parent_of);
    }
    if (threadIdx.x == 0) {
        if (rp.steps_out) rp.steps_out[idx] = steps;
        if (rp.iters_out) rp.iters_out[idx] = iters;
    }
    return true;
}

// As persistent_kernel and batch_kernel of the chain sampler.
template <int T, int ROUTE, bool TREES>
__global__ void __launch_bounds__(T, FT_WAVES) frontier_kernel(GraphDev g, SlotDev sd, RunParams rp) {
    __shared__ FrontierLds<T> lds;
    const SlotPtrs sp = slot_ptrs(sd, (size_t)g.n);
    int64_t done = 0;
    while (true) {
        const int idx = next_item<T>(rp.ctl, lds.tree);
        if (idx >= rp.count) break;
        if (!process_frontier<T, 1 << ROUTE, TREES>(g, sp, lds, dyn_words, rp, ROUTE, sd.fen_len, idx,
                                                    (uint64_t)(rp.first + idx)))
            break;
        ++done;
        if (rp.progress && threadIdx.x == 0)
            __hip_atomic_store(&rp.progress[blockIdx.x], done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

template <int T>
__global__ void __launch_bounds__(T, FT_WAVES) frontier_batch_kernel(BatchArgs a, SlotDev sd, int32_t *ctl,
                                                                     const int64_t *launch) {
    __shared__ FrontierLds<T> lds;
    const SlotPtrs sp = slot_ptrs(sd, (size_t)sd.stride);
    const int64_t L = *launch;
    while (true) {
        const int idx = next_item<T>(ctl, lds.tree);
        if (idx >= a.base[a.k]) break;
        int j = 0;
        while (j + 1 < a.k && idx >= a.base[j + 1]) ++j;
        const BatchJob &job = a.job[j];
        RunParams rp{};
        rp.seed = job.seed;
        rp.mode = RUN_ESTIMATE;
        rp.traversal = job.traversal;
        rp.iter_cap = job.iter_cap;
        rp.ctl = ctl;
        rp.f_out = a.f;
        rp.steps_out = a.steps;
        rp.iters_out = a.iters;
        const uint64_t s = (uint64_t)(job.first + L * (int64_t)(a.base[j + 1] - a.base[j]) + (idx - a.base[j]));
        if (!process_frontier<T, 1 << ROUTE_LDS | 1 << ROUTE_GLOBAL, false>(job.g, sp, lds, dyn_words, rp, job.route,
                                                                            job.g.two_m + 2, idx, s))
            break;
    }
}

// Trees the caller holds (RUN_EVALUATE, RUN_CROSS).
template <int T>
__global__ void __launch_bounds__(T, FT_WAVES) tree_kernel(GraphDev g, SlotDev sd, RunParams rp) {
    __shared__ TreeShared<T> tree;
    const SlotPtrs sp = slot_ptrs(sd, (size_t)g.n);
    int64_t done = 0;
    while (true) {
        // trees that are short and alike, one wavefront's or a workgroup for each: fixed shares,
        // without the counter's 45 ns per tree (1,024 trees of a grid of 64: 0.14 -> 0.11 ms; of
        // a grid of 1,024 it pays to start them one after the other: 0.70, 0.72 ms)
        const bool shares = T == WAVE || ((int)gridDim.x >= rp.count && g.n <= 512);
        const int64_t item = shares ? blockIdx.x + done * gridDim.x : next_item<T>(rp.ctl, tree);
        if (item >= rp.count) break;
        const int idx = (int)item;
        if (shares) __syncthreads();  // the LDS of the tree before is free
        const size_t row = rp.rows ? (size_t)rp.rows[idx] : (size_t)idx;
        const int32_t *par = rp.parents_in + row * (size_t)g.n;
        if (rp.mode == RUN_CROSS) {
            const int64_t d = crossing_edges<T>(g, sp, rp, par, (int32_t)row, idx, tree);
            if (threadIdx.x == 0) rp.f_out[idx] = d;
        } else {
            evaluate_tree<T>(g, sp, tree, dyn_words, path_bits(g.n), rp, sd.fen_len, idx,
                             [&](int v) { return par[v]; });
        }
        if (threadIdx.x == 0) {
            if (rp.steps_out) rp.steps_out[idx] = 0;
            if (rp.iters_out) rp.iters_out[idx] = 0;
        }
        ++done;
        if (rp.progress && threadIdx.x == 0)
            __hip_atomic_store(&rp.progress[blockIdx.x], done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// Dynamic LDS of a workgroup of T threads: the words of the tree being sampled; in
// their place, once its parents are read, what the traversal of its evaluation takes:
// the sweep's list and nodes, or the path sums' map (64 KB above 2^18 vertices, where the
// sweep takes 28: 1,024 trees of a road-like graph of 315,215 vertices take 146 ms at two
// workgroups per CU, 119 at four).
template <int T>
size_t dyn_lds(int route, int64_t n, int traversal) {
    const size_t words = route == ROUTE_LDS ? 4 * (size_t)n : 0;
    const size_t eval = traversal == 2 ? sizeof(SweepLds<T>) : (size_t)path_bits(n) / 8;
    return (std::max(words, eval) + 15) / 16 * 16;
}

template <typename K>
int resident(K kernel, int threads, size_t lds) {
    int blocks = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, kernel, threads, lds) != hipSuccess) return 0;
    return blocks;
}
// Dynamic LDS above 64 KB is a limit of the kernel, shared by every thread of the process: it
// is set to the most any graph takes, so that no call lowers it between another's two steps.
template <typename K>
hipError_t allow_lds(K kernel, size_t lds) {
    constexpr int most = (4 * (int)LDS_MAX_N + 15) / 16 * 16;
    if (lds <= (64u << 10)) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, most);
}

}  // namespace

template <int T, int ROUTE, bool TREES>
static hipError_t launch_frontier_of(const GraphDev &g, const SlotDev &s, const RunParams &rp, int slots,
                                     hipStream_t stream) {
    const size_t lds = dyn_lds<T>(ROUTE, g.n, rp.traversal);
    const hipError_t e = allow_lds(frontier_kernel<T, ROUTE, TREES>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((frontier_kernel<T, ROUTE, TREES>), dim3(slots), dim3(T), lds, stream, g, s, rp);
    return hipGetLastError();
}
hipError_t launch_frontier(const GraphDev &g, const SlotDev &s, const RunParams &rp, int slots, hipStream_t stream) {
    const bool trees = rp.mode == RUN_SAMPLE;
    if (rp.route == ROUTE_GLOBAL)
        return trees ? launch_frontier_of<GT, ROUTE_GLOBAL, true>(g, s, rp, slots, stream)
                     : launch_frontier_of<GT, ROUTE_GLOBAL, false>(g, s, rp, slots, stream);
    return trees ? launch_frontier_of<LT, ROUTE_LDS, true>(g, s, rp, slots, stream)
                 : launch_frontier_of<LT, ROUTE_LDS, false>(g, s, rp, slots, stream);
}
// A batch's workgroups have the threads its largest graph takes, and the most dynamic LDS of
// its jobs with that many threads (grids of 1,024 take 28 KB with 256; the 40 KB of 512 threads
// left a CU three of those workgroups where it holds four).
static bool batch_is_global(const BatchArgs &a) {
    for (int j = 0; j < a.k; ++j)
        if (a.job[j].route == ROUTE_GLOBAL) return true;
    return false;
}
template <int T>
static size_t batch_lds(const BatchArgs &a) {
    size_t lds = 0;
    for (int j = 0; j < a.k; ++j) lds = std::max(lds, dyn_lds<T>(a.job[j].route, a.job[j].g.n, a.job[j].traversal));
    return lds;
}
template <int T>
static hipError_t launch_batch_of(const BatchArgs &a, const SlotDev &s, int32_t *ctl, const int64_t *launch, int slots,
                                  hipStream_t stream) {
    const size_t lds = batch_lds<T>(a);
    const hipError_t e = allow_lds(frontier_batch_kernel<T>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((frontier_batch_kernel<T>), dim3(slots), dim3(T), lds, stream, a, s, ctl, launch);
    return hipGetLastError();
}
hipError_t launch_frontier_batch(const BatchArgs &a, const SlotDev &s, int32_t *ctl, const int64_t *launch,
                                 int slots, hipStream_t stream) {
    return batch_is_global(a) ? launch_batch_of<GT>(a, s, ctl, launch, slots, stream)
                              : launch_batch_of<LT>(a, s, ctl, launch, slots, stream);
}
template <int T>
static hipError_t launch_trees_of(const GraphDev &g, const SlotDev &s, const RunParams &rp, int slots,
                                  hipStream_t stream) {
    hipLaunchKernelGGL((tree_kernel<T>), dim3(slots), dim3(T), dyn_lds<T>(ROUTE_GLOBAL, g.n, rp.traversal), stream, g,
                       s, rp);
    return hipGetLastError();
}
hipError_t launch_tree(const GraphDev &g, const SlotDev &s, const RunParams &rp, int slots, hipStream_t stream) {
    const int threads = tree_threads(g.n, rp.traversal, rp.mode, slots);
    return threads == GT ? launch_trees_of<GT>(g, s, rp, slots, stream)
         : threads == LT ? launch_trees_of<LT>(g, s, rp, slots, stream)
                         : launch_trees_of<WAVE>(g, s, rp, slots, stream);
}
int frontier_blocks_per_cu(int route, int64_t n, int traversal) {
    return route == ROUTE_GLOBAL ? resident(frontier_kernel<GT, ROUTE_GLOBAL, false>, GT, dyn_lds<GT>(route, n, traversal))
                                 : resident(frontier_kernel<LT, ROUTE_LDS, false>, LT, dyn_lds<LT>(route, n, traversal));
}
int frontier_batch_blocks_per_cu(const BatchArgs &a) {
    return batch_is_global(a) ? resident(frontier_batch_kernel<GT>, GT, batch_lds<GT>(a))
                              : resident(frontier_batch_kernel<LT>, LT, batch_lds<LT>(a));
}
int tree_blocks_per_cu(int64_t n, int traversal, int mode, int64_t slots) {
    const int threads = tree_threads(n, traversal, mode, slots);
    return threads == GT ? resident(tree_kernel<GT>, GT, dyn_lds<GT>(ROUTE_GLOBAL, n, traversal))
         : threads == LT ? resident(tree_kernel<LT>, LT, dyn_lds<LT>(ROUTE_GLOBAL, n, traversal))
                         : resident(tree_kernel<WAVE>, WAVE, dyn_lds<WAVE>(ROUTE_GLOBAL, n, traversal));
}

}  // namespace kc
