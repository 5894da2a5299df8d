// kc_tree.h -- device code shared by the sampling kernels: memory and wave
// helpers, the Philox arrows, and everything a sampled tree goes through
// (volumes, numbering, f).  Included by the kernel files only.
//
// The tree code runs in a workgroup of T threads (64: one wavefront) that owns
// one tree.  Threads exchange data through global memory by workgroup-scope
// relaxed atomics (L2-coherent on gfx950), ordered by the workgroup barriers; for
// the 16-byte loads of records still being completed see pin().
#pragma once

#include <type_traits>

#include "kc_internal.h"

namespace kc {
namespace {

constexpr int WAVE = 64;
// Neighbours kept inline in a vertex's 32-byte graph record (see GraphDev::vrec).
constexpr int VREC_INLINE = 6;

// ------------------------------------------------------------ memory helpers

template <typename T>
__device__ __forceinline__ T aload(const T *p) {
    return __hip_atomic_load(const_cast<T *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <typename T>
__device__ __forceinline__ void astore(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <typename T>
__device__ __forceinline__ T afetch_add(T *p, T v) {
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <typename T>
__device__ __forceinline__ T afetch_or(T *p, T v) {
    return __hip_atomic_fetch_or(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <typename T>
__device__ __forceinline__ T afetch_xor(T *p, T v) {
    return __hip_atomic_fetch_xor(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <typename T>
__device__ __forceinline__ T acas(T *p, T expected, T desired) {
    __hip_atomic_compare_exchange_strong(p, &expected, desired, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_WORKGROUP);
    return expected;  // value found at *p
}
// Orders one wavefront's memory operations among its lanes.
__device__ __forceinline__ void sync_wave() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    __builtin_amdgcn_wave_barrier();
}
__device__ __forceinline__ void fence_wg() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup"); }

// ------------------------------------------------------------- wave helpers

__device__ __forceinline__ int rank_in(uint64_t mask) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}
__device__ __forceinline__ int64_t wave_sum(int64_t v) {
    for (int o = WAVE / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}
__device__ __forceinline__ int wave_max(int v) {
    for (int o = WAVE / 2; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o));
    return v;
}

// The first error of a launch stays (whichever threads call this).
__device__ void report_error(int32_t *ctl, int code, int idx) {
    int expected = 0;
    if (__hip_atomic_compare_exchange_strong(&ctl[1], &expected, code, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT))
        __hip_atomic_store(&ctl[2], idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ------------------------------------------------------------------ arrows

// Philox4x32-10 block function (Salmon, Moraes, Dror, Shaw, SC'11): ten
// rounds of two 32x32->64 multiplies with the Weyl key schedule.  Counter
// (k, v, s_lo, s_hi), key (seed_lo, seed_hi).  The neighbour slot is the
// high word of x * deg with x = out0 | out1 << 32, i.e. floor(x deg / 2^64),
// computed from two 32x32 products.
struct Bits {
    uint32_t lo, hi;
};
__device__ __forceinline__ Bits philox_bits(uint64_t seed, uint64_t s, uint32_t v, uint32_t k) {
    uint32_t x0 = k, x1 = v, x2 = (uint32_t)s, x3 = (uint32_t)(s >> 32);
    uint32_t key0 = (uint32_t)seed, key1 = (uint32_t)(seed >> 32);
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        // one full 32x32->64 product each (a single v_mad_u64_u32, not mul_lo + mul_hi)
        const uint64_t a = (uint64_t)0xD2511F53u * x0;
        const uint64_t b = (uint64_t)0xCD9E8D57u * x2;
        const uint32_t y0 = (uint32_t)(b >> 32) ^ x1 ^ key0;
        const uint32_t y2 = (uint32_t)(a >> 32) ^ x3 ^ key1;
        x0 = y0; x1 = (uint32_t)b; x2 = y2; x3 = (uint32_t)a;
        key0 += 0x9E3779B9u;
        key1 += 0xBB67AE85u;
    }
    return Bits{x0, x1};
}
__device__ __forceinline__ uint32_t slot_of(Bits x, uint32_t deg) {
    const uint64_t lowprod = (uint64_t)x.lo * deg;
    const uint64_t highprod = (uint64_t)x.hi * deg + (lowprod >> 32);
    return (uint32_t)(highprod >> 32);
}
__device__ __forceinline__ uint32_t arrow_slot(uint64_t seed, uint64_t s, uint32_t v, uint32_t k,
                                               uint32_t deg) {
    return slot_of(philox_bits(seed, s, v, k), deg);
}

// --------------------------------------------------------- tree traversal

// The numbered tree: one 16-byte record per vertex, two 8-byte words, so that
// every step of the numbering touches one line per vertex it visits:
//   rec[2v]     pending children << 44 | volume while the volumes are summed
//               (starting at deg(v)); then vol(v) | (tin(v) + 1) << 32, the high
//               half 0 until tin is known
//   rec[2v + 1] parent (low half, -1 at the root) | once the vertex is finished,
//               its offset in the parent's interval << 32
struct SlotPtrs {
    unsigned char *state;  // the sampler's block, 20 bytes per vertex
    size_t stride;
    int4 *queue;
    int32_t *cstart;
    uint64_t *rec;
    int32_t *leaf;         // the tree's leaves
    int32_t *grp;          // per 64 vertices: counts of crossing edges
    int64_t *fen;
};

__device__ __forceinline__ int32_t rec_parent(const uint64_t *rec, int v) {
    return (int32_t)(uint32_t)aload(&rec[2 * (size_t)v + 1]);
}
// A record that other threads may be completing is read by one 16-byte load, then pinned:
// the compiler may not load parts of it again or apart, so that what is tested is what is
// used.  Each of its two words is written by one 8-byte store, from "unknown" to the only
// value it can have, and a half of an aligned 16-byte load is read whole: a word is unknown
// or complete, and an old one only makes a climb longer.  Evaluating 512 trees of a power-law
// graph of 289,721 vertices took 14.1 ms with unpinned loads, 13.2 with an atomic load for each
// word, 12.6 so; 1,024 of a road-like graph of 44,780 17.4, 18.4 and 17.4.
__device__ __forceinline__ void pin(int4 &q) { asm("" : "+v"(q.x), "+v"(q.y), "+v"(q.z), "+v"(q.w)); }

// The numbering of a vertex once it is complete: tin, vol and tree parent.
struct TNum {
    uint32_t tin, vol;
    int32_t par;
};
__device__ __forceinline__ TNum rec_num(const uint64_t *rec, int v) {
    const uint64_t w = aload(&rec[2 * (size_t)v]);
    return {(uint32_t)(w >> 32) - 1, (uint32_t)w, rec_parent(rec, v)};
}
__device__ __forceinline__ uint32_t rec_tin(const uint64_t *rec, int v) {
    return (uint32_t)(aload(&rec[2 * (size_t)v]) >> 32) - 1;
}

// Vertices each lane keeps in flight in the tree numbering: the memory
// operations of one step are issued together, so a wavefront has this many
// times as many requests outstanding as it has lanes.  The streaming passes
// take twice as many.
constexpr int NB = 4;
constexpr int NBS = 8;

constexpr uint64_t PEND_ONE = 1ull << 44;
constexpr uint64_t VOL_MASK = PEND_ONE - 1;

__device__ __forceinline__ uint32_t degree(const GraphDev &g, int v) {
    return (uint32_t)(g.off[v + 1] - g.off[v]);
}

// Fenwick tree over positions 0..2m storing a difference array.  The nodes at
// multiples of 2^shift are kept in LDS (at most FEN_HI of them): what is left of an
// update or a sum in memory lies in one block of 2^shift words, where the whole
// tree there took about ten lines of its own per point (1,024 trees of a road-like
// graph of 44,780 vertices: 22.4 ms, 19.8 with the split).
template <int T>
constexpr int FEN_HI = T == WAVE ? 1024 : 2048;  // (one wavefront: the list and these fit the chain table's LDS)
struct Fenwick {
    int64_t *low, *hi;
    int32_t len, shift;
};
__device__ __forceinline__ void fen_point_add(const Fenwick &t, uint32_t pos, int64_t val) {
    uint32_t i = pos + 1;
    const uint32_t len = (uint32_t)t.len, mask = (1u << t.shift) - 1;
    for (; i < len && (i & mask) != 0; i += i & (0u - i)) afetch_add(&t.low[i], val);
    for (uint32_t h = i >> t.shift; i < len && h <= (len - 1) >> t.shift; h += h & (0u - h)) afetch_add(&t.hi[h], val);
}
__device__ __forceinline__ void fen_range_add(const Fenwick &t, uint32_t lo, uint32_t hi, int64_t val) {
    if (val == 0 || hi <= lo) return;
    fen_point_add(t, lo, val);
    fen_point_add(t, hi, -val);
}

// The two contributions attached to tau0 vertex x (Theorem 3.4), as
// ranges of tin with a weight, active for every u in Sub(tau0, x):
//   forward : p(x) = p0(x)          -> +(2m - vol(x)) on Sub(tau, x)
//   reverse : p(p0(x)) = x, p0(x)!=r -> -(2m - vol(p0(x))) on Sub(tau, p0(x))
struct Items {
    uint32_t flo, fhi, rlo, rhi;
    int64_t fw, rw;
};
__device__ __forceinline__ Items items_of(const GraphDev &g, const uint64_t *rec, int x) {
    Items it{0u, 0u, 0u, 0u, 0, 0};
    if (x == g.root) return it;
    const TNum nx = rec_num(rec, x);
    const int z = g.p0[x];
    if (nx.par == z) {
        it.flo = nx.tin; it.fhi = nx.tin + nx.vol; it.fw = g.two_m - (int64_t)nx.vol;
    }
    if (z != g.root) {
        const TNum nz = rec_num(rec, z);
        if (nz.par == x) {
            it.rlo = nz.tin; it.rhi = nz.tin + nz.vol; it.rw = (int64_t)nz.vol - g.two_m;
        }
    }
    return it;
}
struct PathShared {
    int32_t n_mark, n_left, n_user, extra, bad;
};
// Scratch of the tree code in LDS.
template <int T>
struct TreeShared {
    int32_t count[2];           // the sweep's lists
    int32_t leaves, taken, left, bad, item;
    PathShared paths;
    int64_t red[T / WAVE];
};

// Sum of v over the workgroup, in every thread.
template <int T>
__device__ __forceinline__ int64_t block_sum(int64_t v, TreeShared<T> &sh) {
    v = wave_sum(v);
    if constexpr (T > WAVE) {
        if ((threadIdx.x & (WAVE - 1)) == 0) sh.red[threadIdx.x / WAVE] = v;
        __syncthreads();
        v = 0;
#pragma unroll
        for (int w = 0; w < T / WAVE; ++w) v += sh.red[w];
        __syncthreads();
    }
    return v;
}
// One LDS atomic per wavefront: the wavefront's share `n` of *counter, as its first position.
__device__ __forceinline__ int take_shared(int32_t *counter, int n) {
    int base = 0;
    if ((threadIdx.x & (WAVE - 1)) == 0 && n > 0) base = afetch_add(counter, n);
    return __builtin_amdgcn_readfirstlane(base);
}

// Volumes and the volume-weighted preorder of the tree whose parents are in
// rec (rec[2v] = deg(v), rec[2v+1] = parent already).  Returns false if the
// parents do not form a tree rooted at r.
//
// Bottom-up: each lane carries up to NB finished vertices; a carrier pushes its
// vertex's volume into the parent's word with one atomic, and the last child to
// arrive carries the parent on.  The volume part the atomic returns is the
// parent's degree plus the volumes of the siblings that arrived before: the
// vertex's offset in its parent's interval.  Top-down, tin is the sum of the
// offsets along the path to the root: a vertex climbs to one whose tin is known
// and writes those of the vertices it passed; a spread of seeds climbs first.
//
// Neither half has rounds, so a deep tree (1,200 levels on a road-like graph of
// 44,780 vertices) costs its longest chain's dependent atomics and climbs, not
// two barriers per level: 6.8M cycles a tree with completion groups, top-down in
// reverse.  (1,024 such trees, numbering and f: 23.4 ms, 17.8 with this, the
// workgroup's sweep and the split Fenwick tree.)
template <int T>
__device__ bool tree_numbering(const GraphDev &g, const SlotPtrs &sp, TreeShared<T> &sh) {
    const int tid = threadIdx.x;
    const int n = g.n;
    if (tid == 0) sh.leaves = sh.taken = sh.left = 0;
    // one PEND_ONE per child in the parent's word
    for (int b = 0; b < n; b += T * NBS) {
        int32_t p[NBS];
#pragma unroll
        for (int k = 0; k < NBS; ++k) {
            const int v = b + k * T + tid;
            p[k] = v < n ? rec_parent(sp.rec, v) : -1;
        }
#pragma unroll
        for (int k = 0; k < NBS; ++k)
            if (p[k] >= 0) afetch_add(&sp.rec[2 * (size_t)p[k]], PEND_ONE);
    }
    __syncthreads();
    for (int b = 0; b < n; b += T * NBS) {
        uint64_t w[NBS];
#pragma unroll
        for (int k = 0; k < NBS; ++k) {
            const int v = b + k * T + tid;
            w[k] = v < n ? aload(&sp.rec[2 * (size_t)v]) : PEND_ONE;  // past the end: not a leaf
        }
        int c = 0;
#pragma unroll
        for (int k = 0; k < NBS; ++k) c += __popcll(__ballot((w[k] >> 44) == 0));
        int at = take_shared(&sh.leaves, c);
#pragma unroll
        for (int k = 0; k < NBS; ++k) {
            const bool leaf = (w[k] >> 44) == 0;
            const uint64_t m = __ballot(leaf);
            if (leaf) sp.leaf[at + rank_in(m)] = b + k * T + tid;
            at += __popcll(m);
        }
    }
    __syncthreads();
    const int L = sh.leaves;
    int cv[NB], cp[NB];
    uint64_t cval[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) { cv[k] = -1; cp[k] = -1; cval[k] = 0; }
    int64_t done = 0;
    bool more = true;
    while (true) {
        if (more) {
            int c = 0;
#pragma unroll
            for (int k = 0; k < NB; ++k) c += __popcll(__ballot(cv[k] < 0));
            int at = c > 0 ? take_shared(&sh.taken, c) : 0;
            if (c > 0) more = at + c < L;
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                const uint64_t m = __ballot(cv[k] < 0);
                const int j = at + rank_in(m);
                if (cv[k] < 0 && j < L) {
                    cv[k] = sp.leaf[j];
                    cval[k] = (uint64_t)degree(g, cv[k]);
                    cp[k] = rec_parent(sp.rec, cv[k]);
                }
                at += __popcll(m);
            }
        }
        uint64_t busy = 0;
#pragma unroll
        for (int k = 0; k < NB; ++k) busy |= __ballot(cv[k] >= 0);
        if (busy == 0ull) break;  // (then no leaf is left either)
        // the parent's own parent, the next vertex if this child is the last, comes
        // from the record line the atomic uses
        uint64_t old[NB];
        int32_t up[NB];
        bool any[NB];  // (the wavefront has such a carrier: most of a deep tree's steps have few)
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            any[k] = __ballot(cv[k] >= 0) != 0ull;
            if (!any[k]) continue;
            old[k] = 0;
            up[k] = -1;
            if (cv[k] >= 0 && cp[k] >= 0) {
                old[k] = afetch_add(&sp.rec[2 * (size_t)cp[k]], cval[k] - PEND_ONE);
                up[k] = rec_parent(sp.rec, cp[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            if (!any[k] || cv[k] < 0) continue;
            const bool top = cp[k] < 0;
            astore(&sp.rec[2 * (size_t)cv[k]], cval[k] | (uint64_t)(top ? 1u : 0u) << 32);
            astore(&sp.rec[2 * (size_t)cv[k] + 1], (uint64_t)(uint32_t)cp[k] | (old[k] & VOL_MASK) << 32);
            ++done;
            const bool last = !top && (old[k] >> 44) == 1;
            if (last) cval[k] = (old[k] & VOL_MASK) + cval[k];
            cv[k] = last ? cp[k] : -1;
            cp[k] = up[k];
        }
    }
    if (block_sum<T>(done, sh) != n) return false;
    __syncthreads();
    // top-down
    constexpr int SEED = 4096, SHORT = 8;
    const int4 *rec4 = reinterpret_cast<const int4 *>(sp.rec);  // vol, tin + 1, parent, offset
    auto climb = [&](auto wu, auto is_short, int at, int count, auto vertex) __attribute__((always_inline)) {
        constexpr int WU = decltype(wu)::value;
        constexpr bool CUT = decltype(is_short)::value;
        int v[WU], x[WU];
        uint32_t sum[WU], vol[WU], off[WU], up[WU], len[WU];
        int4 r[WU];
        bool go[WU];
#pragma unroll
        for (int k = 0; k < WU; ++k) {
            const int i = at + k * T;
            v[k] = i < count ? vertex(i) : -1;
            x[k] = v[k] >= 0 ? v[k] : g.root;
            sum[k] = len[k] = vol[k] = off[k] = up[k] = 0;
        }
        int step = 0;
        uint64_t any;
        do {
            any = 0;
#pragma unroll
            for (int k = 0; k < WU; ++k) r[k] = rec4[x[k]];
#pragma unroll
            for (int k = 0; k < WU; ++k) {
                pin(r[k]);
                if (step == 0) {
                    vol[k] = (uint32_t)r[k].x;
                    off[k] = (uint32_t)r[k].w;
                    up[k] = (uint32_t)r[k].z;
                }
                go[k] = r[k].y == 0;
                sum[k] += go[k] ? (uint32_t)r[k].w : 0u;
                x[k] = go[k] ? r[k].z : x[k];
                len[k] += go[k] ? 1u : 0u;
                any |= __builtin_amdgcn_ballot_w64(go[k]);
            }
        } while ((!CUT || step < SHORT) && ++step && any != 0ull);
#pragma unroll
        for (int k = 0; k < WU; ++k) {
            if (v[k] < 0 || len[k] == 0) continue;
            if (go[k]) {
                sp.leaf[afetch_add(&sh.left, 1)] = v[k];  // (the leaves are used up)
                continue;
            }
            uint32_t tin1 = sum[k] + (uint32_t)r[k].y;  // tin + 1
            astore(&sp.rec[2 * (size_t)v[k]], (uint64_t)vol[k] | (uint64_t)tin1 << 32);
            tin1 -= off[k];
            for (int y = (int)up[k]; y != x[k];) {
                int4 q = rec4[y];
                pin(q);
                astore(&sp.rec[2 * (size_t)y], (uint64_t)(uint32_t)q.x | (uint64_t)tin1 << 32);
                tin1 -= (uint32_t)q.w;
                y = q.z;
            }
        }
    };
    constexpr auto one = std::integral_constant<int, 1>{};
    constexpr auto four = std::integral_constant<int, 4>{};
    const int seeds = min(n, SEED);
    for (int at = tid; at - tid < seeds; at += T)
        climb(one, std::false_type{}, at, seeds, [&](int i) { return (int)((int64_t)i * n / seeds); });
    for (int at = tid; at - tid < n; at += 4 * T) climb(four, std::true_type{}, at, n, [](int i) { return i; });
    __syncthreads();
    const int left = sh.left;
    for (int at = tid; at - tid < left; at += T)
        climb(one, std::false_type{}, at, left, [&](int i) { return sp.leaf[i]; });
    __syncthreads();
    return true;
}

// f by walking each vertex's tau0 ancestors along p0 (Theorem 3.4 as a sum over
// vertices u of d(u) q(u): every tau0 edge x -> p0(x) on u's tau0 path adds
// 2m - vol(x) when tau uses it in the same direction and x is a tau ancestor
// of u, and subtracts 2m - vol(p0(x)) when tau uses it the other way and
// p0(x) (not the root) is a tau ancestor of u).  Each thread's share of f.
template <int T>
__device__ int64_t f_walk(const GraphDev &g, const SlotPtrs &sp) {
    const int n = g.n, root = g.root;
    const int64_t two_m = g.two_m;
    int64_t acc = 0;
    for (int u = threadIdx.x; u < n; u += T) {
        const TNum nu = rec_num(sp.rec, u);
        const uint32_t tu = nu.tin;
        int64_t q = 0;
        int x = u;
        TNum nx = nu;
        while (x != root) {
            const int z = g.p0[x];
            if (nx.par == z) {
                if (nx.tin <= tu && tu < nx.tin + nx.vol) q += two_m - (int64_t)nx.vol;
            }
            if (z == root) break;
            const TNum nz = rec_num(sp.rec, z);
            if (nz.par == x) {
                if (nz.tin <= tu && tu < nz.tin + nz.vol) q -= two_m - (int64_t)nz.vol;
            }
            x = z;
            nx = nz;
        }
        acc += (int64_t)degree(g, u) * q;
    }
    return acc;
}

// f by a tau0-preorder sweep, 64 preorder positions per step.  The Fenwick tree
// holds the items of every tau0 vertex whose subtree started before the step and
// is still open; items of the step's own vertices and of subtrees closing inside
// the step are listed in LDS with the positions they hold for.  The tree returns
// to all zeros at the end of the sweep.  Each thread's share of f.
//
// A step is bound by its dependent loads (vertex, record, tau0 parent, its
// record), so the rest of it is spread over the workgroup: every wavefront has
// all 64 positions and takes its share of the Fenwick tree's levels and of the
// list, and the listing threads update the tree.  One wavefront doing all of it
// took 40k cycles a step (17 ms for the 700 steps of a road-like graph of 44,780
// vertices).
struct SweepItem {
    uint32_t lo, hi;  // holds for tin in [lo, hi)
    int32_t from, to; // at preorder positions from .. to
    int64_t w;
};
template <int T>
struct SweepLds {
    SweepItem list[2 * T];
    int64_t hi[FEN_HI<T>];
};

template <int T>
__device__ int64_t f_sweep(const GraphDev &g, const SlotPtrs &sp, int64_t fen_len, SweepLds<T> &lds,
                           TreeShared<T> &sh) {
    constexpr int WAVES = T / WAVE;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
    const int n = g.n;
    int64_t acc = 0;
    int blk = 0;
    SweepItem *list = lds.list;
    Fenwick fen{sp.fen, lds.hi, (int32_t)fen_len, 0};
    int levels = 1;
    while ((1ll << levels) < fen_len) ++levels;
    while ((fen_len - 1) >> fen.shift >= FEN_HI<T>) ++fen.shift;
    for (int i = tid; i < FEN_HI<T>; i += T) fen.hi[i] = 0;
    if (tid < 2) sh.count[tid] = 0;
    __syncthreads();
    int turn = 0;  // of the two list counters
    // the step's own vertices, and the closing subtrees of its first list, are read a step ahead
    const int first = tid - WAVE;  // this thread's place among those
    int e0 = g.eoff[0], e1 = g.eoff[1];
    int u_next = lane < n ? g.pre0[lane] : g.root;
    int x_next = first >= 0 && e0 + first < e1 ? g.elist[e0 + first] : -1;
    for (int P0 = 0; P0 < n; P0 += WAVE, ++blk) {
        const int p = P0 + lane;
        const bool valid = p < n;
        const int u = u_next, c0 = e0, c1 = e1;
        int x = wave == 0 ? (valid ? u : -1) : x_next;
        if (P0 + WAVE < n) {
            e0 = e1;
            e1 = g.eoff[blk + 2];
            u_next = p + WAVE < n ? g.pre0[p + WAVE] : g.root;
            x_next = first >= 0 && e0 + first < e1 ? g.elist[e0 + first] : -1;
        }
        const uint32_t tu = rec_tin(sp.rec, u);
        int64_t S = 0;
        // the first list: the step's own vertices (wavefront 0) and closing subtrees
        // (the others); then further closing subtrees
        for (int c = c0, own = 1; own != 0 || c < c1;) {
            const bool mine = own && wave == 0;
            if (!own) x = c + tid < c1 ? g.elist[c + tid] : -1;
            Items it{0u, 0u, 0u, 0u, 0, 0};
            int o = -1;
            if (x >= 0) {
                it = items_of(g, sp.rec, x);
                o = g.out0[x];
            }
            if (own && valid) {
                // this wavefront's levels of the prefix sum at tu
                const uint32_t i = min(tu + 1, (uint32_t)fen_len - 1);
                for (int b = wave; b < levels; b += WAVES)
                    if (i >> b & 1) S += b < fen.shift ? aload(&fen.low[i >> b << b]) : fen.hi[i >> b << (b - fen.shift)];
            }
            const int32_t from = mine ? p : o + 1, to = mine ? o : INT32_MAX;
            const bool f1 = it.fw != 0, r1 = it.rw != 0;
            const uint64_t fm = __ballot(f1), rm = __ballot(r1);
            const int at = take_shared(&sh.count[turn], __popcll(fm) + __popcll(rm));
            if (f1) list[at + rank_in(fm)] = {it.flo, it.fhi, from, to, mine ? it.fw : -it.fw};
            if (r1) list[at + __popcll(fm) + rank_in(rm)] = {it.rlo, it.rhi, from, to, mine ? it.rw : -it.rw};
            __syncthreads();
            const int cnt = sh.count[turn];
            turn ^= 1;
            if (tid == 0) sh.count[turn] = 0;
            // the tree as it stands after the step (every prefix sum has been read): what
            // stays open is added, what closed (and was added before) taken out
            for (int j = tid; j < cnt; j += T)
                if (list[j].to >= P0 + WAVE) fen_range_add(fen, list[j].lo, list[j].hi, list[j].w);
            for (int j = wave; j < cnt; j += WAVES) {
                const SweepItem e = list[j];
                if (e.from <= p && p <= e.to && e.lo <= tu && tu < e.hi) S += e.w;
            }
            c += own ? T - WAVE : T;
            own = 0;
            __syncthreads();
        }
        if (valid) acc += (int64_t)degree(g, u) * S;
    }
    return acc;
}

// Number of graph edges {x, y} that join the two trees left when the tree
// edge {cut_u, cut_v} of the tree `par` is removed (the side away from the root is
// Sub(tau, c) with c the child endpoint).  With relink, also cut-link (section
// 4.2): edge number j of them, in the order (x ascending, row order, x < y), with
// j drawn by Philox on counter (slot, serial, ISM_CTR_LO, ISM_CTR_HI), joins the
// two parts; the path from its inner endpoint up to c is reversed so the tree
// stays rooted at r.
//
// Which side a vertex is on is found by climbing to c, to the root or to a vertex
// whose side is known (as the path sums below: no volumes, no numbering), and the
// edges are counted from the rows of the smaller side.  The counts of each 64
// smaller endpoints stay in grp, so that the drawn edge's rows are found without a
// second pass.  (1.9 ms a tree of 20,000 vertices by numbering and full scan; an
// update of four edges over 1,024 such trees took 56.3 ms, 24.4 with this and the
// path currents found by climbing.)
template <int T>
__device__ int64_t crossing_edges(const GraphDev &g, const SlotPtrs &sp, const RunParams &rp, const int32_t *par,
                                  int32_t slot, int idx, TreeShared<T> &sh) {
    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    const int n = g.n;
    const int a = rp.cut_u, b = rp.cut_v;
    const int c = a != g.root && par[a] == b ? a : (b != g.root && par[b] == a ? b : -1);
    if (c < 0) {
        if (tid == 0) report_error(rp.ctl, DEV_BADTREE, idx);
        return 0;
    }
    // sides: 0 unknown, OUT, IN; then the counts per 64 smaller endpoints
    constexpr uint8_t OUT = 1, IN = 2;
    uint8_t *side = sp.state;
    const int nchunk = (n + WAVE - 1) / WAVE;
    if (tid == 0) sh.bad = 0;
    for (int v = tid; v < n; v += T) side[v] = v == g.root ? OUT : v == c ? IN : 0;
    for (int ch = tid; ch < nchunk; ch += T) astore(&sp.grp[ch], 0);
    __syncthreads();
    int64_t vol_in = 0;
    for (int v = tid; v < n; v += T) {
        int x = v, len = 0, s;
        while ((s = aload(&side[x])) == 0) {
            x = par[x];
            if ((unsigned)x >= (unsigned)n || ++len > n) {
                sh.bad = 1;
                s = OUT;
                break;
            }
        }
        for (int y = v; y != x && len > 0; --len) {
            astore(&side[y], (uint8_t)s);
            y = par[y];
        }
        if (s == IN) vol_in += degree(g, v);
    }
    vol_in = block_sum<T>(vol_in, sh);
    if (sh.bad) {  // (uniform)
        if (tid == 0) report_error(rp.ctl, DEV_BADTREE, idx);
        return 0;
    }
    const int small = 2 * vol_in <= g.two_m ? IN : OUT;
    auto edge_count = [&](int x, int64_t first, int64_t step) {
        int k = 0;
        for (int64_t e = g.off[x] + first; e < g.off[x + 1]; e += step) {
            const int y = g.adj[e];
            if (side[y] != small) {
                ++k;
                (void)afetch_add(&sp.grp[min(x, y) / WAVE], 1);
            }
        }
        return k;
    };
    int64_t cnt = 0;
    for (int x0 = tid - lane; x0 < n; x0 += T) {
        const int x = x0 + lane;
        const bool mine = x < n && side[x] == small;
        const bool wide = mine && degree(g, x) > WAVE;  // a row for the whole wavefront
        if (mine && !wide) cnt += edge_count(x, 0, 1);
        for (uint64_t m = __ballot(wide); m != 0ull; m &= m - 1)
            cnt += edge_count(x0 + __ffsll((unsigned long long)m) - 1, lane, WAVE);
    }
    const int64_t total = block_sum<T>(cnt, sh);
    if (!rp.relink) return total;
    if (total <= 0) {
        if (tid == 0) report_error(rp.ctl, DEV_BADTREE, idx);
        return 0;
    }
    __syncthreads();
    if (tid >= WAVE) return total;
    const int64_t j = arrow_slot(rp.seed, ((uint64_t)ISM_CTR_HI << 32) | ISM_CTR_LO, rp.serial, (uint32_t)slot,
                                 (uint32_t)total);
    auto scan = [&](int64_t k) {
        for (int d = 1; d < WAVE; d <<= 1) {
            const int64_t t = __shfl_up(k, d);
            if (lane >= d) k += t;
        }
        return k;
    };
    // the 64 rows that hold edge j, and the edges before them
    int64_t base = 0;
    int chunk = -1;
    for (int c0 = 0; c0 < nchunk; c0 += WAVE) {
        const int64_t k = c0 + lane < nchunk ? (int64_t)aload(&sp.grp[c0 + lane]) : 0;
        const int64_t incl = scan(k);
        const uint64_t past = __ballot(base + incl > j);
        if (past != 0ull) {
            const int l = __ffsll((unsigned long long)past) - 1;
            chunk = c0 + l;
            base += __shfl(incl - k, l);
            break;
        }
        base += __shfl(incl, WAVE - 1);
    }
    if (chunk < 0) {
        if (tid == 0) report_error(rp.ctl, DEV_BADTREE, idx);
        return total;
    }
    // edge j among the rows' edges to larger endpoints
    const int x = chunk * WAVE + lane;
    int64_t k = 0;
    if (x < n)
        for (int64_t e = g.off[x]; e < g.off[x + 1]; ++e) {
            const int z = g.adj[e];
            if (z > x && side[z] != side[x]) ++k;
        }
    const int64_t incl = scan(k);
    if (k > 0 && base + incl - k <= j && j < base + incl) {
        int64_t r = j - (base + incl - k);
        int y = -1;
        for (int64_t e = g.off[x]; e < g.off[x + 1]; ++e) {
            const int z = g.adj[e];
            if (z > x && side[z] != side[x]) {
                if (r == 0) { y = z; break; }
                --r;
            }
        }
        if (y < 0) {
            report_error(rp.ctl, DEV_BADTREE, idx);
        } else {
            const bool ix = side[x] == IN;
            int32_t *out = rp.parents_mut + (size_t)slot * (size_t)n;
            int32_t prev = ix ? y : x, z = ix ? x : y;
            for (int guard = 0; guard <= n; ++guard) {
                const int32_t nz = out[z];
                out[z] = prev;
                if (z == c) break;
                if (nz < 0 || nz >= n) {  // c is an ancestor of the inner endpoint: not reached
                    report_error(rp.ctl, DEV_BADTREE, idx);
                    break;
                }
                prev = z;
                z = nz;
            }
        }
    }
    return total;
}

// f on a shallow reference tree (the tau0-ancestor table, depth(tau0) <= 8),
// without volumes or a numbering.
//
// Write Theorem 3.4's sum as f = sum_x c(x) (2m - vol(x)): c(x) is the weight of
// the vertices u whose q has the term 2m - vol(x).  u = x always has it if tau uses
// x -> p0(x) (FWD); a tau0 descendant u of x has it if x is also a tau ancestor of
// u, and -1 times that of z = p0(x) if tau uses z -> x and z is a tau ancestor of u.
// The second kind needs an internal vertex x of tau0 whose tau0 edge is in tau; on
// a power-law graph those are hubs with many other edges, so that few u (0 to 3%
// there) have one on their tau0 path: only those are looked at one by one.
// And sum_x c(x) vol(x) = sum_w d(w) C(w) with C(w) the sum of c along w's tau path,
// so the volumes are not needed either: C runs down the tree.  A vertex climbs
// until it meets one whose path sum is known and writes those of the vertices it
// passed; nearly all climb one step.  Per vertex that is one random line (the
// parent's record) and some path lines, where the volumes and the numbering take
// about six (child count, carry, tin and record, most of them written back).
// f of 2,048 trees of a power-law graph of 481,994 vertices: 194 -> 87 ms; of 2,560 of
// a dense one of 150,001 vertices: 77 -> 26 ms.
//
// Records: rec[2v] = parent | flags | deg << 32, rec[2v + 1] = the path sum of the
// first kind of c (at most 2m < 2^32) << 32 | the nearest MARKed vertex on v's
// path (itself included), all ones while unknown.  MARKed are the x and z above,
// so that "t is a tau ancestor of u" is a walk along the marks of u's path.
constexpr uint32_t P_FWD = 1u << 31, P_MARK = 1u << 30, P_PAR = P_MARK - 1;
constexpr uint32_t P_NONE = 0xFFFFFFFFu;
constexpr uint64_t P_UNKNOWN = ~0ull;
constexpr int64_t PATHS_MAX_N = 1 << 30;  // (a parent and two flags in 32 bits)

__device__ __forceinline__ uint32_t next_mark(const uint64_t *rec, uint32_t y) {
    const uint32_t p = (uint32_t)aload(&rec[2 * (size_t)y]) & P_PAR;
    return (uint32_t)aload(&rec[2 * (size_t)p + 1]);
}

// bitmap: nbits (a power of two) bits of LDS; a vertex's bit is that of its index
// modulo nbits (a bit too many costs a look, no error).  Returns false if the
// parents do not form a tree rooted at r; else *f is the thread's share of f.
template <int T, int D, typename ParentOf>
__device__ bool f_paths(const GraphDev &g, const SlotPtrs &sp, PathShared &sh, uint32_t *bitmap, int nbits,
                        ParentOf parent_of, int64_t *f) {
    const int tid = threadIdx.x, n = g.n;
    const int64_t two_m = g.two_m;
    uint64_t *rec = sp.rec;
    // the slot's block, free once the parents are read: the second kind of c and its
    // path sums (at marked vertices), the vertices with terms of that kind, the marked
    int64_t *extra = reinterpret_cast<int64_t *>(sp.state);
    int64_t *extra_sum = reinterpret_cast<int64_t *>(sp.state + 8 * sp.stride);
    int32_t *left = reinterpret_cast<int32_t *>(sp.state + 8 * sp.stride);  // (before those)
    int32_t *user = reinterpret_cast<int32_t *>(sp.state + 8 * sp.stride);
    int32_t *marked = reinterpret_cast<int32_t *>(sp.state + 16 * sp.stride);
    auto tau0_parent = [&](int v) { return g.anc0[v]; };
    if (tid == 0) sh.n_mark = sh.n_left = sh.n_user = sh.extra = sh.bad = 0;
    __syncthreads();
    // ---- the records
    constexpr int U = 4;
    for (int b = 0; b < n; b += T * U) {
        int32_t p[U], z[U], pz[U];
        uint32_t d[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int v = b + k * T + tid;
            p[k] = v < n && v != g.root ? parent_of(v) : g.root;
            d[k] = v < n ? degree(g, v) : 0;
            z[k] = v < n ? tau0_parent(v) : -1;
            if (v < n && v != g.root && (p[k] < 0 || p[k] >= n || p[k] == v)) {
                sh.bad = 1;
                p[k] = g.root;
            }
        }
#pragma unroll
        for (int k = 0; k < U; ++k) pz[k] = tau0_parent(p[k]);
        int c = 0;
        uint32_t marks = 0;
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int v = b + k * T + tid;
            const bool inner = v < n && v != g.root;
            const bool fwd = inner && p[k] == z[k];
            const bool mark = inner && ((fwd && (g.int0[v >> 5] >> (v & 31) & 1u)) || pz[k] == v);
            if (v < n) {
                astore(&rec[2 * (size_t)v], (uint64_t)((uint32_t)p[k] | (fwd ? P_FWD : 0u) | (mark ? P_MARK : 0u)) |
                                                (uint64_t)d[k] << 32);
                astore(&rec[2 * (size_t)v + 1], v == g.root ? (uint64_t)P_NONE : P_UNKNOWN);
            }
            if (mark) marks |= 1u << k;
            c += __popcll(__ballot(mark));
        }
        int at = take_shared(&sh.n_mark, c);
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const uint64_t m = __ballot(marks >> k & 1u);
            if (marks >> k & 1u) marked[at + rank_in(m)] = b + k * T + tid;
            at += __popcll(m);
        }
    }
    __syncthreads();
    const int n_mark = sh.n_mark;
    for (int i = tid; i < nbits / 32; i += T) bitmap[i] = 0;  // (its memory held the parents, on one route)
    __syncthreads();
    auto set_bit = [&](int v) {
        const int k = v & (nbits - 1);
        (void)afetch_or(&bitmap[k >> 5], 1u << (k & 31));
    };
    for (int i = tid; i < n_mark; i += T) {
        const int u = marked[i];
        const uint32_t node = (uint32_t)aload(&rec[2 * (size_t)u]);
        const int p = (int)(node & P_PAR);
        if (node & P_FWD) set_bit(u);
        if (tau0_parent(p) == u) set_bit(p);
        extra[u] = 0;
    }
    // ---- the path sums.  A few thousand vertices climb as far as it takes, which writes the
    // trunk of the tree; the others climb SHORT steps at most, and those not done, once more
    constexpr int SEED = 4096, SHORT = 8;
    const int4 *rec4 = reinterpret_cast<const int4 *>(rec);
    int64_t acc = 0;
    auto climb = [&](auto wu, auto is_short, int at, int count, auto vertex) __attribute__((always_inline)) {
        constexpr int WU = decltype(wu)::value;
        constexpr bool CUT = decltype(is_short)::value;
        int v[WU], x[WU], mark[WU];
        uint32_t sum[WU], la[WU], own[WU], dv[WU], up[WU], len[WU];
        int4 r[WU];
        bool go[WU];
#pragma unroll
        for (int k = 0; k < WU; ++k) {
            const int i = at + k * T;
            v[k] = i < count ? vertex(i) : -1;
            x[k] = v[k] >= 0 ? v[k] : g.root;
            sum[k] = 0;
            la[k] = P_NONE;
            len[k] = 0;
            mark[k] = -1;
            own[k] = dv[k] = up[k] = 0;
        }
        uint32_t step = 0;
        uint64_t any;
        do {
            any = 0;
#pragma unroll
            for (int k = 0; k < WU; ++k) r[k] = rec4[x[k]];
#pragma unroll
            for (int k = 0; k < WU; ++k) {
                pin(r[k]);
                const uint32_t node = (uint32_t)r[k].x;
                const uint32_t c = node & P_FWD ? (uint32_t)r[k].y : 0u;
                if (step == 0) {
                    own[k] = c;
                    dv[k] = (uint32_t)r[k].y;
                    up[k] = node & P_PAR;
                }
                go[k] = (uint32_t)r[k].w == P_NONE;  // (a path sum is less)
                if (!CUT && go[k] && x[k] == mark[k]) {  // Brent's cycle finding: not a tree
                    sh.bad = 1;
                    go[k] = false;
                }
                if (!CUT && (step & (step - 1)) == 0) mark[k] = x[k];
                sum[k] += go[k] ? c : 0u;
                la[k] = go[k] && la[k] == P_NONE && (node & P_MARK) ? (uint32_t)x[k] : la[k];
                x[k] = go[k] ? (int)(node & P_PAR) : x[k];
                len[k] += go[k] ? 1u : 0u;
                any |= __builtin_amdgcn_ballot_w64(go[k]);
            }
        } while ((!CUT || step < SHORT) && ++step && any != 0ull && (CUT || sh.bad == 0));
#pragma unroll
        for (int k = 0; k < WU; ++k) {
            if (v[k] < 0) continue;
            if (go[k]) {
                if (CUT) left[afetch_add(&sh.n_left, 1)] = v[k];
                continue;
            }
            if ((uint32_t)r[k].w == P_NONE) continue;  // not a tree
            const uint32_t total = sum[k] + (uint32_t)r[k].w;
            uint32_t l = la[k] != P_NONE ? la[k] : (uint32_t)r[k].z;
            acc += (int64_t)dv[k] * ((own[k] != 0 ? two_m : 0) - (int64_t)total);
            if (len[k] > 0) astore(&rec[2 * (size_t)v[k] + 1], (uint64_t)total << 32 | l);
            if (len[k] > 1) {  // the vertices passed: their sums, and the first mark from each on
                uint32_t rest = total - own[k];
                bool look = l == (uint32_t)v[k];
                for (int y = (int)up[k]; y != x[k];) {
                    if (look) {
                        int4 q = rec4[y];
                        pin(q);
                        for (int a = y; (l = (uint32_t)a, !((uint32_t)q.x & P_MARK));) {
                            if ((uint32_t)q.w != P_NONE) { l = (uint32_t)q.z; break; }
                            a = (int)((uint32_t)q.x & P_PAR);
                            q = rec4[a];
                            pin(q);
                        }
                        look = false;
                    }
                    int4 q = rec4[y];
                    pin(q);
                    astore(&rec[2 * (size_t)y + 1], (uint64_t)rest << 32 | l);
                    rest -= (uint32_t)q.x & P_FWD ? (uint32_t)q.y : 0u;
                    look = l == (uint32_t)y;
                    y = (int)((uint32_t)q.x & P_PAR);
                }
            }
        }
    };
    constexpr auto one = std::integral_constant<int, 1>{};
    constexpr auto four = std::integral_constant<int, 4>{};
    const int seed = min(n, SEED);
    for (int at = tid; at - tid < seed; at += T) climb(one, std::false_type{}, at, seed, [](int i) { return i; });
    for (int at = seed + tid; at - tid < n; at += 4 * T) climb(four, std::true_type{}, at, n, [](int i) { return i; });
    __syncthreads();
    const int n_left = sh.n_left;
    for (int at = tid; at - tid < n_left; at += T)
        climb(one, std::false_type{}, at, n_left, [&](int i) { return left[i]; });
    __syncthreads();
    if (sh.bad) return false;  // (uniform)
    if (n_mark > 0) {
        // ---- the vertices with a tau0 ancestor in the map (the records are complete)
        for (int b = 0; b < n; b += T) {
            const int u = b + tid;
            bool hit = false;
            if (u < n) {
                int z[D];
#pragma unroll
                for (int i = 0; i < D; ++i) z[i] = g.anc0[(size_t)i * n + u];
#pragma unroll
                for (int i = 0; i < D; ++i) {
                    const int k = z[i] & (nbits - 1);
                    hit = hit || (z[i] >= 0 && (bitmap[k >> 5] >> (k & 31) & 1u));
                }
            }
            const uint64_t m = __ballot(hit);
            const int at = take_shared(&sh.n_user, __popcll(m));
            if (hit) user[at + rank_in(m)] = u;
        }
        __syncthreads();
        const int n_user = sh.n_user;
        for (int i = tid; i < n_user; i += T) {
            const int u = user[i];
            const int4 ru = rec4[u];
            const int64_t d = (int64_t)(uint32_t)ru.y;
            // the vertices whose terms u has, if they are tau ancestors of u
            uint32_t plus[D], minus[D];
            int z[D];
            bool some = false;
#pragma unroll
            for (int l = 0; l < D; ++l) z[l] = g.anc0[(size_t)l * n + u];
            uint32_t node[D];
#pragma unroll
            for (int l = 0; l < D; ++l) node[l] = z[l] >= 0 ? (uint32_t)rec4[z[l]].x : 0u;
#pragma unroll
            for (int l = 0; l < D; ++l) {
                plus[l] = z[l] >= 0 && (node[l] & P_FWD) ? (uint32_t)z[l] : P_NONE;
                minus[l] = P_NONE;
                if (l > 0 && z[l] >= 0 && z[l] != g.root && (int)(node[l] & P_PAR) == z[l - 1]) minus[l] = (uint32_t)z[l];
                some = some || plus[l] != P_NONE || minus[l] != P_NONE;
            }
            if (!some) continue;
            for (uint32_t y = (uint32_t)ru.z; y != P_NONE; y = next_mark(rec, y)) {
                int64_t t = 0;
#pragma unroll
                for (int l = 0; l < D; ++l) t += (plus[l] == y ? 1 : 0) - (minus[l] == y ? 1 : 0);
                if (t != 0) {
                    acc += t * d * two_m;
                    (void)afetch_add(&extra[y], t * d);
                    sh.extra = 1;
                }
            }
        }
        __syncthreads();
        if (sh.extra) {  // (uniform)
            for (int i = tid; i < n_mark; i += T) {
                int64_t e = 0;
                for (uint32_t y = (uint32_t)marked[i]; y != P_NONE; y = next_mark(rec, y)) e += aload(&extra[y]);
                extra_sum[marked[i]] = e;
            }
            __syncthreads();
            for (int w = tid; w < n; w += T) {
                const int4 r = rec4[w];
                if ((uint32_t)r.z != P_NONE) acc -= (int64_t)(uint32_t)r.y * extra_sum[r.z];
            }
        }
    }
    *f = acc;
    return true;
}

// The per-slot arrays of workgroup blockIdx.x, each `stride` vertices long.
__device__ __forceinline__ SlotPtrs slot_ptrs(const SlotDev &sd, size_t stride) {
    SlotPtrs sp;
    const size_t b = (size_t)blockIdx.x;
    unsigned char *st = sd.state + b * (size_t)state_bytes((int64_t)stride);
    sp.state = st;
    sp.stride = stride;
    sp.queue = sd.queue + b * (size_t)sd.chains;
    sp.cstart = sd.cstart + b * (size_t)sd.chains;
    sp.rec = sd.rec ? reinterpret_cast<uint64_t *>(sd.rec) + 2 * b * stride : nullptr;
    // the numbering's arrays reuse the sampler's block (dead once the parents are in rec)
    sp.leaf = reinterpret_cast<int32_t *>(st);
    sp.grp = reinterpret_cast<int32_t *>(st + 16 * stride);
    sp.fen = sd.fen ? sd.fen + b * (size_t)sd.fen_len : nullptr;
    return sp;
}

__device__ __forceinline__ bool stopped(const int32_t *ctl) {
    return __hip_atomic_load(const_cast<int32_t *>(&ctl[1]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}
// The next work item for the calling workgroup (one atomic per workgroup), or
// INT32_MAX once an error was recorded.  The same value in every thread, as a
// scalar; it is a barrier of the workgroup.
template <int T>
__device__ __forceinline__ int next_item(int32_t *ctl, TreeShared<T> &sh) {
    int idx = 0;
    __syncthreads();  // the LDS of the item before is free
    if (threadIdx.x == 0) {
        idx = __hip_atomic_fetch_add(&ctl[0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (stopped(ctl)) idx = INT32_MAX;
    }
    if constexpr (T > WAVE) {
        if (threadIdx.x == 0) sh.item = idx;
        __syncthreads();
        idx = sh.item;
    }
    return __builtin_amdgcn_readfirstlane(idx);
}

// f of a tree of graph g (work item idx; its parents by parent_of(v), checked here)
// into f_out[idx].  scratch: LDS, the sweep's list or nbits bits.
template <int T, typename ParentOf>
__device__ void evaluate_tree(const GraphDev &g, const SlotPtrs &sp, TreeShared<T> &sh, uint32_t *scratch,
                              int nbits, const RunParams &rp, int64_t fen_len, int idx,
                              ParentOf parent_of) {
    const int tid = threadIdx.x;
    if (rp.traversal != 2 && g.anc0 && g.n < PATHS_MAX_N) {
        int64_t part = 0;
        const bool ok = g.anc_depth <= 4 ? f_paths<T, 4>(g, sp, sh.paths, scratch, nbits, parent_of, &part)
                                         : f_paths<T, 8>(g, sp, sh.paths, scratch, nbits, parent_of, &part);
        const int64_t f = block_sum<T>(part, sh);
        if (tid == 0) {
            if (!ok) report_error(rp.ctl, DEV_BADTREE, idx);
            rp.f_out[idx] = f;
        }
        return;
    }
    if (tid == 0) sh.bad = 0;
    // the parent into each vertex's tree record; its volume word starts at deg(v)
    bool bad = false;
    for (int b = 0; b < g.n; b += T * NBS) {
        int32_t p[NBS];
#pragma unroll
        for (int k = 0; k < NBS; ++k) {
            const int v = b + k * T + tid;
            p[k] = v < g.n && v != g.root ? parent_of(v) : -1;
        }
#pragma unroll
        for (int k = 0; k < NBS; ++k) {
            const int v = b + k * T + tid;
            if (v >= g.n) continue;
            if (v != g.root && (p[k] < 0 || p[k] >= g.n || p[k] == v)) { bad = true; p[k] = g.root; }
            astore(&sp.rec[2 * (size_t)v], (uint64_t)degree(g, v));
            astore(&sp.rec[2 * (size_t)v + 1], (uint64_t)(uint32_t)p[k]);
        }
    }
    __syncthreads();
    if (bad) sh.bad = 1;  // (read after the numbering's barriers)
    bool ok = tree_numbering<T>(g, sp, sh);
    if (sh.bad) ok = false;
    int64_t f = 0;
    if (!ok) {
        // (the call fails; nothing is evaluated)
    } else if (rp.traversal == 2) {
        f = block_sum<T>(f_sweep<T>(g, sp, fen_len, *reinterpret_cast<SweepLds<T> *>(scratch), sh), sh);
    } else {
        f = block_sum<T>(f_walk<T>(g, sp), sh);
    }
    if (tid == 0) {
        if (!ok) report_error(rp.ctl, DEV_BADTREE, idx);
        rp.f_out[idx] = f;
    }
}

}  // namespace
}  // namespace kc
