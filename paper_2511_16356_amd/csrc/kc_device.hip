// kc_device.hip -- the chain sampler, and the kernels around the samplers: edge
// updates of resident trees, exact sums, fills and counters.
//
// Uniform spanning trees by Wilson's algorithm (paper section 2.2 and Algorithm
// 1), organised as cooperative cycle popping.  The k-th draw at vertex v of
// sample s always uses the same Philox4x32-10 arrow, so the tree and the
// per-vertex draw counts are the unique cycle-popping outcome of those arrow
// stacks, whatever order the pops happen in.  Two samplers find it:
//
//   the frontier sampler (kc_frontier.hip), one workgroup per sample, for graphs
//   whose words fit LDS and for larger ones with short walks;
//   the chain sampler (here), one wavefront per sample, for large graphs with long
//   walks, and for calls with many samples of a graph that leaves few workgroups of
//   the other in flight: up to 64 lanes drive loop-erased walks ("chains") of the
//   same sample at once; a chain whose arrow lands on another chain's path is parked
//   in an LDS table and its lane moves on.
//
// Which one a call takes is kc_host::route_of.
//
// Every kernel takes sample after sample from a counter and evaluates f of each
// tree where it was sampled (kc_tree.h); sum f and sum f^2 are exact, in 128-bit
// integers.
//
// Cross-lane communication through global memory uses workgroup-scope
// relaxed atomics (L2-coherent on gfx950) ordered by workgroup fences; every
// lane of a sample of the chain sampler is in the same wavefront.

#include <algorithm>

#include "kc_tree.h"

namespace kc {
namespace {

// ------------------------------------------------------------ sampler state

// Two 8-byte words per (sample, vertex), in two arrays, so that the claim
// (an atomic on the tag word) and the read of the arrow word go to different
// cache lines and overlap:
//   tag word   low half: bits 0..30 tag (0 = arrow not revealed ("free"),
//              1 = in the tree from the start, 2 + c + CH g = on the path of
//              chain c in its generation g); bit 31 need (the vertex's turn as
//              a walk start passed while it was on a path)
//              high half: 1 + the first of the chains parked on this vertex
//              (their head's arrow points here), 0 if none; the list continues
//              through the chain table's wnext links
//   arrow word low half: the current arrow target (the tree parent at the
//              end); high half: how many arrows the vertex has drawn
// A free vertex's tag word is 0; a start vertex's is T_TREE.  A path that
// reaches the tree joins it as a whole: its chain records the generation as
// finished (fin in LDS), and every vertex tagged with a finished generation is
// a tree vertex from then on, with no write to its tag word.  Every change of
// a tag word is one atomic operation, so claims, parks, need marks and erases
// of the same round may meet on a vertex in any order.
constexpr uint32_t T_FREE = 0, T_TREE = 1, T_CHAIN0 = 2;

__device__ __forceinline__ uint32_t *tag_high(uint64_t *w) { return reinterpret_cast<uint32_t *>(w) + 1; }
__device__ __forceinline__ uint64_t arrow_of(int32_t nxt, uint32_t drw) {
    return (uint64_t)(uint32_t)nxt | ((uint64_t)drw << 32);
}
constexpr uint32_t TW_TAG = (1u << 31) - 1;
constexpr uint32_t TW_NEED = 1u << 31;
constexpr int GEN_MAX = 32767;  // generations of one chain id (fin is int16)

// A chain is a loop-erased path of revealed arrows owned by one walk: from
// its start vertex to its head.  A lane drives at most one chain at a time.
// When the head's arrow lands on another chain's path, the chain is parked
// (it joins the vertex's waiter list) and the lane takes other work; the chain is
// woken when that vertex is popped (resume there), and joins the tree with
// the chain it waits on.  A start vertex that already lies on a path is skipped with its
// need bit set; if it is popped later its eraser queues it for a restart.
// Popped vertices are also offered as optional extra starts (a small LIFO):
// revealing any free vertex is work the cycle-popping order fixes anyway.
// Chain-table sizes the kernel is built for (chains per sample).  More chains
// let more walks proceed at once in one sample (fewer rounds per sample);
// fewer chains let more samples share a CU (more samples in flight).
#define KC_CHAIN_VARIANTS(X) X(1024) X(2048)
constexpr int MAX_CHAINS = 2048;
constexpr int HINTS = 128; // optional restart hints

enum : int { CS_FREE = 0, CS_ACTIVE = 1, CS_PARKED = 2, CS_QUEUED = 3, CS_DONE = 4 };
enum : int { T_RESUME = 0, T_POP = 2 };

// Lane modes.  Each issues exactly one round of memory operations per sampler
// round, and all lanes' operations are in flight together.
enum : int {
    M_IDLE = 0,    // no work
    M_LOOK = 1,    // look at `tgt` and claim it if free (first publishing the head's
                   // new arrow if one was drawn)
    M_PARK = 2,    // join the waiter list of `tgt` if its tag word is still `seen`
    M_NEED = 3,    // set the need bit of start vertex `tgt` if its tag word is still `seen`
    M_ADJ = 4,     // the drawn neighbour lies beyond the inline ones: fetch it
    M_ERASE0 = 5,  // popping: load the kept vertex `tgt` (the new head)
    M_ERASE = 6,   // popping: free `tgt`, follow next until `stopv`
    M_FETCH = 7    // lean looks: load the arrow word and graph record of the head just claimed
};

template <int CH>
struct SamplerShared {
    int32_t block[CH];   // parked: vertex the head's arrow points at
    int16_t up[CH];      // parked: chain owning `block`
    int16_t wnext[CH];   // parked: next / previous chain parked on the same vertex (-1: none)
    int16_t wprev[CH];
    int8_t state[CH];    // CS_*
    int16_t fin[CH];     // last generation of the chain id whose path joined the tree (-1: none);
                         // the id's current generation is fin + 1
    int16_t ring[CH];    // free chain ids, taken first in, first out (so generations grow evenly)
    int32_t hint[HINTS];
};

struct SamplerWS {
    uint64_t *tagw;
    uint64_t *arrow;
    int32_t *rq;   // restart ring (n entries)
    int4 *queue;   // ready tasks (CH entries): {chain, kind, e, stop}
    int32_t *start; // chain start vertices (CH entries)
};

// Cooperative cycle popping of one sample by one wavefront.
//
// Every chain runs Wilson's loop-erased walk with loops popped explicitly
// (each vertex of a popped cycle becomes free and draws its next arrow when
// revisited).  Parked chains form a wait-for forest (chain -> owner of the
// vertex it points at); when a park closes a cycle in it, that is a cycle of
// current arrows spanning several chains, and it is popped as a whole.  Only
// genuine cycles of current arrows are ever popped, so the result is the
// cycle-popping outcome of the arrow stacks: independent of timing, of
// `walkers`, of the chain table and of which free vertices are started.
//
// A round: idle lanes take work; every busy lane issues its memory operations
// (one dependent round trip); the results are applied (draws from the head's
// inline neighbours, wakes, pushes); chains that reached the tree finish, with
// the parked chains that wait on them; newly parked chains are checked for a
// cycle of the wait-for forest, all in lockstep.
//
// Returns the total number of draws, or -1 (error recorded in ctl).
template <int CH, bool LEAN>
__device__ int64_t sample_tree(const GraphDev &g, const SamplerWS &ws, SamplerShared<CH> &sh,
                               uint64_t seed, uint64_t s, int walkers, int64_t iter_cap,
                               int32_t *ctl, int idx, int64_t *iters_used, int32_t root_u,
                               int32_t root_v) {
    const int lane = threadIdx.x;
    const int n = g.n, root = g.root;
    const bool two_roots = root_u >= 0;  // start from {u, v} instead of {root}
    uint64_t *__restrict__ tagw = ws.tagw;
    uint64_t *__restrict__ arw = ws.arrow;
    for (int v = lane; v < n; v += WAVE) {
        const bool in_tree = two_roots ? (v == root_u || v == root_v) : v == root;
        astore(&tagw[v], (uint64_t)(in_tree ? T_TREE : T_FREE));
        astore(&arw[v], arrow_of(-1, 0));
    }
    for (int c = lane; c < CH; c += WAVE) {
        sh.state[c] = CS_FREE;
        sh.fin[c] = -1;
        sh.ring[c] = (int16_t)c;
    }
    fence_wg();
    __syncthreads();

    const bool worker = lane < walkers;
    int mode = M_IDLE, chain = -1, cur = -1, tgt = -1, stopv = -1;
    uint32_t ctag = 0, dcur = 0;
    bool haspath = false;  // M_LOOK: the chain has a path (not a fresh start)
    bool pend = false;     // M_LOOK: publish arrow (cur -> tgt, dcur) first
    uint64_t seen = 0;     // M_PARK / M_NEED: expected tag word
    int adjpos = 0;        // M_ADJ: CSR position of the drawn neighbour
    // graph record of the head `cur`: CSR offset, degree, first neighbours (plain scalars,
    // so that the record stays in registers)
    int hoff = 0, hdeg = 0, hn0 = -1, hn1 = -1, hn2 = -1, hn3 = -1, hn4 = -1, hn5 = -1;
    // wave-uniform bookkeeping
    int next_start = 0, q_head = 0, q_tail = 0, f_head = 0, f_tail = CH, parked = 0, hint_top = 0;
    int64_t rq_head = 0, rq_tail = 0;
    int64_t iters = 0, mysteps = 0;
    int err = 0;

    // tag of chain c's path in its current generation
    auto tag_of = [&](int c) __attribute__((always_inline)) {
        return T_CHAIN0 + (uint32_t)c + (uint32_t)CH * (uint32_t)(sh.fin[c] + 1);
    };
    // a tree vertex: a start vertex, or on a path whose generation has joined the tree
    auto in_tree = [&](uint32_t t) __attribute__((always_inline)) {
        if (t < T_CHAIN0) return t == T_TREE;
        const uint32_t x = t - T_CHAIN0;
        return (int)(x / (uint32_t)CH) <= (int)sh.fin[x % (uint32_t)CH];
    };

    // the head `cur` (its graph record in registers, dcur draws so far) draws its next arrow;
    // called once per round for the lanes that set `drawing`
    auto draw = [&]() __attribute__((always_inline)) {
        const uint32_t deg = (uint32_t)hdeg;
        const uint32_t j = arrow_slot(seed, s, (uint32_t)cur, dcur, deg);
        mysteps++;
        dcur += 1;
        haspath = true;
        if (j < (uint32_t)VREC_INLINE) {
            // select in registers: pairs first, then the pair (an indexed read of the
            // record would place it in scratch memory)
            const bool odd = (j & 1u) != 0u;
            int p01 = odd ? hn1 : hn0;
            int p23 = odd ? hn3 : hn2;
            int p45 = odd ? hn5 : hn4;
            asm volatile("" : "+v"(p01), "+v"(p23), "+v"(p45));
            tgt = j < 2u ? p01 : (j < 4u ? p23 : p45);
            pend = true;
            mode = M_LOOK;
        } else {
            adjpos = hoff + (int)j;
            mode = M_ADJ;
        }
    };

    while (true) {
        // ---- phase 0: idle lanes take tasks, restarts, fresh starts, then hints
        {
            const uint64_t idle = __ballot(worker && mode == M_IDLE);
            const int nidle = __popcll(idle);
            const int take_q = min(nidle, q_tail - q_head);
            int left = nidle - take_q, room = f_tail - f_head;
            const int take_r = (int)min((int64_t)min(left, room), rq_tail - rq_head);
            left -= take_r; room -= take_r;
            const int take_s = min(min(left, room), n - next_start);
            left -= take_s; room -= take_s;
            const int take_h = min(min(left, room), hint_top);
            if (worker && mode == M_IDLE) {
                const int r = rank_in(idle);
                const int k = r - take_q;
                pend = false;
                // a lane that takes work reads all four sources at clamped, always
                // valid indices and keeps the one it needs, so its loads and those of
                // the other lanes are in flight together; lanes that take nothing
                // read nothing (a round with nothing to take has no load here)
                int4 t = make_int4(0, 0, 0, 0);
                int32_t t_rq = 0, t_ord = 0, t_hint = 0;
                if (r < take_q + take_r + take_s + take_h) {
                    t = ws.queue[(q_head + max(0, min(r, take_q - 1))) & (CH - 1)];
                    t_rq = aload(&ws.rq[(rq_head + max(0, min(k, take_r - 1))) % n]);
                    t_ord = aload(&g.order[max(0, min(next_start + k - take_r, n - 1))]);
                    t_hint = sh.hint[max(0, min(hint_top - 1 - (k - take_r - take_s), HINTS - 1))];
                }
                if (r < take_q) {
                    chain = t.x;
                    ctag = tag_of(chain);
                    if (t.y == T_RESUME) {
                        tgt = t.z;
                        haspath = true;
                        mode = M_LOOK;
                    } else {
                        tgt = t.z;
                        stopv = t.w;
                        mode = M_ERASE0;
                    }
                } else if (k < take_r + take_s + take_h) {
                    chain = sh.ring[(f_head + k) & (CH - 1)];
                    ctag = tag_of(chain);
                    tgt = k < take_r ? t_rq : (k < take_r + take_s ? t_ord : t_hint);
                    astore(&ws.start[chain], tgt);
                    haspath = false;
                    mode = M_LOOK;
                }
                if (mode != M_IDLE) sh.state[chain] = CS_ACTIVE;
            }
            q_head += take_q;
            rq_head += take_r;
            next_start += take_s;
            hint_top -= take_h;
            f_head += take_r + take_s + take_h;
        }
        if (__ballot(mode != M_IDLE) == 0ull) {
            if (next_start < n || q_tail != q_head || parked != 0 || rq_tail != rq_head)
                err = DEV_PROTOCOL;
            break;
        }
        if (++iters > iter_cap) err = DEV_LIMIT;
        if (err == 0 && mode != M_IDLE && mode != M_ADJ && (unsigned)tgt >= (unsigned)n)
            err = DEV_PROTOCOL;
        if (err == 0 && mode == M_ADJ && (unsigned)adjpos >= (unsigned)g.two_m) err = DEV_PROTOCOL;
        const int m0 = err == 0 ? mode : M_IDLE;

        // ---- memory: every lane issues its operations before any result is used
        const bool do_cas = m0 == M_LOOK || m0 == M_PARK || m0 == M_NEED;
        const bool do_xchg = m0 == M_ERASE;
        // a lean look at a walk's next vertex is the claim alone: most such looks
        // meet the tree, and a claimed vertex's arrow word and record are fetched
        // in the next round (M_FETCH)
        // (LEAN: a compile-time choice, so that a kernel without lean looks carries none of it)
        const bool thin = LEAN && m0 == M_LOOK && haspath;
        const bool fetch = LEAN && m0 == M_FETCH;
        const bool do_arrow = (m0 == M_LOOK && !thin) || m0 == M_ERASE0 || fetch || do_xchg;
        const bool do_rec = (m0 == M_LOOK && !thin) || m0 == M_ERASE0 || fetch;
        if (m0 == M_LOOK && pend) astore(&arw[cur], arrow_of(tgt, dcur));
        int4 r0 = make_int4(0, 0, 0, 0), r1 = make_int4(0, 0, 0, 0);
        const int rv = fetch ? cur : tgt;  // the vertex whose words are read
        if (do_rec) {
            r0 = g.vrec[2 * (size_t)rv];
            r1 = g.vrec[2 * (size_t)rv + 1];
        }
        // (each operation returns into a register of its own: a shared one would make
        // every later issue wait for the earlier operations' results)
        uint64_t o_cas = 0, o_xchg = 0, o_tag = 0;
        if (do_cas) {
            const uint64_t expect = m0 == M_LOOK ? (uint64_t)T_FREE : seen;
            const uint64_t want = m0 == M_LOOK ? (uint64_t)ctag
                                : m0 == M_PARK ? ((seen & 0xffffffffull) | ((uint64_t)(chain + 1) << 32))
                                               : (seen | TW_NEED);
            o_cas = acas(&tagw[tgt], expect, want);
        }
        if (do_xchg)
            o_xchg = __hip_atomic_exchange(&tagw[tgt], (uint64_t)T_FREE, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
        if (m0 == M_ERASE0) o_tag = aload(&tagw[tgt]);
        uint64_t ar = 0;
        if (do_arrow) ar = aload(&arw[rv]);
        auto take_record = [&]() __attribute__((always_inline)) {
            hoff = r0.x; hdeg = r0.y; hn0 = r0.z; hn1 = r0.w;
            hn2 = r1.x; hn3 = r1.y; hn4 = r1.z; hn5 = r1.w;
        };
        int32_t y = -1;
        if (m0 == M_ADJ) y = g.adj[adjpos];
        const uint64_t o64 = do_cas ? o_cas : (do_xchg ? o_xchg : o_tag);

        // ---- apply the results
        bool retire = false, park = false, drawing = false, finish = false;
        int park_head = -1;
        int wake_kind = -1, wake_vtx = -1, wake_head = -1, restart_vtx = -1, hint_vtx = -1;
        const uint32_t old = (uint32_t)o64;
        const uint32_t tg = old & TW_TAG;
        const int32_t nt = (int32_t)(uint32_t)ar;
        const uint32_t dt = (uint32_t)(ar >> 32);
        if (m0 == M_LOOK) {
            const bool drew = pend;  // the arrow into tgt was just published
            pend = false;
            if (old == T_FREE) {
                // claimed: the new head draws at once (after a lean look, next round)
                cur = tgt;
                if (thin) {
                    mode = M_FETCH;
                } else {
                    dcur = dt;
                    take_record();
                    drawing = true;
                }
            } else if (tg == ctag) {
                // own path: the new arrow closed a loop at tgt; pop it, keep tgt as head
                if (!drew) err = DEV_PROTOCOL;
                stopv = tgt;
                if (thin) {
                    mode = M_ERASE0;  // reads tgt's words, then erases from its arrow on
                } else {
                    cur = tgt;
                    dcur = dt;
                    take_record();
                    tgt = nt;
                    mode = M_ERASE;
                }
            } else if (in_tree(tg)) {
                if (haspath) finish = true;  // the path reaches the tree and joins it
                else retire = true;          // a fresh chain whose start is already in the tree
            } else if (tg >= T_CHAIN0) {
                seen = o64;
                mode = haspath ? M_PARK : M_NEED;
            } else {
                err = DEV_PROTOCOL;
            }
        } else if (m0 == M_PARK || m0 == M_NEED) {
            if (o64 == seen) {
                if (m0 == M_PARK) {
                    park = true;  // joined the list; recorded below
                    park_head = (int)(seen >> 32) - 1;
                } else {
                    retire = true;  // need mark set: the fresh chain has nothing to retrace
                }
            } else if (o64 == (uint64_t)T_FREE) {
                mode = M_LOOK;  // popped meanwhile: look again
            } else if (in_tree(tg)) {
                if (m0 == M_PARK) finish = true;
                else retire = true;
            } else if (tg >= T_CHAIN0 && tg != ctag) {
                seen = o64;  // another park or a new owner: try again
            } else {
                err = DEV_PROTOCOL;
            }
        } else if (m0 == M_ADJ) {
            tgt = y;
            pend = true;
            mode = M_LOOK;
        } else if (m0 == M_ERASE) {
            if (tg != ctag) err = DEV_PROTOCOL;
            wake_head = (int)(o64 >> 32) - 1;
            if (wake_head >= 0) { wake_kind = T_RESUME; wake_vtx = tgt; }
            if (old & TW_NEED) restart_vtx = tgt;
            else hint_vtx = tgt;
            if (nt == stopv) drawing = true; else tgt = nt;
        } else if (m0 == M_ERASE0) {
            if (tg != ctag) err = DEV_PROTOCOL;
            cur = tgt;
            dcur = dt;
            take_record();
            if (nt == stopv) drawing = true;
            else { mode = M_ERASE; tgt = nt; }
        } else if (fetch) {
            dcur = dt;
            take_record();
            drawing = true;
        }
        if (drawing) draw();
        // paths that reached the tree join it: their generation is finished
        auto finish_chain = [&](int c) __attribute__((always_inline)) {
            if ((int)sh.fin[c] + 1 > GEN_MAX) err = DEV_LIMIT;
            sh.fin[c] = (int16_t)(sh.fin[c] + 1);
            sh.state[c] = CS_DONE;
        };
        if (finish) finish_chain(chain);
        __syncthreads();
        // a new park on a path that has joined the tree (in this round, or since its
        // owner was looked at) joins the tree with it instead
        if (park && in_tree(tg)) {
            park = false;
            finish = true;
            finish_chain(chain);
        }
        // new parks join their vertex's list before any wake walks a list
        if (park) {
            int h = park_head;
            if ((unsigned)(h + 1) > (unsigned)CH) { err = DEV_PROTOCOL; h = -1; }
            sh.wnext[chain] = (int16_t)h;
            sh.wprev[chain] = -1;
            if (h >= 0) sh.wprev[h] = (int16_t)chain;
            sh.block[chain] = tgt;
            sh.up[chain] = (int16_t)((tg - T_CHAIN0) % (uint32_t)CH);
            sh.state[chain] = CS_PARKED;
        }
        // popped vertices: need-restarts to the restart ring, the rest offered as hints
        {
            const uint64_t qm = __ballot(restart_vtx >= 0);
            if (restart_vtx >= 0) astore(&ws.rq[(rq_tail + rank_in(qm)) % n], (int32_t)restart_vtx);
            rq_tail += __popcll(qm);
            const uint64_t hm = __ballot(hint_vtx >= 0);
            if (hint_vtx >= 0) {
                const int k = hint_top + rank_in(hm);
                if (k < HINTS) sh.hint[k] = hint_vtx;
            }
            hint_top = min(HINTS, hint_top + __popcll(hm));
        }
        // retired chains return to the free ring
        {
            const uint64_t rm = __ballot(retire);
            if (retire) {
                sh.ring[(f_tail + rank_in(rm)) & (CH - 1)] = (int16_t)chain;
                sh.state[chain] = CS_FREE;
                mode = M_IDLE;
                chain = -1;
            }
            f_tail += __popcll(rm);
        }
        const uint64_t pm0 = __ballot(park);
        parked += __popcll(pm0);
        __syncthreads();
        // the chains whose walk reached the tree go back to the free ring at once; a
        // parked chain whose head's arrow points into a path that joined the tree
        // joins it too, transitively (a scan of the chain table per step, only
        // while chains are parked), and goes back to the ring as it is found.
        // Their state reads "done" until the closure is over.
        const uint64_t fm = __ballot(finish);
        if (fm != 0ull) {
            const int f0 = f_tail;
            if (finish) sh.ring[(f_tail + rank_in(fm)) & (CH - 1)] = (int16_t)chain;
            f_tail += __popcll(fm);
            __syncthreads();
            for (int pass = 0; parked > 0; ++pass) {
                int tot = 0;
                for (int c0 = 0; c0 < CH; c0 += WAVE) {
                    const int c = c0 + lane;
                    const bool join = sh.state[c] == CS_PARKED && sh.state[sh.up[c]] == CS_DONE;
                    const uint64_t jm = __ballot(join);
                    if (join) {
                        finish_chain(c);
                        sh.ring[(f_tail + rank_in(jm)) & (CH - 1)] = (int16_t)c;
                    }
                    f_tail += __popcll(jm);
                    tot += __popcll(jm);
                }
                __syncthreads();
                parked -= tot;
                if (tot == 0) break;
                if (pass > CH) { err = DEV_PROTOCOL; break; }
            }
            for (int i = f0 + lane; i < f_tail; i += WAVE) sh.state[sh.ring[i & (CH - 1)]] = CS_FREE;
            if (finish) {
                mode = M_IDLE;
                chain = -1;
            }
            __syncthreads();
        }
        // wake the chains parked on vertices that were popped or joined the tree:
        // each such lane walks the list its atomic detached, one chain per pass
        if ((unsigned)(wake_head + 1) > (unsigned)CH) { err = DEV_PROTOCOL; wake_head = -1; }
#pragma unroll 1
        for (int pass = 0;; ++pass) {
            const uint64_t wm = __ballot(wake_head >= 0);
            if (wm == 0ull) break;
            if (pass == CH) {  // longer than the chain table: the lists are broken
                err = DEV_PROTOCOL;
                break;
            }
            if (wake_head >= 0) {
                const int c = wake_head;
                if (sh.state[c] != CS_PARKED || sh.block[c] != wake_vtx) err = DEV_PROTOCOL;
                ws.queue[(q_tail + rank_in(wm)) & (CH - 1)] = make_int4(c, wake_kind, wake_vtx, 0);
                sh.state[c] = CS_QUEUED;
                wake_head = sh.wnext[c];
                if ((unsigned)(wake_head + 1) > (unsigned)CH) { err = DEV_PROTOCOL; wake_head = -1; }
            }
            q_tail += __popcll(wm);
            parked -= __popcll(wm);
        }
        __syncthreads();

        // ---- new parks: each looks for a cycle of parked chains through its own
        // new owner link, all lanes in lockstep (a chain woken above is no longer
        // parked).  A walk that runs into a cycle closed by another new park
        // stops there (Brent's cycle finding), so every walk ends within a few
        // times the number of chains.  A cycle is found by each new park on it;
        // its smallest chain index identifies it, and the lowest such lane pops
        // it, one cycle at a time.  (Most rounds park nothing and skip this.)
        if (pm0 != 0ull) {
            const int c = chain;
            bool walking = ((pm0 >> lane) & 1ull) != 0ull && sh.state[c] == CS_PARKED;
            bool on_cycle = false;
            int hare = 0, tort = 0, cmin = c, power = 1, lam = 1;
            if (walking) {
                const int x0 = sh.up[c];
                if (sh.state[x0] != CS_PARKED) {
                    walking = false;
                } else {
                    cmin = min(c, x0);
                    tort = x0;
                    hare = sh.up[x0];
                }
            }
#pragma unroll 1
            for (int step = 0; __ballot(walking) != 0ull; ++step) {
                if (walking) {
                    if (hare == c) {
                        on_cycle = true;
                        walking = false;
                    } else if (sh.state[hare] != CS_PARKED || hare == tort) {
                        walking = false;  // reaches a walking chain, or another new cycle
                    } else if (step >= 4 * CH) {
                        err = DEV_PROTOCOL;  // longer than any walk through the chain table
                        walking = false;
                    } else {
                        cmin = min(cmin, hare);
                        if (power == lam) {
                            tort = hare;
                            power <<= 1;
                            lam = 0;
                        }
                        hare = sh.up[hare];
                        ++lam;
                    }
                }
            }
            uint64_t todo = __ballot(on_cycle);
            while (todo != 0ull) {
                const int L = __ffsll((unsigned long long)todo) - 1;
                const int key = __shfl(cmin, L);
                todo &= ~__ballot(on_cycle && cmin == key);
                int ncyc = 0;
                if (lane == L) {
                    // the chains c -> up(c) -> ... -> c form a cycle of arrows: pop all
                    // of them; each keeps the vertex where its predecessor entered it
                    // and leaves the waiter list of the vertex it was parked on
                    int prev = c, m;
                    do {
                        m = sh.up[prev];
                        const int wp = sh.wprev[m], wn = sh.wnext[m];
                        if (wp >= 0) sh.wnext[wp] = (int16_t)wn;
                        else astore(tag_high(&tagw[sh.block[m]]), (uint32_t)(wn + 1));
                        if (wn >= 0) sh.wprev[wn] = (int16_t)wp;
                        ws.queue[(q_tail + ncyc) & (CH - 1)] = make_int4(m, T_POP, sh.block[prev], sh.block[m]);
                        sh.state[m] = CS_QUEUED;
                        ++ncyc;
                        prev = m;
                    } while (m != c && ncyc <= CH);
                }
                ncyc = __shfl(ncyc, L);
                parked -= ncyc;
                q_tail += ncyc;
                __syncthreads();
            }
            if (((pm0 >> lane) & 1ull) != 0ull) {
                mode = M_IDLE;
                chain = -1;
            }
        }
        fence_wg();
        if (__ballot(err != 0) != 0ull) break;
    }
    const int e = wave_max(err);
    if (e != 0) {
        report_error(ctl, e, idx);
        return -1;
    }
    *iters_used = iters;
    return wave_sum(mysteps);
}

// ------------------------------------------------------------ the kernels

// The sampler's arrays inside a slot's state block.
__device__ __forceinline__ SamplerWS sampler_ws(const SlotPtrs &sp) {
    SamplerWS ws;
    ws.tagw = reinterpret_cast<uint64_t *>(sp.state);
    ws.arrow = reinterpret_cast<uint64_t *>(sp.state + 8 * sp.stride);
    ws.rq = reinterpret_cast<int32_t *>(sp.state + 16 * sp.stride);
    ws.queue = sp.queue;
    ws.start = sp.cstart;
    return ws;
}

// The sampler and the sweep run one after the other: one LDS block serves both.
constexpr int CHAIN_BITS = 1 << 16;
template <int CH>
union KernelShared {
    SamplerShared<CH> samp;
    SweepLds<WAVE> sweep;
    uint32_t bitmap[CHAIN_BITS / 32];
};

// The evaluation of a chain sampler's tree: a function of its own, so that its
// registers do not weigh on the sampler's.  Inlined, a tree took 12 to 15% longer
// (road network of 44,780 vertices, 512 trees: 6,940 ms against 6,120 ms; grid of
// 102,400, 8 trees: 538 ms against 478 ms).
template <int CH>
__device__ __attribute__((noinline)) void evaluate_chain_tree(const GraphDev &g, const SlotPtrs &sp,
                                                              TreeShared<WAVE> &tree, KernelShared<CH> &lds,
                                                              const RunParams &rp, int64_t fen_len, int idx) {
    const uint64_t *arrow = sampler_ws(sp).arrow;
    evaluate_tree<WAVE>(g, sp, tree, lds.bitmap, min(CHAIN_BITS, path_bits(g.n)), rp, fen_len, idx,
                        [&](int v) { return (int32_t)(uint32_t)aload(&arrow[v]); });
}

// One sample s (work item idx) of graph g through the whole path in the
// calling workgroup: the tree, then (except in RUN_SAMPLE) its numbering and
// f.  Returns false when the workgroup must stop (an error was recorded).
template <int CH, bool LEAN>
__device__ bool process_one(const GraphDev &g, const SlotPtrs &sp, KernelShared<CH> &lds, TreeShared<WAVE> &tree,
                            const RunParams &rp, int64_t fen_len, int idx, uint64_t s) {
    const int lane = threadIdx.x;
    const size_t n = (size_t)g.n;
    int64_t iters = 0;
    const SamplerWS ws = sampler_ws(sp);
    const int64_t steps = sample_tree<CH, LEAN>(g, ws, lds.samp, rp.seed, s, rp.walkers, rp.iter_cap, rp.ctl, idx,
                                                &iters, rp.root_u, rp.root_v);
    if (steps < 0) return false;
    if (rp.mode == RUN_SAMPLE) {
        int32_t *po = rp.parents_out + (size_t)idx * n;
        uint32_t *co = rp.cnt_out ? rp.cnt_out + (size_t)idx * n : nullptr;
        for (int v = lane; v < g.n; v += WAVE) {
            const uint64_t ar = aload(&ws.arrow[v]);
            po[v] = (int32_t)(uint32_t)ar;  // -1 at vertices that started in the tree
            if (co) co[v] = (uint32_t)(ar >> 32);
        }
    } else {
        evaluate_chain_tree<CH>(g, sp, tree, lds, rp, fen_len, idx);
    }
    if (rp.steps_out && lane == 0) rp.steps_out[idx] = steps;
    if (rp.iters_out && lane == 0) rp.iters_out[idx] = iters;
    return true;
}

// Waves per SIMD the kernel is built to fit: three at 1,024 chains (168 VGPRs;
// the LDS then allows ten workgroups per CU), two at 2,048 (LDS allows five).
template <int CH>
constexpr int waves_per_simd() { return CH <= 1024 ? 3 : 2; }

template <int CH, bool LEAN>
__global__ void __launch_bounds__(WAVE) __attribute__((amdgpu_waves_per_eu(waves_per_simd<CH>())))
persistent_kernel(GraphDev g, SlotDev sd, RunParams rp) {
    __shared__ KernelShared<CH> lds;
    __shared__ TreeShared<WAVE> tree;
    const SlotPtrs sp = slot_ptrs(sd, (size_t)g.n);
    int64_t done = 0;
    while (true) {
        const int idx = next_item<WAVE>(rp.ctl, tree);
        if (idx >= rp.count) break;
        if (!process_one<CH, LEAN>(g, sp, lds, tree, rp, sd.fen_len, idx, (uint64_t)(rp.first + idx))) break;
        // samples finished by this workgroup, for a host that watches a long batch
        ++done;
        if (rp.progress && threadIdx.x == 0)
            __hip_atomic_store(&rp.progress[blockIdx.x], done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// One persistent launch over the samples of several graphs (a batch): work
// item idx belongs to the job j with base[j] <= idx < base[j + 1], and is
// sample first[j] + launch * count[j] + (idx - base[j]) of that job's graph,
// where `launch` counts the launches of the batch so far (read from device
// memory, advanced by advance_kernel after each launch).  Every item's f,
// draws and rounds go to position idx of the batch arrays.
template <int CH, bool LEAN>
__global__ void __launch_bounds__(WAVE) __attribute__((amdgpu_waves_per_eu(waves_per_simd<CH>())))
batch_kernel(BatchArgs a, SlotDev sd, int32_t *ctl,
                                                     const int64_t *launch) {
    __shared__ KernelShared<CH> lds;
    __shared__ TreeShared<WAVE> tree;
    const SlotPtrs sp = slot_ptrs(sd, (size_t)sd.stride);
    const int64_t L = *launch;
    while (true) {
        const int idx = next_item<WAVE>(ctl, tree);
        if (idx >= a.base[a.k]) break;
        int j = 0;
        while (j + 1 < a.k && idx >= a.base[j + 1]) ++j;
        const BatchJob &job = a.job[j];
        RunParams rp{};
        rp.seed = job.seed;
        rp.mode = RUN_ESTIMATE;
        rp.walkers = job.walkers;
        rp.traversal = job.traversal;
        rp.iter_cap = job.iter_cap;
        rp.ctl = ctl;
        rp.f_out = a.f;
        rp.steps_out = a.steps;
        rp.iters_out = a.iters;
        const uint64_t s = (uint64_t)(job.first + L * (int64_t)(a.base[j + 1] - a.base[j]) + (idx - a.base[j]));
        if (!process_one<CH, LEAN>(job.g, sp, lds, tree, rp, job.g.two_m + 2, idx, s)) break;
    }
}

// Launch counter of a batch: one more launch done; the status word is cleared
// by the next launch's reset.
__global__ void advance_kernel(int64_t *launch) {
    if (threadIdx.x == 0) *launch += 1;
}

// Resident trees that contain one of the deleted edges {u, v} (as u -> v or
// v -> u in the parent array): flags[t] = 1.  One thread per (tree, edge).
__global__ void flag_trees_kernel(const int32_t *par, int32_t count, int64_t n, const int32_t *eu,
                                  const int32_t *ev, int32_t ne, uint8_t *flags) {
    const int64_t total = (int64_t)count * ne;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t t = i / ne;
        const int k = (int)(i - t * ne);
        const int32_t u = eu[k], v = ev[k];
        const int32_t *row = par + t * n;
        if (row[u] == v || row[v] == u) flags[t] = 1;
    }
}

// The places of a path's vertices: pos[path[i]] = i, -1 elsewhere (two launches).
__global__ void clear_pos_kernel(int32_t *pos, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        pos[i] = -1;
}
__global__ void set_pos_kernel(const int32_t *path, int32_t len, int32_t *pos) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < len; i += gridDim.x * blockDim.x) pos[path[i]] = i;
}

// Signed count of the edges of a fixed u -> v path that a tree's own u -> v
// path uses (+1 along the path's direction, -1 against it); its mean over
// uniform spanning trees is the effective resistance R(u, v) (Kirchhoff: the
// tree path's direction on an edge has mean equal to the unit current there,
// and currents summed along any u -> v path give the potential difference).
// The edges x -> p(x) from u up to the root count as the path runs along them,
// those from v up the other way; the tree edges above both cancel, so the tree
// needs no numbering (1.9 ms for 1,024 trees of 20,000 vertices with one).  Two
// threads per tree, bound by the longer climb's dependent loads.
__global__ void path_current_kernel(const int32_t *par, int32_t count, int64_t n, const int32_t *path, int32_t len,
                                    const int32_t *pos, int64_t *c, int32_t *ctl) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x, t = i >> 1;
    int64_t sum = 0;
    if (t < count) {
        const int32_t *row = par + (int64_t)t * n;
        int32_t x = (i & 1) ? path[len - 1] : path[0];
        int64_t guard = 0;
        for (int32_t p; (p = row[x]) >= 0 && p < n; x = p) {
            const int32_t k = pos[x];
            if (k >= 0) {
                if (k + 1 < len && path[k + 1] == p) ++sum;
                else if (k > 0 && path[k - 1] == p) --sum;
            }
            if (++guard > n) {
                report_error(ctl, DEV_BADTREE, t);
                break;
            }
        }
    }
    const int64_t other = __shfl_xor(sum, 1);
    if (t < count && (i & 1) == 0) c[t] = sum - other;
}

// Trees drawn with u and v in the tree from the start (a two-tree forest
// rooted at u and v): add the edge v -> u, then re-orient the path from r so
// that every vertex points toward r.  One thread per tree.
__global__ void reroot_kernel(int32_t *par, int32_t count, int64_t n, int32_t u, int32_t v, int32_t r) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= count) return;
    int32_t *row = par + (int64_t)t * n;
    row[v] = u;
    int32_t prev = -1, x = r;
    for (int64_t guard = 0; x != -1 && guard <= n; ++guard) {
        const int32_t nx = row[x];
        row[x] = prev;
        prev = x;
        x = nx;
    }
}

// link-cut (section 4.2) on resident trees rows[t]: the tree path between u
// and v (lengths su from u and sv from v up to their lowest common ancestor)
// has d = su + sv edges; d_out[t] = d.  With relink, edge number j (drawn by
// Philox on counter (slot, serial, ISM_CTR_LO, ISM_CTR_HI); edges counted
// from u upward, then from v upward) is removed and {u, v} added: the path
// from the endpoint on j's side up to the cut edge is reversed.  One thread
// per tree.
__global__ void link_cut_kernel(int32_t *par, const int32_t *rows, int32_t count, int64_t n, int32_t u,
                                int32_t v, uint64_t seed, uint32_t serial, int relink, int64_t *d_out,
                                int32_t *ctl) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= count) return;
    const int32_t slot = rows[t];
    int32_t *row = par + (int64_t)slot * n;
    auto depth_of = [&](int32_t x) {
        int64_t d = 0;
        while (d <= n && row[x] != -1) {
            x = row[x];
            ++d;
        }
        return d;
    };
    int64_t du = depth_of(u), dv = depth_of(v);
    if (du > n || dv > n) {
        report_error(ctl, DEV_BADTREE, t);
        return;
    }
    int32_t x = u, y = v;
    int64_t su = 0, sv = 0;
    for (; du > dv; --du, ++su) x = row[x];
    for (; dv > du; --dv, ++sv) y = row[y];
    for (; x != y; ++su, ++sv) {
        x = row[x];
        y = row[y];
    }
    const int64_t d = su + sv;
    d_out[t] = d;
    if (!relink) return;
    if (d <= 0) {
        report_error(ctl, DEV_BADTREE, t);
        return;
    }
    const int64_t j = arrow_slot(seed, ((uint64_t)ISM_CTR_HI << 32) | ISM_CTR_LO, serial, (uint32_t)slot,
                                 (uint32_t)d);
    const bool u_side = j < su;
    int32_t prev = u_side ? v : u, z = u_side ? u : v;
    const int64_t steps = u_side ? j : j - su;
    for (int64_t i = 0; i <= steps; ++i) {
        const int32_t nz = row[z];
        row[z] = prev;
        prev = z;
        z = nz;
    }
}

__global__ void reset_ctl_kernel(int32_t *ctl) {
    if (threadIdx.x < 4) ctl[threadIdx.x] = 0;
}

__global__ void zero_i64_kernel(int64_t *p, int64_t len) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < len;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

// Exact sums of f and f^2 (128-bit) and of the draw counts of items
// base[b] .. base[b+1]-1 into out[b], one block b per range (a single range:
// base = {0, count}).
struct Ranges {
    int32_t base[BATCH_MAX + 1];
};

__global__ void __launch_bounds__(256) reduce_kernel(const int64_t *f, const int64_t *steps,
                                                     const int64_t *iters, Ranges r, ReduceOut *outs) {
    const int32_t lo = r.base[blockIdx.x], count = r.base[blockIdx.x + 1] - lo;
    f += lo;
    if (steps) steps += lo;
    if (iters) iters += lo;
    ReduceOut *out = outs + blockIdx.x;
    __shared__ unsigned __int128 sh_s[256];
    __shared__ unsigned __int128 sh_q[256];
    __shared__ int64_t sh_t[256];
    __shared__ int64_t sh_i[256];
    unsigned __int128 s = 0, q = 0;
    int64_t t = 0, it = 0;
    for (int i = threadIdx.x; i < count; i += 256) {
        const __int128 x = f[i];
        s += (unsigned __int128)x;
        q += (unsigned __int128)(x * x);
        if (steps) t += steps[i];
        if (iters) it += iters[i];
    }
    sh_s[threadIdx.x] = s;
    sh_q[threadIdx.x] = q;
    sh_t[threadIdx.x] = t;
    sh_i[threadIdx.x] = it;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            sh_s[threadIdx.x] += sh_s[threadIdx.x + w];
            sh_q[threadIdx.x] += sh_q[threadIdx.x + w];
            sh_t[threadIdx.x] += sh_t[threadIdx.x + w];
            sh_i[threadIdx.x] += sh_i[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out->sum_lo = (uint64_t)sh_s[0];
        out->sum_hi = (int64_t)(uint64_t)(sh_s[0] >> 64);
        out->sq_lo = (uint64_t)sh_q[0];
        out->sq_hi = (uint64_t)(sh_q[0] >> 64);
        out->steps = sh_t[0];
        out->iters = sh_i[0];
    }
}

}  // namespace

hipError_t launch_reset_ctl(int32_t *ctl, hipStream_t stream) {
    hipLaunchKernelGGL(reset_ctl_kernel, dim3(1), dim3(64), 0, stream, ctl);
    return hipGetLastError();
}

bool valid_chains(int chains) {
#define KC_CASE(C) if (chains == C) return true;
    KC_CHAIN_VARIANTS(KC_CASE)
#undef KC_CASE
    return false;
}

hipError_t launch_persistent(const GraphDev &g, const SlotDev &s, const RunParams &rp, int chains,
                             int slots, hipStream_t stream) {
    if (rp.mode != RUN_SAMPLE && rp.mode != RUN_ESTIMATE) return launch_tree(g, s, rp, slots, stream);
    if (rp.route != ROUTE_CHAINS) return launch_frontier(g, s, rp, slots, stream);
#define KC_CASE(C)                                                                                   \
    if (chains == C) {                                                                              \
        if (rp.lean)                                                                                \
            hipLaunchKernelGGL((persistent_kernel<C, true>), dim3(slots), dim3(WAVE), 0, stream, g, s, rp); \
        else                                                                                        \
            hipLaunchKernelGGL((persistent_kernel<C, false>), dim3(slots), dim3(WAVE), 0, stream, g, s, rp); \
        return hipGetLastError();                                                                   \
    }
    KC_CHAIN_VARIANTS(KC_CASE)
#undef KC_CASE
    return hipErrorInvalidValue;
}

int sampler_chains() { return MAX_CHAINS; }

int batch_blocks_per_cu(int chains) {
    int blocks = 0;
#define KC_CASE(C)                                                                                   \
    if (chains == C) {                                                                              \
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, batch_kernel<C, false>, WAVE, 0) != \
            hipSuccess)                                                                             \
            return 0;                                                                               \
        return blocks;                                                                              \
    }
    KC_CHAIN_VARIANTS(KC_CASE)
#undef KC_CASE
    return 0;
}

int persistent_blocks_per_cu(int chains) {
    int blocks = 0;
#define KC_CASE(C)                                                                                   \
    if (chains == C) {                                                                              \
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, persistent_kernel<C, false>, WAVE, 0) !=   \
            hipSuccess)                                                                             \
            return 0;                                                                               \
        return blocks;                                                                              \
    }
    KC_CHAIN_VARIANTS(KC_CASE)
#undef KC_CASE
    return 0;
}

hipError_t launch_reduce(const int64_t *f, const int64_t *steps, const int64_t *iters, int32_t count,
                         ReduceOut *out, hipStream_t stream) {
    Ranges r{};
    r.base[0] = 0;
    r.base[1] = count;
    hipLaunchKernelGGL(reduce_kernel, dim3(1), dim3(256), 0, stream, f, steps, iters, r, out);
    return hipGetLastError();
}

hipError_t launch_batch(const BatchArgs &a, const SlotDev &s, int32_t *ctl, int64_t *launch, ReduceOut *out,
                        int chains, int slots, hipStream_t stream) {
    if (a.k < 1 || a.k > BATCH_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(reset_ctl_kernel, dim3(1), dim3(64), 0, stream, ctl);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // lean looks when every job of the batch takes them
    bool lean = true;
    for (int j = 0; j < a.k; ++j) lean = lean && a.job[j].lean != 0;
#define KC_CASE(C)                                                                                \
    if (chains == C) {                                                                           \
        if (lean)                                                                                \
            hipLaunchKernelGGL((batch_kernel<C, true>), dim3(slots), dim3(WAVE), 0, stream, a, s, ctl, launch); \
        else                                                                                     \
            hipLaunchKernelGGL((batch_kernel<C, false>), dim3(slots), dim3(WAVE), 0, stream, a, s, ctl, launch); \
        e = hipGetLastError();                                                                   \
    }
    e = hipErrorInvalidValue;
    if (batch_is_frontier(a)) e = launch_frontier_batch(a, s, ctl, launch, slots, stream);
    else { KC_CHAIN_VARIANTS(KC_CASE) }
#undef KC_CASE
    if (e != hipSuccess) return e;
    Ranges r{};
    for (int j = 0; j <= a.k; ++j) r.base[j] = a.base[j];
    hipLaunchKernelGGL(reduce_kernel, dim3(a.k), dim3(256), 0, stream, a.f, a.steps, a.iters, r, out);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(advance_kernel, dim3(1), dim3(64), 0, stream, launch);
    return hipGetLastError();
}

hipError_t launch_reroot(int32_t *par, int32_t count, int64_t n, int32_t u, int32_t v, int32_t r,
                         hipStream_t stream) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(reroot_kernel, dim3((unsigned)((count + 63) / 64)), dim3(64), 0, stream, par, count, n,
                       u, v, r);
    return hipGetLastError();
}

hipError_t launch_link_cut(int32_t *par, const int32_t *rows, int32_t count, int64_t n, int32_t u, int32_t v,
                           uint64_t seed, uint32_t serial, int relink, int64_t *d_out, int32_t *ctl,
                           hipStream_t stream) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(link_cut_kernel, dim3((count + 63) / 64), dim3(64), 0, stream, par, rows, count, n, u, v,
                       seed, serial, relink, d_out, ctl);
    return hipGetLastError();
}

hipError_t launch_path_currents(const int32_t *par, int32_t count, int64_t n, const int32_t *path, int32_t len,
                                int32_t *pos, int64_t *c, int32_t *ctl, hipStream_t stream) {
    if (count <= 0 || len < 2) return hipErrorInvalidValue;
    hipLaunchKernelGGL(reset_ctl_kernel, dim3(1), dim3(64), 0, stream, ctl);
    hipLaunchKernelGGL(clear_pos_kernel, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 4096)), dim3(256), 0, stream,
                       pos, n);
    hipLaunchKernelGGL(set_pos_kernel, dim3((unsigned)std::min<int64_t>((len + 255) / 256, 4096)), dim3(256), 0, stream,
                       path, len, pos);
    hipLaunchKernelGGL(path_current_kernel, dim3((unsigned)((2 * (int64_t)count + 63) / 64)), dim3(64), 0, stream, par,
                       count, n, path, len, pos, c, ctl);
    return hipGetLastError();
}

hipError_t launch_flag_trees(const int32_t *par, int32_t count, int64_t n, const int32_t *eu,
                             const int32_t *ev, int32_t ne, uint8_t *flags, hipStream_t stream) {
    const int64_t total = (int64_t)count * ne;
    if (total <= 0) return hipSuccess;
    int64_t blocks = (total + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(flag_trees_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, par, count, n, eu, ev,
                       ne, flags);
    return hipGetLastError();
}

hipError_t launch_zero_i64(int64_t *p, int64_t len, hipStream_t stream) {
    if (len <= 0) return hipSuccess;
    int64_t blocks = (len + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(zero_i64_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, p, len);
    return hipGetLastError();
}

}  // namespace kc
