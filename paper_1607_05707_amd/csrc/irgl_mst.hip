// Boruvka minimum spanning forest: the workload the paper uses to show the
// Atomic construct (Section 3, the find-minimum-cross-component-edge kernel).
//
// Every vertex starts as its own component.  A round is three phases of one
// persistent cooperative launch, separated by the grid barrier:
//   1. find-min-edge: a ForAll over the worklist (all vertices in round 0,
//      then the vertices that still had a cross-component edge, the kernel's
//      Retry-style re-push) finds each vertex's lightest edge to another
//      component and makes it its component's candidate inside an atomic
//      section;
//   2. every component root hooks to the component at the other end of its
//      chosen edge and emits that edge into the forest (a pair of components
//      that chose the same edge keeps the smaller id as root and emits the
//      edge once);
//   3. pointer jumping flattens the hooks (iterated while Any(changed), with
//      the block-aggregated reduction), and every vertex moves to its new root.
// The loop ends when a round's worklist is empty.
//
// Edges are compared in the total order (weight, smaller endpoint, larger
// endpoint), so the minimum forest is unique and no cycle can form.  An
// undirected edge {u, v} is named by its canonical entry: the CSR index of
// the u -> v entry with u < v; (weight << 32 | canonical entry) is then a
// 64-bit key in the same order (entries of a row are sorted by destination).
//
// The atomic section updates two words of the component, its lightest
// weight and its edge, together.  Three compilations of it (IRGL_LOCK_*):
//   packed  - the MI355X form: the two words are one 64-bit key, updated
//             with a single 64-bit atomicMin;
//   spin    - the blocking Atomic: a compare-and-swap lock per component in
//             a divergence-safe retry loop (the lock holder runs its section
//             and releases inside the same loop iteration, so lanes of one
//             wavefront waiting on each other cannot deadlock);
//   ticket  - the same section under a ticket lock.
// Before taking a lock a lane reads the component's weight: weights only
// fall during phase 1, so a candidate heavier than a stale read cannot win.
// The lanes of a wavefront that offer to the same component first reduce
// their candidates to one (cooperative conversion, Sections 3.5 and 4.2,
// applied to the atomic section), so a giant component sees one lock
// acquisition or atomic per wavefront instead of one per vertex.
// Every lock wait is bounded by a wall-clock limit (IRGL_ERR_WATCHDOG).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>

#include "irgl.h"
#include "irgl_device.h"

namespace irgl_shared {
irgl_status note_hip_failure(hipError_t e);
irgl_status caller_csr(const irgl_graph_s *g, int *device, irgl_csr *out);
}  // namespace irgl_shared

namespace irgl {
namespace mst {

constexpr unsigned long long kNoKey = ~0ull;
constexpr int kTBlock = 4096;   // ... this many or more: the whole workgroup
constexpr int kMstQueue = 256;  // LDS push staging per wavefront
constexpr int kMstU = 4;        // entries per lane per step: their columns and weights, then their
                                // components, are in flight together (phase() in irgl_device.h)
constexpr int kMstChase = 32;   // hooks a root follows in one pass
constexpr int kMstSample = 256; // entries sampled for the dominant component
constexpr int kMstShare = 64;   // ... which holds at least this many of them

struct MstParams {
    int32_t n;
    const int32_t *row_ptr;
    const int32_t *col;
    const uint32_t *w;
    int32_t *comp;               // component (root id) of every vertex
    int32_t *hook;               // per root: the root it joins this round
    unsigned long long *key;     // packed: per root, weight << 32 | canonical entry
    uint32_t *minwt;             // spin / ticket: per root, the weight ...
    int32_t *minedge;            // ... and the canonical entry of its chosen edge
    uint32_t *lock;              // spin: per root lock word
    uint32_t *ticket;            // ticket: per root next ticket ...
    uint32_t *serving;           // ... and the ticket being served
    int32_t *wl0, *wl1;          // worklists of vertices that still had a cross edge
    int32_t *forest;             // emitted forest edges (canonical entries), capacity n
    int32_t *repmin;             // per root: smallest vertex id of its tree
    // per vertex: the row key and the canonical entry of the lightest cross
    // edge found last (in arrays that this lock kind does not use)
    unsigned long long *best;
    int32_t *bestentry;
    uint8_t *in_forest;          // optional: per CSR entry, 1 for both directions of forest edges
    int32_t *comp_out;           // optional: smallest vertex id of each vertex's tree
    unsigned long long *weight;  // forest weight (device)
    Ctrl *ctrl;
    Stats *dstats;
    uint32_t lock_kind;
    uint32_t max_rounds;
    unsigned long long wd_ticks;
    unsigned long long spin_ticks;
    uint32_t barrier;
};

// The launch reuses control-block counters: cnt[] for the rotating worklist
// counts, red[] for the pointer-jumping reduction, forest for the number of
// emitted forest edges.

template <int B>
struct MstSmem {
    static constexpr int NW = B / kWave;
    int queue[NW][kMstQueue];
    int fill[NW];
    uint32_t base;
    int flag;
    int owner;
    int big_v, big_r0, big_r1;
    unsigned long long red[NW];
    unsigned long long wsum[NW];
    int dsum[NW];
    // gather tier: the workgroup's rows concatenated (exclusive scan of the
    // degrees), each slot's owner found by a binary search
    int gstart[B];
    int gr0[B];
    int gv[B];
    int gc[B];
    int sample[kMstSample];
    unsigned long long vmin[B];  // per row: lightest cross edge as (w << 32 | neighbour)
};

// For a fixed vertex v, ordering its edges {v, u} by (w, smaller endpoint,
// larger endpoint) is ordering them by (w, u): an edge to u < v has the
// smaller endpoint u < v, an edge to u > v has v.  So a row's lightest cross
// edge is the minimum of the 64-bit row key w << 32 | u.

// The row key of entry k of a lane's kMstU entries, folded into `fold`, for
// those that lead to another component.  In the first round every vertex is
// its own component, so the components need no look at memory.
template <class Fold>
__device__ __forceinline__ void cross_entries(const MstParams &p, const int (&e)[kMstU], const bool (&act)[kMstU],
                                              const int (&v)[kMstU], const int (&c)[kMstU], bool first, Fold fold) {
    int u[kMstU], cu[kMstU];
    uint32_t w[kMstU];
#pragma unroll
    for (int k = 0; k < kMstU; ++k) {
        u[k] = p.col[e[k]];
        w[k] = p.w[e[k]];
    }
    phase(u);
    if (first) {  // uniform
#pragma unroll
        for (int k = 0; k < kMstU; ++k) cu[k] = u[k];
    } else {
#pragma unroll
        for (int k = 0; k < kMstU; ++k) cu[k] = p.comp[u[k]];
        phase(cu);
    }
    phase(w);
#pragma unroll
    for (int k = 0; k < kMstU; ++k)
        if (act[k] && u[k] != v[k] && cu[k] != c[k])
            fold(k, (static_cast<unsigned long long>(w[k]) << 32) | static_cast<uint32_t>(u[k]));
}

// Row key minimum of entries [r0, r1) of vertex v in component c, this
// thread's share of a workgroup's B threads.
template <int B>
__device__ __forceinline__ unsigned long long scan_row(const MstParams &p, int v, int c, int r0, int r1, int tid,
                                                       bool first, unsigned long long &scanned) {
    unsigned long long b = kNoKey;
    for (int x = r0; x < r1; x += B * kMstU) {
        int e[kMstU], vs[kMstU], cs[kMstU];
        bool act[kMstU];
#pragma unroll
        for (int k = 0; k < kMstU; ++k) {
            e[k] = x + k * B + tid;
            act[k] = e[k] < r1;
            scanned += act[k] ? 1u : 0u;
            e[k] = min(e[k], r1 - 1);
            vs[k] = v;
            cs[k] = c;
        }
        cross_entries(p, e, act, vs, cs, first, [&](int, unsigned long long key) { b = min(b, key); });
    }
    return b;
}

__device__ __forceinline__ unsigned long long wave_min(unsigned long long b) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) b = min(b, static_cast<unsigned long long>(__shfl_xor(b, off, kWave)));
    return b;
}

// The entry u -> v of u's row (rows sorted by destination: binary search,
// then a linear scan if the row is not sorted), or -1.
__device__ __forceinline__ int find_entry(const MstParams &p, int u, int v) {
    int a = p.row_ptr[u], b = p.row_ptr[u + 1];
    const int r0 = a, r1 = b;
    while (a < b) {
        const int mid = (a + b) >> 1;
        if (p.col[mid] < v) a = mid + 1;
        else b = mid;
    }
    if (a < r1 && p.col[a] == v) return a;
    for (int e = r0; e < r1; ++e)
        if (p.col[e] == v) return e;
    return -1;
}

// The row (source vertex) of CSR entry e.
__device__ __forceinline__ int row_of(const MstParams &p, int e) {
    int a = 0, b = p.n;  // largest v with row_ptr[v] <= e
    while (b - a > 1) {
        const int mid = (a + b) >> 1;
        if (p.row_ptr[mid] <= e) a = mid;
        else b = mid;
    }
    return a;
}

// Candidate key (weight << 32 | canonical entry) of row key rk of vertex v,
// or kNoKey.  The canonical entry is the smaller endpoint's entry.
__device__ __forceinline__ unsigned long long candidate_key(const MstParams &p, int v, unsigned long long rk) {
    if (rk == kNoKey) return kNoKey;
    const int u = static_cast<int>(rk & 0xFFFFFFFFull);
    const int canon = find_entry(p, min(u, v), max(u, v));
    if (canon < 0) {  // no reverse entry: the CSR is not symmetric
        set_error(p.ctrl, IRGL_ERR_INVALID_GRAPH, false);
        return kNoKey;
    }
    return (rk & 0xFFFFFFFF00000000ull) | static_cast<uint32_t>(canon);
}

// The atomic section of find-min-edge: make `k` the candidate of component
// c if it is lighter.  Called by every lane; `want` says whether this lane
// has a candidate.
__device__ __forceinline__ void offer(const MstParams &p, int c, unsigned long long k, bool want) {
    if (p.lock_kind == IRGL_LOCK_PACKED) {
        if (want && k < p.key[c]) atomicMin(&p.key[c], k);
        return;
    }
    const uint32_t wt = static_cast<uint32_t>(k >> 32);
    const int32_t edge = static_cast<int32_t>(k & 0xFFFFFFFFull);
    // a candidate heavier than a (possibly stale, never lower) read cannot win
    bool pending = want && wt <= p.minwt[c];
    const bool ticket = p.lock_kind == IRGL_LOCK_TICKET;
    uint32_t mine = 0;
    if (pending && ticket) mine = atomicAdd(&p.ticket[c], 1u);
    const unsigned long long t0 = wall_clock64();
    // The loop leaves only when no lane of the wavefront is pending (a
    // wave-uniform test at the top).  With a per-lane exit the compiler may
    // legally move the section and its release after the loop, where a lane
    // holding the lock waits, masked off, for lanes of its own wavefront
    // that spin on that lock: the divergence deadlock the Atomic construct
    // exists to avoid.  Here the section runs in the iteration that took the
    // lock, before the next test.
    for (;;) {
        if (__ballot(pending) == 0ull) break;
        if (pending) {
            const bool held = ticket ? load_agent(&p.serving[c]) == mine : atomicCAS(&p.lock[c], 0u, 1u) == 0u;
            if (held) {
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                const uint32_t cw = load_agent(&p.minwt[c]);
                const int32_t ce = static_cast<int32_t>(load_agent(reinterpret_cast<uint32_t *>(&p.minedge[c])));
                if (wt < cw || (wt == cw && (ce < 0 || edge < ce))) {
                    store_agent(&p.minwt[c], wt);
                    store_agent(reinterpret_cast<uint32_t *>(&p.minedge[c]), static_cast<uint32_t>(edge));
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                if (ticket) store_agent(&p.serving[c], mine + 1u);
                else store_agent(&p.lock[c], 0u);
                pending = false;
            } else if (wall_clock64() - t0 > p.spin_ticks) {
                set_error(p.ctrl, kErrWatchdog, true);
                pending = false;
            }
        }
        __builtin_amdgcn_s_sleep(1);
    }
}

// The component's chosen key after phase 1 (kNoKey: none).
__device__ __forceinline__ unsigned long long chosen(const MstParams &p, int c) {
    if (p.lock_kind == IRGL_LOCK_PACKED) return p.key[c];
    const int32_t e = p.minedge[c];
    return e < 0 ? kNoKey : (static_cast<unsigned long long>(p.minwt[c]) << 32) | static_cast<uint32_t>(e);
}

template <int B>
__device__ __forceinline__ unsigned long long block_sum(MstSmem<B> &sm, unsigned long long x) {
    constexpr int NW = B / kWave;
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) x += __shfl_xor(x, off, kWave);
    __syncthreads();
    if (lane_id() == 0) sm.wsum[threadIdx.x / kWave] = x;
    __syncthreads();
    unsigned long long t = 0;
#pragma unroll
    for (int k = 0; k < NW; ++k) t += sm.wsum[k];
    return t;
}

// A vertex of the component that most of a fixed sample of the entries lead
// to, if that is a quarter of them or more, else -1.  Every workgroup finds
// the same one.
template <int B>
__device__ __forceinline__ int dominant(const MstParams &p, MstSmem<B> &sm) {
    static_assert(B >= kMstSample && kMstSample % kWave == 0, "one thread per sample");
    const int tid = threadIdx.x;
    const uint32_t m = static_cast<uint32_t>(p.row_ptr[p.n]);
    if (m == 0u) return -1;  // uniform
    int u = 0, c = -1, best = 0;
    if (tid < kMstSample) {
        const uint32_t e = static_cast<uint32_t>((static_cast<unsigned long long>(tid) * 0x9E3779B97F4A7C15ull >> 32) *
                                                     static_cast<unsigned long long>(m) >> 32);
        u = p.col[e];
        c = p.comp[u];
        sm.sample[tid] = c;
    }
    __syncthreads();
    if (tid < kMstSample) {
        for (int k = 0; k < kMstSample; ++k) best += sm.sample[k] == c ? 1 : 0;
        best = best << 16 | tid;  // ties: the last sample
    }
    unsigned long long top = ~0ull - static_cast<unsigned long long>(best);
    top = wave_min(top);
    if (lane_id() == 0) sm.red[tid / kWave] = top;
    __syncthreads();
    for (int k = 0; k < B / kWave; ++k) top = min(top, sm.red[k]);
    const int got = static_cast<int>(~0ull - top);
    if (tid == (got & 0xFFFF)) sm.owner = u;
    __syncthreads();
    const int x = sm.owner;
    __syncthreads();
    return (got >> 16) >= kMstShare ? x : -1;
}

// Phase 1 over worklist `in` (identity when null) of cnt_in vertices; pushes
// the vertices that have a cross edge.  Rows of kTBlock or more entries are
// scanned by the whole workgroup one at a time; the other rows of a tile are
// concatenated and dealt to the lanes in full rounds (load-balanced gather),
// each slot folding its edge into its row's minimum with an LDS atomicMin.
template <int B>
__device__ __forceinline__ void find_min_edges(const MstParams &p, MstSmem<B> &sm, Team tm, const int32_t *in,
                                               uint32_t cnt_in, WaveQueue &wq, uint32_t *cnt_out,
                                               int32_t *out, unsigned long long &scanned, int skip) {
    constexpr int NW = B / kWave;
    const int tid = threadIdx.x, lane = lane_id(), wid = tid / kWave;
    const bool first = in == nullptr;  // every vertex is its own component
    for (uint32_t base = tm.id * B; base < cnt_in; base += tm.size * B) {
        const uint32_t i = base + tid;
        int v = -1, c = -1, r0 = 0, r1 = 0;
        unsigned long long rk = kNoKey;
        bool kept = false;
        if (i < cnt_in) {
            v = in ? in[i] : static_cast<int>(i);
            c = p.comp[v];
            r0 = p.row_ptr[v];
            r1 = p.row_ptr[v + 1];
            if (!first) {
                // the lightest cross edge of the round before is the lightest
                // still, if it is a cross edge still: cross edges only get
                // fewer (RMAT-20: rounds 2 and 3 scanned every row again, 300
                // us each)
                rk = p.best[v];
                kept = p.comp[static_cast<uint32_t>(rk)] != c;
            }
            if (c == skip) {  // the others will reach it
                v = -1;
                kept = false;
                r1 = r0;
            }
            if (kept) r1 = r0;
            else rk = kNoKey;
        }
        int deg = r1 - r0;
        // workgroup tier: one large row at a time
        while (__syncthreads_or(deg >= kTBlock)) {
            if (deg >= kTBlock) sm.owner = tid;
            __syncthreads();
            if (sm.owner == tid) {
                sm.big_v = v;
                sm.big_r0 = r0;
                sm.big_r1 = r1;
                deg = 0;
            }
            __syncthreads();
            const int bv = sm.big_v;
            const unsigned long long b = wave_min(scan_row<B>(p, bv, p.comp[bv], sm.big_r0, sm.big_r1, tid, first, scanned));
            if (lane == 0) sm.red[wid] = b;
            __syncthreads();
            if (sm.owner == tid) {
                for (int k = 0; k < NW; ++k) rk = min(rk, sm.red[k]);
            }
            __syncthreads();
        }
        // gather tier
        const int incl = wave_inclusive_scan(deg);
        if (lane == kWave - 1) sm.dsum[wid] = incl;
        sm.vmin[tid] = kNoKey;
        __syncthreads();
        int total = 0, wpre = 0;
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            wpre += (k < wid) ? sm.dsum[k] : 0;
            total += sm.dsum[k];
        }
        sm.gstart[tid] = wpre + incl - deg;
        sm.gr0[tid] = r0;
        sm.gv[tid] = v;
        sm.gc[tid] = c;
        __syncthreads();
        // a lane takes kMstU consecutive slots, mostly of one row: it folds
        // them in a register and touches the row's minimum once (an LDS
        // atomic per entry, most of a wavefront's on one row, was the bound)
        for (int done = 0; done < total; done += B * kMstU) {
            int e[kMstU], o[kMstU], vs[kMstU], cs[kMstU];
            bool act[kMstU];
            const int s0 = done + tid * kMstU;
            int ow = 0;
            if (s0 < total) {
#pragma unroll
                for (int step = B / 2; step > 0; step >>= 1)
                    if (sm.gstart[ow + step] <= s0) ow += step;
            }
#pragma unroll
            for (int k = 0; k < kMstU; ++k) {
                const int slot = s0 + k;
                act[k] = slot < total;
                while (act[k] && ow < B - 1 && sm.gstart[ow + 1] <= slot) ++ow;
                o[k] = ow;
                e[k] = act[k] ? sm.gr0[ow] + (slot - sm.gstart[ow]) : 0;
                vs[k] = sm.gv[ow];
                cs[k] = sm.gc[ow];
                scanned += act[k] ? 1u : 0u;
            }
            int row = o[0];
            unsigned long long low = kNoKey;
            cross_entries(p, e, act, vs, cs, first, [&](int k, unsigned long long key) {
                if (o[k] != row) {
                    if (low != kNoKey) atomicMin(&sm.vmin[row], low);
                    row = o[k];
                    low = kNoKey;
                }
                low = min(low, key);
            });
            if (low != kNoKey) atomicMin(&sm.vmin[row], low);
        }
        __syncthreads();
        if (deg > 0) rk = sm.vmin[tid];
        unsigned long long k = kNoKey;
        if (kept) {
            k = (rk & 0xFFFFFFFF00000000ull) | static_cast<uint32_t>(p.bestentry[v]);
        } else if (v >= 0) {
            k = candidate_key(p, v, rk);
            if (k != kNoKey) {
                p.best[v] = rk;
                p.bestentry[v] = static_cast<int32_t>(static_cast<uint32_t>(k));
            }
        }
        const bool has = k != kNoKey;
        // Cooperative conversion of the atomic section: the candidates of the
        // wavefront's lanes that share the first candidate lane's component
        // (in later rounds most lanes are in one giant component) are reduced
        // to their minimum, and only that lane enters the section for them.
        bool want = has;
        const unsigned long long cm = __ballot(has);
        if (cm) {
            const int leader = __ffsll(static_cast<long long>(cm)) - 1;
            const int cl = __shfl(c, leader, kWave);
            const bool same = has && c == cl;
            const unsigned long long kk = wave_min(same ? k : kNoKey);
            if (same) {
                want = lane == leader;
                k = kk;
            }
        }
        offer(p, c, k, want);
        wq.push(has, v, cnt_out, out, static_cast<uint32_t>(p.n), p.ctrl);
        __syncthreads();  // the gather arrays are rewritten by the next tile
    }
}

// Five waves per SIMD: 1280 workgroups of 256 threads, the most an explicit
// grid may ask for.
template <int B>
__global__ __launch_bounds__(B) __attribute__((amdgpu_waves_per_eu(fit_waves<B, 5>()))) void mst_kernel(MstParams p) {
    __shared__ MstSmem<B> sm;
    const Team tm = whole_grid();
    BarrierState bs = make_barrier_state(p.wd_ticks, p.barrier);
    Ctrl *ctrl = p.ctrl;
    const int wid = threadIdx.x / kWave;
    const uint32_t n = static_cast<uint32_t>(p.n);
    const uint32_t stride = tm.size * B;
    const uint32_t gid = tm.id * B + threadIdx.x;
    const bool lead = tm.id == 0 && threadIdx.x == 0;
    unsigned long long scanned = 0, items = 0, added = 0;
    uint32_t round = 0;
    uint32_t jumps = 0;  // pointer-jumping passes so far (rotates the reduction words)
    // A vertex of the component that holds most entries, once there is one.
    // That component chooses no edge from then on: every other component
    // still chooses its lightest, so each joins another and the forest is the
    // same, but its rows (nearly all of the graph in the last rounds, whose
    // vertices would find no edge to another component) are not scanned.  The
    // same vertex names it in every round, so its vertices may leave the
    // worklist for good.
    int x0 = -1;
    uint32_t *const fcnt = &ctrl->forest;
    bool ok = true;
    for (;; ++round) {
        const uint32_t cnt_in = round == 0 ? n : min(load_agent(&ctrl->cnt[round % 3]), n);
        if (cnt_in == 0) break;
        if (round >= p.max_rounds) {
            if (lead) set_error(ctrl, kErrIterLimit, false);
            break;
        }
        items += cnt_in;
        if (lead) store_agent(&ctrl->cnt[(round + 2) % 3], 0u);
        const int32_t *in = round == 0 ? nullptr : ((round & 1u) ? p.wl1 : p.wl0);
        int32_t *out = (round & 1u) ? p.wl0 : p.wl1;
        WaveQueue wq{sm.queue[wid], 0, kMstQueue};
        // phase 1: find-min-edge with the atomic section
        if (round > 0 && x0 < 0) x0 = dominant<B>(p, sm);
        find_min_edges<B>(p, sm, tm, in, cnt_in, wq, &ctrl->cnt[(round + 1) % 3], out, scanned,
                          x0 < 0 ? -2 : p.comp[x0]);
        block_drain<B>(wq, sm.fill, &sm.base, &ctrl->cnt[(round + 1) % 3], out, n, ctrl);
        if (!(ok = grid_barrier(ctrl, bs, &sm.flag, nullptr, tm))) break;
        // phase 2: hook every root with a candidate, emit its edge through the
        // wavefront's LDS queue (one atomic per wavefront and step on the one
        // forest counter was 0.18 of the phase's 0.21 ms on RMAT-20)
        for (uint32_t base2 = tm.id * B; base2 < n; base2 += stride) {
            const uint32_t c = base2 + threadIdx.x;
            bool emit = false;
            int e = 0;
            if (c < n && p.comp[c] == static_cast<int32_t>(c)) {
                const unsigned long long k = chosen(p, static_cast<int>(c));
                if (k != kNoKey) {
                    e = static_cast<int>(k & 0xFFFFFFFFull);
                    const int lo = row_of(p, e), hi = p.col[e];
                    const int other = p.comp[lo] == static_cast<int32_t>(c) ? hi : lo;
                    const int c2 = p.comp[other];
                    const bool mutual = chosen(p, c2) == k;
                    p.hook[c] = (mutual && static_cast<int>(c) < c2) ? static_cast<int32_t>(c) : c2;
                    emit = !(mutual && static_cast<int>(c) > c2);
                    if (emit) added += static_cast<unsigned long long>(k >> 32);
                }
            }
            wq.push(emit, e, fcnt, p.forest, n, ctrl);
        }
        block_drain<B>(wq, sm.fill, &sm.base, fcnt, p.forest, n, ctrl);
        if (!(ok = grid_barrier(ctrl, bs, &sm.flag, nullptr, tm))) break;
        // phase 3: pointer jumping over the hooks, While Any(unfinished): a
        // root follows its hooks for up to kMstChase steps, which ends most
        // phases after one pass (concurrent writes only put an ancestor
        // nearer the end in place of another)
        for (uint32_t pass = 0;; ++jumps, ++pass) {
            // the hooks form a forest (edge keys strictly fall along a hook
            // chain), so its depth is below n and log2 n passes flatten it
            if (pass > p.max_rounds) {
                if (lead) set_error(ctrl, kErrInternal, false);
                ok = false;
                break;
            }
            // red[(jumps + 1) % 3] was last read after pass jumps - 2, before
            // the barrier of pass jumps - 1; it is next set in pass jumps + 1
            uint32_t *red = &ctrl->red[jumps % 3];
            if (lead) store_agent(&ctrl->red[(jumps + 1) % 3], 0u);
            bool changed = false;
            for (uint32_t c = gid; c < n; c += stride) {
                if (p.comp[c] != static_cast<int32_t>(c)) continue;
                const int32_t h0 = p.hook[c];
                int32_t h = h0, hh = p.hook[h0];
                for (int k = 0; k < kMstChase && hh != h; ++k) {
                    h = hh;
                    hh = p.hook[h];
                }
                if (h != h0) p.hook[c] = h;
                changed |= hh != h;
            }
            if (__syncthreads_or(changed) && threadIdx.x == 0) atomicOr(red, 1u);
            if (!(ok = grid_barrier(ctrl, bs, &sm.flag, nullptr, tm))) break;
            if (load_agent(red) == 0u) {
                ++jumps;
                break;
            }
        }
        if (!ok) break;
        // every vertex joins its new root; the roots' candidates are cleared
        for (uint32_t v = gid; v < n; v += stride) {
            p.comp[v] = p.hook[p.comp[v]];
            if (p.lock_kind == IRGL_LOCK_PACKED) {
                p.key[v] = kNoKey;
            } else {
                p.minwt[v] = kInf;
                p.minedge[v] = -1;
            }
        }
        if (!(ok = grid_barrier(ctrl, bs, &sm.flag, nullptr, tm))) break;
        // (a root's hook is itself again: roots that kept their id were the
        // hook forest's roots)
    }
    const unsigned long long wsum = block_sum<B>(sm, added);
    const unsigned long long ssum = block_sum<B>(sm, scanned);
    if (threadIdx.x == 0) {
        if (wsum) atomicAdd(p.weight, wsum);
        atomicAdd(&ctrl->edges, ssum);
        if (tm.id == 0) {
            ctrl->iterations = round;
            ctrl->items = items;
        }
    }
    if (ok) ok = grid_barrier(ctrl, bs, &sm.flag, nullptr, tm);
    if (ok) {
        // smallest vertex id of every tree, then the per-entry marks.  The
        // dominant component's is one minimum per thread and one atomic per
        // wavefront (its 620,000 atomics on one word took 2.9 ms of 6.3 on
        // RMAT-20); of the others a wavefront's lanes that share the first
        // lane's component leave it to that lane (consecutive lanes hold
        // consecutive ids), and a lane whose id is no smaller than the word
        // it reads, which only falls, has nothing to do.
        if (x0 < 0) x0 = dominant<B>(p, sm);
        const int32_t big = x0 < 0 ? -2 : p.comp[x0];
        uint32_t low = kInf;
        for (uint32_t base3 = tm.id * B; base3 < n; base3 += stride) {
            const uint32_t v = base3 + threadIdx.x;
            const bool live = v < n;
            const int cv = live ? p.comp[v] : -1;
            bool mine = live && cv != big;
            if (live && !mine) low = min(low, v);
            const unsigned long long lm = __ballot(mine);
            if (lm) {
                const int leader = __ffsll(static_cast<long long>(lm)) - 1;
                const int cl = __shfl(cv, leader, kWave);
                if (cv == cl && lane_id() != leader) mine = false;
            }
            if (mine && static_cast<int32_t>(v) < p.repmin[cv]) atomicMin(&p.repmin[cv], static_cast<int32_t>(v));
        }
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) low = min(low, static_cast<uint32_t>(__shfl_xor(low, off, kWave)));
        if (lane_id() == 0 && low != kInf) atomicMin(&p.repmin[big], static_cast<int32_t>(low));
        const uint32_t nf = min(load_agent(fcnt), n);
        if (p.in_forest) {
            for (uint32_t k = gid; k < nf; k += stride) {
                const int e = p.forest[k];
                const int lo = row_of(p, e), hi = p.col[e];
                p.in_forest[e] = 1;
                const int r = find_entry(p, hi, lo);
                if (r >= 0) p.in_forest[r] = 1;
            }
        }
        ok = grid_barrier(ctrl, bs, &sm.flag, nullptr, tm);
        if (ok && p.comp_out)
            for (uint32_t v = gid; v < n; v += stride) p.comp_out[v] = p.repmin[p.comp[v]];
    }
    // statistics: the last workgroup to leave publishes them
    if (threadIdx.x == 0) {
        const uint32_t prev = __hip_atomic_fetch_add(&ctrl->done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        if (prev == tm.size - 1 && p.dstats) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            Stats *s = p.dstats;
            s->status = static_cast<int32_t>(load_agent(&ctrl->error));
            s->iterations = ctrl->iterations;
            s->items = ctrl->items;
            s->edges = __hip_atomic_load(&ctrl->edges, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s->max_frontier = 0;
            s->grid = static_cast<int32_t>(tm.size);
            s->block = B;
            s->heavy_pulls = 0;
            s->frontier_edges = load_agent(fcnt);
        }
    }
}

__global__ void mst_init_kernel(MstParams p, unsigned long long m) {
    const unsigned long long stride = static_cast<unsigned long long>(gridDim.x) * blockDim.x;
    const unsigned long long t = static_cast<unsigned long long>(blockIdx.x) * blockDim.x + threadIdx.x;
    for (unsigned long long v = t; v < static_cast<unsigned long long>(p.n); v += stride) {
        p.comp[v] = static_cast<int32_t>(v);
        p.hook[v] = static_cast<int32_t>(v);
        p.repmin[v] = 0x7FFFFFFF;
        if (p.lock_kind == IRGL_LOCK_PACKED) {  // the other arrays are not this kind's
            p.key[v] = kNoKey;
            continue;
        }
        p.minwt[v] = kInf;
        p.minedge[v] = -1;
        p.lock[v] = 0;
        p.ticket[v] = 0;
        p.serving[v] = 0;
    }
    if (p.in_forest)
        for (unsigned long long e = t; e < m; e += stride) p.in_forest[e] = 0;
    if (t == 0) {
        Ctrl *c = p.ctrl;
        for (int k = 0; k < 3; ++k) {
            c->cnt[k] = 0;
            c->red[k] = 0;
        }
        c->forest = 0;
        reset_barrier_words(c);
        c->error = 0;
        c->fatal = 0;
        c->done = 0;
        c->iterations = 0;
        c->items = 0;
        c->edges = 0;
        *p.weight = 0;
    }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
constexpr size_t kAlignB = 256;
constexpr size_t align_b(size_t x) { return (x + kAlignB - 1) / kAlignB * kAlignB; }

struct MstLayout {
    size_t ctrl, comp, hook, key, minwt, minedge, lock, ticket, serving, wl0, wl1, forest, repmin, weight, total;
};

MstLayout mst_layout(int64_t n) {
    MstLayout L;
    const size_t nb = align_b(static_cast<size_t>(n) * 4);
    L.ctrl = 0;
    L.comp = align_b(sizeof(Ctrl));
    L.hook = L.comp + nb;
    L.key = L.hook + nb;
    L.minwt = L.key + align_b(static_cast<size_t>(n) * 8);
    L.minedge = L.minwt + nb;  // (the two hold n 64-bit words for the packed kind)
    L.lock = L.minedge + nb;
    L.ticket = L.lock + nb;
    L.serving = L.ticket + nb;
    L.wl0 = L.serving + nb;
    L.wl1 = L.wl0 + nb;
    L.forest = L.wl1 + nb;
    L.repmin = L.forest + nb;
    L.weight = L.repmin + nb;
    L.total = L.weight + kAlignB;
    return L;
}

#define MST_HIP(call)                                                   \
    do {                                                                \
        hipError_t e_ = (call);                                         \
        if (e_ != hipSuccess) return irgl_shared::note_hip_failure(e_); \
    } while (0)

template <int B>
irgl_status mst_grid(int dev, int requested, int *grid) {
    int cus = 0, per_cu = 0;
    MST_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    MST_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, mst_kernel<B>, B, 0));
    // at most 6 waves per SIMD are co-resident on gfx950 (the same cap as
    // every other cooperative launch of the library)
    per_cu = std::min(per_cu, std::max(1, 24 / (B / kWave)));
    const int limit = per_cu * cus;
    if (limit <= 0 || requested < 0 || requested > limit) return IRGL_ERR_CONFIG;
    *grid = requested ? requested : limit;
    return IRGL_OK;
}

// Workgroups a graph repays: one thread for about twelve entries (four for a
// vertex), in steps of 32 workgroups; every further one costs each of the
// three or more barriers of a round (us per forest at 32 / 128 / 512
// workgroups of 512 threads: R-MAT 13, 158K entries, 217 / 232 / 310; R-MAT
// 17, 2.9M, 991 / 468 / 481; road-like 150^2 347 / 320 / 437, 1200^2 10694 /
// 3119 / 1587).
int mst_workgroups(int64_t n, int64_t m, int block) {
    const int64_t groups = (m + 4 * n) / 12 / block;
    return static_cast<int>(std::min<int64_t>(1 << 20, (groups + 31) / 32 * 32 + (groups == 0 ? 32 : 0)));
}

template <int B>
irgl_status mst_launch(MstParams &p, int64_t m, int dev, int requested, hipStream_t s) {
    int grid = 0;
    irgl_status st = mst_grid<B>(dev, requested, &grid);
    if (st) return st;
    // ... and at most 1024 threads per compute unit (us at 1024 / 1280
    // workgroups of 256: uniform 600,000 x 12 1312 / 1384, 2M x 16 2923 /
    // 3048; road-like 2048^2 3380 / 3283)
    if (!requested) {
        int cus = 0;
        MST_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
        grid = std::min({grid, mst_workgroups(p.n, m, B), cus * (1024 / B)});
    }
    void *args[] = {&p};
    MST_HIP(hipLaunchCooperativeKernel(reinterpret_cast<const void *>(mst_kernel<B>), dim3(grid), dim3(B), args, 0,
                                       s));
    return IRGL_OK;
}

}  // namespace mst
}  // namespace irgl

using namespace irgl::mst;

extern "C" {

irgl_status irgl_mst_workspace_bytes(irgl_graph g, size_t *bytes) {
    int dev = 0;
    irgl_csr csr;
    irgl_status st = irgl_shared::caller_csr(g, &dev, &csr);
    if (st) return st;
    if (!bytes) return IRGL_ERR_INVALID_ARGUMENT;
    *bytes = mst_layout(csr.n).total;
    return IRGL_OK;
}

irgl_status irgl_mst(irgl_graph g, uint64_t *weight, int32_t *component, uint8_t *in_forest, void *ws,
                     size_t ws_bytes, void *stream, irgl_stats *dstats, const irgl_mst_config *cfg) {
    int dev = 0;
    irgl_csr csr;
    irgl_status st = irgl_shared::caller_csr(g, &dev, &csr);
    if (st) return st;
    if (!weight || !ws) return IRGL_ERR_INVALID_ARGUMENT;
    if (!csr.w && csr.m > 0) return IRGL_ERR_NO_WEIGHTS;  // an edgeless graph needs none
    // RMAT-22, ms at workgroups x threads: 6.3 at 256x512, 6.2 at 512x256, 5.4 at 512x512
    const int block = (cfg && cfg->block) ? cfg->block : 512;
    if (block != 256 && block != 512 && block != 1024) return IRGL_ERR_CONFIG;
    const uint32_t kind = cfg ? cfg->lock : IRGL_LOCK_PACKED;
    if (kind > IRGL_LOCK_TICKET) return IRGL_ERR_CONFIG;
    const uint32_t barrier = cfg ? cfg->barrier : IRGL_BARRIER_XCD;
    if (barrier > IRGL_BARRIER_WORKGROUP) return IRGL_ERR_CONFIG;
    if (csr.m >= (1ll << 31)) return IRGL_ERR_TOO_LARGE;  // canonical entries are 31-bit
    const MstLayout L = mst_layout(csr.n);
    if (ws_bytes < L.total) return IRGL_ERR_WORKSPACE_TOO_SMALL;
    int cur = -1;
    MST_HIP(hipGetDevice(&cur));
    if (cur != dev) MST_HIP(hipSetDevice(dev));
    int khz = 0;
    MST_HIP(hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev));
    if (khz <= 0) khz = 100000;
    char *base = static_cast<char *>(ws);
    MstParams p;
    std::memset(&p, 0, sizeof(p));
    p.n = csr.n;
    p.row_ptr = csr.row_ptr;
    p.col = csr.col;
    p.w = csr.w;
    p.comp = reinterpret_cast<int32_t *>(base + L.comp);
    p.hook = reinterpret_cast<int32_t *>(base + L.hook);
    p.key = reinterpret_cast<unsigned long long *>(base + L.key);
    p.minwt = reinterpret_cast<uint32_t *>(base + L.minwt);
    p.minedge = reinterpret_cast<int32_t *>(base + L.minedge);
    p.lock = reinterpret_cast<uint32_t *>(base + L.lock);
    p.ticket = reinterpret_cast<uint32_t *>(base + L.ticket);
    p.serving = reinterpret_cast<uint32_t *>(base + L.serving);
    p.wl0 = reinterpret_cast<int32_t *>(base + L.wl0);
    p.wl1 = reinterpret_cast<int32_t *>(base + L.wl1);
    p.forest = reinterpret_cast<int32_t *>(base + L.forest);
    p.repmin = reinterpret_cast<int32_t *>(base + L.repmin);
    p.best = reinterpret_cast<unsigned long long *>(base + (kind == IRGL_LOCK_PACKED ? L.minwt : L.key));
    p.bestentry = reinterpret_cast<int32_t *>(base + (kind == IRGL_LOCK_SPIN ? L.ticket : L.lock));
    p.in_forest = in_forest;
    p.comp_out = component;
    p.weight = reinterpret_cast<unsigned long long *>(weight);
    p.ctrl = reinterpret_cast<irgl::Ctrl *>(base + L.ctrl);
    p.dstats = reinterpret_cast<irgl::Stats *>(dstats);
    p.lock_kind = kind;
    // components at least halve every round: ceil(log2 n) + 2 rounds suffice
    uint32_t rounds = 2;
    for (int64_t x = 1; x < csr.n; x <<= 1) ++rounds;
    p.max_rounds = rounds;
    const uint32_t wd_ms = (cfg && cfg->watchdog_ms) ? cfg->watchdog_ms : 20000u;
    p.wd_ticks = static_cast<unsigned long long>(wd_ms) * static_cast<unsigned long long>(khz);
    p.spin_ticks = p.wd_ticks;
    p.barrier = barrier;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const unsigned long long m = static_cast<unsigned long long>(csr.m);
    const int fill = static_cast<int>(std::min<int64_t>(65535, (std::max<int64_t>(csr.n, csr.m) + 255) / 256));
    hipLaunchKernelGGL(mst_init_kernel, dim3(std::max(fill, 1)), dim3(256), 0, s, p, m);
    MST_HIP(hipGetLastError());
    switch (block) {
        case 256: st = mst_launch<256>(p, csr.m, dev, cfg ? cfg->grid : 0, s); break;
        case 512: st = mst_launch<512>(p, csr.m, dev, cfg ? cfg->grid : 0, s); break;
        default: st = mst_launch<1024>(p, csr.m, dev, cfg ? cfg->grid : 0, s); break;
    }
    if (cur != dev) (void)hipSetDevice(cur);
    return st;
}

}  // extern "C"
