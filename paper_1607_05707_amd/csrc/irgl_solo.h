// Solo runs: consecutive small invocations of the Iterate loop, run by the
// team's first workgroup alone while the others wait at the next team
// barrier.
//
// A small invocation costs its barrier and its instructions, not its work:
// 3.6 us for a barrier of 256 workgroups (1.9 us of arrivals and polling, the
// rest the cache invalidation of 32 workgroups per XCD, one after another),
// then worklist, counters and drain through memory that all XCDs share.
// Here the worklists and counters live in LDS, only the wavefronts that hold
// items take part, and the barrier is the workgroup's.
#pragma once

#include "irgl_expand.h"

namespace irgl {

// A solo run pops worklists of at most kSoloItems vertices (kSoloPer per
// thread of its wavefronts, looked up together; fewer in a workgroup with
// fewer wavefronts) with at most kSoloEdges edges, and leaves larger ones to
// the team: one compute unit looks up about one scattered address per clock.
// It also ends after kSoloSteps invocations, so that the host abort flag is
// seen every few milliseconds, and once a share of the watchdog's bound has
// passed: the other workgroups wait at one barrier all the while.  The clock
// is read every kSoloClock invocations (a full one takes about 10 us, so a
// bound of 1 ms is kept with half of it to spare; one of 512 invocations on
// 1000 items each took longer).
constexpr int kSoloWaves = 8;
constexpr int kSoloPer = 2;
constexpr uint32_t kSoloItems = kSoloWaves * kWave * kSoloPer;
constexpr uint32_t kSoloEdges = 4096;
constexpr uint32_t kSoloSteps = 512;
constexpr uint32_t kSoloClock = 8;
constexpr unsigned long long kSoloShare = 4;
// After a run of fewer than kSoloWorth invocations kSoloHold team invocations follow.
constexpr uint32_t kSoloWorth = 3;
constexpr uint32_t kSoloHold = 8;
// Far lists of at most this many entries are transferred solo.
constexpr uint32_t kSoloFar = 2048;
// Rows of at most this many edges are walked by the thread that popped them;
// a wavefront with a longer one deals its edges to its lanes.
constexpr int kSoloRow = 8;

// The largest worklist a solo run is entered with: about kSoloEdges edges at
// the graph's mean out-degree.
__host__ __device__ __forceinline__ uint32_t solo_items(int64_t n, int64_t m) {
    const int64_t mean = m / (n > 0 ? n : 1) + 1;
    const int64_t k = static_cast<int64_t>(kSoloEdges) / mean;
    return static_cast<uint32_t>(k < 1 ? 1 : (k > kSoloItems ? kSoloItems : k));
}

// Pushes of a solo run: the next worklist in LDS (what does not fit goes to
// the outgoing worklist in memory), the far list in memory with its counter
// in LDS.
struct SoloPushers {
    int *list;
    uint32_t list_cap;
    uint32_t *cnt;
    int32_t *out;
    uint32_t cap;
    int32_t *far_out;
    uint32_t *far_cnt;
    uint32_t far_cap;
    Sink sk;  // the control block that errors go to
    uint32_t fmin = kInf;
    const int32_t *deg_rp = nullptr;
    unsigned long long mf = 0;
    uint32_t tries = 0;
    uint32_t wins = 0;
    // Positions of the lanes' items: one LDS atomic per wavefront for all U.
    template <int U>
    __device__ __forceinline__ bool reserve(const bool (&p)[U], uint32_t (&at)[U], uint32_t *c) {
        uint32_t total = 0;
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const unsigned long long m = __ballot(p[k]);
            at[k] = total + lane_rank(m);
            total += static_cast<uint32_t>(__popcll(m));
        }
        if (total == 0) return false;  // uniform across the wavefront
        uint32_t base = 0;
        if (lane_id() == 0) base = atomicAdd(c, total);
        base = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(base)));
#pragma unroll
        for (int k = 0; k < U; ++k) at[k] += base;
        return true;
    }
    template <int U>
    __device__ __forceinline__ void push_near(const bool (&p)[U], const int (&item)[U]) {
        uint32_t at[U];
        if (!reserve(p, at, cnt)) return;
#pragma unroll
        for (int k = 0; k < U; ++k) {
            if (!p[k]) continue;
            if (at[k] < list_cap) list[at[k]] = item[k];
            else if (at[k] < cap) out[at[k]] = item[k];
            else set_error(sk.ctrl, kErrOverflow, false);
        }
    }
    template <int U>
    __device__ __forceinline__ void push_far(const bool (&p)[U], const int (&item)[U]) {
        uint32_t at[U];
        if (!reserve(p, at, far_cnt)) return;
#pragma unroll
        for (int k = 0; k < U; ++k) {
            if (!p[k]) continue;
            if (at[k] < far_cap) far_out[at[k]] = item[k];
            else set_error(sk.ctrl, kErrOverflow, false);
        }
    }
    __device__ __forceinline__ void near(bool p, int item) {
        const bool ps[1] = {p};
        const int is[1] = {item};
        push_near(ps, is);
    }
    __device__ __forceinline__ void far(bool p, int item) {
        const bool ps[1] = {p};
        const int is[1] = {item};
        push_far(ps, is);
    }
};

// Loop state that a solo run continues from and leaves behind.
struct SoloState {
    uint32_t it, tr, thresh;
    unsigned long long items, m_seen;
    uint32_t max_frontier;
};

// Run solo invocations from the worklist `in` of cnt_in vertices (which every
// workgroup found small enough) and leave the worklist they end with in
// `out`.  All threads of the workgroup call it.  Returns the items left;
// `edges` grows by this thread's share of the scanned edges.  trace_begin(it,
// items) says whether an invocation is traced, trace_end(it, edges scanned by
// this thread so far, busy ticks, pushers) records it.  `until`: the
// wall-clock tick that ends the run.
template <int B, class Op, class MakeOp, class Begin, class End>
__device__ __forceinline__ uint32_t solo_run(const int32_t *in, uint32_t cnt_in, int32_t *out, uint32_t cap,
                                             uint32_t n, const int32_t *__restrict__ row_ptr,
                                             const int32_t *__restrict__ col, uint32_t *val, uint32_t *expd,
                                             uint32_t *far_flag, uint32_t *stamp, int32_t *far0, int32_t *far1,
                                             uint32_t far_cap, uint32_t delta, uint32_t max_iter, Ctrl *ctrl,
                                             Smem<B> &sm, SoloState &st, unsigned long long &edges,
                                             unsigned long long until, MakeOp make, Begin trace_begin,
                                             End trace_end) {
    constexpr int kU = 4;
    constexpr int J = kSoloPer;
    constexpr int kWaves = B / kWave < kSoloWaves ? B / kWave : kSoloWaves;
    constexpr uint32_t kThreads = kWaves * kWave;
    constexpr uint32_t kItems = kThreads * kSoloPer;
    constexpr uint32_t kList = 4 * B;
    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int wid = tid / kWave;
    const bool works = wid < kWaves;  // the other wavefronts only keep the barriers
    __syncthreads();  // the queues' space is free: every wavefront has drained its own
    for (uint32_t i = tid; i < cnt_in; i += B) sm.solo[0][i] = in[i];
    if (tid == 0) {
        sm.solo_cnt[0] = cnt_in;
        sm.solo_cnt[1] = 0u;
        sm.solo_sum = 0ull;
        sm.solo_steps = kSoloSteps;
        sm.solo_until = until;
        if (Op::kFar) {
            sm.solo_far[st.tr & 1u] = min(load_agent(&ctrl->far_cnt[st.tr % 3]), far_cap);
            sm.solo_fmin[st.tr & 1u] = load_agent(&ctrl->far_min[st.tr % 3]);
            sm.solo_far[(st.tr & 1u) ^ 1u] = 0u;
            sm.solo_fmin[(st.tr & 1u) ^ 1u] = kInf;
        }
    }
    SoloPushers pu{nullptr, min(kList, cap), nullptr, out, cap, nullptr, nullptr, far_cap,
                   Sink{nullptr, nullptr, cap, ctrl, nullptr}};
    uint32_t step = 0, cnt = 0;
    __syncthreads();
    for (;; ++step) {
        const uint32_t most = sm.solo_steps;
        cnt = min(sm.solo_cnt[step % 3], cap);
        uint32_t far_n = 0;
        if (cnt == 0) {
            if (!Op::kFar) break;
            far_n = min(sm.solo_far[st.tr & 1u], far_cap);
            if (far_n == 0 || far_n > kSoloFar) break;
        }
        if (cnt > kItems || st.it >= max_iter || step >= most) break;
        if (tid == 0) sm.solo_cnt[(step + 2) % 3] = 0u;
        const bool traced = trace_begin(st.it, cnt);
        const unsigned long long t0 = traced ? wall_clock64() : 0ull;
        pu.list = sm.solo[(step & 1u) ^ 1u];
        pu.cnt = &sm.solo_cnt[(step + 1) % 3];
        if (cnt == 0) {
            if constexpr (Op::kFar) {
                // transfer: far list tr -> next worklist / far list tr + 1
                const uint32_t lo = max(st.thresh, sm.solo_fmin[st.tr & 1u]);
                const uint32_t t_new = lo >= kInf - delta ? kInf : lo + delta;
                const uint32_t nx = (st.tr & 1u) ^ 1u;
                pu.far_out = nx ? far1 : far0;
                pu.far_cnt = &sm.solo_far[nx];
                far_transfer<B>((st.tr & 1u) ? far1 : far0, far_n, n, st.thresh, t_new, val, far_flag, stamp, st.it,
                                pu, Team{0u, 1u});
                __syncthreads();  // the old list has been read
                if (tid == 0) {
                    sm.solo_far[st.tr & 1u] = 0u;
                    sm.solo_fmin[st.tr & 1u] = kInf;
                }
                st.thresh = t_new;
                ++st.tr;
            }
        } else {
            // look up every item at once; nothing is changed before the
            // worklist is known to be small enough
            const bool mine = works && static_cast<uint32_t>(wid) * kWave < cnt;  // uniform across the wavefront
            int v[J], r0[J], r1[J];
            uint32_t dv[J], last[J];
            bool wide = false;
            if (mine) {
                const int *const list = sm.solo[step & 1u];
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    const uint32_t i = static_cast<uint32_t>(j) * kThreads + static_cast<uint32_t>(tid);
                    v[j] = i < cnt ? list[i] : -1;
                    if (i < cnt && static_cast<uint32_t>(v[j]) >= n) {  // never expected: a corrupt worklist entry
                        set_error(ctrl, kErrInternal, false);
                        v[j] = -1;
                    }
                    r0[j] = r1[j] = 0;
                    dv[j] = 0u;
                    last[j] = kInf;
                    if (v[j] >= 0) {
                        r0[j] = row_ptr[v[j]];
                        r1[j] = row_ptr[v[j] + 1];
                        if (Op::kFar) {
                            dv[j] = __hip_atomic_load(&val[v[j]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                            last[j] = expd[v[j]];
                        }
                    }
                }
                phase(r0);
                phase(r1);
                int total = 0;
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    // SSSP: expanded at this distance before: nothing to relax
                    if (Op::kFar && v[j] >= 0 && last[j] == dv[j]) r1[j] = r0[j];
                    // a row beyond the edge limit counts as the limit + 1, so the sum fits
                    total += min(r1[j] - r0[j], static_cast<int>(kSoloEdges) + 1);
                    wide |= r1[j] - r0[j] > kSoloRow;
                }
                total = wave_inclusive_scan(total);
                if (lane == kWave - 1) sm.wsum[wid] = total;
            } else if (works && lane == 0) {
                sm.wsum[wid] = 0;
            }
            __syncthreads();
            int all = 0;
#pragma unroll
            for (int k = 0; k < kWaves; ++k) all += sm.wsum[k];
            if (static_cast<uint32_t>(all) > kSoloEdges) break;  // uniform: the team takes it
            if (mine) {
                const Op op = make(st.it, st.thresh, st.tr);
                if (Op::kFar) {
                    pu.far_out = (st.tr & 1u) ? far1 : far0;
                    pu.far_cnt = &sm.solo_far[st.tr & 1u];
                }
                const bool gather = __ballot(wide) != 0ull;
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    const int deg = r1[j] - r0[j];
                    if (Op::kFar && deg > 0) expd[v[j]] = dv[j];
                    edges += static_cast<unsigned long long>(deg);
                    if (!gather) {
                        // short rows: each thread walks its own
                        for (int x = 0; __ballot(x < deg) != 0ull; x += kU) {
                            int e[kU], sv[kU];
                            uint32_t sval[kU];
                            bool act[kU];
#pragma unroll
                            for (int k = 0; k < kU; ++k) {
                                act[k] = x + k < deg;
                                e[k] = act[k] ? r0[j] + x + k : 0;
                                sv[k] = v[j];
                                sval[k] = dv[j];
                            }
                            relax_and_push<kU>(op, col, e, act, sv, sval, pu);
                        }
                    } else {
                        // the wavefront's rows, concatenated and dealt to its
                        // lanes (the gather tier of expand() in one wavefront)
                        const int inc = wave_inclusive_scan(deg);
                        const int total = __builtin_amdgcn_readlane(inc, kWave - 1);
                        __builtin_amdgcn_wave_barrier();
                        sm.gstart[tid] = inc - deg;
                        sm.gr0[tid] = r0[j];
                        sm.vtx[tid] = v[j];
                        sm.vval[tid] = dv[j];
                        __builtin_amdgcn_wave_barrier();
                        for (int done = 0; done < total; done += kWave * kU) {
                            int e[kU], sv[kU];
                            uint32_t sval[kU];
                            bool act[kU];
#pragma unroll
                            for (int k = 0; k < kU; ++k) {
                                const int slot = done + k * kWave + lane;
                                act[k] = slot < total;
                                int o = wid * kWave;
#pragma unroll
                                for (int s = kWave / 2; s > 0; s >>= 1)
                                    if (sm.gstart[o + s] <= slot) o += s;
                                e[k] = act[k] ? sm.gr0[o] + (slot - sm.gstart[o]) : 0;
                                sv[k] = sm.vtx[o];
                                sval[k] = sm.vval[o];
                            }
                            relax_and_push<kU>(op, col, e, act, sv, sval, pu);
                        }
                    }
                }
            }
            st.m_seen += static_cast<unsigned long long>(all);
            st.items += cnt;
            st.max_frontier = max(st.max_frontier, cnt);
            if (traced) trace_end(st.it, edges, wall_clock64() - t0, pu);
        }
        if (Op::kFar && __ballot(pu.fmin != kInf) != 0ull) {
            uint32_t m = pu.fmin;
#pragma unroll
            for (int d = 1; d < kWave; d <<= 1) m = min(m, static_cast<uint32_t>(__shfl_xor(m, d, kWave)));
            if (lane == 0) atomicMin(&sm.solo_fmin[st.tr & 1u], m);
            pu.fmin = kInf;
        }
        ++st.it;
        if (step % kSoloClock == kSoloClock - 1 && tid == 0 && wall_clock64() > sm.solo_until) sm.solo_steps = 0u;
        __syncthreads();
    }
    // what is left: the worklist to memory, the counters to the control block
    const uint32_t have = min(cnt, min(kList, cap));
    unsigned long long deg = 0;
    for (uint32_t i = tid; i < cnt; i += B) {
        const int x = i < have ? sm.solo[step & 1u][i] : out[i];
        if (i < have) out[i] = x;
        if (!Op::kFar && static_cast<uint32_t>(x) < n) deg += static_cast<unsigned long long>(row_ptr[x + 1] - row_ptr[x]);
    }
    if (deg) atomicAdd(&sm.solo_sum, deg);
    __syncthreads();  // solo_sum is complete; the queues' space may be used again
    return cnt;
}

}  // namespace irgl
