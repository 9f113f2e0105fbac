// Level-scheduled triangular solves (Sec. 2.6, Alg. 3), as one persistent
// launch per triangle in which rows of successive levels are solved inside a
// workgroup with their dependencies held in LDS.
//
// Plan (built once per factor on the host by plan.hpp's make_plan):
//  * the rows are cut into parts: x-y tiles spanning all z for a recognised
//    grid stencil, otherwise contiguous row ranges, numbered in the order the
//    triangle is solved. Every dependency of a row lies in its own part or in an
//    earlier part, so the parts can be claimed in order from a ticket counter:
//    a part only ever waits for parts already claimed by running workgroups,
//    hence no deadlock at any occupancy or grid size;
//  * inside a part the rows are laid out by (level, row) (Alg. 3's order) and
//    cut into sub-segments of at most 64 rows of one level.
//
// Execution (k_trsv_blk): one workgroup per part: solver wavefronts (one by
// default), a writer wavefront and prefetching wavefronts.
//  * Prefetchers stream the next sub-segments into a ring of LDS slots: the
//    right-hand side (gathered by row, or read in plan order for the upper
//    solve of an L-then-U chain), the row's entries, and the values of
//    dependencies in earlier parts, polled from global memory until final;
//  * the solver takes sub-segments in order, reads dependencies inside the part
//    from a small LDS ring of recent results and dependencies outside it from
//    the slot, and publishes each result to the polled copy (below). It never
//    waits on global memory itself;
//  * the writer copies the part's results from the polled copy to the outputs
//    by row or in the other triangle's order, scattered stores kept off the
//    solver's path.
//  * Every wait is bounded: a wave that has polled `spin` times (the limit set by
//    hec_set_spin_limit) gives up, records the failure in the schedule's error
//    word and in its workgroup's abort flag, and every wave then leaves its loops
//    and the launch ends normally, with garbage in its outputs; the host reports
//    the failure (HEC_ERR_TIMEOUT) at its next synchronisation. Only a broken plan,
//    a lost store or a misuse (two streams on one schedule) can get there.
//  * Readiness of a value across parts is the value itself: each triangle
//    keeps an internal copy of its results in plan order, pre-filled with a
//    signalling-NaN bit pattern that arithmetic never produces; results are
//    stored to it and polled from it with device-coherent (agent scope)
//    accesses, so only single-location coherence is needed and no cache-wide
//    fence is issued. A sub-segment's results are 64 consecutive positions, so
//    these stores are whole cache lines; the outputs by row (or in the other
//    triangle's order) are plain stores. In an L-then-U chain the lower launch
//    fills the upper solve's copy and the upper launch refills the lower one
//    for the next chain, so the chain is exactly two launches.
#include <algorithm>
#include <climits>
#include <cmath>
#include <type_traits>

#include "hec_internal.hpp"

namespace hec {

namespace {

constexpr int kWaves = 16;  // solver wavefronts first, then prefetching wavefronts, the writer last
constexpr int kWriterBatch = 8;  // sub-segments' worth of positions the writer copies at a time
constexpr int kBlkThreads = 64 * kWaves;
constexpr int kBatch = 8;           // entries loaded per batch by a prefetcher lane
using plan::kPad;
using plan::kSub;
using plan::align16;
using plan::ctrl_bytes;
using plan::ctrl_head;
using plan::lds_bytes;
using plan::Slot;

template <class T> struct Sentinel;
template <> struct Sentinel<double> {
    using U = unsigned long long;
    static constexpr U bits = 0x7FF4DEADBEEF1234ull;  // signalling NaN: never produced by arithmetic
    static constexpr U qnan = 0x7FF8000000000000ull;
};
template <> struct Sentinel<float> {
    using U = unsigned int;
    static constexpr U bits = 0x7FA0BEEFu;
    static constexpr U qnan = 0x7FC00000u;
};

template <class T>
__device__ __forceinline__ typename Sentinel<T>::U load_coherent(const T *p) {
    using U = typename Sentinel<T>::U;
    return __hip_atomic_load((U *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Publishes a solved value. A right-hand side that carries the sentinel's own
// bit pattern (and reaches the output untouched by arithmetic) is replaced by
// a quiet NaN, so no waiting row can mistake a final value for "not ready".
template <class T>
__device__ __forceinline__ void store_coherent(T *p, T v) {
    using U = typename Sentinel<T>::U;
    U u;
    __builtin_memcpy(&u, &v, sizeof(T));
    if (u == Sentinel<T>::bits) u = Sentinel<T>::qnan;
    __hip_atomic_store((U *)p, u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <class T>
__device__ __forceinline__ T from_bits(typename Sentinel<T>::U u) {
    T v;
    __builtin_memcpy(&v, &u, sizeof(T));
    return v;
}

// Vectors of one triangular solve. b: right-hand side, read at bmap[q] for
// position q when bmap is given, else by row (b_by_row) or in plan order; xq:
// the results in plan order, the copy dependent rows poll (pre-filled with the
// sentinel); x: optional output by row; yother: optional output at the plan's
// per-position index (`other`, -1: not written) -- the other triangle's plan
// order, or a caller's vector; fill: a vector of nfill elements the kernel sets
// to the sentinel for the next solve (the polled copy of the other triangle of
// an L-then-U chain).
template <class T>
struct SolveIO {
    const T *b;
    const int32_t *bmap;
    int32_t b_by_row;
    T *xq, *x, *yother, *fill;
    int64_t nfill;
};

// Sets io.fill to the sentinel: a grid-stride loop at kernel start.
template <class T>
__device__ __forceinline__ void fill_sentinel(const SolveIO<T> &io) {
    if (!io.fill) return;
    const T s = from_bits<T>(Sentinel<T>::bits);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < io.nfill; i += (int64_t)gridDim.x * blockDim.x)
        io.fill[i] = s;
}

struct PlanArgs {
    int32_t nparts, K, ldq, W, D, S;  // S: most sub-segments in one part
    const int32_t *part_ss, *part_pos, *ss_pos, *ss_need, *grow, *other, *enc;
    uint32_t *err;  // the schedule's error word: set when a wait gives up
    uint32_t spin;  // polls a wait makes before it gives up
};

// Records a wait that gave up: the schedule's error word (read by the host).
__device__ __forceinline__ void record_timeout(uint32_t *err) {
    __hip_atomic_store(err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Another wave gave up somewhere on the device (checked now and then by long waits).
__device__ __forceinline__ bool timed_out(const uint32_t *err) {
    return __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u;
}

// First poll of a dependency outside the part: only lanes whose entry has one
// load (a lane-masked load); the others get 0, which is never the sentinel. (A
// shared dummy address for those lanes would send a device-coherent load per
// wavefront and entry to one cache line from every compute unit: a hot spot that
// slows every access mapped to the same memory channel.)
template <class T>
__device__ __forceinline__ typename Sentinel<T>::U first_poll(const T *x, int e) {
    return e >= 0 ? load_coherent(x + e) : (typename Sentinel<T>::U)0;
}

template <class T, bool UPPER, int KC, int NS>
__global__ __launch_bounds__(kBlkThreads) void k_trsv_blk(PlanArgs P, const T *__restrict__ val,
                                                          const T *__restrict__ piv, SolveIO<T> io,
                                                          uint32_t *sync, const int32_t *skip) {
    using U = typename Sentinel<T>::U;
    constexpr U SENT = Sentinel<T>::bits;
    if (skip && *skip) return;  // uniform: no workgroup touches the counters
    fill_sentinel(io);
    T *const xq = io.xq;
    T *const x = io.x;
    T *const yother = io.yother;
    extern __shared__ __align__(16) char smem[];
    constexpr int NP = kWaves - NS - 1;
    const int D = P.D, K = P.K, W = P.W;
    int *done = (int *)smem;  // per solver wavefront: the next sub-segment it solves
    int *filled = done + plan::kMaxSolvers;
    int *s_part = filled + D;
    int *s_abort = s_part + 1;  // a wave of this workgroup gave up a wait
    const uint32_t zero_off = (uint32_t)(ctrl_head(D) - 16);
    int *sspos = (int *)(smem + ctrl_head(D));
    int *ssneed = (int *)(smem + ctrl_head(D) + plan::ss_bytes(P.S));
    const uint32_t sx_off = (uint32_t)ctrl_bytes(D, P.S, NS);
    T *sx = (T *)(smem + sx_off);
    const uint32_t slots_off = sx_off + (uint32_t)align16((size_t)W * sizeof(T));
    const Slot<T, UPPER> L{KC};
    const uint32_t sb = (uint32_t)L.bytes();
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    if (threadIdx.x < 4) ((int *)(smem + zero_off))[threadIdx.x] = 0;
    if (threadIdx.x == 0) *s_abort = 0;
    // every slot's dependency addresses start at the zero word: a solver that gave up a
    // wait may still read the header of a slot that was never filled (the reads stay in
    // range; nothing it computes is published)
    for (int t = threadIdx.x; t < D * KC * kSub; t += blockDim.x)
        ((uint32_t *)(smem + slots_off + (t / (KC * kSub)) * sb + L.a()))[t % (KC * kSub)] = zero_off;
    // A wait that has spun `spin` times gives up: it marks the workgroup and the device.
    // Waves of the workgroup see the mark within 64 polls; other workgroups' long polls
    // look at the device's error word as often.
    // (every calling lane stores the mark: callers are wave-uniform, so lane 0 may not be among them)
    auto give_up = [&]() {
        __hip_atomic_store(s_abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        record_timeout(P.err);
    };
    auto wg_aborted = [&]() { return __hip_atomic_load(s_abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != 0; };
    // one more poll of a wait: true when the wait must stop (given up here or elsewhere).
    // Called in wave-uniform control flow only, so a wave stops as a whole; the answer
    // is made a scalar (read from the first lane) so that the compiler keeps the loops
    // and flags that depend on it uniform (scalar branches, no exec-mask bookkeeping)
    auto spun_out = [&](uint32_t &it, bool device_wide) {
        ++it;
        bool stop = it > P.spin;
        if (!stop && (it & 63) == 0) stop = wg_aborted() || (device_wide && timed_out(P.err));
        stop = __builtin_amdgcn_readfirstlane((int)stop) != 0;
        if (stop) give_up();
        return stop;
    };

    for (;;) {
        __syncthreads();
        if (*s_abort) break;  // uniform: read by every thread after the barrier
        if (threadIdx.x == 0) *s_part = (int)atomicAdd(&sync[0], 1u);
        if ((int)threadIdx.x < plan::kMaxSolvers) done[threadIdx.x] = (int)threadIdx.x < NS ? (int)threadIdx.x : INT_MAX;
        if ((int)threadIdx.x < D) filled[threadIdx.x] = -1;
        __syncthreads();
        const int p = *s_part;
        if (p >= P.nparts) break;
        const int kb = P.part_ss[p], nss = P.part_ss[p + 1] - kb, pos0 = P.part_pos[p];
        for (int t = threadIdx.x; t <= nss; t += blockDim.x) {
            sspos[t] = P.ss_pos[kb + t];
            if constexpr (NS > 1)
                if (t < nss) ssneed[t] = P.ss_need[kb + t];
        }
        __syncthreads();

        if (wave < NS) {
            // ---------------- solvers: one LDS round trip and KC fused multiply-adds per row.
            // Solver wavefront w takes the part's sub-segments w, w + NS, ...; with NS > 1 a
            // sub-segment first waits until every sub-segment below its dependency bound is
            // solved (the `done` counters), which orders its reads of the ring of results
            // after their writes. The next own sub-segment's header and dependency
            // addresses are read while the current one is computed (two register sets used
            // alternately), so the only dependent LDS access of a step is the read of its
            // dependencies' values.
            __builtin_amdgcn_s_setprio(3);
            struct Head {
                T b, d;
                int q0, cnt, need;
                uint32_t ad[KC];
            };
            const int w0 = wave;
            auto adv = [&](int sl) {  // slot of the next own sub-segment (NS <= D)
                sl += NS;
                return sl >= D ? sl - D : sl;
            };
            int ready = w0;  // own sub-segments below `ready` are known to be filled
            bool bail = false;  // a wait gave up: stop taking sub-segments
            // Waits until own sub-segment r (in slot sl) is filled; returns one past the
            // run of consecutive own filled sub-segments starting at r (at most 8 looked
            // at). Lane u reads the flag of own sub-segment r + u*NS, so the eight flags
            // take one LDS round trip; relaxed loads suffice: a slot's contents are
            // complete before its flag is written (the prefetcher waits for its LDS
            // writes first), LDS accesses of one wavefront complete in order, and the
            // signal fence keeps the compiler from moving slot reads above the check.
            auto scan = [&](int r, int sl) -> int {
                const int u = lane & 7, want = r + u * NS;
                int s2 = sl + u * NS;
                s2 -= D * (int)((unsigned)s2 / (unsigned)D);
                uint32_t it = 0;
                for (;;) {
                    const int f = __hip_atomic_load(&filled[s2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    const uint64_t m = __ballot(lane < 8 && want < nss && f == want);
                    const int ok = __builtin_ctzll(~m);  // own filled sub-segments r, r + NS, ... in a row
                    if (ok > 0) {
                        __atomic_signal_fence(__ATOMIC_SEQ_CST);
                        return r + ok * NS;
                    }
                    if (spun_out(it, false)) {
                        bail = true;
                        return r;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
            };
            // With several solvers: waits until every sub-segment below `need` is solved.
            // done[v] only grows and holds the next sub-segment solver v takes, so all below
            // `need` are solved once every counter reaches it (unused counters hold
            // INT_MAX; lane v reads counter v & 7). Relaxed loads suffice as in scan.
            auto wait_need = [&](int need) {
                if constexpr (NS == 1) return;  // one solver: its own earlier sub-segments are solved
                const int v = lane & (plan::kMaxSolvers - 1);
                uint32_t it = 0;
                for (;;) {
                    const int dv = __hip_atomic_load(&done[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    if (__ballot(dv < need) == 0) break;
                    if (spun_out(it, false)) {
                        bail = true;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
                __atomic_signal_fence(__ATOMIC_SEQ_CST);
            };
            auto load_head = [&](int r, int sl, Head &H) {
                const char *p2 = smem + slots_off + sl * sb;
                H.q0 = sspos[r];
                H.cnt = sspos[r + 1] - H.q0;
                H.need = 0;
                if constexpr (NS > 1) H.need = ssneed[r];
                H.b = ((const T *)(p2 + L.b()))[lane];
                H.d = (T)1;
                if constexpr (UPPER) H.d = ((const T *)(p2 + L.d()))[lane];
#pragma unroll
                for (int u = 0; u < KC; ++u) H.ad[u] = ((const uint32_t *)(p2 + L.a()))[u * kSub + lane];
            };
            // Two register sets fit the 128-VGPR budget of a 1024-thread workgroup for
            // rows of up to 64 bytes of values; longer rows load the next header after
            // the step instead (nxt is then cur).
            constexpr bool kPipe = KC * sizeof(T) <= 64;
            // One sub-segment: cur is loaded; nxt receives own sub-segment rel + NS.
            auto step = [&](int rel, int slot, Head &cur, Head &nxt) {
                const int nslot = adv(slot);
                const char *p2 = smem + slots_off + slot * sb;
                const bool pre = kPipe && rel + NS < ready;
                T acc = cur.b;
                // entries in chunks of at most 8 (bounds the live registers of long rows)
                constexpr int CH = KC < 8 ? KC : 8;
#pragma unroll
                for (int c0 = 0; c0 < KC; c0 += CH) {
                    T xv[CH], av[CH];
#pragma unroll
                    for (int u = 0; u < CH; ++u) av[u] = ((const T *)(p2 + L.v()))[(c0 + u) * kSub + lane];
                    if (c0 == 0) wait_need(cur.need);
#pragma unroll
                    for (int u = 0; u < CH; ++u) xv[u] = *(const T *)(smem + cur.ad[c0 + u]);
                    if (c0 == 0 && pre) load_head(rel + NS, nslot, nxt);
#pragma unroll
                    for (int u = 0; u < CH; ++u) acc -= av[u] * xv[u];
                }
                if constexpr (UPPER) acc = acc * cur.d;  // the pivot's reciprocal, formed by the prefetcher
                if (lane < cur.cnt && !bail) {  // (after a give-up nothing more is published)
                    sx[(cur.q0 - pos0 + lane) & (W - 1)] = acc;
                    store_coherent(xq + cur.q0 + lane, acc);
                }
                // publish: the results in the ring are readable and the slot is free. A lone
                // solver releases every 4 sub-segments (only prefetchers wait on it).
                if (NS > 1 || (rel & 3) == 3 || rel + NS >= nss) {
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                    if (lane == 0) __hip_atomic_store(&done[w0], rel + NS, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
                if (kPipe && !pre && rel + NS < nss) {
                    ready = scan(rel + NS, nslot);
                    load_head(rel + NS, nslot, nxt);  // (after a give-up: read, never used)
                }
                return nslot;
            };
            int slot = w0 % D;
            if constexpr (kPipe) {
                // A give-up is looked at once per pair of steps: the data flow between the
                // two register sets stays the same on every path (a check between the
                // steps made the compiler copy one set into the other, measured 7% slower
                // on the 128^3 pair); the second step of a pair then publishes nothing.
                Head h0, h1;
                if (w0 < nss) {
                    ready = scan(w0, slot);
                    load_head(w0, slot, h0);
                }
                for (int rel = w0; rel < nss && !bail; rel += 2 * NS) {
                    slot = step(rel, slot, h0, h1);
                    if (rel + NS < nss) slot = step(rel + NS, slot, h1, h0);
                }
            } else {
                for (int rel = w0; rel < nss; rel += NS) {
                    if (rel >= ready) ready = scan(rel, slot);
                    if (bail) break;
                    Head h;
                    load_head(rel, slot, h);
                    slot = step(rel, slot, h, h);
                }
            }
            __builtin_amdgcn_s_setprio(0);
        } else if (wave == kWaves - 1) {
            // ---------------- writer: the part's results go to the outputs by row (x) and in the
            // other order (yother), read back from the polled copy, where a final value is
            // its own ready flag. The part's positions are consecutive; each lane takes
            // every 64th of kWriterBatch * 64 at a time, once the solvers' progress counters
            // have passed them.
            if (x || yother) {
                const int pend_part = P.part_pos[p + 1];
                constexpr int WB = kWriterBatch;
                for (int c = pos0; c < pend_part; c += WB * kSub) {
                    const int cend = min(c + WB * kSub, pend_part);
                    U v[WB];
                    int gi[WB], po[WB];
#pragma unroll
                    for (int k = 0; k < WB; ++k) {
                        const int q = c + k * kSub + lane;
                        const bool live = q < cend;
                        gi[k] = live && x ? P.grow[q] : -1;
                        po[k] = live && yother && P.other ? P.other[q] : -1;
                        v[k] = live ? SENT : (U)0;
                    }
                    bool quit = false;
                    uint32_t it = 0;
                    for (;;) {  // all sub-segments below the smallest counter are solved
                        int m = INT_MAX;
#pragma unroll
                        for (int u = 0; u < plan::kMaxSolvers; ++u)
                            m = min(m, __hip_atomic_load(&done[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
                        if (sspos[min(m, nss)] >= cend) break;
                        if (spun_out(it, false)) {
                            quit = true;
                            break;
                        }
                        __builtin_amdgcn_s_sleep(8);
                    }
                    if (quit) break;
                    bool pend = true;
                    it = 0;
                    while (pend) {  // the solvers' coherent stores may still be on their way
#pragma unroll
                        for (int k = 0; k < WB; ++k)
                            if (v[k] == SENT) v[k] = load_coherent(xq + c + k * kSub + lane);
                        bool mine = false;
#pragma unroll
                        for (int k = 0; k < WB; ++k) mine |= v[k] == SENT;
                        pend = __ballot(mine) != 0;  // uniform: the wave waits as a whole
                        if (pend && spun_out(it, true)) {
                            quit = true;
                            break;
                        }
                        if (pend) __builtin_amdgcn_s_sleep(2);
                    }
                    if (quit) break;
#pragma unroll
                    for (int k = 0; k < WB; ++k) {
                        const T r = from_bits<T>(v[k]);
                        if (gi[k] >= 0) x[gi[k]] = r;
                        if (po[k] >= 0) yother[po[k]] = r;
                    }
                }
            }
        } else {
            // ---------------- prefetchers: every lane of a slot is written (idle lanes get padding)
            // Each prefetching wavefront keeps two of its sub-segments in flight: while
            // the right-hand side and the polls of one are outstanding, the row data and
            // first entries of its next one (NP later) are already loading.
            // Only the LDS writes wait for the solver to release the slot.
            constexpr int B = KC < kBatch ? KC : kBatch;
            constexpr bool kPfPipe = KC == 4;  // two register sets fit the 128-VGPR budget for short rows only
            struct Pre {
                int q0, cnt, gi, po;
                T dd;
                int es[B];
                T vs[B];
            };
            auto issue = [&](int r, Pre &R) {  // everything indexed by position: one round trip
                R.q0 = sspos[r];
                R.cnt = sspos[r + 1] - R.q0;
                const bool live = lane < R.cnt;
                const int q = R.q0 + (live ? lane : 0);
                R.gi = live && io.b_by_row && !io.bmap ? P.grow[q] : 0;
                // upper: the reciprocal of u_ii (correctly rounded), so that the solver's
                // step multiplies instead of dividing; the result is within about one
                // rounding of the quotient
                R.dd = (T)1;
                if constexpr (UPPER) R.dd = live ? (T)1 / piv[q] : (T)1;
#pragma unroll
                for (int u = 0; u < B; ++u) {
                    R.es[u] = kPad;
                    R.vs[u] = (T)0;
                    if (live && u < K) {
                        R.es[u] = P.enc[(size_t)u * P.ldq + q];
                        R.vs[u] = val[(size_t)u * P.ldq + q];
                    }
                }
            };
            // every lane polls all its entries at once; entries without an outside
            // dependency read a constant zero. A repeated poll reloads only the entries
            // still pending (a load per entry and lane that is already final, or that
            // has no outside dependency, was measured slower: 420 against 353 us for the
            // 128^3 pair, the extra device-coherent loads crowding the memory side)
            bool quit = false;  // a wait gave up: stop filling slots
            auto poll = [&](const int (&es)[B], U (&xs)[B]) {
                bool pend = false;
#pragma unroll
                for (int u = 0; u < B; ++u) pend |= xs[u] == SENT;
                uint32_t it = 0;
                while (__ballot(pend) != 0) {  // uniform: the wave polls as a whole
                    if (spun_out(it, true)) {
                        quit = true;
                        return;
                    }
                    __builtin_amdgcn_s_sleep(1);
#pragma unroll
                    for (int u = 0; u < B; ++u)
                        if (xs[u] == SENT) xs[u] = load_coherent(xq + es[u]);
                    pend = false;
#pragma unroll
                    for (int u = 0; u < B; ++u) pend |= xs[u] == SENT;
                }
            };
            // entries and dependency addresses (known before any poll completes)
            auto put = [&](char *sl, uint32_t so, int s0, const int (&es)[B], const T (&vs)[B]) {
#pragma unroll
                for (int u = 0; u < B; ++u) {
                    const int s = s0 + u;
                    const uint32_t xe_at = so + (uint32_t)(L.xe() + (size_t)(s * kSub + lane) * sizeof(T));
                    uint32_t at = zero_off;  // padding: value 0 times a zero
                    if (es[u] >= 0) at = xe_at;
                    else if (es[u] != kPad) at = sx_off + (uint32_t)(((-1 - es[u]) & (W - 1)) * sizeof(T));
                    ((uint32_t *)(sl + L.a()))[s * kSub + lane] = at;
                    ((T *)(sl + L.v()))[s * kSub + lane] = vs[u];
                }
            };
            // the polled values of dependencies outside the part (other entries never read theirs)
            auto put_xe = [&](char *sl, int s0, const int (&es)[B], const U (&xs)[B]) {
#pragma unroll
                for (int u = 0; u < B; ++u)
                    if (es[u] >= 0) ((T *)(sl + L.xe()))[(s0 + u) * kSub + lane] = from_bits<T>(xs[u]);
            };
            auto process = [&](int rel, Pre &cur, Pre &nxt) {
                const int slot = rel % D;
                const uint32_t so = slots_off + slot * sb;
                char *sl = smem + so;
                const bool live = lane < cur.cnt;
                const int q = cur.q0 + (live ? lane : 0);
                const T bb = live ? io.b[io.bmap ? io.bmap[q] : io.b_by_row ? cur.gi : q] : (T)0;
                U xs[B];
#pragma unroll
                for (int u = 0; u < B; ++u) xs[u] = first_poll(xq, cur.es[u]);
                if (kPfPipe && rel + NP < nss) issue(rel + NP, nxt);
                // the slot's previous sub-segment, rel - D, must be solved; everything but the
                // outside values goes in before the polls, so that only those and the flag
                // follow the last poll
                const int prev = rel - D;
                if (prev >= 0) {
                    uint32_t it = 0;
                    while (__hip_atomic_load(&done[prev & (NS - 1)], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) <= prev) {
                        if (spun_out(it, false)) {
                            quit = true;
                            return;
                        }
                        __builtin_amdgcn_s_sleep(4);
                    }
                }
                put(sl, so, 0, cur.es, cur.vs);
                ((T *)(sl + L.b()))[lane] = bb;
                if constexpr (UPPER) ((T *)(sl + L.d()))[lane] = cur.dd;
                poll(cur.es, xs);
                if (quit) return;
                put_xe(sl, 0, cur.es, xs);
                for (int s0 = B; s0 < KC; s0 += B) {  // rows longer than one batch
                    int es[B];
                    T vs[B];
#pragma unroll
                    for (int u = 0; u < B; ++u) {
                        es[u] = kPad;
                        vs[u] = (T)0;
                        if (live && s0 + u < K) {
                            es[u] = P.enc[(size_t)(s0 + u) * P.ldq + q];
                            vs[u] = val[(size_t)(s0 + u) * P.ldq + q];
                        }
                    }
                    U xs2[B];
#pragma unroll
                    for (int u = 0; u < B; ++u) xs2[u] = first_poll(xq, es[u]);
                    put(sl, so, s0, es, vs);
                    poll(es, xs2);
                    if (quit) return;
                    put_xe(sl, s0, es, xs2);
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                if (lane == 0) __hip_atomic_store(&filled[slot], rel, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
            };
            const int w = wave - NS;
            if constexpr (kPfPipe) {
                Pre p0, p1;
                if (w < nss) issue(w, p0);
                for (int rel = w; rel < nss && !quit; rel += 2 * NP) {
                    process(rel, p0, p1);
                    if (rel + NP < nss && !quit) process(rel + NP, p1, p0);
                }
            } else {
                for (int rel = w; rel < nss && !quit; rel += NP) {
                    Pre p0;
                    issue(rel, p0);
                    process(rel, p0, p0);
                }
            }
        }
    }
    if (threadIdx.x == 0) {
        uint32_t d = atomicAdd(&sync[1], 1u);
        if (d == gridDim.x - 1) {
            __hip_atomic_store(&sync[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&sync[1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// Triangles whose rows are too long for the LDS slots (more than 32 entries: ILU(3)
// fill, irregular matrices). Rows in level order, each level's rows of more than
// kRowShort entries first; a wavefront solves one long row or kRowGroup short ones
// (8 lanes a row), the lanes striding the row's entries, which are stored row by row.
// Workgroups claim kRowWaves consecutive items at a time from a ticket counter, the next
// claim already on its way while the current items are solved, and poll every
// dependency in global memory: an item only waits for items of earlier levels, claimed
// before it by running workgroups, so the lowest unfinished item can always proceed.
//
// Bound: a level costs one device-coherent store and load between compute units (1.2 us
// measured) plus the row's own loads, which are issued levels ahead of time because
// 2048 wavefronts hold more rows than a level has. One row per lane over a padded slab
// (every row walking the longest row's slots, one batch of polls after another) took
// 5.78 ms for the L-then-U pair of a 60,000-row power-law ILU(0) (rows of 4 to 512
// entries, 31 levels); this takes 0.15 ms.
using plan::kRowGroup;
using plan::kRowShort;
constexpr int kRowWaves = 8;   // wavefronts per workgroup, one item each per claim

template <class T, bool UPPER>
__global__ __launch_bounds__(64 * kRowWaves) void k_trsv_row(int32_t nitems, const int2 *__restrict__ items,
                                                             const int32_t *__restrict__ ptr,
                                                             const int32_t *__restrict__ grow,
                                                             const int32_t *__restrict__ other,
                                                             const int32_t *__restrict__ enc,
                                                             const T *__restrict__ val, const T *__restrict__ piv,
                                                             SolveIO<T> io, uint32_t *sync, const int32_t *skip,
                                                             uint32_t *err, uint32_t spin) {
    using U = typename Sentinel<T>::U;
    constexpr U SENT = Sentinel<T>::bits;
    if (skip && *skip) return;
    fill_sentinel(io);
    // by the round's parity: its claim, and whether a wave gave up in the round before
    __shared__ int s_claim[2], s_abort[2];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // rows q0 .. q0 + cnt - 1, G lanes each; false: a wait gave up
    auto solve = [&](auto gsz, auto bsz, int32_t q0, int32_t cnt) {
        constexpr int G = decltype(gsz)::value, B = decltype(bsz)::value;
        const int g = lane % G, r = lane / G;
        const bool live = r < cnt;
        const int32_t q = q0 + (live ? r : 0);
        const int32_t e1 = live ? ptr[q + 1] : 0;
        int32_t e = live ? ptr[q] + g : 0;
        const bool lead = live && g == 0;
        const int32_t gi = lead ? grow[q] : 0;
        const T rhs = lead ? io.b[io.bmap ? io.bmap[q] : io.b_by_row ? gi : q] : (T)0;
        T pv = (T)1;
        if constexpr (UPPER) pv = lead ? piv[q] : (T)1;
        T acc = (T)0;
        while (__ballot(e < e1) != 0) {
            uint32_t it = 0;
            int es[B];
            T vs[B];
            U xs[B];
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const bool in = e + u * G < e1;
                es[u] = in ? enc[e + u * G] : kPad;
                vs[u] = in ? val[e + u * G] : (T)0;
            }
#pragma unroll
            for (int u = 0; u < B; ++u) xs[u] = first_poll(io.xq, es[u]);
            for (;;) {  // only the pending entries are reloaded
                bool pend = false;
#pragma unroll
                for (int u = 0; u < B; ++u) pend |= xs[u] == SENT;
                if (__ballot(pend) == 0) break;
                ++it;
                if (it > spin || ((it & 63) == 0 && timed_out(err))) return false;
                __builtin_amdgcn_s_sleep(1);
#pragma unroll
                for (int u = 0; u < B; ++u)
                    if (xs[u] == SENT) xs[u] = load_coherent(io.xq + es[u]);
            }
#pragma unroll
            for (int u = 0; u < B; ++u)
                if (es[u] != kPad) acc += vs[u] * from_bits<T>(xs[u]);
            e += G * B;
        }
#pragma unroll
        for (int o = G / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
        if (lead) {
            T v = rhs - acc;
            if constexpr (UPPER) v = v / pv;
            store_coherent(io.xq + q, v);
            if (io.x) io.x[gi] = v;
            if (io.yother) {
                const int32_t o = other[q];
                if (o >= 0) io.yother[o] = v;
            }
        }
        return true;
    };
    if (threadIdx.x == 0) {
        s_abort[0] = s_abort[1] = 0;
        s_claim[0] = (int)atomicAdd(&sync[0], 1u);
    }
    for (int round = 0;; ++round) {
        __syncthreads();
        const int c = s_claim[round & 1];
        if (s_abort[round & 1] || (int64_t)c * kRowWaves >= nitems) break;  // uniform: read after the barrier
        uint32_t next = 0;
        if (threadIdx.x == 0) next = atomicAdd(&sync[0], 1u);
        const int i = c * kRowWaves + wave;
        if (i < nitems) {
            const int2 item = items[i];
            const int32_t q0 = __builtin_amdgcn_readfirstlane(item.x), cnt = __builtin_amdgcn_readfirstlane(item.y);
            const bool ok = cnt > 0 ? solve(std::integral_constant<int, 64 / kRowGroup>(),
                                            std::integral_constant<int, 4>(), q0, cnt)
                                    : solve(std::integral_constant<int, 64>(), std::integral_constant<int, 8>(), q0, 1);
            if (!ok) {  // nothing more is published; every wave of the workgroup leaves at the barrier
                record_timeout(err);
                s_abort[(round + 1) & 1] = 1;
            }
        }
        if (threadIdx.x == 0) s_claim[(round + 1) & 1] = (int)next;
    }
    if (threadIdx.x == 0) {  // the last workgroup out resets the counters for the next launch
        const uint32_t d = atomicAdd(&sync[1], 1u);
        if (d == gridDim.x - 1) {
            __hip_atomic_store(&sync[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&sync[1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// ---------------------------------------------------------------------------
// Wavefront solve of a triangle on a 3D grid (plan.hpp's GridPlan): one tile of 8 x 8
// columns per workgroup, tiles claimed in order from a ticket counter (a tile only
// waits for tiles claimed before it, held by running workgroups).
//
// Lane (ma, mb) of the solver solves its column's row at c-index s - ma - mb - lag at step
// s, lag = kGridLag for each 16 lanes before it. Its dependencies: the row behind it along c,
// solved by the lane itself a step earlier (a register); from the left, lane - 1 a step earlier
// (a DPP shift); from below, lane - 8: in the same 16 lanes a DPP shift too, else, which is
// what the lag is for, read from LDS a step ahead; on the tile's low faces the values that
// the tiles before it hand over through global memory.
//
// Bound: the path across the tiles, 30 of them for 128 x 128 columns, each 11 to 15 steps and
// the way of a value from one compute unit to the next; a step is one wavefront's instruction
// issue. So everything else is kept off the solver, which takes blocks of 4 steps without a
// branch inside:
//  * loaders stream the coefficients (packed by claim, step and lane) and the right-hand side
//    of 8 steps each into registers and, when the ring has room, into a ring of 32 LDS slots;
//    the solver reads a block's slots while it computes the one before;
//  * a poller for each low face brings in its 8 values a step, 8 steps at a time, with
//    device-coherent loads until they are not the sentinel, and counts the leading steps that
//    have all theirs; the solver looks at the count and the values in one LDS round trip;
//  * the solver stores the high faces' results for the next tiles at the end of a block (the
//    corner on the a-face only, where the tile above reads it too); writers take all results
//    from LDS to the output, by row or in padded tile-step order for the intermediate of an
//    L-then-U chain; a slot is loaded again once its results were read.
// Lanes without a row at a step have zero coefficients and a zero right-hand side: they
// compute zeros (or, once a solution holds infinities, NaN) that reach no row.
// Readiness of a face value is the value itself, as in the blocked kernel: the face buffer
// holds the sentinel before the launch (filled by the previous launch of an L-then-U chain,
// or by a fill kernel before a lone solve).
// With the neighbours' values passed through LDS cells, a check of the faces and the stores to
// the output in every step, a step took 131 ns and a tile 2.9 us after the one before; here 78
// and 2.7. 128^3 L-then-U pair 233 -> 201 us, one triangle 142 -> 104. Measured and not taken
// (the pair, against the state at the time): blocks of 2 steps (265 : 232) and of 8 (229 : 204,
// registers), a lag of 2 (250 : 232), 12 wavefronts (281 : 250, registers), a look at the faces
// in every step (263 : 261), a block's inputs read again after a wait (250 : 232).
constexpr int kGridWaves = 8;  // the solver, two face pollers, the writers, then loaders
constexpr int kGridWriters = 2;
constexpr int kGridLoaders = kGridWaves - 3 - kGridWriters;
constexpr int kGridRing = 32;  // steps in LDS
static_assert((kGridRing & (kGridRing - 1)) == 0 && kGridRing % 8 == 0, "ring");

struct GridArgs {
    int32_t NA, NB, NC, PA, PB, S, nclaims;
    int64_t sa, sb, sc;
    uint32_t *err;  // the schedule's error word
    uint32_t spin;  // polls before a wait gives up
};

// b: right-hand side by row; x: results by row; face: the triangle's face buffer
// ([claim][face][step][8] in the giving tile's steps, sentinel-filled); fill: nfill elements set to the
// sentinel for a later solve (may be NULL). bpad / xpad: b / x in padded tile-step
// order instead, the lower plan's position (claim * S + step) * 64 + lane, which the
// upper plan visits in reverse (its claim c, step s, lane l is the lower plan's
// position total - 1 - (c S + s) 64 - l): the intermediate of an L-then-U chain, read
// and written 512 contiguous bytes a step instead of a row-by-row gather.
template <class T>
struct GridIO {
    const T *b;
    T *x;
    T *face;
    T *fill;
    int64_t nfill;
    int32_t bpad, xpad;
};

// Two values loaded and stored together (in FP64 64 lanes read 16 bytes from LDS in 10 cycles,
// two 8-byte reads in one ds_read2st64 in 18).
template <class T>
struct alignas(2 * sizeof(T)) Two {
    T x, y;
};

// Dynamic LDS of k_trsv_grid: control words, slots [ring][SLOT], rows [ring][kGridRow],
// a row of zeros. A slot: the pairs (back, below) and (left, right-hand side) of the 64 lanes;
// upper: (back, below), (left, reciprocal pivot), then the right-hand sides. A row: 8 values
// from the b-face, the 64 results, 8 values from the a-face.
constexpr int kGridBlock = 4;  // steps of the solver between two looks at what has arrived
using plan::kGridLag;
constexpr size_t kGridCtrl = 512;
constexpr int kGridRow = 80;
template <bool UPPER>
constexpr int kGridSlot = UPPER ? 320 : 256;
template <class T, bool UPPER>
constexpr size_t grid_lds_bytes() {
    return kGridCtrl + ((size_t)kGridRing * (kGridSlot<UPPER> + kGridRow) + kGridRow) * sizeof(T);
}

// LDS accesses of one wavefront complete in order: only the compiler is held, so that a value
// stored before is what another lane of the wavefront reads after.
__device__ __forceinline__ void lds_order() {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_wave_barrier();
}

// v of the lane K before in the same 16 lanes; lanes without one: `first`.
template <int K, class T>
__device__ __forceinline__ T row_shift(T first, T v) {
    constexpr int kRowShr = 0x110 + K;  // DPP row_shr:K
    int f[sizeof(T) / 4], x[sizeof(T) / 4];
    __builtin_memcpy(f, &first, sizeof(T));
    __builtin_memcpy(x, &v, sizeof(T));
#pragma unroll
    for (int k = 0; k < (int)(sizeof(T) / 4); ++k) x[k] = __builtin_amdgcn_update_dpp(f[k], x[k], kRowShr, 0xF, 0xF, false);
    __builtin_memcpy(&v, x, sizeof(T));
    return v;
}

// The same, 0 in lanes without one (no register to copy first).
template <int K, class T>
__device__ __forceinline__ T row_shift0(T v) {
    int x[sizeof(T) / 4];
    __builtin_memcpy(x, &v, sizeof(T));
#pragma unroll
    for (int k = 0; k < (int)(sizeof(T) / 4); ++k) x[k] = __builtin_amdgcn_mov_dpp(x[k], 0x110 + K, 0xF, 0xF, true);
    __builtin_memcpy(&v, x, sizeof(T));
    return v;
}

template <class T, bool UPPER>
__global__ __launch_bounds__(64 * kGridWaves) void k_trsv_grid(GridArgs G, const T *__restrict__ coef, GridIO<T> io,
                                                               uint32_t *sync, const int32_t *skip) {
    using U = typename Sentinel<T>::U;
    constexpr U SENT = Sentinel<T>::bits;
    constexpr int NCOEF = UPPER ? plan::kGridCoefUpper : plan::kGridCoefLower;
    constexpr int TA = plan::kGT, TB = plan::kGT, RS = kGridRow, RM = kGridRing - 1;
    constexpr int FS = TA;  // face entries per step in each face's buffer
    constexpr int SLOT = kGridSlot<UPPER>;
    constexpr int NB = kGridBlock, D = kGridLag;
    static_assert(TA == 8 && TB == 8 && 8 % NB == 0 && D >= 1 && D < NB, "lanes are 8 x 8 columns, blocks 8 steps");
    if (skip && *skip) return;  // uniform: no workgroup touches the counters
    if (io.fill) {
        const T sv = from_bits<T>(SENT);
        for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < io.nfill;
             i += (int64_t)gridDim.x * blockDim.x)
            io.fill[i] = sv;
    }
    extern __shared__ __align__(16) char gsm[];
    int *const filled = (int *)gsm;          // [ring]: step whose coefficients and rhs a slot holds
    int *const s_done = filled + kGridRing;  // steps the solver has finished
    int *const s_claim = s_done + 1;
    int *const s_abort = s_done + 2;
    int *const s_faces = s_done + 4;         // [2]: leading steps whose a-face (b-face) values are all in their rows
    int *const s_prog = s_done + 6;          // [writers]: all blocks of a writer below this step are read
    int *const s_none = s_done + 32;         // [64]: written by lanes that have nothing to say
    T *const slots = (T *)(gsm + kGridCtrl);
    T *const rows = slots + kGridRing * SLOT;
    T *const zeros = rows + kGridRing * RS;
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    // wavefront 4 is on the solver's SIMD: a poller, which computes little
    const int wave = wid == 4 ? 2 : wid >= 2 && wid < 4 ? wid + 1 : wid;
    const int ma = lane & 7, mb = lane >> 3;
    auto lag = [](int l) { return kGridLag * (l >> 4); };
    auto skew = [&](int l) { return (l & 7) + (l >> 3) + lag(l); };  // lane l's row at step s: c-index s - skew
    if (threadIdx.x == 0) *s_abort = 0;
    for (int t = threadIdx.x; t < RS; t += blockDim.x) zeros[t] = (T)0;
    auto lds_load = [](const int *p) {
        return __builtin_amdgcn_readfirstlane(__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
    };
    auto lds_publish = [&](int *p, int v) {  // after this wavefront's LDS accesses above it (they complete in order)
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        if (lane == 0) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    // one more poll of a wait (wave-uniform callers): true when the wait must stop
    auto spun_out = [&](uint32_t &it, bool device_wide) {
        ++it;
        bool stop = it > G.spin;
        if (!stop && (it & 63) == 0) stop = lds_load(s_abort) != 0 || (device_wide && timed_out(G.err));
        stop = __builtin_amdgcn_readfirstlane((int)stop) != 0;
        if (stop) {
            __hip_atomic_store(s_abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            record_timeout(G.err);
        }
        return stop;
    };
    const int S8 = (G.S + lag(63) + 7) / 8 * 8;  // whole blocks: the last steps hold no row
    for (;;) {
        __syncthreads();
        if (*s_abort) break;  // uniform: read by every thread after the barrier
        if (threadIdx.x == 0) {
            *s_claim = (int)atomicAdd(&sync[0], 1u);
            *s_done = s_faces[0] = s_faces[1] = 0;
        }
        if (threadIdx.x < kGridRing) filled[threadIdx.x] = -1;
        if ((int)threadIdx.x < kGridWriters) s_prog[threadIdx.x] = 0;
        __syncthreads();
        const int c = __builtin_amdgcn_readfirstlane(*s_claim);
        if (c >= G.nclaims) break;
        const int mta = c % G.PA, mtb = c / G.PA;
        const int32_t ta = UPPER ? G.PA - 1 - mta : mta, tb = UPPER ? G.PB - 1 - mtb : mtb;
        // global a and b of the column of lane (ma', mb')
        auto col_a = [&](int m) { return ta * TA + (UPPER ? TA - 1 - m : m); };
        auto col_b = [&](int m) { return tb * TB + (UPPER ? TB - 1 - m : m); };
        // row of lane l's column at its c-index mc, -1: none
        auto row_of = [&](int l, int32_t mc) -> int64_t {
            const int32_t ga = col_a(l & 7), gb = col_b(l >> 3);
            return ga < G.NA && gb < G.NB && (uint32_t)mc < (uint32_t)G.NC
                       ? ga * G.sa + gb * G.sb + (UPPER ? G.NC - 1 - mc : mc) * G.sc : -1;
        };
        // Vectors by row are read and written 8 steps at a time, so that a wavefront's access
        // falls on few cache lines (at one step the lanes' rows lie on 15 planes): access i of
        // 8 takes, with columns running along the unit stride, 8 steps of the 8 columns from
        // 8 i, else a column per lane at the step whose rows lie on plane i (mod 8).
        const bool along = G.sc == 1;
        auto acc_col = [&](int i) { return along ? 8 * i + (lane >> 3) : lane; };
        auto acc_step = [&](int i) { return along ? lane & 7 : (skew(lane) + i) & 7; };
        // this lane's padded tile-step position at step 0, and its change per step
        const int64_t pq = ((int64_t)c * G.S - lag(lane)) * 64 + lane;
        const int64_t p0 = UPPER ? (int64_t)G.nclaims * G.S * 64 - 1 - pq : pq, pd = UPPER ? -64 : 64;
        if (wave == 0) {
            // ---------------- solver
            __builtin_amdgcn_s_setprio(3);
            // this lane's face store (if any): a-face by mb (the corner too), b-face by ma
            const bool fst = (ma == TA - 1 && (mta < G.PA - 1 || (mb == TB - 1 && mtb < G.PB - 1))) ||
                             (ma != TA - 1 && mb == TB - 1 && mtb < G.PB - 1);
            T *const fp = io.face + ((int64_t)c * 2 + (ma == TA - 1 ? 0 : 1)) * S8 * FS + (ma == TA - 1 ? mb : ma);
            int *const done = lane == 0 ? s_done : s_none + lane;
            T xp = (T)0;  // this lane's result of the previous step (0: none)
            int ready = 0;   // steps known to be loaded
            int fready = 0;  // steps known to have their face values
            bool bail = false;
            auto look = [&](int s0) {  // looks at the flags of the ring from step s0, in one LDS round trip
                const int want = s0 + (lane & RM);
                const int f = __hip_atomic_load(&filled[want & RM], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                const uint64_t out = __ballot(f != want);
                ready = max(ready, s0 + (out ? min(__builtin_ctzll(out), kGridRing) : kGridRing));
                __atomic_signal_fence(__ATOMIC_SEQ_CST);
            };
            struct Blk {  // a block's inputs
                Two<T> c0[NB], c1[NB];
                T b[NB], fa[NB], nb[D];  // nb: the values from below of the first steps
            };
            // step u of the block whose slots start at sl
            auto load_slot = [&](const T *sl, int u, Blk &H) {
                H.c0[u] = ((const Two<T> *)(sl + u * SLOT))[lane];
                H.c1[u] = ((const Two<T> *)(sl + u * SLOT))[64 + lane];
                if constexpr (UPPER) H.b[u] = sl[u * SLOT + 256 + lane];
            };
            // block s0's coefficients and right-hand sides, waited for until they are loaded
            auto load_slots = [&](int s0, Blk &H) {
                uint32_t it = 0;
                for (look(s0); ready < s0 + NB && !bail; look(s0)) bail = spun_out(it, false);
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    load_slot(slots + (s0 & RM) * SLOT, u, H);
                    __asm__ volatile("" : "+v"(H.c0[u].x), "+v"(H.c0[u].y), "+v"(H.c1[u].x), "+v"(H.c1[u].y));
                    if constexpr (UPPER) __asm__ volatile("" : "+v"(H.b[u]));
                }
            };
            // block s0's face values, waited for until they are in: the counts are read before the
            // values, so that a look that finds them needs no second one
            auto load_faces = [&](int s0, Blk &H) {
                const T *const row = rows + (s0 & RM) * RS;
                uint32_t it = 0;
                for (;;) {
                    const int f = __hip_atomic_load(s_faces + (lane & 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    __atomic_signal_fence(__ATOMIC_SEQ_CST);
                    T b[D];
#pragma unroll
                    for (int u = 0; u < NB; ++u) H.fa[u] = row[u * RS + 72 + mb];
#pragma unroll
                    for (int u = 0; u < D; ++u) b[u] = row[u * RS + ma];
#pragma unroll
                    for (int u = 0; u < NB; ++u) __asm__ volatile("" : "+v"(H.fa[u]));
#pragma unroll
                    for (int u = 0; u < D; ++u) {
                        __asm__ volatile("" : "+v"(b[u]));
                        H.nb[u] = mb == 0 ? b[u] : H.nb[u];
                    }
                    fready = min(__builtin_amdgcn_readlane(f, 0), __builtin_amdgcn_readlane(f, 1));
                    if (fready >= s0 + NB || bail) break;
                    bail = spun_out(it, false);
                }
                __atomic_signal_fence(__ATOMIC_SEQ_CST);
            };
            // The steps of block s0, whose inputs are in cur. The next block's are read into nxt,
            // a step's worth in each step (from slots in range that may not be loaded yet: read
            // again then). A taken branch costs as much as four instructions of a step, so there
            // is none here: lanes without a row compute zeros (or, once a solution holds
            // infinities, NaN) that reach no row and face entries that no tile reads.
            auto run = [&](int s0, Blk &cur, Blk &nxt) {
                const int s1 = s0 + NB;
                if (__builtin_expect(ready < s1 + NB, 0)) look(s1);
                const bool loaded = ready >= s1 + NB, faced = fready >= s1 + NB;
                T *const r0 = rows + (s0 & RM) * RS, *const r1 = rows + (s1 & RM) * RS;
                const T *const sx = slots + (s1 & RM) * SLOT;
                // the value from below at step s0 + u + D: lanes of the b-face in that step's row,
                // others in the row of 1 + D steps before it
                const T *const bm = r0 + (mb == 0 ? D * RS : -RS) + lane;
                const T *const bp = (s0 == 0 ? zeros : rows + ((s0 - 1) & RM) * RS) + lane;
                const T *const b0 = mb == 0 ? bm : bp;
                const T *const be = mb == 0 ? r1 - (NB - D) * RS + lane : bm;
                T *const fb = fp + (int64_t)s0 * FS;
                T acc[NB], nb[NB];
#pragma unroll
                for (int u = 0; u < D; ++u) nb[u] = cur.nb[u];
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    const T bel = (u == 0 ? b0 : u < NB - D ? bm : be)[u * RS];
                    if (u + D < NB)
                        nb[u + D < NB ? u + D : 0] = bel;
                    else
                        nxt.nb[u + D < NB ? 0 : u + D - NB] = bel;
                    load_slot(sx, u, nxt);
                    nxt.fa[u] = r1[u * RS + 72 + mb];
                    T left = row_shift0<1>(xp);
                    __asm__ volatile("" : "+v"(left));  // (every lane shifts: not under the condition below)
                    left = ma == 0 ? cur.fa[u] : left;
                    const T below = row_shift<8>(nb[u], xp);
                    T v;
                    if constexpr (!UPPER) {  // columns ascending (c along z): back, below, left
                        v = cur.c1[u].y - cur.c0[u].x * xp;
                        v -= cur.c0[u].y * below;
                        v -= cur.c1[u].x * left;
                    } else {  // left, below, back; then the reciprocal pivot
                        v = cur.b[u] - cur.c1[u].x * left;
                        v -= cur.c0[u].y * below;
                        v -= cur.c0[u].x * xp;
                        v *= cur.c1[u].y;
                    }
                    (r0 + u * RS)[8 + lane] = v;
                    lds_order();  // other lanes read v from there in the next step
                    acc[u] = xp = v;
                }
                // an arithmetic result is never the signalling-NaN sentinel (IEEE mode quiets
                // NaN operands), so no check is needed before publishing it
                if (fst) {
#pragma unroll
                    for (int u = 0; u < NB; ++u) {
                        U bits;
                        __builtin_memcpy(&bits, &acc[u], sizeof(T));
                        __hip_atomic_store((U *)(fb + u * FS), bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                }
                __atomic_signal_fence(__ATOMIC_SEQ_CST);
                __hip_atomic_store(done, s1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (__builtin_expect(!loaded && s1 < S8, 0)) load_slots(s1, nxt);  // (after a give-up: never used)
                if (__builtin_expect(!faced, 1)) {
                    if (s1 < S8) load_faces(s1, nxt);
                }
            };
            Blk h0, h1;
#pragma unroll
            for (int u = 0; u < D; ++u) h0.nb[u] = (T)0;
            load_slots(0, h0);
            load_faces(0, h0);
            for (int s0 = 0; s0 < S8 && !bail; s0 += 2 * NB) {
                run(s0, h0, h1);
                if (s0 + NB < S8 && !bail) run(s0 + NB, h1, h0);
            }
            __builtin_amdgcn_s_setprio(0);
        } else if (wave <= 2) {
            // ---------------- face pollers, one per face: lane 8 q + j polls entry j of step w + q;
            // a value goes into the step's row once, when it has arrived and the solver is done
            // with the row's previous use; the window moves on by the leading steps that have
            // all theirs
            const bool on_a = wave == 1;
            const int q = lane >> 3, j = lane & 7, lg = on_a ? lag(8 * j) : 0;
            // a-face entry j: a-face of the tile before along a; b-face entry j: b-face of the
            // tile below, its corner (j = 7) on that tile's a-face
            // (the faces are in the order of the giving tile's steps)
            const T *const fsrc = io.face + j + (on_a       ? ((int64_t)(c - 1) * 2 + 0) * S8 * FS + (TA - 1) * FS
                                                 : ((int64_t)(c - G.PA) * 2 + (j == TA - 1 ? 0 : 1)) * S8 * FS +
                                                       (TB - 1 + lag(63)) * FS);
            T *const gp = rows + (on_a ? 72 + j : j);
            const bool has = on_a ? mta > 0 && col_b(j) < G.NB : mtb > 0 && col_a(j) < G.NA;
            int w = 0;
            if ((on_a ? mta : mtb) == 0) {  // no tile before it on this side: zeros, and nothing to poll
                for (int r = q; r < kGridRing; r += 8) gp[r * RS] = (T)0;
                lds_publish(s_faces + wave - 1, INT_MAX);
                w = S8;
            }
            bool wr = false;  // this lane's value of step w + q is in its row
            uint32_t it = 0;
            int dn = 0;  // steps the solver is known to have finished
            while (w < S8) {
                const int st = w + q;
                if (w + 8 > dn + kGridRing) dn = lds_load(s_done);
                const bool can = !wr && st < S8 && st < dn + kGridRing;
                const bool need = can && has && (uint32_t)(st - lg - j) < (uint32_t)G.NC;
                const U v = need ? load_coherent(fsrc + (int64_t)st * FS) : (U)0;
                if (can && (!need || v != SENT)) {
                    gp[(st & RM) * RS] = need ? from_bits<T>(v) : (T)0;
                    wr = true;
                }
                uint64_t t = __ballot(wr || st >= S8);  // bit 8 q ends up set when all of step w + q is in
                t &= t >> 4;
                t &= t >> 2;
                t &= t >> 1;
                t = ~t & 0x0101010101010101ull;
                const int k = t ? __builtin_ctzll(t) >> 3 : 8;  // leading steps of the window with all their values
                if (k == 0) {
                    if (spun_out(it, true)) break;
                    continue;
                }
                it = 0;
                lds_publish(s_faces + wave - 1, w + k);
                const int from = lane + 8 * k;  // lane l takes over lane l + 8 k's entry
                const int nw = __shfl((int)wr, from < 64 ? from : lane);
                wr = from < 64 && nw != 0;
                w += k;
            }
        } else if (wave < 3 + kGridWriters) {
            // ---------------- writers: blocks of 8 steps in turn
            const int wi = wave - 3;
            for (int s0 = 8 * wi; s0 < S8; s0 += 8 * kGridWriters) {
                uint32_t it = 0;
                bool quit = false;
                while (lds_load(s_done) < s0 + 8) {
                    if (spun_out(it, false)) {
                        quit = true;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(2);
                }
                if (quit) break;
                __atomic_signal_fence(__ATOMIC_SEQ_CST);
                auto result = [&](int l, int u) {
                    return rows[((s0 + u) & RM) * RS + 8 + l];
                };
                T v[8];
                if (io.xpad) {
#pragma unroll
                    for (int u = 0; u < 8; ++u) v[u] = result(lane, u);
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        if (row_of(lane, s0 + u - skew(lane)) >= 0) io.x[p0 + (s0 + u) * pd] = v[u];
                } else {
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = result(acc_col(i), acc_step(i));
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const int64_t row = row_of(acc_col(i), s0 + acc_step(i) - skew(acc_col(i)));
                        if (row >= 0) io.x[row] = v[i];
                    }
                }
                lds_publish(s_prog + wi, s0 + 8 * kGridWriters);
            }
            lds_publish(s_prog + wi, INT_MAX);
        } else {
            // ---------------- loaders: blocks of 8 consecutive steps in turn, each in flight at
            // once; a block waits in registers until its slots' previous results were read, so
            // that what is in flight does not end with the ring
            for (int s0 = (wave - 3 - kGridWriters) * 8; s0 < S8; s0 += kGridLoaders * 8) {
                T cv[8][NCOEF], bv[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int s = s0 + u;
                    const int o = s - lag(lane);  // the packed order has no lag
                    const bool in = (uint32_t)o < (uint32_t)G.S;
                    const T *cp = coef + ((int64_t)c * G.S + (in ? o : 0)) * NCOEF * 64 + lane;
#pragma unroll
                    for (int k = 0; k < NCOEF; ++k) cv[u][k] = in ? cp[k * 64] : (T)0;
                    const int64_t at = io.bpad ? row_of(lane, s - skew(lane)) >= 0 ? p0 + s * pd : -1
                                               : row_of(acc_col(u), s0 + acc_step(u) - skew(acc_col(u)));
                    bv[u] = at >= 0 ? io.b[at] : (T)0;
                }
                uint32_t it = 0;
                bool quit = false;
                for (;;) {
                    int m = INT_MAX;
#pragma unroll
                    for (int k = 0; k < kGridWriters; ++k) m = min(m, lds_load(s_prog + k));
                    if (m >= s0 + 8 - kGridRing) break;
                    if (spun_out(it, false)) {
                        quit = true;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(2);
                }
                if (quit) break;
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    T *const sl = slots + ((s0 + u) & RM) * SLOT;
                    ((Two<T> *)sl)[lane] = Two<T>{cv[u][0], cv[u][1]};
                    if constexpr (UPPER)
                        ((Two<T> *)sl)[64 + lane] = Two<T>{cv[u][2], cv[u][3]};
                    else
                        sl[128 + 2 * lane] = cv[u][2];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int st = io.bpad ? u : acc_step(u), l = io.bpad ? lane : acc_col(u);
                    slots[((s0 + st) & RM) * SLOT + (UPPER ? 256 + l : 129 + 2 * l)] = bv[u];
                }
                __atomic_signal_fence(__ATOMIC_SEQ_CST);
                if (lane < 8)
                    __hip_atomic_store(&filled[(s0 + lane) & RM], s0 + lane, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {  // the last workgroup out resets the counters for the next launch
        const uint32_t d = atomicAdd(&sync[1], 1u);
        if (d == gridDim.x - 1) {
            __hip_atomic_store(&sync[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&sync[1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// ---------------------------------------------------------------------------
// Wavefront solve of a triangle on a 2D grid: tiles of 64 columns side by side (64 x 1
// GridPlan), one wavefront solving a tile: at step s lane l solves the row at c-index
// s - l of its column. Its two dependencies were solved at step s - 1, by the lane itself
// (a register) and by lane l - 1, whose value one DPP shift over the wavefront brings in;
// lane 0 keeps the shift's old operand, the face value from the tile before.
//
// Bound: the chain of steps, one wavefront's instruction issue: two fused multiply-adds,
// two DPP moves, four LDS accesses. So everything else is kept off the solver:
//  * loaders stream the coefficients and the right-hand side into a ring of 64 LDS slots,
//    8 steps each in flight per wavefront;
//  * a poller brings in the face values, 32 steps at a time;
//  * the solver puts each result in the place of the right-hand side it came from, and two
//    writers take the results from there to the face buffer (device-coherent) and to the
//    output; a slot is loaded again once its result was read.
// Blocks of 8 steps: a block starts when its slots are loaded and its face values are in;
// the next block's slots are read into registers while it computes if they are loaded
// already. Lanes without a row at a step have zero coefficients and a zero right-hand
// side: they compute zeros (or, once a solution holds infinities, NaN) that reach no row.
// With the neighbours' values passed through LDS cells and all stores in the solver a step
// took 132 ns; here 45 (54 with the streams of a long chain beside it; 701 x 653 L-then-U
// pair 473 -> 215 us, 64 x 64 54 -> 28 us).
constexpr int kG2Waves = 8, kG2Ring = 64, kG2Batch = 8, kG2Writers = 2;
constexpr int kG2Loaders = kG2Waves - 2 - kG2Writers;  // after the solver, the poller and the writers
constexpr int kG2Row = 68;  // elements of a step in the ring of right-hand sides: 4 more than the lanes, so
                            // that 8 steps x 8 columns read or written at once fall on different banks
constexpr size_t kG2Ctrl = 512;
static_assert(plan::kGT2 == 64, "one lane per column of a tile");

template <class T, bool UPPER>
constexpr size_t grid2_lds_bytes() {
    constexpr int NC2 = UPPER ? plan::kGrid2CoefUpper : plan::kGrid2CoefLower;
    return kG2Ctrl + (size_t)kG2Ring * sizeof(T) + (size_t)kG2Ring * (NC2 * 64 + kG2Row) * sizeof(T);
}

// The coefficients back and left of a row, loaded and stored together.
template <class T>
struct alignas(2 * sizeof(T)) Pair {
    T back, left;
};

// v of the lane before, lane 0: `first`.
template <class T>
__device__ __forceinline__ T shift_lane(T first, T v) {
    constexpr int kWaveShr1 = 0x138;  // DPP wave_shr:1
    if constexpr (sizeof(T) == 8) {
        int f[2], x[2];
        __builtin_memcpy(f, &first, 8);
        __builtin_memcpy(x, &v, 8);
        x[0] = __builtin_amdgcn_update_dpp(f[0], x[0], kWaveShr1, 0xF, 0xF, false);
        x[1] = __builtin_amdgcn_update_dpp(f[1], x[1], kWaveShr1, 0xF, 0xF, false);
        __builtin_memcpy(&v, x, 8);
    } else {
        int f, x;
        __builtin_memcpy(&f, &first, 4);
        __builtin_memcpy(&x, &v, 4);
        x = __builtin_amdgcn_update_dpp(f, x, kWaveShr1, 0xF, 0xF, false);
        __builtin_memcpy(&v, &x, 4);
    }
    return v;
}

// Lane 0: v of lane u of its 16 (other lanes: unspecified). u is a compile-time constant.
template <int u, class T>
__device__ __forceinline__ T lane_to_first(T v) {
    if constexpr (u == 0) return v;
    constexpr int kRowShl = 0x100 + u;  // DPP row_shl:u
    int x[sizeof(T) / 4];
    __builtin_memcpy(x, &v, sizeof(T));
#pragma unroll
    for (int k = 0; k < (int)(sizeof(T) / 4); ++k) x[k] = __builtin_amdgcn_update_dpp(0, x[k], kRowShl, 0xF, 0xF, true);
    __builtin_memcpy(&v, x, sizeof(T));
    return v;
}

template <class T, bool UPPER>
__global__ __launch_bounds__(64 * kG2Waves) void k_trsv_grid2(GridArgs G, const T *__restrict__ coef, GridIO<T> io,
                                                              uint32_t *sync, const int32_t *skip) {
    using U = typename Sentinel<T>::U;
    constexpr U SENT = Sentinel<T>::bits;
    constexpr int NC2 = UPPER ? plan::kGrid2CoefUpper : plan::kGrid2CoefLower;  // back, left (and reciprocal pivot)
    constexpr int RM = kG2Ring - 1;
    if (skip && *skip) return;  // uniform: no workgroup touches the counters
    if (io.fill) {
        const T sv = from_bits<T>(SENT);
        for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < io.nfill;
             i += (int64_t)gridDim.x * blockDim.x)
            io.fill[i] = sv;
    }
    extern __shared__ __align__(16) char gsm[];
    int *const filled = (int *)gsm;        // [ring]: step whose coefficients and rhs a slot holds
    int *const s_done = filled + kG2Ring;  // steps the solver has finished
    int *const s_faces = s_done + 1;       // leading steps whose face value is in the ring
    int *const s_claim = s_done + 2;
    int *const s_abort = s_done + 3;
    int *const s_prog = s_done + 4;        // [writers]: all blocks of a writer below this step are read
    T *const fring = (T *)(gsm + kG2Ctrl);               // [ring] face values
    Pair<T> *const cpr = (Pair<T> *)(fring + kG2Ring);   // [ring][64] coefficients
    T *const rhs = (T *)(cpr + kG2Ring * 64);            // [ring][kG2Row] right-hand side, then result
    T *const rpv = rhs + kG2Ring * kG2Row;               // [ring][64] reciprocal pivot (upper)
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    // wavefront 4 is on the solver's SIMD: the poller, which computes little
    const int wave = wid == 4 ? 1 : wid >= 1 && wid < 4 ? wid + 1 : wid;
    if (threadIdx.x == 0) *s_abort = 0;
    auto lds_load = [](const int *p) {
        return __builtin_amdgcn_readfirstlane(__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
    };
    auto lds_publish = [&](int *p, int v) {  // after this wavefront's LDS accesses above it (they complete in order)
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        if (lane == 0) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    // one more poll of a wait (wave-uniform callers): true when the wait must stop
    auto spun_out = [&](uint32_t &it, bool device_wide) {
        ++it;
        bool stop = it > G.spin;
        if (!stop && (it & 63) == 0) stop = lds_load(s_abort) != 0 || (device_wide && timed_out(G.err));
        stop = __builtin_amdgcn_readfirstlane((int)stop) != 0;
        if (stop) {
            __hip_atomic_store(s_abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            record_timeout(G.err);
        }
        return stop;
    };
    const int S8 = (G.S + 7) / 8 * 8;  // whole blocks: the steps past S hold no row
    for (;;) {
        __syncthreads();
        if (*s_abort) break;  // uniform: read by every thread after the barrier
        if (threadIdx.x == 0) {
            *s_claim = (int)atomicAdd(&sync[0], 1u);
            *s_done = 0;
            *s_faces = 0;
        }
        if (threadIdx.x < kG2Ring) filled[threadIdx.x] = -1;
        if ((int)threadIdx.x < kG2Writers) s_prog[threadIdx.x] = 0;
        if (threadIdx.x < kG2Ring) fring[threadIdx.x] = (T)0;  // (a tile without one before it: no poller writes)
        __syncthreads();
        const int c = __builtin_amdgcn_readfirstlane(*s_claim);
        if (c >= G.nclaims) break;
        const int32_t ta = UPPER ? G.PA - 1 - c : c;
        // row of column l of the tile at its c-index mc, -1: none
        auto row_of = [&](int l, int32_t mc) -> int64_t {
            const int32_t ga = ta * 64 + (UPPER ? 63 - l : l);
            return ga < G.NA && (uint32_t)mc < (uint32_t)G.NC ? ga * G.sa + (UPPER ? G.NC - 1 - mc : mc) * G.sc : -1;
        };
        // Vectors by row are read and written 8 steps at a time, so that a wavefront's access
        // falls on few cache lines (a step alone has 64 rows on 64 lines: 50 us more on the
        // 701 x 653 pair): access i of 8 takes, with columns running along the unit stride,
        // 8 steps of the 8 columns from 8 i (8 rows in a row of memory each), else, with
        // neighbouring columns adjacent in memory, a column per lane at step (lane + i) mod 8
        // (lanes in a row of memory at the same c-index).
        const bool along = G.sc == 1;
        auto acc_col = [&](int i) { return along ? 8 * i + (lane >> 3) : lane; };
        auto acc_step = [&](int i) { return along ? lane & 7 : (lane + i) & 7; };
        // this lane's padded tile-step position at step 0, and its change per step
        const int64_t pq = (int64_t)c * G.S * 64 + lane;
        const int64_t p0 = UPPER ? (int64_t)G.nclaims * G.S * 64 - 1 - pq : pq, pd = UPPER ? -64 : 64;
        const bool has_face = c > 0, has_next = c + 1 < G.nclaims;

        if (wave == 0) {
            // ---------------- solver
            __builtin_amdgcn_s_setprio(3);
            struct Blk {  // a block's inputs
                Pair<T> cv[8];
                T bv[8], pv[8], fv;  // fv: lane u holds step u's face value
            };
            int ready = 0, fready = has_face ? 0 : INT_MAX;  // steps known to be loaded / to have their face value
            bool bail = false;
            auto ensure = [&](int s0) {  // block s0 loaded and its faces in
                uint32_t it = 0;
                while (ready < s0 + 8 && !bail) {  // 8 flags, one per lane, in one LDS round trip
                    const int want = s0 + (lane & 7);
                    const int f = __hip_atomic_load(&filled[want & RM], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    if (__ballot(f != want) == 0)
                        ready = s0 + 8;
                    else if (spun_out(it, false))
                        bail = true;
                }
                it = 0;
                while (fready < s0 + 8 && !bail) {
                    fready = lds_load(s_faces);
                    if (fready < s0 + 8 && spun_out(it, false)) bail = true;
                }
                __atomic_signal_fence(__ATOMIC_SEQ_CST);
            };
            auto load = [&](int s0, Blk &H) {
                const int o = (s0 & RM) * 64 + lane;
                const T *const b = rhs + (s0 & RM) * kG2Row + lane;
                H.fv = fring[(s0 & RM) + (lane & 7)];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    H.cv[u] = cpr[o + u * 64];
                    H.bv[u] = b[u * kG2Row];
                    H.pv[u] = (T)1;
                    if constexpr (UPPER) H.pv[u] = rpv[o + u * 64];
                }
            };
            // the block's inputs have arrived (said to the compiler, which otherwise waits for
            // the next block's reads as well before the first step of this one)
            auto arrived = [&](Blk &H) {
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    __asm__ volatile("" : "+v"(H.cv[u].back), "+v"(H.cv[u].left), "+v"(H.bv[u]));
                    if constexpr (UPPER) __asm__ volatile("" : "+v"(H.pv[u]));
                }
                __asm__ volatile("" : "+v"(H.fv));
            };
            T xp = (T)0;  // this lane's result of the previous step (0: none)
            // the steps of block s0, whose inputs are in cur; those of the next one are read
            // into nxt meanwhile, and again once they are there if they were not yet
            auto block = [&](int s0, Blk &cur, Blk &nxt) {
                const int s1 = s0 + 8;
                const bool pre = ready >= s1 + 8 && fready >= s1 + 8;
                // the flags of the 16 steps from the next block: read now, looked at below
                const int want = s1 + (lane & 15);
                const int fl = __hip_atomic_load(&filled[want & RM], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                const int ff = __hip_atomic_load(s_faces, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                load(s1, nxt);
                T *const o = rhs + (s0 & RM) * kG2Row + lane;
                auto step = [&](auto uc) {
                    constexpr int u = decltype(uc)::value;
                    const T left = shift_lane<T>(lane_to_first<u>(cur.fv), xp);
                    T acc;
                    if constexpr (!UPPER) {
                        acc = cur.bv[u] - cur.cv[u].back * xp;
                        acc -= cur.cv[u].left * left;
                    } else {
                        acc = cur.bv[u] - cur.cv[u].left * left;
                        acc -= cur.cv[u].back * xp;
                        acc *= cur.pv[u];
                    }
                    o[u * kG2Row] = acc;
                    xp = acc;
                };
                step(std::integral_constant<int, 0>());
                step(std::integral_constant<int, 1>());
                step(std::integral_constant<int, 2>());
                step(std::integral_constant<int, 3>());
                step(std::integral_constant<int, 4>());
                step(std::integral_constant<int, 5>());
                step(std::integral_constant<int, 6>());
                step(std::integral_constant<int, 7>());
                lds_publish(s_done, s1);
                const uint32_t out = (uint32_t)__ballot(fl != want) & 0xFFFFu;  // steps not loaded yet
                if ((out & 0xFFu) == 0) ready = max(ready, s1 + (out == 0 ? 16 : 8));
                if (has_face) fready = max(fready, __builtin_amdgcn_readfirstlane(ff));
                if (!pre && s1 < S8) {
                    ensure(s1);
                    load(s1, nxt);  // (after a give-up: in range, never published)
                }
                arrived(nxt);
            };
            Blk h0, h1;
            ensure(0);
            load(0, h0);
            arrived(h0);
            for (int s0 = 0; s0 < S8 && !bail; s0 += 16) {
                block(s0, h0, h1);
                if (s0 + 8 < S8 && !bail) block(s0 + 8, h1, h0);
            }
            __builtin_amdgcn_s_setprio(0);
        } else if (wave == 1) {
            // ---------------- face poller: lane l < 32 polls step w + l; a value goes into the ring
            // once, when it has arrived and the solver is done with the entry's previous use;
            // the window moves on by the leading steps that have their value
            if (has_face) {
                const T *const fsrc = io.face + (int64_t)(c - 1) * G.S;
                int w = 0;
                bool wr = false;  // this lane's value of step w + lane is in the ring
                uint32_t it = 0;
                while (w < S8) {
                    const int dn = lds_load(s_done);
                    const int st = w + lane;
                    const bool can = lane < 32 && !wr && st < S8 && st < dn + kG2Ring;
                    const bool need = can && st < G.NC;
                    const U v = need ? load_coherent(fsrc + st) : (U)0;
                    if (can && (!need || v != SENT)) {
                        fring[st & RM] = need ? from_bits<T>(v) : (T)0;
                        wr = true;
                    }
                    const uint64_t m = __ballot(wr || (lane < 32 && st >= S8)) & 0xFFFFFFFFull;
                    const int k = __builtin_ctzll(~m);  // leading steps of the window with their value
                    if (k == 0) {
                        if (spun_out(it, true)) break;
                        __builtin_amdgcn_s_sleep(1);
                        continue;
                    }
                    it = 0;
                    lds_publish(s_faces, min(w + k, S8));
                    const int from = lane + k;  // lane l takes over lane l + k's step
                    const int nw = __shfl((int)wr, from < 64 ? from : lane);
                    wr = from < 32 && nw != 0;
                    w += k;
                }
            }
        } else if (wave < 2 + kG2Writers) {
            // ---------------- writers: blocks of 8 steps in turn; the results of lane 63, which the
            // tile after this one waits for, first
            const int wi = wave - 2;
            T *const fdst = io.face + (int64_t)c * G.S;
            for (int s0 = 8 * wi; s0 < S8; s0 += 8 * kG2Writers) {
                uint32_t it = 0;
                bool quit = false;
                while (lds_load(s_done) < s0 + 8) {
                    if (spun_out(it, false)) {
                        quit = true;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(2);
                }
                if (quit) break;
                __atomic_signal_fence(__ATOMIC_SEQ_CST);
                const T *const p = rhs + (s0 & RM) * kG2Row;
                if (has_next) {
                    const int mc = s0 + lane - 63;
                    if (lane < 8 && (uint32_t)mc < (uint32_t)G.NC)
                        store_coherent(fdst + mc, p[lane * kG2Row + 63]);
                }
                T v[8];
                if (io.xpad) {
#pragma unroll
                    for (int u = 0; u < 8; ++u) v[u] = p[u * kG2Row + lane];
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        if (row_of(lane, s0 + u - lane) >= 0) io.x[p0 + (s0 + u) * pd] = v[u];
                } else {
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = p[acc_step(i) * kG2Row + acc_col(i)];
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const int64_t row = row_of(acc_col(i), s0 + acc_step(i) - acc_col(i));
                        if (row >= 0) io.x[row] = v[i];
                    }
                }
                lds_publish(s_prog + wi, s0 + 8 * kG2Writers);
            }
            lds_publish(s_prog + wi, INT_MAX);
        } else {
            // ---------------- loaders: runs of kG2Batch consecutive steps in turn, each run in
            // flight at once; a run waits until its slots' previous results were read
            constexpr int B = kG2Batch;
            static_assert(B == 8, "the accesses by row take blocks of 8 steps");
            for (int s0 = (wave - 2 - kG2Writers) * B; s0 < S8; s0 += kG2Loaders * B) {
                uint32_t it = 0;
                bool quit = false;
                for (;;) {
                    int m = INT_MAX;
#pragma unroll
                    for (int k = 0; k < kG2Writers; ++k) m = min(m, lds_load(s_prog + k));
                    if (m >= s0 + B - kG2Ring) break;
                    if (spun_out(it, false)) {
                        quit = true;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(2);
                }
                if (quit) break;
                Pair<T> cv[B];
                T bv[B], pv[B];
#pragma unroll
                for (int u = 0; u < B; ++u) {
                    const int s = s0 + u;
                    const bool in = s < G.S;
                    const T *cp = coef + ((int64_t)c * G.S + (in ? s : 0)) * NC2 * 64;
                    cv[u] = in ? ((const Pair<T> *)cp)[lane] : Pair<T>{};
                    if constexpr (UPPER) pv[u] = in ? cp[128 + lane] : (T)0;
                    const int64_t at = io.bpad ? row_of(lane, s - lane) >= 0 ? p0 + s * pd : -1
                                               : row_of(acc_col(u), s0 + acc_step(u) - acc_col(u));
                    bv[u] = at >= 0 ? io.b[at] : (T)0;
                }
#pragma unroll
                for (int u = 0; u < B; ++u) {
                    const int o = ((s0 + u) & RM) * 64 + lane;
                    cpr[o] = cv[u];
                    if constexpr (UPPER) rpv[o] = pv[u];
                }
                T *const rb = rhs + (s0 & RM) * kG2Row;
#pragma unroll
                for (int u = 0; u < B; ++u)
                    rb[io.bpad ? u * kG2Row + lane : acc_step(u) * kG2Row + acc_col(u)] = bv[u];
                __atomic_signal_fence(__ATOMIC_SEQ_CST);
                if (lane < B)
                    __hip_atomic_store(&filled[(s0 + lane) & RM], s0 + lane, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {  // the last workgroup out resets the counters for the next launch
        const uint32_t d = atomicAdd(&sync[1], 1u);
        if (d == gridDim.x - 1) {
            __hip_atomic_store(&sync[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&sync[1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// Whether every off-diagonal entry of the factor joins neighbours on the grid: *bad is set
// where one does not.
__global__ __launch_bounds__(256) void k_grid_check(int32_t n, int32_t nx, int32_t ny, int32_t nz,
                                                    const int32_t *__restrict__ LUp, const int32_t *__restrict__ LUj,
                                                    int32_t *bad) {
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t x = i % nx, y = (i / nx) % ny, z = i / (nx * ny);
    bool ok = true;
    for (int32_t e = LUp[i]; e < LUp[i + 1]; ++e) {
        const int32_t d = LUj[e] - i, a = d < 0 ? -d : d;
        if (d == 0) continue;
        // (nx or ny may be 1: any of the axes an offset fits will do)
        ok = ok && ((a == 1 && (d < 0 ? x > 0 : x + 1 < nx)) || (a == nx && (d < 0 ? y > 0 : y + 1 < ny)) ||
                    (a == nx * ny && (d < 0 ? z > 0 : z + 1 < nz)));
    }
    if (!ok) *bad = 1;
}

// Packed coefficients of a wavefront plan, one thread per step and lane: the factor's
// values at the row's neighbours behind it (0 where it has none, or where the lane has no
// row) and, for the upper triangle, the reciprocal of the pivot. 3D grid: [claim][step][k]
// [lane] with k = back, below, left, reciprocal. 2D grid: per step the pairs (back, left)
// of the 64 lanes, then the reciprocal of each.
template <class T>
__global__ __launch_bounds__(256) void k_grid_coef(int64_t total, int upper, int32_t NA, int32_t NB, int32_t NC,
                                                   int32_t PA, int32_t PB, int TA, int32_t S, int64_t sa, int64_t sb,
                                                   int64_t sc, const int32_t *__restrict__ LUp,
                                                   const int32_t *__restrict__ LUj, const int32_t *__restrict__ diag,
                                                   const double *__restrict__ LUx, T *__restrict__ out) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= total) return;
    const int lane = (int)(q & 63);
    const int64_t cs = q >> 6;  // claim * S + step
    const int64_t claim = cs / S;
    const plan::GridCell g = plan::grid_cell(NA, NB, NC, PA, PB, TA, upper != 0, claim, lane, (int32_t)(cs - claim * S));
    T v[4] = {};
    if (g.valid) {
        const int64_t row = g.ga * sa + g.gb * sb + g.gc * sc;
        const int64_t sg = upper ? 1 : -1;
        const int32_t d = diag[row];
        const int32_t e0 = upper ? d + 1 : LUp[row], e1 = upper ? LUp[row + 1] : d;
        for (int32_t e = e0; e < e1; ++e) {
            const int64_t o = (LUj[e] - row) * sg;
            const T a = (T)LUx[e];
            if (o == sc) v[0] = a;
            else if (o == sb) v[1] = a;
            else if (o == sa) v[2] = a;
        }
        if (upper) v[3] = (T)1 / (T)LUx[d];
    }
    if (TA == plan::kGT) {
        T *const o = out + cs * 64 * (3 + upper) + lane;
        for (int k = 0; k < 3 + upper; ++k) o[k * 64] = v[k];
    } else {
        T *const o = out + cs * 64 * (2 + upper);
        ((Pair<T> *)o)[lane] = Pair<T>{v[0], v[2]};
        if (upper) o[128 + lane] = v[3];
    }
}

// The pivots of an upper wavefront plan, one thread per step and lane (1 where it has no row).
template <class T>
__global__ __launch_bounds__(256) void k_grid_piv(int64_t total, int32_t NA, int32_t NB, int32_t NC, int32_t PA,
                                                  int32_t PB, int TA, int32_t S, int64_t sa, int64_t sb, int64_t sc,
                                                  const int32_t *__restrict__ diag, const double *__restrict__ LUx,
                                                  T *__restrict__ out) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= total) return;
    const int64_t claim = (q >> 6) / S;
    const plan::GridCell g =
        plan::grid_cell(NA, NB, NC, PA, PB, TA, true, claim, (int)(q & 63), (int32_t)((q >> 6) - claim * S));
    out[q] = g.valid ? (T)LUx[diag[g.ga * sa + g.gb * sb + g.gc * sc]] : (T)1;
}

// Before a single-triangle solve: the output filled with the sentinel.
template <class T>
__global__ __launch_bounds__(256) void k_trsv_fill(int64_t n, T *x, const int32_t *skip) {
    if (skip && *skip) return;
    int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q < n) x[q] = from_bits<T>(Sentinel<T>::bits);
}

// dst[q] = src[map[q]] (0 where map[q] < 0), optional FP32 copy.
__global__ __launch_bounds__(256) void k_gather(size_t n, const int32_t *__restrict__ map,
                                                const double *__restrict__ src, double *__restrict__ dst,
                                                float *__restrict__ dst32) {
    size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    int32_t m = map[q];
    double v = m >= 0 ? src[m] : 0.0;
    dst[q] = v;
    if (dst32) dst32[q] = (float)v;
}

int max_lds_per_block() {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 64 * 1024;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess || v <= 0)
        return 64 * 1024;
    return std::min(v, 160 * 1024);
}

template <class T, bool UPPER>
void launch_blk(const hec_tri &tri, uint32_t *sync, uint32_t *err, const SolveIO<T> &io, hipStream_t s,
                const int32_t *skip) {
    const uint32_t spin = spin_limit();
    T *const yother = io.yother;
    if (tri.nparts == 0 && tri.nitems == 0) return;
    const bool f64 = sizeof(T) == 8;
    if (!tri.blocked) {
        const T *val = f64 ? (const T *)tri.val.get() : (const T *)tri.val32.get();
        const T *piv = UPPER ? (f64 ? (const T *)tri.piv.get() : (const T *)tri.piv32.get()) : nullptr;
        const int grid = std::min((tri.nitems + kRowWaves - 1) / kRowWaves, 256);
        k_trsv_row<T, UPPER><<<grid, 64 * kRowWaves, 0, s>>>(tri.nitems, (const int2 *)tri.items.get(),
                                                             tri.row_ptr.get(), tri.grow.get(),
                                                             yother ? tri.other.get() : nullptr, tri.enc.get(), val,
                                                             piv, io, sync, skip, err, spin);
        HEC_CHECK_LAUNCH();
        return;
    }
    const size_t lds = f64 ? tri.lds64 : tri.lds32;
    PlanArgs P{tri.nparts, tri.K, tri.ldq, tri.W, f64 ? tri.D64 : tri.D32, tri.S,
               tri.part_ss.get(), tri.part_pos.get(), tri.ss_pos.get(), tri.ss_need.get(), tri.grow.get(),
               yother ? tri.other.get() : nullptr, tri.enc.get(), err, spin};
    const T *val, *piv = nullptr;
    if constexpr (sizeof(T) == 8) {
        val = tri.val.get();
        if (UPPER) piv = tri.piv.get();
    } else {
        val = tri.val32.get();
        if (UPPER) piv = tri.piv32.get();
    }
    const int grid = std::min(tri.nparts, 256);
    auto go = [&](auto kc, auto ns) {
        constexpr int KC = decltype(kc)::value, NS = decltype(ns)::value;
        static bool attr_set = false;  // one per instantiation
        if (!attr_set) {
            HEC_HIP(hipFuncSetAttribute((const void *)k_trsv_blk<T, UPPER, KC, NS>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, max_lds_per_block()));
            attr_set = true;
        }
        k_trsv_blk<T, UPPER, KC, NS><<<grid, kBlkThreads, lds, s>>>(P, val, piv, io, sync, skip);
    };
    // the planner gives 1 or plan::kSolvers solver wavefronts
    auto go_kc = [&](auto ns) {
        switch (tri.KC) {
            case 4: go(std::integral_constant<int, 4>(), ns); break;
            case 8: go(std::integral_constant<int, 8>(), ns); break;
            case 16: go(std::integral_constant<int, 16>(), ns); break;
            default: go(std::integral_constant<int, 32>(), ns); break;
        }
    };
    if (tri.NS == 1)
        go_kc(std::integral_constant<int, 1>());
    else if constexpr (plan::kSolvers > 1)
        go_kc(std::integral_constant<int, plan::kSolvers>());
    HEC_CHECK_LAUNCH();
}

template <class T, bool UPPER>
void launch_grid(const hec_grid &g, uint32_t *sync, uint32_t *err, const GridIO<T> &io, hipStream_t s,
                 const int32_t *skip) {
    const int32_t nclaims = g.PA * g.PB;
    GridArgs G{g.NA, g.NB, g.NC, g.PA, g.PB, g.S, nclaims, g.sa, g.sb, g.sc, err, spin_limit()};
    const T *coef;
    if constexpr (sizeof(T) == 8)
        coef = g.coef.get();
    else
        coef = g.coef32.get();
    const int grid = std::min(nclaims, 1024);
    auto go = [&](auto kernel, size_t lds, int waves, bool &attr_set) {
        if (!attr_set) {
            HEC_HIP(hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
            attr_set = true;
        }
        kernel<<<grid, 64 * waves, lds, s>>>(G, coef, io, sync, skip);
    };
    static bool attr3 = false, attr2 = false;  // one per instantiation
    static_assert(grid_lds_bytes<T, UPPER>() <= 160 * 1024 && grid2_lds_bytes<T, UPPER>() <= 160 * 1024, "LDS");
    if (g.TA == plan::kGT)
        go(k_trsv_grid<T, UPPER>, grid_lds_bytes<T, UPPER>(), kGridWaves, attr3);
    else
        go(k_trsv_grid2<T, UPPER>, grid2_lds_bytes<T, UPPER>(), kG2Waves, attr2);
    HEC_CHECK_LAUNCH();
}

// The wavefront path of trsv_launch (both triangles have grid plans; not RAS).
template <class T>
void trsv_launch_grid(const hec_levels_s &lv, uint32_t which, const T *b, T *x, hipStream_t s,
                      const int32_t *skip) {
    T *fL, *fU, *yp;
    if constexpr (sizeof(T) == 8) {
        fL = lv.fL64.get();
        fU = lv.fU64.get();
        yp = lv.yp64.get();
    } else {
        fL = lv.fL32.get();
        fU = lv.fU32.get();
        yp = lv.yp32.get();
    }
    const int64_t nface = lv.lower.grid.face_elems();
    uint32_t *sync = const_cast<uint32_t *>(lv.sync.get());
    uint32_t *err = sync + kLevelsErrWord;
    if (which == HEC_LU) {
        // fL is sentinel-filled between chains (by level_schedule, then by every upper
        // launch); the lower launch fills fU for the upper one
        // the intermediate goes through yp in padded tile-step order
        launch_grid<T, false>(lv.lower.grid, sync, err, GridIO<T>{b, yp, fL, fU, nface, 0, 1}, s, skip);
        launch_grid<T, true>(lv.upper.grid, sync + 2, err, GridIO<T>{yp, x, fU, fL, nface, 1, 0}, s, skip);
        return;
    }
    // a lone triangle: fU, free between calls, is filled right before
    k_trsv_fill<T><<<ceil_div(nface, 256), 256, 0, s>>>(nface, fU, skip);
    HEC_CHECK_LAUNCH();
    if (which == HEC_LOWER)
        launch_grid<T, false>(lv.lower.grid, sync, err, GridIO<T>{b, x, fU, nullptr, 0}, s, skip);
    else
        launch_grid<T, true>(lv.upper.grid, sync + 2, err, GridIO<T>{b, x, fU, nullptr, 0}, s, skip);
}

}  // namespace

template <class T>
void trsv_launch(const hec_levels_s &lv, uint32_t which, const T *b, T *x, hipStream_t s, const int32_t *skip) {
    const int64_t n = lv.n, nf = lv.nf;
    if (n == 0) return;
    T *qL, *qU, *yp;
    if constexpr (sizeof(T) == 8) {
        qL = lv.qL64.get();
        qU = lv.qU64.get();
        yp = lv.yp64.get();
    } else {
        qL = lv.qL32.get();
        qU = lv.qU32.get();
        yp = lv.yp32.get();
    }
    if (lv.lower.grid.on && lv.upper.grid.on) {
        trsv_launch_grid<T>(lv, which, b, x, s, skip);
        return;
    }
    uint32_t *sync = const_cast<uint32_t *>(lv.sync.get());
    uint32_t *err = sync + kLevelsErrWord;
    if (which == HEC_LU) {
        // qL is sentinel-filled between calls (by level_schedule, then by every upper
        // launch); the lower launch fills qU for the upper one: two launches in all.
        // Restricted additive Schwarz: the lower solve reads b through the stacked
        // rows' system rows (bmap); the upper solve writes each owned row's result to
        // x through `other`, overlap rows nowhere.
        if (lv.ras) {
            launch_blk<T, false>(lv.lower, sync, err, SolveIO<T>{b, lv.lower.bmap.get(), 0, qL, nullptr, yp, qU, nf}, s,
                                 skip);
            launch_blk<T, true>(lv.upper, sync + 2, err, SolveIO<T>{yp, nullptr, 0, qU, nullptr, x, qL, nf}, s, skip);
        } else {
            launch_blk<T, false>(lv.lower, sync, err, SolveIO<T>{b, nullptr, 1, qL, nullptr, yp, qU, nf}, s, skip);
            launch_blk<T, true>(lv.upper, sync + 2, err, SolveIO<T>{yp, nullptr, 0, qU, x, nullptr, qL, nf}, s, skip);
        }
        return;
    }
    // one triangle: qU, free between calls, holds the polled copy; qL keeps its fill
    k_trsv_fill<T><<<ceil_div(nf, 256), 256, 0, s>>>(nf, qU, skip);
    HEC_CHECK_LAUNCH();
    if (which == HEC_LOWER)
        launch_blk<T, false>(lv.lower, sync, err, SolveIO<T>{b, nullptr, 1, qU, x, nullptr, nullptr, 0}, s, skip);
    else
        launch_blk<T, true>(lv.upper, sync + 2, err, SolveIO<T>{b, nullptr, 1, qU, x, nullptr, nullptr, 0}, s, skip);
}

void trsv_init_levels(hec_levels_s &lv, hipStream_t s) {
    const int64_t n = lv.nf;
    if (n == 0) return;
    if (lv.qL64.get()) {
        k_trsv_fill<double><<<ceil_div(n, 256), 256, 0, s>>>(n, lv.qL64.get(), nullptr);
        HEC_CHECK_LAUNCH();
    }
    if (lv.qL32.get()) {
        k_trsv_fill<float><<<ceil_div(n, 256), 256, 0, s>>>(n, lv.qL32.get(), nullptr);
        HEC_CHECK_LAUNCH();
    }
    const int64_t nface = lv.fL64.get() ? lv.lower.grid.face_elems() : 0;
    if (nface) {
        k_trsv_fill<double><<<ceil_div(nface, 256), 256, 0, s>>>(nface, lv.fL64.get(), nullptr);
        HEC_CHECK_LAUNCH();
        if (lv.fL32.get()) {
            k_trsv_fill<float><<<ceil_div(nface, 256), 256, 0, s>>>(nface, lv.fL32.get(), nullptr);
            HEC_CHECK_LAUNCH();
        }
    }
}

void level_only(const hec_ilu_s &M, bool upper, hec_tri &tri) {
    if (!upper) {  // kept from the factorisation
        tri.nlev = (int32_t)M.hlptr.size() - 1;
        tri.hlevel_ptr = M.hlptr;
        tri.hperm = M.hlperm;
        return;
    }
    tri.nlev = plan::compute_levels(M.n, M.hLUp.data(), M.hLUj.data(), M.hdiag.data(), upper, tri.hlevel_ptr,
                                    tri.hperm);
}

void build_grid(const hec_ilu_s &M, hec_grid &lower, hec_grid &upper, hipStream_t s) {
    lower = hec_grid();
    upper = hec_grid();
    plan::GridPlan P[2];
    for (int u = 0; u < 2; ++u)
        if (!plan::grid_plan_shape(M.n, M.gnx, M.gny, M.gnz, u != 0, P[u])) return;
    DevBuf<int32_t> bad(1);
    int32_t hbad = 0;
    HEC_HIP(hipMemsetAsync(bad.get(), 0, sizeof(int32_t), s));
    k_grid_check<<<ceil_div(M.n, 256), 256, 0, s>>>(M.n, M.gnx, M.gny, M.gnz, M.LUp.get(), M.LUj.get(), bad.get());
    HEC_CHECK_LAUNCH();
    bad.download(&hbad, 1, s);
    HEC_HIP(hipStreamSynchronize(s));
    if (hbad) return;
    for (int u = 0; u < 2; ++u) {
        hec_grid &g = u ? upper : lower;
        const plan::GridPlan &Q = P[u];
        g.TA = Q.TA;
        g.NA = Q.NA;
        g.NB = Q.NB;
        g.NC = Q.NC;
        g.PA = Q.PA;
        g.PB = Q.PB;
        g.S = Q.S;
        g.sa = Q.sa;
        g.sb = Q.sb;
        g.sc = Q.sc;
        const int64_t total = g.pad_elems();
        const int ncoef = Q.ncoef - (g.TA == plan::kGT2 ? 1 : 0);
        auto pack = [&](auto &buf) {
            buf.alloc((size_t)total * ncoef);
            k_grid_coef<<<ceil_div(total, 256), 256, 0, s>>>(total, u, g.NA, g.NB, g.NC, g.PA, g.PB, g.TA, g.S, g.sa,
                                                             g.sb, g.sc, M.LUp.get(), M.LUj.get(), M.diag.get(),
                                                             M.LUx.get(), buf.get());
            HEC_CHECK_LAUNCH();
        };
        pack(g.coef);
        if (M.has_f32) pack(g.coef32);
        g.on = true;
    }
}

void build_grid_pivots(const hec_ilu_s &M, hec_grid &g, hipStream_t s) {
    const int64_t total = g.pad_elems();
    auto pack = [&](auto &buf) {
        buf.alloc((size_t)total);
        k_grid_piv<<<ceil_div(total, 256), 256, 0, s>>>(total, g.NA, g.NB, g.NC, g.PA, g.PB, g.TA, g.S, g.sa, g.sb,
                                                        g.sc, M.diag.get(), M.LUx.get(), buf.get());
        HEC_CHECK_LAUNCH();
    };
    pack(g.piv);
    if (M.has_f32) pack(g.piv32);
}

template void trsv_launch<double>(const hec_levels_s &, uint32_t, const double *, double *, hipStream_t,
                                  const int32_t *);
template void trsv_launch<float>(const hec_levels_s &, uint32_t, const float *, float *, hipStream_t,
                                 const int32_t *);

void build_tri(const hec_ilu_s &M, bool upper, hec_tri &tri, const hec_tri *upper_plan, hipStream_t s) {
    const int32_t n = M.n;
    plan::HostPlan P;
    plan::make_plan(n, M.hLUp.data(), M.hLUj.data(), M.hdiag.data(), M.gnx, M.gny, M.gnz, upper, M.has_f32,
                    max_lds_per_block() - 256, P, false, M.hblocks.empty() ? nullptr : &M.hblocks, plan::kSolvers, 0,
                    false);
    std::vector<int32_t> rptr, items;  // row-polling plan: entry ranges and items (first position, rows)
    if (n > 0 && !P.blocked)
        plan::make_row_plan(n, M.hLUp.data(), M.hLUj.data(), M.hdiag.data(), upper, kRowShort, kRowGroup, P, rptr,
                            items);
    tri.nlev = P.nlev;
    tri.hlevel_ptr = std::move(P.level_ptr);
    tri.hperm = std::move(P.perm);
    tri.K = P.K;
    tri.KC = P.KC;
    tri.ldq = P.ldq;
    if (n == 0) return;
    tri.blocked = P.blocked;
    tri.nparts = P.nparts;
    tri.nss = P.nss;
    tri.W = P.W;
    tri.S = P.S;
    tri.D64 = P.D64;
    tri.D32 = P.D32;
    tri.lds64 = P.lds64;
    tri.lds32 = P.lds32;
    if (!P.blocked) {
        tri.nitems = (int32_t)items.size() / 2;
        tri.items.alloc(items.size());
        tri.items.upload(items.data(), items.size(), s);
        tri.row_ptr.alloc(rptr.size());
        tri.row_ptr.upload(rptr.data(), rptr.size(), s);
    }
    tri.part_ss.alloc(P.part_ss.size());
    tri.part_ss.upload(P.part_ss.data(), P.part_ss.size(), s);
    tri.part_pos.alloc(P.part_pos.size());
    tri.part_pos.upload(P.part_pos.data(), P.part_pos.size(), s);
    tri.ss_pos.alloc(P.ss_pos.size());
    tri.ss_pos.upload(P.ss_pos.data(), P.ss_pos.size(), s);
    tri.NS = P.NS;
    if (!P.ss_need.empty()) {
        tri.ss_need.alloc(P.ss_need.size());
        tri.ss_need.upload(P.ss_need.data(), P.ss_need.size(), s);
    }
    tri.grow.alloc(n);
    tri.grow.upload(P.grow.data(), n, s);
    const bool ras = !M.hext_row.empty();
    if (ras && !upper) {  // right-hand side of each position: the system row of its stacked row
        std::vector<int32_t> bm(n);
        for (int32_t q = 0; q < n; ++q) bm[q] = M.hext_row[P.grow[q]];
        tri.bmap.alloc(n);
        tri.bmap.upload(bm.data(), n, s);
        HEC_HIP(hipStreamSynchronize(s));
    }
    if (ras && upper) {  // owned rows write their result to the system vector, overlap rows nowhere
        std::vector<int32_t> om(n);
        for (int32_t q = 0; q < n; ++q) {
            const int32_t row = P.grow[q], sys = M.hext_row[row];
            om[q] = M.hown[sys] == row ? sys : -1;
        }
        tri.other.alloc(n);
        tri.other.upload(om.data(), n, s);
        HEC_HIP(hipStreamSynchronize(s));
    }
    if (!upper && upper_plan) {
        // position of each lower-plan row in the upper plan
        std::vector<int32_t> up_pos(n), other(n);
        for (int32_t q = 0; q < n; ++q) up_pos[upper_plan->hgrow[q]] = q;
        for (int32_t q = 0; q < n; ++q) other[q] = up_pos[P.grow[q]];
        tri.other.alloc(n);
        tri.other.upload(other.data(), n, s);
        HEC_HIP(hipStreamSynchronize(s));  // `other` is uploaded from host memory that ends here
    }
    const size_t slab = P.enc.size();  // K * ldq slots, or the entries of a row-polling plan
    tri.enc.alloc(slab);
    tri.enc.upload(P.enc.data(), slab, s);
    tri.val.alloc(slab);
    if (M.has_f32) tri.val32.alloc(slab);
    DevBuf<int32_t> dsrc(slab);
    if (slab) {
        dsrc.upload(P.src.data(), slab, s);
        k_gather<<<ceil_div(slab, 256), 256, 0, s>>>(slab, dsrc.get(), M.LUx.get(), tri.val.get(), tri.val32.get());
        HEC_CHECK_LAUNCH();
    }
    DevBuf<int32_t> dp;
    if (upper) {
        tri.piv.alloc(tri.ldq);
        if (M.has_f32) tri.piv32.alloc(tri.ldq);
        dp.alloc(tri.ldq);
        dp.upload(P.psrc.data(), tri.ldq, s);
        k_gather<<<ceil_div(tri.ldq, 256), 256, 0, s>>>(tri.ldq, dp.get(), M.LUx.get(), tri.piv.get(),
                                                        tri.piv32.get());
        HEC_CHECK_LAUNCH();
    }
    HEC_HIP(hipStreamSynchronize(s));
    tri.hgrow = std::move(P.grow);
}

void build_flat(const hec_ilu_s &M, bool upper, hec_tri &tri, hipStream_t s) {
    const int32_t n = M.n;
    plan::HostPlan P;
    plan::make_plan(n, M.hLUp.data(), M.hLUj.data(), M.hdiag.data(), 0, 0, 0, upper, M.has_f32, 0, P, true);
    hec_flat &f = tri.flat;
    f.K = P.K;
    f.ldq = P.ldq;
    f.nchunks = n ? (int32_t)P.chunks.size() - 1 : 0;
    if (n == 0) return;
    f.chunk_ptr.alloc(P.chunks.size());
    f.chunk_ptr.upload(P.chunks.data(), P.chunks.size(), s);
    f.row.alloc(n);
    f.row.upload(P.grow.data(), n, s);
    const size_t slab = (size_t)P.K * P.ldq;
    f.col.alloc(slab);
    f.col.upload(P.enc.data(), slab, s);
    f.val.alloc(slab);
    if (M.has_f32) f.val32.alloc(slab);
    DevBuf<int32_t> dsrc(slab);
    if (slab) {
        dsrc.upload(P.src.data(), slab, s);
        k_gather<<<ceil_div(slab, 256), 256, 0, s>>>(slab, dsrc.get(), M.LUx.get(), f.val.get(), f.val32.get());
        HEC_CHECK_LAUNCH();
    }
    DevBuf<int32_t> dp;
    if (upper) {
        f.piv.alloc(P.ldq);
        if (M.has_f32) f.piv32.alloc(P.ldq);
        dp.alloc(P.ldq);
        dp.upload(P.psrc.data(), P.ldq, s);
        k_gather<<<ceil_div(P.ldq, 256), 256, 0, s>>>(P.ldq, dp.get(), M.LUx.get(), f.piv.get(), f.piv32.get());
        HEC_CHECK_LAUNCH();
    }
    HEC_HIP(hipStreamSynchronize(s));
}

}  // namespace hec
