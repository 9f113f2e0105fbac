// ILU(k) (Sec. 2.4, Eq. (7)-(10), Alg. 2) and level schedules (Sec. 2.6,
// Eq. (11), Alg. 3), plus their C entry points and trsv_levels'.
//
// Symbolic work (the fill pattern S_k, the levels) is integer work done once
// per matrix on the host. The numeric factorisation runs on the device, in one
// launch whose rows wait for the rows they eliminate with.
#include <algorithm>
#include <cmath>
#include <memory>

#include "hec_internal.hpp"

namespace hec {

// ------------------------------------------------------------------ host symbolic work

// Symbolic ILU(k): S_k = {(i,j) : level(i,j) <= k} with the level rule of
// Eq. (9)-(10). Row i starts from A's pattern at level 0; pivots p < i are
// taken in increasing order and each merges the kept upper part of row p with
// level lev(i,p) + lev(p,j) + 1. Candidates above k are never inserted: they
// can neither be kept nor act as pivots.
static void symbolic_iluk(int32_t n, const int32_t *Ap, const int32_t *Aj, int32_t k,
                          std::vector<int32_t> &LUp, std::vector<int32_t> &LUj, std::vector<int32_t> &diag) {
    LUp.assign(n + 1, 0);
    diag.assign(n, -1);
    LUj.clear();
    if (k == 0) {
        LUj.assign(Aj, Aj + Ap[n]);
        for (int32_t i = 0; i <= n; ++i) LUp[i] = Ap[i];
        for (int32_t i = 0; i < n; ++i)
            for (int32_t e = Ap[i]; e < Ap[i + 1] && diag[i] < 0; ++e)
                if (Aj[e] == i) diag[i] = e;
        return;
    }
    LUj.reserve((size_t)Ap[n] * 2);
    std::vector<int32_t> LUlev;
    LUlev.reserve((size_t)Ap[n] * 2);
    std::vector<std::pair<int32_t, int32_t>> row;  // (column, level), ascending column
    for (int32_t i = 0; i < n; ++i) {
        row.clear();
        for (int32_t e = Ap[i]; e < Ap[i + 1]; ++e) row.emplace_back(Aj[e], 0);
        for (size_t t = 0; t < row.size() && row[t].first < i; ++t) {
            int32_t p = row[t].first, lp = row[t].second;
            // merge the upper part of row p (final, kept entries only)
            size_t pos = t + 1;
            for (int32_t u = diag[p] + 1; u < LUp[p + 1]; ++u) {
                int32_t j = LUj[u];
                int32_t lv = lp + LUlev[u] + 1;
                if (lv > k) continue;
                while (pos < row.size() && row[pos].first < j) ++pos;
                if (pos < row.size() && row[pos].first == j) {
                    if (lv < row[pos].second) row[pos].second = lv;
                } else {
                    row.insert(row.begin() + pos, std::make_pair(j, lv));
                }
            }
        }
        for (auto &cl : row) {
            if (cl.first == i) diag[i] = (int32_t)LUj.size();
            LUj.push_back(cl.first);
            LUlev.push_back(cl.second);
        }
        LUp[i + 1] = (int32_t)LUj.size();
    }
}

// ------------------------------------------------------------------ numeric ILU kernel

// Numeric elimination (Alg. 2 restricted to S_k) in one launch. Some lanes take a row i: for
// each stored p < i in ascending order, l_ip = a_ip / u_pp, then a_ij -= l_ip * u_pj for every
// stored (p, j), j > p, that is also in row i, the lanes taking the entries of row p. A row is
// worked on apart (in LDS, or where it is too long for that in its entries of `in`) and written
// to `out` once; `out` starts filled with a signalling NaN that arithmetic never produces, so an
// entry of row p is polled until it is final (device-coherent accesses).
// Workgroups claim four items from a ticket counter, a wavefront each, the next claim on its
// way meanwhile: an item, rows of one level of L, only waits for items of earlier levels,
// claimed before it by running workgroups. Every wait is bounded (spin_limit).
//
// An item is up to four rows of at most kIluShort entries, 16 lanes each, or one longer row
// with the whole wavefront: chosen row by row, so that a long row costs the others nothing.
// Four rows of kIluShort (7.5 KB) and one of kIluLds (10 KB) take a wavefront about the same LDS:
// 40 KB a workgroup, three of them on a compute unit. Rows beyond kIluLds look their columns up
// and keep their values in memory. With kIluLds = 97, 256, 512 and 1,024 a 60,000-row power-law
// matrix (rows of 4 to 512) takes 1.71, 1.63, 1.38 and 1.78 ms, 20,000 rows of 4 to 2,000 2.31,
// 2.19, 2.24 and 2.78 (514 with a launch per level).
//
// Bound: the chain of levels, each a store and a load between compute units and one
// division and update per pivot. With a launch per level and one thread per row, its
// loads one after another, a level took 15 us (60^3 ILU(0), 178 levels: 2.7 ms), 45 us
// with ILU(1) rows and 9.5 ms with rows of up to 512 entries (60,000-row power-law
// matrix: 285 ms); now 0.57, 2.7 (75 x 62 x 51 ILU(1), 15.4 ms before) and 1.38 ms in all.
// The values are the same bit for bit.
constexpr unsigned long long kIluSent = 0x7FF4DEADBEEF1234ull;
constexpr int kIluShort = 96;  // most entries of a row that shares a wavefront with three others
constexpr int kIluLds = 512;   // most entries of a row worked on in LDS
constexpr int kIluGroup = 4;   // rows of a short item

struct IluArgs {
    int32_t nitems;
    const int2 *items;  // (first row in perm, rows; 0 rows: one row of more than kIluShort entries)
    const int32_t *perm, *LUp, *LUj, *diag;
    double *in;  // start values; a row beyond kIluLds entries is worked on there
    double *out;
    int32_t *zero_pivot;
    uint32_t *sync, *err;  // ticket; set when a wait gave up
    uint32_t spin;         // polls of a wait before it gives up
};

// LDS of a wavefront's rows: per entry its value, its column and, if it is a pivot's, the
// pivot's diagonal and the end of its row.
template <bool LONG>
constexpr int ilu_wave_entries() {
    return LONG && kIluLds > kIluGroup * kIluShort ? kIluLds : kIluGroup * kIluShort;
}
template <bool LONG>
constexpr size_t ilu_lds_bytes() {
    return (size_t)4 * ilu_wave_entries<LONG>() * (sizeof(double) + 3 * sizeof(int32_t));
}

// LONG: there are rows of more than kIluShort entries.
template <bool LONG>
__global__ __launch_bounds__(256) void k_ilu_rows(IluArgs A) {
    using U = unsigned long long;
    extern __shared__ __align__(16) char ism[];
    __shared__ int s_claim[2], s_abort[2];  // by the round's parity
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double *const wvals = (double *)ism + wave * ilu_wave_entries<LONG>();
    int32_t *const wints = (int32_t *)((double *)ism + 4 * ilu_wave_entries<LONG>()) + wave * 3 * ilu_wave_entries<LONG>();
    auto poll = [&](const double *p) {
        return __hip_atomic_load((const U *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto gave_up = [&](uint32_t &it) {  // one more poll of a wait (wave-uniform)
        ++it;
        if (it > A.spin) return true;
        if ((it & 63) == 0 && __hip_atomic_load(A.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u) return true;
        __builtin_amdgcn_s_sleep(1);
        return false;
    };
    struct Piv {  // pivot row p: this lane's entry u of its upper part, its place in row i, and u_pp
        int32_t u, pe, f;
        U v, d;
        const double *pv, *pd;
    };
    constexpr int NP = 4;  // pivots whose entries are waited for together
    // Rows q0 .. q0 + cnt - 1 of perm, G lanes each, in LDS (at most CAP entries) or in `in`
    // (CAP = 0); false: a wait gave up.
    auto factor = [&](auto gc, auto cc, int32_t q0, int32_t cnt) {
        constexpr int G = decltype(gc)::value, CAP = decltype(cc)::value;
        const int g = lane % G, grp = lane / G;
        const bool live = grp < cnt;
        const int32_t i = A.perm[q0 + (live ? grp : 0)];
        const int32_t b0 = A.LUp[i], len = live ? A.LUp[i + 1] - b0 : 0, nl = live ? A.diag[i] - b0 : 0;
        double *const vals = CAP ? wvals + grp * CAP : A.in + b0;
        int32_t *const lcols = wints + grp * 3 * CAP, *const pdiag = lcols + CAP, *const pend = pdiag + CAP;
        const int32_t *const cols = CAP ? lcols : A.LUj + b0;
        auto order = [] {  // what the row's lanes stored is what they read after
            if constexpr (CAP != 0)  // (LDS accesses of a wavefront complete in order: only the compiler is held)
                __atomic_signal_fence(__ATOMIC_SEQ_CST);
            else
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            __builtin_amdgcn_wave_barrier();
        };
        if constexpr (CAP != 0) {
            for (int e = g; e < len; e += G) {
                const int32_t c = A.LUj[b0 + e];
                lcols[e] = c;
                vals[e] = A.in[b0 + e];
                if (e < nl) {
                    pdiag[e] = A.diag[c];
                    pend[e] = A.LUp[c + 1];
                }
            }
        }
        order();
        auto diag_of = [&](int e) { return CAP ? pdiag[e] : A.diag[cols[e]]; };   // of pivot e, in LUx
        auto end_of = [&](int e) { return CAP ? pend[e] : A.LUp[cols[e] + 1]; };  // of pivot e's row
        auto place = [&](int e, int32_t j) -> int32_t {  // of column j in row i past entry e, -1: not stored
            int lo = e + 1, hi = len;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (cols[mid] < j) lo = mid + 1;
                else hi = mid;
            }
            return lo < len && cols[lo] == j ? lo : -1;
        };
        // entry u of pivot e's row (only looked up where row i has its column)
        auto load = [&](int e, int32_t u, bool in, Piv &P) {
            P.u = u;
            P.f = in && u < P.pe ? place(e, A.LUj[u]) : -1;
            P.v = 0;
            if (P.f >= 0) {
                P.pv = A.out + u;
                P.v = poll(P.pv);
            }
        };
        bool stop = false;  // the row met a zero pivot: the rest of it stays as it is
        for (int e0 = 0; __ballot(e0 < nl) != 0; e0 += NP) {
            Piv P[NP];
#pragma unroll
            for (int k = 0; k < NP; ++k) {
                const bool in = e0 + k < nl;
                const int32_t pd = in ? diag_of(e0 + k) : 0;
                P[k].pe = in ? end_of(e0 + k) : 0;
                P[k].pd = P[k].pv = A.out + pd;
                P[k].d = in ? poll(P[k].pd) : 0;
                load(e0 + k, in ? pd + 1 + g : 0, in, P[k]);
            }
            uint32_t it = 0;
            for (;;) {  // until the entries of all NP pivots are final; only the pending ones are loaded again
                bool pending = false;
#pragma unroll
                for (int k = 0; k < NP; ++k) pending |= P[k].v == kIluSent || P[k].d == kIluSent;
                if (__ballot(pending) == 0) break;
                if (gave_up(it)) return false;
#pragma unroll
                for (int k = 0; k < NP; ++k) {
                    if (P[k].v == kIluSent) P[k].v = poll(P[k].pv);
                    if (P[k].d == kIluSent) P[k].d = poll(P[k].pd);
                }
            }
#pragma unroll
            for (int k = 0; k < NP; ++k) {
                const int e = e0 + k;
                const double upp = __longlong_as_double((long long)P[k].d);
                if (e < nl && !stop && upp == 0.0) {
                    if (g == 0) atomicMax(A.zero_pivot, cols[e] + 1);
                    stop = true;
                }
                const bool act = e < nl && !stop;
                const double lip = act ? vals[e] / upp : 0.0;
                order();
                if (act && g == 0) vals[e] = lip;
                if (act && P[k].f >= 0) vals[P[k].f] -= lip * __longlong_as_double((long long)P[k].v);
                // entries of row p past the first G
                for (int32_t u = P[k].u + G; __ballot(act && u < P[k].pe) != 0; u += G) {
                    load(e, u, act, P[k]);
                    it = 0;
                    while (__ballot(P[k].v == kIluSent) != 0) {
                        if (gave_up(it)) return false;
                        if (P[k].v == kIluSent) P[k].v = poll(P[k].pv);
                    }
                    if (act && P[k].f >= 0) vals[P[k].f] -= lip * __longlong_as_double((long long)P[k].v);
                }
                order();
            }
        }
        for (int e = g; e < len; e += G) {
            U v = (U)__double_as_longlong(vals[e]);
            if (v == kIluSent) v = 0x7FF8000000000000ull;  // an input that is the sentinel: a quiet NaN
            __hip_atomic_store((U *)(A.out + b0 + e), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        order();
        return true;
    };
    auto item_rows = [&](int2 item) {
        const int32_t q0 = __builtin_amdgcn_readfirstlane(item.x), cnt = __builtin_amdgcn_readfirstlane(item.y);
        if constexpr (LONG) {
            if (cnt == 0) {
                const int32_t i = A.perm[q0];
                const int32_t len = __builtin_amdgcn_readfirstlane(A.LUp[i + 1] - A.LUp[i]);
                if (len <= kIluLds)
                    return factor(std::integral_constant<int, 64>(), std::integral_constant<int, kIluLds>(), q0, 1);
                return factor(std::integral_constant<int, 64>(), std::integral_constant<int, 0>(), q0, 1);
            }
        }
        return factor(std::integral_constant<int, 64 / kIluGroup>(), std::integral_constant<int, kIluShort>(), q0, cnt);
    };
    if (threadIdx.x == 0) {
        s_abort[0] = s_abort[1] = 0;
        s_claim[0] = (int)atomicAdd(A.sync, 1u);
    }
    for (int round = 0;; ++round) {
        __syncthreads();
        const int c = s_claim[round & 1];
        if (s_abort[round & 1] || (int64_t)c * 4 >= A.nitems) break;  // uniform: read after the barrier
        uint32_t next = 0;
        if (threadIdx.x == 0) next = atomicAdd(A.sync, 1u);
        const int t = c * 4 + wave;
        if (t < A.nitems && !item_rows(A.items[t])) {
            __hip_atomic_store(A.err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_abort[(round + 1) & 1] = 1;
        }
        if (threadIdx.x == 0) s_claim[(round + 1) & 1] = (int)next;
    }
}

__global__ __launch_bounds__(256) void k_ilu_fill(size_t n, double *__restrict__ out) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) ((unsigned long long *)out)[i] = kIluSent;
}

// Where a wait of k_ilu_rows gave up or its start values find no memory: the rows of one level
// of L a launch, one thread per row, in place; all rows p were finished by earlier launches.
__global__ __launch_bounds__(256) void k_ilu_level(int32_t cnt, const int32_t *__restrict__ rows,
                                                   const int32_t *__restrict__ LUp,
                                                   const int32_t *__restrict__ LUj,
                                                   const int32_t *__restrict__ diag, double *LUx,
                                                   int32_t *zero_pivot) {
    int32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= cnt) return;
    int32_t i = rows[t];
    int32_t b = LUp[i + 1], di = diag[i];
    for (int32_t e = LUp[i]; e < di; ++e) {
        int32_t p = LUj[e];
        int32_t dp = diag[p];
        double upp = LUx[dp];
        if (upp == 0.0) {
            atomicMax(zero_pivot, p + 1);
            return;
        }
        double lip = LUx[e] / upp;
        LUx[e] = lip;
        int32_t f = e + 1;
        int32_t pe = LUp[p + 1];
        for (int32_t u = dp + 1; u < pe && f < b; ++u) {
            int32_t j = LUj[u];
            while (f < b && LUj[f] < j) ++f;
            if (f < b && LUj[f] == j) LUx[f] -= lip * LUx[u];
        }
    }
}

__global__ __launch_bounds__(256) void k_check_diag(int32_t n, const int32_t *__restrict__ diag,
                                                    const double *__restrict__ LUx, int32_t *zero_pivot) {
    int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n && LUx[diag[i]] == 0.0) atomicMax(zero_pivot, i + 1);
}

template <class S, class D>
__global__ __launch_bounds__(256) void k_convert(size_t n, const S *__restrict__ src, D *__restrict__ dst) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = (D)src[i];
}

}  // namespace hec

using namespace hec;

// The numeric phase in one launch (k_ilu_rows): M's values from x0, its entries' start values.
// zero_pivot: 0, or one past a row whose pivot is zero. false: M's values are not formed (a wait
// gave up, or no memory for the start values beside the factor's).
static bool numeric_rows(hec_ilu_s &M, int32_t nlev, const double *x0, int32_t &zero_pivot, hipStream_t s) {
    const int32_t n = M.n;
    enum : int { FLAG = 0, TICKET = 1, ERR = 2, NFLAGS = 4 };  // zero pivot (row + 1), claims, given up
    auto is_long = [&](int32_t i) { return M.hLUp[i + 1] - M.hLUp[i] > kIluShort; };
    bool any_long = false;
    for (int32_t i = 0; i < n && !any_long; ++i) any_long = is_long(i);
    std::vector<int32_t> perm, items;  // perm: inside each level the long rows, which take longest, first
    items.reserve(2 * ((size_t)n / kIluGroup + nlev));
    if (any_long) perm = M.hlperm;
    for (int32_t l = 0; l < nlev; ++l) {
        const int32_t b = M.hlptr[l + 1];
        int32_t q = M.hlptr[l];
        if (any_long) {
            const int32_t a = q;
            q = (int32_t)(std::stable_partition(perm.begin() + a, perm.begin() + b, is_long) - perm.begin());
            for (int32_t t = a; t < q; ++t) items.insert(items.end(), {t, 0});
        }
        for (; q < b; q += kIluGroup) {
            items.push_back(q);
            items.push_back(std::min(kIluGroup, b - q));
        }
    }
    const int32_t nitems = (int32_t)(items.size() / 2);
    if (nitems == 0) return true;
    DevBuf<int32_t> dperm, dflag, ditems;
    DevBuf<double> din;
    try {
        dperm.alloc(n);
        dflag.alloc(NFLAGS);
        ditems.alloc(items.size());
        din.alloc(M.nnz);
    } catch (const Error &e) {
        if (e.code != HEC_ERR_NOMEM) throw;
        (void)hipGetLastError();  // not for the next launch's check
        return false;
    }
    dperm.upload(any_long ? perm.data() : M.hlperm.data(), n, s);
    ditems.upload(items.data(), items.size(), s);
    din.upload(x0, M.nnz, s);
    HEC_HIP(hipMemsetAsync(dflag.get(), 0, NFLAGS * sizeof(int32_t), s));
    k_ilu_fill<<<ceil_div(M.nnz, 256), 256, 0, s>>>(M.nnz, M.LUx.get());
    HEC_CHECK_LAUNCH();
    const IluArgs args{nitems,       (const int2 *)ditems.get(), dperm.get(),  M.LUp.get(), M.LUj.get(),
                       M.diag.get(), din.get(),                  M.LUx.get(), dflag.get() + FLAG,
                       (uint32_t *)dflag.get() + TICKET, (uint32_t *)dflag.get() + ERR, spin_limit()};
    const unsigned grid = std::min(ceil_div(nitems, 4), 1024u);
    if (any_long)
        k_ilu_rows<true><<<grid, 256, ilu_lds_bytes<true>(), s>>>(args);
    else
        k_ilu_rows<false><<<grid, 256, ilu_lds_bytes<false>(), s>>>(args);
    HEC_CHECK_LAUNCH();
    int32_t hflag[NFLAGS] = {};
    dflag.download(hflag, NFLAGS, s);
    HEC_HIP(hipStreamSynchronize(s));
    zero_pivot = hflag[FLAG];
    return hflag[ERR] == 0;
}

// The same with a launch per level (k_ilu_level), which waits for nothing and works in place:
// what numeric_rows could not form.
static void numeric_levels(hec_ilu_s &M, int32_t nlev, const double *x0, int32_t &zero_pivot, hipStream_t s) {
    DevBuf<int32_t> dperm(M.n), dflag(1);
    dperm.upload(M.hlperm.data(), M.n, s);
    HEC_HIP(hipMemsetAsync(dflag.get(), 0, sizeof(int32_t), s));
    M.LUx.upload(x0, M.nnz, s);
    for (int32_t l = 1; l < nlev; ++l) {  // level 0 rows have no L entries: nothing to do
        const int32_t a = M.hlptr[l], cnt = M.hlptr[l + 1] - a;
        k_ilu_level<<<ceil_div(cnt, 256), 256, 0, s>>>(cnt, dperm.get() + a, M.LUp.get(), M.LUj.get(), M.diag.get(),
                                                       M.LUx.get(), dflag.get());
        HEC_CHECK_LAUNCH();
    }
    dflag.download(&zero_pivot, 1, s);
    HEC_HIP(hipStreamSynchronize(s));
}

// ILU(k) of a CSR matrix (validated, every diagonal stored): host symbolic phase
// (Eq. (9)-(10)), device numeric phase (Alg. 2 restricted to S_k).
static std::unique_ptr<hec_ilu_s> factor_csr(int32_t n, const int32_t *Ap, const int32_t *Aj, const double *Ax,
                                            int32_t k, uint32_t flags, hipStream_t s) {
    auto M = std::make_unique<hec_ilu_s>();
    OwnerScope own(&M->dev_bytes);
    M->n = n;
    M->k = k;
    M->has_f32 = (flags & HEC_KEEP_F32) != 0;
    symbolic_iluk(n, Ap, Aj, k, M->hLUp, M->hLUj, M->hdiag);
    plan::detect_grid(n, Ap, Aj, M->gnx, M->gny, M->gnz);
    M->nnz = M->hLUp[n];
    // A's values scattered into S_k, fill entries start at 0 (k = 0: S_0 is A's pattern)
    std::vector<double> scat;
    if (M->nnz != Ap[n]) {
        scat.assign(M->nnz, 0.0);
        for (int32_t i = 0; i < n; ++i) {
            int32_t f = M->hLUp[i];
            for (int32_t e = Ap[i]; e < Ap[i + 1]; ++e) {
                while (M->hLUj[f] < Aj[e]) ++f;
                scat[f] = Ax[e];
            }
        }
    }
    const double *x0 = scat.empty() ? Ax : scat.data();
    M->LUp.alloc(n + 1);
    M->LUj.alloc(M->nnz);
    M->diag.alloc(n);
    M->LUx.alloc(M->nnz);
    M->LUp.upload(M->hLUp.data(), n + 1, s);
    M->LUj.upload(M->hLUj.data(), M->nnz, s);
    M->diag.upload(M->hdiag.data(), n, s);
    // numeric elimination in level order of L
    const int32_t nlev =
        plan::compute_levels(n, M->hLUp.data(), M->hLUj.data(), M->hdiag.data(), false, M->hlptr, M->hlperm);
    int32_t zp = 0;
    if (!numeric_rows(*M, nlev, x0, zp, s)) numeric_levels(*M, nlev, x0, zp, s);
    if (zp) fail(HEC_ERR_ZERO_PIVOT, "zero pivot in row " + std::to_string(zp - 1));
    // every pivot u_ii must be nonzero for the backward substitution, also
    // those of rows that no later row uses
    if (n) {
        DevBuf<int32_t> dflag(1);
        HEC_HIP(hipMemsetAsync(dflag.get(), 0, sizeof(int32_t), s));
        k_check_diag<<<ceil_div(n, 256), 256, 0, s>>>(n, M->diag.get(), M->LUx.get(), dflag.get());
        HEC_CHECK_LAUNCH();
        dflag.download(&zp, 1, s);
        HEC_HIP(hipStreamSynchronize(s));
        if (zp) fail(HEC_ERR_ZERO_PIVOT, "zero pivot in row " + std::to_string(zp - 1));
    }
    if (M->has_f32) {
        M->LUx32.alloc(M->nnz);
        if (M->nnz)
            k_convert<double, float><<<ceil_div(M->nnz, 256), 256, 0, s>>>(M->nnz, M->LUx.get(),
                                                                           M->LUx32.get());
        HEC_CHECK_LAUNCH();
        HEC_HIP(hipStreamSynchronize(s));
    }
    M->n_sys = n;
    return M;
}

// Sec. 2.5, restricted additive Schwarz on one device: the rows are cut into
// nblocks contiguous blocks (the sequence partition), each block is extended by
// `overlap` layers of graph neighbours (rows reached through A's stored
// entries), and the extended blocks are stacked into one block-diagonal matrix
// that keeps only the entries of A inside each extended block. ext_row: system
// row of each stacked row; bstart: first stacked row of each block; own: the
// stacked row (inside its own block) of each system row.
static void ras_stack(int32_t n, const int32_t *Ap, const int32_t *Aj, const double *Ax, int32_t nblocks,
                      int32_t overlap, std::vector<int32_t> &Sp, std::vector<int32_t> &Sj, std::vector<double> &Sx,
                      std::vector<int32_t> &ext_row, std::vector<int32_t> &bstart, std::vector<int32_t> &own) {
    const int32_t R = (int32_t)(((int64_t)n + nblocks - 1) / nblocks);
    const int32_t nb = n ? (n + R - 1) / R : 0;
    std::vector<int32_t> stamp(n, -1), loc(n, 0);
    own.assign(n, -1);
    ext_row.clear();
    bstart.assign(1, 0);
    Sp.assign(1, 0);
    Sj.clear();
    Sx.clear();
    std::vector<int32_t> cur, layer, next;
    for (int32_t b = 0; b < nb; ++b) {
        const int32_t s0 = b * R, e0 = std::min(n, s0 + R);
        cur.clear();
        for (int32_t i = s0; i < e0; ++i) {
            stamp[i] = b;
            cur.push_back(i);
        }
        layer = cur;
        for (int32_t l = 0; l < overlap; ++l) {
            next.clear();
            for (int32_t i : layer)
                for (int32_t e = Ap[i]; e < Ap[i + 1]; ++e)
                    if (stamp[Aj[e]] != b) {
                        stamp[Aj[e]] = b;
                        next.push_back(Aj[e]);
                    }
            cur.insert(cur.end(), next.begin(), next.end());
            layer.swap(next);
        }
        std::sort(cur.begin(), cur.end());
        const int32_t base = (int32_t)ext_row.size();
        for (size_t t = 0; t < cur.size(); ++t) loc[cur[t]] = (int32_t)t;
        for (size_t t = 0; t < cur.size(); ++t) {
            const int32_t i = cur[t];
            ext_row.push_back(i);
            if (i >= s0 && i < e0) own[i] = base + (int32_t)t;
            for (int32_t e = Ap[i]; e < Ap[i + 1]; ++e)
                if (stamp[Aj[e]] == b) {
                    Sj.push_back(base + loc[Aj[e]]);
                    Sx.push_back(Ax[e]);
                }
            Sp.push_back((int32_t)Sj.size());
        }
        bstart.push_back((int32_t)ext_row.size());
    }
}

namespace hec {

void check_levels(const hec_levels_s &lv, hipStream_t s) {
    if (!lv.sync.get()) return;
    uint32_t *errw = const_cast<uint32_t *>(lv.sync.get()) + kLevelsErrWord;
    uint32_t e = 0;
    HEC_HIP(hipMemcpyAsync(&e, errw, sizeof(e), hipMemcpyDeviceToHost, s));
    HEC_HIP(hipStreamSynchronize(s));
    if (e) {
        const uint32_t zero = 0;
        HEC_HIP(hipMemcpyAsync(errw, &zero, sizeof(zero), hipMemcpyHostToDevice, s));
        HEC_HIP(hipStreamSynchronize(s));
        fail(HEC_ERR_TIMEOUT, "a wait of the triangular solve gave up (its dependency never became ready); "
                              "the results of the solves since the last check are not valid");
    }
}

}  // namespace hec

extern "C" {

hec_status ilu_factor(int32_t n, const int32_t *Ap, const int32_t *Aj, const double *Ax, int32_t k, uint32_t flags,
                      void *stream, hec_ilu *out) {
    return guarded([&] {
        if (!out) fail(HEC_ERR_INVALID_ARG, "out is NULL");
        *out = nullptr;
        validate_csr(n, Ap, Aj, Ax);
        if (k < 0) fail(HEC_ERR_INVALID_ARG, "k < 0");
        if (flags & ~HEC_KEEP_F32) fail(HEC_ERR_INVALID_ARG, "unknown flags");
        for (int32_t i = 0; i < n; ++i) {
            bool d = false;
            for (int32_t e = Ap[i]; e < Ap[i + 1] && !d; ++e) d = Aj[e] == i;
            if (!d) fail(HEC_ERR_INVALID_ARG, "row " + std::to_string(i) + " has no stored diagonal");
        }
        hipStream_t s = as_stream(stream);
        StreamScope scope(s);
        auto M = factor_csr(n, Ap, Aj, Ax, k, flags, s);
        *out = M.release();
    });
}

hec_status ilu_factor_ras(int32_t n, const int32_t *Ap, const int32_t *Aj, const double *Ax, int32_t k,
                          int32_t nblocks, int32_t overlap, uint32_t flags, void *stream, hec_ilu *out) {
    return guarded([&] {
        if (!out) fail(HEC_ERR_INVALID_ARG, "out is NULL");
        *out = nullptr;
        validate_csr(n, Ap, Aj, Ax);
        if (k < 0) fail(HEC_ERR_INVALID_ARG, "k < 0");
        if (nblocks < 1) fail(HEC_ERR_INVALID_ARG, "nblocks < 1");
        if (overlap < 0) fail(HEC_ERR_INVALID_ARG, "overlap < 0");
        if (flags & ~HEC_KEEP_F32) fail(HEC_ERR_INVALID_ARG, "unknown flags");
        for (int32_t i = 0; i < n; ++i) {
            bool d = false;
            for (int32_t e = Ap[i]; e < Ap[i + 1] && !d; ++e) d = Aj[e] == i;
            if (!d) fail(HEC_ERR_INVALID_ARG, "row " + std::to_string(i) + " has no stored diagonal");
        }
        std::vector<int32_t> Sp, Sj, ext_row, bstart, own;
        std::vector<double> Sx;
        ras_stack(n, Ap, Aj, Ax, nblocks, overlap, Sp, Sj, Sx, ext_row, bstart, own);
        const int64_t nf = (int64_t)ext_row.size();
        if (nf > INT32_MAX / 2 || (int64_t)Sj.size() > INT32_MAX)
            fail(HEC_ERR_INVALID_ARG, "extended blocks too large for 32-bit indices");
        hipStream_t s = as_stream(stream);
        StreamScope scope(s);
        auto M = factor_csr((int32_t)nf, Sp.data(), Sj.data(), Sx.data(), k, flags, s);
        M->n_sys = n;
        M->nblocks = (int32_t)bstart.size() - 1;
        M->overlap = overlap;
        M->gnx = M->gny = M->gnz = 0;
        M->hblocks.swap(bstart);
        M->hext_row.swap(ext_row);
        M->hown.swap(own);
        *out = M.release();
    });
}

hec_status ilu_info(hec_ilu M, int32_t *n, int64_t *nnz) {
    return guarded([&] {
        if (!M) fail(HEC_ERR_INVALID_ARG, "null factor");
        if (n) *n = M->n;
        if (nnz) *nnz = M->nnz;
    });
}

hec_status ilu_export(hec_ilu M, int32_t *LUp, int32_t *LUj, double *LUx) {
    return guarded([&] {
        if (!M) fail(HEC_ERR_INVALID_ARG, "null factor");
        if (LUp) std::copy(M->hLUp.begin(), M->hLUp.end(), LUp);
        if (LUj) std::copy(M->hLUj.begin(), M->hLUj.end(), LUj);
        if (LUx) {
            M->LUx.download(LUx, M->nnz, M->LUx.st);
            HEC_HIP(hipStreamSynchronize(M->LUx.st));
        }
    });
}

hec_status ilu_ras_export(hec_ilu M, int32_t *n_sys, int32_t *nblocks, int32_t *block_start, int32_t *ext_row,
                          int32_t *own) {
    return guarded([&] {
        if (!M) fail(HEC_ERR_INVALID_ARG, "null factor");
        const bool ras = !M->hext_row.empty();
        if (n_sys) *n_sys = M->n_sys;
        if (nblocks) *nblocks = ras ? M->nblocks : 1;
        if (block_start) {
            if (ras) {
                std::copy(M->hblocks.begin(), M->hblocks.end(), block_start);
            } else {
                block_start[0] = 0;
                block_start[1] = M->n;
            }
        }
        if (ext_row) {
            if (ras) std::copy(M->hext_row.begin(), M->hext_row.end(), ext_row);
            else for (int32_t i = 0; i < M->n; ++i) ext_row[i] = i;
        }
        if (own) {
            if (ras) std::copy(M->hown.begin(), M->hown.end(), own);
            else for (int32_t i = 0; i < M->n; ++i) own[i] = i;
        }
    });
}

hec_status ilu_destroy(hec_ilu M) {
    delete M;
    return HEC_OK;
}

hec_status level_schedule(hec_ilu M, void *stream, hec_levels *out) {
    return guarded([&] {
        if (!out) fail(HEC_ERR_INVALID_ARG, "out is NULL");
        *out = nullptr;
        if (!M) fail(HEC_ERR_INVALID_ARG, "null factor");
        hipStream_t s = as_stream(stream);
        StreamScope scope(s);
        auto lv = std::make_unique<hec_levels_s>();
        OwnerScope own(&lv->dev_bytes);
        lv->n = M->n_sys;
        lv->nf = M->n;
        lv->ras = !M->hext_row.empty();
        if (!lv->ras && trsv_grid_enabled()) {  // the wavefront plans: both triangles or neither
            build_grid(*M, lv->lower.grid, lv->upper.grid, s);
        }
        if (lv->lower.grid.on) {  // the level schedules only (levels_export, the batched copies)
            level_only(*M, true, lv->upper);
            level_only(*M, false, lv->lower);
        } else {
            build_tri(*M, true, lv->upper, nullptr, s);
            build_tri(*M, false, lv->lower, &lv->upper, s);
        }
        if (!lv->ras && M->n <= HEC_BATCH_MAX_N) {  // small enough for the batched solver
            if (batch_takes_grid(lv->upper.grid)) {
                build_grid_pivots(*M, lv->upper.grid, s);
            } else {
                build_flat(*M, false, lv->lower, s);
                build_flat(*M, true, lv->upper, s);
            }
        }
        lv->sync.alloc(kLevelsSyncWords);
        HEC_HIP(hipMemsetAsync(lv->sync.get(), 0, kLevelsSyncWords * sizeof(uint32_t), s));
        const int64_t ny = lv->lower.grid.on ? std::max<int64_t>(M->n, lv->lower.grid.pad_elems()) : M->n;
        lv->yp64.alloc(ny);
        if (M->has_f32) lv->yp32.alloc(ny);
        if (!lv->lower.grid.on) {
            lv->qL64.alloc(M->n);
            lv->qU64.alloc(M->n);
            if (M->has_f32) {
                lv->qL32.alloc(M->n);
                lv->qU32.alloc(M->n);
            }
        } else {
            const int64_t nface = lv->lower.grid.face_elems();
            lv->fL64.alloc(nface);
            lv->fU64.alloc(nface);
            if (M->has_f32) {
                lv->fL32.alloc(nface);
                lv->fU32.alloc(nface);
            }
        }
        trsv_init_levels(*lv, s);
        HEC_HIP(hipStreamSynchronize(s));
        *out = lv.release();
    });
}

hec_status levels_info(hec_levels lv, int32_t *n, int32_t *nlev_lower, int32_t *nlev_upper) {
    return guarded([&] {
        if (!lv) fail(HEC_ERR_INVALID_ARG, "null levels");
        if (n) *n = lv->n;
        if (nlev_lower) *nlev_lower = lv->lower.nlev;
        if (nlev_upper) *nlev_upper = lv->upper.nlev;
    });
}

hec_status levels_grid(hec_levels lv, int32_t *grid) {
    return guarded([&] {
        if (!lv || !grid) fail(HEC_ERR_INVALID_ARG, "null levels or output");
        *grid = lv->lower.grid.on && lv->upper.grid.on ? 1 : 0;
    });
}

hec_status levels_export(hec_levels lv, int32_t *lower_ptr, int32_t *lower_perm, int32_t *upper_ptr,
                         int32_t *upper_perm) {
    return guarded([&] {
        if (!lv) fail(HEC_ERR_INVALID_ARG, "null levels");
        if (lower_ptr) std::copy(lv->lower.hlevel_ptr.begin(), lv->lower.hlevel_ptr.end(), lower_ptr);
        if (lower_perm) std::copy(lv->lower.hperm.begin(), lv->lower.hperm.end(), lower_perm);
        if (upper_ptr) std::copy(lv->upper.hlevel_ptr.begin(), lv->upper.hlevel_ptr.end(), upper_ptr);
        if (upper_perm) std::copy(lv->upper.hperm.begin(), lv->upper.hperm.end(), upper_perm);
    });
}

hec_status levels_destroy(hec_levels lv) {
    delete lv;
    return HEC_OK;
}

hec_status levels_check(hec_levels lv, void *stream) {
    return guarded([&] {
        if (!lv) fail(HEC_ERR_INVALID_ARG, "null levels");
        check_levels(*lv, as_stream(stream));
    });
}

hec_status trsv_levels(hec_ilu M, hec_levels lv, uint32_t which, hec_dtype prec, const void *b, void *x,
                       void *stream) {
    return guarded([&] {
        if (!M || !lv) fail(HEC_ERR_INVALID_ARG, "null factor or levels");
        if (M->n_sys != lv->n || M->n != lv->nf) fail(HEC_ERR_INVALID_ARG, "factor and levels differ in size");
        if (which != HEC_LOWER && which != HEC_UPPER && which != HEC_LU) fail(HEC_ERR_INVALID_ARG, "bad `which`");
        if (lv->ras && which != HEC_LU)
            fail(HEC_ERR_INVALID_ARG, "a RAS factor is applied as a whole (HEC_LU): its triangles are over the stacked blocks");
        if (lv->n > 0 && (!b || !x)) fail(HEC_ERR_INVALID_ARG, "b or x is NULL");
        if (b == x && lv->n > 0) fail(HEC_ERR_INVALID_ARG, "b and x must not overlap");
        hipStream_t s = as_stream(stream);
        StreamScope scope(s);
        if (prec == HEC_F64) {
            trsv_launch<double>(*lv, which, (const double *)b, (double *)x, s);
        } else if (prec == HEC_F32) {
            if (!M->has_f32 || (!lv->yp32.get() && lv->n > 0))
                fail(HEC_ERR_INVALID_ARG, "factor has no FP32 copy (HEC_KEEP_F32)");
            trsv_launch<float>(*lv, which, (const float *)b, (float *)x, s);
        } else {
            fail(HEC_ERR_INVALID_ARG, "bad dtype");
        }
    });
}

}  // extern "C"
