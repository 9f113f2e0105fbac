// Batched restarted GMRES for many small systems (the serving path): one
// persistent launch solves every system of a batch, one workgroup per system,
// and the launch (descriptor upload, kernel, result download) is recorded once
// into a hipGraph per batch context and replayed for each batch.
//
// Per system the method is that of gmres_solve (Sec. 2.7; right preconditioning
// with M = LU of Eq. (7)-(8); Alg. 3 level order for the triangular solves),
// carried out by the workgroup alone:
//  * SpMV over the HEC arrays (Alg. 1: the ELL slab, then the CSR remainder),
//    one row per thread, FP64 accumulation;
//  * the preconditioner solve: a factor with wavefront plans (ILU(0) of a grid
//    stencil) level by level of the grid, in place on a vector in LDS (b_grid); any
//    other in level order (Eq. (11), Alg. 3) over a level-ordered copy of each
//    triangle: 64-row chunks of one level are taken by the wavefronts in turn,
//    and a row reads each dependency from LDS as
//    soon as it is final (the LDS vectors start filled with a signalling-NaN
//    pattern that arithmetic never produces), so no barrier separates levels;
//  * classical Gram-Schmidt applied twice in three passes over the basis,
//    deterministic block reductions, Givens rotations and the small least-squares solve in FP64 in LDS;
//  * cycles restart from the FP64 true residual. precision 1: each cycle uses the
//    FP32 copies of the matrix and factor values (FP64 vectors and arithmetic),
//    asked for a reduction of inner_rtol, and the FP64 true residual refines.
// Nothing a workgroup computes depends on the other systems of the batch, so a
// system's result is bit-identical alone and in any batch.
#include <algorithm>
#include <chrono>
#include <climits>
#include <cmath>
#include <mutex>

#include "hec_internal.hpp"

namespace hec {
namespace {

constexpr int kBT = 512;          // threads per system (256 registers each: deep loads instead of more wavefronts)
constexpr int kBW = kBatchWaves;  // wavefronts per system
static_assert(kBW == kBT / 64, "wavefronts of a workgroup");
constexpr int kBMaxM = 32;        // largest restart length
constexpr int kBRedStride = 33;   // per-wavefront partial sums in LDS

// Pointers that the kernel reads from memory, said to be global: taken as generic they
// become flat accesses, which wait for everything in flight, LDS included.
#ifdef __HIP_DEVICE_COMPILE__
#define HEC_GLOBAL __attribute__((address_space(1)))
#else
#define HEC_GLOBAL
#endif
template <class T>
HEC_GLOBAL T *as_global(T *p) {
    return (HEC_GLOBAL T *)p;
}
#ifdef __HIP_DEVICE_COMPILE__
#define HEC_CONST __attribute__((address_space(4)))
#define HEC_LDS __attribute__((address_space(3)))
#else
#define HEC_CONST
#define HEC_LDS
#endif
using LDouble = HEC_LDS double;
using LInt = HEC_LDS int;
using GDouble = HEC_GLOBAL double;
using GFloat = HEC_GLOBAL float;
using GInt = HEC_GLOBAL int32_t;
template <class VT> struct GlobalOf;
template <> struct GlobalOf<double> { using type = GDouble; };
template <> struct GlobalOf<float> { using type = GFloat; };
template <class VT> using Global = typename GlobalOf<VT>::type;

struct BatchSys {
    int32_t n, K, ld, has_rem;
    const GInt *ell_col;
    const GDouble *ell_val;
    const GFloat *ell_val32;
    const GInt *rem_ptr, *rem_col;
    const GDouble *rem_val;
    const GFloat *rem_val32;
    // level-ordered triangles (lower, upper): chunk starts, position -> row,
    // dependency rows and values at s*ldq + q, pivots (upper)
    int32_t KL, KU, ldq, nchL, nchU;
    const GInt *chL, *rowL, *colL, *chU, *rowU, *colU;
    const GDouble *valL, *valU, *pivU;
    const GFloat *valL32, *valU32, *pivU32;
    // wavefront plans (both triangles, 0 tiles: none): packed coefficients of PA x PB tiles
    int32_t ntiles, TA, NA, NB, NC, PA, PB, S;
    int64_t sa, sb, sc;
    const GDouble *coefL, *coefU;
    const GFloat *coefL32, *coefU32;
    const GDouble *gpiv;  // the upper plan's pivots, a value per step and lane
    const GFloat *gpiv32;
    const GDouble *b;
    GDouble *x;
    GDouble *ws;  // (2m + 3) * n doubles: V (m+1), Z (m), r, w
};

struct BatchHead {
    int32_t count, restart, maxit, x0_zero;
    uint32_t spin;  // polls a wait for a dependency makes before it gives up
    double rtol, target, inner_rtol;
};

struct BatchOut {
    int32_t status, iterations, restarts, ir_steps;
    double rel_res_true, rel_res_est;
};

// LDS layout of one system (dynamic): ly[max_n] | lz[max_n] | red[kBW][33] |
// H[(m+1)][m] | cs[m] | sn[m] | g[m+1] | y[m] | h2[m] | sc[8] (sc[6]: two flags of the grid
// solves, sc[7]: the give-up flag, ints)
struct Lds {
    double *ly, *lz, *red, *H, *cs, *sn, *g, *y, *h2, *sc;
};

__host__ __device__ inline size_t batch_lds_bytes(int max_n, int m) {
    return sizeof(double) * (2 * (size_t)max_n + kBW * kBRedStride + (size_t)(m + 1) * m + 5 * (size_t)m + 1 + 8);
}

constexpr unsigned long long kSent = 0x7FF4DEADBEEF1234ull;  // signalling NaN: never produced by arithmetic
constexpr unsigned long long kQNaN = 0x7FF8000000000000ull;

template <class VT> __device__ __forceinline__ const Global<VT> *ellv(const BatchSys &S);
template <> __device__ __forceinline__ const GDouble *ellv<double>(const BatchSys &S) { return S.ell_val; }
template <> __device__ __forceinline__ const GFloat *ellv<float>(const BatchSys &S) { return S.ell_val32; }
template <class VT> __device__ __forceinline__ const Global<VT> *remv(const BatchSys &S);
template <> __device__ __forceinline__ const GDouble *remv<double>(const BatchSys &S) { return S.rem_val; }
template <> __device__ __forceinline__ const GFloat *remv<float>(const BatchSys &S) { return S.rem_val32; }
template <class VT> __device__ __forceinline__ const Global<VT> *fval(const BatchSys &S, bool up);
template <> __device__ __forceinline__ const GDouble *fval<double>(const BatchSys &S, bool up) {
    return up ? S.valU : S.valL;
}
template <> __device__ __forceinline__ const GFloat *fval<float>(const BatchSys &S, bool up) {
    return up ? S.valU32 : S.valL32;
}
template <class VT> __device__ __forceinline__ const Global<VT> *fpiv(const BatchSys &S);
template <> __device__ __forceinline__ const GDouble *fpiv<double>(const BatchSys &S) { return S.pivU; }
template <> __device__ __forceinline__ const GFloat *fpiv<float>(const BatchSys &S) { return S.pivU32; }

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// Sums of the per-thread partials p[0..nv) over the workgroup, in a fixed order;
// out[k] (LDS) receives sum k. Ends with a barrier.
template <int NV>
__device__ __forceinline__ void block_sums(const double (&p)[NV], int nv, const Lds &L, double *out) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        if (k < nv) {
            const double s = wave_sum(p[k]);
            if (lane == 0) L.red[wave * kBRedStride + k] = s;
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < nv) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < kBW; ++w) t += L.red[w * kBRedStride + threadIdx.x];
        out[threadIdx.x] = t;
    }
    __syncthreads();
}

__device__ __forceinline__ double block_norm(const GDouble *v, int n, const Lds &L) {
    double p[1] = {0.0};
    for (int i = threadIdx.x; i < n; i += kBT) p[0] += v[i] * v[i];
    block_sums<1>(p, 1, L, L.sc);
    return sqrt(L.sc[0]);
}

// y = A x (z == nullptr) or y = z - A x; Alg. 1 order: ELL entries, then remainder. The
// loads of 8 entries of a row, then their gathers, are in flight together.
template <class VT, class X>
__device__ __forceinline__ void b_spmv(const BatchSys &S, const X *x, GDouble *y, const GDouble *z) {
    const Global<VT> *ev = ellv<VT>(S);
    const Global<VT> *rv = remv<VT>(S);
    for (int i = threadIdx.x; i < S.n; i += kBT) {
        double s = 0.0;
        for (int k0 = 0; k0 < S.K; k0 += 8) {
            int j[8];
            VT a[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const size_t e = (size_t)(k0 + u) * S.ld + i;
                j[u] = k0 + u < S.K ? S.ell_col[e] : i;
                a[u] = k0 + u < S.K ? ev[e] : (VT)0;
            }
            double xv[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) xv[u] = x[j[u]];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (k0 + u < S.K) s += (double)a[u] * xv[u];
        }
        if (S.has_rem)
            for (int e = S.rem_ptr[i]; e < S.rem_ptr[i + 1]; ++e) s += (double)rv[e] * x[S.rem_col[e]];
        y[i] = z ? z[i] - s : s;
    }
    __syncthreads();
}

__device__ __forceinline__ unsigned long long lds_load_bits(const double *p) {
    return __hip_atomic_load((const unsigned long long *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// One triangle in level order: wavefront w takes every kBW-th chunk from w (each at
// most 64 rows of one level); a row waits in LDS for each dependency to leave the
// sentinel. Every dependency lies in an earlier chunk, so the lowest unfinished
// chunk can always proceed. Lower: dst = L^{-1} src (src in global memory, unit
// diagonal). Upper: dst = U^{-1} src (src in LDS), also stored to out.
template <class VT, bool UPPER, class Src>
__device__ __forceinline__ void b_tri(const BatchSys &S, const Src *src, double *dst, GDouble *out, uint32_t spin,
                      int *timed_out) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nch = UPPER ? S.nchU : S.nchL, K = UPPER ? S.KU : S.KL, ldq = S.ldq;
    const GInt *ch = UPPER ? S.chU : S.chL, *rowp = UPPER ? S.rowU : S.rowL, *colp = UPPER ? S.colU : S.colL;
    const Global<VT> *valp = fval<VT>(S, UPPER);
    for (int c = wave; c < nch; c += kBW) {
        const int q = ch[c] + lane;
        if (q >= ch[c + 1]) continue;
        const int row = rowp[q];
        double acc = src[row];
        for (int s0 = 0; s0 < K; s0 += 8) {
            int j[8];
            double a[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int s = s0 + u;
                j[u] = s < K ? colp[(size_t)s * ldq + q] : INT_MIN;
                a[u] = j[u] >= 0 ? (double)valp[(size_t)s * ldq + q] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (j[u] < 0) continue;
                unsigned long long bits = lds_load_bits(dst + j[u]);
                uint32_t it = 0;
                while (bits == kSent) {
                    if (++it > spin) {  // give up: the row goes on with a NaN, the system reports it
                        *timed_out = 1;
                        bits = kQNaN;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                    bits = lds_load_bits(dst + j[u]);
                }
                acc -= a[u] * __longlong_as_double((long long)bits);
            }
        }
        if constexpr (UPPER) acc = acc / (double)fpiv<VT>(S)[q];
        unsigned long long r = (unsigned long long)__double_as_longlong(acc);
        if (r == kSent) r = kQNaN;  // keep a final value distinguishable from "not ready"
        if (out) out[row] = __longlong_as_double((long long)r);
        __hip_atomic_store((unsigned long long *)(dst + row), r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
}

// v of the lane before (lane 0: `first`).
__device__ __forceinline__ double lane_before(double first, double v) {
    int f[2], x[2];
    __builtin_memcpy(f, &first, 8);
    __builtin_memcpy(x, &v, 8);
    x[0] = __builtin_amdgcn_update_dpp(f[0], x[0], 0x138, 0xF, 0xF, false);  // DPP wave_shr:1
    x[1] = __builtin_amdgcn_update_dpp(f[1], x[1], 0x138, 0xF, 0xF, false);
    __builtin_memcpy(&v, x, 8);
    return v;
}

template <class T>
__device__ __forceinline__ T *uniform_ptr(T *p) {
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (T *)(((uint64_t)hi << 32) | lo);
}
template <class T>
__device__ __forceinline__ T *uniform_lds(T *p) {
    return (T *)(uintptr_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)p);
}

template <class VT> __device__ __forceinline__ const Global<VT> *gcoef(const HEC_CONST BatchSys &S, bool up);
template <> __device__ __forceinline__ const GDouble *gcoef<double>(const HEC_CONST BatchSys &S, bool up) {
    return up ? S.coefU : S.coefL;
}
template <> __device__ __forceinline__ const GFloat *gcoef<float>(const HEC_CONST BatchSys &S, bool up) {
    return up ? S.coefU32 : S.coefL32;
}
template <class VT> __device__ __forceinline__ const Global<VT> *gpiv(const HEC_CONST BatchSys &S);
template <> __device__ __forceinline__ const GDouble *gpiv<double>(const HEC_CONST BatchSys &S) { return S.gpiv; }
template <> __device__ __forceinline__ const GFloat *gpiv<float>(const HEC_CONST BatchSys &S) { return S.gpiv32; }

// One triangle of a factor with wavefront plans, in place on y (LDS, by row): level by
// level of the grid, a lane per column, wavefront w holding the columns of tiles (claims)
// w, w + kBW, .. (NT of them at most), with a barrier between levels unless one tile holds
// all columns. A row's three dependencies are its neighbours' results of the level before:
// the one along the column in a register, the others in LDS (on a 2D grid, FLAT, from the
// lane before by a shift; lane 0 reads the tile before it). Bound: the chain of levels, an
// LDS round trip and three fused multiply-adds each; the coefficients, which come from L2
// or beyond, are loaded 12 (8 in 3D) levels ahead, shared among NT tiles (4 ahead, a level
// took 0.4 us). In level order with polled dependencies a 63 x 63 system's two triangles
// took 142 us and a 16^3 system's 59; now 33 and 29. A row of U is divided by its pivot in FP64,
// as in level order (FP32 pivots too): a product with the packed reciprocal, in FP32 an FP32
// number, has up to 2^-24 more error a row; 48 systems of 1,000 to 4,200 rows took 5.3 ms
// with it and take 5.7 to 5.9. The quotient from a reciprocal of its own and one correction by the
// remainder, with the guards that makes it the same for every operand: 6.0 ms.
// Not inlined: with its registers allocated apart from the solver's, the levels ahead stay
// in registers (a spill reload in the loop waits for every load in flight).
template <class VT, bool UPPER, bool FLAT, bool MANY, int NT>
__device__ __attribute__((noinline)) void b_grid(const HEC_CONST BatchSys *sys, LDouble *y, LInt *timed_out, LInt *done,
                                                 uint32_t spin_v) {
    // (arguments of a call arrive in vector registers: made uniform again)
    const HEC_CONST BatchSys &S = *uniform_ptr(sys);
    y = uniform_lds(y);
    timed_out = uniform_lds(timed_out);
    done = uniform_lds(done);
    const uint32_t spin = __builtin_amdgcn_readfirstlane(spin_v);
    const Global<VT> *const coef = gcoef<VT>(S, UPPER);
    const Global<VT> *const piv = gpiv<VT>(S);
    constexpr int TA = FLAT ? plan::kGT2 : plan::kGT, TB = 64 / TA, U = (FLAT ? 12 : 8) / NT, LEFT = FLAT ? 1 : 2;
    constexpr int NC = FLAT ? (UPPER ? plan::kGrid2CoefUpper : plan::kGrid2CoefLower)
                            : (UPPER ? plan::kGridCoefUpper : plan::kGridCoefLower);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nlev = S.NA + S.NB + S.NC - 2;
    if (!MANY && wave > 0) {  // one wavefront has all columns: the others wait for its end
        uint32_t it = 0;
        while (*(volatile LInt *)done == 0) {
            if (++it > spin) {
                *timed_out = 1;
                break;
            }
            __builtin_amdgcn_s_sleep(16);
        }
        return;
    }
    const int ma = lane % TA, mb = lane / TA;
    const int sc = UPPER ? -(int)S.sc : (int)S.sc;
    const int da = UPPER ? (int)S.sa : -(int)S.sa, db = UPPER ? (int)S.sb : -(int)S.sb;
    struct Lev {
        VT cv[NC];  // back, (below,) left, (pivot)
        double b;
    };
    struct Tile {
        int first, ncl, row0;  // level of this lane's first row; its rows; where the first is
        int oa, ob;            // from a row to its left and below neighbour (0: none, whose coefficient is 0 ..
        bool has_a, has_b;     // .. and whose value is taken as 0)
        const Global<VT> *base, *pbase;  // the tile's coefficients and pivots (uniform)
        int t0;                // level t is the tile's step t + t0
        double xp;             // this lane's result of the level before
        Lev ring[U];
    } T[NT];
    // coefficients of level t, steps past the tile's ends clamped (no lane has a row there),
    // and the right-hand side (no other row is stored to it)
    auto load = [&](const Tile &T, int t, Lev &H) {
        const int st = min(max(t + T.t0, 0), S.S - 1);
        const Global<VT> *cp = T.base + (size_t)st * (64 * NC);
        if constexpr (FLAT) {  // the pair (back, left) of the lane
            H.cv[0] = cp[2 * lane];
            H.cv[1] = cp[2 * lane + 1];
        } else {
#pragma unroll
            for (int k = 0; k <= LEFT; ++k) H.cv[k] = cp[k * 64 + lane];
        }
        if constexpr (UPPER) H.cv[LEFT + 1] = T.pbase[(size_t)st * 64 + lane];
        const int idx = t - T.first;
        H.b = y[(unsigned)idx < (unsigned)T.ncl ? T.row0 + idx * sc : 0];
    };
    auto step = [&](Tile &T, int t, const Lev &H) {
        const int idx = t - T.first;
        const bool ok = (unsigned)idx < (unsigned)T.ncl;
        const int row = ok ? T.row0 + idx * sc : 0;
        double left, below = 0.0;
        if constexpr (FLAT) {
            double face = 0.0;
            if (MANY && lane == 0 && ok && T.has_a) face = y[row + T.oa];
            left = lane_before(face, T.xp);
        } else {
            left = y[row + (ok ? T.oa : 0)];
            below = y[row + (ok ? T.ob : 0)];
            left = T.has_a ? left : 0.0;
            below = T.has_b ? below : 0.0;
        }
        double acc;
        if constexpr (!UPPER) {
            acc = H.b - (double)H.cv[0] * T.xp;
            if constexpr (!FLAT) acc -= (double)H.cv[1] * below;
            acc -= (double)H.cv[LEFT] * left;
        } else {
            acc = H.b - (double)H.cv[LEFT] * left;
            if constexpr (!FLAT) acc -= (double)H.cv[1] * below;
            acc -= (double)H.cv[0] * T.xp;
            acc = acc / (double)H.cv[LEFT + 1];
        }
        if (ok) y[row] = acc;
        T.xp = ok ? acc : 0.0;
    };
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        const bool mine = wave + k * kBW < S.ntiles;  // (a wavefront without a tile only takes part in the barriers)
        const int c = mine ? wave + k * kBW : 0;
        const int mta = c % S.PA, mtb = c / S.PA;
        const int ta = UPPER ? S.PA - 1 - mta : mta, tb = UPPER ? S.PB - 1 - mtb : mtb;
        const int ga = ta * TA + (UPPER ? TA - 1 - ma : ma), gb = tb * TB + (UPPER ? TB - 1 - mb : mb);
        const bool act = mine && ga < S.NA && gb < S.NB;
        T[k].t0 = (UPPER ? S.PA * TA - S.NA + S.PB * TB - S.NB : 0) - mta * TA - mtb * TB;
        T[k].first = ma + mb - T[k].t0;
        T[k].ncl = act ? S.NC : 0;
        T[k].row0 = act ? (int)(ga * S.sa + gb * S.sb + (UPPER ? (S.NC - 1) * S.sc : 0)) : 0;
        T[k].has_a = act && (UPPER ? ga + 1 < S.NA : ga > 0);
        T[k].has_b = act && (UPPER ? gb + 1 < S.NB : gb > 0);
        T[k].oa = T[k].has_a ? da : 0;
        T[k].ob = T[k].has_b ? db : 0;
        T[k].base = coef + (size_t)c * S.S * (64 * NC);
        T[k].pbase = piv + (size_t)c * S.S * 64;
        T[k].xp = 0.0;
    }
    // the loads of the first levels in the order the loop issues them: where the two orders
    // differ, the compiler's wait for the oldest load is a wait for almost all of them
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int k = 0; k < NT; ++k) load(T[k], u, T[k].ring[u]);
        __asm__ volatile("" ::: "memory");
    }
    for (int t = 0; t < nlev; t += U) {  // (levels past the last have no rows)
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int k = 0; k < NT; ++k) {
                const Lev H = T[k].ring[u];
                load(T[k], t + U + u, T[k].ring[u]);
                step(T[k], t + u, H);
            }
            // the level's results are in LDS (a full barrier would also wait for the loads ahead)
            if (MANY) __asm__ volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        }
    }
    if (!MANY && lane == 0) *(volatile LInt *)done = 1;
}

// One triangle with a wavefront plan, by the shape of its tiles.
template <class VT, bool UPPER>
__device__ __forceinline__ void b_grid_tri(const BatchSys &S, const BatchSys *sys, double *y, uint32_t spin,
                                           int *timed_out, int *done) {
    const auto *sc = (const HEC_CONST BatchSys *)sys;
    auto *ly = (LDouble *)y;
    auto *lt = (LInt *)timed_out, *ld = (LInt *)done;
    if (S.TA == plan::kGT2) {
        if (S.ntiles == 1) b_grid<VT, UPPER, true, false, 1>(sc, ly, lt, ld, spin);
        else b_grid<VT, UPPER, true, true, 1>(sc, ly, lt, ld, spin);
    } else if (S.ntiles <= kBW) {
        b_grid<VT, UPPER, false, true, 1>(sc, ly, lt, ld, spin);
    } else {
        b_grid<VT, UPPER, false, true, 2>(sc, ly, lt, ld, spin);
    }
}

// out = U^{-1} L^{-1} v (Eq. (7)-(8)), also left in LDS, where it is whole on return; returns
// where. No barrier follows the stores to out on the grid path: every thread may read its own
// rows of it (i, i + kBT, ..), for others' it needs one.
template <class VT>
__device__ __forceinline__ const double *b_prec(const BatchSys &S, const BatchSys *sys, const GDouble *v, GDouble *out, const Lds &L,
                                                uint32_t spin, int *timed_out) {
    if (S.ntiles > 0) {
        int *const done = (int *)(L.sc + 6);  // the lower, the upper solve has ended
        if (threadIdx.x < 2) done[threadIdx.x] = 0;
        for (int i = threadIdx.x; i < S.n; i += kBT) L.ly[i] = v[i];
        __syncthreads();
        b_grid_tri<VT, false>(S, sys, L.ly, spin, timed_out, done);
        __syncthreads();
        b_grid_tri<VT, true>(S, sys, L.ly, spin, timed_out, done + 1);
        __syncthreads();
        for (int i = threadIdx.x; i < S.n; i += kBT) out[i] = L.ly[i];
        return L.ly;
    }
    const double sent = __longlong_as_double((long long)kSent);
    for (int i = threadIdx.x; i < S.n; i += kBT) {
        L.ly[i] = sent;
        L.lz[i] = sent;
    }
    __syncthreads();
    b_tri<VT, false>(S, v, L.ly, (GDouble *)nullptr, spin, timed_out);
    __syncthreads();
    b_tri<VT, true>(S, L.ly, L.lz, out, spin, timed_out);
    __syncthreads();
    return L.lz;
}

// One classical Gram-Schmidt pass over the basis V (nv <= NB vectors of n elements):
//   MODE 1: sums = V^T w;   MODE 2: w -= V h, sums = V^T w;   MODE 3: w -= V h, sums[0] = w.w
// Every thread takes rows i, i + kBT, .., all of a row's basis entries in flight at once
// and used for the update and the sums together, so that the two applications read the
// basis three times instead of four. A butterfly that halves the sums in each step reduces
// a wavefront's sums at once; the wavefronts' sums are added in a fixed order.
template <int MODE, int NB>
__device__ __forceinline__ void b_cgs_pass(const GDouble *V, int n, int nv, GDouble *w, const double *h, double *sums,
                                           const Lds &L) {
    constexpr int NS = MODE == 3 ? 1 : NB;
    constexpr int R = NB >= 32 ? 1 : 32 / NB;  // rows in flight together
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double acc[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) acc[k] = 0.0;
    for (int i0 = threadIdx.x; i0 < n; i0 += kBT * R) {
        double v[R][NB], wi[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            // (rows past the last read its entries and count as zero: no branches between the loads)
            const int i = min(i0 + r * kBT, n - 1);
            wi[r] = w[i];
#pragma unroll
            for (int k = 0; k < NB; ++k) v[r][k] = k < nv ? V[(size_t)k * n + i] : 0.0;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = i0 + r * kBT;
            if constexpr (MODE != 1) {
#pragma unroll
                for (int k = 0; k < NB; ++k)
                    if (k < nv) wi[r] -= v[r][k] * h[k];
                if (i < n) w[i] = wi[r];
            }
            wi[r] = i < n ? wi[r] : 0.0;
            if constexpr (MODE == 3) {
                acc[0] += wi[r] * wi[r];
            } else {
#pragma unroll
                for (int k = 0; k < NB; ++k) acc[k] += v[r][k] * wi[r];
            }
        }
    }
#pragma unroll
    for (int o = 32, cnt = NS; o > 0; o >>= 1) {  // a lane ends with the sum of its bits' index
        if (cnt > 1) {
            cnt >>= 1;
            const bool up = (lane & o) != 0;
#pragma unroll
            for (int k = 0; k < NS / 2; ++k)
                if (k < cnt) {
                    const double lo = acc[k], hi = acc[k + cnt];
                    const double rlo = __shfl_xor(lo, o), rhi = __shfl_xor(hi, o);
                    acc[k] = up ? hi + rhi : lo + rlo;
                }
        } else {
            acc[0] += __shfl_xor(acc[0], o);
        }
    }
    constexpr int PER = 64 / NS;  // lanes that hold the same sum
    if (lane % PER == 0) L.red[wave * kBRedStride + lane / PER] = acc[0];
    __syncthreads();
    if ((int)threadIdx.x < (MODE == 3 ? 1 : nv)) {
        double t = 0.0;
#pragma unroll
        for (int q = 0; q < kBW; ++q) t += L.red[q * kBRedStride + threadIdx.x];
        sums[threadIdx.x] = t;
    }
    __syncthreads();
}

// w orthogonalised twice against nv vectors, the coefficients' sum in h1; returns ||w||.
template <int NB>
__device__ __forceinline__ double b_cgs(const GDouble *V, int n, int nv, GDouble *w, double *h1, double *h2, const Lds &L) {
    b_cgs_pass<1, NB>(V, n, nv, w, nullptr, h1, L);
    b_cgs_pass<2, NB>(V, n, nv, w, h1, h2, L);
    b_cgs_pass<3, NB>(V, n, nv, w, h2, L.sc, L);
    if ((int)threadIdx.x < nv) h1[threadIdx.x] += h2[threadIdx.x];
    __syncthreads();
    return sqrt(L.sc[0]);
}

// One GMRES cycle from the residual r (norm beta > 0): at most mcyc Arnoldi
// steps, stopping once the rotated residual estimate is <= tol; x += Z y.
// Returns the steps taken; *est receives the last estimate.
template <class VT>
__device__ __forceinline__ int b_cycle(const BatchSys &S, const BatchSys *sys, int m, int mcyc, double tol, const GDouble *r, double beta, const Lds &L,
                       double *est, uint32_t spin, int *timed_out) {
    const int n = S.n;
    GDouble *V = S.ws, *Z = V + (size_t)(m + 1) * n, *w = Z + (size_t)m * n + n;
    for (int i = threadIdx.x; i < n; i += kBT) V[i] = r[i] / beta;
    if (threadIdx.x == 0) L.g[0] = beta;
    __syncthreads();
    int j = 0;
    double res = beta;
    while (j < mcyc) {
        GDouble *vj = V + (size_t)j * n, *zj = Z + (size_t)j * n;
        const double *const zl = b_prec<VT>(S, sys, vj, zj, L, spin, timed_out);
        b_spmv<VT>(S, zl, w, nullptr);
        // classical Gram-Schmidt, twice
        const int nv = j + 1;
        double *const h1 = L.y, *const h2 = L.h2;
        const double hn = nv <= 8    ? b_cgs<8>(V, n, nv, w, h1, h2, L)
                          : nv <= 16 ? b_cgs<16>(V, n, nv, w, h1, h2, L)
                                     : b_cgs<32>(V, n, nv, w, h1, h2, L);
        if (threadIdx.x <= j) L.H[threadIdx.x * m + j] = h1[threadIdx.x];
        __syncthreads();
        if (threadIdx.x == 0) {
            // previous rotations, then the one that zeroes H[j+1][j]
            for (int k = 0; k < j; ++k) {
                const double a = L.H[k * m + j], b = L.H[(k + 1) * m + j];
                L.H[k * m + j] = L.cs[k] * a + L.sn[k] * b;
                L.H[(k + 1) * m + j] = -L.sn[k] * a + L.cs[k] * b;
            }
            const double a = L.H[j * m + j];
            const double d = hypot(a, hn);
            const double c = d > 0.0 ? a / d : 1.0, s = d > 0.0 ? hn / d : 0.0;
            L.cs[j] = c;
            L.sn[j] = s;
            L.H[j * m + j] = d;
            L.g[j + 1] = -s * L.g[j];
            L.g[j] = c * L.g[j];
            L.sc[1] = fabs(L.g[j + 1]);
        }
        __syncthreads();
        res = L.sc[1];
        ++j;
        if (res <= tol || hn == 0.0 || j == mcyc) break;
        GDouble *vn = V + (size_t)j * n;
        for (int i = threadIdx.x; i < n; i += kBT) vn[i] = w[i] / hn;
        __syncthreads();
    }
    // y = H(0:j, 0:j)^{-1} g(0:j), then x += Z y
    if (threadIdx.x == 0) {
        for (int k = j - 1; k >= 0; --k) {
            double t = L.g[k];
            for (int c = k + 1; c < j; ++c) t -= L.H[k * m + c] * L.y[c];
            L.y[k] = L.H[k * m + k] != 0.0 ? t / L.H[k * m + k] : 0.0;
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += kBT) {
        double xi = S.x[i];
        for (int k = 0; k < j; ++k) xi += Z[(size_t)k * n + i] * L.y[k];
        S.x[i] = xi;
    }
    __syncthreads();
    *est = res;
    return j;
}

// VT: the value type of the cycles (FP32 copies with precision 1).
template <class VT>
__global__ __launch_bounds__(kBT) void k_gmres_batch(const BatchHead *__restrict__ head,
                                                     const BatchSys *__restrict__ sys, BatchOut *__restrict__ out,
                                                     int max_n) {
    const BatchHead H = *head;
    if ((int)blockIdx.x >= H.count) return;
    const BatchSys S = sys[blockIdx.x];
    extern __shared__ __align__(16) char bsmem[];
    const int m = H.restart;
    Lds L;
    L.ly = (double *)bsmem;
    L.lz = L.ly + max_n;
    L.red = L.lz + max_n;
    L.H = L.red + kBW * kBRedStride;
    L.cs = L.H + (size_t)(m + 1) * m;
    L.sn = L.cs + m;
    L.g = L.sn + m;
    L.y = L.g + m + 1;
    L.h2 = L.y + m;
    L.sc = L.h2 + m;
    const int n = S.n;
    GDouble *r = S.ws + (size_t)(2 * m + 1) * n;
    BatchOut o{HEC_OK, 0, 0, 0, 0.0, 0.0};
    // a wait for a dependency gave up in this system's solves (a word of the scalar area;
    // no static LDS: the kernel's dynamic LDS may take the whole workgroup limit)
    int *const timed_out = (int *)(L.sc + 7);
    if (threadIdx.x == 0) *timed_out = 0;
    const double bnorm = block_norm(S.b, n, L);  // (its barriers publish the flag's reset)
    if (bnorm == 0.0 || n == 0) {
        for (int i = threadIdx.x; i < n; i += kBT) S.x[i] = 0.0;
    } else {
        if (H.x0_zero)
            for (int i = threadIdx.x; i < n; i += kBT) S.x[i] = 0.0;
        __syncthreads();
        b_spmv<double>(S, S.x, r, S.b);
        double res = block_norm(r, n, L);
        int cycles = 0;
        while (res / bnorm > H.target && o.iterations < H.maxit) {
            const int mcyc = min(m, H.maxit - o.iterations);
            double est = 0.0;
            int jd;
            if constexpr (sizeof(VT) == 8) {
                jd = b_cycle<double>(S, sys + blockIdx.x, m, mcyc, H.target * bnorm, r, res, L, &est, H.spin, timed_out);
            } else {
                const double tol = fmax(H.inner_rtol * res, 0.5 * H.target * bnorm);
                jd = b_cycle<float>(S, sys + blockIdx.x, m, mcyc, tol, r, res, L, &est, H.spin, timed_out);
                o.ir_steps++;
            }
            o.rel_res_est = est / bnorm;
            o.iterations += jd;
            cycles++;
            b_spmv<double>(S, S.x, r, S.b);
            res = block_norm(r, n, L);
            if (jd == 0) break;
        }
        o.restarts = max(0, cycles - 1);
        o.rel_res_true = res / bnorm;
        if (!(res / bnorm <= H.target)) o.status = HEC_ERR_NOT_CONVERGED;
    }
    __syncthreads();
    if (*timed_out) o.status = HEC_ERR_TIMEOUT;
    if (threadIdx.x == 0) out[blockIdx.x] = o;
}

}  // namespace
}  // namespace hec

// Batch context: pinned descriptor staging, device descriptors and results,
// per-system workspaces, and the recorded graph.
struct hec_batch_s {
    int32_t capacity = 0, restart = 0, max_n = 0;
    bool use_graph = true;
    size_t lds = 0;
    hipStream_t bs = nullptr;   // the context's own stream (graphs are recorded and replayed on it)
    hipEvent_t ev = nullptr;
    hec::BatchHead *h_head = nullptr;
    hec::BatchSys *h_sys = nullptr;
    hec::BatchOut *h_out = nullptr;
    int64_t dev_bytes = 0;      // device bytes of the buffers below
    hec::DevBuf<hec::BatchHead> d_head;
    hec::DevBuf<hec::BatchSys> d_sys;
    hec::DevBuf<hec::BatchOut> d_out;
    hec::DevBuf<double> d_ws;
    hipGraph_t graph[2] = {};         // by precision: each has its kernel
    hipGraphExec_t exec[2] = {};
    ~hec_batch_s() {
        for (auto e : exec)
            if (e) (void)hipGraphExecDestroy(e);
        for (auto g : graph)
            if (g) (void)hipGraphDestroy(g);
        if (bs) (void)hipStreamSynchronize(bs);
        d_ws.release();  // in order on bs, before it is destroyed
        d_out.release();
        d_sys.release();
        d_head.release();
        if (h_out) (void)hipHostFree(h_out);
        if (h_sys) (void)hipHostFree(h_sys);
        if (h_head) (void)hipHostFree(h_head);
        if (ev) (void)hipEventDestroy(ev);
        if (bs) (void)hipStreamDestroy(bs);
    }
};

namespace hec {
namespace {

// Kernel launch plus the copies around it, on the context's stream.
void enqueue_batch(hec_batch_s &B, bool mixed) {
    HEC_HIP(hipMemcpyAsync(B.d_head.get(), B.h_head, sizeof(BatchHead), hipMemcpyHostToDevice, B.bs));
    HEC_HIP(hipMemcpyAsync(B.d_sys.get(), B.h_sys, sizeof(BatchSys) * B.capacity, hipMemcpyHostToDevice, B.bs));
    if (mixed)
        k_gmres_batch<float><<<B.capacity, kBT, B.lds, B.bs>>>(B.d_head.get(), B.d_sys.get(), B.d_out.get(), B.max_n);
    else
        k_gmres_batch<double><<<B.capacity, kBT, B.lds, B.bs>>>(B.d_head.get(), B.d_sys.get(), B.d_out.get(), B.max_n);
    HEC_CHECK_LAUNCH();
    HEC_HIP(hipMemcpyAsync(B.h_out, B.d_out.get(), sizeof(BatchOut) * B.capacity, hipMemcpyDeviceToHost, B.bs));
}

int max_dyn_lds() {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 64 * 1024;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess || v <= 0)
        return 64 * 1024;
    return std::min(v, 160 * 1024);
}

}  // namespace
}  // namespace hec

using namespace hec;

extern "C" {

hec_status batch_create(int32_t capacity, int32_t restart, int32_t max_n, int32_t use_graph, hec_batch *out) {
    return guarded([&] {
        if (!out) fail(HEC_ERR_INVALID_ARG, "out is NULL");
        *out = nullptr;
        if (capacity < 1 || capacity > 65535) fail(HEC_ERR_INVALID_ARG, "capacity must be in [1, 65535]");
        if (restart < 1 || restart > kBMaxM) fail(HEC_ERR_INVALID_ARG, "restart must be in [1, 32]");
        if (max_n < 1 || max_n > HEC_BATCH_MAX_N) fail(HEC_ERR_INVALID_ARG, "max_n must be in [1, HEC_BATCH_MAX_N]");
        std::unique_ptr<hec_batch_s> B(new hec_batch_s());
        B->capacity = capacity;
        B->restart = restart;
        B->max_n = max_n;
        B->use_graph = use_graph != 0;
        B->lds = batch_lds_bytes(max_n, restart);
        if ((int64_t)B->lds > max_dyn_lds()) fail(HEC_ERR_INVALID_ARG, "max_n too large for the workgroup's LDS");
        // once per process; a failure is reported (and taken off the runtime's last-error
        // slot, where it would otherwise surface in the caller's next HIP call)
        static const hipError_t attr = [] {
            const hipError_t e = hipFuncSetAttribute((const void *)k_gmres_batch<double>,
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, max_dyn_lds());
            return e != hipSuccess ? e
                                   : hipFuncSetAttribute((const void *)k_gmres_batch<float>,
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, max_dyn_lds());
        }();
        if (attr != hipSuccess) {
            (void)hipGetLastError();
            fail(HEC_ERR_HIP, std::string("hipFuncSetAttribute(k_gmres_batch): ") + hipGetErrorString(attr));
        }
        HEC_HIP(hipStreamCreateWithFlags(&B->bs, hipStreamNonBlocking));
        HEC_HIP(hipEventCreateWithFlags(&B->ev, hipEventDisableTiming));
        HEC_HIP(hipHostMalloc((void **)&B->h_head, sizeof(BatchHead), hipHostMallocDefault));
        HEC_HIP(hipHostMalloc((void **)&B->h_sys, sizeof(BatchSys) * capacity, hipHostMallocDefault));
        HEC_HIP(hipHostMalloc((void **)&B->h_out, sizeof(BatchOut) * capacity, hipHostMallocDefault));
        std::memset(B->h_sys, 0, sizeof(BatchSys) * capacity);
        {
            StreamScope scope(B->bs);
            OwnerScope own(&B->dev_bytes);
            B->d_head.alloc(1);
            B->d_sys.alloc(capacity);
            B->d_out.alloc(capacity);
            B->d_ws.alloc((size_t)(2 * restart + 3) * max_n * capacity);
            HEC_HIP(hipStreamSynchronize(B->bs));
        }
        *out = B.release();
    });
}

hec_status batch_destroy(hec_batch B) {
    return guarded([&] { delete B; });
}

hec_status gmres_solve_batched(hec_batch B, int32_t count, const hec_matrix *A, const hec_ilu *M,
                               const hec_levels *lv, const double *const *b, double *const *x,
                               const hec_solve_opts *o, hec_solve_info *info, void *stream) {
    auto t0 = std::chrono::steady_clock::now();
    hec_status st = guarded([&] {
        if (!B || !o) fail(HEC_ERR_INVALID_ARG, "null batch context or options");
        if (count < 0 || count > B->capacity) fail(HEC_ERR_INVALID_ARG, "count must be in [0, capacity]");
        if (count > 0 && (!A || !M || !lv || !b || !x)) fail(HEC_ERR_INVALID_ARG, "null array argument");
        if (o->restart != B->restart) fail(HEC_ERR_INVALID_ARG, "restart differs from the batch context's");
        if (o->maxit < 0) fail(HEC_ERR_INVALID_ARG, "maxit < 0");
        if (!(o->rtol > 0.0)) fail(HEC_ERR_INVALID_ARG, "rtol must be > 0");
        if (o->precision != 0 && o->precision != 1) fail(HEC_ERR_INVALID_ARG, "precision must be 0 or 1");
        const bool mixed = o->precision == 1;
        const size_t per = (size_t)(2 * B->restart + 3) * B->max_n;
        // the previous batch (if any) has completed: every call synchronises before it returns
        for (int32_t i = 0; i < count; ++i) {
            hec_matrix a = A[i];
            hec_ilu f = M[i];
            hec_levels l = lv[i];
            if (!a || !f || !l) fail(HEC_ERR_INVALID_ARG, "null handle in the batch");
            if (a->n != f->n || a->n != l->n || f->n != f->n_sys)
                fail(HEC_ERR_INVALID_ARG, "matrix, factor and levels differ in size (or a RAS factor)");
            if (a->n > B->max_n) fail(HEC_ERR_INVALID_ARG, "system larger than the batch context's max_n");
            if (a->n > 0 && (!b[i] || !x[i])) fail(HEC_ERR_INVALID_ARG, "b or x is NULL");
            if (mixed && (!a->has_f32 || !f->has_f32))
                fail(HEC_ERR_INVALID_ARG, "mixed precision needs HEC_KEEP_F32 on the matrix and the factor");
            const hec_grid &gl = l->lower.grid, &gu = l->upper.grid;
            const bool by_grid = gl.on && batch_takes_grid(gu) && gu.piv.get();
            if (a->n > 0 && !by_grid && (l->lower.flat.nchunks == 0 || l->upper.flat.nchunks == 0))
                fail(HEC_ERR_INVALID_ARG, "levels handle has no level-ordered copy (n above HEC_BATCH_MAX_N)");
            BatchSys &S = B->h_sys[i];
            S.n = a->n;
            S.K = a->K;
            S.ld = a->ld;
            S.has_rem = a->nnz_rem > 0;
            S.ell_col = as_global(a->ell_col.get());
            S.ell_val = as_global(a->ell_val.get());
            S.ell_val32 = as_global(a->ell_val32.get());
            S.rem_ptr = as_global(a->rem_ptr.get());
            S.rem_col = as_global(a->rem_col.get());
            S.rem_val = as_global(a->rem_val.get());
            S.rem_val32 = as_global(a->rem_val32.get());
            const hec_flat &fl = l->lower.flat, &fu = l->upper.flat;
            S.KL = fl.K;
            S.KU = fu.K;
            S.ldq = fl.ldq;
            S.nchL = fl.nchunks;
            S.nchU = fu.nchunks;
            S.ntiles = 0;
            if (by_grid) {
                S.ntiles = gl.PA * gl.PB;
                S.TA = gl.TA;
                S.NA = gl.NA;
                S.NB = gl.NB;
                S.NC = gl.NC;
                S.PA = gl.PA;
                S.PB = gl.PB;
                S.S = gl.S;
                S.sa = gl.sa;
                S.sb = gl.sb;
                S.sc = gl.sc;
                S.coefL = as_global(gl.coef.get());
                S.coefU = as_global(gu.coef.get());
                S.coefL32 = as_global(gl.coef32.get());
                S.coefU32 = as_global(gu.coef32.get());
                S.gpiv = as_global(gu.piv.get());
                S.gpiv32 = as_global(gu.piv32.get());
            }
            S.chL = as_global(fl.chunk_ptr.get());
            S.rowL = as_global(fl.row.get());
            S.colL = as_global(fl.col.get());
            S.valL = as_global(fl.val.get());
            S.valL32 = as_global(fl.val32.get());
            S.chU = as_global(fu.chunk_ptr.get());
            S.rowU = as_global(fu.row.get());
            S.colU = as_global(fu.col.get());
            S.valU = as_global(fu.val.get());
            S.valU32 = as_global(fu.val32.get());
            S.pivU = as_global(fu.piv.get());
            S.pivU32 = as_global(fu.piv32.get());
            S.b = as_global(b[i]);
            S.x = as_global(x[i]);
            S.ws = as_global(B->d_ws.get() + per * i);
        }
        BatchHead &Hh = *B->h_head;
        Hh.count = count;
        Hh.restart = B->restart;
        Hh.maxit = o->maxit;
        Hh.x0_zero = o->x0_zero;
        Hh.spin = spin_limit();
        Hh.rtol = o->rtol;
        Hh.target = mixed && o->ir_rtol > 0.0 ? std::min(o->ir_rtol, o->rtol) : o->rtol;
        Hh.inner_rtol = o->inner_rtol > 0.0 ? o->inner_rtol : 1e-4;
        if (count == 0) return;
        // order after the caller's stream (b, x and the handles' setup), run, wait
        hipStream_t us = as_stream(stream);
        HEC_HIP(hipEventRecord(B->ev, us));
        HEC_HIP(hipStreamWaitEvent(B->bs, B->ev, 0));
        if (B->use_graph) {
            if (!B->exec[mixed]) {
                HEC_HIP(hipStreamBeginCapture(B->bs, hipStreamCaptureModeThreadLocal));
                try {
                    enqueue_batch(*B, mixed);
                } catch (...) {
                    hipGraph_t g = nullptr;
                    (void)hipStreamEndCapture(B->bs, &g);
                    if (g) (void)hipGraphDestroy(g);
                    throw;
                }
                HEC_HIP(hipStreamEndCapture(B->bs, &B->graph[mixed]));
                HEC_HIP(hipGraphInstantiate(&B->exec[mixed], B->graph[mixed], nullptr, nullptr, 0));
            }
            HEC_HIP(hipGraphLaunch(B->exec[mixed], B->bs));
        } else {
            enqueue_batch(*B, mixed);
        }
        HEC_HIP(hipStreamSynchronize(B->bs));
    });
    const double secs = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    if (info && B && o) {
        for (int32_t i = 0; i < count && i <= B->capacity - 1; ++i) {
            hec_solve_info &f = info[i];
            f = hec_solve_info{};
            if (st == HEC_OK) {
                const BatchOut &r = B->h_out[i];
                f.status = r.status;
                f.iterations = r.iterations;
                f.restarts = r.restarts;
                f.ir_steps = r.ir_steps;
                f.rel_res_true = r.rel_res_true;
                f.rel_res_est = r.rel_res_est;
            } else {
                f.status = st;
            }
            f.seconds = secs;
        }
    }
    if (st == HEC_OK && B) {
        for (int32_t i = 0; i < count; ++i)
            if (B->h_out[i].status == HEC_ERR_TIMEOUT) {
                set_last_error("a wait of a system's triangular solve gave up (hec_set_spin_limit)");
                return HEC_ERR_TIMEOUT;
            }
        for (int32_t i = 0; i < count; ++i)
            if (B->h_out[i].status != HEC_OK) {
                set_last_error("a system of the batch did not converge");
                return HEC_ERR_NOT_CONVERGED;
            }
    }
    return st;
}

}  // extern "C"
