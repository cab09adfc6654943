// Device helpers shared by the streaming kernels and the fast evaluation:
// fixed-order workgroup reductions, partial records and the last-arrival
// election, the start of the CG's line search, and the end of a gradient
// pass.  NT is the workgroup size.
#pragma once

#include <algorithm>
#include <cmath>

#include "internal.h"

namespace uvm {
namespace {

// ---------------------------------------------------------------- reductions
// Sum K doubles over the workgroup; every thread receives the totals.
template <int K, int NT = NTHR>
__device__ __forceinline__ void block_sum(double (&v)[K]) {
    constexpr int NW = NT / 64;
    __shared__ double red[K][NW];
#pragma unroll
    for (int x = 0; x < K; ++x) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v[x] += __shfl_xor(v[x], o, 64);
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    __syncthreads();
    if (lane == 0) {
#pragma unroll
        for (int x = 0; x < K; ++x) red[x][wave] = v[x];
    }
    __syncthreads();
#pragma unroll
    for (int x = 0; x < K; ++x) {
        double t[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) t[w] = red[x][w];
#pragma unroll
        for (int o = 1; o < NW; o <<= 1)
#pragma unroll
            for (int w = 0; w + o < NW; w += 2 * o) t[w] += t[w + o];
        v[x] = t[0];
    }
}

__device__ __forceinline__ double block_min(double v) {
    __shared__ double red[NTHR / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    __syncthreads();
    if (lane == 0) red[wave] = v;
    __syncthreads();
    return fmin(fmin(red[0], red[1]), fmin(red[2], red[3]));
}

// Partial records are written and read at device coherence (relaxed
// agent-scope atomic stores and loads: they bypass the caches that are not
// coherent between the chiplets), so that the workgroup that finishes a
// reduction in the same launch reads every other workgroup's record.
__device__ __forceinline__ void coh_store(double *p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void coh_store(float *p, float v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double coh_load(const double *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sum slot `s` (K slots starting at s0) of n_items partial records of NPART
// doubles starting at `base`, in index order (strided per thread, then the
// fixed workgroup reduction).
template <int K, int NT = NTHR>
__device__ __forceinline__ void sum_partials(const double *base, int n_items, int s0, double (&out)[K]) {
#pragma unroll
    for (int x = 0; x < K; ++x) out[x] = 0.0;
    for (int it = threadIdx.x; it < n_items; it += NT) {
#pragma unroll
        for (int x = 0; x < K; ++x) out[x] += coh_load(base + (size_t)it * NPART + s0 + x);
    }
    block_sum<K, NT>(out);
}

// Two record sets in one pass, their loads issued together (one memory round
// trip instead of two): slots [s0, s0 + K) of na records at `a` and slots
// [s1, s1 + L) of nb records at `b`, each summed in index order exactly as
// sum_partials does.  Past a set's end a thread reads a stand-in record of
// the other set (never of an empty one) and adds -0.0, an exact identity.
template <int K, int L, int NT = NTHR>
__device__ __forceinline__ void sum_partials2(const double *a, int na, int s0, double (&oa)[K], const double *b,
                                              int nb, int s1, double (&ob)[L]) {
    double v[K + L];
#pragma unroll
    for (int x = 0; x < K + L; ++x) v[x] = 0.0;
    const int nmax = na > nb ? na : nb;
    // four rounds of loads in flight (the sums stay in record order)
    constexpr int U = 4;
    for (int i0 = threadIdx.x; i0 < nmax; i0 += U * NT) {
        double la[U][K], lb[U][L];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int it = i0 + u * NT;
            const bool oka = it < na, okb = it < nb;
            if (!oka && !okb) continue;
            const double *ra = oka ? a + (size_t)it * NPART + s0 : b + (size_t)it * NPART + s1;
            const double *rb = okb ? b + (size_t)it * NPART + s1 : ra;
#pragma unroll
            for (int x = 0; x < K; ++x) la[u][x] = coh_load(ra + (oka ? x : 0));
#pragma unroll
            for (int x = 0; x < L; ++x) lb[u][x] = coh_load(rb + (okb ? x : 0));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int it = i0 + u * NT;
#pragma unroll
            for (int x = 0; x < K; ++x) v[x] += it < na ? la[u][x] : -0.0;
#pragma unroll
            for (int x = 0; x < L; ++x) v[K + x] += it < nb ? lb[u][x] : -0.0;
        }
    }
    block_sum<K + L, NT>(v);
#pragma unroll
    for (int x = 0; x < K; ++x) oa[x] = v[x];
#pragma unroll
    for (int x = 0; x < L; ++x) ob[x] = v[K + x];
}

// Sums of slots [0, K) and minima of slots [K, K + MN) of n_items records,
// one pass over the records (the sums in the order of sum_partials).
template <int K, int MN>
__device__ __forceinline__ void sum_min_partials(const double *base, int n_items, double (&sums)[K],
                                                 double (&mins)[MN]) {
#pragma unroll
    for (int x = 0; x < K; ++x) sums[x] = 0.0;
#pragma unroll
    for (int x = 0; x < MN; ++x) mins[x] = INFINITY;
    for (int it = threadIdx.x; it < n_items; it += NTHR) {
        double l[K + MN];
#pragma unroll
        for (int x = 0; x < K + MN; ++x) l[x] = coh_load(base + (size_t)it * NPART + x);
#pragma unroll
        for (int x = 0; x < K; ++x) sums[x] += l[x];
#pragma unroll
        for (int x = 0; x < MN; ++x) mins[x] = fmin(mins[x], l[K + x]);
    }
    block_sum<K>(sums);
#pragma unroll
    for (int x = 0; x < MN; ++x) mins[x] = block_min(mins[x]);
}

// Arrival of workgroup `rank` of the n of image c at the end of a partial-sum
// pass, once thread 0 has stored this workgroup's partial record (coh_store):
// returns true (in every thread) in exactly one workgroup per image and
// launch, the last to arrive, which may then read every record of the image
// (coh_load) and finish the image's reduction in a fixed order.  Thread 0
// waits for its record's store to complete before it counts itself in, so the
// last arrival finds every record in place.  The counters only elect that
// workgroup (the sums never depend on arrival order) and are left at zero for
// the next launch; no workgroup waits for another.
//
// Atomics on one address are served one after the other, and the workgroups
// of a pass end together: more than ARRIVE_FLAT of them count themselves in on
// CTR_SUB counters, whose last arrivals then count on the image's main one.
// (About 10 ns an arrival: 1,024 workgroups on one counter, 1024^2 FP32,
// k_cg_init 19.8 -> 10.2 us and k_cg_dir 27.3 -> 21.0; with 34 of them a
// second counter costs as much as it saves, 5.5 -> 5.7.)
constexpr int ARRIVE_FLAT = 128;
__device__ __forceinline__ bool arrive_last(unsigned *ctr, int c, int rank, int n) {
    __shared__ unsigned s_last;
    __syncthreads();
    if (threadIdx.x == 0) {
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_s_waitcnt(0);   // this workgroup's record stored
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        unsigned *p = ctr + (size_t)c * CTR_STRIDE;
        auto count = [](unsigned *x, unsigned expected) {
            const unsigned t = __hip_atomic_fetch_add(x, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const bool last = t + 1 == expected;
            if (last) __hip_atomic_store(x, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return last;
        };
        bool last;
        if (n <= ARRIVE_FLAT) {
            last = count(p, (unsigned)n);
        } else {
            const int sub = rank % CTR_SUB;
            last = count(p + (1 + sub) * CTR_LINE, (unsigned)((n - sub + CTR_SUB - 1) / CTR_SUB)) &&
                   count(p, (unsigned)CTR_SUB);
        }
        s_last = last ? 1u : 0u;
    }
    __syncthreads();
    return s_last != 0;
}

// ---- line search: exact minimisation of the convex phi on [0, alpha_max]
//   phi'(al)  = b + a al + lambda sum d (ln((I + al d)/M) + 1)
//   phi''(al) = a + lambda sum d^2 / (I + al d)
// The entropy part of phi' increases with al, so phi'(al) >= phi'(0) + a al
// and the minimiser lies below -phi'(0)/a: that bounds a search without
// alpha_max.  The start knows phi', phi'' at 0 and, from the direction's
// visibility pass, at alpha_max, which settles a step that reaches alpha_max
// without any pass.  Each pass evaluates phi', phi'' at LS_K trial steps
// inside the bracket [LO, HI] and keeps the smallest bracket.  With HI
// evaluated the trials are the root of the cubic Hermite interpolant of phi'
// on the bracket, the Newton steps from both ends, the secant step and points
// 1e-3 and 1e-6 of the bracket either side of the cubic's root; with HI an
// unevaluated bound, a geometric ladder from the Newton step to HI; with no
// bound, factors of 4 from the Newton step.  A bracket narrowed to 1e-13 (or
// the last pass) accepts the cubic's root.  The state is advanced identically
// by every workgroup of the channel.
enum { PH_SEARCH = 0, PH_DONE = 3 };
static_assert(LS_K == 8, "the bracket proposal fills eight trial steps");

__device__ __forceinline__ void ls_finish(double *st, double al) {
    st[LSS_PHASE] = PH_DONE;
    st[LSS_ALPHA] = al;
#pragma unroll
    for (int m = 0; m < LS_K; ++m) st[LSS_T0 + m] = al;
}

// Root in [lo, hi] of the cubic Hermite interpolant p of phi' from its values
// f0 < 0 < f1 and slopes h0, h1 at the ends, by Newton's method on the unit
// parameter s of the bracket, safeguarded by bisection of the sub-bracket on
// which p changes sign.
__device__ double hermite_root(double lo, double hi, double f0, double f1, double h0, double h1) {
    const double w = hi - lo, d0 = h0 * w, d1 = h1 * w;
    double sl = 0.0, sh = 1.0;
    double s = f0 / (f0 - f1);
    if (!(s > 0.0 && s < 1.0)) s = 0.5;
    for (int it = 0; it < 64; ++it) {
        const double s2 = s * s, s3 = s2 * s;
        const double p = (2.0 * s3 - 3.0 * s2 + 1.0) * f0 + (s3 - 2.0 * s2 + s) * d0 + (3.0 * s2 - 2.0 * s3) * f1 +
                         (s3 - s2) * d1;
        if (p == 0.0) break;
        if (p < 0.0) sl = s;
        else sh = s;
        const double dp = 6.0 * (s2 - s) * (f0 - f1) + (3.0 * s2 - 4.0 * s + 1.0) * d0 + (3.0 * s2 - 2.0 * s) * d1;
        double sn = dp != 0.0 ? s - p / dp : 0.5 * (sl + sh);
        if (!(sn > sl && sn < sh)) sn = 0.5 * (sl + sh);
        if (sn == s) break;
        s = sn;
    }
    return fmin(fmax(lo + s * w, lo), hi);
}

__device__ __forceinline__ double ls_cubic(const double *st) {
    return hermite_root(st[LSS_LO], st[LSS_HI], st[LSS_FLO], st[LSS_FHI], st[LSS_HLO], st[LSS_HHI]);
}

__device__ void ls_propose(double *st) {
    const double lo = st[LSS_LO], hi = st[LSS_HI];
    const double tn = lo - st[LSS_FLO] / st[LSS_HLO];   // > lo (FLO < 0, HLO > 0)
    double t[LS_K];
    if (hi < 0.0) {
        double x = (tn > lo && isfinite(tn)) ? tn : (lo > 0.0 ? 2.0 * lo : 1.0);
        for (int m = 0; m < LS_K; ++m, x *= 4.0) t[m] = x;
    } else if (st[LSS_HI_EVAL] == 0.0) {
        const double t0 = (tn > lo && tn < hi) ? tn : lo + 0.5 * (hi - lo);
        const double r = log(hi / t0) / (LS_K - 1);
        for (int m = 0; m < LS_K - 1; ++m) t[m] = t0 * exp(r * m);
        t[LS_K - 1] = hi;
    } else {
        const double w = hi - lo;
        const double rc = ls_cubic(st);
        t[0] = rc;
        t[1] = tn;
        t[2] = hi - st[LSS_FHI] / st[LSS_HHI];
        t[3] = lo - st[LSS_FLO] * w / (st[LSS_FHI] - st[LSS_FLO]);
        t[4] = rc - 1e-3 * w;
        t[5] = rc + 1e-3 * w;
        t[6] = rc - 1e-6 * w;
        t[7] = rc + 1e-6 * w;
        for (int m = 0; m < LS_K; ++m)
            if (!(t[m] > lo && t[m] < hi)) t[m] = lo + (m + 1) * w / (LS_K + 1);
    }
    for (int i = 1; i < LS_K; ++i)   // ascending (insertion sort)
        for (int j = i; j > 0 && t[j] < t[j - 1]; --j) {
            const double x = t[j]; t[j] = t[j - 1]; t[j - 1] = x;
        }
#pragma unroll
    for (int m = 0; m < LS_K; ++m) st[LSS_T0 + m] = t[m];
}

// Start from a, b, e1 = lambda sum d (ln(I/M) + 1), e2 = lambda sum d^2/I
// (so phi'(0) = b + e1, phi''(0) = a + e2), alpha_max and, when am_eval, the
// entropy parts f_am, h_am of phi', phi'' at alpha_max.
__device__ void ls_init(double *st, double a, double b, double e1, double e2, double amax, bool stop,
                        bool am_eval, double f_am, double h_am) {
    st[LSS_A] = a;
    st[LSS_B] = b;
    st[LSS_AMAX] = isfinite(amax) ? amax : -1.0;
    st[LSS_STOP] = stop ? 1.0 : 0.0;
    st[LSS_LO] = 0.0;
    st[LSS_HI] = isfinite(amax) ? amax : -1.0;
    st[LSS_FLO] = b + e1;
    st[LSS_HLO] = a + e2;
    st[LSS_FHI] = 0.0;
    st[LSS_HHI] = 0.0;
    st[LSS_HI_EVAL] = 0.0;
    st[LSS_PHASE] = PH_SEARCH;
    if (stop || !(st[LSS_FLO] < 0.0) || !(st[LSS_HLO] > 0.0) || (isfinite(amax) && amax <= 0.0)) {
        ls_finish(st, 0.0);
        return;
    }
    if (isfinite(amax) && am_eval) {
        const double fa = b + a * amax + f_am;
        if (fa <= 0.0) {   // phi' <= 0 on all of [0, alpha_max]
            ls_finish(st, amax);
            return;
        }
        st[LSS_FHI] = fa;
        st[LSS_HHI] = a + h_am;
        st[LSS_HI_EVAL] = 1.0;
    } else if (!isfinite(amax) && a > 0.0) {
        st[LSS_HI] = -st[LSS_FLO] / a;
    }
    ls_propose(st);
}

// The end of a gradient pass, by the last of the image's n_rec workgroups to
// arrive (their records are in ppart):
//   mode 1: Phi, chi^2 (from the visibility pass's partials) and S (from the
//           image pass's partials) into the scalars and, if given, `user`;
//   mode 2: the Polak-Ribiere beta (clipped at 0), |gt|^2 and the iteration
//           count; all scalars copied to `user`.
// With the fast evaluation (TR) the gradient pass has the sum S itself (slot
// 0 of its records in mode 1, 2 in mode 2), and mode 2 is also the end of the
// step: Phi, chi^2 (the spread's partials), S, alpha and alpha_max.
struct GradTail {
    unsigned *ctr;
    const double *vispart;
    const int *ivis_base;
    const double *pp_S;
    const double *ls;                   // TR: line-search states
    double *scal;
    double *chan;
    double *user;
    // graph replays of a one-image CG step: the history buffer's address and
    // the replay counter (the scalars go to row *hist_ctr); null otherwise
    const long long *hist_ptr;
    long long *hist_ctr;
};

inline GradTail make_grad_tail(const uvmem_ctx *c, int mode, double *user) {
    const bool hist = mode == 2 && c->hist_in_grad, tr = c->tr_lg > 0;
    unsigned *ctr = c->d_ctr + (size_t)CTR_GRAD * c->nimg * CTR_STRIDE;
    const int *trbase = mode == 2 ? c->d_trsbase : c->d_trgbase;   // spread or gather records
    return GradTail{ctr, tr ? c->d_trpart : c->d_vispart, tr ? trbase : c->d_ivis_base, c->d_ppart, c->d_ls,
                    c->d_scal, c->d_chan, user,
                    hist ? c->d_hist_ptr : nullptr, hist ? c->d_iter_ctr : nullptr};
}

template <int NT, bool TR>
__device__ __forceinline__ void grad_tail(int mode, int c, int rank, int n_rec, const double *ppart, double lam,
                                          const GradTail &tail) {
    if ((mode != 1 && mode != 2) || !arrive_last(tail.ctr, c, rank, n_rec)) return;
    double *sc = tail.scal + (size_t)c * UVMEM_NSCAL;
    if (mode == 1) {
        double x2[1], S[1];
        const int v0 = tail.ivis_base[c], v1 = tail.ivis_base[c + 1];
        sum_partials2<1, 1, NT>(tail.vispart + (size_t)v0 * NPART, v1 - v0, 0, x2,
                                (TR ? ppart : tail.pp_S) + (size_t)c * n_rec * NPART, n_rec, 0, S);
        if (threadIdx.x == 0) {
            const double chi2 = 0.5 * x2[0];
            sc[UVMEM_S_PHI] = chi2 + lam * S[0];
            sc[UVMEM_S_CHI2] = chi2;
            sc[UVMEM_S_S] = S[0];
            if (tail.user) {
                double *u = tail.user + (size_t)c * UVMEM_NSCAL;
                u[UVMEM_S_PHI] = sc[UVMEM_S_PHI];
                u[UVMEM_S_CHI2] = chi2;
                u[UVMEM_S_S] = S[0];
            }
        }
        return;
    }
    double gg[TR ? 3 : 2], x2[1];
    if constexpr (TR) {
        const int v0 = tail.ivis_base[c], v1 = tail.ivis_base[c + 1];
        sum_partials2<1, 3, NT>(tail.vispart + (size_t)v0 * NPART, v1 - v0, 0, x2,
                                ppart + (size_t)c * n_rec * NPART, n_rec, 0, gg);
    } else {
        sum_partials<2, NT>(ppart + (size_t)c * n_rec * NPART, n_rec, 0, gg);
    }
    if (threadIdx.x == 0) {
        double *ch = tail.chan + (size_t)c * CH_N;
        if constexpr (TR) {
            const double *lsc = tail.ls + (size_t)c * LSS_N;
            const double chi2 = 0.5 * x2[0], al = lsc[LSS_ALPHA];
            sc[UVMEM_S_PHI] = chi2 + lam * gg[2];
            sc[UVMEM_S_CHI2] = chi2;
            sc[UVMEM_S_S] = gg[2];
            sc[UVMEM_S_ALPHA] = al;
            sc[UVMEM_S_ALPHA_MAX] = lsc[LSS_AMAX] < 0.0 ? INFINITY : lsc[LSS_AMAX];
            if (al == 0.0) ch[CH_STOP] = 1.0;
        }
        const double gold = ch[CH_GG_OLD];
        const bool stop = ch[CH_STOP] != 0.0;
        double beta = 0.0;
        if (!stop && gold > 0.0) beta = fmax(0.0, (gg[0] - gg[1]) / gold);
        sc[UVMEM_S_BETA] = beta;
        sc[UVMEM_S_GNORM2] = gg[0];
        if (sc[UVMEM_S_ALPHA] != 0.0) sc[UVMEM_S_ITER] += 1.0;
        if (tail.user) {
            for (int x = 0; x < UVMEM_NSCAL; ++x) tail.user[(size_t)c * UVMEM_NSCAL + x] = sc[x];
        }
        if (tail.hist_ptr) {
            double *hb = reinterpret_cast<double *>(tail.hist_ptr[0]);
            const long long t = tail.hist_ctr[0];
            if (hb) {
                for (int x = 0; x < UVMEM_NSCAL; ++x) hb[t * UVMEM_NSCAL + x] = sc[x];
            }
            tail.hist_ctr[0] = t + 1;
        }
    }
}

}  // namespace
}  // namespace uvm
