// Streaming kernels around the DFT contractions: attenuation prologue,
// visibility sums (residual, chi^2, line-search scalars), gradient
// finalisation with the entropy term, and the projected-CG step.
//
// Every reduction is FP64 and has a fixed order: a workgroup sums its
// elements in a fixed thread/stride pattern, then across waves in LDS; the
// per-channel totals sum the workgroup partials in index order.  Consumers
// that need a per-channel total recompute it from the partials themselves
// (every workgroup of the channel gets the same bits), which keeps each CG
// phase to one launch without atomics.
#include <cmath>
#include <type_traits>

#include "internal.h"
#include "reduce.h"

namespace uvm {
namespace {

// ---------------------------------------------------------------- fill
template <typename R>
__global__ void k_fill(R *__restrict__ x, R value, long long count) {
    long long i = (long long)blockIdx.x * NTHR + threadIdx.x;
    long long stride = (long long)gridDim.x * NTHR;
    for (; i < count; i += stride) x[i] = value;
}

// ---------------------------------------------------------------- prologue
// B = A o I written into the padded operand image; optional entropy partial
// S = sum I ln(I/M) and the domain flag (I <= 0 or NaN).
template <typename R>
__global__ __launch_bounds__(NTHR) void k_prologue(const R *__restrict__ I, const R *__restrict__ beam,
                                                   R *__restrict__ bop, const int *__restrict__ ichan_base,
                                                   double *__restrict__ ppart,
                                                   int *__restrict__ flag, int n, int np, int n_pb, int pb_len,
                                                   double M, int with_entropy) {
    const int c = blockIdx.x / n_pb, pb = blockIdx.x % n_pb;   // image plane, pixel block
    const long long npix = (long long)n * n;
    const R *Ic = I + (size_t)c * npix;
    const int ch0 = ichan_base[c], ch1 = ichan_base[c + 1];   // the channels that see this image
    double s[1] = {0.0};
    int bad = 0;
    for (int r = 0; r < pb_len / NTHR; ++r) {
        long long p = (long long)pb * pb_len + r * NTHR + threadIdx.x;
        if (p >= npix) break;
        const int i = (int)(p / n), j = (int)(p % n);
        const R x = Ic[p];
        for (int ch = ch0; ch < ch1; ++ch)
            bop[(size_t)ch * np * np + (size_t)i * np + j] = beam[(size_t)ch * npix + p] * x;
        if (with_entropy) {
            const double xd = (double)x;
            if (!(xd > 0.0)) bad = 1;
            else s[0] += xd * log(xd / M);
        }
    }
    if (with_entropy) {
        if (bad) atomicOr(flag, 1);
        block_sum<1>(s);
        if (threadIdx.x == 0) coh_store(ppart + ((size_t)c * n_pb + pb) * NPART + 0, s[0]);
    }
}

// ---------------------------------------------------------------- visibilities
// mode 0: out[k] = V_k (model visibilities)
// mode 1: R_k = V_k - Vo_k -> R; partial[0] = sum w |R|^2
// mode 2: Vd_k = V_k -> Vd; partial[0] = sum w |Vd|^2, partial[1] = sum w Re(conj(R) Vd)
// mode 3: R_k += alpha_c Vd_k; partial[0] = sum w |R|^2
// mode 4: R is a caller's coefficient vector, only read (w may be null)
// with_max (modes 1, 3, 4): partial[2] = max over the item of w max(|Re R|, |Im R|)
// One visibility item (index `item`); `alpha` is the step length of mode 3.
__device__ __forceinline__ void vis_item(const VisItem it, int item, const double2 *__restrict__ vpart,
                                         int n_parts, long long ztot, const double2 *__restrict__ vo,
                                         const float *__restrict__ w, double2 *__restrict__ R,
                                         double2 *__restrict__ Vd, double2 *__restrict__ out,
                                         double *__restrict__ vispart, int mode, int with_max, double alpha) {
    double acc[2] = {0.0, 0.0};
    double cmax = 0.0;   // max |Re|, |Im| of the adjoint's coefficients w R (mode 4: R alone)
    constexpr int U = 2;   // visibilities per thread and round, loads issued together
    for (long long k0 = it.kbeg; k0 < it.kend; k0 += U * NTHR) {
        // the loads that do not depend on the forward partials are issued
        // first, then every block's partials (four blocks in flight), which
        // are summed in block order; indices past the item's end are clamped
        // and null arrays replaced by the partials, so that no load sits
        // behind a branch (values loaded that way are never used)
        const double2 *anyv = vpart ? vpart : R;
        const float *wsrc = w ? w : reinterpret_cast<const float *>(anyv);
        const double2 *lsrc = mode == 1 ? vo : mode >= 2 ? R : anyv;
        const double2 *l2src = mode == 3 ? Vd : anyv;
        double ww[U];
        double2 ld[U], ld2[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const long long k = k0 + threadIdx.x + (long long)u * NTHR;
            const long long kc = k < it.kend ? k : it.kend - 1;
            const float wr = wsrc[kc];
            ww[u] = w ? (double)wr : 1.0;
            ld[u] = lsrc[kc];
            ld2[u] = l2src[kc];
        }
        double2 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = make_double2(0.0, 0.0);
        if (mode < 3) {
            constexpr int PB = 4;
            for (int ib0 = 0; ib0 < n_parts; ib0 += PB) {
                double2 pv[PB][U];
#pragma unroll
                for (int b = 0; b < PB; ++b)
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const long long k = k0 + threadIdx.x + (long long)u * NTHR;
                        const long long kc = k < it.kend ? k : it.kend - 1;
                        const int ibc = ib0 + b < n_parts ? ib0 + b : n_parts - 1;
                        pv[b][u] = vpart[(size_t)ibc * ztot + kc];
                    }
                // blocks past the last add -0.0, an exact identity (no branch
                // between the loads and the sums)
#pragma unroll
                for (int b = 0; b < PB; ++b) {
                    const bool okb = ib0 + b < n_parts;
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        v[u].x += okb ? pv[b][u].x : -0.0;
                        v[u].y += okb ? pv[b][u].y : -0.0;
                    }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const long long k = k0 + threadIdx.x + (long long)u * NTHR;
            if (k >= it.kend) continue;
            const double wv = ww[u];
            if (mode == 0) {
                out[k] = v[u];
            } else if (mode == 1) {
                const double2 o = ld[u];
                const double2 r = make_double2(v[u].x - (double)o.x, v[u].y - (double)o.y);
                R[k] = r;
                acc[0] += wv * (r.x * r.x + r.y * r.y);
                cmax = fmax(cmax, wv * fmax(fabs(r.x), fabs(r.y)));
            } else if (mode == 2) {
                Vd[k] = v[u];
                const double2 r = ld[u];
                acc[0] += wv * (v[u].x * v[u].x + v[u].y * v[u].y);
                acc[1] += wv * (r.x * v[u].x + r.y * v[u].y);
            } else if (mode == 3) {
                const double2 d = ld2[u];
                double2 r = ld[u];
                r.x += alpha * d.x;
                r.y += alpha * d.y;
                R[k] = r;
                acc[0] += wv * (r.x * r.x + r.y * r.y);
                cmax = fmax(cmax, wv * fmax(fabs(r.x), fabs(r.y)));
            } else {
                const double2 r = ld[u];
                cmax = fmax(cmax, wv * fmax(fabs(r.x), fabs(r.y)));
            }
        }
    }
    if (mode != 0 && mode != 4) {
        block_sum<2>(acc);
        if (threadIdx.x == 0) {
            coh_store(vispart + (size_t)item * NPART + 0, acc[0]);
            coh_store(vispart + (size_t)item * NPART + 1, acc[1]);
        }
    }
    if (with_max && mode != 0 && mode != 2) {
        cmax = -block_min(-cmax);
        if (threadIdx.x == 0) coh_store(vispart + (size_t)item * NPART + 2, cmax);
    }
}

// Visibility pass over the context's items (modes 0, 1, 3 and 4 above).
__global__ __launch_bounds__(NTHR) void k_vis(const VisItem *__restrict__ items,
                                              const double2 *__restrict__ vpart, int n_parts, long long ztot,
                                              const double2 *__restrict__ vo, const float *__restrict__ w,
                                              double2 *__restrict__ R, double2 *__restrict__ Vd,
                                              double2 *__restrict__ out, const double *__restrict__ scal,
                                              double *__restrict__ vispart, const int *__restrict__ chan_img,
                                              int mode, int with_max) {
    const VisItem it = items[blockIdx.x];
    const int img = chan_img ? chan_img[it.chan] : 0;
    const double alpha = mode == 3 ? scal[(size_t)img * UVMEM_NSCAL + UVMEM_S_ALPHA] : 0.0;
    vis_item(it, blockIdx.x, vpart, n_parts, ztot, vo, w, R, Vd, out, vispart, mode, with_max, alpha);
}

// ---------------------------------------------------------------- gradient
// G = sum over the channel's split-K slots of gpart (fixed order);
// mode 0: out = A o G (adjoint only)
// mode 1: out = A o G + lambda (ln(I/M) + 1)            (grad Phi)
// mode 2: as 1 into g; gt = g with zeros on the active set; partials
//         [0] = gt_new . gt_new, [1] = gt_new . gt_old; gt updated in place.
// mode 3: out = scale_img x G without the attenuation (dirty image / PSF).
// With a focus-of-attention mask, pixels outside it are not free: modes 1
// and 2 write 0 there (gradient and projected gradient).
// The last workgroup of an image finishes modes 1 and 2 (grad_tail).
// TR (fast evaluation, several channels per image): the planes hold sums over
// channels with A applied already; mode 1 also sums S and checks the domain,
// mode 2 first takes the CG step I <- max(I + alpha d, M).
struct GradStep {
    const void *dir;
    int *flag;
};
template <typename R, int RP, typename PT, bool TR>
__global__ __launch_bounds__(NTHR) void k_grad(const PT *__restrict__ gpart, const int *__restrict__ slot_base,
                                               const int *__restrict__ ichan_base,
                                               const R *__restrict__ beam, R *__restrict__ I,
                                               R *__restrict__ out, R *__restrict__ gt,
                                               double *__restrict__ ppart, const double *__restrict__ img_scale,
                                               const unsigned char *__restrict__ mask, int n, int np, int n_pb,
                                               int pb_len, double M, double Mb, double lam, int mode,
                                               GradTail tail, GradStep step) {
    const int c = blockIdx.x / n_pb, pb = blockIdx.x % n_pb;
    const double al = TR && mode == 2 ? tail.ls[(size_t)c * LSS_N + LSS_ALPHA] : 0.0;
    int bad = 0;
    const long long npix = (long long)n * n;
    const int ch0 = ichan_base[c], ch1 = ichan_base[c + 1];   // the channels that see this image
    const size_t np2 = (size_t)np * np;
    constexpr int NA = TR ? 3 : 2;
    double acc[NA] = {};
    // groups of RP pixels per thread; fixed-order sum over the slots with
    // 8 slots x RP pixels of independent loads in flight
    for (int g0 = 0; g0 < pb_len; g0 += RP * NTHR) {
        size_t off[RP];
        bool okp[RP];
#pragma unroll
        for (int r = 0; r < RP; ++r) {
            const long long p = (long long)pb * pb_len + g0 + r * NTHR + threadIdx.x;
            okp[r] = g0 + r * NTHR < pb_len && p < npix;
            const long long pc = okp[r] ? p : 0;
            off[r] = (size_t)(pc / n) * np + (size_t)(pc % n);
        }
        // per-pixel inputs of the epilogue and the first channel's beam,
        // loaded ahead of the slot sums, unconditionally (from a stand-in
        // array where one is absent or unused, so that no load sits behind a
        // branch; such values are never used)
        const R *Isrc = mode == 1 || mode == 2 ? I : gt;
        const unsigned char *msrc = mask ? mask : reinterpret_cast<const unsigned char *>(gt);
        const size_t bbase = (size_t)(ch0 < ch1 ? ch0 : 0) * npix;
        R xI[RP], xgt[RP], bm0[RP];
        unsigned char mk[RP];
#pragma unroll
        for (int r = 0; r < RP; ++r) {
            const long long p = (long long)pb * pb_len + g0 + r * NTHR + threadIdx.x;
            const long long pc = okp[r] ? p : 0;
            const size_t q = (size_t)c * npix + pc;
            xI[r] = Isrc[q];
            xgt[r] = gt[q];
            mk[r] = msrc[q];
            bm0[r] = beam[bbase + pc];
        }
        // grad chi^2 = sum over the image's channels of A_ch o (sum of the
        // channel's slots)
        double AG[RP];
#pragma unroll
        for (int r = 0; r < RP; ++r) AG[r] = 0.0;
        for (int ch = ch0; ch < (TR ? ch0 + 1 : ch1); ++ch) {
            const int s0 = slot_base[ch], s1 = slot_base[ch + 1];
            double Gs[RP];
#pragma unroll
            for (int r = 0; r < RP; ++r) Gs[r] = 0.0;
            int s = s0;
            // UL slots x RP pixels of independent loads in flight (32 slots
            // when a thread owns one pixel), then batches of 8; the sum
            // stays in slot order
            constexpr int UL = RP == 1 ? 32 : 8;
            auto batch = [&](auto ul) {
                constexpr int B = decltype(ul)::value;
                double v[RP][B];
#pragma unroll
                for (int r = 0; r < RP; ++r)
#pragma unroll
                    for (int u = 0; u < B; ++u) v[r][u] = (double)gpart[(size_t)(s + u) * np2 + off[r]];
#pragma unroll
                for (int r = 0; r < RP; ++r)
#pragma unroll
                    for (int u = 0; u < B; ++u) Gs[r] += v[r][u];
                s += B;
            };
            while (s + UL <= s1) batch(std::integral_constant<int, UL>());
            if constexpr (UL > 8)
                while (s + 8 <= s1) batch(std::integral_constant<int, 8>());
            for (; s < s1; ++s) {
#pragma unroll
                for (int r = 0; r < RP; ++r) Gs[r] += (double)gpart[(size_t)s * np2 + off[r]];
            }
#pragma unroll
            for (int r = 0; r < RP; ++r) {
                const long long p = (long long)pb * pb_len + g0 + r * NTHR + threadIdx.x;
                const double A = TR || mode == 3 ? 1.0 : ch == ch0 ? (double)bm0[r] : (double)beam[(size_t)ch * npix + p];
                if (okp[r]) AG[r] += A * Gs[r];
            }
        }
#pragma unroll
        for (int r = 0; r < RP; ++r) {
            if (!okp[r]) continue;
            const long long p = (long long)pb * pb_len + g0 + r * NTHR + threadIdx.x;
            const size_t q = (size_t)c * npix + p;
            double gv = AG[r];
            if (mode == 3) gv *= img_scale[c];
            double x = (double)xI[r];
            if (mode == 1 || mode == 2) {
                if (TR && mode == 2 && al != 0.0) {
                    const R xr = (R)fmax(x + al * (double)reinterpret_cast<const R *>(step.dir)[q], Mb);
                    I[q] = xr;
                    x = (double)xr;
                }
                const double lg = log(x / M);
                if (TR) {
                    if (!(x > 0.0)) bad = 1;
                    else acc[mode == 1 ? 0 : NA - 1] += x * lg;
                }
                gv += lam * (lg + 1.0);
                if (mask && !mk[r]) gv = 0.0;
            }
            const R gr = (R)gv;
            out[q] = gr;
            if (mode == 2) {
                const bool act = (x <= Mb * (1.0 + BOUND_TOL)) && ((double)gr > 0.0);
                const double gnew = act ? 0.0 : (double)gr;
                const double gold = (double)xgt[r];
                gt[q] = (R)gnew;
                acc[0] += gnew * gnew;
                acc[1] += gnew * gold;
            }
        }
    }
    if (mode == 2 || (TR && mode == 1)) {
        if (TR && bad) atomicOr(step.flag, 1);
        block_sum<NA>(acc);
        if (threadIdx.x == 0) {
#pragma unroll
            for (int x = 0; x < NA; ++x) coh_store(ppart + ((size_t)c * n_pb + pb) * NPART + x, acc[x]);
        }
    }
    grad_tail<NTHR, TR>(mode, c, pb, n_pb, ppart, lam, tail);
}

// ---------------------------------------------------------------- CG
// Initial projected gradient gt = g off the active set, partial |gt|^2; the
// last workgroup of an image starts its CG bookkeeping.
template <typename R>
__global__ __launch_bounds__(NTHR) void k_cg_init(const R *__restrict__ I, const R *__restrict__ g,
                                                  R *__restrict__ gt, R *__restrict__ dir,
                                                  double *__restrict__ ppart, int n, int n_pb, int pb_len, double Mb,
                                                  unsigned *__restrict__ ctr, double *__restrict__ scal,
                                                  double *__restrict__ chan) {
    const int c = blockIdx.x / n_pb, pb = blockIdx.x % n_pb;
    const long long npix = (long long)n * n;
    double acc[1] = {0.0};
    for (int r = 0; r < pb_len / NTHR; ++r) {
        const long long p = (long long)pb * pb_len + r * NTHR + threadIdx.x;
        if (p >= npix) break;
        const size_t q = (size_t)c * npix + p;
        const double x = (double)I[q], gv = (double)g[q];
        const bool act = (x <= Mb * (1.0 + BOUND_TOL)) && (gv > 0.0);
        const double gn = act ? 0.0 : gv;
        gt[q] = (R)gn;
        dir[q] = (R)0;
        acc[0] += gn * gn;
    }
    block_sum<1>(acc);
    if (threadIdx.x == 0) coh_store(ppart + ((size_t)c * n_pb + pb) * NPART + 0, acc[0]);
    if (!arrive_last(ctr, c, pb, n_pb)) return;
    double gg[1];
    sum_partials<1>(ppart + (size_t)c * n_pb * NPART, n_pb, 0, gg);
    if (threadIdx.x == 0) {
        double *sc = scal + (size_t)c * UVMEM_NSCAL;
        sc[UVMEM_S_ALPHA] = 0.0;
        sc[UVMEM_S_BETA] = 0.0;
        sc[UVMEM_S_GNORM2] = gg[0];
        sc[UVMEM_S_ALPHA_MAX] = 0.0;
        sc[UVMEM_S_ITER] = 0.0;
        double *ch = chan + (size_t)c * CH_N;
        for (int x = 0; x < CH_N; ++x) ch[x] = 0.0;
        ch[CH_GG_OLD] = gg[0];
        ch[CH_STOP] = gg[0] == 0.0 ? 1.0 : 0.0;
    }
}

// Steps 1-3: d <- -gt + beta d, projected onto the feasible directions at the
// bound (d = 0 on the active set, d >= 0 on the other bound pixels), stored
// with B = A o d for the forward model; partials of gt . d and, for this
// direction and for the restart direction -gt, of the entropy parts of
// phi'(0) - b and phi''(0) - a and of alpha_max.  The last workgroup of an
// image takes step 2: restart with d = -gt when gt . d >= 0 (it then rewrites
// the image's d and B itself, which a restart alone needs; bop null: no B), stop when the
// projected gradient is zero; it keeps the chosen direction's totals and
// starts the line search of an image that has no visibilities.
template <typename R>
__global__ __launch_bounds__(NTHR) void k_cg_dir(const R *__restrict__ I, const R *__restrict__ g,
                                                 const R *__restrict__ gt, R *__restrict__ dir,
                                                 const R *__restrict__ beam, R *__restrict__ bop,
                                                 const int *__restrict__ ichan_base,
                                                 const double *__restrict__ scal, double *__restrict__ chan,
                                                 double *__restrict__ ppart, int n, int np, int n_pb, int pb_len,
                                                 double M, double Mb, double lam, unsigned *__restrict__ ctr,
                                                 const int *__restrict__ ivis_base, double *__restrict__ ls) {
    const int c = blockIdx.x / n_pb, pb = blockIdx.x % n_pb;
    const long long npix = (long long)n * n;
    const double beta = scal[(size_t)c * UVMEM_NSCAL + UVMEM_S_BETA];
    const bool stop = chan[(size_t)c * CH_N + CH_STOP] != 0.0;
    const int ch0 = ichan_base[c], ch1 = ichan_base[c + 1];   // the channels that see this image
    // [0] gt . d; entropy parts [1], [2] of d and [3], [4] of -gt
    double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    double am_d = INFINITY, am_s = INFINITY;
    for (int r = 0; r < pb_len / NTHR; ++r) {
        const long long p = (long long)pb * pb_len + r * NTHR + threadIdx.x;
        if (p >= npix) break;
        const size_t q = (size_t)c * npix + p;
        const double x = (double)I[q], gv = (double)g[q], gtv = (double)gt[q];
        // the first channel's beam with the other loads (the stores below
        // would otherwise hold it back)
        const R bm0 = ch0 < ch1 ? beam[(size_t)ch0 * npix + p] : R(0);
        double d = -gtv + beta * (double)dir[q];
        const bool atb = x <= Mb * (1.0 + BOUND_TOL);
        if (atb && gv > 0.0) d = 0.0;
        else if (atb) d = fmax(d, 0.0);
        if (stop) d = 0.0;
        const R dr = (R)d;
        // device-coherent stores: a restart rewrites these pixels from the
        // last workgroup, which may run on another chiplet, and no cache may
        // keep an older copy to write back after it
        coh_store(dir + q, dr);
        const int i = (int)(p / n), j = (int)(p % n);
        for (int ch = ch0; ch < ch1 && bop; ++ch)
            coh_store(bop + (size_t)ch * np * np + (size_t)i * np + j,
                      (ch == ch0 ? bm0 : beam[(size_t)ch * npix + p]) * dr);
        d = (double)dr;
        const double s = stop ? 0.0 : -gtv;
        const double lg = log(x / M) + 1.0;
        acc[0] += gtv * d;
        acc[1] += d * lg;
        acc[2] += d * d / x;
        acc[3] += s * lg;
        acc[4] += s * s / x;
        if (d < 0.0) am_d = fmin(am_d, (x - Mb) / (-d));
        if (s < 0.0) am_s = fmin(am_s, (x - Mb) / (-s));
    }
    block_sum<5>(acc);
    am_d = block_min(am_d);
    am_s = block_min(am_s);
    if (threadIdx.x == 0) {
        double *pp = ppart + ((size_t)c * n_pb + pb) * NPART;
        for (int m = 0; m < 5; ++m) coh_store(pp + m, acc[m]);
        coh_store(pp + 5, am_d);
        coh_store(pp + 6, am_s);
    }
    if (!arrive_last(ctr, c, pb, n_pb)) return;
    double t[5];
    double amm[2];
    sum_min_partials<5, 2>(ppart + (size_t)c * n_pb * NPART, n_pb, t, amm);
    const double am0 = amm[0], am1 = amm[1];
    const double gg = scal[(size_t)c * UVMEM_NSCAL + UVMEM_S_GNORM2];
    const bool restart = t[0] >= 0.0;
    const bool stop_now = stop || gg == 0.0;
    if (threadIdx.x == 0) {
        double *ch = chan + (size_t)c * CH_N;
        if (stop_now) ch[CH_STOP] = 1.0;
        ch[CH_RESTART] = restart ? 1.0 : 0.0;
        ch[CH_GTD] = restart ? -gg : t[0];
        ch[CH_GG_OLD] = gg;
        ch[CH_E1] = restart ? t[3] : t[1];
        ch[CH_E2] = restart ? t[4] : t[2];
        ch[CH_AMAX] = restart ? am1 : am0;
        // no visibility workgroup will start this image's line search
        if (ivis_base[c + 1] == ivis_base[c])
            ls_init(ls + (size_t)c * LSS_N, 0.0, 0.0, lam * ch[CH_E1], lam * ch[CH_E2], ch[CH_AMAX], stop_now,
                    false, 0.0, 0.0);
    }
    // a stopped image's direction is zero already (gt = 0 or stop)
    if (!restart || stop_now) return;
    for (long long p = threadIdx.x; p < npix; p += NTHR) {
        const size_t q = (size_t)c * npix + p;
        const R dr = (R)(-(double)gt[q]);
        coh_store(dir + q, dr);
        const int i = (int)(p / n), j = (int)(p % n);
        for (int ch = ch0; ch < ch1 && bop; ++ch)
            coh_store(bop + (size_t)ch * np * np + (size_t)i * np + j, beam[(size_t)ch * npix + p] * dr);
    }
}

// The line search itself is described with its start (reduce.h).

// Advance the state with phi'(T_m) = f[m], phi''(T_m) = h[m].
__device__ void ls_update(double *st, const double *f, const double *h) {
    if ((int)st[LSS_PHASE] == PH_DONE) return;
    int m = 0;
    while (m < LS_K && f[m] <= 0.0) ++m;
    if (m > 0 && f[m - 1] == 0.0) { ls_finish(st, st[LSS_T0 + m - 1]); return; }
    if (m > 0) {
        st[LSS_LO] = st[LSS_T0 + m - 1];
        st[LSS_FLO] = f[m - 1];
        st[LSS_HLO] = h[m - 1];
    }
    if (m < LS_K) {
        st[LSS_HI] = st[LSS_T0 + m];
        st[LSS_FHI] = f[m];
        st[LSS_HHI] = h[m];
        st[LSS_HI_EVAL] = 1.0;
    } else if (st[LSS_HI] >= 0.0 && st[LSS_HI_EVAL] == 0.0 && st[LSS_T0 + LS_K - 1] == st[LSS_HI]) {
        // phi'(HI) <= 0 at an unevaluated end: HI is alpha_max, the minimiser
        // on [0, alpha_max], or the bound -phi'(0)/a, where phi' >= 0, so the
        // root up to rounding
        ls_finish(st, st[LSS_HI]);
        return;
    }
    const double lo = st[LSS_LO], hi = st[LSS_HI];
    if (st[LSS_HI_EVAL] != 0.0 && hi - lo <= 1e-13 * hi) {
        ls_finish(st, ls_cubic(st));
        return;
    }
    ls_propose(st);
}

// Accepted step when the pass budget ran out: the cubic's root in the
// bracket, or the largest step known to descend.
__device__ double ls_fallback(const double *st) {
    return st[LSS_HI_EVAL] != 0.0 ? ls_cubic(st) : st[LSS_LO];
}

// Sum the LS_K (phi' entropy part, phi'' entropy part) partials of a channel
// and turn them into phi', phi'' at the trial steps.
__device__ __forceinline__ void ls_eval(const double *st, const double *pp, int n_pb, double lam,
                                        double *f, double *h) {
    double e[2 * LS_K];
    sum_partials<2 * LS_K>(pp, n_pb, 0, e);
#pragma unroll
    for (int m = 0; m < LS_K; ++m) {
        const double t = st[LSS_T0 + m];
        f[m] = st[LSS_B] + st[LSS_A] * t + lam * e[2 * m];
        h[m] = st[LSS_A] + lam * e[2 * m + 1];
    }
}

// Step 5: Vd and the partials of a = sum w |Vd|^2 and b = sum w Re(conj(R) Vd)
// (the first n_visit workgroups, one visibility item each), and the entropy
// parts of phi', phi'' at alpha_max (pixel workgroups of the images that have
// visibilities; zero without a finite alpha_max).  The last workgroup of an
// image starts its line search from these totals and the direction pass's.
template <typename R>
__global__ __launch_bounds__(NTHR) void k_cg_vis(const VisItem *__restrict__ items, int n_visit,
                                                 const double2 *__restrict__ vpart, int n_parts, long long ztot,
                                                 const float *__restrict__ w, double2 *__restrict__ Rv,
                                                 double2 *__restrict__ Vd, double *__restrict__ vispart,
                                                 const int *__restrict__ chan_img, const int *__restrict__ ivis_base,
                                                 const R *__restrict__ I, const R *__restrict__ dir,
                                                 double *__restrict__ ppart, int n, int n_pb, int pb_len, double M,
                                                 double lam, const double *__restrict__ chan,
                                                 double *__restrict__ ls, unsigned *__restrict__ ctr) {
    int img, rank = -1;   // the workgroup's pixel block, if it has one
    if ((int)blockIdx.x < n_visit) {
        const VisItem it = items[blockIdx.x];
        img = chan_img[it.chan];
        vis_item(it, blockIdx.x, vpart, n_parts, ztot, nullptr, w, Rv, Vd, nullptr, vispart, 2, 0, 0.0);
    } else {
        const int blk = (int)blockIdx.x - n_visit;
        img = blk / n_pb;
        const int pb = rank = blk % n_pb;
        const long long npix = (long long)n * n;
        // the thread's first pixel, loaded ahead of the image's scalars
        // (pixel 0 stands in past the end)
        const long long p_1 = (long long)pb * pb_len + threadIdx.x;
        const size_t q_1 = (size_t)img * npix + (p_1 < npix ? p_1 : 0);
        const R d_1 = dir[q_1], x_1 = I[q_1];
        if (ivis_base[img + 1] == ivis_base[img]) return;   // started by the direction pass
        const double *chc = chan + (size_t)img * CH_N;
        const double am = chc[CH_AMAX];
        double acc[2] = {0.0, 0.0};
        if (isfinite(am) && chc[CH_STOP] == 0.0) {
            for (int r = 0; r < pb_len / NTHR; ++r) {
                const long long p = (long long)pb * pb_len + r * NTHR + threadIdx.x;
                if (p >= npix) break;
                const size_t q = (size_t)img * npix + p;
                const double d = r == 0 ? (double)d_1 : (double)dir[q];
                if (d == 0.0) continue;
                const double x = (r == 0 ? (double)x_1 : (double)I[q]) + am * d;
                acc[0] += d * (log(x / M) + 1.0);
                acc[1] += d * d / x;
            }
        }
        block_sum<2>(acc);
        if (threadIdx.x == 0) {
            coh_store(ppart + ((size_t)img * n_pb + pb) * NPART + 0, acc[0]);
            coh_store(ppart + ((size_t)img * n_pb + pb) * NPART + 1, acc[1]);
        }
    }
    const int v0 = ivis_base[img], v1 = ivis_base[img + 1];
    if (!arrive_last(ctr, img, rank < 0 ? (int)blockIdx.x - v0 : v1 - v0 + rank, v1 - v0 + n_pb)) return;
    double ab[2], fh[2];
    sum_partials2<2, 2>(vispart + (size_t)v0 * NPART, v1 - v0, 0, ab, ppart + (size_t)img * n_pb * NPART, n_pb, 0,
                        fh);
    if (threadIdx.x == 0) {
        const double *ch = chan + (size_t)img * CH_N;
        ls_init(ls + (size_t)img * LSS_N, ab[0], ab[1], lam * ch[CH_E1], lam * ch[CH_E2], ch[CH_AMAX],
                ch[CH_STOP] != 0.0, true, lam * fh[0], lam * fh[1]);
    }
}

// Pass of the line search: every workgroup of an image reads the state and
// evaluates the phi', phi'' partials at its LS_K trial steps; the last
// workgroup to arrive advances the state with the totals (in the last pass,
// a search that has not converged takes its fallback step).  A converged
// search makes the whole image skip the pass.
template <typename R>
__global__ __launch_bounds__(NTHR) void k_ls_step(const R *__restrict__ I, const R *__restrict__ dir,
                                                  double *__restrict__ ls, double *__restrict__ ppart,
                                                  int n, int n_pb, int pb_len, double M, double lam, int last_pass,
                                                  unsigned *__restrict__ ctr) {
    const int c = blockIdx.x / n_pb, pb = blockIdx.x % n_pb;
    const long long npix = (long long)n * n;
    // the thread's first pixel, loaded ahead of the state (pixel 0 stands in
    // past the end)
    const long long p_1 = (long long)pb * pb_len + threadIdx.x;
    const size_t q_1 = (size_t)c * npix + (p_1 < npix ? p_1 : 0);
    const R d_1 = dir[q_1], x_1 = I[q_1];
    __shared__ double st[LSS_N];
    double *lsc = ls + (size_t)c * LSS_N;
    if (threadIdx.x < LSS_N) st[threadIdx.x] = lsc[threadIdx.x];
    __syncthreads();
    if ((int)st[LSS_PHASE] == PH_DONE) return;
    double tr[LS_K];
#pragma unroll
    for (int m = 0; m < LS_K; ++m) tr[m] = st[LSS_T0 + m];
    double acc[2 * LS_K];
#pragma unroll
    for (int m = 0; m < 2 * LS_K; ++m) acc[m] = 0.0;
    for (int r = 0; r < pb_len / NTHR; ++r) {
        const long long p = (long long)pb * pb_len + r * NTHR + threadIdx.x;
        if (p >= npix) break;
        const size_t q = (size_t)c * npix + p;
        const double d = r == 0 ? (double)d_1 : (double)dir[q];
        if (d == 0.0) continue;
        const double x0 = r == 0 ? (double)x_1 : (double)I[q];
#pragma unroll
        for (int m = 0; m < LS_K; ++m) {
            const double x = x0 + tr[m] * d;
            acc[2 * m] += d * (log(x / M) + 1.0);
            acc[2 * m + 1] += d * d / x;
        }
    }
    block_sum<2 * LS_K>(acc);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int m = 0; m < 2 * LS_K; ++m) coh_store(ppart + ((size_t)c * n_pb + pb) * NPART + m, acc[m]);
    }
    if (!arrive_last(ctr, c, pb, n_pb)) return;
    double f[LS_K], h[LS_K];
    ls_eval(st, ppart + (size_t)c * n_pb * NPART, n_pb, lam, f, h);
    if (threadIdx.x == 0) {
        ls_update(st, f, h);
        if (last_pass && (int)st[LSS_PHASE] != PH_DONE) ls_finish(st, ls_fallback(st));
    }
    __syncthreads();
    if (threadIdx.x < LSS_N) lsc[threadIdx.x] = st[threadIdx.x];
}

// Step 8: I <- max(I + alpha d, M) with the accepted step and the entropy
// partial of the new image (pixel workgroups); R <- R + alpha Vd and its
// chi^2 partials (visibility workgroups, one item each).  The last
// workgroup of an image stores Phi, chi^2, S, alpha and alpha_max.
template <typename R>
__global__ __launch_bounds__(NTHR) void k_cg_update(R *__restrict__ I, const R *__restrict__ dir,
                                                    const double *__restrict__ ls, double *__restrict__ pp_out,
                                                    double *__restrict__ scal, double *__restrict__ chan,
                                                    int *__restrict__ flag,
                                                    int n, int n_pb, int pb_len, double M, double Mb, double lam,
                                                    const VisItem *__restrict__ vitems, const float *__restrict__ w,
                                                    double2 *__restrict__ Rv, const double2 *__restrict__ Vd,
                                                    double *__restrict__ vispart, const int *__restrict__ chan_img,
                                                    const int *__restrict__ ivis_base, int n_pixwg, int with_max,
                                                    unsigned *__restrict__ ctr) {
    const bool visw = (int)blockIdx.x >= n_pixwg;
    const int vi = (int)blockIdx.x - n_pixwg;
    const VisItem vit = visw ? vitems[vi] : VisItem{};
    const int c = visw ? chan_img[vit.chan] : (int)blockIdx.x / n_pb, pb = visw ? -1 : (int)blockIdx.x % n_pb;
    const long long npix = (long long)n * n;
    const double *lsc = ls + (size_t)c * LSS_N;
    const double al = lsc[LSS_ALPHA];
    if (visw) {
        vis_item(vit, vi, nullptr, 0, 0, nullptr, w, Rv, const_cast<double2 *>(Vd), nullptr, vispart, 3, with_max, al);
    } else {
        double acc[1] = {0.0};
        int bad = 0;
        for (int r = 0; r < pb_len / NTHR; ++r) {
            const long long p = (long long)pb * pb_len + r * NTHR + threadIdx.x;
            if (p >= npix) break;
            const size_t q = (size_t)c * npix + p;
            // I and d are loaded together, before the step is known (selects,
            // not a branch, so that the load of d is not deferred behind it)
            const double x0 = (double)I[q], dv = (double)dir[q];
            const R xr = (R)fmax(x0 + al * dv, Mb);
            const bool moved = al != 0.0;
            double x = moved ? (double)xr : x0;
            if (moved) I[q] = xr;
            if (!(x > 0.0)) bad = 1;
            else acc[0] += x * log(x / M);
        }
        if (bad) atomicOr(flag, 1);
        block_sum<1>(acc);
        if (threadIdx.x == 0) coh_store(pp_out + ((size_t)c * n_pb + pb) * NPART + 0, acc[0]);
    }
    const int v0 = ivis_base[c], v1 = ivis_base[c + 1];
    if (!arrive_last(ctr, c, visw ? n_pb + vi - v0 : pb, n_pb + v1 - v0)) return;
    double x2[1], S[1];
    sum_partials2<1, 1>(vispart + (size_t)v0 * NPART, v1 - v0, 0, x2, pp_out + (size_t)c * n_pb * NPART, n_pb, 0,
                        S);
    if (threadIdx.x == 0) {
        double *sc = scal + (size_t)c * UVMEM_NSCAL;
        const double chi2 = 0.5 * x2[0];
        sc[UVMEM_S_PHI] = chi2 + lam * S[0];
        sc[UVMEM_S_CHI2] = chi2;
        sc[UVMEM_S_S] = S[0];
        sc[UVMEM_S_ALPHA] = al;
        sc[UVMEM_S_ALPHA_MAX] = lsc[LSS_AMAX] < 0.0 ? INFINITY : lsc[LSS_AMAX];
        if (al == 0.0) chan[(size_t)c * CH_N + CH_STOP] = 1.0;
    }
}

// History copy for graph replays: dst = *hist_ptr + ctr * (C * NSCAL).
__global__ void k_copy_hist(const double *__restrict__ scal, const long long *__restrict__ hist_ptr,
                            long long *__restrict__ ctr, int count) {
    double *base = reinterpret_cast<double *>(hist_ptr[0]);
    const long long t = ctr[0];
    if (base) {
        for (int x = threadIdx.x; x < count; x += blockDim.x) base[t * count + x] = scal[x];
    }
    __syncthreads();
    if (threadIdx.x == 0) ctr[0] = t + 1;
}

__global__ void k_set_hist(long long *__restrict__ hist_ptr, long long *__restrict__ ctr, long long hist) {
    if (threadIdx.x == 0) {
        hist_ptr[0] = hist;
        ctr[0] = 0;
    }
}

template <typename R> inline R *P(void *p) { return reinterpret_cast<R *>(p); }
template <typename R> inline const R *CP(const void *p) { return reinterpret_cast<const R *>(p); }

inline int pix_grid(const uvmem_ctx *c) { return c->nimg * c->n_pb; }
// Partial records of the pixel passes: buffer 0 holds the prologue's entropy
// partials until the evaluation's gradient pass has read them; every CG pass
// writes buffer 1 and its last workgroups read it in the same launch.
inline double *pp(const uvmem_ctx *c, int buf) {
    return c->d_ppart + (size_t)buf * c->nimg * std::max(c->n_pb, c->n_trrec) * NPART;
}
inline unsigned *ctr(const uvmem_ctx *c, int site) { return c->d_ctr + (size_t)site * c->nimg * CTR_STRIDE; }
// The fp16 split adjoint scales its coefficients by the channel's max |w R|,
// which the visibility pass leaves in slot 2 of its partial records.
inline int adj_scaled(const uvmem_ctx *c) { return c->prec == UVMEM_FP16X3 && !c->tr_lg ? 1 : 0; }

template <typename R>
hipError_t t_prologue(const uvmem_ctx *c, const void *I, int with_entropy, hipStream_t st) {
    hipLaunchKernelGGL(k_prologue<R>, dim3(pix_grid(c)), dim3(NTHR), 0, st, CP<R>(I), CP<R>(c->d_beam),
                       P<R>(c->d_bop), c->d_ichan_base, pp(c, 0), c->d_flag, c->n, c->np, c->n_pb, c->pix_blk, c->M,
                       with_entropy);
    return hipGetLastError();
}

// k_grad with 4 pixels per thread and round when the pixel blocks are long
// enough, else 1 (more workgroups, fewer loads in flight per thread); the
// split-K partials are FP32 for the split precisions, else FP64
template <typename R, typename PT, bool TR>
void grad_launch_t(const uvmem_ctx *c, const void *I, void *out, double *ppart, int mode, double *user,
                   hipStream_t st) {
    const PT *gp = static_cast<const PT *>(c->d_gpart);
    // gradients (modes 1, 2) follow the region-restricted adjoint and its slots
    const int *slots = (mode == 1 || mode == 2) && c->has_region ? c->d_slot_base_m : c->d_slot_base;
    const GradTail tail = make_grad_tail(c, mode, user);
    const GradStep step{c->d_dir, c->d_flag};
    R *img = P<R>(const_cast<void *>(I));   // written by a TR step only
    if (c->pix_blk >= 4 * NTHR)
        hipLaunchKernelGGL((k_grad<R, 4, PT, TR>), dim3(pix_grid(c)), dim3(NTHR), 0, st, gp, slots, c->d_ichan_base,
                           CP<R>(c->d_beam), img, P<R>(out), P<R>(c->d_gt), ppart, c->d_wscale, c->d_mask, c->n,
                           c->np, c->n_pb, c->pix_blk, c->M, c->Mb, c->lam, mode, tail, step);
    else
        hipLaunchKernelGGL((k_grad<R, 1, PT, TR>), dim3(pix_grid(c)), dim3(NTHR), 0, st, gp, slots, c->d_ichan_base,
                           CP<R>(c->d_beam), img, P<R>(out), P<R>(c->d_gt), ppart, c->d_wscale, c->d_mask, c->n,
                           c->np, c->n_pb, c->pix_blk, c->M, c->Mb, c->lam, mode, tail, step);
}

template <typename R>
void grad_launch(const uvmem_ctx *c, const void *I, void *out, double *ppart, int mode, double *user,
                 hipStream_t st) {
    if (c->tr_lg)
        grad_launch_t<R, double, true>(c, I, out, ppart, mode, user, st);
    else if (c->gpart_f32)
        grad_launch_t<R, float, false>(c, I, out, ppart, mode, user, st);
    else
        grad_launch_t<R, double, false>(c, I, out, ppart, mode, user, st);
}

template <typename R>
hipError_t t_cg_init_dir(const uvmem_ctx *c, const void *I, hipStream_t st) {
    hipLaunchKernelGGL(k_cg_init<R>, dim3(pix_grid(c)), dim3(NTHR), 0, st, CP<R>(I), CP<R>(c->d_g),
                       P<R>(c->d_gt), P<R>(c->d_dir), pp(c, 1), c->n, c->n_pb, c->pix_blk, c->Mb,
                       ctr(c, CTR_INIT), c->d_scal, c->d_chan);
    return hipGetLastError();
}

// The CG step in three phases around the DFT launches (phase 0: before the
// forward model, 1: between forward and adjoint, 2: after the adjoint).
template <typename R>
hipError_t t_cg_phase(const uvmem_ctx *c, void *I, double *user, int phase, hipStream_t st) {
    const dim3 gp(pix_grid(c)), blk(NTHR);
    if (phase == 0) {
        // 1-3. direction update and projection, restart test and stop, B = A o d,
        // alpha_max and the entropy parts of phi'(0), phi''(0)
        hipLaunchKernelGGL(k_cg_dir<R>, gp, blk, 0, st, CP<R>(I), CP<R>(c->d_g), CP<R>(c->d_gt), P<R>(c->d_dir),
                           CP<R>(c->d_beam), c->tr_lg ? (R *)nullptr : P<R>(c->d_bop), c->d_ichan_base, c->d_scal,
                           c->d_chan, pp(c, 1), c->n,
                           c->np, c->n_pb, c->pix_blk, c->M, c->Mb, c->lam, ctr(c, CTR_DIR), c->d_ivis_base,
                           c->d_ls);
        return hipGetLastError();
    }
    if (phase == 1) {
        // 5. Vd, the quadratic coefficients a, b of chi^2 along d and phi'
        // at alpha_max; the line search starts from them
        // (the fast evaluation's forward has done all of that)
        if (c->n_visit && !c->tr_lg)
            hipLaunchKernelGGL(k_cg_vis<R>, dim3(c->n_visit + pix_grid(c)), blk, 0, st, c->d_vis, c->n_visit,
                               c->d_vpart, c->has_region ? c->n_vparts_m : c->n_vparts, (long long)c->ztot,
                               c->d_w, c->d_R, c->d_Vd, c->d_vispart, c->d_chan_img, c->d_ivis_base, CP<R>(I),
                               CP<R>(c->d_dir), pp(c, 1), c->n, c->n_pb, c->pix_blk, c->M, c->lam, c->d_chan,
                               c->d_ls, ctr(c, CTR_VIS));
        // 6-7. line-search passes (the last one accepts a step)
        const int L = c->ls_steps;
        for (int t = 0; t < L; ++t)
            hipLaunchKernelGGL(k_ls_step<R>, gp, blk, 0, st, CP<R>(I), CP<R>(c->d_dir), c->d_ls, pp(c, 1), c->n,
                               c->n_pb, c->pix_blk, c->M, c->lam, t == L - 1 ? 1 : 0, ctr(c, CTR_LS));
        // 8-9. I <- max(I + alpha d, M) and its entropy partial (pixel
        // workgroups); R <- R + alpha Vd and the chi^2 partials (visibility
        // workgroups); Phi of the new image
        // (the fast evaluation does this in its spread and gradient passes)
        if (c->tr_lg) return hipGetLastError();
        hipLaunchKernelGGL(k_cg_update<R>, dim3(pix_grid(c) + c->n_visit), blk, 0, st, P<R>(I), CP<R>(c->d_dir),
                           c->d_ls, pp(c, 1), c->d_scal, c->d_chan, c->d_flag, c->n, c->n_pb, c->pix_blk, c->M,
                           c->Mb, c->lam, c->d_vis, c->d_w, c->d_R, c->d_Vd, c->d_vispart, c->d_chan_img,
                           c->d_ivis_base, pix_grid(c), adj_scaled(c), ctr(c, CTR_UPD));
        return hipGetLastError();
    }
    // 10-12. gradient at the new point, projected gradient, beta and the scalars
    return launch_grad(c, I, c->d_g, 2, user, st);
}

}  // namespace

__global__ void k_fill_c(double2 *__restrict__ x, double2 value, long long count) {
    long long i = (long long)blockIdx.x * NTHR + threadIdx.x;
    const long long stride = (long long)gridDim.x * NTHR;
    for (; i < count; i += stride) x[i] = value;
}

hipError_t launch_fill_c(const uvmem_ctx *c, double2 *x, double re, double im, hipStream_t st) {
    const long long count = c->ztot;
    if (count == 0) return hipSuccess;
    const int blocks = (int)std::min<long long>((count + NTHR - 1) / NTHR, 4096);
    hipLaunchKernelGGL(k_fill_c, dim3(blocks), dim3(NTHR), 0, st, x, make_double2(re, im), count);
    return hipGetLastError();
}

hipError_t launch_fill(const uvmem_ctx *c, void *img, double value, hipStream_t st) {
    const long long count = (long long)c->nimg * c->n * c->n;
    const int blocks = (int)std::min<long long>((count + NTHR - 1) / NTHR, 4096);
    if (c->prec == UVMEM_FP64)
        hipLaunchKernelGGL(k_fill<double>, dim3(blocks), dim3(NTHR), 0, st, P<double>(img), value, count);
    else
        hipLaunchKernelGGL(k_fill<float>, dim3(blocks), dim3(NTHR), 0, st, P<float>(img), (float)value, count);
    return hipGetLastError();
}

hipError_t launch_prologue(const uvmem_ctx *c, const void *I, int with_entropy, hipStream_t st) {
    if (c->tr_lg) return hipSuccess;   // part of the fast evaluation's first pass
    return c->prec == UVMEM_FP64 ? t_prologue<double>(c, I, with_entropy, st)
                                 : t_prologue<float>(c, I, with_entropy, st);
}

hipError_t launch_vis_sum(const uvmem_ctx *c, int mode, double2 *out, hipStream_t st) {
    if (c->n_visit == 0 || c->tr_lg) return hipSuccess;   // part of the fast evaluation's forward
    hipLaunchKernelGGL(k_vis, dim3(c->n_visit), dim3(NTHR), 0, st, c->d_vis, c->d_vpart, c->n_vparts,
                       (long long)c->ztot, c->d_vo, c->d_w, c->d_R, c->d_Vd, out, c->d_scal, c->d_vispart,
                       c->d_chan_img, mode, adj_scaled(c));
    return hipGetLastError();
}

hipError_t launch_vis_sum_raw(const VisItem *items, int n_items, const double2 *vpart, int n_parts, long long ztot,
                              double2 *out, hipStream_t st) {
    if (n_items == 0) return hipSuccess;
    hipLaunchKernelGGL(k_vis, dim3(n_items), dim3(NTHR), 0, st, items, vpart, n_parts, ztot,
                       (const double2 *)nullptr, (const float *)nullptr, (double2 *)nullptr, (double2 *)nullptr,
                       out, (const double *)nullptr, (double *)nullptr, (const int *)nullptr, 0, 0);
    return hipGetLastError();
}

hipError_t launch_coef_max(const uvmem_ctx *c, const double2 *coef, hipStream_t st) {
    if (c->n_visit == 0 || !adj_scaled(c)) return hipSuccess;
    hipLaunchKernelGGL(k_vis, dim3(c->n_visit), dim3(NTHR), 0, st, c->d_vis, c->d_vpart, c->n_vparts,
                       (long long)c->ztot, c->d_vo, (const float *)nullptr, const_cast<double2 *>(coef), c->d_Vd,
                       (double2 *)nullptr, c->d_scal, c->d_vispart, c->d_chan_img, 4, 1);
    return hipGetLastError();
}

hipError_t launch_grad(const uvmem_ctx *c, const void *I, void *out, int mode, double *user_scal, hipStream_t st) {
    if (c->tr_lg) {
        // the inverse's last pass; it does the rest itself unless an image
        // sums several channels
        const hipError_t e = launch_tr_rows_inv(c, I, out, mode, user_scal, st);
        if (e != hipSuccess || c->nimg == c->nchan) return e;
    }
    if (c->prec == UVMEM_FP64) grad_launch<double>(c, I, out, pp(c, 1), mode, user_scal, st);
    else grad_launch<float>(c, I, out, pp(c, 1), mode, user_scal, st);
    return hipGetLastError();
}

hipError_t launch_cg_init_dir(const uvmem_ctx *c, const void *I, hipStream_t st) {
    return c->prec == UVMEM_FP64 ? t_cg_init_dir<double>(c, I, st) : t_cg_init_dir<float>(c, I, st);
}

hipError_t launch_copy_scal(const uvmem_ctx *c, double *, long long *ctr, hipStream_t st) {
    hipLaunchKernelGGL(k_copy_hist, dim3(1), dim3(NTHR), 0, st, c->d_scal,
                       reinterpret_cast<const long long *>(c->d_hist_ptr), ctr, c->nimg * UVMEM_NSCAL);
    return hipGetLastError();
}

hipError_t launch_set_hist(const uvmem_ctx *c, double *hist, hipStream_t st) {
    hipLaunchKernelGGL(k_set_hist, dim3(1), dim3(64), 0, st, c->d_hist_ptr, c->d_iter_ctr,
                       (long long)(uintptr_t)hist);
    return hipGetLastError();
}

hipError_t launch_cg_phase(const uvmem_ctx *c, void *I, double *user, int phase, hipStream_t st) {
    return c->prec == UVMEM_FP64 ? t_cg_phase<double>(c, I, user, phase, st)
                                 : t_cg_phase<float>(c, I, user, phase, st);
}

hipError_t launch_cg_step(const uvmem_ctx *c, void *I, double *user, hipStream_t st) {
    hipError_t e;
    if ((e = launch_cg_phase(c, I, user, 0, st)) != hipSuccess) return e;
    if ((e = launch_forward(c, I, st, 1, 2, nullptr)) != hipSuccess) return e;
    if ((e = launch_cg_phase(c, I, user, 1, st)) != hipSuccess) return e;
    if ((e = launch_adjoint(c, c->d_R, c->d_w, st, 1, 0, 1)) != hipSuccess) return e;
    return launch_cg_phase(c, I, user, 2, st);
}

}  // namespace uvm
