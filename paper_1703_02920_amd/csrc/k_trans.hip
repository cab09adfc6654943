// Fast exact evaluation of the direct DFT and its adjoint on gfx950.
//
// Both contractions of k_dft.hip cost Z N^2.  Here the same sums are
// evaluated to working precision through an oversampled grid (a non-uniform
// FFT; the window is the Kaiser-Bessel function, whose transform is closed
// form): with x_m = m, m = j - N/2, L = 2^lg >= 2 N and a window phi of W
// grid nodes,
//   e^{-2 pi i a m} = (1 / phi^(m / L)) sum_q phi(q - a L) e^{-2 pi i q m / L}  (1 + eps),
// so that
//   V_k = sum_{p,q near (b_k L, a_k L)} phi phi G[q][p],
//   G = DFT_L of B[i][j] / (phi^(m_i / L) phi^(m_j / L)) zero-padded to L x L,
// and the adjoint is the transpose of that map.  eps is set by W alone:
// W = 17 reaches FP64 rounding (measured against extended precision: 4e-15 of
// |V| on 64^2 to 300^2 images, where the direct FP64 sum is at 4e-15 to
// 1.1e-14), W = 9 stays near 1e-8 (4e-8 for a source in a corner of the image).
// The transforms compute in FP64 in every context; windows, tile products and
// what is stored between kernels follow the precision (see Tile below).
//
// The image is real, hence V(-u, -v) = conj V(u, v): visibilities are kept
// with a_k in [0, 1/2] (the others negated and conjugated once at finalize)
// and the grid holds only the columns q = -H .. L/2 + H, H = (W - 1) / 2.
// Visibilities are sorted by bin of TB x TB nearest nodes; a bin's windows
// fit one TS x TS node tile (TS = TB + W - 1 = 16 or 32), and both directions
// work on such tiles with FP64 or FP32 matrix instructions: gathering is
// T = (tile) (column windows) followed by a short dot with the row windows,
// spreading is (column windows x coefficient)^T (row windows) with the
// visibilities as the contraction dimension.  Overlapping tiles are summed
// in a fixed order when the inverse transform reads them, so results are
// bitwise reproducible.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <type_traits>
#include <vector>

#include "internal.h"
#include "reduce.h"

namespace uvm {
namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

// Two types follow the precision: S, in which grids, half spectra and tiles
// are stored (the transforms compute in FP64 whatever it is), and A, that of
// the windows and the tile products (float for the split precisions only,
// whose contraction accumulates in FP32 too).  S is float for the split
// precisions, double for FP64; FP32 and FP16X3 contexts store the forward's
// half spectra and grid as double and the adjoint's tiles and half spectra as
// float.  The
// window's correction makes the forward grid of a source in the image's corner
// eleven times its visibilities, cancelled again by the window sums: rounded
// to FP32 there, a corner source was 1.1e-7 off (the FP32 contraction 6e-8),
// in FP64 4e-8, and images whose flux passes FP32 overflowed, in
// FP16X3 too, whose contraction scales its operands.  (FP32, 23 channels of
// 512^2, shared: 291 -> 334 us, one image 0 to 3 %; FP16X3 512^2 x 999,600
// 93 -> 97 to 100, many channels up to 14 %.)  Matrix
// instructions 16 x 16 x 4: lane l supplies A[l%16][l/16] and
// B[l/16][l%16] and holds D[drow(l/16, r)][l%16] in register r.  vec4: four
// window values read from LDS at once, aligned as their rows are (16 bytes; a
// plain vector of four doubles claims 32, which every other row is not).
template <typename S> struct Tile;
template <> struct Tile<double> {
    typedef doublex4 acc;
    typedef double vec4 __attribute__((ext_vector_type(4), aligned(16)));
    typedef double2 c2;
    static __device__ __forceinline__ acc mma(double a, double b, acc c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int drow(int g, int r) { return 4 * r + g; }
    static constexpr int PAD = 2;   // row padding of the LDS windows: 16 bytes
};
template <> struct Tile<float> {
    typedef floatx4 acc;
    typedef float vec4 __attribute__((ext_vector_type(4), aligned(16)));
    typedef float2 c2;
    static __device__ __forceinline__ acc mma(float a, float b, acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int drow(int g, int r) { return 4 * g + r; }
    static constexpr int PAD = 4;
};
template <typename S> using C2 = typename Tile<S>::c2;
__device__ __forceinline__ double2 wide(double2 a) { return a; }
__device__ __forceinline__ double2 wide(float2 a) { return make_double2((double)a.x, (double)a.y); }
template <typename S> __device__ __forceinline__ C2<S> narrow(double x, double y) { return C2<S>{(S)x, (S)y}; }

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
// multiplication by -i (forward) or +i (inverse)
template <bool INV>
__device__ __forceinline__ double2 crot(double2 a) {
    return INV ? make_double2(-a.y, a.x) : make_double2(a.y, -a.x);
}

// ---------------------------------------------------------------- FFT
// In-place radix-R butterflies, outputs in natural order.
template <bool INV>
__device__ __forceinline__ void dft4(double2 &a0, double2 &a1, double2 &a2, double2 &a3) {
    const double2 s0 = cadd(a0, a2), d0 = csub(a0, a2), s1 = cadd(a1, a3), d1 = crot<INV>(csub(a1, a3));
    a0 = cadd(s0, s1);
    a1 = cadd(d0, d1);
    a2 = csub(s0, s1);
    a3 = csub(d0, d1);
}
template <bool INV>
__device__ __forceinline__ void dft8(double2 (&v)[8]) {
    constexpr double C = 0.70710678118654752440;
    double2 e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6];
    double2 o0 = v[1], o1 = v[3], o2 = v[5], o3 = v[7];
    dft4<INV>(e0, e1, e2, e3);
    dft4<INV>(o0, o1, o2, o3);
    // o_k *= e^{-+ 2 pi i k / 8}
    const double2 r1 = crot<INV>(o1), r3 = crot<INV>(o3);
    o1 = make_double2(C * (o1.x + r1.x), C * (o1.y + r1.y));
    o2 = crot<INV>(o2);
    o3 = make_double2(C * (r3.x - o3.x), C * (r3.y - o3.y));
    v[0] = cadd(e0, o0);
    v[1] = cadd(e1, o1);
    v[2] = cadd(e2, o2);
    v[3] = cadd(e3, o3);
    v[4] = csub(e0, o0);
    v[5] = csub(e1, o1);
    v[6] = csub(e2, o2);
    v[7] = csub(e3, o3);
}

// LDS element of sequence position o: one pad element per eight keeps the
// stride-8 stores of the first pass on distinct banks.
__device__ __forceinline__ constexpr int fpad(int o) { return o + (o >> 3); }

// Radix of pass p for L = 2^LG (0 past the last): eights first, then fours.
__host__ __device__ constexpr int fft_radix(int lg, int p) {
    // lg = 3 e + 2 f with f in {0, 1, 2}
    const int f = lg % 3 == 0 ? 0 : lg % 3 == 2 ? 1 : 2;
    const int e = (lg - 2 * f) / 3;
    return p < e ? 8 : p < e + f ? 4 : 0;
}
constexpr int fft_threads(int lg) { return (1 << lg) / 8; }

// One Stockham pass: thread t of L/8 holds, for butterfly b < 8/R and leg r,
// sequence position (t + b L/8) + r L/R; Ns is the product of the earlier
// radices.  Multiplies by the pass's twiddles and transforms in registers.
template <int LG, int R, int NS, bool INV>
__device__ __forceinline__ void fft_butterflies(double2 (&v)[8], int t, const double2 *__restrict__ tw) {
    constexpr int L = 1 << LG, T = L / 8, NB = 8 / R;
    if constexpr (NS > 1) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int k = ((t + b * T) & (NS - 1)) * (L / (NS * R));
            auto w = [&](int m) {
                double2 x = tw[k * m];
                if (INV) x.y = -x.y;
                return x;
            };
            const double2 w1 = w(1), w2 = w(2);
            v[b * R + 1] = cmul(v[b * R + 1], w1);
            v[b * R + 2] = cmul(v[b * R + 2], w2);
            const double2 w3 = cmul(w1, w2);
            v[b * R + 3] = cmul(v[b * R + 3], w3);
            if constexpr (R == 8) {
                const double2 w4 = w(4);
                v[4] = cmul(v[4], w4);
                v[5] = cmul(v[5], cmul(w1, w4));
                v[6] = cmul(v[6], cmul(w2, w4));
                v[7] = cmul(v[7], cmul(w3, w4));
            }
        }
    }
    if constexpr (R == 8) {
        dft8<INV>(v);
    } else {
#pragma unroll
        for (int b = 0; b < NB; ++b) dft4<INV>(v[b * 4], v[b * 4 + 1], v[b * 4 + 2], v[b * 4 + 3]);
    }
}

// Passes P.. of the transform of L = 2^LG points held 8 per thread by the
// L/8 threads of a sequence, exchanged through s (fpad'ed); every sequence of
// the workgroup runs in step (__syncthreads).  On return leg r of butterfly b
// holds output position (t + b L/8) + r L/R of the last pass's radix R.
template <int LG, int P, int NS, bool INV>
__device__ __forceinline__ void fft_passes(double2 (&v)[8], int t, double2 *s, const double2 *__restrict__ tw) {
    constexpr int L = 1 << LG, T = L / 8;
    constexpr int R = fft_radix(LG, P), RN = fft_radix(LG, P + 1);
    fft_butterflies<LG, R, NS, INV>(v, t, tw);
    if constexpr (RN != 0) {
        __syncthreads();   // the buffer's earlier readers are done
#pragma unroll
        for (int b = 0; b < 8 / R; ++b) {
            const int jj = t + b * T;
            const int base = (jj / NS) * (NS * R) + (jj & (NS - 1));
#pragma unroll
            for (int r = 0; r < R; ++r) s[fpad(base + r * NS)] = v[b * R + r];
        }
        __syncthreads();
#pragma unroll
        for (int b = 0; b < 8 / RN; ++b)
#pragma unroll
            for (int r = 0; r < RN; ++r) v[b * RN + r] = s[fpad(t + b * T + r * (L / RN))];
        fft_passes<LG, P + 1, NS * R, INV>(v, t, s, tw);
    }
}
// Radix of the last pass.
constexpr int fft_last(int lg) {
    int p = 0;
    while (fft_radix(lg, p + 1)) ++p;
    return fft_radix(lg, p);
}
// Output position of register x (leg x % R of butterfly x / R).
template <int LG>
__device__ __forceinline__ int fft_out(int t, int x) {
    constexpr int R = fft_last(LG);
    return t + (x / R) * ((1 << LG) / 8) + (x % R) * ((1 << LG) / R);
}

// Whether output register x, or input leg r, can lie in the image at all: the
// image takes at most a quarter of the positions at either end (L >= 2 N).
template <int LG>
__device__ __forceinline__ constexpr bool fft_live(int x) {
    return fft_last(LG) == 8 ? (x < 2 || x >= 6) : (x % 4 == 0 || x % 4 == 3);
}
__device__ __forceinline__ constexpr bool leg_live(int r) { return r < 2 || r >= 6; }

// Image index of transform position p (pixel offset p or p - L), -1 in the
// zero padding.
__device__ __forceinline__ int pix_of(int p, int L, int n) {
    const int half = n / 2;
    return p < half ? p + half : p >= L - half ? p - (L - half) : -1;
}

// Sequences per workgroup: enough for a whole wave at the short lengths, two
// rows above so that a column access has 32 bytes (FP32 half spectra, one row
// at L = 1024: one 512^2 image 6.3 -> 5.9 us, but 23 channels 29.5 -> 34.7),
// one column.
constexpr int row_seqs(int lg) { return tr_row_seqs(lg); }
constexpr int col_seqs(int lg) { return lg <= 6 ? 8 : lg <= 7 ? 4 : lg <= 8 ? 2 : 1; }

// Row block of a workgroup.  The row passes touch 2 NF rows of every column,
// less than a 128-byte line of X or Y: the blocks of a line go to one XCD
// (workgroups are dealt to the eight in turn), next to each other in time, so
// that its L2 holds the line for all of them.  FP32 half spectra, 1024^2:
// forward rows 11.8 -> 9.9 us, inverse rows 42.3 -> 39.8; 23 channels of
// 512^2: 32.6 -> 29.5 and 49.3 -> 43.0.
template <typename S, int NF> __device__ __forceinline__ int row_block() {
    constexpr int G = NF >= 8 ? 1 : 64 / ((int)sizeof(C2<S>) * NF) > 1 ? 64 / ((int)sizeof(C2<S>) * NF) : 1;
    const int b = blockIdx.x, k = b / 8;
    if (G == 1 || b >= (int)gridDim.x / (8 * G) * (8 * G)) return b;
    return (k / G * 8 + b % 8) * G + k % G;
}

// DIR: the image is a CG direction, and the row pass also sums the entropy
// parts of phi', phi'' at alpha_max (partials [0], [1]; zero without a finite
// alpha_max).  Done by the first channel of each image; one record per
// workgroup, gridDim.x per image.
template <typename R> struct RowArgs {
    const R *img;               // the image, or the direction
    const R *I;                 // DIR: the current point
    const R *beam;
    const int *chan_img, *ichan_base;
    const double *chan;         // DIR: CG bookkeeping
    double *pp;
    double M;
};

// Rows: two rows (i, i + 1) of B = A o img form one complex sequence; their
// spectra are separated by symmetry and stored as X[q + H][i], i contiguous,
// for the columns q = -H .. L/2 + H.  Bound by latency (loads, three or four
// exchanges through LDS, stores) for one image: 5 us at 256^2, at 1024^2 9.6
// (bf16x3) and 12.0 (FP32, whose half spectra are FP64); 23 channels
// of 512^2 in FP32 102 MB stored in 36.8 us (51 MB as FP32 in 29.5).  With the
// attenuation in a launch of its own 1024^2 took 9.5 + 12.
template <int LG, typename R, typename S, bool DIR>
__global__ __launch_bounds__(row_seqs(LG) * fft_threads(LG)) void k_tr_rows_fwd(
    const RowArgs<R> ra, C2<S> *__restrict__ X, const double2 *__restrict__ tw, const double *__restrict__ dec,
    int n, int H) {
    constexpr int L = 1 << LG, T = fft_threads(LG), NF = row_seqs(LG);
    __shared__ double2 s[NF][fpad(L)];
    const int f = threadIdx.x / T, t = threadIdx.x % T;
    const int rows0 = row_block<S, NF>() * NF * 2;
    const int c = blockIdx.y, i0 = rows0 + 2 * f;
    const int Lx = L / 2 + 2 * H + 1;
    const int im = ra.chan_img[c];
    double2 v[8];
    const bool live = i0 < n;   // n is even
    const size_t r0 = (size_t)(live ? i0 : 0) * n, npix = (size_t)n * n;
    const R *x0 = ra.img + im * npix + r0, *A0 = ra.beam + c * npix + r0;
    const double d0 = live ? dec[i0] : 0.0, d1 = live ? dec[i0 + 1] : 0.0;
    R px[8], py[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        v[r] = make_double2(0.0, 0.0);
        px[r] = py[r] = R(0);
        if (!leg_live(r)) continue;
        const int j = pix_of(t + r * T, L, n);
        const int jc = j < 0 ? 0 : j;
        px[r] = x0[jc];
        py[r] = x0[n + jc];
        const R bx = A0[jc] * px[r], by = A0[n + jc] * py[r];
        const double dj = dec[jc];
        v[r] = j < 0 ? make_double2(0.0, 0.0) : make_double2((double)bx * (d0 * dj), (double)by * (d1 * dj));
    }
    if constexpr (DIR) {
        if (ra.ichan_base[im] == c) {   // uniform over the workgroup
            double acc[2] = {0.0, 0.0};
            const double *ch = ra.chan + (size_t)im * CH_N;
            const double am = ch[CH_AMAX];
            if (isfinite(am) && ch[CH_STOP] == 0.0) {
                const R *I0 = ra.I + im * npix + r0;
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    const int j = leg_live(r) ? pix_of(t + r * T, L, n) : -1;
                    if (!live || j < 0) continue;
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const double d = (double)(u ? py[r] : px[r]);
                        if (d == 0.0) continue;
                        const double x = (double)I0[u * n + j] + am * d;
                        acc[0] += d * (log(x / ra.M) + 1.0);
                        acc[1] += d * d / x;
                    }
                }
            }
            block_sum<2, NF * T>(acc);
            if (threadIdx.x == 0) {
                double *rec = ra.pp + ((size_t)im * gridDim.x + blockIdx.x) * NPART;
                rec[0] = acc[0];
                rec[1] = acc[1];
            }
        }
    }
    fft_passes<LG, 0, 1, false>(v, t, s[f], tw);
    __syncthreads();
#pragma unroll
    for (int x = 0; x < 8; ++x) s[f][fpad(fft_out<LG>(t, x))] = v[x];
    __syncthreads();
    for (int e = threadIdx.x; e < Lx * NF; e += NF * T) {
        const int qc = e / NF, g = e % NF;
        const int i = rows0 + 2 * g;
        if (i >= n) continue;
        const int q = (qc - H) & (L - 1), qm = (H - qc) & (L - 1);
        const double2 z = s[g][fpad(q)], zm = s[g][fpad(qm)];
        C2<S> *o = X + ((size_t)c * Lx + qc) * n + i;
        o[0] = narrow<S>(0.5 * (z.x + zm.x), 0.5 * (z.y - zm.y));
        o[1] = narrow<S>(0.5 * (z.y + zm.y), 0.5 * (zm.x - z.x));
    }
}

// Columns: X[q][i] -> G[q][p], p = 0 .. L - 1 contiguous.  One sequence a
// workgroup: 12 us at 1024^2 in bf16x3 (17 MB written; 14 in FP32, whose grid
// is FP64), 3.4 to 3.9 at 256^2, where it is latency.
template <int LG, typename S>
__global__ __launch_bounds__(col_seqs(LG) * fft_threads(LG)) void k_tr_cols_fwd(
    const C2<S> *__restrict__ X, C2<S> *__restrict__ G, const double2 *__restrict__ tw, int n, int Lx, int Lg) {
    constexpr int L = 1 << LG, T = fft_threads(LG), NF = col_seqs(LG);
    __shared__ double2 s[NF][fpad(L)];
    const int f = threadIdx.x / T, t = threadIdx.x % T;
    const int c = blockIdx.y, qc = blockIdx.x * NF + f;
    const bool live = qc < Lx;
    const C2<S> *x = X + ((size_t)c * Lx + (live ? qc : 0)) * n;
    double2 v[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        v[r] = make_double2(0.0, 0.0);
        if (!leg_live(r)) continue;
        const int i = pix_of(t + r * T, L, n);
        const double2 y = wide(x[i < 0 ? 0 : i]);
        v[r] = i < 0 ? make_double2(0.0, 0.0) : y;
    }
    fft_passes<LG, 0, 1, false>(v, t, s[f], tw);
    if (!live) return;
    C2<S> *o = G + ((size_t)c * Lg + qc) * L;
#pragma unroll
    for (int y = 0; y < 8; ++y) o[fft_out<LG>(t, y)] = narrow<S>(v[y].x, v[y].y);
}

// ---------------------------------------------------------------- windows
// W nodes, TB nodes per bin side, TS = TB + W - 1 nodes per tile side.
template <int W> struct Win;
template <> struct Win<9> {
    static constexpr int TB = 8, TS = 16, NE = TR_NE9;
};
template <> struct Win<17> {
    static constexpr int TB = 16, TS = 32, NE = TR_NE17;
};

// Index of the wave in its workgroup; SC: uniform to the compiler, so that
// spans, items and loop bounds are scalar.
template <bool SC> __device__ __forceinline__ int wave_index() {
    const int wave = threadIdx.x >> 6;
    return SC ? __builtin_amdgcn_readfirstlane(wave) : wave;
}

// The per-wave LDS exchange: other lanes' stores are visible after it.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Window buffers of one wave, per axis, laid out for the reader: the gather
// takes four consecutive nodes of a visibility at a time (VIS: rows of
// visibilities), the spread four consecutive visibilities of a node; rows
// padded by 16 bytes so that the 16 rows a 128-bit read takes start in
// different banks.
template <int W, typename S, bool VIS> struct WinBuf {
    static constexpr int ROWS = VIS ? 32 : Win<W>::TS, LEN = (VIS ? Win<W>::TS : 32) + Tile<S>::PAD;
    S v[2][ROWS][LEN];
    static_assert(sizeof(S) * LEN % alignof(typename Tile<S>::vec4) == 0 && alignof(typename Tile<S>::vec4) <= 16,
                  "rows of the 16-byte aligned buffer are aligned for reads of four");
    __device__ __forceinline__ S &at(int axis, int vis, int node) {
        return VIS ? v[axis][vis][node] : v[axis][node][vis];
    }
};

// Window values of 32 visibilities into s (zero off the window): lane l takes
// visibility l % 32 of the batch, axis l / 32 (0: columns, 1: rows), whose
// grid coordinate is X = a L or b L.  Tap u of a visibility whose nearest node
// is at tile offset `off` sits at off + u; taps u and W - 1 - u are E +- z O,
// E and O the even and odd parts in z = 2 (X - nearest node) of the tap's
// polynomial (coefficients in poly: NE even and NE odd ones per tap pair,
// uniform over the wave).  A lane past the item's end (ok false) writes some
// finite window at offset 0; whoever uses it drops the result or multiplies
// by a zero coefficient.
template <int W, typename S, bool VIS>
__device__ __forceinline__ void windows32(WinBuf<W, S, VIS> &s, double X, bool ok, int L, int n0,
                                          const S *__restrict__ poly) {
    constexpr int H = (W - 1) / 2, NE = Win<W>::NE;
    typedef float floatv4 __attribute__((ext_vector_type(4)));
    const int lane = threadIdx.x & 63, vv = lane & 31, axis = lane >> 5;
    floatv4 *z4 = reinterpret_cast<floatv4 *>(&s);
    static_assert(sizeof(s) % (64 * 16) == 0 || sizeof(s) % 16 == 0, "whole 16-byte elements");
    constexpr int N4 = (int)(sizeof(s) / 16);
#pragma unroll
    for (int m = 0; m < (N4 + 63) / 64; ++m)
        if (N4 % 64 == 0 || lane + 64 * m < N4) z4[lane + 64 * m] = floatv4{0.f, 0.f, 0.f, 0.f};
    const double nd = rint(X);
    const S z = (S)(2.0 * (X - nd)), z2 = z * z;
    const int off = ok ? (((int)nd & (L - 1)) - n0) : 0;
    wave_sync();
    // 140 FP64 coefficients are more than the scalar registers hold: they are
    // read again for every batch (the compiler is kept from moving them out of
    // the batch loop, where it spilled them to vector lanes, 240 instructions
    // a batch to read back; 256^2 FP64 x 99,840: spread 24.8 -> 22.9 us)
    int at0 = 0;
    if constexpr (W == 17) asm volatile("" : "+s"(at0));
    poly += at0;
    S *row = &s.at(axis, vv, off);
    constexpr int ST = VIS ? 1 : WinBuf<W, S, VIS>::LEN;   // from node to node
#pragma unroll
    for (int u = 0; u <= H; ++u) {
        const S *pe = poly + u * 2 * NE, *po = pe + NE;
        S e = pe[NE - 1], o = po[NE - 1];
#pragma unroll
        for (int m = NE - 2; m >= 0; --m) {
            e = fma(e, z2, pe[m]);
            if (u < H) o = fma(o, z2, po[m]);
        }
        if (u < H) {
            row[u * ST] = fma(z, o, e);
            row[(W - 1 - u) * ST] = fma(-z, o, e);
        } else {
            row[u * ST] = e;
        }
    }
}

// x + y after exchanging 16-lane rows (SW16: odd rows of x with even rows of
// y) or half waves (upper half of x with lower half of y): row or half r of
// the result holds the sum over a pair of rows (halves) of x (r even / lower)
// or of y.
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
template <bool SW16>
__device__ __forceinline__ uintx2 swap32(unsigned x, unsigned y) {
    if constexpr (SW16) return __builtin_amdgcn_permlane16_swap(x, y, false, false);
    else return __builtin_amdgcn_permlane32_swap(x, y, false, false);
}
template <bool SW16>
__device__ __forceinline__ double swap_add(double x, double y) {
    const long long bx = __double_as_longlong(x), by = __double_as_longlong(y);
    const uintx2 lo = swap32<SW16>((unsigned)bx, (unsigned)by);
    const uintx2 hi = swap32<SW16>((unsigned)(bx >> 32), (unsigned)(by >> 32));
    return __longlong_as_double(((long long)hi.x << 32) | lo.x) + __longlong_as_double(((long long)hi.y << 32) | lo.y);
}
template <bool SW16>
__device__ __forceinline__ float swap_add(float x, float y) {
    const uintx2 v = swap32<SW16>(__float_as_uint(x), __float_as_uint(y));
    return __uint_as_float(v.x) + __uint_as_float(v.y);
}

// e with 2^(e-1) <= |x| < 2^e (the least for zero, subnormal and non-finite x).
constexpr int EXP_LEAST = -1022;
__device__ __forceinline__ int exponent(double x) {
    const int e = (int)((unsigned long long)__double_as_longlong(x) >> 52 & 2047u);
    return e == 0 || e == 2047 ? EXP_LEAST : e - 1022;
}

// What the gather does with V_k (component by component):
//   TV_OUT: out[caller's index] = V_k
//   TV_RES: R_k = V_k - Vo_k; partial [0] = sum w |R|^2
//   TV_DIR: Vd_k = V_k; partials [0] = sum w |Vd|^2, [1] = sum w Re(conj(R) Vd)
// (each workgroup's partials in record blockIdx.x of `part`).
enum { TV_OUT, TV_RES, TV_DIR };

// TV_DIR: the last workgroup of an image starts its line search from the
// totals of a and b, the row pass's entropy parts and the direction pass's.
struct DirTail {
    const int *chan_img, *gbase;
    unsigned *ctr;
    const double *pp;
    int n_rec;
    const double *chan;
    double *ls;
    double lam;
};

// Gather: a workgroup's four waves take one span of consecutive items each
// (spans are cut to equal cost at finalize); an item's grid tile is held in
// registers.  The visibilities of a span are consecutive, so the next batch's
// coordinates are loaded while the current one computes.  Bound by the issue
// of matrix (FP64 products 42 % of the cycles, FP32 34 %) and vector
// instructions (22 and 30 %) and by LDS (35 %), at three waves a SIMD, not by
// its 52 bytes a visibility.  1024^2 x 5,000,250 with the residual: FP32 158
// us (gather 216 and a residual pass of 47 apart), split 100 (FP64 tiles 160);
// 256^2 x 99,840 FP64 18.5.
template <int W, typename S, typename A, int MODE>
__global__ __launch_bounds__(64 * TR_WAVES) void k_tr_interp(
    const int2 *__restrict__ spans, const TrItem *__restrict__ items, const double *__restrict__ a,
    const double *__restrict__ b, const C2<S> *__restrict__ G, const A *__restrict__ poly, int L, int Lg,
    long long ztot, double *__restrict__ out, const double *__restrict__ ref, const float *__restrict__ w,
    const unsigned *__restrict__ perm, double *__restrict__ part, const DirTail dt) {
    constexpr int H = (W - 1) / 2, TB = Win<W>::TB, TS = Win<W>::TS, NT = TS / 16, NS = TS / 4;
    // PAIR: both halves of a batch side by side, and scalar spans and loop
    // bounds (256^2 x 64 channels, split: 219 -> 205 us; 512^2 27.3 -> 25.6).
    // Nine FP64 taps fill the scalar registers with coefficients: spilled
    // there, 1024^2 FP32 158 -> 167 us.
    constexpr bool PAIR = W == 17 || sizeof(A) == 4;
    typedef typename Tile<A>::acc acc_t;
    // an FP64 grid into FP32 products: each tile is scaled by its own power of
    // two, exactly, so that the products have the range of the grid
    constexpr bool SCALED = sizeof(S) > sizeof(A);
    __shared__ __attribute__((aligned(16))) WinBuf<W, A, true> s[TR_WAVES];
    // step x of a contraction takes the columns 16 (x / 4) + 4 g + x % 4, and
    // the tile's rows are permuted so that register r of lane group g holds
    // row 4 g + r: a lane then reads its windows four at a time
    auto ccol = [&](int x, int g) { return 16 * (x / 4) + 4 * g + x % 4; };
    const int wave = wave_index<PAIR>(), lane = threadIdx.x & 63;
    const int q = lane & 15, g = lane >> 4;
    const int2 span = spans[blockIdx.x * TR_WAVES + wave];
    const double *ab = lane < 32 ? a : b;
    double acc0 = 0.0, acc1 = 0.0;
    double xn = 0.0;
    // coordinates of the batch at k (past the end: some visibility's)
    auto fetch = [&](long long k) {
        k += lane & 31;
        xn = ab[k < ztot ? k : ztot - 1];
    };
    if (span.x < span.y) fetch(items[span.x].kbeg);
    // this lane's visibility in a batch and component of the result
    const int vl = 16 * (g >> 1) + q, comp = g & 1;
    for (int item = span.x; item < span.y; ++item) {
        const TrItem it = items[item];
        A gr[NT][NS], gi[NT][NS];
        const int qr = sizeof(A) == 8 ? 4 * (q & 3) + (q >> 2) : q;
        C2<S> raw[NT][NS];
#pragma unroll
        for (int x = 0; x < NS; ++x) {
            const C2<S> *col = G + ((size_t)it.chan * Lg + it.bx * TB + ccol(x, g)) * L;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                raw[t][x] = col[(it.by * TB - H + 16 * t + qr) & (L - 1)];
            }
        }
        // SCALED: the tile's power of two, the largest exponent in it
        int ex = 0;
        if constexpr (SCALED) {
            ex = EXP_LEAST;
#pragma unroll
            for (int x = 0; x < NS; ++x)
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    ex = max(ex, max(exponent(raw[t][x].x), exponent(raw[t][x].y)));
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) ex = max(ex, __shfl_xor(ex, o, 64));
        }
#pragma unroll
        for (int x = 0; x < NS; ++x)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                gr[t][x] = (A)(SCALED ? (S)ldexp((double)raw[t][x].x, -ex) : raw[t][x].x);
                gi[t][x] = (A)(SCALED ? (S)ldexp((double)raw[t][x].y, -ex) : raw[t][x].y);
            }
        const int n0 = TB * (lane < 32 ? it.bx : it.by);
        for (long long k0 = it.kbeg; k0 < it.kend; k0 += 32) {
            const double X = xn * (double)L;
            fetch(k0 + 32 < it.kend ? k0 + 32 : it.kend);
            const long long kv = k0 + vl;
            const bool ok = kv < it.kend;
            const long long kc = ok ? kv : it.kend - 1;
            double rv = 0.0;
            float wv = 0.f;
            unsigned pk = 0;
            if constexpr (MODE == TV_OUT) {
                pk = perm[kc];
            } else {
                rv = ref[2 * kc + comp];
                wv = w[kc];
            }
            windows32<W, A, true>(s[wave], X, k0 + (lane & 31) < it.kend, L, n0, poly);
            wave_sync();
            // the sums of N halves of 16 visibilities, side by side, from h0
            A half[2] = {A(0), A(0)};
            auto sums = [&](auto N, int h0) {
                constexpr int NHALF = decltype(N)::value;
                typedef typename Tile<A>::vec4 S4;
                acc_t ar[NHALF][NT], ai[NHALF][NT];
#pragma unroll
                for (int h = 0; h < NHALF; ++h)
#pragma unroll
                    for (int t = 0; t < NT; ++t) ar[h][t] = ai[h][t] = acc_t{A(0), A(0), A(0), A(0)};
#pragma unroll
                for (int cb = 0; cb < NS / 4; ++cb) {
                    S4 wx[NHALF];
#pragma unroll
                    for (int h = 0; h < NHALF; ++h)
                        wx[h] = *reinterpret_cast<const S4 *>(&s[wave].v[0][16 * (h0 + h) + q][4 * g + 16 * cb]);
#pragma unroll
                    for (int x = 0; x < 4; ++x)
#pragma unroll
                        for (int h = 0; h < NHALF; ++h)
#pragma unroll
                            for (int t = 0; t < NT; ++t) {
                                ar[h][t] = Tile<A>::mma(gr[t][4 * cb + x], wx[h][x], ar[h][t]);
                                ai[h][t] = Tile<A>::mma(gi[t][4 * cb + x], wx[h][x], ai[h][t]);
                            }
                }
#pragma unroll
                for (int h = 0; h < NHALF; ++h) {
                    A vr = A(0), vi = A(0);
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        const S4 wy = *reinterpret_cast<const S4 *>(&s[wave].v[1][16 * (h0 + h) + q][4 * g + 16 * t]);
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            vr = fma(wy[r], ar[h][t][r], vr);
                            vi = fma(wy[r], ai[h][t][r], vi);
                        }
                    }
                    half[h0 + h] = swap_add<true>(vr, vi);
                }
            };
            constexpr std::integral_constant<int, 1> one;
            constexpr std::integral_constant<int, 2> two;
            if constexpr (PAIR) {
                if (k0 + 16 < it.kend) sums(two, 0);
                else sums(one, 0);
            } else {
                sums(one, 0);
                if (k0 + 16 < it.kend) sums(one, 1);
            }
            // lane group g now gets component g % 2 of visibility 16 (g / 2) + q
            double v = (double)swap_add<false>(half[0], half[1]);
            if constexpr (SCALED) v = ldexp(v, ex);
            if (ok) {
                if constexpr (MODE == TV_OUT) {
                    out[2 * (size_t)(pk >> 1) + comp] = comp && (pk & 1u) ? -v : v;
                } else if constexpr (MODE == TV_RES) {
                    const double r = v - rv;
                    out[2 * kv + comp] = r;
                    acc0 += (double)wv * (r * r);
                } else {
                    out[2 * kv + comp] = v;
                    acc0 += (double)wv * (v * v);
                    acc1 += (double)wv * (rv * v);
                }
            }
            wave_sync();
        }
    }
    if constexpr (MODE != TV_OUT) {
        __shared__ double red[2][TR_WAVES];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            acc0 += __shfl_xor(acc0, o, 64);
            acc1 += __shfl_xor(acc1, o, 64);
        }
        if (lane == 0) {
            red[0][wave] = acc0;
            red[1][wave] = acc1;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
#pragma unroll
            for (int x = 0; x < 2; ++x)
                coh_store(part + (size_t)blockIdx.x * NPART + x, (red[x][0] + red[x][1]) + (red[x][2] + red[x][3]));
        }
    }
    if constexpr (MODE == TV_DIR) {
        const int im = dt.chan_img[items[spans[blockIdx.x * TR_WAVES].x].chan];
        const int v0 = dt.gbase[im], v1 = dt.gbase[im + 1];
        if (!arrive_last(dt.ctr, im, (int)blockIdx.x - v0, v1 - v0)) return;
        double ab2[2], fh[2];
        sum_partials2<2, 2>(part + (size_t)v0 * NPART, v1 - v0, 0, ab2, dt.pp + (size_t)im * dt.n_rec * NPART,
                            dt.n_rec, 0, fh);
        if (threadIdx.x == 0) {
            const double *ch = dt.chan + (size_t)im * CH_N;
            ls_init(dt.ls + (size_t)im * LSS_N, ab2[0], ab2[1], dt.lam * ch[CH_E1], dt.lam * ch[CH_E2], ch[CH_AMAX],
                    ch[CH_STOP] != 0.0, true, dt.lam * fh[0], dt.lam * fh[1]);
        }
    }
}

// Spread, the visibilities as the contraction dimension: as the gather, a
// workgroup's four waves take one span of items of equal cost each and store
// an item's tile in its slot, tiles[slot][column][row].  A bin of several
// items has workgroups of its own (waves[].z = live waves > 0), whose waves
// sum an item each and add their sums in LDS in wave order into one tile.
// DEEP (contexts with a deep bin): its waves sum several items each.  Where
// an item's sum is FP32 these are added in FP64 (sixteen registers, a wave or
// two less on a SIMD, hence a variant of its own), and the tiles, fewer but
// larger, are stored in FP64.
// Bound as the gather, its matrix share smaller (33 % in FP64).  1024^2 x
// 5,000,250: FP32 195 us (items of unequal cost in groups of four 273), split
// 116 (FP64 tiles 196); 256^2 x 99,840 FP64 22.8.
// perm (may be null): coef is in the caller's order (index << 1 | negated).
// STEP (a CG step): the coefficients are R + alpha Vd, which also replace R;
// the chi^2 partial of the workgroup goes to its record in part.
struct StepArgs {
    double2 *R;
    const double2 *Vd;
    const double *ls;
    double *part;
};
template <int W, typename S, typename A, bool STEP, bool DEEP>
__global__ __launch_bounds__(64 * TR_WAVES) void k_tr_spread(const int4 *__restrict__ waves,
                                                            const TrItem *__restrict__ items,
                                                            const double *__restrict__ a,
                                                            const double *__restrict__ b,
                                                            const double2 *__restrict__ coef,
                                                            const float *__restrict__ w,
                                                            const unsigned *__restrict__ perm,
                                                            C2<S> *__restrict__ tiles,
                                                            const A *__restrict__ poly, int L,
                                                            long long ztot, const StepArgs sa) {
    constexpr int TB = Win<W>::TB, TS = Win<W>::TS, NT = TS / 16;
    typedef typename Tile<A>::acc acc_t;
    __shared__ __attribute__((aligned(16))) WinBuf<W, A, false> s[TR_WAVES];
    __shared__ __attribute__((aligned(16))) A sc[TR_WAVES][2][32];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int q = lane & 15, g = lane >> 4;
    const int4 span = waves[blockIdx.x * TR_WAVES + wave];   // first item, end, live waves of a shared bin
    const double *ab = lane < 32 ? a : b;
    acc_t ar[NT][NT], ai[NT][NT];
    constexpr bool WIDE = DEEP && sizeof(A) == 4;
    static_assert(!WIDE || NT == 1, "one accumulator tile");
    double wr[4] = {0.0, 0.0, 0.0, 0.0}, wi[4] = {0.0, 0.0, 0.0, 0.0};
    // the next batch's data are loaded while the current one computes; the
    // visibilities of a span are consecutive, so that includes the next item's
    double xn = 0.0, chi = 0.0;
    float wn = 1.f;
    double2 cn = make_double2(0.0, 0.0), dn = cn;
    const double al = STEP ? sa.ls[(size_t)span.w * LSS_N + LSS_ALPHA] : 0.0;
    auto fetch = [&](long long k0) {
        const long long k = k0 + (lane & 31), kc = k < ztot ? k : ztot - 1;
        xn = ab[kc];
        if (w) wn = w[kc];
        if constexpr (STEP) {
            cn = sa.R[kc];
            dn = sa.Vd[kc];
        } else {
            const unsigned pk = perm ? perm[kc] : 0u;
            cn = coef[perm ? (long long)(pk >> 1) : kc];
            if (pk & 1u) cn.y = -cn.y;
        }
    };
    auto at = [&](int x, int y, int r) { return (16 * x + Tile<A>::drow(g, r)) * TS + 16 * y + q; };
    if (span.x < span.y) fetch(items[span.x].kbeg);
    for (int item = span.x; item < span.y; ++item) {
        const TrItem it = items[item];
        const int n0 = TB * (lane < 32 ? it.bx : it.by);
        // (FP64 sums of the same bin go on; a scalar branch)
        if (!DEEP || WIDE || __builtin_amdgcn_readfirstlane(span.z == 0 || item == span.x)) {
#pragma unroll
            for (int x = 0; x < NT; ++x)
#pragma unroll
                for (int y = 0; y < NT; ++y) ar[x][y] = ai[x][y] = acc_t{A(0), A(0), A(0), A(0)};
        }
        for (long long k0 = it.kbeg; k0 < it.kend; k0 += 32) {
            const bool ok = k0 + (lane & 31) < it.kend;
            if (lane < 32) {
                double2 cv = cn;
                if constexpr (STEP) {
                    cv.x += al * dn.x;
                    cv.y += al * dn.y;
                    if (ok) {
                        sa.R[k0 + lane] = cv;
                        chi += (double)wn * (cv.x * cv.x + cv.y * cv.y);
                    }
                }
                sc[wave][0][lane] = ok ? (A)(cv.x * (double)wn) : A(0);
                sc[wave][1][lane] = ok ? (A)(cv.y * (double)wn) : A(0);
            }
            windows32<W, A, false>(s[wave], xn * (double)L, ok, L, n0, poly);
            fetch(k0 + 32 < it.kend ? k0 + 32 : it.kend);
            wave_sync();
            // halves of 16 visibilities (zero coefficients past the end), the
            // contraction's step m of lane group g taking visibility 4 g + m
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (k0 + 16 * h >= it.kend) break;
                typedef typename Tile<A>::vec4 S4;
                const int v0 = 16 * h + 4 * g;
                const S4 cr = *reinterpret_cast<const S4 *>(&sc[wave][0][v0]);
                const S4 ci = *reinterpret_cast<const S4 *>(&sc[wave][1][v0]);
                S4 kx[NT], ky[NT];
#pragma unroll
                for (int y = 0; y < NT; ++y) {
                    kx[y] = *reinterpret_cast<const S4 *>(&s[wave].v[0][16 * y + q][v0]);
                    ky[y] = *reinterpret_cast<const S4 *>(&s[wave].v[1][16 * y + q][v0]);
                }
#pragma unroll
                for (int m = 0; m < 4; ++m)
#pragma unroll
                    for (int x = 0; x < NT; ++x) {
                        const A pr = kx[x][m] * cr[m], pi = kx[x][m] * ci[m];
#pragma unroll
                        for (int y = 0; y < NT; ++y) {
                            ar[x][y] = Tile<A>::mma(pr, ky[y][m], ar[x][y]);
                            ai[x][y] = Tile<A>::mma(pi, ky[y][m], ai[x][y]);
                        }
                    }
            }
            wave_sync();
        }
        if (WIDE && span.z != 0) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                wr[r] += (double)ar[0][0][r];
                wi[r] += (double)ai[0][0][r];
            }
        }
        if (span.z == 0) {
            C2<S> *o = tiles + (size_t)it.slot * (TS * TS);
#pragma unroll
            for (int x = 0; x < NT; ++x)
#pragma unroll
                for (int y = 0; y < NT; ++y)
#pragma unroll
                    for (int r = 0; r < 4; ++r) o[at(x, y, r)] = C2<S>{(S)ar[x][y][r], (S)ai[x][y][r]};
        }
    }
    if constexpr (STEP) {
        __shared__ double red[TR_WAVES];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) chi += __shfl_xor(chi, o, 64);
        if (lane == 0) red[wave] = chi;
        __syncthreads();
        if (threadIdx.x == 0) sa.part[(size_t)blockIdx.x * NPART] = (red[0] + red[1]) + (red[2] + red[3]);
    }
    if (span.z == 0) return;   // uniform over the workgroup
    // waves 1.. leave their sums in LDS, wave 0 adds them in order
    typedef typename std::conditional<WIDE, double, A>::type B;
    C2<B> *buf = reinterpret_cast<C2<B> *>(&s[0]);
    static_assert((TR_WAVES - 1) * TS * TS * sizeof(C2<B>) <= sizeof(s), "wave sums fit the window buffers");
    __syncthreads();
    if (wave > 0 && wave < span.z) {
#pragma unroll
        for (int x = 0; x < NT; ++x)
#pragma unroll
            for (int y = 0; y < NT; ++y)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    buf[(wave - 1) * TS * TS + at(x, y, r)] =
                        C2<B>{WIDE ? (B)wr[r] : (B)ar[x][y][r], WIDE ? (B)wi[r] : (B)ai[x][y][r]};
    }
    __syncthreads();
    if (wave > 0) return;
    C2<S> *o = tiles + (size_t)items[span.x].slot * (TS * TS);
#pragma unroll
    for (int x = 0; x < NT; ++x)
#pragma unroll
        for (int y = 0; y < NT; ++y)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                C2<B> t{WIDE ? (B)wr[r] : (B)ar[x][y][r], WIDE ? (B)wi[r] : (B)ai[x][y][r]};
                for (int v = 1; v < span.z; ++v) {
                    const C2<B> w = buf[(v - 1) * TS * TS + at(x, y, r)];
                    t.x += w.x;
                    t.y += w.y;
                }
                o[at(x, y, r)] = C2<S>{(S)t.x, (S)t.y};
            }
}

// Inverse columns: node (q, p) sums the tiles that cover it (at most two bin
// columns by two bin rows, each bin's slots in order), then the transform
// over p; the image rows are kept: Y[q][i].  Bound by the latency of the tile
// loads (slots, tiles, further tiles in rounds): 19 us at 1024^2 (31 with a
// tile at a time), 7.4 at 256^2, 76 for 23 channels of 512^2 (101 with FP64
// tiles).
template <int LG, int W, typename TT, typename S>
__global__ __launch_bounds__(col_seqs(LG) * fft_threads(LG)) void k_tr_cols_inv(
    const C2<TT> *__restrict__ tiles, const int2 *__restrict__ bin_slot, C2<S> *__restrict__ Y,
    const double2 *__restrict__ tw, int n, int Lx, int nbx) {
    constexpr int L = 1 << LG, T = fft_threads(LG), NF = col_seqs(LG);
    constexpr int H = (W - 1) / 2, TB = Win<W>::TB, TS = Win<W>::TS, NBY = L / TB;
    __shared__ double2 s[NF][fpad(L)];
    const int f = threadIdx.x / T, t = threadIdx.x % T;
    const int c = blockIdx.y, qc = blockIdx.x * NF + f;
    const bool live = qc < Lx;
    const int2 *bins = bin_slot + (size_t)c * nbx * NBY;
    double2 v[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) v[r] = make_double2(0.0, 0.0);
    if (live) {
        const int bxh = qc / TB;
#pragma unroll
        for (int dx = 1; dx >= 0; --dx) {
            const int bx = bxh - dx;
            if (bx < 0 || bx >= nbx) continue;
            const int co = (qc - bx * TB) * TS;
            int s0[8][2], s1[8][2];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const int pr = (t + r * T + H) & (L - 1);
                const int bh = pr / TB, bl = (bh - 1) & (NBY - 1);
                const int2 l = bins[bx * NBY + bl], h = bins[bx * NBY + bh];
                s0[r][0] = l.x;
                s1[r][0] = l.y;
                s0[r][1] = h.x;
                s1[r][1] = h.y;
            }
            // the first tile of every covering bin in one round of loads
            // (slot 0 stands in for an empty bin), further ones after them
            C2<TT> y[8][2];
#pragma unroll
            for (int r = 0; r < 8; ++r)
#pragma unroll
                for (int d = 0; d < 2; ++d) {
                    const int off = co + ((t + r * T + H) & (TB - 1)) + (d == 0 ? TB : 0);
                    const int x = s0[r][d] < s1[r][d] ? s0[r][d] : 0;
                    y[r][d] = tiles[(size_t)x * (TS * TS) + off];
                }
#pragma unroll
            for (int r = 0; r < 8; ++r)
#pragma unroll
                for (int d = 0; d < 2; ++d)
                    if (s0[r][d] < s1[r][d]) v[r] = cadd(v[r], wide(y[r][d]));
            int most = 0;
#pragma unroll
            for (int r = 0; r < 8; ++r)
#pragma unroll
                for (int d = 0; d < 2; ++d) most = max(most, s1[r][d] - s0[r][d]);
            // (a round of all sixteen at a time: one load latency a round)
            for (int k = 1; k < most; ++k) {
#pragma unroll
                for (int r = 0; r < 8; ++r)
#pragma unroll
                    for (int d = 0; d < 2; ++d) {
                        const int off = co + ((t + r * T + H) & (TB - 1)) + (d == 0 ? TB : 0);
                        const int x = s0[r][d] + k < s1[r][d] ? s0[r][d] + k : 0;
                        y[r][d] = tiles[(size_t)x * (TS * TS) + off];
                    }
#pragma unroll
                for (int r = 0; r < 8; ++r)
#pragma unroll
                    for (int d = 0; d < 2; ++d)
                        if (s0[r][d] + k < s1[r][d]) v[r] = cadd(v[r], wide(y[r][d]));
            }
        }
    }
    fft_passes<LG, 0, 1, true>(v, t, s[f], tw);
    if (!live) return;
    C2<S> *o = Y + ((size_t)c * Lx + qc) * n;
#pragma unroll
    for (int x = 0; x < 8; ++x) {
        if (!fft_live<LG>(x)) continue;
        const int i = pix_of(fft_out<LG>(t, x), L, n);
        if (i >= 0) o[i] = narrow<S>(v[x].x, v[x].y);
    }
}

// The gradient pass of an image with one channel, pixel by pixel (modes as
// k_grad with TR): the adjoint, grad Phi with the sum S, the CG's image
// update, gradient and projected gradient, or the dirty image.
template <typename R> struct RowGrad {
    const R *beam, *dir;
    R *I, *out, *gt;            // I is written by a CG step only
    int *flag;
    double *pp;
    const double *img_scale;
    const unsigned char *mask;
    double M, Mb, lam;
    int mode;
    GradTail tail;
};

// Inverse rows: the real part over the half grid of two image rows at once
// (their Hermitian halves packed as one complex sequence), times the window's
// inverse transform.  The workgroup's NF row pairs start at rows0.
template <int LG, typename S> struct RowsInv {
    static constexpr int L = 1 << LG, T = fft_threads(LG), NF = row_seqs(LG);
    static constexpr int LXM = L / 2 + 2 * TR_HMAX + 1;
    // per pair: the half spectra of two rows, then (reused) the exchange of
    // the transform
    static constexpr int NSH = 2 * LXM > fpad(L) ? 2 * LXM : fpad(L);
    static constexpr int NE = (LXM + T - 1) / T;
    C2<S> h0[NE], h1[NE];

    // The half spectra, all loads in flight together (rows past the image:
    // its first ones, never used).
    __device__ __forceinline__ void load(const C2<S> *Y, int c, int rows0, int n, int H) {
        const int Lx = L / 2 + 2 * H + 1;
#pragma unroll
        for (int m = 0; m < NE; ++m) {
            const int e = threadIdx.x + m * NF * T;
            const int qc = e / NF < Lx ? e / NF : Lx - 1, ir = rows0 + 2 * (e % NF);
            const C2<S> *y = Y + ((size_t)c * Lx + qc) * n + (ir < n ? ir : 0);
            h0[m] = y[0];
            h1[m] = y[1];
        }
    }
    // Transforms them; register x then holds the two rows' sums at position
    // fft_out(t, x).
    __device__ __forceinline__ void run(double2 (*s)[NSH], double2 (&v)[8], const double2 *tw, int H, int t) {
        const int f = threadIdx.x / T;
        const int Lx = L / 2 + 2 * H + 1;
#pragma unroll
        for (int m = 0; m < NE; ++m) {
            const int e = threadIdx.x + m * NF * T;
            if (e >= Lx * NF) continue;
            s[e % NF][2 * (e / NF)] = wide(h0[m]);
            s[e % NF][2 * (e / NF) + 1] = wide(h1[m]);
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int q = t + r * T, qm = (L - q) & (L - 1);
            auto col = [&](int x) { return x <= L / 2 + H ? x + H : x >= L - H ? x - (L - H) : -1; };
            const int cp = col(q), cm = col(qm);
            double2 z = make_double2(0.0, 0.0);
            if (cp >= 0) {
                const double2 a = s[f][2 * cp], b = s[f][2 * cp + 1];
                z.x += a.x - b.y;
                z.y += a.y + b.x;
            }
            if (cm >= 0) {
                const double2 a = s[f][2 * cm], b = s[f][2 * cm + 1];
                z.x += a.x + b.y;
                z.y += b.x - a.y;
            }
            v[r] = make_double2(0.5 * z.x, 0.5 * z.y);
        }
        fft_passes<LG, 0, 1, true>(v, t, s[f], tw);
    }
};

// Several channels of one image: workgroup (x, y) sums A_c x (its rows) over
// the y-th share of the channels (no A for the dirty image, mode 3) into plane
// y, which the gradient kernel then sums (a plane per channel cost 56 us here
// and 51 us there on 23 channels of 512^2; shares of three channels 46 and 20).
template <int LG, typename R, typename S>
__global__ __launch_bounds__(row_seqs(LG) * fft_threads(LG)) void k_tr_rows_sum(
    const C2<S> *__restrict__ Y, double *__restrict__ plane, const R *__restrict__ beam, int nchan, int mode,
    const double2 *__restrict__ tw, const double *__restrict__ dec, int n, int np, int H) {
    typedef RowsInv<LG, S> RI;
    constexpr int L = RI::L, T = RI::T, NF = RI::NF;
    __shared__ double2 s[NF][RI::NSH];
    const int f = threadIdx.x / T, t = threadIdx.x % T;
    const int rows0 = row_block<S, NF>() * NF * 2, i = rows0 + 2 * f;
    const bool live = i < n;
    const int c0 = (int)((long long)nchan * blockIdx.y / gridDim.y);
    const int c1 = (int)((long long)nchan * (blockIdx.y + 1) / gridDim.y);
    double acc[8][2];
#pragma unroll
    for (int x = 0; x < 8; ++x) acc[x][0] = acc[x][1] = 0.0;
#pragma unroll 1
    for (int c = c0; c < c1; ++c) {
        RI ri;
        ri.load(Y, c, rows0, n, H);
        R A[8][2];
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            if (!fft_live<LG>(x)) continue;
            const int j = pix_of(fft_out<LG>(t, x), L, n);
#pragma unroll
            for (int u = 0; u < 2; ++u) A[x][u] = beam[live && j >= 0 ? ((size_t)c * n + i + u) * n + j : 0];
        }
        double2 v[8];
        __syncthreads();   // the last channel's exchange has been read
        ri.run(s, v, tw, H, t);
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            if (!fft_live<LG>(x)) continue;
            acc[x][0] += mode == 3 ? v[x].x : (double)A[x][0] * v[x].x;
            acc[x][1] += mode == 3 ? v[x].y : (double)A[x][1] * v[x].y;
        }
    }
    if (!live) return;
    const double d0 = dec[i], d1 = dec[i + 1];
    double *o = plane + ((size_t)blockIdx.y * np + i) * np;
#pragma unroll
    for (int x = 0; x < 8; ++x) {
        const int j = fft_live<LG>(x) ? pix_of(fft_out<LG>(t, x), L, n) : -1;
        if (j < 0) continue;
        const double dj = dec[j];
        o[j] = acc[x][0] * (d0 * dj);
        o[np + j] = acc[x][1] * (d1 * dj);
    }
}

// One channel per image: the rows go straight through the gradient pass (14 +
// 25 us apart at 1024^2, 29 together in an evaluation, 47 at the end of a CG
// step).  A third of it is the end of the reductions: stores drained, two
// atomics and two rounds of loads across chiplets.
template <int LG, typename R, typename S>
__global__ __launch_bounds__(row_seqs(LG) * fft_threads(LG)) void k_tr_rows_inv(
    const C2<S> *__restrict__ Y, const RowGrad<R> rg, const double2 *__restrict__ tw,
    const double *__restrict__ dec, int n, int H) {
    typedef RowsInv<LG, S> RI;
    constexpr int L = RI::L, T = RI::T, NF = RI::NF;
    __shared__ double2 s[NF][RI::NSH];
    const int f = threadIdx.x / T, t = threadIdx.x % T;
    const int c = blockIdx.y, rows0 = row_block<S, NF>() * NF * 2;
    const int i = rows0 + 2 * f;
    const bool live = i < n;
    RI ri;
    ri.load(Y, c, rows0, n, H);
    // the pixels' data, loaded ahead of the transform
    R pI[8][2], pA[8][2], pd[8][2], pg[8][2];
    double lg[8][2];
    double al = 0.0;
    if (rg.mode == 2) al = rg.tail.ls[(size_t)c * LSS_N + LSS_ALPHA];
#pragma unroll
    for (int x = 0; x < 8; ++x) {
        if (!fft_live<LG>(x)) continue;
        const int j = pix_of(fft_out<LG>(t, x), L, n);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const size_t q = live && j >= 0 ? ((size_t)c * n + i + u) * n + j : 0;
            pA[x][u] = rg.beam[q];
            if (rg.mode == 1 || rg.mode == 2) pI[x][u] = rg.I[q];
            if (rg.mode == 2) {
                pd[x][u] = rg.dir[q];
                pg[x][u] = rg.gt[q];
            }
        }
    }
    // the pixels' logarithms, while the spectra are on their way and without
    // a branch between them: their long dependent chains overlap (a pixel
    // off the image: ln 1)
    if (rg.mode == 1 || rg.mode == 2) {
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            if (!fft_live<LG>(x)) continue;
            const int j = pix_of(fft_out<LG>(t, x), L, n);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const R x0 = pI[x][u];
                if (rg.mode == 2) pI[x][u] = al != 0.0 ? (R)fmax((double)x0 + al * (double)pd[x][u], rg.Mb) : x0;
                const double xi = live && j >= 0 ? (double)pI[x][u] : rg.M;
                lg[x][u] = log(xi / rg.M);
            }
        }
    }
    double2 v[8];
    ri.run(s, v, tw, H, t);
    const double d0 = live ? dec[i] : 0.0, d1 = live ? dec[i + 1] : 0.0;
    const int mode = rg.mode;
    double acc[3] = {0.0, 0.0, 0.0};
    int bad = 0;
    const double scale = mode == 3 ? rg.img_scale[c] : 1.0;
#pragma unroll
    for (int x = 0; x < 8; ++x) {
        const int j = fft_live<LG>(x) ? pix_of(fft_out<LG>(t, x), L, n) : -1;
        if (!live || j < 0) continue;
        const double dj = dec[j];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const size_t q = ((size_t)c * n + i + u) * n + j;
            const double G = u ? v[x].y * (d1 * dj) : v[x].x * (d0 * dj);
            double gv = mode == 3 ? G * scale : (double)pA[x][u] * G;
            double xi = 0.0;
            if (mode == 1 || mode == 2) {
                xi = (double)pI[x][u];
                if (mode == 2 && al != 0.0) rg.I[q] = pI[x][u];
                if (!(xi > 0.0)) bad = 1;
                else acc[mode == 1 ? 0 : 2] += xi * lg[x][u];
                gv += rg.lam * (lg[x][u] + 1.0);
                if (rg.mask && !rg.mask[q]) gv = 0.0;
            }
            const R gr = (R)gv;
            rg.out[q] = gr;
            if (mode == 2) {
                const bool act = (xi <= rg.Mb * (1.0 + BOUND_TOL)) && ((double)gr > 0.0);
                const double gnew = act ? 0.0 : (double)gr;
                const double gold = (double)pg[x][u];
                rg.gt[q] = (R)gnew;
                acc[0] += gnew * gnew;
                acc[1] += gnew * gold;
            }
        }
    }
    constexpr int NTH = NF * T;
    const int rows = gridDim.x;
    if (mode == 1 || mode == 2) {
        if (bad) atomicOr(rg.flag, 1);
        block_sum<3, NTH>(acc);
        if (threadIdx.x == 0) {
#pragma unroll
            for (int x = 0; x < 3; ++x) coh_store(rg.pp + ((size_t)c * rows + blockIdx.x) * NPART + x, acc[x]);
        }
    }
    grad_tail<NTH, true>(mode, c, blockIdx.x, rows, rg.pp, rg.lam, rg.tail);
}

// dst[caller's order] = src[bin order], conjugated where negated (dir = 0);
// the reverse for dir = 1.
__global__ void k_tr_permute(const double2 *__restrict__ src, double2 *__restrict__ dst,
                             const unsigned *__restrict__ perm, long long count, int dir) {
    long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (; k < count; k += stride) {
        const unsigned pk = perm[k];
        double2 v = dir ? src[pk >> 1] : src[k];
        if (pk & 1u) v.y = -v.y;
        dst[dir ? k : (long long)(pk >> 1)] = v;
    }
}

// ---------------------------------------------------------------- set-up
// Coordinates of raw visibility k: a in [0, 1/2], b in [-1/2, 1/2] (the sums
// have period one in both; the reduction is exact), and whether the pair was
// negated.
__device__ __forceinline__ bool reduce_ab(double u, double v, double cell, double &a, double &b) {
    // (products rounded before the reduction, as the coordinates of the direct
    // contraction are: no fused multiply-subtract)
    a = __dmul_rn(u, cell);
    b = __dmul_rn(v, cell);
    a -= rint(a);
    b -= rint(b);
    const bool neg = a < 0.0;
    if (neg) {
        a = -a;
        b = -b;
    }
    return neg;
}

// Sort keys: the bin of every visibility, channel by channel.
__global__ __launch_bounds__(NTHR) void k_tr_keys(const VisItem *__restrict__ items, const double *__restrict__ u,
                                                  const double *__restrict__ v, double cell,
                                                  unsigned *__restrict__ key, unsigned *__restrict__ val, int L,
                                                  int tb, int nbx, int nby) {
    const VisItem it = items[blockIdx.x];
    for (long long k = it.kbeg + threadIdx.x; k < it.kend; k += NTHR) {
        double a, b;
        const bool neg = reduce_ab(u[k], v[k], cell, a, b);
        const int nx = (int)rint(a * (double)L), ny = (int)rint(b * (double)L) & (L - 1);
        key[k] = ((unsigned)it.chan * nbx + nx / tb) * nby + ny / tb;
        val[k] = (unsigned)k << 1 | (neg ? 1u : 0u);
    }
}

// Stable least-significant-digit radix sort, 8 bits a pass: digit counts of
// SORT_BLK consecutive elements per block, their prefix sums (digit major),
// then every block places its elements in order (ranks within a wave by
// matching digits, waves and rounds in element order).
constexpr int SORT_BLK = 4096;

__global__ __launch_bounds__(NTHR) void k_sort_count(const unsigned *__restrict__ key, long long count, int shift,
                                                     unsigned *__restrict__ hist, int nblk) {
    __shared__ unsigned h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const long long k0 = (long long)blockIdx.x * SORT_BLK;
    for (int r = 0; r < SORT_BLK / NTHR; ++r) {
        const long long k = k0 + r * NTHR + threadIdx.x;
        if (k < count) atomicAdd(&h[(key[k] >> shift) & 255u], 1u);
    }
    __syncthreads();
    hist[(size_t)threadIdx.x * nblk + blockIdx.x] = h[threadIdx.x];
}

// Exclusive prefix sums of one digit's block counts (a workgroup per digit),
// its total into tot[digit].
__global__ __launch_bounds__(NTHR) void k_sort_scan(unsigned *__restrict__ hist, unsigned *__restrict__ tot,
                                                    int nblk) {
    __shared__ unsigned s[NTHR];
    unsigned *h = hist + (size_t)blockIdx.x * nblk;
    unsigned run = 0;
    for (int b0 = 0; b0 < nblk; b0 += NTHR) {
        const int b = b0 + threadIdx.x;
        const unsigned x = b < nblk ? h[b] : 0u;
        s[threadIdx.x] = x;
        __syncthreads();
        for (int o = 1; o < NTHR; o <<= 1) {
            const unsigned y = threadIdx.x >= (unsigned)o ? s[threadIdx.x - o] : 0u;
            __syncthreads();
            s[threadIdx.x] += y;
            __syncthreads();
        }
        if (b < nblk) h[b] = run + s[threadIdx.x] - x;
        run += s[NTHR - 1];
        __syncthreads();
    }
    if (threadIdx.x == 0) tot[blockIdx.x] = run;
}

__global__ __launch_bounds__(NTHR) void k_sort_place(const unsigned *__restrict__ key,
                                                     const unsigned *__restrict__ val, long long count, int shift,
                                                     const unsigned *__restrict__ hist,
                                                     const unsigned *__restrict__ tot, int nblk,
                                                     unsigned *__restrict__ key2, unsigned *__restrict__ val2) {
    constexpr int NW = NTHR / 64, PER = SORT_BLK / NW;
    __shared__ unsigned cnt[NW][256];   // next position of each digit, per wave
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const long long k0 = (long long)blockIdx.x * SORT_BLK + (long long)wave * PER;
    for (int x = lane; x < 256; x += 64) cnt[wave][x] = 0;
    __syncthreads();
    for (int r = 0; r < PER / 64; ++r) {
        const long long k = k0 + r * 64 + lane;
        if (k < count) atomicAdd(&cnt[wave][(key[k] >> shift) & 255u], 1u);
    }
    __syncthreads();
    {
        const int d = threadIdx.x;   // digit
        unsigned base = hist[(size_t)d * nblk + blockIdx.x];
        for (int x = 0; x < d; ++x) base += tot[x];
        for (int x = 0; x < NW; ++x) {
            const unsigned y = cnt[x][d];
            cnt[x][d] = base;
            base += y;
        }
    }
    __syncthreads();
    for (int r = 0; r < PER / 64; ++r) {
        const long long k = k0 + r * 64 + lane;
        const bool ok = k < count;
        const unsigned kk = ok ? key[k] : 0u;
        const unsigned d = (kk >> shift) & 255u;
        unsigned long long same = __ballot(ok);
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const unsigned long long bm = __ballot((d >> m) & 1u);
            same &= (d >> m) & 1u ? bm : ~bm;
        }
        const unsigned rank = __popcll(same & ((1ull << lane) - 1ull));
        unsigned at = 0;
        if (ok) at = cnt[wave][d] + rank;
        wave_sync();
        if (ok && rank == 0) cnt[wave][d] = at + (unsigned)__popcll(same);
        wave_sync();
        if (ok) {
            key2[at] = kk;
            val2[at] = val[k];
        }
    }
}

// start[t] = first position whose key is >= t, for t = 0 .. nkeys (nkeys: the
// number of bins of all channels).
__global__ __launch_bounds__(NTHR) void k_tr_bounds(const unsigned *__restrict__ key, long long count,
                                                    int *__restrict__ start, unsigned nkeys) {
    const long long k = (long long)blockIdx.x * NTHR + threadIdx.x;
    if (k > count) return;
    const unsigned lo = k == 0 ? 0u : key[k - 1] + 1u;
    const unsigned hi = k == count ? nkeys : key[k];
    for (unsigned t = lo; t <= hi; ++t) start[t] = (int)k;
}

// The sorted arrays.  A pointing's visibilities are rotated to the image
// centre: V^o e^{-2 pi i (u x0 + v y0)}, phase reduced mod 1.
__global__ __launch_bounds__(NTHR) void k_tr_gather(const VisItem *__restrict__ items, const double *__restrict__ u,
                                                    const double *__restrict__ v, const float2 *__restrict__ vis,
                                                    const float *__restrict__ w, const unsigned *__restrict__ val,
                                                    double cell, const double2 *__restrict__ centre,
                                                    double *__restrict__ a, double *__restrict__ b,
                                                    double2 *__restrict__ vo, float *__restrict__ ws,
                                                    unsigned *__restrict__ perm) {
    const VisItem it = items[blockIdx.x];
    const double2 x0 = centre[it.chan];
    for (long long d = it.kbeg + threadIdx.x; d < it.kend; d += NTHR) {
        const unsigned p = val[d];
        const long long k = p >> 1;
        double av, bv;
        reduce_ab(u[k], v[k], cell, av, bv);
        a[d] = av;
        b[d] = bv;
        ws[d] = w[k];
        perm[d] = p;
        const float2 o = vis[k];
        double re = o.x, im = o.y;
        if (x0.x != 0.0 || x0.y != 0.0) {
            const double ph = u[k] * x0.x + v[k] * x0.y;
            double sn, cs;
            sincospi(2.0 * (ph - rint(ph)), &sn, &cs);
            const double t = re * cs + im * sn;
            im = im * cs - re * sn;
            re = t;
        }
        vo[d] = make_double2(re, p & 1u ? -im : im);
    }
}

// A = exp(-4 ln2 |x - x0|^2 / fwhm^2) of one channel.
template <typename R>
__global__ void k_beam(R *__restrict__ beam, int n, double cell, double cx, double cy, double fwhm) {
    const long long npix = (long long)n * n;
    long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (; p < npix; p += stride) {
        const double x = (double)((int)(p % n) - n / 2) * cell - cx;
        const double y = (double)((int)(p / n) - n / 2) * cell - cy;
        beam[p] = (R)exp(-4.0 * 0.69314718055994530942 * (x * x + y * y) / (fwhm * fwhm));
    }
}

inline double *tr_pp(const uvmem_ctx *c, int buf) {
    return c->d_ppart + (size_t)buf * c->nimg * std::max(c->n_pb, c->n_trrec) * NPART;
}

template <int LG, typename R, typename S>
hipError_t fwd_lg(const uvmem_ctx *c, const void *I, int what, hipStream_t st) {
    const int H = c->tr_h, L = 1 << LG, Lx = L / 2 + 2 * H + 1;
    constexpr int T = fft_threads(LG), RS = row_seqs(LG), CS = col_seqs(LG);
    const dim3 gr(c->n_trrec, c->nchan), gc((Lx + CS - 1) / CS, c->nchan), br(RS * T);
    const RowArgs<R> ra{(const R *)(what == 2 ? c->d_dir : I), (const R *)I, (const R *)c->d_beam, c->d_chan_img,
                        c->d_ichan_base, c->d_chan, tr_pp(c, 1), c->M};
    C2<S> *X = (C2<S> *)c->d_trx;
    if (what == 2)
        hipLaunchKernelGGL((k_tr_rows_fwd<LG, R, S, true>), gr, br, 0, st, ra, X, c->d_trtw, c->d_trdec, c->n, H);
    else
        hipLaunchKernelGGL((k_tr_rows_fwd<LG, R, S, false>), gr, br, 0, st, ra, X, c->d_trtw, c->d_trdec, c->n, H);
    hipLaunchKernelGGL((k_tr_cols_fwd<LG, S>), gc, dim3(CS * T), 0, st, X, (C2<S> *)c->d_trg, c->d_trtw, c->n, Lx,
                       c->tr_lgc);
    return hipGetLastError();
}

template <int LG, int W, typename TT, typename S>
hipError_t inv_lg(const uvmem_ctx *c, hipStream_t st) {
    const int H = c->tr_h, L = 1 << LG, Lx = L / 2 + 2 * H + 1;
    constexpr int T = fft_threads(LG), CS = col_seqs(LG);
    hipLaunchKernelGGL((k_tr_cols_inv<LG, W, TT, S>), dim3((Lx + CS - 1) / CS, c->nchan), dim3(CS * T), 0, st,
                       (const C2<TT> *)c->d_trtile, c->d_trbin, (C2<S> *)c->d_trx, c->d_trtw, c->n, Lx, c->tr_nbx);
    return hipGetLastError();
}

template <int LG, typename R, typename S>
hipError_t rows_inv_lg(const uvmem_ctx *c, const void *I, void *out, int mode, double *user, hipStream_t st) {
    constexpr int T = fft_threads(LG), RS = row_seqs(LG);
    const dim3 br(RS * T);
    const C2<S> *Y = (const C2<S> *)c->d_trx;
    if (c->nimg == c->nchan) {
        const RowGrad<R> rg{(const R *)c->d_beam, (const R *)c->d_dir, (R *)const_cast<void *>(I), (R *)out,
                            (R *)c->d_gt, c->d_flag, tr_pp(c, 1), c->d_wscale, c->d_mask, c->M, c->Mb, c->lam, mode,
                            make_grad_tail(c, mode, user)};
        hipLaunchKernelGGL((k_tr_rows_inv<LG, R, S>), dim3(c->n_trrec, c->nchan), br, 0, st, Y, rg, c->d_trtw,
                           c->d_trdec, c->n, c->tr_h);
    } else {
        hipLaunchKernelGGL((k_tr_rows_sum<LG, R, S>), dim3(c->n_trrec, c->n_trplane), br, 0, st, Y,
                           (double *)c->d_gpart, (const R *)c->d_beam, c->nchan, mode, c->d_trtw, c->d_trdec, c->n,
                           c->np, c->tr_h);
    }
    return hipGetLastError();
}

// f(std::integral_constant<int, lg>()) for the context's transform length.
template <typename F>
hipError_t with_lg(const uvmem_ctx *c, F f) {
    switch (c->tr_lg) {
    case 6: return f(std::integral_constant<int, 6>());
    case 7: return f(std::integral_constant<int, 7>());
    case 8: return f(std::integral_constant<int, 8>());
    case 9: return f(std::integral_constant<int, 9>());
    case 10: return f(std::integral_constant<int, 10>());
    case 11: return f(std::integral_constant<int, 11>());
    case 12: return f(std::integral_constant<int, 12>());
    }
    return hipErrorInvalidValue;
}

template <int W, typename S, typename A, int MODE>
void interp_mode(const uvmem_ctx *c, double2 *out, const double2 *ref, hipStream_t st) {
    hipLaunchKernelGGL((k_tr_interp<W, S, A, MODE>), dim3(c->n_trgroup), dim3(64 * TR_WAVES), 0, st, c->d_trspan,
                       c->d_tritem, c->d_a, c->d_b, (const C2<S> *)c->d_trg, (const A *)c->d_trpoly, 1 << c->tr_lg,
                       c->tr_lgc, (long long)c->ztot, (double *)out, (const double *)ref, c->d_w, c->d_trperm,
                       c->d_trpart,
                       DirTail{c->d_chan_img, c->d_trgbase, c->d_ctr + (size_t)CTR_VIS * c->nimg * CTR_STRIDE, tr_pp(c, 1),
                               c->n_trrec, c->d_chan, c->d_ls, c->lam});
}
template <int W, typename S, typename A>
hipError_t interp_w(const uvmem_ctx *c, int what, double2 *out, hipStream_t st) {
    if (what == 0) interp_mode<W, S, A, TV_OUT>(c, out, nullptr, st);
    else if (what == 1) interp_mode<W, S, A, TV_RES>(c, c->d_R, c->d_vo, st);
    else interp_mode<W, S, A, TV_DIR>(c, c->d_Vd, c->d_R, st);
    return hipGetLastError();
}

template <int W, typename S, typename A, bool STEP, bool DEEP>
void spread_w(const uvmem_ctx *c, const double2 *coef, const float *w, const unsigned *perm, hipStream_t st) {
    hipLaunchKernelGGL((k_tr_spread<W, S, A, STEP, DEEP>), dim3(c->n_trspread), dim3(64 * TR_WAVES), 0, st, c->d_trspread,
                       c->d_tritem, c->d_a, c->d_b, coef, w, perm, (C2<S> *)c->d_trtile, (const A *)c->d_trpoly,
                       1 << c->tr_lg, (long long)c->ztot, StepArgs{c->d_R, c->d_Vd, c->d_ls, c->d_trpart});
}

// f(image type, S forward, S adjoint, A, width) of the context's precision.
template <int W> using width = std::integral_constant<int, W>;
template <typename F>
hipError_t with_prec(const uvmem_ctx *c, F f) {
    if (c->prec == UVMEM_FP64) return f(double(), double(), double(), double(), width<17>());
    if (c->prec == UVMEM_FP32) return f(float(), double(), float(), double(), width<9>());
    if (c->prec == UVMEM_FP16X3) return f(float(), double(), float(), float(), width<9>());
    return f(float(), float(), float(), float(), width<9>());
}

}  // namespace

hipError_t launch_tr_forward(const uvmem_ctx *c, const void *I, int what, double2 *out, hipStream_t st) {
    return with_prec(c, [&](auto r, auto s, auto, auto a, auto w) {
        typedef decltype(r) R;
        typedef decltype(s) S;
        const hipError_t e =
            with_lg(c, [&](auto lg) { return fwd_lg<decltype(lg)::value, R, S>(c, I, what, st); });
        return e != hipSuccess ? e : interp_w<decltype(w)::value, S, decltype(a)>(c, what, out, st);
    });
}

hipError_t launch_tr_adjoint(const uvmem_ctx *c, const double2 *coef, const float *w, const unsigned *perm,
                             int step, hipStream_t st) {
    return with_prec(c, [&](auto, auto, auto s, auto a, auto ww) {
        typedef decltype(s) S;
        typedef decltype(a) A;
        constexpr int W = decltype(ww)::value;
        auto run = [&](auto deep) {
            constexpr bool DEEP = decltype(deep)::value;
            typedef typename std::conditional<DEEP, double, S>::type TT;   // of the tiles
            if (step) spread_w<W, TT, A, true, DEEP>(c, coef, w, perm, st);
            else spread_w<W, TT, A, false, DEEP>(c, coef, w, perm, st);
            return with_lg(c, [&](auto lg) { return inv_lg<decltype(lg)::value, W, TT, S>(c, st); });
        };
        return c->tr_deep ? run(std::true_type()) : run(std::false_type());
    });
}

hipError_t launch_tr_rows_inv(const uvmem_ctx *c, const void *I, void *out, int mode, double *user_scal,
                              hipStream_t st) {
    return with_prec(c, [&](auto r, auto, auto s, auto, auto) {
        return with_lg(c, [&](auto lg) {
            return rows_inv_lg<decltype(lg)::value, decltype(r), decltype(s)>(c, I, out, mode, user_scal, st);
        });
    });
}

hipError_t launch_beam(const uvmem_ctx *c, int chan) {
    const size_t npix = (size_t)c->n * c->n;
    const dim3 grid((unsigned)std::min<size_t>((npix + NTHR - 1) / NTHR, 4096)), blk(NTHR);
    if (c->prec == UVMEM_FP64)
        hipLaunchKernelGGL(k_beam<double>, grid, blk, 0, nullptr, (double *)c->d_beam + chan * npix, c->n, c->cell,
                           c->cx[chan], c->cy[chan], c->fwhm[chan]);
    else
        hipLaunchKernelGGL(k_beam<float>, grid, blk, 0, nullptr, (float *)c->d_beam + chan * npix, c->n, c->cell,
                           c->cx[chan], c->cy[chan], c->fwhm[chan]);
    return hipGetLastError();
}

hipError_t launch_tr_sort(const uvmem_ctx *c, const double *u, const double *v, const float *vis, const float *w,
                          std::vector<int> &start) {
    const long long count = c->ztot;
    const int L = 1 << c->tr_lg, nblk = (int)((count + SORT_BLK - 1) / SORT_BLK);
    const unsigned nkeys = (unsigned)c->nchan * c->tr_nbx * c->tr_nby;
    unsigned *key = (unsigned *)c->d_Vd, *val = key + count, *key2 = val + count, *val2 = key2 + count;
    // one scratch allocation: pointing centres, digit counts, bin starts
    char *scratch = nullptr;
    std::vector<double2> hc(c->nchan);
    for (int ch = 0; ch < c->nchan; ++ch) hc[ch] = make_double2(c->cx[ch], c->cy[ch]);
    const size_t cbytes = hc.size() * sizeof(double2), hcount = ((size_t)nblk + 1) * 256;
    start.resize((size_t)nkeys + 1);
    hipError_t e = hipMalloc((void **)&scratch, cbytes + (hcount + start.size()) * sizeof(int));
    double2 *centre = (double2 *)scratch;
    unsigned *hist = (unsigned *)(scratch + cbytes);
    int *dstart = (int *)(hist + hcount);
    if (e == hipSuccess) e = hipMemcpy(centre, hc.data(), cbytes, hipMemcpyHostToDevice);
    if (e == hipSuccess) {
        unsigned *tot = hist + (size_t)nblk * 256;
        hipLaunchKernelGGL(k_tr_keys, dim3(c->n_visit), dim3(NTHR), 0, nullptr, c->d_vis, u, v, c->cell, key, val, L,
                           c->tr_w - 1, c->tr_nbx, c->tr_nby);
        for (int shift = 0; shift < 32 && (nkeys - 1) >> shift; shift += 8) {
            hipLaunchKernelGGL(k_sort_count, dim3(nblk), dim3(NTHR), 0, nullptr, key, count, shift, hist, nblk);
            hipLaunchKernelGGL(k_sort_scan, dim3(256), dim3(NTHR), 0, nullptr, hist, tot, nblk);
            hipLaunchKernelGGL(k_sort_place, dim3(nblk), dim3(NTHR), 0, nullptr, key, val, count, shift, hist, tot,
                               nblk, key2, val2);
            std::swap(key, key2);
            std::swap(val, val2);
        }
        hipLaunchKernelGGL(k_tr_bounds, dim3((unsigned)(count / NTHR + 1)), dim3(NTHR), 0, nullptr, key, count,
                           dstart, nkeys);
        hipLaunchKernelGGL(k_tr_gather, dim3(c->n_visit), dim3(NTHR), 0, nullptr, c->d_vis, u, v,
                           (const float2 *)vis, w, val, c->cell, centre, c->d_a, c->d_b, c->d_vo, c->d_w,
                           c->d_trperm);
        e = hipGetLastError();
        // (waits for the kernels)
        const hipError_t e2 = hipMemcpy(start.data(), dstart, start.size() * sizeof(int), hipMemcpyDeviceToHost);
        if (e == hipSuccess) e = e2;
    }
    if (scratch) (void)hipFree(scratch);
    return e;
}

hipError_t launch_tr_permute(const uvmem_ctx *c, const double2 *src, double2 *dst, int to_bins, hipStream_t st) {
    if (c->ztot == 0) return hipSuccess;
    const int blocks = (int)std::min<long long>((c->ztot + NTHR - 1) / NTHR, 4096);
    hipLaunchKernelGGL(k_tr_permute, dim3(blocks), dim3(NTHR), 0, st, src, dst, c->d_trperm, (long long)c->ztot,
                       to_bins);
    return hipGetLastError();
}

}  // namespace uvm
