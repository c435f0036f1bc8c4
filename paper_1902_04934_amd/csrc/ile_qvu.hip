// Q, U, V of Eq. (8) from frequency-domain series: the band-limited,
// noise-weighted inner products of Eq. (2) as sums over the n-point FFT grid
// f_i = i df (i < n/2), (i - n) df (i >= n/2).
//
//   k_fd_g        g_k,i = 2 df / S_k,i d_k,i exp(2 pi i f_i t0), the part of
//                 the products that the modes share (0 outside
//                 f_min < |f_i| < f_max), and the transforms' tables
//   k_fd_first,   the inverse FFT of the products conj(h_lm,i) g_k,i,
//   k_fd_second   Q_k,lm[s] = sum_i conj(h_lm,i) g_k,i exp(2 pi i i s / n), Q at
//                 t0 + s / (n df): one row in LDS (n <= 1024), or for larger
//                 n = N1 N2 the four-step form, N1 transforms of length N2
//                 over strided columns (of the products, formed as they are
//                 read), a twiddle, N2 transforms of length N1; each transform
//                 self-sorting radix-8 passes in LDS.  Beside them
//                 U_k[a][b] = sum_i w_k,i conj(h_a,i) h_b,i and
//                 V_k[a][b] = sum_i w_k,i h_a,-i h_b,i (w = 2 df / S in the
//                 band): all (a, b) over a run of bins from one read of h, then
//                 the runs added in order
//
// All of it is bound by latency and by passes over memory that the caches
// serve, not by HBM (23 MB at 3 x 21 rows of 16384 bins, 4.5 us at the rate of
// a large copy): so the products are not written and read back, a transform
// takes three LDS passes where radix 2 took seven, U and V read h once a run
// instead of once a pair (a gigabyte through L2), and the two halves share
// their launches.  At that size: 12.7 (products) + 17.3 + 13.8 (transforms) +
// 42.4 us (U, V) before, 3.1 + 24.8 + 14.6 us now; as launches of their own the
// last two are 16.8 + 11.2 and 20.9 + 7.6.  The blocking call: 112.8 -> 54.2 us.
#include "ile_internal.h"

#include <math.h>

#include <algorithm>

namespace {

constexpr int FD_T = 256;

__device__ inline double fd_freq(int64_t i, int64_t n, double df)
{
    return (double)(i < n / 2 ? i : i - n) * df;
}

// 2 df / S in the open band, else 0; sets bad for a bad spectrum there
__device__ inline double fd_weight(double f, double S, double df, double f_min, double f_max,
                                   bool &bad)
{
    const double af = fabs(f);
    if (!(af > f_min && af < f_max)) return 0.0;
    if (!(S > 0.0) || !isfinite(S)) {
        bad = true;
        return 0.0;
    }
    return 2.0 * df / S;
}

// exp(2 pi i j / n), by quadrant-exact arithmetic
__device__ inline double2 root(int64_t j, int64_t n)
{
    double sn, cs;
    sincospi(2.0 * (double)j / (double)n, &sn, &cs);
    return make_double2(cs, sn);
}

// Also the transforms' tables, once instead of in every workgroup: tab holds
// exp(2 pi i j / N2) and exp(2 pi i j / n) for j < N2, then exp(2 pi i j / N1)
// for j < N1 (N1 = 1 when a row is one transform, N2 = n).
__global__ __launch_bounds__(FD_T) void k_fd_g(const double2 *__restrict__ d,
                                               const double *__restrict__ psd, int64_t n,
                                               double df, double f_min, double f_max, double t0,
                                               int n_det, int N1, int N2,
                                               double2 *__restrict__ tab,
                                               double2 *__restrict__ g, int32_t *err)
{
    const int64_t i = (int64_t)blockIdx.x * FD_T + threadIdx.x;
    const int k = blockIdx.y;
    if (k == n_det) {
        if (i < N2) tab[i] = root(i, N2);
        else if (i < 2 * N2) tab[i] = root(i - N2, n);
        else if (i < 2 * N2 + N1) tab[i] = root(i - 2 * N2, N1);
        return;
    }
    if (i >= n) return;
    const double f = fd_freq(i, n, df);
    bool bad = false;
    const double w = fd_weight(f, psd[(int64_t)k * n + i], df, f_min, f_max, bad);
    const double2 dk = d[(int64_t)k * n + i];
    bad |= !isfinite(dk.x) || !isfinite(dk.y);
    double sn, cs;
    sincospi(2.0 * f * t0, &sn, &cs);
    g[(int64_t)k * n + i] = make_double2(w * (dk.x * cs - dk.y * sn), w * (dk.x * sn + dk.y * cs));
    if (bad) atomicOr(err, 1);
}

// conj(h) g; bad for a non-finite h
__device__ inline double2 fd_product(double2 h, double2 g, bool &bad)
{
    bad |= !isfinite(h.x) || !isfinite(h.y);
    return make_double2(h.x * g.x + h.y * g.y, h.x * g.y - h.y * g.x);
}

__device__ inline double2 cmul(double2 a, double2 b)
{
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ inline double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ inline double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ inline double2 muli(double2 a) { return make_double2(-a.y, a.x); }   // i a

// In-place inverse DFTs (exp(+2 pi i jk/R)) of R values
__device__ inline void dft(double2 (&v)[2])
{
    const double2 a = v[0];
    v[0] = cadd(a, v[1]);
    v[1] = csub(a, v[1]);
}
__device__ inline void dft(double2 (&v)[4])
{
    const double2 a = cadd(v[0], v[2]), b = csub(v[0], v[2]);
    const double2 c = cadd(v[1], v[3]), d = muli(csub(v[1], v[3]));
    v[0] = cadd(a, c);
    v[1] = cadd(b, d);
    v[2] = csub(a, c);
    v[3] = csub(b, d);
}
__device__ inline void dft(double2 (&v)[8])
{
    double2 e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    dft(e);
    dft(o);
    const double s = 0.70710678118654752440;
    o[1] = make_double2(s * (o[1].x - o[1].y), s * (o[1].x + o[1].y));     // exp(i pi/4)
    o[2] = muli(o[2]);
    o[3] = make_double2(-s * (o[3].x + o[3].y), s * (o[3].x - o[3].y));    // exp(3 i pi/4)
#pragma unroll
    for (int k = 0; k < 4; k++) {
        v[k] = cadd(e[k], o[k]);
        v[k + 4] = csub(e[k], o[k]);
    }
}

// A workgroup's sequences live in one LDS buffer of at most FFT_PTS values, a
// slot left free after every eight, so that the strided stores of a pass
// fall in different banks.
constexpr int FFT_PTS = 8 * FD_T;
__host__ __device__ inline int fft_pad(int i) { return i + (i >> 3); }

// One self-sorting pass of radix R over nb sequences of length 2^lg (sub-length
// len = 2^lg / st): t = p st + q reads x[q + st (p + c len/R)], and element k
// of its DFT times exp(2 pi i p k / len) goes to [q + st (R p + k)].  In place:
// every thread holds its 8 values between the reads and the writes.
template <int R>
__device__ inline void fft_pass(double2 *s, const double2 *tw, int nb, int lg, int lgst)
{
    constexpr int LR = R == 8 ? 3 : R == 4 ? 2 : 1, NJ = 8 / R;
    const int lgh = lg - LR, lgm = lg - lgst - LR, LS = fft_pad(1 << lg), st = 1 << lgst;
    double2 v[NJ][R];
#pragma unroll
    for (int j = 0; j < NJ; j++) {
        const int t = threadIdx.x + FD_T * j, sq = t >> lgh, w = t & ((1 << lgh) - 1);
        const int p = w >> lgst, q = w & (st - 1);
        if (sq >= nb) continue;
        const double2 *x = s + sq * LS;
#pragma unroll
        for (int c = 0; c < R; c++) v[j][c] = x[fft_pad(q + ((p + (c << lgm)) << lgst))];
        dft(v[j]);
#pragma unroll
        for (int k = 1; k < R; k++) v[j][k] = cmul(v[j][k], tw[(p * k) << lgst]);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NJ; j++) {
        const int t = threadIdx.x + FD_T * j, sq = t >> lgh, w = t & ((1 << lgh) - 1);
        const int p = w >> lgst, q = w & (st - 1);
        if (sq >= nb) continue;
        double2 *x = s + sq * LS;
#pragma unroll
        for (int k = 0; k < R; k++) x[fft_pad(q + ((R * p + k) << lgst))] = v[j][k];
    }
    __syncthreads();
}

// Inverse DFT (unnormalized, exp(+2 pi i jk/L)) of nb sequences of length L =
// 2^lg, nb L <= FFT_PTS.  Every thread of the block must call it; the values
// and the table are in place, a barrier behind them.
__device__ inline void lds_ifft(double2 *s, const double2 *tw, int nb, int lg)
{
    for (int lgst = 0; lgst < lg;) {
        const int left = lg - lgst;
        if (left >= 3) {
            fft_pass<8>(s, tw, nb, lg, lgst);
            lgst += 3;
        } else if (left == 2) {
            fft_pass<4>(s, tw, nb, lg, lgst);
            lgst += 2;
        } else {
            fft_pass<2>(s, tw, nb, lg, lgst);
            lgst += 1;
        }
    }
}

// one workgroup per row (k, a), the whole row in LDS (n = 2^lg <= 1024)
__device__ __forceinline__ void fft_row_block(int row, const double2 *__restrict__ h,
                                              const double2 *__restrict__ g,
                                              const double2 *__restrict__ tab, int lg, int n_lm,
                                              double2 *__restrict__ y, int32_t *err)
{
    extern __shared__ double2 sh[];
    const int n = 1 << lg, k = row / n_lm, a = row % n_lm;
    double2 *tw = sh + fft_pad(n) + 1;
    bool bad = false;
    for (int e = threadIdx.x; e < n; e += FD_T)
        sh[fft_pad(e)] = fd_product(h[(int64_t)a * n + e], g[(int64_t)k * n + e], bad);
    for (int j = threadIdx.x; j < n; j += FD_T) tw[j] = tab[j];
    if (bad) atomicOr(err, 1);
    __syncthreads();
    lds_ifft(sh, tw, 1, lg);
    for (int e = threadIdx.x; e < n; e += FD_T) y[(int64_t)row * n + e] = sh[fft_pad(e)];
}

// Four-step, first half: columns i1 in [c0, c0 + 2^lgB) of the N1 x N2 view
// x[i1 + N1 i2] of the row's products; transform over i2, twiddle
// exp(2 pi i i1 s2 / n), store t[s2 N1 + i1] (2^lgB consecutive i1:
// contiguous).  The twiddle of m = i1 s2 is the product of two tables' entries,
// exp(2 pi i (m mod N2) / n) and the transform's own exp(2 pi i (m / N2) N2 / n)
// = tw of length N1.
__device__ __forceinline__ void fft_a_block(int bx, int row, const double2 *__restrict__ h,
                                            const double2 *__restrict__ g,
                                            const double2 *__restrict__ tab,
                                            double2 *__restrict__ t, int lg1, int lg2, int lgB,
                                            int n_lm, int32_t *err)
{
    extern __shared__ double2 sh[];
    const int N2 = 1 << lg2, B = 1 << lgB, LS = fft_pad(N2);
    const int64_t n = (int64_t)1 << (lg1 + lg2);
    double2 *tw = sh + B * LS, *tf = tw + N2, *tc = lg1 == lg2 ? tw : tf + N2;
    const int k = row / n_lm, a = row % n_lm, c0 = bx * B;
    bool bad = false;
    for (int e = threadIdx.x; e < B * N2; e += FD_T) {
        const int b = e & (B - 1), i2 = e >> lgB;
        const int64_t i = c0 + b + ((int64_t)i2 << lg1);
        sh[b * LS + fft_pad(i2)] = fd_product(h[a * n + i], g[k * n + i], bad);
    }
    for (int j = threadIdx.x; j < 2 * N2; j += FD_T) tw[j] = tab[j];
    if (lg1 != lg2)
        for (int j = threadIdx.x; j < 1 << lg1; j += FD_T) tc[j] = tab[2 * N2 + j];
    if (bad) atomicOr(err, 1);
    __syncthreads();
    lds_ifft(sh, tw, B, lg2);
    for (int e = threadIdx.x; e < B * N2; e += FD_T) {
        const int b = e & (B - 1), s2 = e >> lgB;
        const int m = (c0 + b) * s2;   // < n
        const double2 z = cmul(sh[b * LS + fft_pad(s2)], cmul(tc[m >> lg2], tf[m & (N2 - 1)]));
        t[row * n + ((int64_t)s2 << lg1) + c0 + b] = z;
    }
}

// Four-step, second half: rows s2 in [d0, d0 + 2^lgB) of t (contiguous over
// i1); transform over i1 and store y[s2 + N2 s1].
__device__ __forceinline__ void fft_c_block(int bx, int rw, const double2 *__restrict__ t,
                                            const double2 *__restrict__ tab,
                                            double2 *__restrict__ y, int lg1, int lg2, int lgB)
{
    extern __shared__ double2 sh[];
    const int N1 = 1 << lg1, B = 1 << lgB, LS = fft_pad(N1);
    const int64_t row = (int64_t)rw << (lg1 + lg2);
    double2 *tw = sh + B * LS;
    const int d0 = bx * B;
    for (int e = threadIdx.x; e < B * N1; e += FD_T) {
        const int i1 = e & (N1 - 1), b = e >> lg1;
        sh[b * LS + fft_pad(i1)] = t[row + ((int64_t)(d0 + b) << lg1) + i1];
    }
    for (int j = threadIdx.x; j < N1; j += FD_T) tw[j] = tab[(2 << lg2) + j];
    __syncthreads();
    lds_ifft(sh, tw, B, lg1);
    for (int e = threadIdx.x; e < B * N1; e += FD_T) {
        const int b = e & (B - 1), s1 = e >> lgB;
        y[row + d0 + b + ((int64_t)s1 << lg2)] = sh[b * LS + fft_pad(s1)];
    }
}

// U, V over the bins [i0, i0 + per) of detector k: a thread keeps the sums of
// 2 x 2 pairs (a, b) in registers, G groups of threads share the bins of each
// staged block of ub, and the groups' sums are added in group order.  part
// [run][a][b][4] (Re U, Im U, Re V, Im V) and used[run] = 1, or used = 0 when
// no bin of the run is in the band.
constexpr int UV_B = 64;   // most bins staged at once
__device__ __forceinline__ void uv_part_block(int run, int runs, const double2 *__restrict__ h,
                                              const double *__restrict__ psd, int64_t n, int n_lm,
                                              int per, int ub, double df, double f_min,
                                              double f_max, double *__restrict__ part,
                                              int32_t *__restrict__ used)
{
    extern __shared__ double2 sh[];
    __shared__ double s_w[UV_B];
    const int k = run / runs;
    const int n2 = (n_lm + 1) / 2, np = 2 * n2, G = min(FD_T / (n2 * n2), 8);
    // [bin][mode] (n_lm padded to even): h, h at -f
    double2 *sx = sh, *sz = sx + ub * np;
    const int grp = threadIdx.x / (n2 * n2), u = threadIdx.x % (n2 * n2);
    const int a0 = 2 * (u / n2), b0 = 2 * (u % n2);
    double acc[2][2][4] = {};
    int any_run = 0;
    for (int s0 = 0; s0 < per; s0 += ub) {
        const int64_t i0 = (int64_t)(run - k * runs) * per + s0;
        // the band is known before its spectrum arrives: a block outside it
        // reads nothing
        int any = 0;
        double w = 0.0;
        if (threadIdx.x < ub && i0 + threadIdx.x < n) {
            bool bad = false;
            const int64_t i = i0 + threadIdx.x;
            const double f = fabs(fd_freq(i, n, df));
            any = f > f_min && f < f_max;
            if (any) w = fd_weight(f, psd[k * n + i], df, f_min, f_max, bad);
        }
        if (!__syncthreads_or(any)) continue;
        any_run = 1;
        if (threadIdx.x < ub) s_w[threadIdx.x] = w;
        for (int e = threadIdx.x; e < ub * np; e += FD_T) {
            const int c = e & (ub - 1), a = e / ub;
            const int64_t i = i0 + c;
            const bool in = a < n_lm && i < n;
            const int64_t ia = in ? a * n : 0, ii = in ? i : 0;
            double2 x = h[ia + ii], z = h[ia + (ii == 0 ? 0 : n - ii)];
            if (!in) x = z = make_double2(0.0, 0.0);
            sx[c * np + a] = x;
            sz[c * np + a] = z;
        }
        __syncthreads();
        if (grp < G)
            for (int c = grp; c < ub; c += G) {
                const double wc = s_w[c];
                if (wc == 0.0) continue;
                double2 x[2], z[2], y[2];
#pragma unroll
                for (int q = 0; q < 2; q++) {
                    x[q] = sx[c * np + a0 + q];
                    z[q] = sz[c * np + a0 + q];
                    y[q] = sx[c * np + b0 + q];
                    y[q] = make_double2(wc * y[q].x, wc * y[q].y);
                }
#pragma unroll
                for (int p = 0; p < 2; p++)
#pragma unroll
                    for (int q = 0; q < 2; q++) {
                        double *s = acc[p][q];
                        s[0] = fma(x[p].x, y[q].x, fma(x[p].y, y[q].y, s[0]));    // conj(x) y
                        s[1] = fma(x[p].x, y[q].y, fma(-x[p].y, y[q].x, s[1]));
                        s[2] = fma(z[p].x, y[q].x, fma(-z[p].y, y[q].y, s[2]));   // z y
                        s[3] = fma(z[p].x, y[q].y, fma(z[p].y, y[q].x, s[3]));
                    }
            }
        __syncthreads();
    }
    if (threadIdx.x == 0) used[run] = any_run;
    if (!any_run) return;
    // groups in order through LDS (the staging area: [np][np][4] doubles)
    double *red = reinterpret_cast<double *>(sh);
    for (int q = 0; q < G; q++) {
        if (grp == q)
#pragma unroll
            for (int p = 0; p < 2; p++)
#pragma unroll
                for (int r = 0; r < 2; r++)
#pragma unroll
                    for (int c = 0; c < 4; c++) {
                        double *s = red + ((a0 + p) * np + b0 + r) * 4 + c;
                        *s = q == 0 ? acc[p][r][c] : *s + acc[p][r][c];
                    }
        __syncthreads();
    }
    for (int e = threadIdx.x; e < n_lm * n_lm * 4; e += FD_T) {
        const int c = e & 3, ab = e >> 2, a = ab / n_lm, b = ab % n_lm;
        part[(int64_t)run * n_lm * n_lm * 4 + e] = red[(a * np + b) * 4 + c];
    }
}

// the runs of each detector in order, sixteen interleaved sums an entry (the
// reads are independent: a run not in the band holds whatever was there, and is
// not added)
constexpr int UV_S = 16;
__device__ __forceinline__ void uv_sum_block(int bx, int k, const double *__restrict__ part,
                                             const int32_t *__restrict__ used, int runs, int n_lm,
                                             double *__restrict__ U, double *__restrict__ V)
{
    constexpr int NS = UV_S, NE = FD_T / NS;
    __shared__ double red[NS][NE];
    const int le = threadIdx.x % NE, s = threadIdx.x / NE;
    const int ne = n_lm * n_lm * 4, e = bx * NE + le;
    double v = 0.0;
    if (e < ne) {
        const double *pk = part + (int64_t)k * runs * ne + e;
#pragma unroll 16
        for (int r = s; r < runs; r += NS) {
            const double x = pk[(int64_t)r * ne];
            v += used[k * runs + r] ? x : 0.0;
        }
    }
    red[s][le] = v;
    __syncthreads();
    if (s != 0 || e >= ne) return;
    for (int q = 1; q < NS; q++) v += red[q][le];
    const int c = e & 3;
    const int64_t o = 2 * ((int64_t)k * n_lm * n_lm + (e >> 2)) + (c & 1);
    (c < 2 ? U : V)[o] = v;
}

// What one launch needs of both halves of the work.
struct fd_args {
    const double2 *h, *g, *tab;
    const double *psd;
    double2 *t, *Q;
    double *part, *U, *V;
    int32_t *used, *err, *err_host;
    int64_t n;
    int n_det, n_lm, lg1, lg2, lgA, lgC;
    int runs, per, ub;
    double df, f_min, f_max;
};

// The transforms and the U, V sums do not depend on each other and neither
// fills the chip for long: one launch holds the workgroups of the sums over the
// runs and those of the first half of the transforms (ROW: of the whole rows),
// the next those of the second half and of the runs' sums.
template <bool ROW> __global__ __launch_bounds__(FD_T) void k_fd_first(fd_args A)
{
    const int nuv = A.runs * A.n_det;
    if ((int)blockIdx.x < nuv) {
        uv_part_block(blockIdx.x, A.runs, A.h, A.psd, A.n, A.n_lm, A.per, A.ub, A.df, A.f_min,
                      A.f_max, A.part, A.used);
        return;
    }
    const int b = blockIdx.x - nuv;
    if (ROW) {
        fft_row_block(b, A.h, A.g, A.tab, A.lg2, A.n_lm, A.Q, A.err);
    } else {
        const int lgx = A.lg1 - A.lgA;
        fft_a_block(b & ((1 << lgx) - 1), b >> lgx, A.h, A.g, A.tab, A.t, A.lg1, A.lg2, A.lgA,
                    A.n_lm, A.err);
    }
}

template <bool ROW> __global__ __launch_bounds__(FD_T) void k_fd_second(fd_args A)
{
    const int bk = (A.n_lm * A.n_lm * 4 + FD_T / UV_S - 1) / (FD_T / UV_S), nuv = bk * A.n_det;
    if ((int)blockIdx.x < nuv) {
        if (blockIdx.x == 0 && threadIdx.x == 0) *A.err_host = *A.err;
        uv_sum_block(blockIdx.x % bk, blockIdx.x / bk, A.part, A.used, A.runs, A.n_lm, A.U, A.V);
        return;
    }
    if (!ROW) {
        const int b = blockIdx.x - nuv, lgx = A.lg2 - A.lgC;
        fft_c_block(b & ((1 << lgx) - 1), b >> lgx, A.t, A.tab, A.Q, A.lg1, A.lg2, A.lgC);
    }
}

inline int log2i(int64_t n)
{
    int lg = 0;
    while (((int64_t)1 << lg) < n) lg++;
    return lg;
}

// Bins of a staged block (two arrays of them within 48 KB of LDS) and of a run:
// at most 256 runs a detector, each a whole number of blocks.
inline int uv_block(int n_lm) { return n_lm <= 24 ? UV_B : UV_B / 2; }
inline int uv_per(int64_t n, int n_lm)
{
    const int ub = uv_block(n_lm);
    const int64_t per = (n + 255) / 256;
    return (int)(std::max<int64_t>(1, (per + ub - 1) / ub) * ub);
}
inline int uv_runs(int64_t n, int n_lm) { return (int)((n + uv_per(n, n_lm) - 1) / uv_per(n, n_lm)); }

constexpr int FFT_ROW = 1024;   // longest row transformed by one workgroup
constexpr int TAB = 3 * 1024;   // the transforms' tables

}  // namespace

size_t ile_fd_tmp_bytes(int64_t n, int n_det, int n_lm)
{
    const size_t t = n > FFT_ROW ? (size_t)n_det * n_lm * n * 16 : 0;
    const size_t runs = (size_t)n_det * uv_runs(n, n_lm);
    return (size_t)(n_det * n + TAB) * 16 + t + runs * n_lm * n_lm * 32 + runs * 4 + 64;
}

hipError_t ile_launch_qvu(const double *h, const double *d, const double *psd, int64_t n,
                          int n_det, int n_lm, double df, double f_min, double f_max, double t0,
                          double *Q, double *U, double *V, void *tmp, int32_t *err,
                          int32_t *err_host, hipEvent_t e0, hipEvent_t e1, hipStream_t st)
{
    const bool row = n <= FFT_ROW;
    const int lg = log2i(n), rows = n_det * n_lm;
    fd_args A{};
    A.lg2 = row ? lg : lg / 2;
    A.lg1 = lg - A.lg2;   // both <= 10 for n <= 2^20
    const int N1 = 1 << A.lg1, N2 = 1 << A.lg2;
    double2 *tab = (double2 *)tmp, *g = tab + TAB;
    A.h = (const double2 *)h;
    A.g = g;
    A.tab = tab;
    A.psd = psd;
    A.t = g + (size_t)n_det * n;
    A.Q = (double2 *)Q;
    A.part = (double *)(A.t + (row ? 0 : (size_t)rows * n));
    A.U = U;
    A.V = V;
    A.err = err;
    A.err_host = err_host;
    A.n = n;
    A.n_det = n_det;
    A.n_lm = n_lm;
    A.runs = uv_runs(n, n_lm);
    A.per = uv_per(n, n_lm);
    A.ub = uv_block(n_lm);
    A.used = (int32_t *)(A.part + (size_t)n_det * A.runs * n_lm * n_lm * 4);
    A.df = df;
    A.f_min = f_min;
    A.f_max = f_max;
    const int64_t ng = std::max<int64_t>(n, 2 * N2 + N1);
    hipLaunchKernelGGL(k_fd_g, dim3((unsigned)((ng + FD_T - 1) / FD_T), n_det + 1), dim3(FD_T), 0, st,
                       (const double2 *)d, psd, n, df, f_min, f_max, t0, n_det, N1, N2, tab, g, err);
    hipError_t e = hipEventRecord(e0, st);
    if (e != hipSuccess) return e;
    const int n2 = (n_lm + 1) / 2;
    const size_t luv = std::max<size_t>((size_t)2 * A.ub * 2 * n2 * sizeof(double2),
                                        (size_t)4 * n2 * n2 * 4 * sizeof(double));
    const int nuv1 = A.runs * n_det,
              nuv2 = (n_lm * n_lm * 4 + FD_T / UV_S - 1) / (FD_T / UV_S) * n_det;
    if (row) {
        const size_t lr = (fft_pad((int)n) + 1 + n) * sizeof(double2);
        hipLaunchKernelGGL(k_fd_first<true>, dim3(nuv1 + rows), dim3(FD_T), std::max(luv, lr), st, A);
        hipLaunchKernelGGL(k_fd_second<true>, dim3(nuv2), dim3(FD_T), 0, st, A);
    } else {
        // sequences per workgroup: up to 16 (runs of 256 bytes) within FFT_PTS
        // and 64 KB with the tables
        A.lgA = std::min(4, log2i(FFT_PTS) - A.lg2);
        A.lgC = std::min(4, log2i(FFT_PTS) - A.lg1);
        const size_t ta = 2 * (size_t)N2 + (A.lg1 != A.lg2 ? N1 : 0);
        const auto lds_a = [&] { return (((size_t)fft_pad(N2) << A.lgA) + ta) * sizeof(double2); };
        while (A.lgA > 0 && lds_a() > 64 * 1024) A.lgA--;
        const size_t lc = (((size_t)fft_pad(N1) << A.lgC) + N1) * sizeof(double2);
        hipLaunchKernelGGL(k_fd_first<false>, dim3(nuv1 + (unsigned)rows * (N1 >> A.lgA)), dim3(FD_T),
                           std::max(luv, lds_a()), st, A);
        hipLaunchKernelGGL(k_fd_second<false>, dim3(nuv2 + (unsigned)rows * (N2 >> A.lgC)), dim3(FD_T),
                           lc, st, A);
    }
    e = hipGetLastError();
    return e != hipSuccess ? e : hipEventRecord(e1, st);
}
