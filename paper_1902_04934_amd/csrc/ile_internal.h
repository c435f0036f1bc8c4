// ile_internal.h -- device-side parameter blocks and launch wrappers shared
// by the HIP kernels (ile_kernels.hip) and the C-ABI host code (ile_api.cpp).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include "ile.h"

// Enum fields and arguments arrive from C callers, where any int may sit in
// them; C++ must not load an out-of-range value as the enum type, so the
// ABI reads them as 32-bit integers and validates those.
template <typename E> inline int32_t enum_raw(const E &e)
{
    static_assert(sizeof(E) == sizeof(int32_t), "4-byte enum");
    int32_t v;
    memcpy(&v, &e, sizeof v);
    return v;
}

#define ILE_NPAR 7
#define ILE_MAX_TERMS 160   // Wigner-d terms over all modes (l <= 6, <= 32 modes)
#define ILE_LMAX 6

// Everything the kernels need about one intrinsic point and the detector
// network, passed by value as a kernel argument.
struct ile_geom {
    int n_det, n_lm, n_t, half;      // half = (n_t - 1) / 2
    int n_q;                         // length of each Q series
    int s_max;                       // largest valid window start, n_q - n_t
    // phased matrix-core engine: bins of a chunk and the LDS stride of a
    // sample's row of them (one more); set per launch from the LDS budget
    int wcap, wrow;
    double t0;                       // time of Q[0]
    double dt;                       // 1 / srate
    double d_ref, gmst, t_ref_max;
    double r[ILE_MAX_DET][3];        // site vectors [m]
    double D[ILE_MAX_DET][9];        // detector tensors
    // ordering key: Hilbert index of the window starts of up to 3 detectors
    int key_lo[3];
    int key_shift;                   // log2 of the cell width in samples
    int key_bits;                    // bits per axis
    int key_dims;                    // detectors used in the key
    // -2Y_lm as sums of a_t cos(i/2)^pc_t sin(i/2)^ps_t, times e^{i m phi}
    int mode_m[ILE_MAX_LM];
    int mode_first[ILE_MAX_LM];
    int mode_nterm[ILE_MAX_LM];
    double term_a[ILE_MAX_TERMS];
    // the powers pc_t | ps_t << 8, 32-bit so that the kernels read them with
    // scalar loads (a byte field of a kernel argument is a vector load)
    int term_pw[ILE_MAX_TERMS];
    int n_pw;                        // powers 0 .. n_pw - 1 of cos and sin(i/2) used
    int m_max;                       // largest |m| of the modes
    // surrogate form: per-sample vectors z [N][n_lm] used in place of -2Y_lm
    // (the n_lm "modes" are then basis functions), or null
    const double2 *ext_y;
};

// Device pointers of one intrinsic point of a batch.
struct ile_point_dev {
    const void *Q;            // planar Q (context precision)
    const double2 *U, *V;
    const double *smp;        // samples [7][N]
    int64_t N;
    const int32_t *perm;      // sorted order (local indices)
    const int32_t *shifts;    // window starts [n_det][N]
    double *out;              // lnLmargT [N]
    // phased engine: the point's per-sample terms (ile_launch_terms_multi, tile
    // order from position 0) and what they are formed from, the samples'
    // records and the packed triangles (ile_pack_uv); or all null, and the
    // tiles form them
    double *terms;
    const struct ile_sample_rec *rec;
    const double *uvt;
};

// A sample as the per-sample terms read it: parameters 0 .. 5 (t_ref is in the
// window starts) and the window starts (all -1 for an invalid sample, 0 past
// n_det).  One 64-byte line, so gathering records through the sample order
// reads no more memory than a copy in that order would.
struct __attribute__((aligned(16))) ile_sample_rec {
    double th[6];
    int32_t s[ILE_MAX_DET];
};
static_assert(sizeof(ile_sample_rec) == 64, "one line");

// Speed of light [m/s].
constexpr double kIleC = 299792458.0;

__device__ inline bool sample_ok(const ile_geom &g, const double th[7])
{
    bool fin = true;
#pragma unroll
    for (int p = 0; p < 7; p++) fin = fin && isfinite(th[p]);
    return fin && th[5] > 0.0 && th[4] >= -1.0 && th[4] <= 1.0 &&
           fabs(th[6]) <= g.t_ref_max;
}

// Window starts of a sample: s_k = floor((t_ref + tau_k - t0)/dt + 1/2) - half
// with the arrival delay tau_k; false (s then undefined) if the sample or a
// window is out of range.  Operation order as written, no contraction, so that
// the window rounding agrees with an independent evaluation except within
// 1e-9 of a tie.
__device__ inline bool window_starts(const ile_geom &g, const double th[7],
                                     int (&s)[ILE_MAX_DET])
{
#pragma clang fp contract(off)
    bool ok = sample_ok(g, th);
    const double h = th[0] - g.gmst;
    const double cd = cos(th[1]);
    const double n0 = cd * cos(h);
    const double n1 = cd * sin(h);
    const double n2 = sin(th[1]);
#pragma unroll
    for (int k = 0; k < ILE_MAX_DET; k++) {
        s[k] = 0;
        if (k < g.n_det) {
            const double nr = n0 * g.r[k][0] + n1 * g.r[k][1] + n2 * g.r[k][2];
            const double tau = -nr / kIleC;
            const double x = (th[6] + tau - g.t0) / g.dt;
            const double xs = floor(x + 0.5) - (double)g.half;
            if (xs >= 0.0 && xs <= (double)g.s_max)
                s[k] = (int)xs;
            else
                ok = false;
        }
    }
    return ok;
}

// A sample's record, or (rec null) its window starts.
__device__ inline void store_starts(const ile_geom &g, const double th[7],
                                    const int (&s)[ILE_MAX_DET], bool ok, ile_sample_rec *rec,
                                    int32_t *shifts, int64_t i, int64_t N)
{
    if (rec) {
        ile_sample_rec R;
#pragma unroll
        for (int p = 0; p < 6; p++) R.th[p] = th[p];
#pragma unroll
        for (int k = 0; k < ILE_MAX_DET; k++) R.s[k] = ok ? s[k] : -1;
        rec[i] = R;
    } else {
#pragma unroll
        for (int k = 0; k < ILE_MAX_DET; k++)
            if (k < g.n_det) shifts[k * N + i] = ok ? s[k] : -1;
    }
}

// Counting sort of the samples by key, three kernels: the keys are counted and
// every sample takes its slot in its bucket (block_count_slot), the counts
// are scanned within blocks of ILE_SCAN_BLOCK (ile_launch_scan), and a sample's
// place is its bucket's offset, its scan block's (the prefix of the block
// totals, which each workgroup of the scatter forms in LDS: cheaper than two
// more kernels over the counts) and its slot.
#define ILE_SCAN_BLOCK 4096
#define ILE_PREP_T 1024

// Counts key in table for every live thread of the workgroup (ILE_PREP_T
// threads, all of which call it) and returns the thread's slot: the bucket's
// count before the workgroup's, plus the thread's rank among the
// workgroup's samples of that key.  Equal keys of a workgroup are merged in
// an LDS hash table first, so that a table entry takes one atomic per
// workgroup that holds its key: concentrated draws fall into a few buckets,
// where the atomics of one address are serial.
__device__ inline uint32_t block_count_slot(uint32_t *table, uint32_t key, bool live)
{
    constexpr int NS = 2 * ILE_PREP_T;
    constexpr uint32_t kFree = 0xffffffffu;   // no key (fewer than 2^25 buckets)
    __shared__ uint32_t hk[NS], hc[NS], hb[NS];
    for (int i = threadIdx.x; i < NS; i += ILE_PREP_T) {
        hk[i] = kFree;
        hc[i] = 0;
    }
    __syncthreads();
    uint32_t at = (key * 2654435761u) >> 16 & (NS - 1), r = 0;
    if (live) {
        for (;;) {   // at most ILE_PREP_T of the NS entries are ever taken
            uint32_t have = hk[at];
            if (have == kFree) have = atomicCAS(&hk[at], kFree, key);
            if (have == kFree || have == key) break;
            at = (at + 1) & (NS - 1);
        }
        r = atomicAdd(&hc[at], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < NS; i += ILE_PREP_T)
        if (hc[i]) hb[i] = atomicAdd(&table[hk[i]], hc[i]);
    __syncthreads();
    return live ? hb[at] + r : 0u;
}

// Exclusive prefix of the nb scan-block totals into pre (LDS, nb words), by a
// workgroup of 256 threads, all of which call it.
__device__ inline void scan_prefix(const uint32_t *bsum, int nb, uint32_t *pre)
{
    __shared__ uint32_t ws[4];
    const int t = threadIdx.x, lane = t & 63, per = (nb + 255) / 256;
    uint32_t sum = 0;
    for (int j = t * per; j < min((t + 1) * per, nb); j++) sum += bsum[j];
    uint32_t inc = sum;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t u = __shfl_up(inc, off);
        if (lane >= off) inc += u;
    }
    if (lane == 63) ws[t >> 6] = inc;
    __syncthreads();
    uint32_t run = inc - sum;
    for (int w = 0; w < (t >> 6); w++) run += ws[w];
    for (int j = t * per; j < min((t + 1) * per, nb); j++) {
        pre[j] = run;
        run += bsum[j];
    }
    __syncthreads();
}

// Largest of a wave's values, in every lane.
__device__ inline double wave_max(double x)
{
    for (int off = 32; off > 0; off >>= 1) x = fmax(x, __shfl_xor(x, off));
    return x;
}

// A workgroup's NV sums of T values each (a thread's v[k] into sm[k][t]) by the
// fixed tree (t, t + T/2), (t, t + T/4), ..., of which the first wave does all:
// one barrier.  In lane 0 of that wave.
template <int T, int NV>
__device__ inline void tree_sum(double (&v)[NV], double (*sm)[T])
{
    const int t = threadIdx.x;
#pragma unroll
    for (int k = 0; k < NV; k++) sm[k][t] = v[k];
    __syncthreads();
    if (t >= 64) return;
#pragma unroll
    for (int k = 0; k < NV; k++) {
        double x[T / 64];
#pragma unroll
        for (int j = 0; j < T / 64; j++) x[j] = sm[k][t + 64 * j];
#pragma unroll
        for (int h = T / 128; h > 0; h >>= 1)
#pragma unroll
            for (int j = 0; j < h; j++) x[j] += x[j + h];
        for (int off = 32; off > 0; off >>= 1) x[0] += __shfl_down(x[0], off);
        v[k] = x[0];
    }
}

// The result of a partial (M, S1, S2, n, maxL).
__device__ inline void finish_one(double M, double S1, double S2, double n, double ML,
                                  double *res)
{
    if (M == -INFINITY || n == 0.0) {
        res[0] = -INFINITY;
        res[1] = 0.0;
        res[2] = 0.0;
        res[3] = NAN;
    } else {
        res[0] = M + log(S1) - log(n);
        res[1] = S1;
        res[2] = S1 * S1 / S2;
        const double var = S2 / (S1 * S1) - 1.0 / n;
        res[3] = var > 0.0 ? sqrt(var) : 0.0;
    }
    res[4] = ML;
    res[5] = n;
}

// Ordering key of a sample: its cell (window starts of up to three
// detectors, each in cells of 2^key_shift positions, key_bits bits per axis)
// numbered along the Hilbert curve, so that runs of consecutive keys stay
// compact in every axis (tiles of consecutive samples then span narrower
// windows than along a Morton order).  Skilling's transpose form (J.
// Skilling, "Programming the Hilbert curve", AIP Conf. Proc. 707, 381, 2004),
// then the transposed bits interleaved from the most significant.
__device__ inline uint32_t cell_key(const ile_geom &g, const int *s)
{
    const int n = g.key_dims, b = g.key_bits;
    if (n < 1 || b < 1) return 0;   // a single cell
    uint32_t x[3] = {0, 0, 0};
#pragma unroll
    for (int d = 0; d < 3; d++)
        if (d < n) {
            int c = (s[d] - g.key_lo[d]) >> g.key_shift;
            c = c < 0 ? 0 : c;
            c = c > (1 << b) - 1 ? (1 << b) - 1 : c;
            x[d] = (uint32_t)c;
        }
    const uint32_t top = 1u << (b - 1);
    for (uint32_t q = top; q > 1; q >>= 1) {
        const uint32_t p = q - 1;
#pragma unroll
        for (int i = 0; i < 3; i++)
            if (i < n) {
                if (x[i] & q) {
                    x[0] ^= p;
                } else {
                    const uint32_t t = (x[0] ^ x[i]) & p;
                    x[0] ^= t;
                    x[i] ^= t;
                }
            }
    }
#pragma unroll
    for (int i = 1; i < 3; i++)
        if (i < n) x[i] ^= x[i - 1];
    const uint32_t last = n == 3 ? x[2] : n == 2 ? x[1] : x[0];
    uint32_t t = 0;
    for (uint32_t q = top; q > 1; q >>= 1)
        if (last & q) t ^= q - 1;
    uint32_t key = 0;
    for (int bit = b - 1; bit >= 0; bit--)
#pragma unroll
        for (int i = 0; i < 3; i++)
            if (i < n) key = (key << 1) | (((x[i] ^ t) >> bit) & 1u);
    return key;
}

// K steps of the matrix-core contraction (4 real rows = 2 modes each); the
// device Q holds 4 * ksp_of(n_lm) rows per detector (rows 2a and 2a+1 = Re,
// Im of mode a, the rest zero).
__device__ inline double ipow(double x, int n)
{
    double r = 1.0;
    for (int i = 0; i < n; i++) r *= x;
    return r;
}

// -2Y_lm(iota, phi) of mode a from the per-mode Wigner-d term table.
__device__ inline double2 sylm_dev(const ile_geom &g, int a, double cos_iota,
                                   double phi)
{
    double c = sqrt(0.5 * (1.0 + cos_iota));   // cos(iota/2)
    double s = sqrt(0.5 * (1.0 - cos_iota));   // sin(iota/2)
    double sum = 0.0;
    const int t0 = g.mode_first[a], nt = g.mode_nterm[a];
    for (int t = t0; t < t0 + nt; t++)
        sum += g.term_a[t] * ipow(c, g.term_pw[t] & 255) * ipow(s, g.term_pw[t] >> 8);
    double sm, cm;
    sincos((double)g.mode_m[a] * phi, &sm, &cm);
    return make_double2(sum * cm, sum * sm);
}

// The tables that harmonics are read from, register arrays read at indices that
// are the same in every lane: powers of cos(iota/2), sin(iota/2) by repeated
// products from 1, and e^{i m phi} = (e^{i phi})^m, |m| <= ILE_LMAX.
constexpr int kPw = 2 * ILE_LMAX + 1;
__device__ __forceinline__ void ylm_tables(double cos_iota, double phi, double (&cp)[kPw],
                                           double (&sp)[kPw], double (&er)[kPw],
                                           double (&ei)[kPw])
{
    const double c = sqrt(0.5 * (1.0 + cos_iota)), sn = sqrt(0.5 * (1.0 - cos_iota));
    cp[0] = sp[0] = 1.0;
#pragma unroll
    for (int q = 1; q < kPw; q++) {
        cp[q] = cp[q - 1] * c;
        sp[q] = sp[q - 1] * sn;
    }
    double s1, c1;
    sincos(phi, &s1, &c1);
    er[ILE_LMAX] = 1.0;
    ei[ILE_LMAX] = 0.0;
#pragma unroll
    for (int m = 1; m <= ILE_LMAX; m++) {
        const double pr = er[ILE_LMAX + m - 1], pi = ei[ILE_LMAX + m - 1];
        er[ILE_LMAX + m] = fma(pr, c1, -(pi * s1));
        ei[ILE_LMAX + m] = fma(pr, s1, pi * c1);
        er[ILE_LMAX - m] = er[ILE_LMAX + m];
        ei[ILE_LMAX - m] = -ei[ILE_LMAX + m];
    }
}

// -2Y_lm of mode a from the tables: its Wigner-d terms, then e^{i m phi}.
__device__ __forceinline__ double2 ylm_entry(const ile_geom &g, int a, const double (&cp)[kPw],
                                             const double (&sp)[kPw], const double (&er)[kPw],
                                             const double (&ei)[kPw])
{
    const int u0 = g.mode_first[a], nt = g.mode_nterm[a];
    double sum = 0.0;
    for (int u = u0; u < u0 + nt; u++)
        sum += g.term_a[u] * cp[g.term_pw[u] & 255] * sp[g.term_pw[u] >> 8];
    const int mi = ILE_LMAX + g.mode_m[a];
    return make_double2(sum * er[mi], sum * ei[mi]);
}

__host__ __device__ inline int ksp_of(int n_lm) { return (2 * n_lm + 3) / 4; }

// K steps (32 rows each) of the BF16 hi/lo contraction: the rows are
// [Q_hi (2 n_lm); Q_lo (2 n_lm); Q_hi (2 n_lm)], zero-padded; the device Q
// holds them K-contiguous per position: [n_det][n_q][32 * ksb_of(n_lm)] bf16.
__host__ __device__ inline int ksb_of(int n_lm) { return (6 * n_lm + 31) / 32; }

// Packed triangles of the quadratic term: detector by detector, four rows a0 ..
// a0 + 3 at a time, first their diagonal entries, then column by column b =
// a0 + 1 .. n_lm - 1 their entries (a, b), zeros where b <= a or a >= n_lm; an
// entry is (Re U_h, Im U_h, Re V_s, Im V_s) of the Hermitian part of U and the
// symmetric part of V.  Four groups of zeros follow the last (they are fetched,
// not used).  Doubles needed, then the packing itself from U, V
// [n_det][n_lm][n_lm] complex.
inline size_t ile_pack_uv_doubles(int n_det, int n_lm)
{
    size_t groups = 0;
    for (int a0 = 0; a0 < n_lm; a0 += 4) groups += n_lm - a0;
    return 16 * (n_det * groups + 4);
}
inline void ile_pack_uv(int n_det, int n_lm, const double *U, const double *V, double *out)
{
    memset(out, 0, ile_pack_uv_doubles(n_det, n_lm) * sizeof(double));
    for (int k = 0; k < n_det; k++)
        for (int a0 = 0; a0 < n_lm; a0 += 4)
            for (int c = a0; c < n_lm; c++, out += 16)   // c = a0: the diagonal
                for (int i = 0; i < 4 && a0 + i < n_lm; i++) {
                    const int a = a0 + i, b = c == a0 ? a : c;
                    if (c != a0 && b <= a) continue;
                    const size_t e = 2 * (((size_t)k * n_lm + a) * n_lm + b),
                                 f = 2 * (((size_t)k * n_lm + b) * n_lm + a);
                    double *o = out + 4 * i;
                    o[0] = 0.5 * (U[e] + U[f]);
                    o[1] = 0.5 * (U[e + 1] - U[f + 1]);
                    o[2] = 0.5 * (V[e] + V[f]);
                    o[3] = 0.5 * (V[e + 1] + V[f + 1]);
                }
}

// Tuning of the contraction kernel.
struct ile_tune {
    int tile_samples;   // samples per workgroup tile (16)
    int threads;        // positions per G block of the pipelined engines: 128 .. 512
    int engine;         // 0: FMA on the vector ALUs, 1: matrix cores, producer and
                        // consumer waves; 3: matrix cores, phased waves
    int lds_budget;     // phased engine: dynamic LDS per workgroup in bytes (0: default)
};
bool ile_tune_supported(ile_precision prec, const ile_tune &tu);
// Sets the phased engine's block width in g (wcap, wrow) for this tuning;
// zero for the other engines.
void ile_contract_prepare(ile_geom &g, ile_precision prec, const ile_tune &tu);

// Launch wrappers (ile_kernels.hip).  All are asynchronous on `st`.
hipError_t ile_launch_fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t st);
// n complex values all finite? else bit 0 of *flag.
hipError_t ile_launch_finite(const double *z, int64_t n, int32_t *flag, hipStream_t st);
// Source rows r0 .. r0 + nr - 1 (row k n_lm + a: detector k, mode a) of Q,
// positions i0 .. i0 + ni - 1, from raw [nr][ni] complex to the planar layout
// dst [n_det][4 ksp_of(n_lm)][n_q] of double (fp64) or float: rows 2a, 2a + 1 =
// Re, Im of mode a; a detector's zero rows are written with its last mode.
hipError_t ile_launch_planar(const double *raw, int r0, int nr, int64_t i0, int64_t ni, int n_lm,
                             int64_t n_q, bool fp64, void *dst, hipStream_t st);
// Window starts and ordering keys of N samples: records into rec or (rec null)
// window starts [n_det][N] into shifts; the bucket counts and every sample's
// slot in its bucket into hist and slot (hist null: neither).  Invalid samples
// take the last bucket and set bit 0 of *err.
hipError_t ile_launch_prep(const ile_geom &g, const double *smp, int64_t N, ile_sample_rec *rec,
                           int32_t *shifts, uint32_t *keys, uint32_t *slot, uint32_t *hist,
                           uint32_t n_buckets, int32_t *err, hipStream_t st);
// Exclusive scan within blocks of ILE_SCAN_BLOCK of the n counts v, the block
// totals into tmp.
hipError_t ile_launch_scan(uint32_t *v, int64_t n, uint32_t *tmp, hipStream_t st);
int64_t ile_scan_tmp_words(int64_t n);
// perm: the samples in key order, from the scanned counts of n_buckets.
hipError_t ile_launch_scatter(const uint32_t *keys, const uint32_t *slot, int64_t N,
                              const uint32_t *offs, const uint32_t *bsum, int64_t n_buckets,
                              int32_t *perm, hipStream_t st);
// The same order from the keys alone, by comparing all pairs: N at most
// ile_rank_max(), where one kernel of N^2 comparisons takes less time than
// the counts' clearing, scan and scatter.
int64_t ile_rank_max();
hipError_t ile_launch_rank(const uint32_t *keys, int64_t N, int32_t *perm, hipStream_t st);
hipError_t ile_launch_identity(int32_t *perm, int64_t N, hipStream_t st);
// Per-sample terms of Eq. (7) that the phased engine reads instead of
// forming them in its tiles (kernel k_terms, run by ile_launch_contract
// before the tiles that read them): for tile position i (sample perm[i])
// the fields f = 0 .. F - 1 (F = ile_terms_fields) at terms[16 F (r / 16) +
// 16 f + r % 16], r = i - t0, t0 the first position of the launch (a
// tile's fields are contiguous): q (the quadratic term), a validity flag (1
// or 0), (d_ref/D) F_k (re, im) for each detector, -2Y_lm (re, im) for
// each mode, then for each detector a pair of integers: the sample's window
// start less its tile's smallest, and (first two positions of a tile) that
// smallest start and the spread of the tile's starts; q, the F_k and the
// windows are zero for an invalid sample.  Whole tiles are written.
int ile_terms_fields(const ile_geom &g);
bool ile_contract_uses_terms(ile_precision prec, const ile_tune &tu);
// The terms of positions 0 .. n-1 of every point, one launch (max_lm: the
// points' largest number of modes).
hipError_t ile_launch_terms_multi(const ile_geom *geoms, const ile_point_dev *pts, int n_points,
                                  int max_lm, int64_t n, hipStream_t st);
// Positions per launch of the terms (a multiple of 16): the buffer for N
// samples holds ile_terms_fields x min(N, ILE_TERMS_CHUNK) doubles.
#define ILE_TERMS_CHUNK ((int64_t)1 << 21)
// uvt: the packed triangles (ile_pack_uv); terms: a buffer of
// ile_terms_fields x cap doubles, cap >= 16 a multiple of 16 (both used when
// ile_contract_uses_terms, else may be null).
// rec: the samples' records when ile_contract_uses_terms (smp and shifts are
// then not read), else null.
hipError_t ile_launch_contract(const ile_geom &g, ile_precision prec,
                               const ile_tune &tu, const double *smp, int64_t N,
                               const int32_t *perm, const int32_t *shifts,
                               const void *Q, const double *U, const double *V,
                               const ile_sample_rec *rec, const double *uvt, double *terms,
                               int64_t cap, double *out, double *series,
                               hipStream_t st);
size_t ile_contract_lds_bytes(const ile_geom &g, ile_precision prec,
                              const ile_tune &tu);
hipError_t ile_launch_prior(uint64_t seed, int64_t first, int64_t N,
                            double d_min, double d_max, double t_ref_max,
                            double *smp, int64_t ld, double *ln_p, hipStream_t st);
// Importance-sampling reduction of N values into a 5-double partial
// {M, S1, S2, n, maxL} with S1 = sum e^{lnw-M}, S2 = sum e^{2(lnw-M)}.
int ile_reduce_blocks();
// res (if not null): the n_part partials at parts, of which partial is the
// last, merged in order and finished into result[6].
hipError_t ile_launch_reduce(const double *lnL, const double *ln_p,
                             const double *ln_q, int64_t N, double *tmp,
                             double *partial, const double *parts, int n_part, double *res,
                             hipStream_t st);
// flag[0] | flag[1] to the first word of host and res[0 .. 5] to host[1 .. 6] (pinned
// host memory; either may be null).
hipError_t ile_launch_fetch(const int32_t *flag, const double *res, double *host,
                            hipStream_t st);
// Adaptive sampler (ile_sampler.hip): histogram state P[2][nb], C[2][nb+1].
int ile_hist_max_bins();
hipError_t ile_launch_hist_uniform(int nb, double *P, double *C, hipStream_t st);
hipError_t ile_launch_hist_cdf(int nb, const double *P, double *C, hipStream_t st);
hipError_t ile_launch_hist_draw(uint64_t seed, int64_t first, int64_t N, int nb,
                                const double *P, const double *C, double d_min,
                                double d_max, double t_ref_max, double *smp, int64_t ld,
                                double *ln_p, double *ln_q, int32_t *bins, hipStream_t st);
size_t ile_hist_refit_tmp_doubles(int64_t N, int nb);
hipError_t ile_launch_hist_refit(const int32_t *bins, int64_t ld, const double *lnL,
                                 const double *ln_p, const double *ln_q, int64_t N, int nb,
                                 double floor_w, double scale, double *tmp, double *P,
                                 double *C, hipStream_t st);
// Batched form (ile_batch.hip + the persistent contraction).
size_t ile_contract_dyn_bytes(const ile_geom &g, ile_precision prec, const ile_tune &tu);
// Allows the persistent kernel of this tuning `dyn` bytes of dynamic LDS;
// call outside stream capture, before ile_launch_contract_batched.
hipError_t ile_contract_batched_allow(ile_precision prec, const ile_tune &tu, size_t dyn);
hipError_t ile_launch_contract_batched(ile_precision prec, const ile_tune &tu,
                                       const ile_geom *geoms, const ile_point_dev *pts,
                                       const int2 *items, int n_items, unsigned *counter,
                                       int grid, size_t dyn, bool terms, hipStream_t st);
hipError_t ile_launch_prior_multi(const uint64_t *seed_dev, const int64_t *offs, int n_points,
                                  int64_t n_total, double d_min, double d_max,
                                  double t_ref_max, double *smp, hipStream_t st);
hipError_t ile_launch_prep_multi(const ile_geom *geoms, const int64_t *offs, int n_points,
                                 int64_t n_total, const double *smp, ile_sample_rec *rec,
                                 int32_t *shifts, uint32_t *keys, uint32_t *slot,
                                 uint32_t *hist, uint32_t B, int32_t *err, hipStream_t st);
hipError_t ile_launch_scatter_multi(const uint32_t *keys, const uint32_t *slot,
                                    const int64_t *offs, int n_points, int64_t n_total,
                                    const uint32_t *pos, const uint32_t *bsum,
                                    int64_t n_buckets, int32_t *perm, hipStream_t st);
// tmp: ile_reduce_points_tmp(n_points) doubles.  host (pinned): the error flag
// in its first word, then the 6 n_points results from its second double.
size_t ile_reduce_points_tmp(int n_points);
hipError_t ile_launch_reduce_points(const double *out, const double *lw, const int64_t *offs,
                                    int n_points, double *tmp, const int32_t *err, double *host,
                                    hipStream_t st);
hipError_t ile_launch_batch_lw(const double *lp, const double *lq, int64_t n_total, double *lw,
                               int32_t *err, hipStream_t st);
hipError_t ile_launch_to_bf16_split(const double *Q, int64_t n, void *dst,
                                    hipStream_t st);

// ------------------------------------ surrogate (linear-basis) form
// z_b = sum_lm c_lm,b(lambda) -2Y_lm(iota, phi) per joint sample (rows 0..6
// extrinsic, row 7 lambda of smp [8][N]); gp holds the physical modes' Y
// tables; err bit 0 for lambda outside [-1, 1] (z = NaN).  A: the packed
// coefficients, mode by mode and power by power of lambda the n_b complex
// values, padded with zeros to groups of eight (ile_pack_rom_doubles; a group
// more follows the last).
size_t ile_pack_rom_doubles(int n_lm, int n_b, int n_pow);
void ile_pack_rom(int n_lm, int n_b, int n_pow, const double *A, double *out);
hipError_t ile_launch_rom_z(const ile_geom &gp, const double *smp, int64_t N, const double *A,
                            int n_b, int n_pow, double *Z, int32_t *err, hipStream_t st);

// ------------------------------------ Q, U, V from the frequency domain
// Q [n_det][n_lm][n] complex, U, V [n_det][n_lm][n_lm] complex from the mode
// and data transforms and the spectra (n a power of two in [2, 2^20]); err bit
// 0 for a non-finite input or a non-positive spectrum in the band, copied to
// the host word err_host (mapped host memory, valid once the stream has been
// waited for).  tmp: ile_fd_tmp_bytes; the kernels that transform lie between
// the events.
size_t ile_fd_tmp_bytes(int64_t n, int n_det, int n_lm);
hipError_t ile_launch_qvu(const double *h, const double *d, const double *psd, int64_t n,
                          int n_det, int n_lm, double df, double f_min, double f_max, double t0,
                          double *Q, double *U, double *V, void *tmp, int32_t *err,
                          int32_t *err_host, hipEvent_t e0, hipEvent_t e1, hipStream_t st);

// ------------------------------------------------ extrinsic harvest
// weights: w = exp(ln w - max ln w), ln w = lnL + ln p - ln q (NULL: 0),
// part: ile_hv_parts() + 1 doubles; err bit 0: an invalid ln p / ln q, bit 1:
// no finite positive weight.  pick (u is [2][n_out]): err bit 2 for a uniform
// outside [0, 1) in either row.
int ile_hv_parts();
hipError_t ile_launch_hv_weights(const double *lnL, const double *ln_p, const double *ln_q,
                                 int64_t n, double *w, double *part, int32_t *err,
                                 hipStream_t st);
hipError_t ile_launch_hv_pick(const double *cdf, int64_t n, const double *u, int64_t n_out,
                              int64_t *idx, int32_t *err, hipStream_t st);
hipError_t ile_launch_hv_gather(const double *smp, int64_t ld, const int64_t *idx, int64_t m,
                                double *sel, hipStream_t st);
// one wave per row of series[m][n_t]; theta [7][ld_out] may be NULL
hipError_t ile_launch_hv_bin(const double *series, int64_t m, int n_t, const double *v,
                             const double *sel, double srate, int32_t *bins, double *theta,
                             int64_t ld_out, hipStream_t st);

// ------------------------------------------------ learned proposal (MDN)
// Network sizes and the flat parameter layout (W1 | b1 | W2 | b2 | W3 | b3,
// row-major, masked entries held at zero) documented in ile.h.
#define ILE_MDN_D 7
#define ILE_MDN_H 128
#define ILE_MDN_C 16
#define ILE_MDN_O 336
#define ILE_MDN_OFF_W1 0
#define ILE_MDN_OFF_B1 896
#define ILE_MDN_OFF_W2 1024
#define ILE_MDN_OFF_B2 17408
#define ILE_MDN_OFF_W3 17536
#define ILE_MDN_OFF_B3 60544
#define ILE_MDN_NPARAM 60880
#define ILE_MDN_W3T_LD 384    // rows of the transposed W3 copy, zero past 336
#define ILE_MDN_NPART 36608   // per-workgroup partial: unmasked gradient tiles, loss sum, weight sum
#define ILE_MDN_TILE 64       // samples per workgroup pass

// MADE masks: hidden unit k has degree k mod 6; unit k sees inputs
// i <= deg(k); layer-2 unit k2 sees k1 with deg(k1) <= deg(k2); output o
// (dimension o / 48) sees units with deg(k) < o / 48.  Biases are free.
__host__ __device__ inline bool ile_mdn_trainable(int j)
{
    if (j < 0 || j >= ILE_MDN_NPARAM) return false;
    if (j < ILE_MDN_OFF_B1) return (j % ILE_MDN_D) <= (j / ILE_MDN_D) % 6;
    if (j < ILE_MDN_OFF_W2) return true;
    if (j < ILE_MDN_OFF_B2) {
        const int q = j - ILE_MDN_OFF_W2;
        return (q % ILE_MDN_H) % 6 <= (q / ILE_MDN_H) % 6;
    }
    if (j < ILE_MDN_OFF_W3) return true;
    if (j < ILE_MDN_OFF_B3) {
        const int q = j - ILE_MDN_OFF_W3;
        return (q % ILE_MDN_H) % 6 < (q / ILE_MDN_H) / (3 * ILE_MDN_C);
    }
    return true;
}

// Transform between the sample vector and the network's inputs.
struct ile_mdn_tr {
    double origin[3];   // ra, psi, phi origins
    double mean[7], scale[7];
    double d_min, d_max, t_ref_max, sigma_floor;
    double sigma_scale;   // kappa of draws and densities (training: 1)
};

// Device state of one proposal.
struct ile_mdn_dev {
    float *theta, *m, *v;               // [NPARAM] master weights and Adam moments
    __bf16 *W2b, *W3b;                  // [o][k] copies (forward operands)
    __bf16 *W2t, *W3t;                  // [k][o] copies (backward operands)
    ile_mdn_tr *tr;                     // transform
};

// Defensive mixture with the histogram proposal (nb = 0 or eps = 0: none).
struct ile_mdn_mix {
    int nb;
    const double *P, *C;   // histogram state [2][nb], [2][nb+1]
    double eps;
};

hipError_t ile_launch_mdn_cast(const ile_mdn_dev &M, hipStream_t st);
// ln q of n samples x[7][ld] (optionally mixed), or draws of n samples
// (counters first..first+n-1 of key seed) with their ln p and ln q.
hipError_t ile_launch_mdn_logpdf(const ile_mdn_dev &M, const ile_mdn_mix &mix,
                                 const double *x, int64_t ld, int64_t n, double *ln_q,
                                 int grid, hipStream_t st);
hipError_t ile_launch_mdn_sample(const ile_mdn_dev &M, const ile_mdn_mix &mix,
                                 uint64_t seed, int64_t first, int64_t n, double *x,
                                 int64_t ld, double *ln_p, double *ln_q, int grid,
                                 hipStream_t st);
// Training pieces.  prepare: z~ and tempered weights; cdf: inclusive
// prefix sums of the weights.
// fit: tempering (ESS target ess_frac of the finite samples) into stats =
// {max ln w, beta}, and (if fit_transform) the transform into tr; ws is a
// workspace of ile_mdn_fit_ws_doubles() doubles.
hipError_t ile_launch_mdn_fit(const double *x, int64_t ld, const double *lnw, int64_t n,
                              double ess_frac, ile_mdn_tr *tr, double *stats, double *ws,
                              bool fit_transform, hipStream_t st);
size_t ile_mdn_fit_ws_doubles();
hipError_t ile_launch_mdn_prepare(const ile_mdn_tr *tr, const double *x, int64_t ld,
                                  const double *lnw, int64_t n, const double *stats,
                                  float *z, double *w, hipStream_t st);
// the same with given weights w_in (NULL: 1) instead of tempered ones
hipError_t ile_launch_mdn_prepare_w(const ile_mdn_tr *tr, const double *x, int64_t ld,
                                    const double *w_in, int64_t n, float *z, double *w,
                                    hipStream_t st);
hipError_t ile_launch_mdn_cdf(const double *w, int64_t n, double *cdf, double *ws,
                              hipStream_t st);   // ws: ile_mdn_fit_ws_doubles() doubles
// count minibatch draws (index i with probability w_i / sum w), Philox
// counters (draw, 0, 0x4D444E54) of key seed
hipError_t ile_launch_mdn_draw_idx(uint64_t seed, int64_t count, const double *cdf, int64_t n,
                                   int32_t *idx, hipStream_t st);
// Forward + backward of a batch: per-workgroup partials [grid][NPART].
hipError_t ile_launch_mdn_grad(const ile_mdn_dev &M, const float *z, int64_t ldz,
                               const int32_t *idx, const double *w, int batch, float *part,
                               hipStream_t st);
// Reduce the partials in fixed order; mask; write the gradient (grad may be
// NULL) and the loss; if adam, take one Adam step number `step` (1-based).
hipError_t ile_launch_mdn_update(const ile_mdn_dev &M, const float *part, int n_part,
                                 float *grad, double *loss, bool adam, int64_t step, double lr,
                                 hipStream_t st);
hipError_t ile_launch_lnw(const double *lnL, const double *ln_p, const double *ln_q, int64_t n,
                          double *lnw, hipStream_t st);

// cross-object accessors (defined in ile_api.cpp / ile_prop_api.cpp)
hipStream_t ile_ctx_stream(const ile_ctx *c);
int ile_ctx_hist(const ile_ctx *c, const double **P, const double **C);   // nb, or 0
const ile_mdn_dev &ile_prop_dev(const ile_prop *p);
hipStream_t ile_prop_stream(const ile_prop *p);
int ile_prop_grid(const ile_prop *p);

// Zero-noise injection (ile_kernels.hip): detector responses d[n_det][n] of
// theta (device, 7 doubles), then Q [n_det][n_lm][n] (scaled), U and V
// [n_lm][n_lm] (complex interleaved).
hipError_t ile_launch_inject(const ile_geom &g, const double *h, int n, const double *theta,
                             double *d, hipStream_t st);
hipError_t ile_launch_inject_qv(int n_det, int n_lm, int n, const double *h, const double *d,
                                double scale, double *Q, double *U, double *V, hipStream_t st);
