// ile_kernels.hip -- gfx950 kernels of the ILE likelihood hot path.
//
// Paper: arXiv:1902.04934.  Sec. II.A defines the per-sample likelihood
// (Eq. (7), matrix form Eq. (10)) and its time marginalization (Eq. (9));
// Sec. II.B describes the GPU step whose most costly part is the contraction
// of Q over detector-dependent time windows; Sec. II.C the Monte Carlo
// accuracy measure.
//
// Pipeline for a block of N samples:
//   k_prep        window starts s_k per (sample, detector), validity,
//                 ordering key (Hilbert index of the window starts), the
//                 sample's record and its slot among the samples of its key
//   k_scan_local, k_scatter   the samples' order by key (cells of nearby
//                 windows) from the counts; k_rank: by pairs, for small N
//   k_terms       per sample in tile order: harmonics, antenna factors and the
//                 quadratic term of Eq. (7) (FP64 and FP32 phased engine)
//   k_contract_ph per tile of 16 samples: the coefficients in LDS; per time
//                 chunk and detector the products sum_lm Re(conj(c) Q[p]) over
//                 the union of the tile's windows on the matrix cores (each Q
//                 value loaded once feeds 16 samples), moved to each sample's
//                 bin row and summed over the detectors; FP64 log-sum-exp over
//                 the bins; deterministic tree at the end
//   k_contract    the same with the per-sample work in the tile, producer and
//                 consumer waves (BF16; selectable for FP64/FP32) or VALU
//   k_red*        FP64 importance-sampling partials {M, S1, S2, n, maxL} and
//                 their result.
#include <hip/hip_runtime.h>

#include <math.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "ile_internal.h"
#include "ile_rng.h"

namespace {

constexpr double kC = 299792458.0;
constexpr double kTwoPi = 6.283185307179586476925;
constexpr double kPi = 3.141592653589793238463;


// ---------------------------------------------------------------- geometry
// Arrival delay at site k relative to the geocentre, tau = -n.r/c, with n
// the unit vector towards the source (Sec. II.A, detector response).  Same
// operation order as written, no contraction, so that the window rounding
// agrees with an independent evaluation except within 1e-9 of a tie.
__device__ inline double delay_dev(const ile_geom &g, int k, double ra,
                                   double dec)
{
#pragma clang fp contract(off)
    double h = ra - g.gmst;
    double n0 = cos(dec) * cos(h);
    double n1 = cos(dec) * sin(h);
    double n2 = sin(dec);
    double nr = n0 * g.r[k][0] + n1 * g.r[k][1] + n2 * g.r[k][2];
    return -nr / kC;
}

// Antenna patterns from the detector tensor: polarization basis X, Y of a
// source at hour angle h = ra - gmst, declination dec, rotated by psi;
// F+ = X.D.X - Y.D.Y, Fx = X.D.Y + Y.D.X.  tr = (sin h, cos h, sin dec,
// cos dec, sin psi, cos psi).
__device__ inline void antenna_trig(const ile_geom &g, int k, const double tr[6], double &fp,
                                    double &fx)
{
    const double sh = tr[0], ch = tr[1], sd = tr[2], cd = tr[3], sp = tr[4], cp = tr[5];
    const double eE[3] = {-sh, ch, 0.0};
    const double eN[3] = {-sd * ch, -sd * sh, cd};
    double X[3], Y[3];
#pragma unroll
    for (int i = 0; i < 3; i++) {
        X[i] = -cp * eE[i] + sp * eN[i];
        Y[i] = sp * eE[i] + cp * eN[i];
    }
    double DX[3], DY[3];
#pragma unroll
    for (int i = 0; i < 3; i++) {
        DX[i] = g.D[k][3 * i] * X[0] + g.D[k][3 * i + 1] * X[1] + g.D[k][3 * i + 2] * X[2];
        DY[i] = g.D[k][3 * i] * Y[0] + g.D[k][3 * i + 1] * Y[1] + g.D[k][3 * i + 2] * Y[2];
    }
    fp = (X[0] * DX[0] + X[1] * DX[1] + X[2] * DX[2]) -
         (Y[0] * DY[0] + Y[1] * DY[1] + Y[2] * DY[2]);
    fx = (X[0] * DY[0] + X[1] * DY[1] + X[2] * DY[2]) +
         (Y[0] * DX[0] + Y[1] * DX[1] + Y[2] * DX[2]);
}

__device__ inline void antenna_dev(const ile_geom &g, int k, double ra,
                                   double dec, double psi, double &fp,
                                   double &fx)
{
    double tr[6];
    sincos(ra - g.gmst, &tr[0], &tr[1]);
    sincos(dec, &tr[2], &tr[3]);
    sincos(psi, &tr[4], &tr[5]);
    antenna_trig(g, k, tr, fp, fx);
}

// Per-sample tables of the tile prologue: the sines and cosines of the
// antenna patterns, powers 0 .. 2 ILE_LMAX of cos(iota/2) and sin(iota/2),
// and e^{i m phi} for |m| <= ILE_LMAX.
constexpr int kProTab = 6 + 2 * kPw + 2 * kPw;   // doubles per sample

__host__ __device__ inline size_t prologue_scratch_bytes(int ts, int nd, int nl)
{
    // s_th[7][ts], s_Y[ts][nl], s_F[ts][nd] (complex), s_qp[ts][nd*nl],
    // the per-sample tables [ts][kProTab]
    return sizeof(double) * (size_t)ts * (7 + 2 * nl + 2 * nd + nd * nl + kProTab);
}

// ------------------------------------------------------------- injection
// Zero-noise injection with a white unit-variance noise spectrum, so the
// inner product of Eq. (2) is <a|b> = sum_i conj(a_i) b_i (circular).
// Detector response to theta (Eqs. (5), (6) and the response below Eq. (6)):
//   d_k[i] = Re(F_k (D_ref/D) sum_a Y_a h_a[(i - lag_k) mod n]),
//   lag_k  = floor((t_ref + tau_k - t0)/dt + 1/2)  (the window rounding).
__global__ __launch_bounds__(256) void k_inject_resp(ile_geom g, const double2 *__restrict__ h,
                                                     int n, const double *__restrict__ th,
                                                     double *d)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= (int64_t)g.n_det * n) return;
    const int k = (int)(t / n), i = (int)(t % n);
    double fp, fx;
    antenna_dev(g, k, th[0], th[1], th[2], fp, fx);
    const double tau = delay_dev(g, k, th[0], th[1]);
    double x;
    {
#pragma clang fp contract(off)
        x = (th[6] + tau - g.t0) / g.dt;
    }
    const int64_t lag = (int64_t)floor(x + 0.5);
    int64_t src = ((int64_t)i - lag) % n;
    if (src < 0) src += n;
    const double kappa = g.d_ref / th[5];
    double re = 0.0, im = 0.0;
    for (int a = 0; a < g.n_lm; a++) {
        const double2 y = sylm_dev(g, a, th[4], th[3]);
        const double2 v = h[(size_t)a * n + src];
        re += y.x * v.x - y.y * v.y;
        im += y.x * v.y + y.y * v.x;
    }
    // Re(F z) with F = F+ + i Fx
    d[t] = kappa * (fp * re - fx * im);
}

// Q_k,a[s] = scale * sum_i conj(h_a[(i - s) mod n]) d_k[i]  (Eq. (8)): one
// workgroup per (k, a) and 256 consecutive s; d and the needed 511 h values
// of each 256-wide chunk of i are staged in LDS; sums run in i order.
__global__ __launch_bounds__(256) void k_inject_corr(int n_lm, int n, const double2 *__restrict__ h,
                                                     const double *__restrict__ d, double scale,
                                                     double2 *Q)
{
    __shared__ double sd[256];
    __shared__ double2 sh[512];
    const int ka = blockIdx.y, k = ka / n_lm, a = ka % n_lm;
    const int s0 = blockIdx.x * 256, t = threadIdx.x, s = s0 + t;
    double re = 0.0, im = 0.0;
    for (int i0 = 0; i0 < n; i0 += 256) {
        sd[t] = i0 + t < n ? d[(size_t)k * n + i0 + t] : 0.0;
        for (int j = t; j < 511; j += 256) {
            int64_t idx = ((int64_t)i0 - s0 - 255 + j) % n;
            if (idx < 0) idx += n;
            sh[j] = h[(size_t)a * n + idx];
        }
        __syncthreads();
        for (int ii = 0; ii < 256; ii++) {
            const double2 v = sh[ii - t + 255];
            re += v.x * sd[ii];
            im -= v.y * sd[ii];
        }
        __syncthreads();
    }
    if (s < n) Q[(size_t)ka * n + s] = make_double2(scale * re, scale * im);
}

// U_ab = sum_i conj(h_a[i]) h_b[i], V_ab = sum_i h_a[i] h_b[i] (Eq. (8));
// one workgroup per (a, b), fixed-order tree sum.
__global__ __launch_bounds__(256) void k_inject_gram(int n_lm, int n, const double2 *__restrict__ h,
                                                     double2 *U, double2 *V)
{
    __shared__ double red[4][256];
    const int a = blockIdx.x / n_lm, b = blockIdx.x % n_lm, t = threadIdx.x;
    double ur = 0, ui = 0, vr = 0, vi = 0;
    for (int i = t; i < n; i += 256) {
        const double2 x = h[(size_t)a * n + i], y = h[(size_t)b * n + i];
        ur += x.x * y.x + x.y * y.y;
        ui += x.x * y.y - x.y * y.x;
        vr += x.x * y.x - x.y * y.y;
        vi += x.x * y.y + x.y * y.x;
    }
    red[0][t] = ur;
    red[1][t] = ui;
    red[2][t] = vr;
    red[3][t] = vi;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (t < w)
            for (int q = 0; q < 4; q++) red[q][t] += red[q][t + w];
        __syncthreads();
    }
    if (t == 0) {
        U[blockIdx.x] = make_double2(red[0][0], red[1][0]);
        V[blockIdx.x] = make_double2(red[2][0], red[3][0]);
    }
}

// ------------------------------------------------------------ data layout
__global__ __launch_bounds__(256) void k_finite(const double2 *__restrict__ z, int64_t n,
                                                int32_t *flag)
{
    bool bad = false;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        bad |= !(isfinite(z[i].x) && isfinite(z[i].y));
    if (bad) atomicOr(flag, 1);
}

// A pass at the copy rate in place of the host's (3 x 21 x 16384 values: 1 ms of
// checks and stores there, with the page faults of a second copy).
template <typename T>
__global__ __launch_bounds__(256) void k_planar(const double2 *__restrict__ raw, int r0,
                                                int64_t i0, int64_t ni, int n_lm, int rp,
                                                int64_t n_q, T *__restrict__ dst)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= ni) return;
    const int r = r0 + blockIdx.y, k = r / n_lm, a = r % n_lm;
    const double2 z = raw[(int64_t)blockIdx.y * ni + i];
    T *d = dst + ((int64_t)k * rp + 2 * a) * n_q + i0 + i;
    d[0] = (T)z.x;
    d[n_q] = (T)z.y;
    if (a == n_lm - 1)
        for (int q = 2; 2 * a + q < rp; q++) d[q * n_q] = (T)0;
}

// ------------------------------------------------------------------ prep
__global__ void k_fill_u32(uint32_t *p, uint32_t v, int64_t n)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// Window starts, keys and (COUNT) bucket slots.  What bounds the counting is
// the atomics of one bucket, which are serial: an atomic per workgroup and key
// takes 22 us of 1e5 samples that fall into a few buckets with workgroups of
// 1024 (30 with 512, 45 with 256; 37 with an atomic per wave and key), 18 of
// draws spread over the prior.
template <int T, bool COUNT>
__global__ __launch_bounds__(T) void k_prep(ile_geom g, const double *__restrict__ smp,
                                                     int64_t N, ile_sample_rec *__restrict__ rec,
                                                     int32_t *__restrict__ shifts,
                                                     uint32_t *__restrict__ keys,
                                                     uint32_t *__restrict__ slot, uint32_t *hist,
                                                     uint32_t n_buckets, int32_t *err)
{
    const int64_t i = (int64_t)blockIdx.x * T + threadIdx.x;
    const bool live = i < N;
    const int64_t il = live ? i : N - 1;
    double th[7];
#pragma unroll
    for (int p = 0; p < 7; p++) th[p] = smp[p * N + il];
    int s[ILE_MAX_DET];
    const bool ok = window_starts(g, th, s);
    const uint32_t key = ok ? cell_key(g, s) : n_buckets - 1;   // invalid samples sort last
    if (live) {
        if (!ok) atomicOr(err, 1);
        store_starts(g, th, s, ok, rec, shifts, i, N);
        keys[i] = key;
    }
    if constexpr (COUNT) {
        const uint32_t r = block_count_slot(hist, key, live);
        if (live) slot[i] = r;
    }
}

// Exclusive scan of the counts within blocks of 1024 threads x 4 values.
constexpr int kScanT = 1024;
constexpr int kScanPer = 4;
static_assert(kScanT * kScanPer == ILE_SCAN_BLOCK, "");

__global__ __launch_bounds__(kScanT) void k_scan_local(uint32_t *v, int64_t n,
                                                       uint32_t *bsum)
{
    __shared__ uint32_t ws[kScanT / 64];
    const int t = threadIdx.x, lane = t & 63;
    const int64_t base = (int64_t)blockIdx.x * ILE_SCAN_BLOCK + (int64_t)t * kScanPer;
    uint32_t x[kScanPer], run = 0;
#pragma unroll
    for (int j = 0; j < kScanPer; j++) {
        x[j] = base + j < n ? v[base + j] : 0u;
        run += x[j];
    }
    uint32_t inc = run;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t u = __shfl_up(inc, off);
        if (lane >= off) inc += u;
    }
    if (lane == 63) ws[t >> 6] = inc;
    __syncthreads();
    uint32_t ex = inc - run, total = 0;
#pragma unroll
    for (int w = 0; w < kScanT / 64; w++) {
        ex += w < (t >> 6) ? ws[w] : 0u;
        total += ws[w];
    }
#pragma unroll
    for (int j = 0; j < kScanPer; j++) {
        if (base + j < n) v[base + j] = ex;
        ex += x[j];
    }
    if (t == 0) bsum[blockIdx.x] = total;
}

// Four bytes a sample are moved: 15 us for 1e6 samples, where taking the slots
// here by atomics and copying the samples into tile order took 183 (the terms
// read records through the order as fast as copies).
__global__ __launch_bounds__(256) void k_scatter(const uint32_t *__restrict__ keys,
                                                 const uint32_t *__restrict__ slot, int64_t N,
                                                 const uint32_t *__restrict__ offs,
                                                 const uint32_t *__restrict__ bsum, int nb,
                                                 int32_t *__restrict__ perm)
{
    extern __shared__ __align__(16) unsigned char dyn_lds[];
    uint32_t *pre = reinterpret_cast<uint32_t *>(dyn_lds);
    scan_prefix(bsum, nb, pre);
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= N) return;
    const uint32_t k = keys[i];
    perm[offs[k] + pre[k / ILE_SCAN_BLOCK] + slot[i]] = (int32_t)i;
}

// A sample's place is the number of keys below its own and of equal keys
// before it.  A workgroup places 64 samples, its waves share the keys, which
// come as scalars: 5 us for 1000 samples, 17 for 10000.
constexpr int kRankT = 1024;
__global__ __launch_bounds__(kRankT) void k_rank(const uint32_t *__restrict__ keys, int N,
                                                 int32_t *__restrict__ perm)
{
    __shared__ int cnt[kRankT / 64][64];
    const int lane = threadIdx.x & 63, b = blockIdx.x, i = b * 64 + lane;
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const uint32_t ki = i < N ? keys[i] : 0xfffffffeu;
    int c = 0;
    for (int q = wv; q * 64 < N; q += kRankT / 64) {
        const int j0 = q * 64;
        const uint32_t lim = ki + (q < b ? 1u : 0u);
        if (q == b || j0 + 64 > N) {   // its own samples, or the last few
            const int kq = (int)(j0 + lane < N ? keys[j0 + lane] : 0xffffffffu);
#pragma unroll 8
            for (int j = 0; j < 64; j++)
                c += (uint32_t)__builtin_amdgcn_readlane(kq, j) <
                     lim + (q == b && j < lane ? 1u : 0u);
        } else {
#pragma unroll
            for (int j = 0; j < 64; j++) c += keys[j0 + j] < lim;
        }
    }
    cnt[wv][lane] = c;
    __syncthreads();
    if (wv == 0 && i < N) {
        int at = 0;
#pragma unroll
        for (int w = 0; w < kRankT / 64; w++) at += cnt[w][lane];
        perm[at] = i;
    }
}

__global__ __launch_bounds__(256) void k_identity(int32_t *perm, int64_t N)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < N) perm[i] = (int32_t)i;
}

// ------------------------------------------------------------ contraction
// One workgroup = one tile of TS samples (in sorted order), NT threads.
// Q is stored planar per detector: row 2a holds Re Q_a, row 2a+1 Im Q_a,
// so Re(conj(c_a) Q_a[p]) = sum over the two rows of C[row] * Qm[row][p].
//
// G phase per (chunk, detector), two engines:
//   ENG_VALU: each thread owns one position p and accumulates G for all TS
//             samples with FMAs; coefficients broadcast from LDS.
//   ENG_MFMA: the G block is the real GEMM  C[TS x 2n_lm] * Qm[2n_lm x p]
//             on v_mfma_f64_16x16x4 (TS = 16 = M); each wave owns N-tiles of
//             16 positions, A (coefficients) from LDS, B (Q) from memory.
// Realign: thread j of the chunk adds G[alpha][s_alpha,k - s_min,k + j] for
// every sample; online FP64 log-sum-exp over the bins each thread owns.
// ENG_PH: the phased matrix-core engine below (FP64 or FP32 operands).
enum { ENG_VALU = 0, ENG_MFMA = 1, ENG_BF16 = 2, ENG_PH = 3 };

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// One 16x16x4 matrix-core step in the precision of the operands.  Output
// layouts on gfx950 (checked with lane-layout probes): f64 gives
// D[l/16 + 4v][l%16], f32 (and bf16 below) D[4(l/16) + v][l%16].
template <typename TQ> struct mfma_acc;
template <> struct mfma_acc<double> {
    using type = v4d;
    static __device__ inline v4d step(double a, double b, v4d c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ inline int row(int r, int v) { return r + 4 * v; }
};
template <> struct mfma_acc<float> {
    using type = v4f;
    static __device__ inline v4f step(float a, float b, v4f c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ inline int row(int r, int v) { return 4 * r + v; }
};

// G block on the matrix cores: Gs[alpha][p] = sum_r A[alpha][r] Qm[r][P0 + p]
// for p < W (<= NT), 16 samples.  v_mfma_f64_16x16x4 on gfx950 (checked
// with a lane-layout probe): lane l supplies A[l%16][l/16] and B[l/16][l%16]
// and receives D[l/16 + 4v][l%16], v = 0..3.  Wave wv computes the N-tiles
// wv, wv+NW, ... (NU of them, wave-uniform) of 16 positions.  Q rows are
// padded with zeros to 4 KSP in memory, so every lane loads a valid row;
// columns past the end of Q are clamped (their results are never read).
template <typename TQ, int NT, int NU>
__device__ inline void mfma_tiles(TQ *Gs, const TQ *coefA, const TQ *Qk, int nq,
                                  int KSP, int P0, int lane, int wv)
{
    constexpr int NW = NT / 64;
    const int row = lane >> 4, col = lane & 15;
    using M = mfma_acc<TQ>;
    typename M::type acc[NU];
    const TQ *qb[NU];
#pragma unroll
    for (int u = 0; u < NU; u++) {
        acc[u] = typename M::type{0, 0, 0, 0};
        qb[u] = Qk + (int64_t)row * nq + min(P0 + 16 * (wv + NW * u) + col, nq - 1);
    }
    const int64_t step = 4 * (int64_t)nq;
    // three operand buffers, each reloaded right after its MFMAs consumed
    // it, so every load is in flight for two k-steps; the k-steps past KSP
    // of the last round are skipped by wave-uniform tests (prefetch indices
    // past the end are clamped and unused)
    const int kl = KSP - 1;
    TQ a0 = coefA[lane], a1 = coefA[min(1, kl) * 64 + lane], a2, b0[NU], b1[NU], b2[NU];
#pragma unroll
    for (int u = 0; u < NU; u++) {
        b0[u] = qb[u][0];
        b1[u] = qb[u][min(1, kl) * step];
    }
    // sched_barrier(0) keeps the compiler from folding the prefetch back
    // next to its use
    for (int ks = 0; ks < KSP; ks += 3) {
        const int k2 = min(ks + 2, kl), k3 = min(ks + 3, kl), k4 = min(ks + 4, kl);
        a2 = coefA[k2 * 64 + lane];
#pragma unroll
        for (int u = 0; u < NU; u++) b2[u] = qb[u][k2 * step];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < NU; u++)
            acc[u] = M::step(a0, b0[u], acc[u]);
        __builtin_amdgcn_sched_barrier(0);
        a0 = coefA[k3 * 64 + lane];
#pragma unroll
        for (int u = 0; u < NU; u++) b0[u] = qb[u][k3 * step];
        __builtin_amdgcn_sched_barrier(0);
        if (ks + 1 < KSP) {
#pragma unroll
            for (int u = 0; u < NU; u++)
                acc[u] = M::step(a1, b1[u], acc[u]);
        }
        __builtin_amdgcn_sched_barrier(0);
        a1 = coefA[k4 * 64 + lane];
#pragma unroll
        for (int u = 0; u < NU; u++) b1[u] = qb[u][k4 * step];
        __builtin_amdgcn_sched_barrier(0);
        if (ks + 2 < KSP) {
#pragma unroll
            for (int u = 0; u < NU; u++)
                acc[u] = M::step(a2, b2[u], acc[u]);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int u = 0; u < NU; u++) {
        const int t = wv + NW * u;
#pragma unroll
        for (int v = 0; v < 4; v++) Gs[M::row(row, v) * NT + 16 * t + col] = (TQ)acc[u][v];
    }
}

template <typename TQ, int NT>
__device__ inline void mfma_gphase(TQ *Gs, const TQ *coefA, const TQ *Qk, int nq,
                                   int KSP, int P0, int W, int lane)
{
    constexpr int NW = NT / 64, TPW = NT / 16 / NW;
    static_assert(TPW == 4, "four N-tiles per wave");
    // wave index in an SGPR so the tile count below is known to be uniform
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ntile = (W + 15) >> 4;
    int nu = ntile > wv ? (ntile - wv + NW - 1) / NW : 0;
    nu = __builtin_amdgcn_readfirstlane(nu < TPW ? nu : TPW);
    switch (nu) {
    case 4: mfma_tiles<TQ, NT, 4>(Gs, coefA, Qk, nq, KSP, P0, lane, wv); break;
    case 3: mfma_tiles<TQ, NT, 3>(Gs, coefA, Qk, nq, KSP, P0, lane, wv); break;
    case 2: mfma_tiles<TQ, NT, 2>(Gs, coefA, Qk, nq, KSP, P0, lane, wv); break;
    case 1: mfma_tiles<TQ, NT, 1>(Gs, coefA, Qk, nq, KSP, P0, lane, wv); break;
    default: break;
    }
}

// BF16 hi/lo contraction on v_mfma_f32_16x16x32_bf16: the K dimension is
// the concatenation [Q_hi; Q_lo; Q_hi] against [C_hi, C_hi, C_lo] (3 x 2 n_lm
// rows, zero-padded to 32 KSB), i.e. C.Q to about 16 significant bits with
// float accumulation.  Q is stored K-contiguous per position
// (Qb[p][32 KSB] bf16), so a lane's 8 consecutive k values are one 16-byte
// load; A comes from LDS in the same [ks][lane][8] order.
template <int NT, int NU>
__device__ inline void bf16_tiles(float *Gs, const v8bf *coefA, const v8bf *Qk, int nq, int KSB,
                                  int P0, int lane, int wv)
{
    constexpr int NW = NT / 64;
    const int row = lane >> 4, col = lane & 15;
    v4f acc[NU];
    const v8bf *qb[NU];
#pragma unroll
    for (int u = 0; u < NU; u++) {
        acc[u] = v4f{0, 0, 0, 0};
        qb[u] = Qk + (int64_t)min(P0 + 16 * (wv + NW * u) + col, nq - 1) * (4 * KSB) + row;
    }
    for (int ks = 0; ks < KSB; ks++) {
        const v8bf a = coefA[ks * 64 + lane];
        v8bf b[NU];
#pragma unroll
        for (int u = 0; u < NU; u++) b[u] = qb[u][4 * ks];
#pragma unroll
        for (int u = 0; u < NU; u++) acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[u], acc[u], 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < NU; u++) {
        const int t = wv + NW * u;
#pragma unroll
        for (int v = 0; v < 4; v++) Gs[(4 * row + v) * NT + 16 * t + col] = acc[u][v];
    }
}

template <int NT>
__device__ inline void bf16_gphase(float *Gs, const v8bf *coefA, const v8bf *Qk, int nq, int KSB,
                                   int P0, int W, int lane)
{
    constexpr int NW = NT / 64, TPW = NT / 16 / NW;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ntile = (W + 15) >> 4;
    int nu = ntile > wv ? (ntile - wv + NW - 1) / NW : 0;
    nu = __builtin_amdgcn_readfirstlane(nu < TPW ? nu : TPW);
    switch (nu) {
    case 4: bf16_tiles<NT, 4>(Gs, coefA, Qk, nq, KSB, P0, lane, wv); break;
    case 3: bf16_tiles<NT, 3>(Gs, coefA, Qk, nq, KSB, P0, lane, wv); break;
    case 2: bf16_tiles<NT, 2>(Gs, coefA, Qk, nq, KSB, P0, lane, wv); break;
    case 1: bf16_tiles<NT, 1>(Gs, coefA, Qk, nq, KSB, P0, lane, wv); break;
    default: break;
    }
}

template <int ENG> __host__ __device__ inline size_t coef_bytes(int ts, int nd, int nl, size_t e)
{
    // VALU: complex [nd][nl][ts]; MFMA: real [nd][KSP][64]; BF16: [nd][KSB][64][8] bf16
    return ENG == ENG_VALU   ? (size_t)nd * nl * ts * 2 * e
           : ENG == ENG_MFMA ? (size_t)nd * ksp_of(nl) * 64 * e
                             : (size_t)nd * ksb_of(nl) * 64 * 8 * 2;
}

// Online log-sum-exp of one bin's contraction per sample (q is constant
// over bins and is subtracted at the end); one exp per sample and bin.
template <typename TQ, int TS>
__device__ __forceinline__ void lse_update(const TQ *L, double *m, double *sacc)
{
#pragma unroll
    for (int al = 0; al < TS; al++) {
        const double x = (double)L[al];
        const double d = x - m[al];
        const double e = exp(-fabs(d));
        const bool gt = d > 0.0;
        sacc[al] = gt ? fma(sacc[al], e, 1.0) : sacc[al] + e;
        m[al] = gt ? x : m[al];
    }
}

// Iterator over the pipeline items (chunk j0 of Jc bins, detector k,
// position block blk).
struct PipeIt {
    int j0, Jc, k, blk;
    bool valid;
};

__device__ __forceinline__ void pipe_first(PipeIt &it, int J, int n_t)
{
    it.j0 = 0;
    it.Jc = min(J, n_t);
    it.k = 0;
    it.blk = 0;
    it.valid = n_t > 0;
}

__device__ __forceinline__ void pipe_next(PipeIt &it, int J, int n_t, int nd,
                                          const int *spread, int NP)
{
    it.blk += NP;
    if (it.blk < it.Jc + spread[it.k]) return;
    it.blk = 0;
    if (++it.k < nd) return;
    it.k = 0;
    it.j0 += J;
    if (it.j0 < n_t) {
        it.Jc = min(J, n_t - it.j0);
        return;
    }
    it.valid = false;
}

__device__ __forceinline__ bool pipe_last_of_chunk(const PipeIt &it, int nd, int spread_last,
                                                   int NP)
{
    return it.k == nd - 1 && it.blk + NP >= it.Jc + spread_last;
}

// Deterministic reduction of the per-thread log-sum-exp states over the
// workgroup, in two halves separated by barriers: each wave writes its
// per-sample maximum (then its per-sample sum of s e^{m - M}) to s_red[wave]
// by a fixed butterfly; the M (then the result) are formed over the waves
// in wave order.  Threads with no state contribute -inf (then 0).
template <int TS>
__device__ inline void lse_wave_max(const double *m, double (*s_red)[TS], int lane, int wv)
{
#pragma unroll
    for (int al = 0; al < TS; al++) {
        double v = m ? m[al] : -INFINITY;
        for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off));
        if (lane == 0) s_red[wv][al] = v;
    }
}
template <int TS>
__device__ inline void lse_wave_sum(const double *m, const double *sacc, const double *s_M,
                                    double (*s_red)[TS], int lane, int wv)
{
#pragma unroll
    for (int al = 0; al < TS; al++) {
        double v = 0.0;
        if (m) v = (m[al] == -INFINITY) ? 0.0 : sacc[al] * exp(m[al] - s_M[al]);
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
        if (lane == 0) s_red[wv][al] = v;
    }
}

// 16-lane reductions of doubles by DPP row rotations (8, 4, 2, 1 lanes) of
// both 32-bit halves: lane i meets the partner value of an xor butterfly
// (after the rotation by n the partials repeat with period n), so every lane
// of the row ends with the same bits.
template <int N>
__device__ inline double row_ror64(double x)
{
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)u, 0x120 + N, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), 0x120 + N, 0xF, 0xF,
                                               false);
    return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}
__device__ inline double row_max64(double x)
{
    x = fmax(x, row_ror64<8>(x));
    x = fmax(x, row_ror64<4>(x));
    x = fmax(x, row_ror64<2>(x));
    return fmax(x, row_ror64<1>(x));
}
__device__ inline double row_sum64(double x)
{
    x += row_ror64<8>(x);
    x += row_ror64<4>(x);
    x += row_ror64<2>(x);
    return x + row_ror64<1>(x);
}

// Matrix-core epilogue: the consumers' per-sample states go through LDS R
// (the free G buffers, [TS][NP] doubles); 16 lanes per sample (threads
// tid < 16 TS) combine the NP entries of their sample in a fixed order, then
// across the 16 lanes.  Pass 1 gives M = max m, pass 2 S = sum s e^{m - M}.
template <int TS, int NP>
__device__ inline double epi_reduce(const double *R, int tid, bool is_max)
{
    const int al = tid >> 4, l16 = tid & 15;
    double v = is_max ? -INFINITY : 0.0;
    for (int c = l16; c < NP; c += 16) {
        const double x = R[al * NP + c];
        v = is_max ? fmax(v, x) : v + x;
    }
    return is_max ? row_max64(v) : row_sum64(v);
}

// Per-sample part of a tile, shared by the engines: the samples, -2Y_lm,
// the antenna patterns, the coefficients c = (d_ref/D) F_k Y_lm in the
// engine's operand layout and the quadratic term q of Eq. (7).  scr is free
// LDS of scr_cap bytes (at least prologue_scratch_bytes); U_k and V_k are
// staged there too when they fit.  s_d receives the absolute window starts
// (0 for invalid samples).  Ends with a barrier.
template <typename TQ, int TS, int NT, int ENG>
__device__ __forceinline__ void tile_prologue(
    const ile_geom &g, int64_t base, const double *__restrict__ smp, int64_t N,
    const int32_t *__restrict__ perm, const int32_t *__restrict__ shifts,
    const double2 *__restrict__ U, const double2 *__restrict__ V, double *scr,
    size_t scr_cap, TQ *coef, double *s_q, int *s_idx, int *s_ok, int (*s_d)[TS])
{
    const int tid = threadIdx.x;
    const int nd = g.n_det, nl = g.n_lm;
    const int KSP = ksp_of(nl);    // k-steps per detector (padded)
    const int KSB = ksb_of(nl);    // BF16 k-steps
    const size_t scr_bytes = prologue_scratch_bytes(TS, nd, nl);
    double *s_th = scr;                                  // [7][TS]
    double2 *s_Y = reinterpret_cast<double2 *>(scr + 7 * TS);   // [TS][nl]
    double2 *s_F = s_Y + TS * nl;                        // [TS][nd]
    double *s_qp = reinterpret_cast<double *>(s_F + TS * nd);   // [TS][nd*nl]
    double *s_tab = s_qp + TS * nd * nl;                 // [TS][kProTab]

    // 1. samples of the tile and, one thread per sample, the trigonometry
    //    every mode and detector of the sample shares
    if (tid < TS) {
        int64_t i = base + tid;
        int idx = -1, ok = 0;
        double th[7] = {0, 0, 0, 0, 0, 1, 0};
        if (i < N) {
            idx = perm[i];
#pragma unroll
            for (int p = 0; p < 7; p++) th[p] = smp[(int64_t)p * N + idx];
            ok = sample_ok(g, th);
            for (int k = 0; k < nd; k++) {
                int s = shifts[(int64_t)k * N + idx];
                ok = ok && s >= 0 && s <= g.s_max;
                s_d[k][tid] = s;
            }
        }
        s_idx[tid] = idx;
        s_ok[tid] = ok;
        if (!ok) {
            th[0] = th[1] = th[2] = th[3] = th[4] = th[6] = 0.0;
            th[5] = 1.0;
            for (int k = 0; k < nd; k++) s_d[k][tid] = 0;
        }
#pragma unroll
        for (int p = 0; p < 7; p++) s_th[p * TS + tid] = th[p];
        double *tb = s_tab + tid * kProTab;
        sincos(th[0] - g.gmst, &tb[0], &tb[1]);
        sincos(th[1], &tb[2], &tb[3]);
        sincos(th[2], &tb[4], &tb[5]);
        // powers of cos(iota/2), sin(iota/2) by repeated products from 1
        const double c = sqrt(0.5 * (1.0 + th[4])), sn = sqrt(0.5 * (1.0 - th[4]));
        double *cp = tb + 6, *sp = cp + kPw;
        double pc = 1.0, ps = 1.0;
        cp[0] = sp[0] = 1.0;
        for (int q = 1; q < kPw; q++) {
            pc *= c;
            ps *= sn;
            cp[q] = pc;
            sp[q] = ps;
        }
        // e^{i m phi} = (e^{i phi})^m, m = -ILE_LMAX .. ILE_LMAX
        double2 *em = reinterpret_cast<double2 *>(sp + kPw);
        double s1, c1;
        sincos(th[3], &s1, &c1);
        double er = 1.0, ei = 0.0;
        em[ILE_LMAX] = make_double2(1.0, 0.0);
        for (int m = 1; m <= ILE_LMAX; m++) {
            const double r2 = er * c1 - ei * s1, i2 = er * s1 + ei * c1;
            er = r2;
            ei = i2;
            em[ILE_LMAX + m] = make_double2(er, ei);
            em[ILE_LMAX - m] = make_double2(er, -ei);
        }
    }
    __syncthreads();

    // 2. harmonics -2Y_lm(iota, phi) (the Wigner-d sum over the mode's
    //    terms, then e^{i m phi}), or the surrogate form's basis vectors, and
    //    the antenna patterns F = F+ + i Fx
    for (int t = tid; t < TS * (nl + nd); t += NT) {
        if (t < TS * nl) {
            const int al = t / nl, a = t - al * nl;
            if (g.ext_y) {
                s_Y[al * nl + a] = s_ok[al] ? g.ext_y[(int64_t)s_idx[al] * nl + a]
                                            : make_double2(0.0, 0.0);
            } else {
                const double *cp = s_tab + al * kProTab + 6, *sp = cp + kPw;
                const int t0 = g.mode_first[a], nt = g.mode_nterm[a];
                double sum = 0.0;
                for (int u = t0; u < t0 + nt; u++)
                    sum += g.term_a[u] * cp[g.term_pw[u] & 255] * sp[g.term_pw[u] >> 8];
                const double2 e = reinterpret_cast<const double2 *>(sp + kPw)[ILE_LMAX + g.mode_m[a]];
                s_Y[al * nl + a] = make_double2(sum * e.x, sum * e.y);
            }
        } else {
            const int u = t - TS * nl;
            const int al = u / nd, k = u - al * nd;
            double fp, fx;
            antenna_trig(g, k, s_tab + al * kProTab, fp, fx);
            s_F[al * nd + k] = make_double2(fp, fx);
        }
    }
    __syncthreads();

    // 3. per detector: the coefficients c = (d_ref/D) F_k Y_lm in the
    //    engine's operand layout (modes a in [nl, 2 KSP) are the zero padding
    //    of the matrix-core K dimension), and the rows of the quadratic term
    //    of Eq. (7).  Only the Hermitian part of U and the symmetric part of V
    //    enter it (Re(Y^H U Y) = Y^H U_h Y, Y^T V Y = Y^T V_s Y), so each row
    //    a sums over b >= a only, the off-diagonal terms twice:
    //      row_a = |F|^2 (U_h,aa |Y_a|^2 + 2 Re(conj(Y_a) sum_{b>a} U_h,ab Y_b))
    //            + Re(F^2 (V_s,aa Y_a^2 + 2 Y_a sum_{b>a} V_s,ab Y_b)).
    //    A thread takes rows a and nl - 1 - a (nl - 1 terms together).
    if (ENG == ENG_BF16) {
        unsigned short *cz = reinterpret_cast<unsigned short *>(coef);
        for (int t = tid; t < nd * KSB * 64 * 8; t += NT) cz[t] = 0;
        __syncthreads();
    }
    const int nlp = ENG == ENG_MFMA ? 2 * KSP : nl;
    const int npr = (nl + 1) / 2;
    const size_t uv_off = (scr_bytes + 15) & ~(size_t)15;
    const bool stage_uv = uv_off + 2 * (size_t)nl * nl * sizeof(double2) <= scr_cap;
    double2 *s_U = reinterpret_cast<double2 *>(reinterpret_cast<unsigned char *>(scr) + uv_off);
    double2 *s_V = s_U + nl * nl;
    for (int k = 0; k < nd; k++) {
        const double2 *Uk = U + (int64_t)k * nl * nl, *Vk = V + (int64_t)k * nl * nl;
        if (stage_uv) {
            for (int e = tid; e < nl * nl; e += NT) {
                const int a = e / nl, b = e - a * nl;
                const double2 u1 = Uk[e], u2 = Uk[b * nl + a], v1 = Vk[e], v2 = Vk[b * nl + a];
                s_U[e] = make_double2(0.5 * (u1.x + u2.x), 0.5 * (u1.y - u2.y));
                s_V[e] = make_double2(0.5 * (v1.x + v2.x), 0.5 * (v1.y + v2.y));
            }
            __syncthreads();
        }
        // coefficients: samples fastest, so the 16 lanes of one (k, a)
        // write neighbouring operand slots
        for (int t = tid; t < TS * nlp; t += NT) {
            const int al = t % TS, a = t / TS;
            double cx = 0.0, cy = 0.0;
            if (a < nl) {
                const double kap = s_ok[al] ? g.d_ref / s_th[5 * TS + al] : 0.0;
                const double2 F = s_F[al * nd + k], Ya = s_Y[al * nl + a];
                cx = kap * (F.x * Ya.x - F.y * Ya.y);
                cy = kap * (F.x * Ya.y + F.y * Ya.x);
            }
            if (ENG == ENG_VALU) {
                coef[((k * nl + a) * TS + al) * 2] = (TQ)cx;
                coef[((k * nl + a) * TS + al) * 2 + 1] = (TQ)cy;
            } else if (ENG == ENG_BF16) {
                // A row k' of [C_hi, C_hi, C_lo]: lane = 16 (k' % 32 / 8) + alpha,
                // element k' % 8, k-step k' / 32
                __bf16 *cb = reinterpret_cast<__bf16 *>(coef) + (size_t)k * KSB * 64 * 8;
                const int R = 2 * nl;
                const double cv[2] = {cx, cy};
#pragma unroll
                for (int c = 0; c < 2; c++) {
                    const __bf16 hi = (__bf16)(float)cv[c];
                    const __bf16 lo = (__bf16)(float)(cv[c] - (double)(float)hi);
                    const int r = 2 * a + c;
                    const int kk[3] = {r, R + r, 2 * R + r};
                    const __bf16 vv[3] = {hi, hi, lo};
#pragma unroll
                    for (int q = 0; q < 3; q++) {
                        const int kp = kk[q];
                        cb[((kp >> 5) * 64 + ((kp & 31) >> 3) * 16 + al) * 8 + (kp & 7)] = vv[q];
                    }
                }
            } else {
                // A operand of k-step ks: lane = 16 * (row within the step) + alpha
                const int r0 = 2 * a;
                coef[(k * KSP + (r0 >> 2)) * 64 + (r0 & 3) * 16 + al] = (TQ)cx;
                coef[(k * KSP + (r0 >> 2)) * 64 + ((r0 & 3) + 1) * 16 + al] = (TQ)cy;
            }
        }
        // rows of the quadratic term, two per thread
        for (int t = tid; t < TS * npr; t += NT) {
            const int al = t % TS, pr = t / TS;
            const double2 F = s_F[al * nd + k];
            const double f2 = F.x * F.x + F.y * F.y;
            const double F2r = F.x * F.x - F.y * F.y, F2i = 2.0 * F.x * F.y;
            const double2 *Yr = s_Y + al * nl;
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const int a = h == 0 ? pr : nl - 1 - pr;
                if (h == 1 && a == pr) break;
                double ur = 0, ui = 0, vr = 0, vi = 0;
                for (int b = a + 1; b < nl; b++) {
                    const double2 Yb = Yr[b];
                    double2 u, v;
                    if (stage_uv) {
                        u = s_U[a * nl + b];
                        v = s_V[a * nl + b];
                    } else {
                        const double2 u1 = Uk[a * nl + b], u2 = Uk[b * nl + a];
                        const double2 v1 = Vk[a * nl + b], v2 = Vk[b * nl + a];
                        u = make_double2(0.5 * (u1.x + u2.x), 0.5 * (u1.y - u2.y));
                        v = make_double2(0.5 * (v1.x + v2.x), 0.5 * (v1.y + v2.y));
                    }
                    ur += u.x * Yb.x - u.y * Yb.y;
                    ui += u.x * Yb.y + u.y * Yb.x;
                    vr += v.x * Yb.x - v.y * Yb.y;
                    vi += v.x * Yb.y + v.y * Yb.x;
                }
                const double2 Ya = Yr[a];
                double2 ud, vd;
                if (stage_uv) {
                    ud = s_U[a * nl + a];
                    vd = s_V[a * nl + a];
                } else {
                    const double2 u1 = Uk[a * nl + a], v1 = Vk[a * nl + a];
                    ud = u1;
                    vd = v1;
                }
                // Y_a (V_s,aa Y_a + 2 w): the complex sum of the V part
                const double wr = vd.x * Ya.x - vd.y * Ya.y + 2.0 * vr;
                const double wi = vd.x * Ya.y + vd.y * Ya.x + 2.0 * vi;
                const double yvr = Ya.x * wr - Ya.y * wi, yvi = Ya.x * wi + Ya.y * wr;
                const double uq = ud.x * (Ya.x * Ya.x + Ya.y * Ya.y) + 2.0 * (Ya.x * ur + Ya.y * ui);
                s_qp[al * (nd * nl) + k * nl + a] = f2 * uq + (F2r * yvr - F2i * yvi);
            }
        }
        if (stage_uv) __syncthreads();   // before the next detector's copy
    }
    __syncthreads();

    static_assert(NT >= 16 * TS, "16 lanes per sample for the quadratic sum");
    if (tid < 16 * TS) {
        const int al = tid >> 4, l16 = tid & 15;
        double sum = 0.0;
        for (int r = l16; r < nd * nl; r += 16) sum += s_qp[al * (nd * nl) + r];
        for (int off = 8; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
        if (l16 == 0) {
            const double kap = s_ok[al] ? g.d_ref / s_th[5 * TS + al] : 0.0;
            s_q[al] = 0.25 * kap * kap * sum;
        }
    }
    __syncthreads();
}

// ------------------------------------------------- per-sample terms
// The per-sample part of Eq. (7) for the phased engine, one lane per sample
// in tile order, so that it runs once per sample over the whole GPU rather
// than in one wave of each tile while the tile's other waves wait: the
// harmonics -2Y_lm(iota, phi) (Wigner-d terms times e^{i m phi}, or the
// surrogate form's vectors), the antenna patterns, the coefficient factors
// (d_ref/D) F_k and the quadratic term
//   q = (d_ref/D)^2 / 4 sum_k [ |F_k|^2 Y^H U_h,k Y + Re(F_k^2 Y^T V_s,k Y) ]
// with U_h the Hermitian part of U_k and V_s the symmetric part of V_k, so
// that only b >= a enters (the off-diagonal terms twice): the host packs the
// upper triangles (ile_pack_uv).
// Output: tile-major, field f of position t0 + r at
// terms[16 F (r / 16) + 16 f + r % 16]; the last n_det fields are integer
// pairs, the sample's window start less the smallest of its tile, and in the
// tile's first two positions that smallest start and the tile's spread.
__host__ __device__ inline int terms_fields(int nd, int nl) { return 2 + 3 * nd + 2 * nl; }

// One lane's sample: its validity, window starts, the sines and cosines of
// the antenna angles, d_ref/D, and the tables the harmonics are read from:
// powers of cos and sin of iota/2 and e^{i m phi}, register arrays (of the
// caller, so that they stay in registers) read at indices that are the same
// in every lane.
struct TermsSample {
    int idx, ok;
    int sd[ILE_MAX_DET];
    double tr[6], kap;
};

__device__ __forceinline__ void terms_intake(const ile_geom &g,
                                             const ile_sample_rec *__restrict__ rec,
                                             const int32_t *__restrict__ perm, int64_t i,
                                             bool live, TermsSample &S, double (&cp)[kPw],
                                             double (&sp)[kPw], double (&er)[kPw],
                                             double (&ei)[kPw])
{
    const int nd = g.n_det;
    S.idx = perm[i];
    const ile_sample_rec R = rec[S.idx];
    double th[6];
#pragma unroll
    for (int p = 0; p < 6; p++) th[p] = R.th[p];
    bool ok = live;
#pragma unroll
    for (int k = 0; k < ILE_MAX_DET; k++) {
        S.sd[k] = R.s[k];
        ok = ok & (k >= nd || (S.sd[k] >= 0 && S.sd[k] <= g.s_max));
    }
    S.ok = ok;
    if (!ok) {
        th[0] = th[1] = th[2] = th[3] = th[4] = 0.0;
        th[5] = 1.0;
    }
    sincos(th[0] - g.gmst, &S.tr[0], &S.tr[1]);
    sincos(th[1], &S.tr[2], &S.tr[3]);
    sincos(th[2], &S.tr[4], &S.tr[5]);
    S.kap = ok ? g.d_ref / th[5] : 0.0;
    ylm_tables(th[4], th[3], cp, sp, er, ei);
}

// -2Y_lm of mode a: the mode's Wigner-d terms, then e^{i m phi}; or the
// surrogate form's vector entry.
__device__ __forceinline__ double2 terms_harmonic(const ile_geom &g, const TermsSample &S, int a,
                                                  const double (&cp)[kPw],
                                                  const double (&sp)[kPw],
                                                  const double (&er)[kPw],
                                                  const double (&ei)[kPw])
{
    if (g.ext_y) return S.ok ? g.ext_y[(int64_t)S.idx * g.n_lm + a] : make_double2(0.0, 0.0);
    return ylm_entry(g, a, cp, sp, er, ei);
}

// Row a of detector k's part of the quadratic term (the b > a sums w_U, w_V
// over the row's entries given), with f2 = |F|^2 and F^2 = (F2r, F2i).  The
// roundings are written out, so that they do not depend on the code around.
__device__ __forceinline__ double terms_row(double2 Ya, double4 d, double ur, double ui,
                                            double vr, double vi, double f2, double F2r,
                                            double F2i)
{
    // Y_a (V_s,aa Y_a + 2 w_V): the complex sum of the V part
    const double wr = fma(2.0, vr, fma(Ya.x, d.z, -(Ya.y * d.w)));
    const double wi = fma(2.0, vi, fma(d.z, Ya.y, Ya.x * d.w));
    const double yvr = fma(Ya.x, wr, -(Ya.y * wi)), yvi = fma(Ya.y, wr, Ya.x * wi);
    const double yu = fma(ur, Ya.x, ui * Ya.y), y2 = fma(Ya.x, Ya.x, Ya.y * Ya.y);
    const double uq = fma(d.x, y2, yu + yu);
    return fma(f2, uq, fma(F2r, yvr, -(F2i * yvi)));
}

// Element n of a 16-lane row's 16 values, in every lane of the row.
template <int n> __device__ __forceinline__ double row_bcast(double x)
{
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)u, 0x150 + n, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), 0x150 + n, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

template <int n> __device__ __forceinline__ double4 row_quad(double x)   // elements n .. n + 3
{
    return make_double4(row_bcast<n>(x), row_bcast<n + 1>(x), row_bcast<n + 2>(x), row_bcast<n + 3>(x));
}

// The products of a group of four entries e (lane l holds value l % 16 of the
// group's 16, the same in every row of lanes), the entries of four rows in one
// column, with the column's harmonic y: for each row
//   u += (e_x + i e_y) y, v += (e_z + i e_w) y,
// each sum taking its e_y (e_w) product first.  An entry's value reaches the
// lanes as the multiply-add's broadcast operand (DPP row_newbcast), which
// costs nothing: the waits before the first one are what a DPP operand needs
// after a vector write of its register.
struct tri_acc {
    double ur, ui, vr, vi;
};
#define TRI_F(acc, sgn, n, y)                                                                \
    "v_fmac_f64_dpp %" acc ", " sgn "%16, %" y " row_newbcast:" n " row_mask:0xf bank_mask:0xf\n\t"
#define TRI_E(ur, ui, vr, vi, n1, n3, y0, y1, s)                                             \
    TRI_F(ur, s, n1, y0) TRI_F(ui, "", n1, y1) TRI_F(vr, s, n3, y0) TRI_F(vi, "", n3, y1)
__device__ __forceinline__ void tri_mac(double e, double2 y, tri_acc (&A)[4])
{
#ifdef __HIP_DEVICE_COMPILE__
    asm("s_nop 4\n\t"
        TRI_E("0", "1", "2", "3", "1", "3", "18", "17", "-")
        TRI_E("4", "5", "6", "7", "5", "7", "18", "17", "-")
        TRI_E("8", "9", "10", "11", "9", "11", "18", "17", "-")
        TRI_E("12", "13", "14", "15", "13", "15", "18", "17", "-")
        TRI_E("0", "1", "2", "3", "0", "2", "17", "18", "")
        TRI_E("4", "5", "6", "7", "4", "6", "17", "18", "")
        TRI_E("8", "9", "10", "11", "8", "10", "17", "18", "")
        TRI_E("12", "13", "14", "15", "12", "14", "17", "18", "")
        : "+&v"(A[0].ur), "+&v"(A[0].ui), "+&v"(A[0].vr), "+&v"(A[0].vi), "+&v"(A[1].ur),
          "+&v"(A[1].ui), "+&v"(A[1].vr), "+&v"(A[1].vi), "+&v"(A[2].ur), "+&v"(A[2].ui),
          "+&v"(A[2].vr), "+&v"(A[2].vi), "+&v"(A[3].ur), "+&v"(A[3].ui), "+&v"(A[3].vr),
          "+&v"(A[3].vi)
        : "v"(e), "v"(y.x), "v"(y.y));
#endif
}
#undef TRI_E
#undef TRI_F

// Smallest (or largest) of a 16-lane row, in every lane, by DPP row rotations.
template <bool MIN> __device__ __forceinline__ int row_red(int x)
{
    const auto f = [](int a, int b) { return MIN ? min(a, b) : max(a, b); };
    x = f(x, __builtin_amdgcn_update_dpp(0, x, 0x128, 0xF, 0xF, false));
    x = f(x, __builtin_amdgcn_update_dpp(0, x, 0x124, 0xF, 0xF, false));
    x = f(x, __builtin_amdgcn_update_dpp(0, x, 0x122, 0xF, 0xF, false));
    return f(x, __builtin_amdgcn_update_dpp(0, x, 0x121, 0xF, 0xF, false));
}

__device__ __forceinline__ void terms_store(const ile_geom &g, const TermsSample &S, double q,
                                            double *tp)
{
    const int nd = g.n_det, nl = g.n_lm;
    tp[0] = 0.25 * S.kap * S.kap * q;
    tp[16] = S.ok ? 1.0 : 0.0;
    const int r = __lane_id() & 15;
#pragma unroll
    for (int k = 0; k < ILE_MAX_DET; k++)
        if (k < nd) {
            const int lo = row_red<true>(S.ok ? S.sd[k] : 0x7fffffff);
            const int hi = row_red<false>(S.ok ? S.sd[k] : -1);
            const int2 w = make_int2(S.ok ? S.sd[k] - lo : 0,
                                     hi < 0 || r > 1 ? 0 : r == 0 ? lo : hi - lo);
            *reinterpret_cast<int2 *>(tp + (2 + 2 * nd + 2 * nl + k) * 16) = w;
        }
}

__device__ __forceinline__ double *terms_slot(const ile_geom &g, double *terms, int64_t r)
{
    return terms + (r >> 4) * (16 * (int64_t)terms_fields(g.n_det, g.n_lm)) + (r & 15);
}

constexpr int kTermsT = 64;    // lanes per block

// Any number of modes: a lane's harmonics are an LDS row of 64 lanes
// (conflict free, and no lane reads another's: no barrier), the first one, no
// row's later column, a register: 21 modes then leave eight waves a CU.  The
// quadratic form takes four rows of the triangle at a time: a column's
// harmonic is read once for four entries, whose sixteen sums are independent,
// and a group of four entries is one 8-byte load a lane (each row of 16 lanes
// holds the whole group), issued four columns ahead; memory is one run over all
// rows and detectors.  What is left is those loads' latency: 1e6 samples, 21
// modes, 3 detectors take 432 us, 147 of them the harmonics and the stores,
// against 161 for the multiply-adds at the vector rate.  A row at a time took
// 663 with an entry as two 16-byte loads of one address (2 KB returned to the
// wave's registers for 32 bytes) and 587 with the broadcast operand; two
// columns ahead 454, with the first harmonic in LDS as well 484.
__device__ __forceinline__ void terms_samples(
    const ile_geom &g, const ile_sample_rec *__restrict__ rec, const int32_t *__restrict__ perm,
    const double *__restrict__ uvt, int64_t t0, int64_t n, double *__restrict__ terms)
{
    extern __shared__ __align__(16) unsigned char dyn_lds[];
    const int lane = threadIdx.x;
    const int64_t r = (int64_t)blockIdx.x * kTermsT + lane;   // position t0 + r
    // the last tile's positions past n are written too, as invalid samples
    // (terms holds whole tiles), so that a tile's 16 lanes are all active
    if (r >= ((n + 15) & ~(int64_t)15)) return;
    const int nd = g.n_det, nl = g.n_lm;
    double2 *Yl = reinterpret_cast<double2 *>(dyn_lds) + lane;   // [nl - 1][64], Yl[b] of mode b + 1
    double *tp = terms_slot(g, terms, r);
    TermsSample S;
    double2 y0 = make_double2(0.0, 0.0);
    {
        double cp[kPw], sp[kPw], er[kPw], ei[kPw];
        terms_intake(g, rec, perm, t0 + min(r, n - 1), r < n, S, cp, sp, er, ei);
        for (int a = 0; a < nl; a++) {
            const double2 y = terms_harmonic(g, S, a, cp, sp, er, ei);
            if (a == 0) y0 = y;
            else Yl[(a - 1) * kTermsT] = y;
            tp[(2 + 2 * nd + 2 * a) * 16] = y.x;
            tp[(3 + 2 * nd + 2 * a) * 16] = y.y;
        }
    }
    const double *p = uvt + (lane & 15);
    double qs = 0.0;
    for (int k = 0; k < nd; k++) {
        double fp, fx;
        antenna_trig(g, k, S.tr, fp, fx);
        tp[(2 + 2 * k) * 16] = S.kap * fp;
        tp[(3 + 2 * k) * 16] = S.kap * fx;
        const double f2 = fp * fp + fx * fx, F2r = fp * fp - fx * fx, F2i = 2.0 * fp * fx;
        for (int a0 = 0; a0 < nl; a0 += 4) {
            // the block's diagonal, then columns a0 + 1 .. nl - 1 (zeros where
            // the column is not past the row's diagonal)
            const double dg = p[0];
            double e0 = p[16], e1 = p[32], e2 = p[48], e3 = p[64];
            tri_acc A[4] = {};
            int b = a0;   // columns b + 1
            for (; b + 4 < nl; b += 4) {
                const double2 ya = Yl[b * kTermsT], yb = Yl[(b + 1) * kTermsT];
                const double2 yc = Yl[(b + 2) * kTermsT], yd = Yl[(b + 3) * kTermsT];
                p += 64;
                const double n0 = p[16], n1 = p[32], n2 = p[48], n3 = p[64];
                tri_mac(e0, ya, A);
                tri_mac(e1, yb, A);
                tri_mac(e2, yc, A);
                tri_mac(e3, yd, A);
                e0 = n0;
                e1 = n1;
                e2 = n2;
                e3 = n3;
            }
            if (b + 1 < nl) {
                tri_mac(e0, Yl[b * kTermsT], A);
                p += 16;
            }
            if (b + 2 < nl) {
                tri_mac(e1, Yl[(b + 1) * kTermsT], A);
                p += 16;
            }
            if (b + 3 < nl) {
                tri_mac(e2, Yl[(b + 2) * kTermsT], A);
                p += 16;
            }
            p += 16;
#pragma unroll
            for (int i = 0; i < 4; i++)
                if (a0 + i < nl) {
                    const double4 d = i == 0 ? row_quad<0>(dg) : i == 1 ? row_quad<4>(dg)
                                    : i == 2 ? row_quad<8>(dg) : row_quad<12>(dg);
                    const double2 ya = i == 0 && a0 == 0 ? y0 : Yl[(a0 + i - 1) * kTermsT];
                    qs += terms_row(ya, d, A[i].ur, A[i].ui, A[i].vr, A[i].vi, f2, F2r, F2i);
                }
        }
    }
    terms_store(g, S, qs, tp);
}

__global__ __launch_bounds__(kTermsT) void k_terms(
    ile_geom g, const ile_sample_rec *__restrict__ rec, const int32_t *__restrict__ perm,
    const double *__restrict__ uvt, int64_t t0, int64_t n, double *__restrict__ terms)
{
    terms_samples(g, rec, perm, uvt, t0, n, terms);
}

// Many points, workgroup row y the point: a point alone leaves the chip part
// empty and its last wave's latency in the open (eight points of 1e5 samples,
// 5 to 21 modes, 213 us against 298 by a launch each).
__global__ __launch_bounds__(kTermsT) void k_terms_multi(const ile_geom *__restrict__ geoms,
                                                         const ile_point_dev *__restrict__ pts,
                                                         int64_t n)
{
    const ile_point_dev &P = pts[blockIdx.y];
    terms_samples(geoms[blockIdx.y], P.rec, P.perm, P.uvt, 0, n, P.terms);
}

static size_t terms_lds_bytes(int n_lm)
{
    return (size_t)kTermsT * (n_lm - 1) * sizeof(double2);
}

// One tile: samples perm[base .. base + TS) of a point (those below N).
template <typename TQ, int TS, int NT, int ENG, bool DUMP>
__device__ __forceinline__ void contract_tile(
    const ile_geom &g, int64_t base, const double *__restrict__ smp, int64_t N,
    const int32_t *__restrict__ perm, const int32_t *__restrict__ shifts,
    const TQ *__restrict__ Q, const double2 *__restrict__ U,
    const double2 *__restrict__ V, double *__restrict__ out,
    double *__restrict__ series)
{
    static_assert(ENG == ENG_VALU || (TS == 16 && NT % 128 == 0), "MFMA tile is 16 samples");
    static_assert(ENG != ENG_BF16 || sizeof(TQ) == 4, "BF16 engine accumulates in float");
    constexpr int NW = NT / 64;
    __shared__ __align__(16) TQ Gs[TS * NT];
    __shared__ double s_q[TS];
    __shared__ int s_idx[TS];      // sample index, -1 if the slot is empty
    __shared__ int s_ok[TS];
    __shared__ int s_d[ILE_MAX_DET][TS];
    __shared__ int s_smin[ILE_MAX_DET], s_spread[ILE_MAX_DET];
    __shared__ double s_red[NW][TS];
    __shared__ double s_M[TS];
    extern __shared__ __align__(16) unsigned char dyn_lds[];
    TQ *coef = reinterpret_cast<TQ *>(dyn_lds);

    const int tid = threadIdx.x;
    const int nd = g.n_det, nl = g.n_lm, nq = g.n_q;
    const int KSP = ksp_of(nl), RP = 4 * KSP;   // k-steps and Q rows per detector (padded)
    const int KSB = ksb_of(nl);                 // BF16 k-steps
    constexpr bool MF = ENG != ENG_VALU;        // matrix-core engines

    // prologue scratch: inside Gs when it fits, else after the coefficients
    const size_t scr_bytes = prologue_scratch_bytes(TS, nd, nl);
    double *scr = scr_bytes <= sizeof(Gs)
                      ? reinterpret_cast<double *>(Gs)
                      : reinterpret_cast<double *>(dyn_lds + coef_bytes<ENG>(TS, nd, nl, sizeof(TQ)));

    tile_prologue<TQ, TS, NT, ENG>(g, base, smp, N, perm, shifts, U, V, scr,
                                   scr == reinterpret_cast<double *>(Gs) ? sizeof(Gs) : 0,
                                   coef, s_q, s_idx, s_ok, s_d);

    // 4. per-detector window range of the tile
    if (tid < nd) {
        const int k = tid;
        int lo = 0x7fffffff, hi = -1;
        for (int al = 0; al < TS; al++)
            if (s_ok[al]) {
                lo = min(lo, s_d[k][al]);
                hi = max(hi, s_d[k][al]);
            }
        if (hi < 0) lo = hi = 0;
        s_smin[k] = lo;
        s_spread[k] = hi - lo;
    }
    __syncthreads();
    if (tid < TS)
        for (int k = 0; k < nd; k++) s_d[k][tid] = s_ok[tid] ? s_d[k][tid] - s_smin[k] : 0;
    __syncthreads();

    int smax_all = 0;
    for (int k = 0; k < nd; k++) smax_all = max(smax_all, s_spread[k]);
    // NP positions per G block: every thread for the vector engine, the
    // producer half of the workgroup for the matrix-core engine
    constexpr int NP = MF ? NT / 2 : NT;
    int J = NP - smax_all;
    if (J < 64) J = 64;

    const int lane = tid & 63, wv = tid >> 6;
    // the result of sample al: (M - q) + log S - log n_t, S = the block sum
    const auto finish_sample = [&](int al, double S) {
        if (s_idx[al] >= 0)
            out[s_idx[al]] = s_ok[al] ? (s_M[al] - s_q[al]) + log(S) - log((double)g.n_t) : NAN;
    };

    if constexpr (ENG == ENG_VALU) {
        double m[TS], sacc[TS];
#pragma unroll
        for (int al = 0; al < TS; al++) {
            m[al] = -INFINITY;
            sacc[al] = 0.0;
        }
        for (int j0 = 0; j0 < g.n_t; j0 += J) {
            const int Jc = min(J, g.n_t - j0);
            // thread tid owns the bins j == tid (mod NT); its bin in this chunk
            const int jrel = ((tid - j0) % NT + NT) % NT;
            const bool has = jrel < Jc;
            TQ L[TS];
#pragma unroll
            for (int al = 0; al < TS; al++) L[al] = (TQ)0;

            for (int k = 0; k < nd; k++) {
                const int Pk = s_smin[k] + j0;
                const int Wk = Jc + s_spread[k];
                const TQ *Qk = Q + (int64_t)k * RP * nq;
                for (int blk = 0; blk < Wk; blk += NT) {
                    const int p = blk + tid;
                    TQ acc[TS];
#pragma unroll
                    for (int al = 0; al < TS; al++) acc[al] = (TQ)0;
                    if (p < Wk) {
                        const TQ *qp = Qk + Pk + p;
                        const TQ *cf = coef + (size_t)k * nl * TS * 2;
                        TQ qnr = qp[0], qni = qp[nq];
                        for (int a = 0; a < nl; a++) {
                            const TQ qr = qnr, qi = qni;
                            // next mode's values are in flight during this mode's FMAs
                            if (a + 1 < nl) {
                                qnr = qp[(int64_t)(2 * a + 2) * nq];
                                qni = qp[(int64_t)(2 * a + 3) * nq];
                            }
                            const TQ *ca = cf + a * TS * 2;
#pragma unroll
                            for (int al = 0; al < TS; al++)
                                acc[al] = fma(ca[2 * al], qr, fma(ca[2 * al + 1], qi, acc[al]));
                        }
                    }
#pragma unroll
                    for (int al = 0; al < TS; al++) Gs[al * NT + tid] = acc[al];
                    __syncthreads();
                    if (has) {
#pragma unroll
                        for (int al = 0; al < TS; al++) {
                            const int ix = s_d[k][al] + jrel - blk;
                            const bool in = (unsigned)ix < (unsigned)NT;
                            const TQ v = Gs[al * NT + (in ? ix : 0)];
                            L[al] += in ? v : (TQ)0;
                        }
                    }
                    __syncthreads();
                }
            }
            if (has) {
                const int j = j0 + jrel;
                if (DUMP) {
                    for (int al = 0; al < TS; al++)
                        if (s_ok[al]) series[(int64_t)s_idx[al] * g.n_t + j] = (double)L[al] - s_q[al];
                }
                lse_update<TQ, TS>(L, m, sacc);
            }
        }
        lse_wave_max<TS>(m, s_red, lane, wv);
        __syncthreads();
        if (tid < TS) {
            double M = s_red[0][tid];
            for (int w = 1; w < NW; w++) M = fmax(M, s_red[w][tid]);
            s_M[tid] = M;
        }
        __syncthreads();
        lse_wave_sum<TS>(m, sacc, s_M, s_red, lane, wv);
        __syncthreads();
        if (tid < TS) {
            double S = s_red[0][tid];
            for (int w = 1; w < NW; w++) S += s_red[w][tid];
            finish_sample(tid, S);
        }
    } else {
        // Producer/consumer pipeline over the items (chunk, detector, block):
        // at step s the producer waves compute item s into Gs buffer s % 2
        // on the matrix cores while the consumer waves realign item s-1 from
        // the other buffer (and run the log-sum-exp at the end of a chunk);
        // one barrier per step.  Both iterators are advanced identically by
        // every thread, so the loop bounds are uniform.
        const bool producer = __builtin_amdgcn_readfirstlane(tid) < NP;
        static_assert(TS * NP * sizeof(double) <= sizeof(Gs), "epilogue states fit the G buffers");
        // Separate loops per role (wave-uniform branch) so that the consumer
        // state and the producer's operand buffers are never live together;
        // both loops take the same steps and meet at one barrier per step.
        PipeIt pi, ci;
        pipe_first(pi, J, g.n_t);
        pipe_first(ci, J, g.n_t);
        if (producer) {
            for (int step = 0; pi.valid || ci.valid; step++) {
                if (pi.valid) {
                    const int k = pi.k;
                    const int P0 = s_smin[k] + pi.j0 + pi.blk;
                    const int W = min(pi.Jc + s_spread[k] - pi.blk, NP);
                    if constexpr (ENG == ENG_BF16)
                        bf16_gphase<NP>(reinterpret_cast<float *>(Gs) + (step & 1) * (TS * NP),
                                        reinterpret_cast<const v8bf *>(coef) + (size_t)k * KSB * 64,
                                        reinterpret_cast<const v8bf *>(Q) + (int64_t)k * nq * 4 * KSB,
                                        nq, KSB, P0, W, lane);
                    else
                        mfma_gphase<TQ, NP>(Gs + (step & 1) * (TS * NP), coef + (size_t)k * KSP * 64,
                                            Q + (int64_t)k * RP * nq, nq, KSP, P0, W, lane);
                    pipe_next(pi, J, g.n_t, nd, s_spread, NP);
                }
                if (step > 0 && ci.valid) pipe_next(ci, J, g.n_t, nd, s_spread, NP);
                __syncthreads();
            }
            // epilogue (the consumers write R between the barriers); threads
            // tid < 16 TS reduce
            const double *R = reinterpret_cast<const double *>(Gs);
            __syncthreads();
            if (tid < 16 * TS) {
                const double M = epi_reduce<TS, NP>(R, tid, true);
                if ((tid & 15) == 0) s_M[tid >> 4] = M;
            }
            __syncthreads();
            __syncthreads();
            if (tid < 16 * TS) {
                const double S = epi_reduce<TS, NP>(R, tid, false);
                if ((tid & 15) == 0) finish_sample(tid >> 4, S);
            }
        } else {
            const int tc = tid - NP;   // consumer index
            double m[TS], sacc[TS];
#pragma unroll
            for (int al = 0; al < TS; al++) {
                m[al] = -INFINITY;
                sacc[al] = 0.0;
            }
            TQ L[TS];
#pragma unroll
            for (int al = 0; al < TS; al++) L[al] = (TQ)0;
            for (int step = 0; pi.valid || ci.valid; step++) {
                if (step > 0 && ci.valid) {
                    const TQ *G = Gs + ((step - 1) & 1) * (TS * NP);
                    const int jrel = ((tc - ci.j0) % NP + NP) % NP;
                    const bool has = jrel < ci.Jc;
                    if (has) {
#pragma unroll
                        for (int al = 0; al < TS; al++) {
                            const int ix = s_d[ci.k][al] + jrel - ci.blk;
                            const bool in = (unsigned)ix < (unsigned)NP;
                            const TQ v = G[al * NP + (in ? ix : 0)];
                            L[al] += in ? v : (TQ)0;
                        }
                    }
                    if (pipe_last_of_chunk(ci, nd, s_spread[nd - 1], NP)) {
                        if (has) {
                            const int j = ci.j0 + jrel;
                            if (DUMP) {
                                for (int al = 0; al < TS; al++)
                                    if (s_ok[al])
                                        series[(int64_t)s_idx[al] * g.n_t + j] =
                                            (double)L[al] - s_q[al];
                            }
                            lse_update<TQ, TS>(L, m, sacc);
                        }
#pragma unroll
                        for (int al = 0; al < TS; al++) L[al] = (TQ)0;
                    }
                    pipe_next(ci, J, g.n_t, nd, s_spread, NP);
                }
                if (pi.valid) pipe_next(pi, J, g.n_t, nd, s_spread, NP);
                __syncthreads();
            }
            // epilogue: the same three barriers as the producers
            double *R = reinterpret_cast<double *>(Gs);
#pragma unroll
            for (int al = 0; al < TS; al++) R[al * NP + tc] = m[al];
            __syncthreads();
            if (tid < 16 * TS) {
                const double M = epi_reduce<TS, NP>(R, tid, true);
                if ((tid & 15) == 0) s_M[tid >> 4] = M;
            }
            __syncthreads();
#pragma unroll
            for (int al = 0; al < TS; al++)
                R[al * NP + tc] = m[al] == -INFINITY ? 0.0 : sacc[al] * exp(m[al] - s_M[al]);
            __syncthreads();
            if (tid < 16 * TS) {
                const double S = epi_reduce<TS, NP>(R, tid, false);
                if ((tid & 15) == 0) finish_sample(tid >> 4, S);
            }
        }
    }
}

// ------------------------------------------------ phased matrix-core engine
// One workgroup of four waves per tile of 16 samples.  On gfx950 an FP64
// matrix-core step holds its SIMD's issue for its whole duration, so the
// vector work and the matrix work of a SIMD add up instead of overlapping.
// The tile is therefore not split into producer and consumer waves (which
// leaves the matrix work on some SIMDs and the vector work on others):
// every wave takes both roles in turn, per chunk of J bins:
//   G phase, one detector k at a time: the windowed products
//            G_k[alpha][p] = sum_r C_k[alpha][r] Qm_k[r][P_k + p] over the
//            union of the chunk's windows (P_k = smin_k + j0), as 16-wide
//            N-tiles dealt to the waves in turn, each result moved to its
//            sample's chunk bin: X[alpha][jj] with jj = p - (s_alpha,k -
//            smin_k), stored for the first detector and added for the
//            others (a barrier between detectors), so X holds the sum over
//            the detectors in ascending order;
//   L phase: lane (alpha, sub), LPS = 16 or 32 lanes per sample, owns the
//            bins j = sub (mod LPS) and folds X[alpha][j - j0] into its
//            log-sum-exp.
// X has one row of J bins per sample whatever the spread of the tile's
// window starts (which only widens the unions), so J is set by the LDS
// budget alone.
//
// Log-sum-exp with a lagging reference: each lane keeps (m, s) with
// s = sum exp(x - m) over its bins, and moves m to x only at its first bin
// or when x > m + kLseSlack, so most bins cost one exp and one add.  The
// 16 lanes of a sample are merged by a fixed tree at the end.  A sample's
// bins, their order within each lane and the merge depend neither on the
// tile it lands in nor on the chunking or the pass, and neither does its
// result.
constexpr double kLseSlack = 64.0;

// a * b + c with c a wave-uniform constant held in scalar registers.  The
// compiler's own selection turns Horner steps into a register copy of the
// constant plus an accumulating FMA (its tied operand); this form needs no
// copy.  Arithmetic only.
__device__ __forceinline__ double fma_sc(double a, double b, double c)
{
    double d;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
    return d;
}

// e^d for d <= kLseSlack, the log-sum-exp's terms: d = n ln2 + r with
// n = rint(d / ln2) and r reduced in two parts (Cody and Waite), so
// |r| <= ln2 / 2; e^r by its Taylor polynomial of degree 13 (truncation
// below 5e-18 relative); then scaled by 2^n.  Arguments below -1000 are
// clamped there (the result underflows to 0 either way), so no overflow or
// NaN test is needed.  Relative error a few ulp.
__device__ __forceinline__ double exp_lse(double d)
{
    // d is never NaN here, so the clamp needs no canonicalization
    asm("v_max_f64 %0, %1, %2" : "=v"(d) : "v"(d), "s"(-1000.0));
    const double n = rint(d * 1.4426950408889634074);
    const double r = fma(-n, 1.9082149292705877000e-10, fma(-n, 6.9314718036912381649e-1, d));
    double p = fma_sc(r, 1.0 / 6227020800.0, 1.0 / 479001600.0);   // 1/13!, 1/12!
    p = fma_sc(p, r, 1.0 / 39916800.0);
    p = fma_sc(p, r, 1.0 / 3628800.0);
    p = fma_sc(p, r, 1.0 / 362880.0);
    p = fma_sc(p, r, 1.0 / 40320.0);
    p = fma_sc(p, r, 1.0 / 5040.0);
    p = fma_sc(p, r, 1.0 / 720.0);
    p = fma_sc(p, r, 1.0 / 120.0);
    p = fma_sc(p, r, 1.0 / 24.0);
    p = fma_sc(p, r, 1.0 / 6.0);
    p = fma(p, r, 0.5);
    p = fma(p, r, 1.0);
    p = fma(p, r, 1.0);
    return ldexp(p, (int)n);
}

template <typename TQ> struct qload;
template <> struct qload<double> {
    static __device__ inline double ld(__amdgpu_buffer_rsrc_t r, int vo, int so)
    {
        typedef unsigned int u2 __attribute__((ext_vector_type(2)));
        const u2 v = __builtin_amdgcn_raw_buffer_load_b64(r, vo, so, 0);
        return __builtin_bit_cast(double, v);
    }
};
template <> struct qload<float> {
    static __device__ inline float ld(__amdgpu_buffer_rsrc_t r, int vo, int so)
    {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, vo, so, 0));
    }
};

// Buffer resource over one detector's Q rows (raw bytes, gfx9 word 3).
template <typename TQ>
__device__ inline __amdgpu_buffer_rsrc_t q_rsrc(const TQ *Qk, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<TQ *>(Qk), (short)0, bytes, 0x00020000);
}

template <typename TQ> struct lds_ptr {
    using type = __attribute__((address_space(3))) TQ;
    static __device__ inline int addr(const TQ *p)
    {
        return (int)(unsigned)(uintptr_t)(type *)const_cast<TQ *>(p);
    }
    static __device__ inline type *at(int a) { return (type *)(uintptr_t)(unsigned)a; }
};

__device__ __forceinline__ int med3(int x, int lo, int hi)
{
    int d;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(d) : "v"(x), "v"(lo), "v"(hi));
    return d;
}

// The products of NU N-tiles tb, tb + NW, ... of one detector, computed
// together so that NU accumulations are in flight: lane l supplies
// A[l%16][l/16] (the detector's coefficients, LDS; one read per k-step serves
// all NU tiles) and B[l/16][l%16] = Qm_k[4 ks + l/16][P + 16 t + l%16] by
// buffer loads, the lane's offset in a VGPR and the k-step's in an SGPR, so a
// load costs no vector instruction.  Columns past the end of Q are clamped
// (past every sample's window: never moved to a bin).  Operands are
// double-buffered: the loads of k-step ks + 1 are issued before the products
// of k-step ks; the first k-step's products take the zero of their
// accumulators as a constant.
template <typename TQ, int NU, int NW>
__device__ __forceinline__ void ph_products(typename mfma_acc<TQ>::type (&acc)[NU],
                                            const TQ *coefk, __amdgpu_buffer_rsrc_t rs,
                                            int qrow0, int nq, int KSP, int P, int tb, int lane)
{
    using M = mfma_acc<TQ>;
    const int rb = (qrow0 + (lane >> 4)) * nq, p = P + 16 * tb + (lane & 15);
    int vo[NU];
#pragma unroll
    for (int u = 0; u < NU; u++) vo[u] = (rb + min(p + 16 * NW * u, nq - 1)) * (int)sizeof(TQ);
    const int kstep = 4 * nq * (int)sizeof(TQ);
    TQ a0 = coefk[lane], a1, b0[NU], b1[NU];
#pragma unroll
    for (int u = 0; u < NU; u++) b0[u] = qload<TQ>::ld(rs, vo[u], 0);
    // k-steps in pairs with every load and product unconditional (a load
    // under a branch is sunk next to its use); an odd last step follows
    const auto load = [&](TQ &a, TQ (&b)[NU], int ks) {
        const int kc = min(ks, KSP - 1);
        a = coefk[kc * 64 + lane];
#pragma unroll
        for (int u = 0; u < NU; u++) b[u] = qload<TQ>::ld(rs, vo[u], kc * kstep);
        __builtin_amdgcn_sched_barrier(0);
    };
    const auto step = [&](TQ a, const TQ (&b)[NU]) {
#pragma unroll
        for (int u = 0; u < NU; u++) acc[u] = M::step(a, b[u], acc[u]);
        __builtin_amdgcn_sched_barrier(0);
    };
    load(a1, b1, 1);
#pragma unroll
    for (int u = 0; u < NU; u++) acc[u] = M::step(a0, b0[u], typename M::type{0, 0, 0, 0});
    __builtin_amdgcn_sched_barrier(0);
    if (KSP == 1) return;
    load(a0, b0, 2);
    step(a1, b1);
    int ks = 2;
    for (; ks + 1 < KSP; ks += 2) {
        load(a1, b1, ks + 1);
        step(a0, b0);
        load(a0, b0, ks + 2);
        step(a1, b1);
    }
    if (ks < KSP) step(a0, b0);
}

// Where a lane's results of one detector go: result v of tile t belongs at
// LDS byte xb[v] + 16 t elements, its sample's bin 16 t + c - dd (dd the
// sample's window start minus the detector's smallest); lo[v] is the slot
// before the sample's first bin.
struct ph_row {
    int xb[4], lo[4];
};

// e^d where the reference moves, kept out of line: inlined, its constants are
// held in some twenty vector registers across the whole tile (FP64 119 against
// 100, and FP32 tiles then spill below the 85 that three workgroups per CU
// leave: 0.805 against 0.774 ms on 2e5 samples, 13 modes, 1103 bins).
__device__ __attribute__((noinline)) double exp_rescale(double d) { return exp(d); }

// The group's results to their samples' bins: stored when `add` is false,
// else added.  Each (alpha, bin) comes from exactly one lane of one tile.  A
// tile whose every result has a bin in the chunk (16 t >= spread, 16 t + 15 <
// Jc) takes its addresses by constant offsets; in the others a result
// outside the chunk is held to the slot just before or just past its row's
// bins (cb bytes after lo), which is never read as a bin: one add and one
// med3 in place of the add, compare, select and shift of a bounds test.
template <typename TQ, int NU, int NW>
__device__ __forceinline__ void ph_store(const typename mfma_acc<TQ>::type (&acc)[NU],
                                         const ph_row &R, int cb, int tb, int spread, int Jc,
                                         bool add)
{
    using P = lds_ptr<TQ>;
    constexpr int TB = 16 * (int)sizeof(TQ);
    int base[4];
#pragma unroll
    for (int v = 0; v < 4; v++) base[v] = R.xb[v] + tb * TB;
#pragma unroll
    for (int u = 0; u < NU; u++) {
        const auto put = [&](auto at) {
            if (add) {
                TQ o[4];
#pragma unroll
                for (int v = 0; v < 4; v++) o[v] = *at(v);
#pragma unroll
                for (int v = 0; v < 4; v++) *at(v) = o[v] + (TQ)acc[u][v];
            } else {
#pragma unroll
                for (int v = 0; v < 4; v++) *at(v) = (TQ)acc[u][v];
            }
        };
        const int c0 = 16 * (tb + u * NW);
        if (c0 >= spread && c0 + 15 < Jc) {
            put([&](int v) { return P::at(base[v] + u * NW * TB); });
        } else {
            int a[4];
#pragma unroll
            for (int v = 0; v < 4; v++)
                a[v] = med3(base[v] + u * NW * TB, R.lo[v], R.lo[v] + cb);
            put([&](int v) { return P::at(a[v]); });
        }
    }
}

// LDS of the phased tile beyond its static arrays: coefficients
// [nd][KSP][64], then 16 bytes (the slot before the first row's first bin)
// and the chunk bins X [TS][xrow], the last of a row's xrow elements being the
// slot past its bins (a tile that forms its own terms has their scratch there
// first).
__host__ __device__ inline size_t ph_dyn_bytes(int ts, int nd, int nl, int wrow, size_t e)
{
    const size_t gb = (size_t)ts * wrow * e + 16;
    const size_t sb = prologue_scratch_bytes(ts, nd, nl);
    return coef_bytes<ENG_MFMA>(ts, nd, nl, e) + (gb > sb ? gb : sb);
}

// L phase of one chunk for one lane of the phased tile: the chunk's bins
// j0 + i, i = o, o + LPS, o + 2 LPS, ... < Jc, of its sample (o chosen by
// the caller so that the lane owns the bins j = sub (mod LPS) whatever the
// chunking), x = X[i] (the sum over the detectors), folded into the lane's
// log-sum-exp (m, s).  srow: the sample's series row at bin j0 when the
// per-bin values are wanted (minus q), else null.
template <typename TQ, int LPS, bool DUMP>
__device__ __forceinline__ void ph_lphase(const TQ *X, int Jc, int o, double &m, double &ssum,
                                          double *srow, double q)
{
    const auto xval = [&](int i) {
        const double x = (double)X[i];
        if (DUMP) srow[i] = x - q;
        return x;
    };
    // the terms e^d: FP64 tiles by exp_lse; FP32 tiles, whose bin values
    // carry FP32 rounding already, by the single-precision exponential (its
    // relative error, a few 1e-8, is below that of the values; the sums and
    // the reference stay FP64)
    const auto ex = [](double d) -> double {
        if constexpr (sizeof(TQ) == 4) return (double)expf((float)d);
        else return exp_lse(d);
    };
    const auto fold = [&](double x) {
        double d = x - m;
        if (d > kLseSlack) {
            ssum = m == -INFINITY ? 0.0 : ssum * exp_rescale(m - x);
            m = x;
            d = 0.0;
        }
        ssum += ex(d);
    };
    // two bins at a time: when neither moves the reference, their exps are
    // independent (the sums are still taken in bin order, as fold would)
    int i = o;
    for (; i + LPS < Jc; i += 2 * LPS) {
        const double x0 = xval(i), x1 = xval(i + LPS);
        const double d0 = x0 - m, d1 = x1 - m;
        if (d0 > kLseSlack || d1 > kLseSlack) {
            fold(x0);
            fold(x1);
        } else {
            const double e0 = ex(d0), e1 = ex(d1);
            ssum += e0;
            ssum += e1;
        }
    }
    if (i < Jc) fold(xval(i));
}

// PRE: the per-sample terms come from k_terms (the tile's block of the
// terms, tile-major from position t0; smp, shifts, U and V are null), else the
// tile forms them (tile_prologue).
// What bounds it: the FP64 matrix steps themselves (a variant without stores
// and log-sum-exp runs its chunks at the matrix rate, 0.82 ms per chunk of 463
// bins for 5e5 samples at 3 detectors and 21 modes), then, since they do not
// overlap them, the vector instructions of the stores and of the log-sum-exp,
// and the prologue's latency (one workgroup of the two on a CU waits in it).
// Stores by constant offsets or med3, the zero accumulators as a constant and
// the prologue in one round of loads (windows relative to the tile already
// in the terms) took a 1e6-sample call from 11.01 to 10.37 ms, and 2e5 FP32
// samples (13 modes, 1103 bins) from 0.835 to 0.743 ms.
template <typename TQ, int TS, int NT, bool DUMP, bool PRE>
__device__ __forceinline__ void contract_tile_ph(
    const ile_geom &g, int64_t base, const double *__restrict__ smp, int64_t N,
    const int32_t *__restrict__ perm, const int32_t *__restrict__ shifts,
    const TQ *__restrict__ Q, const double2 *__restrict__ U,
    const double2 *__restrict__ V, const double *__restrict__ terms, int64_t t0,
    double *__restrict__ out, double *__restrict__ series)
{
    static_assert(TS == 16 && (NT == 256 || NT == 512), "phased tile: 16 samples, 4 or 8 waves");
    constexpr int NW = NT / 64;    // waves
    constexpr int LPS = NT / TS;   // lanes per sample in the L phase
    __shared__ double s_q[TS];
    __shared__ int s_idx[TS], s_ok[TS];
    __shared__ int s_d[ILE_MAX_DET][TS];
    __shared__ int s_smin[ILE_MAX_DET], s_spread[ILE_MAX_DET];
    extern __shared__ __align__(16) unsigned char dyn_lds[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nd = g.n_det, nl = g.n_lm, nq = g.n_q, n_t = g.n_t;
    const int KSP = ksp_of(nl), RP = 4 * KSP;
    const int wcap = g.wcap, wrow = g.wrow;
    TQ *coef = reinterpret_cast<TQ *>(dyn_lds);   // [nd][KSP][64]
    TQ *G = reinterpret_cast<TQ *>(dyn_lds + coef_bytes<ENG_MFMA>(TS, nd, nl, sizeof(TQ)));
    // one buffer resource over all of Q (the host keeps it below 2 GiB)
    const __amdgpu_buffer_rsrc_t rs = q_rsrc<TQ>(Q, nd * RP * nq * (int)sizeof(TQ));

    if constexpr (PRE) {
        // one round of loads: samples, validity, windows and q of the tile,
        // and the factors of the coefficients c = (d_ref/D) F_k Y_lm, written
        // in the matrix-core A layout (modes a in [nl, 2 KSP) are the zero
        // padding of K)
        const double *tb = terms + ((base - t0) >> 4) * (16 * (int64_t)terms_fields(nd, nl));
        const int2 *tw = reinterpret_cast<const int2 *>(tb + (2 + 2 * nd + 2 * nl) * TS);
        if (tid < TS) {
            const int64_t i = base + tid;
            s_idx[tid] = i < N ? perm[i] : -1;
            s_ok[tid] = tb[TS + tid] != 0.0;
            s_q[tid] = tb[tid];
        } else if (tid >= 64 && tid < 64 + TS * nd) {
            const int t = tid - 64;
            const int2 w = tw[t];
            s_d[t / TS][t % TS] = w.x;
            if (t % TS == 0) s_smin[t / TS] = w.y;
            if (t % TS == 1) s_spread[t / TS] = w.y;
        }
        for (int t = tid; t < TS * 2 * KSP; t += NT) {
            const int al = t % TS, a = t / TS;
            // every load unconditional, so that they are one round
            const double *yp = tb + (2 + 2 * nd + 2 * min(a, nl - 1)) * TS + al;
            double yr = yp[0], yi = yp[TS], fr[ILE_MAX_DET], fi[ILE_MAX_DET];
#pragma unroll
            for (int k = 0; k < ILE_MAX_DET; k++) {
                const double *fp = tb + (2 + 2 * min(k, nd - 1)) * TS + al;
                fr[k] = fp[0];
                fi[k] = fp[TS];
            }
            if (a >= nl) yr = yi = 0.0;
            TQ *ca = coef + (a >> 1) * 64 + (a & 1) * 32 + al;
#pragma unroll
            for (int k = 0; k < ILE_MAX_DET; k++)
                if (k < nd) {
                    ca[k * KSP * 64] = (TQ)fma(fr[k], yr, -(fi[k] * yi));
                    ca[k * KSP * 64 + 16] = (TQ)fma(fi[k], yr, fr[k] * yi);
                }
        }
        __syncthreads();
    } else {
        const size_t gbytes = (size_t)TS * wrow * sizeof(TQ);
        const size_t sbytes = prologue_scratch_bytes(TS, nd, nl);
        tile_prologue<TQ, TS, NT, ENG_MFMA>(g, base, smp, N, perm, shifts, U, V,
                                            reinterpret_cast<double *>(G),
                                            gbytes > sbytes ? gbytes : sbytes, coef, s_q,
                                            s_idx, s_ok, s_d);
    }

    // window range of each detector over the tile's valid samples, the
    // windows then relative to its start
    if (!PRE) {
        if (tid < TS) {
            const bool v = s_ok[tid];
            for (int k = 0; k < nd; k++) {
                int lo = v ? s_d[k][tid] : 0x7fffffff, hi = v ? s_d[k][tid] : -1;
                for (int off = 8; off > 0; off >>= 1) {
                    lo = min(lo, __shfl_xor(lo, off, 16));
                    hi = max(hi, __shfl_xor(hi, off, 16));
                }
                if (tid == 0) {
                    s_smin[k] = hi >= 0 ? lo : 0;
                    s_spread[k] = hi >= 0 ? hi - lo : 0;
                }
                s_d[k][tid] = v ? s_d[k][tid] - lo : 0;
            }
        }
        __syncthreads();
    }

    using MA = mfma_acc<TQ>;
    const int al = tid / LPS, sub = tid % LPS, row = lane >> 4, col = lane & 15;
    const bool mem = s_ok[al];
    TQ *X = G + 16 / sizeof(TQ);   // [TS][wrow], the chunk's bins of every sample
    const int xaddr = (int)lds_ptr<TQ>::addr(X);
    double m = -INFINITY, ssum = 0.0;
    const int J = wcap;   // below wrow: the slot after a row's last bin is free
    for (int j0 = 0; j0 < n_t; j0 += J) {
        const int Jc = min(J, n_t - j0);
        // G phase, detector by detector: N-tiles wv, wv + NW, ..., four at
        // a time
        for (int k = 0; k < nd; k++) {
            const int smin = __builtin_amdgcn_readfirstlane(s_smin[k]);
            const int spread = __builtin_amdgcn_readfirstlane(s_spread[k]);
            const int T = (Jc + spread + 15) >> 4;
            ph_row R;
#pragma unroll
            for (int v = 0; v < 4; v++) {
                const int r = MA::row(row, v);
                R.lo[v] = xaddr + (r * wrow - 1) * (int)sizeof(TQ);
                R.xb[v] = R.lo[v] + (1 + col - s_d[k][r]) * (int)sizeof(TQ);
            }
            const TQ *coefk = coef + k * KSP * 64;
            const auto group = [&](auto NUc, int tb) {
                constexpr int NU = decltype(NUc)::value;
                typename MA::type acc[NU];
                ph_products<TQ, NU, NW>(acc, coefk, rs, k * RP, nq, KSP, smin + j0, tb, lane);
                ph_store<TQ, NU, NW>(acc, R, (Jc + 1) * (int)sizeof(TQ), tb, spread, Jc, k > 0);
            };
            for (int tb = wv; tb < T; tb += 4 * NW) {
                switch (min(4, (T - tb + NW - 1) / NW)) {
                case 4: group(std::integral_constant<int, 4>{}, tb); break;
                case 3: group(std::integral_constant<int, 3>{}, tb); break;
                case 2: group(std::integral_constant<int, 2>{}, tb); break;
                default: group(std::integral_constant<int, 1>{}, tb); break;
                }
            }
            __syncthreads();
        }
        // L phase
        if (mem) {
            double *srow = DUMP ? series + (int64_t)s_idx[al] * n_t + j0 : nullptr;
            const int o = (sub - j0) & (LPS - 1);   // first bin j = sub (mod LPS)
            ph_lphase<TQ, LPS, DUMP>(X + al * wrow, Jc, o, m, ssum, srow, s_q[al]);
        }
        __syncthreads();
    }
    // merge the LPS lanes of each sample (fixed tree: 16-lane rows, then the
    // row pair), then the result (M - q) + log S - log n_t
    double M = row_max64(m);
    if (LPS == 32) M = fmax(M, __shfl_xor(M, 16));
    double S = row_sum64(m == -INFINITY ? 0.0 : ssum * exp(m - M));
    if (LPS == 32) S += __shfl_xor(S, 16);
    if (sub == 0 && s_idx[al] >= 0)
        out[s_idx[al]] = s_ok[al] ? (M - s_q[al]) + log(S) - log((double)n_t) : NAN;
}

// Waves per SIMD the register allocation must allow (the second bound of
// __launch_bounds__): the eight-wave phased workgroups per CU that their LDS
// admits, two for FP64 and three for FP32, are four and six waves per SIMD
// (tiles that form the per-sample terms themselves need more registers than
// six waves leave).
template <typename TQ, int NT, bool PRE> constexpr int ph_min_waves()
{
    return NT == 512 ? (sizeof(TQ) == 4 && PRE ? 6 : 4) : 1;
}

template <typename TQ, int TS, int NT, int ENG, bool DUMP>
__global__ __launch_bounds__(NT, 1) void k_contract(
    ile_geom g, const double *__restrict__ smp, int64_t N,
    const int32_t *__restrict__ perm, const int32_t *__restrict__ shifts,
    const TQ *__restrict__ Q, const double2 *__restrict__ U,
    const double2 *__restrict__ V, double *__restrict__ out,
    double *__restrict__ series)
{
    contract_tile<TQ, TS, NT, ENG, DUMP>(g, (int64_t)blockIdx.x * TS, smp, N, perm, shifts, Q, U,
                                         V, out, series);
}

// Persistent form over many intrinsic points: every workgroup takes
// (point, tile) items from a queue in list order (the host sorts the list by
// decreasing cost) until it is empty; every wave reaches the exit.
template <typename TQ, int TS, int NT, int ENG>
__global__ __launch_bounds__(NT, 1) void k_contract_batched(
    const ile_geom *__restrict__ geoms, const ile_point_dev *__restrict__ pts,
    const int2 *__restrict__ items, int n_items, unsigned *counter)
{
    __shared__ int s_item;
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) s_item = (int)atomicAdd(counter, 1u);
        __syncthreads();
        // uniform, so the point's parameters load through the scalar unit
        const int it = __builtin_amdgcn_readfirstlane(s_item);
        if (it >= n_items) break;
        const int2 w = items[it];
        const ile_point_dev &P = pts[w.x];
        contract_tile<TQ, TS, NT, ENG, false>(geoms[w.x], (int64_t)w.y * TS, P.smp, P.N, P.perm,
                                              P.shifts, (const TQ *)P.Q, P.U, P.V, P.out, nullptr);
    }
}

// Many intrinsic points on the phased engine: one workgroup per (point,
// tile) item, in list order (the host sorts the list by decreasing cost and
// the dispatcher starts workgroups in that order).  PRE: every point carries
// its per-sample terms; else the tiles form them.  Not persistent: every
// load of the point's parameters precedes the kernel's only store, so they
// are read through the scalar unit instead of being held in registers
// across a queue loop.
template <typename TQ, int TS, int NT, bool PRE>
__global__ __launch_bounds__(NT, (ph_min_waves<TQ, NT, PRE>())) void k_contract_items(
    const ile_geom *__restrict__ geoms, const ile_point_dev *__restrict__ pts,
    const int2 *__restrict__ items)
{
    const int2 w = items[blockIdx.x];
    const ile_point_dev &P = pts[w.x];
    if (PRE)
        contract_tile_ph<TQ, TS, NT, false, true>(geoms[w.x], (int64_t)w.y * TS, nullptr, P.N,
                                                  P.perm, nullptr, (const TQ *)P.Q, nullptr,
                                                  nullptr, P.terms, 0, P.out, nullptr);
    else
        contract_tile_ph<TQ, TS, NT, false, false>(geoms[w.x], (int64_t)w.y * TS, P.smp, P.N,
                                                   P.perm, P.shifts, (const TQ *)P.Q, P.U, P.V,
                                                   nullptr, 0, P.out, nullptr);
}

// One point on the phased engine with its per-sample terms precomputed:
// tiles of tile positions t0 + 16 blockIdx.x .. (below N), their terms
// tile-major from position t0.
template <typename TQ, int NT, bool DUMP>
__global__ __launch_bounds__(NT, (ph_min_waves<TQ, NT, true>())) void k_contract_ph(
    ile_geom g, int64_t N, const int32_t *__restrict__ perm, const TQ *__restrict__ Q,
    const double *__restrict__ terms, int64_t t0, double *__restrict__ out,
    double *__restrict__ series)
{
    contract_tile_ph<TQ, 16, NT, DUMP, true>(g, t0 + (int64_t)blockIdx.x * 16, nullptr, N, perm,
                                             nullptr, Q, nullptr, nullptr, terms, t0, out,
                                             series);
}

// --------------------------------------------------------------- prior
using ile_rng::u53;

__global__ __launch_bounds__(256) void k_prior(uint64_t seed, int64_t first,
                                               int64_t N, double d_min,
                                               double d_max, double t_ref_max,
                                               double *smp, int64_t ld,
                                               double *ln_p)
{
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= N) return;
    const uint64_t i = (uint64_t)(first + t);
    uint32_t w[16];
    ile_rng::prior_words(seed, i, w);
    {
#pragma clang fp contract(off)
    const double v3 = d_max * d_max * d_max - d_min * d_min * d_min;
    const double ra = 2.0 * kPi * u53(w[0], w[1]);
    const double dec = asin(2.0 * u53(w[2], w[3]) - 1.0);
    const double psi = kPi * u53(w[4], w[5]);
    const double phi = 2.0 * kPi * u53(w[6], w[7]);
    const double ci = 2.0 * u53(w[8], w[9]) - 1.0;
    const double D = cbrt(d_min * d_min * d_min + u53(w[10], w[11]) * v3);
    const double tr = t_ref_max * (2.0 * u53(w[12], w[13]) - 1.0);
    smp[0 * ld + t] = ra;
    smp[1 * ld + t] = dec;
    smp[2 * ld + t] = psi;
    smp[3 * ld + t] = phi;
    smp[4 * ld + t] = ci;
    smp[5 * ld + t] = D;
    smp[6 * ld + t] = tr;
    if (ln_p)
        ln_p[t] = -log(kTwoPi) + log(cos(dec) / 2.0) - log(kPi) - log(kTwoPi) -
                  log(2.0) + log(3.0 * D * D / v3) - log(2.0 * t_ref_max);
    }
}

// ------------------------------------------------------------- reduction
constexpr int kRedBlocks = 256;
constexpr int kRedT = 256;

__device__ inline double lnw_at(const double *lnL, const double *lp,
                                const double *lq, int64_t i)
{
    return lnL[i] + (lp ? lp[i] : 0.0) - (lq ? lq[i] : 0.0);
}

// Partials merged in order, then their result: one thread.
__device__ inline void finish_parts(const double *parts, int n_part, double *res)
{
    double M = -INFINITY, ML = -INFINITY, n = 0.0;
    for (int i = 0; i < n_part; i++) {
        M = fmax(M, parts[5 * i]);
        ML = fmax(ML, parts[5 * i + 4]);
        n += parts[5 * i + 3];
    }
    double S1 = 0.0, S2 = 0.0;
    if (M != -INFINITY)
        for (int i = 0; i < n_part; i++) {
            if (parts[5 * i] == -INFINITY) continue;
            const double e = exp(parts[5 * i] - M);
            S1 = fma(parts[5 * i + 1], e, S1);
            S2 = fma(parts[5 * i + 2] * e, e, S2);
        }
    finish_one(M, S1, S2, n, ML, res);
}

// The partial (M, S1, S2, N, maxL) at partial and, if res, the result of the
// n_part partials at parts (partial the last of them): one thread.
__device__ inline void put_partial(double M, double S1, double S2, int64_t N, double ML,
                                   double *partial, const double *parts, int n_part, double *res)
{
    partial[0] = M;
    partial[1] = S1;
    partial[2] = S2;
    partial[3] = (double)N;
    partial[4] = ML;
    if (res && n_part == 1) finish_one(M, S1, S2, (double)N, ML, res);
    else if (res) finish_parts(parts, n_part, res);
}

// Three kernels for many samples, the last also the result: 13 us at 1e5, where
// every workgroup took the largest of the 256 maxima in one thread and the
// result another kernel: 21.
__global__ __launch_bounds__(kRedT) void k_red_max(const double *__restrict__ lnL,
                                                   const double *__restrict__ lp,
                                                   const double *__restrict__ lq, int64_t N,
                                                   double *__restrict__ tmp)
{
    __shared__ double sm[kRedT / 64], sl[kRedT / 64];
    double M = -INFINITY, ML = -INFINITY;
    for (int64_t i = (int64_t)blockIdx.x * kRedT + threadIdx.x; i < N;
         i += (int64_t)kRedBlocks * kRedT) {
        double w = lnw_at(lnL, lp, lq, i);
        M = w > M ? w : M;
        ML = lnL[i] > ML ? lnL[i] : ML;
    }
    M = wave_max(M);
    ML = wave_max(ML);
    if ((threadIdx.x & 63) == 0) {
        sm[threadIdx.x >> 6] = M;
        sl[threadIdx.x >> 6] = ML;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kRedT / 64; w++) {
            M = fmax(M, sm[w]);
            ML = fmax(ML, sl[w]);
        }
        tmp[blockIdx.x] = M;
        tmp[kRedBlocks + blockIdx.x] = ML;
    }
}

// Largest of the kRedBlocks = kRedT values v, in every thread.
__device__ inline double global_max(const double *v)
{
    static_assert(kRedBlocks == kRedT, "a value a thread");
    __shared__ double sm[kRedT / 64];
    const double x = wave_max(v[threadIdx.x]);
    __syncthreads();   // sm may still be read
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = x;
    __syncthreads();
    double M = sm[0];
    for (int w = 1; w < kRedT / 64; w++) M = fmax(M, sm[w]);
    return M;
}

__global__ __launch_bounds__(kRedT) void k_red_sum(const double *lnL,
                                                   const double *lp,
                                                   const double *lq, int64_t N,
                                                   double *tmp)
{
    __shared__ double sm[2][kRedT];
    const double M = global_max(tmp);
    double s[2] = {0.0, 0.0};
    if (M != -INFINITY) {
        for (int64_t i = (int64_t)blockIdx.x * kRedT + threadIdx.x; i < N;
             i += (int64_t)kRedBlocks * kRedT) {
            const double e = exp(lnw_at(lnL, lp, lq, i) - M);
            s[0] += e;
            s[1] = fma(e, e, s[1]);
        }
    }
    tree_sum<kRedT, 2>(s, sm);
    if (threadIdx.x == 0) {
        tmp[2 * kRedBlocks + blockIdx.x] = s[0];
        tmp[3 * kRedBlocks + blockIdx.x] = s[1];
    }
}

__global__ __launch_bounds__(kRedT) void k_red_final(const double *tmp, int64_t N,
                                                     double *partial, const double *parts,
                                                     int n_part, double *res)
{
    __shared__ double sm[2][kRedT];
    const int t = threadIdx.x;
    double s[2] = {tmp[2 * kRedBlocks + t], tmp[3 * kRedBlocks + t]};
    const double M = global_max(tmp), ML = global_max(tmp + kRedBlocks);
    tree_sum<kRedT, 2>(s, sm);
    if (t == 0) put_partial(M, s[0], s[1], N, ML, partial, parts, n_part, res);
}

// The same partial from one workgroup when N is small (at most
// kRedSmallMax): the three kernels above cost more in launches and in their
// mostly idle blocks than the work.  Same quantities, its own summation tree.
// A thread's PER values are loaded at once and kept, and the result follows
// from the same kernel: 1e4 samples 12 us, most of it the one CU's loads, where
// a loop over the values, twice, took 13 and the result another kernel of 4.
constexpr int kRedSmallT = 1024;
constexpr int64_t kRedSmallMax = 16384;

template <int PER>
__global__ __launch_bounds__(kRedSmallT) void k_red_small(const double *__restrict__ lnL,
                                                          const double *__restrict__ lp,
                                                          const double *__restrict__ lq, int N,
                                                          double *partial, const double *parts,
                                                          int n_part, double *res)
{
    __shared__ double sm[2][kRedSmallT];
    const int t = threadIdx.x;
    double M = -INFINITY, ML = -INFINITY, w[PER], l[PER];
#pragma unroll
    for (int j = 0; j < PER; j++) w[j] = l[j] = -INFINITY;
    if (N > 0) {
        // array by array: a thread's loads of each are in flight together (under
        // a test of lp or lq of their own they would be waited for one by one)
        const auto at = [&](int j) { return min(t + kRedSmallT * j, N - 1); };
        double x[PER];
#pragma unroll
        for (int j = 0; j < PER; j++) l[j] = lnL[at(j)];
#pragma unroll
        for (int j = 0; j < PER; j++) x[j] = 0.0;
        if (lp)
#pragma unroll
            for (int j = 0; j < PER; j++) x[j] = lp[at(j)];
#pragma unroll
        for (int j = 0; j < PER; j++) w[j] = l[j] + x[j];
#pragma unroll
        for (int j = 0; j < PER; j++) x[j] = 0.0;
        if (lq)
#pragma unroll
            for (int j = 0; j < PER; j++) x[j] = lq[at(j)];
#pragma unroll
        for (int j = 0; j < PER; j++) w[j] -= x[j];
    }
#pragma unroll
    for (int j = 0; j < PER; j++) {   // (a value met twice leaves the largest as it is)
        M = w[j] > M ? w[j] : M;
        ML = l[j] > ML ? l[j] : ML;
    }
    M = wave_max(M);
    ML = wave_max(ML);
    if ((t & 63) == 0) {
        sm[0][t >> 6] = M;
        sm[1][t >> 6] = ML;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kRedSmallT / 64; q++) {
        M = fmax(M, sm[0][q]);
        ML = fmax(ML, sm[1][q]);
    }
    __syncthreads();
    double s[2] = {0.0, 0.0};
    if (M != -INFINITY) {
#pragma unroll
        for (int j = 0; j < PER; j++)
            if (t + kRedSmallT * j < N) {
                const double e = exp(w[j] - M);
                s[0] += e;
                s[1] = fma(e, e, s[1]);
            }
    }
    tree_sum<kRedSmallT, 2>(s, sm);
    if (t == 0) put_partial(M, s[0], s[1], N, ML, partial, parts, n_part, res);
}

// The error flag and the result fields to pinned host memory (the flag's
// word, then six doubles from its second): one launch before the wait of a
// call, where two copies took their own.
__global__ void k_fetch(const int32_t *__restrict__ flag, const double *__restrict__ res,
                        double *__restrict__ host)
{
    const int t = threadIdx.x;
    if (t == 0 && flag) *reinterpret_cast<int32_t *>(host) = flag[0] | flag[1];
    if (t >= 1 && t <= 6 && res) host[t] = res[t - 1];
}

inline unsigned nblk(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

template <typename TQ, int TS, int NT, int ENG>
hipError_t launch_contract_t(const ile_geom &g, const double *smp, int64_t N,
                             const int32_t *perm, const int32_t *shifts,
                             const void *Q, const double *U, const double *V,
                             double *out, double *series, hipStream_t st)
{
    size_t dyn = coef_bytes<ENG>(TS, g.n_det, g.n_lm, sizeof(TQ));
    const size_t scr = prologue_scratch_bytes(TS, g.n_det, g.n_lm);
    if (scr > (size_t)TS * NT * sizeof(TQ)) dyn += scr;
    const unsigned grid = nblk(N, TS);
    if (series)
        hipLaunchKernelGGL((k_contract<TQ, TS, NT, ENG, true>), dim3(grid), dim3(NT), dyn, st,
                           g, smp, N, perm, shifts, (const TQ *)Q,
                           (const double2 *)U, (const double2 *)V, out, series);
    else
        hipLaunchKernelGGL((k_contract<TQ, TS, NT, ENG, false>), dim3(grid), dim3(NT), dyn, st,
                           g, smp, N, perm, shifts, (const TQ *)Q,
                           (const double2 *)U, (const double2 *)V, out, series);
    return hipGetLastError();
}

// LDS row stride of the phased engine's bin rows, one more than the bins of a
// chunk: the largest that keeps the coefficients and the rows within `budget`
// bytes, an odd multiple of 128 bytes (the unit) so that rows of neighbouring
// samples start in alternate halves of the 256-byte bank period.  One unit
// where the budget leaves less than that (the device's limit then decides),
// 0 where the coefficients leave nothing.
int ph_wrow(int nd, int nl, size_t e, size_t budget)
{
    const size_t fixed = coef_bytes<ENG_MFMA>(16, nd, nl, e) + 16;   // + the slot past X
    if (budget <= fixed) return 0;
    const int unit = (int)(128 / e);
    const int w = (int)((budget - fixed) / ((size_t)16 * e));
    return unit * (std::max(w / unit - 1, 0) / 2 * 2 + 1);
}

// Default LDS budgets of a phased workgroup: FP64 tiles hold four waves per
// SIMD in registers, two workgroups per CU; FP32 tiles need fewer registers
// and run three per CU.
constexpr size_t kPhBudget64 = 78 * 1024;
constexpr size_t kPhBudget32 = 50 * 1024;

static hipError_t launch_terms(const ile_geom &g, const ile_sample_rec *rec,
                               const int32_t *perm, const double *uvt, int64_t t0, int64_t n,
                               double *terms, hipStream_t st)
{
    hipLaunchKernelGGL(k_terms, dim3(nblk(n, kTermsT)), dim3(kTermsT), terms_lds_bytes(g.n_lm), st,
                       g, rec, perm, uvt, t0, n, terms);
    return hipGetLastError();
}

// Raises kernel fn's dynamic LDS limit on the current device to at least
// dyn bytes (never lowers it: another thread may launch with a larger
// size).  allowed: the kernel's per-device record of what was set.
static hipError_t allow_dyn_lds(const void *fn, size_t dyn, size_t (&allowed)[64])
{
    static std::mutex mu;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(mu);
    if (dyn <= allowed[dev]) return hipSuccess;
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn);
    if (e == hipSuccess) allowed[dev] = dyn;
    return e;
}

template <typename TQ, int NT, bool DUMP>
hipError_t launch_contract_ph(const ile_geom &g, int64_t N, const int32_t *perm,
                              const ile_sample_rec *rec, const void *Q, const double *uvt,
                              double *terms, int64_t cap, double *out, double *series, size_t dyn,
                              hipStream_t st)
{
    // dynamic LDS above the default limit must be allowed per kernel
    static size_t allowed[64] = {};
    hipError_t ea = allow_dyn_lds(reinterpret_cast<const void *>(&k_contract_ph<TQ, NT, DUMP>),
                                  dyn, allowed);
    if (ea != hipSuccess) return ea;
    for (int64_t t0 = 0; t0 < N; t0 += cap) {
        const int64_t n = N - t0 < cap ? N - t0 : cap;
        hipError_t e = launch_terms(g, rec, perm, uvt, t0, n, terms, st);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_contract_ph<TQ, NT, DUMP>), dim3(nblk(n, 16)), dim3(NT), dyn, st, g,
                           N, perm, (const TQ *)Q, (const double *)terms, t0, out, series);
    }
    return hipGetLastError();
}

// Allows the persistent phased kernel `dyn` bytes of dynamic LDS (outside
// any stream capture: the batch calls it before capturing its graph).
template <typename TQ, int NT>
hipError_t allow_batched_ph(size_t dyn)
{
    static size_t allowed[64] = {}, allowed_pre[64] = {};
    hipError_t e = allow_dyn_lds(reinterpret_cast<const void *>(&k_contract_items<TQ, 16, NT, false>),
                                 dyn, allowed);
    if (e != hipSuccess) return e;
    return allow_dyn_lds(reinterpret_cast<const void *>(&k_contract_items<TQ, 16, NT, true>), dyn,
                         allowed_pre);
}

template <typename TQ, int NT>
hipError_t launch_batched_ph(const ile_geom *geoms, const ile_point_dev *pts, const int2 *items,
                             int n_items, size_t dyn, bool pre, hipStream_t st)
{
    hipError_t e = allow_batched_ph<TQ, NT>(dyn);
    if (e != hipSuccess) return e;
    // a dispatch covers fewer than 2^32 work-items: at most 2^22 items each
    constexpr int kMaxItems = 1 << 22;
    for (int i0 = 0; i0 < n_items; i0 += kMaxItems) {
        const int n = n_items - i0 < kMaxItems ? n_items - i0 : kMaxItems;
        if (pre)
            hipLaunchKernelGGL((k_contract_items<TQ, 16, NT, true>), dim3((unsigned)n), dim3(NT),
                               dyn, st, geoms, pts, items + i0);
        else
            hipLaunchKernelGGL((k_contract_items<TQ, 16, NT, false>), dim3((unsigned)n), dim3(NT),
                               dyn, st, geoms, pts, items + i0);
    }
    return hipGetLastError();
}

}  // namespace

// ------------------------------------------------------------ launchers
hipError_t ile_launch_finite(const double *z, int64_t n, int32_t *flag, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const unsigned grid = (unsigned)std::min<int64_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(k_finite, dim3(grid), dim3(256), 0, st, (const double2 *)z, n, flag);
    return hipGetLastError();
}

hipError_t ile_launch_planar(const double *raw, int r0, int nr, int64_t i0, int64_t ni, int n_lm,
                             int64_t n_q, bool fp64, void *dst, hipStream_t st)
{
    if (nr <= 0 || ni <= 0) return hipSuccess;
    const dim3 grid(nblk(ni, 256), nr);
    const int rp = 4 * ksp_of(n_lm);
    if (fp64)
        hipLaunchKernelGGL((k_planar<double>), grid, dim3(256), 0, st, (const double2 *)raw, r0,
                           i0, ni, n_lm, rp, n_q, (double *)dst);
    else
        hipLaunchKernelGGL((k_planar<float>), grid, dim3(256), 0, st, (const double2 *)raw, r0,
                           i0, ni, n_lm, rp, n_q, (float *)dst);
    return hipGetLastError();
}

hipError_t ile_launch_fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u32, dim3(nblk(n, 256)), dim3(256), 0, st, p, v, n);
    return hipGetLastError();
}

hipError_t ile_launch_prep(const ile_geom &g, const double *smp, int64_t N, ile_sample_rec *rec,
                           int32_t *shifts, uint32_t *keys, uint32_t *slot, uint32_t *hist,
                           uint32_t n_buckets, int32_t *err, hipStream_t st)
{
    if (N <= 0) return hipSuccess;
    if (hist)
        hipLaunchKernelGGL((k_prep<ILE_PREP_T, true>), dim3(nblk(N, ILE_PREP_T)), dim3(ILE_PREP_T),
                           0, st, g, smp, N, rec, shifts, keys, slot, hist, n_buckets, err);
    else
        hipLaunchKernelGGL((k_prep<64, false>), dim3(nblk(N, 64)), dim3(64), 0, st, g, smp, N, rec,
                           shifts, keys, slot, hist, n_buckets, err);
    return hipGetLastError();
}

int64_t ile_scan_tmp_words(int64_t n) { return (n + ILE_SCAN_BLOCK - 1) / ILE_SCAN_BLOCK; }

hipError_t ile_launch_scan(uint32_t *v, int64_t n, uint32_t *tmp, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const int64_t nb = ile_scan_tmp_words(n);
    if (nb > ILE_SCAN_BLOCK) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_scan_local, dim3((unsigned)nb), dim3(kScanT), 0, st, v, n, tmp);
    return hipGetLastError();
}

hipError_t ile_launch_scatter(const uint32_t *keys, const uint32_t *slot, int64_t N,
                              const uint32_t *offs, const uint32_t *bsum, int64_t n_buckets,
                              int32_t *perm, hipStream_t st)
{
    if (N <= 0) return hipSuccess;
    const int nb = (int)ile_scan_tmp_words(n_buckets);
    hipLaunchKernelGGL(k_scatter, dim3(nblk(N, 256)), dim3(256), nb * sizeof(uint32_t), st, keys,
                       slot, N, offs, bsum, nb, perm);
    return hipGetLastError();
}

// Whole evaluations (order, terms and tiles) by pairs and by counts: 2 x 5
// modes 36 against 43 us at 1000 samples, 44.3 against 45.3 at 8000, 58 against
// 54 at 13000; 3 x 9 modes, eight times the buckets, 78 against 96, 101 against
// 113 and 155 against 161.
int64_t ile_rank_max() { return 8192; }

hipError_t ile_launch_rank(const uint32_t *keys, int64_t N, int32_t *perm, hipStream_t st)
{
    if (N <= 0) return hipSuccess;
    if (N > ile_rank_max()) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_rank, dim3(nblk(N, 64)), dim3(kRankT), 0, st, keys, (int)N, perm);
    return hipGetLastError();
}

hipError_t ile_launch_identity(int32_t *perm, int64_t N, hipStream_t st)
{
    if (N <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_identity, dim3(nblk(N, 256)), dim3(256), 0, st, perm, N);
    return hipGetLastError();
}

static int kernel_threads(const ile_tune &tu)
{
    return tu.engine == ENG_MFMA ? 2 * tu.threads : tu.threads;
}

static size_t ph_budget(const ile_tune &tu, size_t e)
{
    if (tu.lds_budget > 0) return (size_t)tu.lds_budget;
    return e == 8 ? kPhBudget64 : kPhBudget32;
}

void ile_contract_prepare(ile_geom &g, ile_precision prec, const ile_tune &tu)
{
    if (tu.engine == ENG_PH && prec != ILE_BF16) {
        const size_t e = prec == ILE_FP64 ? 8 : 4;
        g.wrow = ph_wrow(g.n_det, g.n_lm, e, ph_budget(tu, e));
        g.wcap = g.wrow - 1;   // the slot past a row's last bin takes what lies outside
    } else {
        g.wrow = g.wcap = 0;
    }
}

static size_t coef_bytes_of(const ile_geom &g, ile_precision prec, const ile_tune &tu, size_t e)
{
    if (prec == ILE_BF16) return coef_bytes<ENG_BF16>(tu.tile_samples, g.n_det, g.n_lm, e);
    return tu.engine == ENG_MFMA ? coef_bytes<ENG_MFMA>(tu.tile_samples, g.n_det, g.n_lm, e)
                                 : coef_bytes<ENG_VALU>(tu.tile_samples, g.n_det, g.n_lm, e);
}

size_t ile_contract_lds_bytes(const ile_geom &g, ile_precision prec,
                              const ile_tune &tu)
{
    const size_t e = prec == ILE_FP64 ? 8 : 4;
    if (tu.engine == ENG_PH && prec != ILE_BF16) {
        const int w = ph_wrow(g.n_det, g.n_lm, e, ph_budget(tu, e));
        // a row is at least a unit, 16 values or more, a chunk one bin less
        if (w < 16) return (size_t)1 << 30;
        return ph_dyn_bytes(16, g.n_det, g.n_lm, w, e) + 2048;
    }
    const size_t gs = (size_t)tu.tile_samples * (tu.engine == ENG_MFMA ? 2 : 1) * tu.threads * e;
    const size_t coef = coef_bytes_of(g, prec, tu, e);
    const size_t scr = prologue_scratch_bytes(tu.tile_samples, g.n_det, g.n_lm);
    return gs + coef + (scr > gs ? scr : 0) + 4096;
}

bool ile_tune_supported(ile_precision prec, const ile_tune &tu)
{
    if (tu.tile_samples != 16) return false;
    // the phased engine takes FP64 and FP32 operands in workgroups of four
    // or eight waves; its block width follows from the LDS budget
    if (tu.engine == ENG_PH) return prec != ILE_BF16 && (tu.threads == 256 || tu.threads == 512);
    // positions per block: 256 or 512 for both engines; the matrix-core
    // engines also take 128 and 192 (smaller LDS, more workgroups per CU)
    const bool mf_only = tu.threads == 128 || tu.threads == 192;
    if (tu.threads != 256 && tu.threads != 512 && !mf_only) return false;
    if (prec == ILE_BF16) return tu.engine == ENG_MFMA;   // BF16 runs on the matrix cores only
    if (mf_only) return tu.engine == ENG_MFMA;
    return tu.engine == ENG_MFMA || tu.engine == ENG_VALU;
}

int ile_terms_fields(const ile_geom &g) { return terms_fields(g.n_det, g.n_lm); }

hipError_t ile_launch_terms_multi(const ile_geom *geoms, const ile_point_dev *pts, int n_points,
                                  int max_lm, int64_t n, hipStream_t st)
{
    if (n <= 0 || n_points <= 0) return hipSuccess;
    if (max_lm > 64 || n_points > 65535) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_terms_multi, dim3(nblk(n, kTermsT), n_points), dim3(kTermsT),
                       terms_lds_bytes(max_lm), st, geoms, pts, n);
    return hipGetLastError();
}

bool ile_contract_uses_terms(ile_precision prec, const ile_tune &tu)
{
    return tu.engine == ENG_PH && prec != ILE_BF16;
}

hipError_t ile_launch_contract(const ile_geom &g, ile_precision prec,
                               const ile_tune &tu, const double *smp, int64_t N,
                               const int32_t *perm, const int32_t *shifts,
                               const void *Q, const double *U, const double *V,
                               const ile_sample_rec *rec, const double *uvt, double *terms,
                               int64_t cap, double *out, double *series,
                               hipStream_t st)
{
    if (N <= 0) return hipSuccess;
    if (!ile_tune_supported(prec, tu)) return hipErrorInvalidValue;
    if (tu.engine == ENG_PH) {
        ile_geom gp = g;
        ile_contract_prepare(gp, prec, tu);
        if (gp.wrow < 16) return hipErrorInvalidValue;
        if (!uvt || !terms || !rec || cap < 16 || cap % 16) return hipErrorInvalidValue;
        if (g.n_lm > 64) return hipErrorInvalidValue;
        const size_t e = prec == ILE_FP64 ? 8 : 4;
        // one 32-bit buffer range covers the whole series
        if ((size_t)g.n_det * 4 * ksp_of(g.n_lm) * g.n_q * e > 0x7fffffffu)
            return hipErrorInvalidValue;
        const size_t dyn = ph_dyn_bytes(16, g.n_det, g.n_lm, gp.wrow, e);
#define ILE_PH(TQ, NT)                                                                       \
    return series ? launch_contract_ph<TQ, NT, true>(gp, N, perm, rec, Q, uvt, terms, cap,     \
                                                     out, series, dyn, st)                     \
                  : launch_contract_ph<TQ, NT, false>(gp, N, perm, rec, Q, uvt, terms, cap,    \
                                                      out, series, dyn, st)
        if (prec == ILE_FP64) {
            if (tu.threads == 256) ILE_PH(double, 256);
            ILE_PH(double, 512);
        }
        if (tu.threads == 256) ILE_PH(float, 256);
        ILE_PH(float, 512);
#undef ILE_PH
    }
#define ILE_CONTRACT(TQ, NT, ENG) \
    return launch_contract_t<TQ, 16, NT, ENG>(g, smp, N, perm, shifts, Q, U, V, out, series, st)
    if (prec == ILE_FP64) {
        if (tu.engine == ENG_MFMA) {
            // producer + consumer halves: threads = 2 x positions per block
            if (tu.threads == 512) ILE_CONTRACT(double, 1024, ENG_MFMA);
            if (tu.threads == 192) ILE_CONTRACT(double, 384, ENG_MFMA);
            if (tu.threads == 128) ILE_CONTRACT(double, 256, ENG_MFMA);
            ILE_CONTRACT(double, 512, ENG_MFMA);
        }
        if (tu.threads == 512) ILE_CONTRACT(double, 512, ENG_VALU);
        ILE_CONTRACT(double, 256, ENG_VALU);
    }
    if (prec == ILE_BF16) {
        if (tu.threads == 512) ILE_CONTRACT(float, 1024, ENG_BF16);
        if (tu.threads == 192) ILE_CONTRACT(float, 384, ENG_BF16);
        if (tu.threads == 128) ILE_CONTRACT(float, 256, ENG_BF16);
        ILE_CONTRACT(float, 512, ENG_BF16);
    }
    if (tu.engine == ENG_MFMA) {
        if (tu.threads == 512) ILE_CONTRACT(float, 1024, ENG_MFMA);
        if (tu.threads == 192) ILE_CONTRACT(float, 384, ENG_MFMA);
        if (tu.threads == 128) ILE_CONTRACT(float, 256, ENG_MFMA);
        ILE_CONTRACT(float, 512, ENG_MFMA);
    }
    if (tu.threads == 512) ILE_CONTRACT(float, 512, ENG_VALU);
    ILE_CONTRACT(float, 256, ENG_VALU);
#undef ILE_CONTRACT
}

size_t ile_contract_dyn_bytes(const ile_geom &g, ile_precision prec, const ile_tune &tu)
{
    const size_t e = prec == ILE_FP64 ? 8 : 4;
    if (tu.engine == ENG_PH && prec != ILE_BF16)
        return ph_dyn_bytes(16, g.n_det, g.n_lm, ph_wrow(g.n_det, g.n_lm, e, ph_budget(tu, e)), e);
    size_t dyn = coef_bytes_of(g, prec, tu, e);
    const size_t scr = prologue_scratch_bytes(tu.tile_samples, g.n_det, g.n_lm);
    if (scr > (size_t)tu.tile_samples * kernel_threads(tu) * e) dyn += scr;
    return dyn;
}

hipError_t ile_contract_batched_allow(ile_precision prec, const ile_tune &tu, size_t dyn)
{
    if (tu.engine != ENG_PH || prec == ILE_BF16) return hipSuccess;
    if (prec == ILE_FP64)
        return tu.threads == 256 ? allow_batched_ph<double, 256>(dyn)
                                 : allow_batched_ph<double, 512>(dyn);
    return tu.threads == 256 ? allow_batched_ph<float, 256>(dyn) : allow_batched_ph<float, 512>(dyn);
}

hipError_t ile_launch_contract_batched(ile_precision prec, const ile_tune &tu,
                                       const ile_geom *geoms, const ile_point_dev *pts,
                                       const int2 *items, int n_items, unsigned *counter,
                                       int grid, size_t dyn, bool terms, hipStream_t st)
{
    if (!ile_tune_supported(prec, tu)) return hipErrorInvalidValue;
    if (tu.engine == ENG_PH) {
        // one workgroup per item (grid and counter are for the persistent
        // kernels of the other engines)
        if (prec == ILE_FP64)
            return tu.threads == 256
                       ? launch_batched_ph<double, 256>(geoms, pts, items, n_items, dyn, terms, st)
                       : launch_batched_ph<double, 512>(geoms, pts, items, n_items, dyn, terms, st);
        return tu.threads == 256
                   ? launch_batched_ph<float, 256>(geoms, pts, items, n_items, dyn, terms, st)
                   : launch_batched_ph<float, 512>(geoms, pts, items, n_items, dyn, terms, st);
    }
#define ILE_BATCHED(TQ, NT, ENG)                                                              \
    do {                                                                                      \
        hipLaunchKernelGGL((k_contract_batched<TQ, 16, NT, ENG>), dim3(grid), dim3(NT), dyn,   \
                           st, geoms, pts, items, n_items, counter);                          \
        return hipGetLastError();                                                             \
    } while (0)
    if (prec == ILE_FP64) {
        if (tu.engine == ENG_MFMA) {
            if (tu.threads == 512) ILE_BATCHED(double, 1024, ENG_MFMA);
            if (tu.threads == 192) ILE_BATCHED(double, 384, ENG_MFMA);
            if (tu.threads == 128) ILE_BATCHED(double, 256, ENG_MFMA);
            ILE_BATCHED(double, 512, ENG_MFMA);
        }
        if (tu.threads == 512) ILE_BATCHED(double, 512, ENG_VALU);
        ILE_BATCHED(double, 256, ENG_VALU);
    }
    if (prec == ILE_BF16) {
        if (tu.threads == 512) ILE_BATCHED(float, 1024, ENG_BF16);
        if (tu.threads == 192) ILE_BATCHED(float, 384, ENG_BF16);
        if (tu.threads == 128) ILE_BATCHED(float, 256, ENG_BF16);
        ILE_BATCHED(float, 512, ENG_BF16);
    }
    if (tu.engine == ENG_MFMA) {
        if (tu.threads == 512) ILE_BATCHED(float, 1024, ENG_MFMA);
        if (tu.threads == 192) ILE_BATCHED(float, 384, ENG_MFMA);
        if (tu.threads == 128) ILE_BATCHED(float, 256, ENG_MFMA);
        ILE_BATCHED(float, 512, ENG_MFMA);
    }
    if (tu.threads == 512) ILE_BATCHED(float, 512, ENG_VALU);
    ILE_BATCHED(float, 256, ENG_VALU);
#undef ILE_BATCHED
}

hipError_t ile_launch_prior(uint64_t seed, int64_t first, int64_t N,
                            double d_min, double d_max, double t_ref_max,
                            double *smp, int64_t ld, double *ln_p, hipStream_t st)
{
    if (N <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_prior, dim3(nblk(N, 256)), dim3(256), 0, st, seed, first,
                       N, d_min, d_max, t_ref_max, smp, ld, ln_p);
    return hipGetLastError();
}

int ile_reduce_blocks() { return kRedBlocks; }

hipError_t ile_launch_reduce(const double *lnL, const double *ln_p,
                             const double *ln_q, int64_t N, double *tmp,
                             double *partial, const double *parts, int n_part, double *res,
                             hipStream_t st)
{
    if (N <= kRedSmallMax) {
#define ILE_SMALL(PER)                                                                        \
    hipLaunchKernelGGL((k_red_small<PER>), dim3(1), dim3(kRedSmallT), 0, st, lnL, ln_p, ln_q, \
                       (int)N, partial, parts, n_part, res)
        if (N <= 1 * kRedSmallT) ILE_SMALL(1);
        else if (N <= 4 * kRedSmallT) ILE_SMALL(4);
        else if (N <= 8 * kRedSmallT) ILE_SMALL(8);
        else if (N <= 12 * kRedSmallT) ILE_SMALL(12);
        else ILE_SMALL(16);
#undef ILE_SMALL
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_red_max, dim3(kRedBlocks), dim3(kRedT), 0, st, lnL, ln_p,
                       ln_q, N, tmp);
    hipLaunchKernelGGL(k_red_sum, dim3(kRedBlocks), dim3(kRedT), 0, st, lnL, ln_p,
                       ln_q, N, tmp);
    hipLaunchKernelGGL(k_red_final, dim3(1), dim3(kRedT), 0, st, (const double *)tmp,
                       N, partial, parts, n_part, res);
    return hipGetLastError();
}

hipError_t ile_launch_fetch(const int32_t *flag, const double *res, double *host, hipStream_t st)
{
    hipLaunchKernelGGL(k_fetch, dim3(1), dim3(64), 0, st, flag, res, host);
    return hipGetLastError();
}

hipError_t ile_launch_to_bf16_split(const double *, int64_t, void *, hipStream_t)
{
    return hipErrorNotSupported;
}

hipError_t ile_launch_inject(const ile_geom &g, const double *h, int n, const double *theta,
                             double *d, hipStream_t st)
{
    const int64_t tot = (int64_t)g.n_det * n;
    hipLaunchKernelGGL(k_inject_resp, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, g,
                       (const double2 *)h, n, theta, d);
    return hipGetLastError();
}

hipError_t ile_launch_inject_qv(int n_det, int n_lm, int n, const double *h, const double *d,
                                double scale, double *Q, double *U, double *V, hipStream_t st)
{
    hipLaunchKernelGGL(k_inject_corr, dim3((unsigned)((n + 255) / 256), (unsigned)(n_det * n_lm)),
                       dim3(256), 0, st, n_lm, n, (const double2 *)h, d, scale, (double2 *)Q);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_inject_gram, dim3((unsigned)(n_lm * n_lm)), dim3(256), 0, st, n_lm, n,
                       (const double2 *)h, (double2 *)U, (double2 *)V);
    return hipGetLastError();
}
