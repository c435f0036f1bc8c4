// ile_batch.hip -- multi-point kernels of the batched form: many intrinsic
// points (uneven mode counts and window lengths) evaluated together
// (arXiv:1902.04934, Sec. III.B: each ILE instance loops over many
// intrinsic points to amortize its startup).  One launch each for the
// prior draw, window starts and ordering keys, scatter, and the per-point
// reduction; the contraction is the persistent kernel in ile_kernels.hip.
// Samples of point p live at offs[p] .. offs[p+1] of the concatenated
// arrays (SoA [7][N_p] per point); keys put point p in buckets
// [p B, (p+1) B) so one counting sort orders every point at once.
#include <hip/hip_runtime.h>
#include <math.h>

#include "ile_internal.h"
#include "ile_rng.h"

namespace {

constexpr double kPi = 3.141592653589793238463;

__device__ inline int point_of(const int64_t *offs, int n_points, int64_t i)
{
    int lo = 0, hi = n_points - 1;   // last p with offs[p] <= i
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (offs[mid] <= i)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

using ile_rng::u53;

// prior draw: point p uses the Philox stream of key seed + p (the stream of
// ile_draw_prior_dev), sample t of the point counter t
__global__ __launch_bounds__(256) void k_prior_multi(const uint64_t *seed_dev,
                                                     const int64_t *offs, int n_points,
                                                     int64_t n_total, double d_min,
                                                     double d_max, double t_ref_max,
                                                     double *smp)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_total) return;
    const int p = point_of(offs, n_points, i);
    const int64_t o = offs[p], n = offs[p + 1] - o, t = i - o;
    const uint64_t seed = *seed_dev + (uint64_t)p;
    uint32_t w[16];
    ile_rng::prior_words(seed, (uint64_t)t, w);
    double *s = smp + 7 * o;
    {
#pragma clang fp contract(off)
        const double v3 = d_max * d_max * d_max - d_min * d_min * d_min;
        s[0 * n + t] = 2.0 * kPi * u53(w[0], w[1]);
        s[1 * n + t] = asin(2.0 * u53(w[2], w[3]) - 1.0);
        s[2 * n + t] = kPi * u53(w[4], w[5]);
        s[3 * n + t] = 2.0 * kPi * u53(w[6], w[7]);
        s[4 * n + t] = 2.0 * u53(w[8], w[9]) - 1.0;
        s[5 * n + t] = cbrt(d_min * d_min * d_min + u53(w[10], w[11]) * v3);
        s[6 * n + t] = t_ref_max * (2.0 * u53(w[12], w[13]) - 1.0);
    }
}

// window starts, ordering keys and bucket slots (same arithmetic as the
// single-point path)
__global__ __launch_bounds__(ILE_PREP_T) void k_prep_multi(
    const ile_geom *__restrict__ geoms, const int64_t *__restrict__ offs, int n_points,
    int64_t n_total, const double *__restrict__ smp, ile_sample_rec *__restrict__ rec,
    int32_t *__restrict__ shifts, uint32_t *__restrict__ keys, uint32_t *__restrict__ slot,
    uint32_t *hist, uint32_t B, int32_t *err)
{
    const int64_t i = (int64_t)blockIdx.x * ILE_PREP_T + threadIdx.x;
    const bool live = i < n_total;
    const int64_t il = live ? i : n_total - 1;
    const int p = point_of(offs, n_points, il);
    const ile_geom &g = geoms[p];
    const int64_t o = offs[p], n = offs[p + 1] - o, t = il - o;
    const double *s = smp + 7 * o;
    double th[7];
#pragma unroll
    for (int q = 0; q < 7; q++) th[q] = s[q * n + t];
    int sh[ILE_MAX_DET];
    const bool ok = window_starts(g, th, sh);
    // invalid samples last within the point
    const uint32_t key = (uint32_t)p * B + (ok ? cell_key(g, sh) : B - 1);
    if (live) {
        if (!ok) atomicOr(err, 1);
        store_starts(g, th, sh, ok, rec ? rec + o : nullptr,
                     rec ? nullptr : shifts + (int64_t)ILE_MAX_DET * o, t, n);
        keys[i] = key;
    }
    const uint32_t r = block_count_slot(hist, key, live);
    if (live) slot[i] = r;
}

// sorted position -> local sample index of the point
__global__ __launch_bounds__(256) void k_scatter_multi(
    const uint32_t *__restrict__ keys, const uint32_t *__restrict__ slot,
    const int64_t *__restrict__ offs, int n_points, int64_t n_total,
    const uint32_t *__restrict__ pos, const uint32_t *__restrict__ bsum, int nb,
    int32_t *__restrict__ perm)
{
    extern __shared__ uint32_t pre[];
    scan_prefix(bsum, nb, pre);
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n_total) return;
    const int p = point_of(offs, n_points, i);
    const uint32_t k = keys[i];
    perm[pos[k] + pre[k / ILE_SCAN_BLOCK] + slot[i]] = (int32_t)(i - offs[p]);
}

// Per-point reduction: ln w = lnLmargT + (ln p - ln q) (lw = NULL: ln w =
// lnLmargT, the prior draws), fixed-order sums; res[6 p ..] = (ln L_marg,
// n_eff, Kish, sigma, max lnLmargT, n).  Three kernels of kRB workgroups a
// point: the maxima, the sums, and one workgroup a point that finishes and
// writes the host's copy.  Eight points of 1e5 samples: 18 us (83 with one
// workgroup a point, whose chain of 98 exps a thread, twice, was the time).
constexpr int kRT = 256, kRB = 64;

__device__ inline double ln_w(const double *out, const double *lw, int64_t i)
{
    return lw ? out[i] + lw[i] : out[i];
}

// tmp: [4][n_points][kRB] largest ln w, largest lnLmargT, the two sums
__global__ __launch_bounds__(kRT) void k_points_max(const double *__restrict__ out,
                                                    const double *__restrict__ lw,
                                                    const int64_t *__restrict__ offs,
                                                    double *__restrict__ tmp)
{
    __shared__ double sm[2][kRT / 64];
    const int b = blockIdx.x, p = blockIdx.y, t = threadIdx.x;
    const int64_t o = offs[p], n = offs[p + 1] - o;
    double M = -INFINITY, ML = -INFINITY;
#pragma unroll 4
    for (int64_t i = (int64_t)b * kRT + t; i < n; i += kRB * kRT) {
        M = fmax(M, ln_w(out, lw, o + i));
        ML = fmax(ML, out[o + i]);
    }
    M = wave_max(M);
    ML = wave_max(ML);
    if ((t & 63) == 0) {
        sm[0][t >> 6] = M;
        sm[1][t >> 6] = ML;
    }
    __syncthreads();
    if (t == 0) {
        for (int w = 1; w < kRT / 64; w++) {
            M = fmax(M, sm[0][w]);
            ML = fmax(ML, sm[1][w]);
        }
        const int at = p * kRB + b, np = gridDim.y * kRB;
        tmp[at] = M;
        tmp[np + at] = ML;
    }
}

__global__ __launch_bounds__(kRT) void k_points_sum(const double *out, const double *lw,
                                                    const int64_t *offs, double *tmp)
{
    __shared__ double sm[2][kRT];
    const int b = blockIdx.x, p = blockIdx.y, t = threadIdx.x, np = gridDim.y * kRB;
    const int64_t o = offs[p], n = offs[p + 1] - o;
    const double M = wave_max(tmp[p * kRB + (t & 63)]);
    double s[2] = {0.0, 0.0};
    if (M != -INFINITY)
        for (int64_t i = (int64_t)b * kRT + t; i < n; i += kRB * kRT) {
            const double e = exp(ln_w(out, lw, o + i) - M);
            s[0] += e;
            s[1] = fma(e, e, s[1]);
        }
    tree_sum<kRT, 2>(s, sm);
    if (t == 0) {
        const int at = p * kRB + b;
        tmp[2 * np + at] = s[0];
        tmp[3 * np + at] = s[1];
    }
}

__global__ __launch_bounds__(64) void k_points_final(const double *__restrict__ tmp,
                                                     const int64_t *__restrict__ offs,
                                                     const int32_t *__restrict__ err,
                                                     double *__restrict__ host)
{
    const int p = blockIdx.x, t = threadIdx.x, np = gridDim.x * kRB;
    const double M = wave_max(tmp[p * kRB + t]), ML = wave_max(tmp[np + p * kRB + t]);
    double s1 = tmp[2 * np + p * kRB + t], s2 = tmp[3 * np + p * kRB + t];
    for (int off = 32; off > 0; off >>= 1) {
        s1 += __shfl_down(s1, off);
        s2 += __shfl_down(s2, off);
    }
    if (t == 0) finish_one(M, s1, s2, (double)(offs[p + 1] - offs[p]), ML, host + 1 + 6 * p);
    if (t == 0 && p == 0) *reinterpret_cast<int32_t *>(host) = *err;
}
static_assert(kRB == 64, "a partial a lane");

// ln p - ln q of caller-supplied draws (either may be NULL = 0); an invalid
// pair (NaN, ln q = -inf or ln p = +inf) sets bit 2 of the error flag.
__global__ __launch_bounds__(256) void k_batch_lw(const double *lp, const double *lq,
                                                  int64_t n_total, double *lw, int32_t *err)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_total) return;
    const double p = lp ? lp[i] : 0.0, q = lq ? lq[i] : 0.0;
    if (isnan(p) || isnan(q) || q == -INFINITY || p == INFINITY) {
        atomicOr(err, 2);
        lw[i] = NAN;
        return;
    }
    lw[i] = p - q;
}

inline unsigned nblk(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

}  // namespace

hipError_t ile_launch_prior_multi(const uint64_t *seed_dev, const int64_t *offs, int n_points,
                                  int64_t n_total, double d_min, double d_max,
                                  double t_ref_max, double *smp, hipStream_t st)
{
    hipLaunchKernelGGL(k_prior_multi, dim3(nblk(n_total, 256)), dim3(256), 0, st, seed_dev,
                       offs, n_points, n_total, d_min, d_max, t_ref_max, smp);
    return hipGetLastError();
}

hipError_t ile_launch_prep_multi(const ile_geom *geoms, const int64_t *offs, int n_points,
                                 int64_t n_total, const double *smp, ile_sample_rec *rec,
                                 int32_t *shifts, uint32_t *keys, uint32_t *slot,
                                 uint32_t *hist, uint32_t B, int32_t *err, hipStream_t st)
{
    hipLaunchKernelGGL(k_prep_multi, dim3(nblk(n_total, ILE_PREP_T)), dim3(ILE_PREP_T), 0, st,
                       geoms, offs, n_points, n_total, smp, rec, shifts, keys, slot, hist, B, err);
    return hipGetLastError();
}

hipError_t ile_launch_scatter_multi(const uint32_t *keys, const uint32_t *slot,
                                    const int64_t *offs, int n_points, int64_t n_total,
                                    const uint32_t *pos, const uint32_t *bsum,
                                    int64_t n_buckets, int32_t *perm, hipStream_t st)
{
    const int nb = (int)ile_scan_tmp_words(n_buckets);
    hipLaunchKernelGGL(k_scatter_multi, dim3(nblk(n_total, 256)), dim3(256),
                       nb * sizeof(uint32_t), st, keys, slot, offs, n_points, n_total, pos, bsum,
                       nb, perm);
    return hipGetLastError();
}

size_t ile_reduce_points_tmp(int n_points) { return (size_t)4 * kRB * n_points; }

hipError_t ile_launch_reduce_points(const double *out, const double *lw, const int64_t *offs,
                                    int n_points, double *tmp, const int32_t *err, double *host,
                                    hipStream_t st)
{
    if (n_points > 65535) return hipErrorInvalidValue;
    const dim3 grid(kRB, n_points);
    hipLaunchKernelGGL(k_points_max, grid, dim3(kRT), 0, st, out, lw, offs, tmp);
    hipLaunchKernelGGL(k_points_sum, grid, dim3(kRT), 0, st, out, lw, offs, tmp);
    hipLaunchKernelGGL(k_points_final, dim3(n_points), dim3(64), 0, st, (const double *)tmp, offs,
                       err, host);
    return hipGetLastError();
}

hipError_t ile_launch_batch_lw(const double *lp, const double *lq, int64_t n_total, double *lw,
                               int32_t *err, hipStream_t st)
{
    if (n_total <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_batch_lw, dim3(nblk(n_total, 256)), dim3(256), 0, st, lp, lq, n_total,
                       lw, err);
    return hipGetLastError();
}
