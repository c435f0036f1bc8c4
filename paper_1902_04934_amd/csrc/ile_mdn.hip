// ile_mdn.hip -- the learned proposal: a masked autoregressive mixture
// density network over the 7 extrinsic parameters, on the matrix cores.
//
// The paper draws its Monte Carlo samples from an adaptive proposal built
// from one-dimensional histograms (Sec. II.A, Sec. III.C); this network is a
// richer proposal trained on the weighted samples of the first adaptive
// rounds, used in a defensive mixture with the histogram proposal.
//
// Model (parameter layout in ile.h): inputs z~[7] (the transformed sample),
// h1 = tanh(W1 z~ + b1), h2 = tanh(W2 h1 + b2), o = W3 h2 + b3, with MADE
// masks (hidden degree k mod 6) so that dimension d's 16-component Gaussian
// mixture, o[48d .. 48d+47] = (logits, means, scale pre-activations),
// depends on z~_0..z~_{d-1} only.
//
// Arithmetic: layer 1 (7 inputs) in FP32 on the vector ALUs; layers 2 and 3
// on v_mfma_f32_16x16x32_bf16 (BF16 operands, FP32 accumulation); mixture
// densities in FP32; the transform, its Jacobian, ln p and the mixture with
// the histogram proposal in FP64.  One wave evaluates 16 samples: lane
// l = 16 g + r holds sample r's inputs (A layout: row r, k = 8 g .. 8 g + 7
// of each 32-wide K step) and receives outputs for samples 4 g + v, v < 4,
// at column r (D layout); a sample's 16 mixture components therefore sit
// in one 16-lane group and its log-sum-exps are 16-lane butterflies.
//
// Training: each workgroup runs forward and backward for 64 samples and
// writes its gradient as one partial row; a second kernel sums the rows in
// a fixed order and takes the Adam step, so training is bit-reproducible.
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>

#include "ile_internal.h"
#include "ile_rng.h"

namespace {

constexpr int D = ILE_MDN_D, H = ILE_MDN_H, O = ILE_MDN_O;
constexpr int OFF_W1 = ILE_MDN_OFF_W1, OFF_B1 = ILE_MDN_OFF_B1, OFF_W2 = ILE_MDN_OFF_W2,
              OFF_B2 = ILE_MDN_OFF_B2, OFF_W3 = ILE_MDN_OFF_W3, OFF_B3 = ILE_MDN_OFF_B3,
              NPARAM = ILE_MDN_NPARAM, NPART = ILE_MDN_NPART, W3T_LD = ILE_MDN_W3T_LD;
constexpr int WLD = 136;   // LDS row of a [row][128] bf16 array (+16 bytes: no bank conflicts)
constexpr int SLD = 72;    // LDS row of a [unit][64 samples] bf16 array
constexpr int CLD = 104;   // LDS row of a 96-output chunk of dL/do
constexpr int MAXB = 64;   // histogram bins held in LDS
constexpr double kPi = 3.141592653589793238463;
constexpr double kTwoPi = 6.283185307179586476925;
constexpr float kHalfLn2Pi = 0.91893853320467274178f;

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v4bf __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

__device__ inline v4f mfma(v8bf a, v8bf b, v4f c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ inline float softplusf(float x) { return fmaxf(x, 0.f) + log1pf(expf(-fabsf(x))); }

// Branch-free functions at the hardware's transcendental rate for the
// training gradient (a few ulp; the BF16 operands of the products dominate
// its error).  exp and log through the base-2 instructions.
__device__ inline float fexp(float x) { return __builtin_amdgcn_exp2f(x * 1.44269504088896341f); }
__device__ inline float flog(float x) { return __builtin_amdgcn_logf(x) * 0.693147180559945309f; }
__device__ inline float frcp(float x) { return __builtin_amdgcn_rcpf(x); }
// tanh: odd Taylor series through x^9 for |x| < 0.2 (truncation < 1e-9
// relative), else (1 - e) / (1 + e) with e = exp(-2|x|)
__device__ inline float ftanh(float x)
{
    const float ax = fabsf(x), x2 = x * x;
    const float poly = ax + ax * x2 * (-1.f / 3.f + x2 * (2.f / 15.f + x2 * (-17.f / 315.f +
                                                                        x2 * (62.f / 2835.f))));
    const float e = fexp(-2.f * ax);
    const float big = (1.f - e) * frcp(1.f + e);
    return copysignf(ax < 0.2f ? poly : big, x);
}
__device__ inline float fsoftplus(float x) { return fmaxf(x, 0.f) + flog(1.f + fexp(-fabsf(x))); }
__device__ inline float fsigmoid(float x) { return frcp(1.f + fexp(-x)); }

// 16-lane reductions by DPP rotations within a row (8, 4, 2, 1 lanes):
// after the rotation by n the partial values repeat with period n, so
// lane i meets the same partner value as in an xor butterfly, and every
// lane of the group ends with the same bits (each step combines the same
// two operands in either order).  DPP moves data between lanes in the
// VALU, without the LDS round trip of a permute.
template <int N>
__device__ inline float row_ror(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
        0, __builtin_bit_cast(int, x), 0x120 + N, 0xF, 0xF, false));
}
__device__ inline float gmax(float x)
{
    x = fmaxf(x, row_ror<8>(x));
    x = fmaxf(x, row_ror<4>(x));
    x = fmaxf(x, row_ror<2>(x));
    return fmaxf(x, row_ror<1>(x));
}
__device__ inline float gsum(float x)
{
    x += row_ror<8>(x);
    x += row_ror<4>(x);
    x += row_ror<2>(x);
    return x + row_ror<1>(x);
}

// Inclusive prefix sums over a 16-lane row, in the order of a shift by 1, 2, 4
// and 8 lanes (a lane with no source adds 0, which leaves it unchanged), and
// the row's last value in every lane.
template <int CTRL>
__device__ inline float row_dpp(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
        0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
}
__device__ inline float row_scan(float x)
{
    x += row_dpp<0x111>(x);   // row_shr
    x += row_dpp<0x112>(x);
    x += row_dpp<0x114>(x);
    return x + row_dpp<0x118>(x);
}
__device__ inline float row_last(float x) { return row_dpp<0x15F>(x); }   // row_newbcast:15

// Ordering point for LDS data handed between lanes of one wave: a wave's
// LDS accesses are performed in issue order, so it is enough that the
// compiler moves no access across this point (no workgroup barrier).
__device__ inline void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ------------------------------------------------------------ transform
// u in (0,1) of dimension d and ln |du/dx|
__device__ inline double to_unit(const ile_mdn_tr &T, int d, double x, double &ldu)
{
    double y;
    switch (d) {
    case 0:
        y = (x - T.origin[0]) / kTwoPi + 0.5;
        ldu = -log(kTwoPi);
        return y - floor(y);
    case 1:
        ldu = log(cos(x) / 2.0);
        return (sin(x) + 1.0) / 2.0;
    case 2:
        y = (x - T.origin[1]) / kPi + 0.5;
        ldu = -log(kPi);
        return y - floor(y);
    case 3:
        y = (x - T.origin[2]) / kTwoPi + 0.5;
        ldu = -log(kTwoPi);
        return y - floor(y);
    case 4:
        ldu = -log(2.0);
        return (x + 1.0) / 2.0;
    case 5:
        ldu = -log(T.d_max - T.d_min);
        return (x - T.d_min) / (T.d_max - T.d_min);
    default:
        ldu = -log(2.0 * T.t_ref_max);
        return (x + T.t_ref_max) / (2.0 * T.t_ref_max);
    }
}

// inverse of to_unit; periodic parameters wrapped into their prior range (the
// product rounded before the sum, then one fused step, whatever code
// surrounds it, so that a seed's draws do not depend on it)
__device__ inline double wrap_unit(double origin, double u, double period)
{
    double x;
    {
#pragma clang fp contract(off)
        x = origin + (u - 0.5) * period;
    }
    return fma(-period, floor(x / period), x);
}
__device__ inline double from_unit(const ile_mdn_tr &T, int d, double u)
{
    switch (d) {
    case 0: return wrap_unit(T.origin[0], u, kTwoPi);
    case 1: return asin(2.0 * u - 1.0);
    case 2: return wrap_unit(T.origin[1], u, kPi);
    case 3: return wrap_unit(T.origin[2], u, kTwoPi);
    case 4: return 2.0 * u - 1.0;
    case 5: return T.d_min + u * (T.d_max - T.d_min);
    default: return (2.0 * u - 1.0) * T.t_ref_max;
    }
}

// x_d -> z~_d (FP32 network input); returns ln |dz~_d/dx_d|, or -inf when u
// is 0 or 1 (z~ is then 0)
__device__ inline double to_z_dim(const ile_mdn_tr &T, int d, double x, float &z)
{
    double ldu;
    const double u = to_unit(T, d, x, ldu);
    if (!(u > 0.0 && u < 1.0)) {
        z = 0.f;
        return -INFINITY;
    }
    const double lu = log(u), l1u = log1p(-u);
    z = (float)((lu - l1u - T.mean[d]) / T.scale[d]);
    return -log(T.scale[d]) - lu - l1u + ldu;
}

// The dimensions' ln |dz~/dx| summed in order, -inf where any of them is: a
// declination past the poles has a NaN (the logarithm of a negative cosine),
// which must not hide that x is outside another dimension's range.
__device__ inline double sum_lj(const double *lj)
{
    double s = 0.0;
    bool out = false;
#pragma unroll
    for (int d = 0; d < D; d++) {
        out |= lj[d] == -INFINITY;
        s += lj[d];
    }
    return out ? -INFINITY : s;
}

// all dimensions
__device__ inline double to_z(const ile_mdn_tr &T, const double x[7], float z[7])
{
    double lj[D];
#pragma unroll
    for (int d = 0; d < D; d++) lj[d] = to_z_dim(T, d, x[d], z[d]);
    return sum_lj(lj);
}

__device__ inline double logaddexp(double a, double b)
{
    const double m = fmax(a, b);
    if (m == -INFINITY) return -INFINITY;
    return m + log(exp(a - m) + exp(b - m));
}

// ln (q_hist / p) of the histogram proposal at (ra, dec)
__device__ inline double ln_hist_ratio(const double *P, int nb, double ra, double dec)
{
    int br = (int)floor(ra * (nb / kTwoPi));
    int bs = (int)floor((sin(dec) + 1.0) * (0.5 * nb));
    br = min(max(br, 0), nb - 1);
    bs = min(max(bs, 0), nb - 1);
    return log(nb * P[br]) + log(nb * P[nb + bs]);
}

// ---------------------------------------------------------- the layers
// Layer 1 for sample r: units k = 32 ks + 8 g + i as BF16 A fragments.
__device__ inline void layer1(const float *W1, int w1ld, const float *b1, const float z[7],
                              int g, v8bf A[4])
{
#pragma unroll
    for (int ks = 0; ks < 4; ks++) {
#pragma unroll
        for (int i = 0; i < 8; i++) {
            const int k = 32 * ks + 8 * g + i;
            float a = b1[k];
#pragma unroll
            for (int d = 0; d < D; d++) a = fmaf(W1[k * w1ld + d], z[d], a);
            A[ks][i] = (__bf16)tanhf(a);
        }
    }
}

// B fragments of the three layer-3 output tiles of dimension d, [4 ks][3 j].
__device__ inline void load_w3_dim(const __bf16 *W3, int ld, int d, int r, int g, v8bf B[12])
{
#pragma unroll
    for (int ks = 0; ks < 4; ks++)
#pragma unroll
        for (int j = 0; j < 3; j++)
            B[3 * ks + j] = *(const v8bf *)(W3 + (48 * d + 16 * j + r) * ld + 32 * ks + 8 * g);
}

// ln q_d of one sample from its component (lane r of the group): returns
// the log density; sig, rr = (z - mu)/sig, ell = log weight + log normal
// of this component, la = log-sum-exp of the logits.
__device__ inline float mix_lnq(float a, float mu, float rho, float z, float sfloor, float kappa,
                                float &sig, float &rr, float &ell, float &la)
{
    const float ma = gmax(a);
    la = ma + logf(gsum(expf(a - ma)));
    sig = kappa * (sfloor + softplusf(rho));
    rr = (z - mu) / sig;
    ell = a - la - 0.5f * rr * rr - logf(sig) - kHalfLn2Pi;
    const float ml = gmax(ell);
    return ml + logf(gsum(expf(ell - ml)));
}

// mix_lnq with the branch-free functions (training gradient); rs = 1/sig
__device__ inline float mix_lnq_fast(float a, float mu, float rho, float z, float sfloor,
                                     float &rs, float &rr, float &ell, float &la)
{
    const float ma = gmax(a);
    la = ma + flog(gsum(fexp(a - ma)));
    const float sig = sfloor + fsoftplus(rho);
    rs = frcp(sig);
    rr = (z - mu) * rs;
    ell = a - la - 0.5f * rr * rr - flog(sig) - kHalfLn2Pi;
    const float ml = gmax(ell);
    return ml + flog(gsum(fexp(ell - ml)));
}

// ----------------------------------------------------------- inference
// LDS image of a [rows][128] bf16 array in rows of 256 bytes without padding:
// 16-byte chunk c of row m is at chunk c ^ (m mod 16), so that the 16 rows
// one fragment load touches lie in 16 different bank groups.
__device__ inline int swz(int m, int c) { return m * H + ((c ^ (m & 15)) << 3); }

constexpr int IW = 8;            // waves per workgroup
constexpr int IT = 64 * IW;
constexpr int W3ROWS = O - 48;   // dimension 0 has no weights

// The FP64 parts of a tile, out of line: inlined, the constants of their
// exponentials and logarithms are held in registers across the tiles and the
// kernel spills.
struct zterm {
    double lj;
    float z;
};
__device__ __attribute__((noinline)) zterm to_z_call(const ile_mdn_tr &T, int d, double x)
{
    zterm t;
    t.lj = to_z_dim(T, d, x, t.z);
    return t;
}
__device__ __attribute__((noinline)) double from_z_call(const ile_mdn_tr &T, int d, float z)
{
    const double zz = T.mean[d] + T.scale[d] * (double)z;
    return from_unit(T, d, 1.0 / (1.0 + exp(-zz)));
}
__device__ __attribute__((noinline)) double ln_prior_call(const ile_mdn_tr &T, double dec, double D_)
{
    return ile_rng::ln_prior(dec, D_, T.d_min, T.d_max, T.t_ref_max);
}
__device__ __attribute__((noinline)) double ln_hist_call(const double *P, int nb, double ra,
                                                         double dec)
{
    return ln_hist_ratio(P, nb, ra, dec);
}
__device__ __attribute__((noinline)) double ln_mix_call(double eps, double lnn, double lqa)
{
    return logaddexp(log1p(-eps) + lnn, log(eps) + lqa);
}
__device__ __attribute__((noinline)) void hist_call(const double *P, const double *C, int nb,
                                                    uint64_t seed, uint64_t i,
                                                    const ile_mdn_tr &T, double *X)
{
    double x[7];
    uint32_t wd[16];
    ile_rng::prior_words(seed, i, wd);
    int br, bs;
    (void)ile_rng::hist_sample(P, C, nb, wd, T.d_min, T.d_max, T.t_ref_max, x, br, bs);
#pragma unroll
    for (int d = 0; d < D; d++) X[d] = x[d];
}

// Persistent: each workgroup stages W3 in LDS once and its waves loop over
// tiles of 16 samples, one wave a tile, with no barrier between waves.
// SAMPLE: ancestral draw of z~, one dimension per pass, then the density of
// the drawn x by the same code as LOGPDF, so the returned ln q is exactly
// what logpdf gives for it.
//
// The ancestral passes use the masks: a unit of degree e (k mod 6) sees
// z~_0 .. z~_e only, so it is final after pass e, and dimension d needs the
// units of degree below d.  Pass d therefore evaluates the 21 or 22 units of
// degree d - 1 of each layer and no other: their hidden values join those of
// the earlier passes in LDS, and the products run over all 128 units as ever
// (in the same order; the units not yet known have weights of zero and hold
// zeros, set for every tile: weights that BF16 rounds to infinities can make a
// NaN, and 0 times the last tile's would reach this one).  All seven passes
// together are one forward evaluation where they were six, which is what the
// kernel's time was: its tanh and exponentials, a chain a lane waits for at
// one wave per SIMD.  W2 comes from global memory, fetched ahead of the
// layer that uses it, so that LDS holds two waves per SIMD.
// 1e5 draws of the mixture take 242 us (596 with a full evaluation per pass and
// one wave per SIMD; the draws are the same bit for bit).
template <bool SAMPLE>
__global__ __launch_bounds__(IT, 2) void k_mdn_infer(
    const float *__restrict__ theta, const __bf16 *__restrict__ W2b,
    const __bf16 *__restrict__ W3b, const ile_mdn_tr *__restrict__ trp, ile_mdn_mix mix,
    uint64_t seed, int64_t first, int64_t n, double *x_io, int64_t ld, double *ln_p,
    double *ln_q)
{
    __shared__ __attribute__((aligned(16))) __bf16 sW3[W3ROWS * H];
    __shared__ __attribute__((aligned(16))) __bf16 sH1[SAMPLE ? IW : 1][SAMPLE ? 16 * H : 8];
    __shared__ __attribute__((aligned(16))) __bf16 sH2[IW][16 * H];
    __shared__ float sW1[H * 8];
    __shared__ float sb1[H], sb2[H], sb3[O];
    __shared__ float sZ[IW][16 * 8];
    // per sample 16 uniforms, later 8 doubles: x, then ln |dz~/dx|
    __shared__ __attribute__((aligned(16))) float sR[IW][16 * 16];
    __shared__ float sLq[IW][16];
    __shared__ double sP[2 * MAXB], sC[2 * (MAXB + 1)];
    __shared__ ile_mdn_tr sT;

    const int tid = threadIdx.x, lane = tid & 63, r0 = lane & 15, g0 = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int c = tid; c < W3ROWS * 16; c += IT) {
        const int row = c >> 4, col = c & 15;
        *(v8bf *)(sW3 + swz(row, col)) = *(const v8bf *)(W3b + (48 + row) * H + 8 * col);
    }
    for (int j = tid; j < H * 8; j += IT) {
        const int k = j >> 3, d = j & 7;
        sW1[j] = d < D ? theta[OFF_W1 + k * D + d] : 0.f;
    }
    for (int j = tid; j < H; j += IT) {
        sb1[j] = theta[OFF_B1 + j];
        sb2[j] = theta[OFF_B2 + j];
    }
    for (int j = tid; j < O; j += IT) sb3[j] = theta[OFF_B3 + j];
    const bool mixed = mix.nb > 0 && mix.eps > 0.0;
    if (mixed) {
        for (int j = tid; j < 2 * mix.nb; j += IT) sP[j] = mix.P[j];
        for (int j = tid; j < 2 * (mix.nb + 1); j += IT) sC[j] = mix.C[j];
    }
    if (tid == 0) sT = *trp;
    __bf16 *H1s = sH1[SAMPLE ? w : 0], *H2s = sH2[w];
    __syncthreads();
    const float sfloor = (float)sT.sigma_floor, kappa = (float)sT.sigma_scale;
    float *Zs = sZ[w], *Rs = sR[w];
    double *Xs = reinterpret_cast<double *>(Rs);   // [16][8]
    // tile t goes to workgroup t mod grid, its waves in turn
    for (int64_t tile = blockIdx.x + (int64_t)gridDim.x * w; tile * 16 < n;
         tile += (int64_t)gridDim.x * IW) {
        // the lane's place through a value the compiler cannot see, or it
        // would hold every weight fragment in registers across the tiles
        int zero_ = 0;
        asm volatile("" : "+s"(zero_));
        const int r = r0 + zero_, g = g0 + zero_;
        const auto frag = [&](const __bf16 *A, int ks) {   // row r, units 32 ks + 8 g ..
            return *(const v8bf *)(A + swz(r, 4 * ks + g));
        };
        // outputs of dimension d >= 1 for samples 4 g + v, component r
        const auto layer3 = [&](const v8bf (&A2)[4], int d, v4f (&t3)[3]) {
#pragma unroll
            for (int j = 0; j < 3; j++) t3[j] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ks++)
#pragma unroll
                for (int j = 0; j < 3; j++)
                    t3[j] = mfma(A2[ks], *(const v8bf *)(sW3 + swz(48 * (d - 1) + 16 * j + r, 4 * ks + g)),
                                 t3[j]);
        };
        const int64_t i = tile * 16 + r;   // sample of the lanes of column r
        const bool valid = i < n;
        if (SAMPLE) {
            // no unit of this tile is known yet
            v8bf none;
#pragma unroll
            for (int q = 0; q < 8; q++) none[q] = (__bf16)0.f;
#pragma unroll
            for (int c = lane; c < 16 * 16; c += 64) {
                *(v8bf *)(H1s + 8 * c) = none;
                *(v8bf *)(H2s + 8 * c) = none;
            }
            // 16 uniforms per sample: group g computes Philox blocks 2g, 2g+1
#pragma unroll
            for (int bb = 0; bb < 2; bb++) {
                uint32_t q[4];
                ile_rng::block(seed, (uint64_t)(first + i), 2 * g + bb, ile_rng::kTagMdn, q);
                Rs[r * 16 + 4 * g + 2 * bb] = (float)ile_rng::u53(q[0], q[1]);
                Rs[r * 16 + 4 * g + 2 * bb + 1] = (float)ile_rng::u53(q[2], q[3]);
            }
            wave_lds_sync();
            // uniforms 0..6: component choices; 7..14 -> 8 normals (Box-Muller);
            // 15: which member of the defensive mixture draws the sample
            {
                const float a = Rs[r * 16 + 7 + 2 * g], b = Rs[r * 16 + 8 + 2 * g];
                const float rad = sqrtf(-2.f * logf(a));
                float sn, cs;
                sincosf(6.28318530717958648f * b, &sn, &cs);
                Rs[r * 16 + 7 + 2 * g] = rad * cs;
                Rs[r * 16 + 8 + 2 * g] = rad * sn;
            }
            wave_lds_sync();
#pragma unroll 1
            for (int d = 0; d < D; d++) {
                v4f t3[3];
                if (d > 0) {
                    const int e = d - 1;             // the degree that is new
                    const int ne = e < 2 ? 22 : 21;  // its units: e, e + 6, ...
                    // layer-2 rows of those units, in flight during layer 1
                    v8bf B[2][4];
#pragma unroll
                    for (int t = 0; t < 2; t++) {
                        const int k2 = e + 6 * min(16 * t + r, ne - 1);
#pragma unroll
                        for (int ks = 0; ks < 4; ks++)
                            B[t][ks] = *(const v8bf *)(W2b + k2 * H + 32 * ks + 8 * g);
                    }
                    float z[7];
#pragma unroll
                    for (int c = 0; c < D; c++) z[c] = c < d ? Zs[r * 8 + c] : 0.f;
#pragma unroll
                    for (int j0 = 0; j0 < 24; j0 += 4) {
                        const int j = j0 + g, k = e + 6 * min(j, ne - 1);
                        float a = sb1[k];
#pragma unroll
                        for (int c = 0; c < D - 1; c++) a = fmaf(sW1[k * 8 + c], z[c], a);
                        H1s[swz(r, k >> 3) + (k & 7)] = (__bf16)tanhf(a);
                    }
                    wave_lds_sync();
                    v4f acc[2];
                    acc[0] = acc[1] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ks = 0; ks < 4; ks++) {
                        const v8bf A = frag(H1s, ks);
#pragma unroll
                        for (int t = 0; t < 2; t++) acc[t] = mfma(A, B[t][ks], acc[t]);
                    }
#pragma unroll
                    for (int t = 0; t < 2; t++) {
                        const int k2 = e + 6 * min(16 * t + r, ne - 1);
                        const float bb = sb2[k2];
#pragma unroll
                        for (int v = 0; v < 4; v++)
                            H2s[swz(4 * g + v, k2 >> 3) + (k2 & 7)] = (__bf16)tanhf(acc[t][v] + bb);
                    }
                    wave_lds_sync();
                    v8bf A2[4];
#pragma unroll
                    for (int ks = 0; ks < 4; ks++) A2[ks] = frag(H2s, ks);
                    layer3(A2, d, t3);
                } else {
                    // dimension 0 sees no hidden unit: its outputs are the biases
#pragma unroll
                    for (int j = 0; j < 3; j++) t3[j] = v4f{0.f, 0.f, 0.f, 0.f};
                }
#pragma unroll
                for (int v = 0; v < 4; v++) {
                    const int s = 4 * g + v;
                    const float al = t3[0][v] + sb3[48 * d + r];
                    const float mu = t3[1][v] + sb3[48 * d + 16 + r];
                    const float rho = t3[2][v] + sb3[48 * d + 32 + r];
                    // categorical draw: first component whose cumulative weight
                    // exceeds u times the total
                    const float ma = gmax(al);
                    const float cum = row_scan(expf(al - ma));
                    const float tot = row_last(cum);
                    const unsigned long long bal = __ballot(cum > Rs[s * 16 + d] * tot);
                    const unsigned bits = (unsigned)(bal >> (16 * g)) & 0xffffu;
                    const int cs = bits ? __ffs(bits) - 1 : 15;
                    const float sig = kappa * (sfloor + softplusf(rho));
                    if (r == cs) Zs[s * 8 + d] = mu + sig * Rs[s * 16 + 7 + d];
                }
                wave_lds_sync();
            }
        }
        // ---- x: lane (r, g) holds dimensions g and g + 4 of sample r
        bool hist = false;
        if (SAMPLE) {
            hist = mixed && Rs[r * 16 + 15] < (float)mix.eps;
            wave_lds_sync();   // Xs takes the place of Rs
            if (hist && g == 0)
                hist_call(sP, sC, mix.nb, seed, (uint64_t)(first + i), sT, Xs + r * 8);
        }
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int d = g + 4 * h;
            if (d >= D) continue;
            if (SAMPLE) {
                if (!hist) Xs[r * 8 + d] = from_z_call(sT, d, Zs[r * 8 + d]);
            } else {
                const double dflt = d == 5 ? 0.5 * (sT.d_min + sT.d_max)
                                           : d == 6 ? 0.0 : (d == 1 || d == 4) ? 0.1 : 1.0;
                Xs[r * 8 + d] = valid ? x_io[d * ld + i] : dflt;
            }
        }
        wave_lds_sync();
        // ---- density of x: the same code in both modes
        // layer-2 fragments of the first two k-steps, in flight meanwhile
        v8bf B2[2][8];
        const auto load_w2 = [&](int k0) {
#pragma unroll
            for (int ks = 0; ks < 2; ks++)
#pragma unroll
                for (int t = 0; t < 8; t++)
                    B2[ks][t] = *(const v8bf *)(W2b + (16 * t + r) * H + 32 * (k0 + ks) + 8 * g);
        };
        double lp = 0.0, lqa = 0.0;
        if (g == 0) {
            lp = ln_prior_call(sT, Xs[r * 8 + 1], Xs[r * 8 + 5]);
            if (mixed) lqa = lp + ln_hist_call(sP, mix.nb, Xs[r * 8], Xs[r * 8 + 1]);
        }
        double xd[2];
#pragma unroll
        for (int h = 0; h < 2; h++) xd[h] = g + 4 * h < D ? Xs[r * 8 + g + 4 * h] : 0.0;
        wave_lds_sync();
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int d = g + 4 * h;
            if (d >= D) continue;
            const zterm t = to_z_call(sT, d, xd[h]);
            Xs[r * 8 + d] = t.lj;
            Zs[r * 8 + d] = t.z;
        }
        wave_lds_sync();
        {
            float z[7];
#pragma unroll
            for (int e = 0; e < D; e++) z[e] = Zs[r * 8 + e];
            load_w2(0);
            v8bf A1[4];
            layer1(sW1, 8, sb1, z, g, A1);
            v4f acc[8];
#pragma unroll
            for (int t = 0; t < 8; t++) acc[t] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 2; ks++)
#pragma unroll
                for (int t = 0; t < 8; t++) acc[t] = mfma(A1[ks], B2[ks][t], acc[t]);
            load_w2(2);
#pragma unroll
            for (int ks = 0; ks < 2; ks++)
#pragma unroll
                for (int t = 0; t < 8; t++) acc[t] = mfma(A1[2 + ks], B2[ks][t], acc[t]);
#pragma unroll
            for (int t = 0; t < 8; t++) {
                const int k2 = 16 * t + r;
                const float bb = sb2[k2];
#pragma unroll
                for (int v = 0; v < 4; v++)
                    H2s[swz(4 * g + v, k2 >> 3) + (k2 & 7)] = (__bf16)tanhf(acc[t][v] + bb);
            }
            wave_lds_sync();
            v8bf A2[4];
#pragma unroll
            for (int ks = 0; ks < 4; ks++) A2[ks] = frag(H2s, ks);
            float lqz[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (int d = 0; d < D; d++) {
                v4f t3[3];
                if (d > 0)
                    layer3(A2, d, t3);
                else
#pragma unroll
                    for (int j = 0; j < 3; j++) t3[j] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int v = 0; v < 4; v++) {
                    float sig, rr, ell, la;
                    lqz[v] += mix_lnq(t3[0][v] + sb3[48 * d + r], t3[1][v] + sb3[48 * d + 16 + r],
                                      t3[2][v] + sb3[48 * d + 32 + r], Zs[(4 * g + v) * 8 + d],
                                      sfloor, kappa, sig, rr, ell, la);
                }
            }
            if (r == 0)
                for (int v = 0; v < 4; v++) sLq[w][4 * g + v] = lqz[v];
        }
        wave_lds_sync();
        if (SAMPLE && valid)
#pragma unroll
            for (int h = 0; h < 2; h++)
                if (g + 4 * h < D) x_io[(g + 4 * h) * ld + i] = xd[h];
        if (g == 0 && valid) {
            const double jac = sum_lj(Xs + r * 8);
            const double lnn = jac == -INFINITY ? -INFINITY : (double)sLq[w][r] + jac;
            double lq = mixed ? ln_mix_call(mix.eps, lnn, lqa) : lnn;
            if (SAMPLE) {
                // a draw on the boundary of the support (probability 0) has
                // p = 0: a finite ln q makes its weight exactly 0
                if (!(lp > -INFINITY) || !(lq > -INFINITY)) lq = 0.0;
                if (ln_p) ln_p[i] = lp;
            }
            ln_q[i] = lq;
        }
        wave_lds_sync();
    }
}

// ------------------------------------------------------------ training
// Forward and backward of 64 samples (batch slots blockIdx.x*64 ..): the
// workgroup's gradient of  L = -sum_s w_s ln q(z~_s)  (not yet divided by
// sum w), its loss sum and weight sum go to part[blockIdx.x][.].
//
// A batch of 16384 is 256 such workgroups, one per CU, so the time is the
// longest chain of one wave; with a wave per 16 samples each walked all of it
// alone and read all the weights (52.7 us a launch).  Sixteen waves share the
// 64 samples instead, two tiles of 16 samples a wave, so that a weight
// fragment serves both: wave w = 8 p + t takes output tile t of layer 2 and of
// both backward products for tiles 2 p and 2 p + 1, and dimension t < 7 of the
// mixture; the rows of the weight-gradient tiles are dealt to all sixteen.
// Every sum keeps its order, so the gradient is the same bit for bit.  32.8 us
// a launch: 9.6 to the end of layer 2, about 10 for the mixture (its
// exponentials and logarithms), the rest the backward products and the rows.
constexpr int GW = 16, GT = 64 * GW;

// A partial row holds what the masks let through.  With the hidden units in
// the order of their degree (mdn_unit), dimension d's rows of W3 use the first
// mdn_count(d) of them and a row of W2 of degree e the first mdn_count(e + 1),
// so of the 16 x 16 gradient tiles [output][unit] only those left of these
// edges exist: 137 of 232, and the row is 146 KB instead of 244 (of both it is
// the bytes written here and read by the update that count).  Then b1, b2, b3,
// W1, the loss sum and the weight sum.
__host__ __device__ constexpr int mdn_unit(int i)   // i-th unit by degree
{
    return i < 44 ? i / 22 + 6 * (i % 22) : 2 + (i - 44) / 21 + 6 * ((i - 44) % 21);
}
__host__ __device__ constexpr int mdn_count(int e)   // units of degree below e
{
    return e <= 2 ? 22 * e : 44 + 21 * (e - 2);
}
constexpr int N_TILE3 = 93, N_TILE = 137;   // tiles of W3, and with those of W2
struct mdn_tiles {
    unsigned char ot[N_TILE], kt[N_TILE];
    int n3, n;
};
constexpr mdn_tiles make_tiles()
{
    mdn_tiles T{};
    int n = 0;
    for (int ot = 0; ot < O / 16; ot++)
        for (int kt = 0; 16 * kt < mdn_count(ot / 3); kt++, n++) {
            T.ot[n] = (unsigned char)ot;
            T.kt[n] = (unsigned char)kt;
        }
    T.n3 = n;
    for (int ot = 0; ot < H / 16; ot++)
        for (int kt = 0; 16 * kt < mdn_count(mdn_unit(16 * ot + 15) % 6 + 1); kt++, n++) {
            T.ot[n] = (unsigned char)ot;
            T.kt[n] = (unsigned char)kt;
        }
    T.n = n;
    return T;
}
static_assert(make_tiles().n3 == N_TILE3 && make_tiles().n == N_TILE, "tile counts");
__device__ constexpr mdn_tiles kTiles = make_tiles();
constexpr int P_B1 = 256 * N_TILE, P_B2 = P_B1 + H, P_B3 = P_B2 + H, P_W1 = P_B3 + O,
              P_LOSS = P_W1 + H * D, P_WSUM = P_LOSS + 1;
static_assert(P_WSUM < NPART, "partial row");
// parameter index of entry p < P_LOSS of a partial row
__device__ inline int mdn_param_of(int p)
{
    if (p < P_B1) {
        const int tile = p >> 8, r = (p >> 4) & 15;
        const int o = 16 * kTiles.ot[tile] + r, k = mdn_unit(16 * kTiles.kt[tile] + (p & 15));
        return tile < N_TILE3 ? OFF_W3 + o * H + k : OFF_W2 + mdn_unit(o) * H + k;
    }
    return p < P_B2 ? OFF_B1 + p - P_B1
         : p < P_B3 ? OFF_B2 + p - P_B2
         : p < P_W1 ? OFF_B3 + p - P_B3 : OFF_W1 + p - P_W1;
}
constexpr int DLD = 72;    // LDS row of the last dimension's 48 outputs (of 64)
__global__ __launch_bounds__(GT) void k_mdn_grad(
    const float *__restrict__ theta, const __bf16 *__restrict__ W2b,
    const __bf16 *__restrict__ W3b, const __bf16 *__restrict__ W2t,
    const __bf16 *__restrict__ W3t, const ile_mdn_tr *__restrict__ trp,
    const float *__restrict__ zt, int64_t ldz, const int32_t *__restrict__ idx,
    const double *__restrict__ wts, int batch, float *__restrict__ part)
{
    __shared__ float sZ[64 * 8];
    __shared__ float sWt[64];
    __shared__ float sLq[D * 64];                                    // ln q_d of each sample
    __shared__ __attribute__((aligned(16))) __bf16 sH1T[H * SLD];    // h1 [unit][sample]
    __shared__ __attribute__((aligned(16))) __bf16 sH2T[H * SLD];    // h2 [unit][sample]
    __shared__ __attribute__((aligned(16))) __bf16 sDOT[O * SLD];    // dL/do [output][sample]
    __shared__ __attribute__((aligned(16))) __bf16 sHs[4][16 * WLD]; // per tile: h2, then dL/da2 [s][unit]
    // in turn: h1 [s][unit] of each tile; dL/do [s][o] of each tile and pair of
    // dimensions; dL/da2 and dL/da1 [unit][sample]
    constexpr int DOP = 16 * CLD, DOM = 3 * DOP + 16 * DLD;
    static_assert(4 * DOM >= 2 * H * SLD && 4 * DOM >= 4 * 16 * WLD, "shared region");
    __shared__ __attribute__((aligned(16))) __bf16 sU[4 * DOM];
    __shared__ float sPar[OFF_W2 + H + O];   // FP32 W1, b1, b2, b3
    __bf16 *sDA2T = sU, *sDA1T = sU + H * SLD;

    const float *W1 = sPar, *b1 = sPar + OFF_B1, *b2 = sPar + OFF_W2,
                *b3 = sPar + OFF_W2 + H;
    const float sfloor = (float)trp->sigma_floor;
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), t = w & 7, m0 = 2 * (w >> 3);
    const int kr = 16 * t + r;   // the lane's unit as an output of tile t

    // layer-2 fragments first: their loads overlap the staging below
    v8bf B2f[4];
#pragma unroll
    for (int ks = 0; ks < 4; ks++) B2f[ks] = *(const v8bf *)(W2b + kr * H + 32 * ks + 8 * g);
    if (tid < 512) {
        const int s = tid >> 3, d = tid & 7;
        const int64_t b = (int64_t)blockIdx.x * 64 + s;
        const bool valid = b < batch;
        const int64_t row = valid ? (idx ? (int64_t)idx[b] : b) : 0;
        sZ[s * 8 + d] = (valid && d < D) ? zt[d * ldz + row] : 0.f;
        if (d == 7) sWt[s] = valid ? (wts ? (float)wts[row] : 1.f) : 0.f;
    }
    for (int e = tid; e < OFF_W2 + H + O; e += GT)
        sPar[e] = e < OFF_W2 ? theta[OFF_W1 + e]
                : e < OFF_W2 + H ? theta[OFF_B2 + e - OFF_W2] : theta[OFF_B3 + e - OFF_W2 - H];
    __syncthreads();

    // ---- layer 1: wave (m, q) takes units 32 q + 8 g .. of tile m
    {
        const int m = w >> 2, q = w & 3;
        float z[7];
#pragma unroll
        for (int d = 0; d < D; d++) z[d] = sZ[(16 * m + r) * 8 + d];
        v8bf A;
#pragma unroll
        for (int i = 0; i < 8; i++) {
            const int k = 32 * q + 8 * g + i;
            float a = b1[k];
#pragma unroll
            for (int d = 0; d < D; d++) a = fmaf(W1[k * D + d], z[d], a);
            A[i] = (__bf16)ftanh(a);
            sH1T[k * SLD + 16 * m + r] = A[i];
        }
        *(v8bf *)(sU + m * 16 * WLD + r * WLD + 32 * q + 8 * g) = A;
    }
    __syncthreads();
    // ---- layer 2
    float h2v[2][4];
    {
        v4f acc[2];
        acc[0] = acc[1] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 4; ks++)
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const v8bf A = *(const v8bf *)(sU + ((m0 + h) * 16 + r) * WLD + 32 * ks + 8 * g);
                acc[h] = mfma(A, B2f[ks], acc[h]);
            }
        const float bb = b2[kr];
#pragma unroll
        for (int h = 0; h < 2; h++) {
            v4bf pk;
#pragma unroll
            for (int v = 0; v < 4; v++) {
                const float x = ftanh(acc[h][v] + bb);
                h2v[h][v] = x;
                pk[v] = (__bf16)x;
                sHs[m0 + h][(4 * g + v) * WLD + kr] = pk[v];
            }
            *(v4bf *)(sH2T + kr * SLD + 16 * (m0 + h) + 4 * g) = pk;
        }
    }
    v8bf Bn[12];
    if (t < D) load_w3_dim(W3b, H, t, r, g, Bn);
    __syncthreads();

    // ---- layer 3 and the mixture's gradients, dimension t
    if (t < D) {
        const int d = t, p = d >> 1, dd = d & 1;
        const int cld = p < 3 ? CLD : DLD;
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int m = m0 + h, s0 = 16 * m;
            __bf16 *DOc = sU + m * DOM + p * DOP;
            v4f t3[3];
#pragma unroll
            for (int j = 0; j < 3; j++) t3[j] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ks++) {
                const v8bf A = *(const v8bf *)(sHs[m] + r * WLD + 32 * ks + 8 * g);
#pragma unroll
                for (int j = 0; j < 3; j++) t3[j] = mfma(A, Bn[3 * ks + j], t3[j]);
            }
            v4bf ga, gm, gr;
#pragma unroll
            for (int v = 0; v < 4; v++) {
                const int s = 4 * g + v;
                const float al = t3[0][v] + b3[48 * d + r];
                const float mu = t3[1][v] + b3[48 * d + 16 + r];
                const float rho = t3[2][v] + b3[48 * d + 32 + r];
                const float ws = sWt[s0 + s];
                float rs, rr, ell, la;
                const float lq = mix_lnq_fast(al, mu, rho, sZ[(s0 + s) * 8 + d], sfloor, rs, rr, ell, la);
                const float gam = fexp(ell - lq), pi = fexp(al - la);
                if (r == 0) sLq[d * 64 + s0 + s] = lq;
                ga[v] = (__bf16)(-ws * (gam - pi));
                gm[v] = (__bf16)(-ws * gam * rr * rs);
                gr[v] = (__bf16)(-ws * gam * (rr * rr - 1.f) * rs * fsigmoid(rho));
                DOc[s * cld + 48 * dd + r] = ga[v];
                DOc[s * cld + 48 * dd + 16 + r] = gm[v];
                DOc[s * cld + 48 * dd + 32 + r] = gr[v];
            }
            *(v4bf *)(sDOT + (48 * d + r) * SLD + s0 + 4 * g) = ga;
            *(v4bf *)(sDOT + (48 * d + 16 + r) * SLD + s0 + 4 * g) = gm;
            *(v4bf *)(sDOT + (48 * d + 32 + r) * SLD + s0 + 4 * g) = gr;
        }
    } else {
        // outputs 48 .. 63 of the last pair: the padding of its K
#pragma unroll
        for (int h = 0; h < 2; h++)
#pragma unroll
            for (int v = 0; v < 4; v++)
                sU[(m0 + h) * DOM + 3 * DOP + (4 * g + v) * DLD + 48 + r] = (__bf16)0.f;
    }
    // the backward fragments, in flight across the barrier
    v8bf Bt[11];
#pragma unroll
    for (int c = 0; c < 11; c++)
        Bt[c] = *(const v8bf *)(W3t + kr * W3T_LD + 32 * c + 8 * g);
    __syncthreads();

    // ---- dL/dh2 = dL/do W3 (pair p is outputs 96 p ..; the last k-step of the
    // last pair would be all zeros)
    v4f dh[2];
    dh[0] = dh[1] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < 11; c++) {
        const int p = c / 3, ks = c % 3, cld = p < 3 ? CLD : DLD;
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const v8bf A = *(const v8bf *)(sU + (m0 + h) * DOM + p * DOP + r * cld + 32 * ks + 8 * g);
            dh[h] = mfma(A, Bt[c], dh[h]);
        }
    }
    v8bf B2[4];
#pragma unroll
    for (int ks = 0; ks < 4; ks++) B2[ks] = *(const v8bf *)(W2t + kr * H + 32 * ks + 8 * g);
    __syncthreads();   // sU changes hands
    // ---- dL/da2 = dL/dh2 (1 - h2^2)
#pragma unroll
    for (int h = 0; h < 2; h++) {
        v4bf pk;
#pragma unroll
        for (int v = 0; v < 4; v++) {
            pk[v] = (__bf16)(dh[h][v] * (1.f - h2v[h][v] * h2v[h][v]));
            sHs[m0 + h][(4 * g + v) * WLD + kr] = pk[v];
        }
        *(v4bf *)(sDA2T + kr * SLD + 16 * (m0 + h) + 4 * g) = pk;
    }
    __syncthreads();

    // ---- dL/dh1 = W2^T dL/da2, dL/da1 = dL/dh1 (1 - h1^2), h1 recomputed in FP32
    {
        v4f dh1[2];
        dh1[0] = dh1[1] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 4; ks++)
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const v8bf A = *(const v8bf *)(sHs[m0 + h] + r * WLD + 32 * ks + 8 * g);
                dh1[h] = mfma(A, B2[ks], dh1[h]);
            }
        float wk[7];
#pragma unroll
        for (int d = 0; d < D; d++) wk[d] = W1[kr * D + d];
        const float bk = b1[kr];
#pragma unroll
        for (int h = 0; h < 2; h++) {
            v4bf pk;
#pragma unroll
            for (int v = 0; v < 4; v++) {
                const int s = 16 * (m0 + h) + 4 * g + v;
                float a = bk;
#pragma unroll
                for (int d = 0; d < D; d++) a = fmaf(wk[d], sZ[s * 8 + d], a);
                const float x = ftanh(a);
                pk[v] = (__bf16)(dh1[h][v] * (1.f - x * x));
            }
            *(v4bf *)(sDA1T + kr * SLD + 16 * (m0 + h) + 4 * g) = pk;
        }
    }
    __syncthreads();

    // ---- weight gradients over the workgroup's 64 samples
    float *P = part + (size_t)blockIdx.x * NPART;
    // (products taken as (dL/dW)^T tiles, so that each lane holds four
    // consecutive units of one output row: a tile is one 1 KB store)
    for (int e = w; e < N_TILE; e += GW) {
        const bool third = e < N_TILE3;
        const int o = 16 * kTiles.ot[e] + r, k = mdn_unit(16 * kTiles.kt[e] + r);
        const __bf16 *G = (third ? sDOT + o * SLD : sDA2T + mdn_unit(o) * SLD) + 8 * g;
        const __bf16 *X = (third ? sH2T : sH1T) + k * SLD + 8 * g;
        v4f a = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 2; ks++)
            a = mfma(*(const v8bf *)(X + 32 * ks), *(const v8bf *)(G + 32 * ks), a);
        *(v4f *)(P + 256 * e + 16 * r + 4 * g) = a;
    }
    // biases, W1, the loss and the weight sum: one sum a thread
    for (int e = tid; e < O + 2 * H + H * D; e += GT) {
        if (e < O + 2 * H) {
            const __bf16 *row = e < O ? sDOT + e * SLD
                              : e < O + H ? sDA2T + (e - O) * SLD : sDA1T + (e - O - H) * SLD;
            float acc = 0.f;
            for (int s = 0; s < 64; s++) acc += (float)row[s];
            P[e < O ? P_B3 + e : e < O + H ? P_B2 + e - O : P_B1 + e - O - H] = acc;
        } else if (e < O + 2 * H + H * D) {
            const int f = e - O - 2 * H, k = f / D, d = f % D;
            float acc = 0.f;
            for (int s = 0; s < 64; s++) acc = fmaf((float)sDA1T[k * SLD + s], sZ[s * 8 + d], acc);
            P[P_W1 + f] = acc;
        }
    }
    if (w == GW - 1 && lane < 16) {
        // lane 4 m + g: samples 16 m + 4 g .. of tile m, then the tiles in order
        float l = 0.f;
#pragma unroll
        for (int d = 0; d < D; d++)
#pragma unroll
            for (int v = 0; v < 4; v++) l -= sWt[4 * lane + v] * sLq[d * 64 + 4 * lane + v];
        l += __shfl_xor(l, 1);
        l += __shfl_xor(l, 2);
        const float l1 = __shfl(l, 4), l2 = __shfl(l, 8), l3 = __shfl(l, 12);
        if (lane == 0) {
            P[P_LOSS] = l + l1 + l2 + l3;
            float ws = 0.f;
            for (int s = 0; s < 64; s++) ws += sWt[s];
            P[P_WSUM] = ws;
        }
    }
}

__device__ inline void write_copies(const ile_mdn_dev &M, int j, float th)
{
    const __bf16 b = (__bf16)th;
    if (j >= OFF_W2 && j < OFF_B2) {
        const int q = j - OFF_W2, o = q / H, k = q % H;
        M.W2b[o * H + k] = b;
        M.W2t[k * H + o] = b;
    } else if (j >= OFF_W3 && j < OFF_B3) {
        const int q = j - OFF_W3, o = q / H, k = q % H;
        M.W3b[o * H + k] = b;
        M.W3t[k * W3T_LD + o] = b;
    }
}

__global__ __launch_bounds__(256) void k_mdn_cast(ile_mdn_dev M)
{
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j < NPARAM) write_copies(M, j, M.theta[j]);
}

// Sum the partial rows in a fixed order, mask, normalize by the weight sum;
// then one Adam step (beta1 0.9, beta2 0.999, eps 1e-8) on the FP32 weights
// and refresh the BF16 copies.  A workgroup serves 64 entries of the rows with
// four row slices each (rows s, s+4, s+8, ...), so the read of all rows runs at
// four times the occupancy; the slices combine in slice order.  Bound by that
// read, which runs at the rate of a large copy (37 MB of a batch of 16384 in
// 8.5 us; 12.2 us when the rows held the masked entries too).  A masked
// parameter's gradient is zero: its weight and moments are zeros and stay so
// (grad, if wanted, holds zeros there already).
constexpr int UPD_P = 64;   // entries per workgroup
__global__ __launch_bounds__(256) void k_mdn_update(ile_mdn_dev M, const float *__restrict__ part,
                                                    int np, float *grad, double *loss, int adam,
                                                    float bc1, float bc2, float lr)
{
    __shared__ float red_g[4][UPD_P], red_w[4][UPD_P];
    const int jj = threadIdx.x & (UPD_P - 1), sl = threadIdx.x / UPD_P;
    const int p = blockIdx.x * UPD_P + jj;
    float ws = 0.f, gs = 0.f;
    if (p < P_LOSS) {
        // the loads are independent, so unrolling lets many be in flight
#pragma unroll 8
        for (int t = sl; t < np; t += 4) {
            ws += part[(size_t)t * NPART + P_WSUM];
            gs += part[(size_t)t * NPART + p];
        }
    }
    red_g[sl][jj] = gs;
    red_w[sl][jj] = ws;
    __syncthreads();
    if (sl != 0 || p >= P_LOSS) return;
    gs = ((red_g[0][jj] + red_g[1][jj]) + red_g[2][jj]) + red_g[3][jj];
    ws = ((red_w[0][jj] + red_w[1][jj]) + red_w[2][jj]) + red_w[3][jj];
    if (p == 0 && loss) {
        float ls = 0.f;
#pragma unroll 16
        for (int t = 0; t < np; t++) ls += part[(size_t)t * NPART + P_LOSS];
        *loss = ws > 0.f ? (double)ls / (double)ws : 0.0;
    }
    const int j = mdn_param_of(p);
    if (!ile_mdn_trainable(j)) return;
    const float gj = ws > 0.f ? gs / ws : 0.f;
    if (grad) grad[j] = gj;
    if (!adam) return;
    const float m = 0.9f * M.m[j] + 0.1f * gj;
    const float v = 0.999f * M.v[j] + 0.001f * gj * gj;
    M.m[j] = m;
    M.v[j] = v;
    const float th = M.theta[j] - lr * (m / bc1) / (sqrtf(v / bc2) + 1e-8f);
    M.theta[j] = th;
    write_copies(M, j, th);
}

// ------------------------------------------------- training-set pieces

// Transform fit, multi-block with fixed partitions and fixed-order merges
// (bit-reproducible).  Tempering of the training weights w = exp(beta (ln w
// - max)) over the finite ln w: beta = 1 if the Kish effective size
// (sum w)^2 / sum w^2 reaches max(1, ess_frac * count), else 30 halvings of
// [0, 1] keeping the lower end whose effective size reaches it.  Then the
// weighted circular means of ra, psi, phi (origins) and the weighted mean
// and standard deviation of z = logit(u) (scale >= 1e-3).
//
// Workspace ws: [0, 16) the state below, [16, 16 + FB * 16) block partials.
constexpr int FB = 256;   // blocks of the partial-sum kernels
enum { S_MAX = 0, S_TARGET, S_LO, S_HI, S_BEVAL, S_BETA, S_DONE, S_CNT };

// fixed-order tree sum of `nv` values per thread over a 256-thread block;
// thread 0 writes them to out[0..nv)
template <int NV>
__device__ inline void block_sums256(double (&v)[NV], double *red, double *out)
{
    for (int q = 0; q < NV; q++) {
        red[threadIdx.x] = v[q];
        __syncthreads();
        for (int s = 128; s > 0; s >>= 1) {
            if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
            __syncthreads();
        }
        if (threadIdx.x == 0) out[q] = red[0];
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void k_fit_max(const double *__restrict__ lnw, int64_t n,
                                                 double *ws)
{
    __shared__ double red[256];
    double mx = -INFINITY, cnt = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)FB * 256)
        if (isfinite(lnw[i])) {
            mx = fmax(mx, lnw[i]);
            cnt += 1.0;
        }
    red[threadIdx.x] = mx;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
        __syncthreads();
    }
    const double bm = red[0];
    __syncthreads();
    double c1[1] = {cnt};
    double *P = ws + 16 + blockIdx.x * 16;
    block_sums256<1>(c1, red, P + 1);
    if (threadIdx.x == 0) P[0] = bm;
}

// The single-workgroup steps fetch the FB block partials with all their lanes
// (one memory round trip instead of one a partial: 41 us for the moments) into
// LDS, then one thread a sum adds them in block order.
template <int NV>
__device__ inline void fetch_parts(const double *ws, double (*sp)[FB + 1])
{
    for (int e = threadIdx.x; e < FB * NV; e += blockDim.x)
        sp[e % NV][e / NV] = ws[16 + (e / NV) * 16 + e % NV];
    __syncthreads();
}
__device__ inline double sum_parts(const double *sp)
{
    double v = 0.0;
#pragma unroll 16
    for (int b = 0; b < FB; b++) v += sp[b];
    return v;
}

__global__ __launch_bounds__(256) void k_fit_init(double *ws, double ess_frac)
{
    __shared__ double sp[2][FB + 1];
    fetch_parts<2>(ws, sp);
    if (threadIdx.x != 0) return;
    double mx = -INFINITY;
    const double cnt = sum_parts(sp[1]);
    for (int b = 0; b < FB; b++) mx = fmax(mx, sp[0][b]);
    ws[S_MAX] = mx;
    ws[S_CNT] = cnt;
    ws[S_TARGET] = fmax(1.0, ess_frac * cnt);
    ws[S_LO] = 0.0;
    ws[S_HI] = 1.0;
    ws[S_BEVAL] = 1.0;
    ws[S_BETA] = 1.0;
    ws[S_DONE] = cnt > 0 ? 0.0 : 1.0;
}

__global__ __launch_bounds__(256) void k_fit_ess_part(const double *__restrict__ lnw, int64_t n,
                                                      double *ws)
{
    __shared__ double red[256];
    if (ws[S_DONE] != 0.0) return;   // uniform across the grid
    const double m = ws[S_MAX], beta = ws[S_BEVAL];
    double v[2] = {0.0, 0.0};
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)FB * 256) {
        if (!isfinite(lnw[i])) continue;
        const double e = exp(beta * (lnw[i] - m));
        v[0] += e;
        v[1] += e * e;
    }
    block_sums256<2>(v, red, ws + 16 + blockIdx.x * 16);
}

// it = 0 judges beta = 1; it = 1..30 halve [lo, hi]
__global__ __launch_bounds__(256) void k_fit_ess_step(double *ws, int it)
{
    __shared__ double sp[2][FB + 1];
    if (ws[S_DONE] != 0.0) return;   // uniform: thread 0 writes it after the barrier
    fetch_parts<2>(ws, sp);
    if (threadIdx.x != 0) return;
    const double s1 = sum_parts(sp[0]), s2 = sum_parts(sp[1]);
    const bool ok = s2 > 0.0 && s1 * s1 / s2 >= ws[S_TARGET];
    if (it == 0) {
        if (ok) {
            ws[S_BETA] = 1.0;
            ws[S_DONE] = 1.0;
            return;
        }
    } else if (ok) {
        ws[S_LO] = ws[S_BEVAL];
    } else {
        ws[S_HI] = ws[S_BEVAL];
    }
    ws[S_BETA] = ws[S_LO];
    ws[S_BEVAL] = 0.5 * (ws[S_LO] + ws[S_HI]);
}

__device__ inline double fit_weight(const double *ws, double l)
{
    return isfinite(l) ? exp(ws[S_BETA] * (l - ws[S_MAX])) : 0.0;
}

__global__ __launch_bounds__(256) void k_fit_circ_part(const double *__restrict__ x, int64_t ld,
                                                       const double *__restrict__ lnw, int64_t n,
                                                       double *ws)
{
    __shared__ double red[256];
    const int pd[3] = {0, 2, 3};
    const double per[3] = {kTwoPi, kPi, kTwoPi};
    double v[6] = {0, 0, 0, 0, 0, 0};
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)FB * 256) {
        const double wi = fit_weight(ws, lnw[i]);
        if (wi == 0.0) continue;
#pragma unroll
        for (int j = 0; j < 3; j++) {
            double sn, cs;
            sincos(kTwoPi * x[pd[j] * ld + i] / per[j], &sn, &cs);
            v[2 * j] += wi * cs;
            v[2 * j + 1] += wi * sn;
        }
    }
    block_sums256<6>(v, red, ws + 16 + blockIdx.x * 16);
}

__global__ __launch_bounds__(256) void k_fit_circ_fin(double *ws, ile_mdn_tr *tr)
{
    __shared__ double sp[6][FB + 1];
    fetch_parts<6>(ws, sp);
    const int j = threadIdx.x;
    if (j >= 3) return;
    const double per[3] = {kTwoPi, kPi, kTwoPi};
    const double sc = sum_parts(sp[2 * j]), ss = sum_parts(sp[2 * j + 1]);
    tr->origin[j] = atan2(ss, sc) * per[j] / kTwoPi;
}

__global__ __launch_bounds__(256) void k_fit_mom_part(const double *__restrict__ x, int64_t ld,
                                                      const double *__restrict__ lnw, int64_t n,
                                                      const ile_mdn_tr *__restrict__ trp, double *ws)
{
    __shared__ double red[256];
    const ile_mdn_tr T = *trp;
    double v[15];
    for (int q = 0; q < 15; q++) v[q] = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)FB * 256) {
        const double wi = fit_weight(ws, lnw[i]);
        if (wi == 0.0) continue;
        double zz[7];
        bool ok = true;
        for (int d = 0; d < D; d++) {
            double ldu;
            const double u = to_unit(T, d, x[d * ld + i], ldu);
            if (!(u > 0.0 && u < 1.0)) ok = false;
            else zz[d] = log(u) - log1p(-u);
        }
        if (!ok) continue;
        v[0] += wi;
        for (int d = 0; d < D; d++) {
            v[1 + d] += wi * zz[d];
            v[8 + d] += wi * zz[d] * zz[d];
        }
    }
    block_sums256<15>(v, red, ws + 16 + blockIdx.x * 16);
}

__global__ void k_fit_stats_only(const double *ws, double *stats)
{
    if (threadIdx.x != 0) return;
    stats[0] = ws[S_MAX];
    stats[1] = ws[S_BETA];
}

__global__ __launch_bounds__(256) void k_fit_mom_fin(double *ws, ile_mdn_tr *tr, double *stats)
{
    __shared__ double sp[15][FB + 1], v[15];
    fetch_parts<15>(ws, sp);
    if (threadIdx.x < 15) v[threadIdx.x] = sum_parts(sp[threadIdx.x]);
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int d = 0; d < D; d++) {
        const double m = v[0] > 0 ? v[1 + d] / v[0] : 0.0;
        const double var = v[0] > 0 ? v[8 + d] / v[0] - m * m : 1.0;
        tr->mean[d] = m;
        tr->scale[d] = fmax(sqrt(fmax(var, 0.0)), 1e-3);
    }
    stats[0] = ws[S_MAX];
    stats[1] = ws[S_BETA];
}

// z~ (FP32, [7][n]) and training weights: tempered exp(beta (ln w - max))
// when lnw is given, else w_in (or 1); 0 where the transform is undefined.
__global__ __launch_bounds__(256) void k_mdn_prepare(const ile_mdn_tr *__restrict__ trp,
                                                     const double *__restrict__ x, int64_t ld,
                                                     const double *__restrict__ lnw,
                                                     const double *__restrict__ w_in, int64_t n,
                                                     const double *__restrict__ stats, float *z,
                                                     double *w)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const ile_mdn_tr T = *trp;
    double xi[7];
    for (int d = 0; d < D; d++) xi[d] = x[d * ld + i];
    float zz[7];
    const double lj = to_z(T, xi, zz);
    for (int d = 0; d < D; d++) z[d * n + i] = zz[d];
    double wi = w_in ? w_in[i] : 1.0;
    if (lnw) wi = isfinite(lnw[i]) ? exp(stats[1] * (lnw[i] - stats[0])) : 0.0;
    w[i] = lj == -INFINITY ? 0.0 : wi;
}

// inclusive prefix sums: CB blocks of 256 threads, each thread a contiguous
// chunk; chunk totals are scanned in order by one thread, then each chunk
// is written from its offset (fixed order: bit-reproducible)
constexpr int CB = 64;
__global__ __launch_bounds__(256) void k_mdn_cdf_part(const double *__restrict__ w, int64_t n,
                                                      double *tot)
{
    const int64_t T = (int64_t)CB * 256, per = (n + T - 1) / T;
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t lo = t * per < n ? t * per : n, hi = lo + per < n ? lo + per : n;
    double s = 0.0;
    for (int64_t i = lo; i < hi; i++) s += w[i];
    tot[t] = s;
}

// exclusive scan of the CB * 256 chunk totals: each of 256 threads scans 64
// consecutive totals, thread 0 scans the 256 thread sums, each thread adds
// its offset (fixed order).  The totals pass through LDS, so that memory is
// read and written in order and the chains run on LDS and registers (21 us as
// a chain of strided loads and stores).
__global__ __launch_bounds__(256) void k_mdn_cdf_scan(double *tot)
{
    constexpr int PER = CB;   // CB * 256 totals over 256 threads
    __shared__ double st[256][PER + 1], ts[256];
    const int tid = threadIdx.x;
#pragma unroll 16
    for (int e = tid; e < 256 * PER; e += 256) st[e / PER][e % PER] = tot[e];
    __syncthreads();
    double run = 0.0, ex[PER];
#pragma unroll
    for (int i = 0; i < PER; i++) {
        ex[i] = run;
        run += st[tid][i];
    }
    ts[tid] = run;
    __syncthreads();
    if (tid == 0) {
        double acc = 0.0;
        for (int t0 = 0; t0 < 256; t0 += 32) {
            double v[32];
#pragma unroll
            for (int i = 0; i < 32; i++) v[i] = ts[t0 + i];
#pragma unroll
            for (int i = 0; i < 32; i++) {
                ts[t0 + i] = acc;
                acc += v[i];
            }
        }
    }
    __syncthreads();
    const double off = ts[tid];
#pragma unroll
    for (int i = 0; i < PER; i++) st[tid][i] = ex[i] + off;
    __syncthreads();
#pragma unroll 16
    for (int e = tid; e < 256 * PER; e += 256) tot[e] = st[e / PER][e % PER];
}

__global__ __launch_bounds__(256) void k_mdn_cdf_write(const double *__restrict__ w, int64_t n,
                                                       const double *__restrict__ tot, double *cdf)
{
    const int64_t T = (int64_t)CB * 256, per = (n + T - 1) / T;
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t lo = t * per < n ? t * per : n, hi = lo + per < n ? lo + per : n;
    double run = tot[t];
    for (int64_t i = lo; i < hi; i++) {
        run += w[i];
        cdf[i] = run;
    }
}

// draw b of a training call: training index drawn with probability
// w_i / sum w (independent draws; step t of the call uses draws
// t*batch .. t*batch + batch - 1)
__global__ __launch_bounds__(256) void k_mdn_draw_idx(uint64_t seed, int64_t count,
                                                      const double *__restrict__ cdf, int64_t n,
                                                      int32_t *idx)
{
    const int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (b >= count) return;
    uint32_t q[4];
    ile_rng::block(seed, (uint64_t)b, 0u, ile_rng::kTagTrain, q);
    const double target = ile_rng::u53(q[0], q[1]) * cdf[n - 1];
    int64_t lo = 0, hi = n - 1;   // first i with cdf[i] > target
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (cdf[mid] > target)
            hi = mid;
        else
            lo = mid + 1;
    }
    idx[b] = (int32_t)lo;
}

}  // namespace

// ---------------------------------------------------------------- launchers
hipError_t ile_launch_mdn_cast(const ile_mdn_dev &M, hipStream_t st)
{
    hipLaunchKernelGGL(k_mdn_cast, dim3((NPARAM + 255) / 256), dim3(256), 0, st, M);
    return hipGetLastError();
}

hipError_t ile_launch_mdn_logpdf(const ile_mdn_dev &M, const ile_mdn_mix &mix, const double *x,
                                 int64_t ld, int64_t n, double *ln_q, int grid, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    if (mix.nb > MAXB) return hipErrorInvalidValue;
    const int64_t tiles = (n + 15) / 16;
    grid = (int)std::min<int64_t>(tiles, std::max(grid, 1));
    hipLaunchKernelGGL(k_mdn_infer<false>, dim3(grid), dim3(IT), 0, st, M.theta, M.W2b, M.W3b,
                       M.tr, mix, (uint64_t)0, (int64_t)0, n, const_cast<double *>(x), ld,
                       (double *)nullptr, ln_q);
    return hipGetLastError();
}

hipError_t ile_launch_mdn_sample(const ile_mdn_dev &M, const ile_mdn_mix &mix, uint64_t seed,
                                 int64_t first, int64_t n, double *x, int64_t ld, double *ln_p,
                                 double *ln_q, int grid, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    if (mix.nb > MAXB) return hipErrorInvalidValue;
    const int64_t tiles = (n + 15) / 16;
    grid = (int)std::min<int64_t>(tiles, std::max(grid, 1));
    hipLaunchKernelGGL(k_mdn_infer<true>, dim3(grid), dim3(IT), 0, st, M.theta, M.W2b, M.W3b,
                       M.tr, mix, seed, first, n, x, ld, ln_p, ln_q);
    return hipGetLastError();
}

hipError_t ile_launch_mdn_fit(const double *x, int64_t ld, const double *lnw, int64_t n,
                              double ess_frac, ile_mdn_tr *tr, double *stats, double *ws,
                              bool fit_transform, hipStream_t st)
{
    if (n <= 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_fit_max, dim3(FB), dim3(256), 0, st, lnw, n, ws);
    hipLaunchKernelGGL(k_fit_init, dim3(1), dim3(256), 0, st, ws, ess_frac);
    for (int it = 0; it <= 30; it++) {
        hipLaunchKernelGGL(k_fit_ess_part, dim3(FB), dim3(256), 0, st, lnw, n, ws);
        hipLaunchKernelGGL(k_fit_ess_step, dim3(1), dim3(256), 0, st, ws, it);
    }
    if (fit_transform) {
        hipLaunchKernelGGL(k_fit_circ_part, dim3(FB), dim3(256), 0, st, x, ld, lnw, n, ws);
        hipLaunchKernelGGL(k_fit_circ_fin, dim3(1), dim3(256), 0, st, ws, tr);
        hipLaunchKernelGGL(k_fit_mom_part, dim3(FB), dim3(256), 0, st, x, ld, lnw, n,
                           (const ile_mdn_tr *)tr, ws);
        hipLaunchKernelGGL(k_fit_mom_fin, dim3(1), dim3(256), 0, st, ws, tr, stats);
    } else {
        hipLaunchKernelGGL(k_fit_stats_only, dim3(1), dim3(64), 0, st, ws, stats);
    }
    return hipGetLastError();
}

size_t ile_mdn_fit_ws_doubles() { return std::max<size_t>(16 + (size_t)FB * 16, (size_t)CB * 256); }

hipError_t ile_launch_mdn_prepare(const ile_mdn_tr *tr, const double *x, int64_t ld,
                                  const double *lnw, int64_t n, const double *stats, float *z,
                                  double *w, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mdn_prepare, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, tr,
                       x, ld, lnw, (const double *)nullptr, n, stats, z, w);
    return hipGetLastError();
}

hipError_t ile_launch_mdn_prepare_w(const ile_mdn_tr *tr, const double *x, int64_t ld,
                                    const double *w_in, int64_t n, float *z, double *w,
                                    hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mdn_prepare, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, tr,
                       x, ld, (const double *)nullptr, w_in, n, (const double *)nullptr, z, w);
    return hipGetLastError();
}

hipError_t ile_launch_mdn_cdf(const double *w, int64_t n, double *cdf, double *ws,
                              hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mdn_cdf_part, dim3(CB), dim3(256), 0, st, w, n, ws);
    hipLaunchKernelGGL(k_mdn_cdf_scan, dim3(1), dim3(256), 0, st, ws);
    hipLaunchKernelGGL(k_mdn_cdf_write, dim3(CB), dim3(256), 0, st, w, n, (const double *)ws, cdf);
    return hipGetLastError();
}

hipError_t ile_launch_mdn_draw_idx(uint64_t seed, int64_t count, const double *cdf, int64_t n,
                                   int32_t *idx, hipStream_t st)
{
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mdn_draw_idx, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st,
                       seed, count, cdf, n, idx);
    return hipGetLastError();
}

hipError_t ile_launch_mdn_grad(const ile_mdn_dev &M, const float *z, int64_t ldz,
                               const int32_t *idx, const double *w, int batch, float *part,
                               hipStream_t st)
{
    if (batch <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mdn_grad, dim3((batch + 63) / 64), dim3(GT), 0, st, M.theta, M.W2b,
                       M.W3b, M.W2t, M.W3t, M.tr, z, ldz, idx, w, batch, part);
    return hipGetLastError();
}

hipError_t ile_launch_mdn_update(const ile_mdn_dev &M, const float *part, int n_part,
                                 float *grad, double *loss, bool adam, int64_t step, double lr,
                                 hipStream_t st)
{
    const double s = (double)std::max<int64_t>(step, 1);
    const float bc1 = (float)(1.0 - pow(0.9, s)), bc2 = (float)(1.0 - pow(0.999, s));
    if (grad) {   // the masked entries
        hipError_t e = ile_launch_fill_u32((uint32_t *)grad, 0u, NPARAM, st);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_mdn_update, dim3((P_LOSS + UPD_P - 1) / UPD_P), dim3(256), 0, st, M, part,
                       n_part, grad, loss, adam ? 1 : 0, bc1, bc2, (float)lr);
    return hipGetLastError();
}

namespace {
__global__ __launch_bounds__(256) void k_lnw(const double *__restrict__ lnL,
                                             const double *__restrict__ lp,
                                             const double *__restrict__ lq, int64_t n,
                                             double *lnw)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) lnw[i] = lnL[i] + (lp ? lp[i] : 0.0) - (lq ? lq[i] : 0.0);
}
}  // namespace

hipError_t ile_launch_lnw(const double *lnL, const double *ln_p, const double *ln_q, int64_t n,
                          double *lnw, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_lnw, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, lnL, ln_p,
                       ln_q, n, lnw);
    return hipGetLastError();
}
