// Surrogate (linear-basis) form (Sec. V): h_lm(lambda; t) = sum_b
// c_lm,b(lambda) e_b(t) with c_lm,b(lambda) = sum_p A[lm][b][p] lambda^p.
// Eq. (7) over the basis needs, per joint sample, the vector
//   z_b = sum_lm c_lm,b(lambda) -2Y_lm(iota, phi)
// in place of the harmonics; k_rom_z forms it (one lane per sample, the
// harmonics in LDS) and the contraction reads it through ile_geom::ext_y.
#include "ile_internal.h"

#include <math.h>
#include <string.h>

namespace {

// Sixteen products of a group of eight complex coefficients (lane l holds value
// l % 16 of its 16, the same in every row of lanes) with u: z_b += A_b u for its
// eight b.  The coefficients reach the lanes as the multiply-adds' broadcast
// operand (DPP row_newbcast); the wait before the first is what a DPP operand
// needs after a vector write of its register.
#define ROM_F(acc, sgn, n, y)                                                                 \
    "v_fmac_f64_dpp %" acc ", " sgn "%16, %" y " row_newbcast:" n " row_mask:0xf bank_mask:0xf\n\t"
#define ROM_R(a0, a1, n, y0, y1, s) ROM_F(a0, s, n, y0) ROM_F(a1, "", n, y1)
__device__ __forceinline__ void rom_mac(double e, double2 u, double2 (&z)[8])
{
#ifdef __HIP_DEVICE_COMPILE__
    asm("s_nop 4\n\t"
        ROM_R("0", "1", "0", "17", "18", "") ROM_R("2", "3", "2", "17", "18", "")
        ROM_R("4", "5", "4", "17", "18", "") ROM_R("6", "7", "6", "17", "18", "")
        ROM_R("8", "9", "8", "17", "18", "") ROM_R("10", "11", "10", "17", "18", "")
        ROM_R("12", "13", "12", "17", "18", "") ROM_R("14", "15", "14", "17", "18", "")
        ROM_R("0", "1", "1", "18", "17", "-") ROM_R("2", "3", "3", "18", "17", "-")
        ROM_R("4", "5", "5", "18", "17", "-") ROM_R("6", "7", "7", "18", "17", "-")
        ROM_R("8", "9", "9", "18", "17", "-") ROM_R("10", "11", "11", "18", "17", "-")
        ROM_R("12", "13", "13", "18", "17", "-") ROM_R("14", "15", "15", "18", "17", "-")
        : "+&v"(z[0].x), "+&v"(z[0].y), "+&v"(z[1].x), "+&v"(z[1].y), "+&v"(z[2].x), "+&v"(z[2].y),
          "+&v"(z[3].x), "+&v"(z[3].y), "+&v"(z[4].x), "+&v"(z[4].y), "+&v"(z[5].x), "+&v"(z[5].y),
          "+&v"(z[6].x), "+&v"(z[6].y), "+&v"(z[7].x), "+&v"(z[7].y)
        : "v"(e), "v"(u.x), "v"(u.y));
#endif
}
#undef ROM_R
#undef ROM_F

// One lane a sample, NG groups of eight basis elements: the modes' harmonics
// into an LDS row (no lane reads another's: no barrier), then z in registers,
// lambda^p Y_a times the coefficients of (a, p), which are one 8-byte load a
// lane and group, issued a step ahead.  1e5 samples, 21 modes, 21 elements, 4
// powers: 64 us (its multiply-adds alone 21 at the vector rate); 152 with
// Horner sums over coefficients read from LDS by every lane, and a sine and
// cosine a mode.
template <int NG>
__global__ __launch_bounds__(64) void k_rom_z(const ile_geom gp, const double *__restrict__ smp,
                                              int64_t N, const double *__restrict__ A, int n_b,
                                              int n_pow, double2 *__restrict__ Z, int32_t *err)
{
    extern __shared__ double2 rom_y[];   // [n_lm][64]
    const int lane = threadIdx.x, nl = gp.n_lm;
    const int64_t r = (int64_t)blockIdx.x * 64 + lane, i = r < N ? r : N - 1;
    const double lam = smp[7 * N + i], ci = smp[4 * N + i], phi = smp[3 * N + i];
    const bool ok = lam >= -1.0 && lam <= 1.0 && ci >= -1.0 && ci <= 1.0 && isfinite(phi);
    double2 *Y = rom_y + lane;
    {
        double cp[kPw], sp[kPw], er[kPw], ei[kPw];
        ylm_tables(ok ? ci : 0.0, ok ? phi : 0.0, cp, sp, er, ei);
        for (int a = 0; a < nl; a++) Y[a * 64] = ylm_entry(gp, a, cp, sp, er, ei);
    }
    const double *p = A + (lane & 15);
    double e[NG], f[NG];
#pragma unroll
    for (int g = 0; g < NG; g++) e[g] = p[16 * g];
    double2 z[NG][8] = {};
    for (int a = 0; a < nl; a++) {
        double2 u = Y[a * 64];
        for (int q = 0; q < n_pow; q++) {
            p += 16 * NG;
#pragma unroll
            for (int g = 0; g < NG; g++) f[g] = p[16 * g];
#pragma unroll
            for (int g = 0; g < NG; g++) rom_mac(e[g], u, z[g]);
            u.x *= lam;
            u.y *= lam;
#pragma unroll
            for (int g = 0; g < NG; g++) e[g] = f[g];
        }
    }
    if (r >= N) return;
    if (!ok) atomicOr(err, 1);
#pragma unroll
    for (int g = 0; g < NG; g++)
#pragma unroll
        for (int b = 0; b < 8; b++)
            if (8 * g + b < n_b)
                Z[i * n_b + 8 * g + b] = ok ? z[g][b] : make_double2(NAN, NAN);
}

int rom_groups(int n_b) { return (n_b + 7) / 8; }

}  // namespace

size_t ile_pack_rom_doubles(int n_lm, int n_b, int n_pow)
{
    return (size_t)16 * rom_groups(n_b) * (n_lm * n_pow + 1);
}

void ile_pack_rom(int n_lm, int n_b, int n_pow, const double *A, double *out)
{
    memset(out, 0, ile_pack_rom_doubles(n_lm, n_b, n_pow) * sizeof(double));
    const size_t row = (size_t)16 * rom_groups(n_b);
    for (int a = 0; a < n_lm; a++)
        for (int b = 0; b < n_b; b++)
            for (int p = 0; p < n_pow; p++)
                memcpy(out + row * (a * n_pow + p) + 2 * b,
                       A + 2 * (((size_t)a * n_b + b) * n_pow + p), 2 * sizeof(double));
}

hipError_t ile_launch_rom_z(const ile_geom &gp, const double *smp, int64_t N, const double *A,
                            int n_b, int n_pow, double *Z, int32_t *err, hipStream_t st)
{
    if (N <= 0) return hipSuccess;
    if (n_b < 1 || n_b > ILE_MAX_LM || gp.n_lm > ILE_MAX_LM) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((N + 63) / 64));
    const size_t lds = (size_t)64 * gp.n_lm * sizeof(double2);
#define ILE_ROM(NG)                                                                           \
    hipLaunchKernelGGL((k_rom_z<NG>), grid, dim3(64), lds, st, gp, smp, N, A, n_b, n_pow,     \
                       (double2 *)Z, err)
    switch (rom_groups(n_b)) {
    case 1: ILE_ROM(1); break;
    case 2: ILE_ROM(2); break;
    case 3: ILE_ROM(3); break;
    default: ILE_ROM(4); break;
    }
#undef ILE_ROM
    return hipGetLastError();
}
