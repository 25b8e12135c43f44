// Line coefficients and the ray-pair formal solve (the ALI hot loop).
//
// Discretisation (Sec. 3.3, no scattering): on the nodes of a ray pair the second-order
// equation d^2u/dtau^2 = u - S becomes the tridiagonal system
//   -A_i u_{i-1} + (1 + A_i + C_i) u_i - C_i u_{i+1} = S_i,
//   A_i = 2 / (D_-(D_- + D_+)),  C_i = 2 / (D_+(D_- + D_+)),
// with D_-+ the optical-depth steps on either side of node i, and second-order (Auer)
// boundary rows that bring in the incoming intensity at both ends.  The elimination of
// Rybicki & Hummer carries F_i = (1 + A_i F_{i-1}/(1 + F_{i-1})) / C_i.
//
// Both ends are eliminated toward the origin O of the pair, so each ray of the pair is
// one half-sweep from its far end to O.  Writing h_i = (D_- + D_+)/2 and
//   Q_i = F_i / (D_+ (1 + F_i)),   y_i = z_i / D_+
// (z_i the Rybicki-Hummer right-hand side), one elimination step becomes
//   T = h_i + Q_{i-1};  F_i = D_+ T;  E = 1/(1 + F_i);  Q_i = T E;  y_i = (S_i h_i + y_{i-1}) E
// with Q = 1, y = I_boundary, D_- = 0 before the first node, which is exactly the Auer
// boundary row.  No step divides by an optical depth.  The sweep carries Q and y as
// fractions N/D and Y/D (scaled by sqrt 2, which cancels at O), which turns each step
// into three multiply-adds of non-negative numbers with no division (see elim_p).
// At O the two halves combine into
//   u_O = (h_O S_O + y_f + y_b) / (h_O + Q_f + Q_b),   Lambda_OO = h_O / (h_O + Q_f + Q_b),
// and u_O - Lambda_OO S_O = (y_f + y_b) / (h_O + Q_f + Q_b) without cancellation.
//
// Mapping: see formal_solve_kernels.h (one wave per origin point and line block, lanes
// over frequencies and up to five lines per lane sharing the profile, ray segments staged
// in LDS).
#include "nlte_internal.h"

namespace nlte {

// ---------------------------------------------------------------- line coefficients

// Eq. (lines) without the profile, at line centre:
//   k_eta = (h nu/4 pi) n_u A_ul,  k_chi = (h nu/4 pi)(n_l B_lu - n_u B_ul),
// line-centre opacity kappa = k_chi / (sqrt(pi) dnu), dnu = nu v_w / c, S = k_eta / k_chi.
// Non-positive opacity (population inversion) is clamped to kappa = S = 0 and counted.
// One thread per (point, line), a block on whole points.  far (nullable): per point, powers of
// two above the largest kappa and the largest S / I_bdy (at least 1) of its lines, as
// exponents: the formal solve's far-wing test reads these 4 bytes per cell instead of every
// line's coefficients.
template <bool F32>
__global__ __launch_bounds__(256) void k_line_coef(SpeciesDev sp, const CellRec *__restrict__ cell,
                                                   const double *__restrict__ pops, int64_t P,
                                                   void *__restrict__ lc, unsigned long long *__restrict__ maser,
                                                   const double *__restrict__ ibdy, short2 *__restrict__ far)
{
    __shared__ short2 s_far[256];
    const int nl = sp.n_lines, per_block = 256 / nl;
    const int lp = threadIdx.x / nl, l = threadIdx.x - lp * nl;
    const int64_t p = blockIdx.x * (int64_t)per_block + lp;
    const bool on = lp < per_block && p < P;
    if (on) {
        const double *n = pops + p * sp.n_lev;
        double nu_ = sp.nu[l];
        double pre = sp.pre[l];
        double nup = n[sp.lu[l]], nlo = n[sp.ll[l]];
        double keta = pre * nup * sp.A[l];
        double kchi = pre * (nlo * sp.Blu[l] - nup * sp.Bul[l]);
        double kap = 0.0, S = 0.0;
        if (kchi > 0.0) {
            double dnu = nu_ * cell[p].vw / kC;
            kap = kchi / (kSqrtPi * dnu);
            S = keta / kchi;
        } else if (maser) {
            atomicAdd(maser, 1ull);
        }
        if (F32)
            reinterpret_cast<float2 *>(lc)[p * nl + l] = make_float2((float)kap, (float)S);
        else
            reinterpret_cast<double2 *>(lc)[p * nl + l] = make_double2(kap, S);
        if (far) {
            // (without a bound: 32767, above every opacity that far_segment takes for none)
            const double I = ibdy[l];
            const int eI = I > 0.0 ? __builtin_amdgcn_frexp_exp(I) : -1000000;
            const int ek = kap == 0.0 ? -3000 : (isfinite(kap) ? __builtin_amdgcn_frexp_exp(kap) : 32767);
            const int es = S == 0.0 ? 0 : (isfinite(S) ? __builtin_amdgcn_frexp_exp(S) - eI + 1 : 32767);
            s_far[threadIdx.x] = make_short2((short)ek, (short)min(max(es, 0), 32767));
        }
    }
    if (!far) return;
    __syncthreads();
    if (on && l == 0) {
        short2 f = s_far[threadIdx.x];
        for (int i = 1; i < nl; ++i) {
            const short2 v = s_far[threadIdx.x + i];
            f.x = max(f.x, v.x);
            f.y = max(f.y, v.y);
        }
        far[p] = f;
    }
}

hipError_t launch_line_coef(const SpeciesDev &sp, const CellRec *cell, const double *pops, int64_t P, int fp32,
                            void *lc, int64_t *maser_count, const double *ibdy, short2 *far, hipStream_t s)
{
    if (P * sp.n_lines == 0) return hipSuccess;
    const int per_block = 256 / sp.n_lines;
    dim3 grid((unsigned)((P + per_block - 1) / per_block));
    auto *m = reinterpret_cast<unsigned long long *>(maser_count);
    if (fp32)
        hipLaunchKernelGGL(k_line_coef<true>, grid, dim3(256), 0, s, sp, cell, pops, P, lc, m, ibdy, far);
    else
        hipLaunchKernelGGL(k_line_coef<false>, grid, dim3(256), 0, s, sp, cell, pops, P, lc, m, ibdy, far);
    return hipGetLastError();
}

// ---------------------------------------------------------------- formal solve

// The kernels are templates in formal_solve_kernels.h, instantiated per precision in
// fs_fp64.hip and fs_fp32.hip (compiled in parallel).
hipError_t launch_formal_solve(const SolveArgs &a, int fp32, hipStream_t s)
{
    if (a.n_blocks == 0) return hipSuccess;
    return fp32 ? launch_formal_solve_f32(a, s) : launch_formal_solve_f64(a, s);
}

}  // namespace nlte
