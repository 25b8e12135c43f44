// Rate equations of one point (device functions shared by the local and the band
// statistical-equilibrium solves).
#pragma once

#include "device_math.h"
#include "nlte_internal.h"

namespace nlte {

// Rate matrix of one point (Eq. ourALI): u->l = A(1 - L) + B_ul Jeff + C_ul,
// l->u = B_lu Jeff + C_lu, column-sum form M[to][from]; row 0 := conservation
// sum_i n_i = ntot (rhs).  Entry i of the matrix is M[i * STRIDE]: STRIDE 1 in private memory,
// the wave's width where the lanes' matrices lie side by side in LDS.  rhs [n] is nullable
// (zero but for its first entry, ntot).
template <int STRIDE = 1>
__device__ __forceinline__ void rate_matrix(const SpeciesDev &sp, double T, double nh2, double ntot,
                                            const double *Jrow, const double *Lrow, bool with_L, double *M,
                                            double *rhs)
{
    const int n = sp.n_lev;
    for (int i = 0; i < n * n; ++i) M[i * STRIDE] = 0.0;
    if (rhs != nullptr) {
        for (int i = 0; i < n; ++i) rhs[i] = 0.0;
        rhs[0] = ntot;
    }
    // transitions u -> lo with rate Rd and lo -> u with rate Ru: gains and losses (the four
    // entries are read together, one memory latency per pair of levels)
    auto add = [&](int u, int lo, double Rd, double Ru) {
        double *gu = M + (lo * n + u) * STRIDE, *du = M + (u * n + u) * STRIDE, *gl = M + (u * n + lo) * STRIDE,
               *dl = M + (lo * n + lo) * STRIDE;
        const double a = *gu, b = *du, c = *gl, d = *dl;
        *gu = a + Rd;
        *du = b - Rd;
        *gl = c + Ru;
        *dl = d - Ru;
    };
    for (int l = 0; l < sp.n_lines; ++l) {
        const double Lv = with_L ? Lrow[l] : 0.0;
        add(sp.lu[l], sp.ll[l], sp.A[l] * (1.0 - Lv) + sp.Bul[l] * Jrow[l], sp.Blu[l] * Jrow[l]);
    }
    // H2 de-excitation coefficients, linear in T between table points and clamped at the ends:
    // K[j0] + f (K[j1] - K[j0]), with j0 the last table point at or below T.  What does not depend
    // on the pair is formed once (the division of the interpolation and 1/kT; energy
    // differences and weight ratios come with the species): with three divisions per pair, 200,003
    // points of ten levels took 156 us, now 95: at three waves per CU their latency shows.
    int j0 = 0, j1 = 0;
    double f = 0.0;
    if (T >= sp.Ttab[sp.n_T - 1]) {
        j0 = j1 = sp.n_T - 1;
    } else if (T > sp.Ttab[0]) {
        for (int step = 128; step > 0; step >>= 1)
            if (j0 + step <= sp.n_T - 2 && !(T < sp.Ttab[j0 + step])) j0 += step;
        j1 = j0 + 1;
        f = (T - sp.Ttab[j0]) / (sp.Ttab[j1] - sp.Ttab[j0]);
    }
    const double kT = kKB * T, ikT = fmin(1.0 / kT, 1.7e308);
#pragma unroll 2
    for (int ic = 0; ic < sp.n_coll; ++ic) {
        const double *K = sp.Ktab + (int64_t)ic * sp.n_T;
        const double K0 = K[j0], Cul = fma(f, K[j1] - K0, K0) * nh2;
        // detailed balance with the Boltzmann sign.  The exponent is the quotient -dE / kT to its
        // last bit (one correction of the product with 1/kT; where 1/kT leaves the FP64 range it is
        // held at the largest number, so that equal energies give 1) and the exponential the
        // library's: a polynomial of degree 11 in its place saved 5 us more and left the
        // populations 1.5 times further from their 64-bit values.
        const double x = -sp.cdE[ic], y = x * ikT;
        const double Clu = Cul * sp.cg[ic] * exp(fma(fma(-y, kT, x), ikT, y));
        add(sp.cu[ic], sp.cl[ic], Cul, Clu);
    }
    for (int c = 0; c < n; ++c) M[c * STRIDE] = 1.0;
}

// The change statistics of a block of one wave and point p of each lane: its totals (a fixed
// tree over the lanes) into partials[blockIdx.x], and the per-model maximum (non-negative
// doubles order like their bit patterns) once per block, or per point where the block
// straddles a model boundary.
__device__ __forceinline__ void report_change(double mx, double sum, int64_t cnt, int64_t fb, int64_t kept, int64_t p,
                                              int64_t P, const int32_t *model_of, unsigned long long *model_change,
                                              ConvPartial *partials)
{
    const bool one_model = block_in_one_model(model_of, P) != 0;
    if (model_change != nullptr && !one_model && cnt > 0)
        atomicMax(&model_change[model_of[p]], (unsigned long long)__double_as_longlong(mx));
    for (int o = kWave / 2; o > 0; o >>= 1) {
        mx = fmax(mx, __shfl_down(mx, o));
        sum += __shfl_down(sum, o);
        cnt += __shfl_down(cnt, o);
        fb += __shfl_down(fb, o);
        kept += __shfl_down(kept, o);
    }
    if (threadIdx.x != 0) return;
    if (model_change != nullptr && one_model && cnt > 0)
        atomicMax(&model_change[model_of[p]], (unsigned long long)__double_as_longlong(mx));
    if (partials) {
        ConvPartial cp;
        cp.max_change = mx;
        cp.sum_change = sum;
        cp.count = cnt;
        cp.n_fallback = fb;
        cp.n_kept = kept;
        partials[blockIdx.x] = cp;
    }
}

}  // namespace nlte
