// Rate equations of one point (device functions shared by the local and the band
// statistical-equilibrium solves).
#pragma once

#include "nlte_internal.h"

namespace nlte {

// H2 de-excitation coefficient of collision pair ic, linear in T between table points
// and clamped at the ends; j is the table interval holding T (T inside the table).
__device__ __forceinline__ double coll_K(const SpeciesDev &sp, int ic, double T, int j, int where)
{
    const double *K = sp.Ktab + (int64_t)ic * sp.n_T;
    if (where < 0) return K[0];
    if (where > 0) return K[sp.n_T - 1];
    return K[j] + (K[j + 1] - K[j]) * (T - sp.Ttab[j]) / (sp.Ttab[j + 1] - sp.Ttab[j]);
}

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
    // the table interval that holds T: the last j with Ttab[j] <= T
    int where = 0, j = 0;
    if (T <= sp.Ttab[0]) where = -1;
    else if (T >= sp.Ttab[sp.n_T - 1]) where = 1;
    else
        for (int step = 128; step > 0; step >>= 1)
            if (j + step <= sp.n_T - 2 && !(T < sp.Ttab[j + step])) j += step;
    const double kT = kKB * T;
#pragma unroll 2
    for (int ic = 0; ic < sp.n_coll; ++ic) {
        const int u = sp.cu[ic], lo = sp.cl[ic];
        const double Cul = coll_K(sp, ic, T, j, where) * nh2;
        // detailed balance with the Boltzmann sign
        const double Clu = Cul * (sp.g[u] / sp.g[lo]) * exp(-(sp.E[u] - sp.E[lo]) / kT);
        add(u, lo, Cul, Clu);
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
