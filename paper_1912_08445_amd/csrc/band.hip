// Statistical equilibrium with the band ALO (Sec. 3.4): the rate equations of every point
// contain, besides its own populations, the new upper-level populations of the first
// cells of its walks (the cells the band of one node reaches).  For line (u -> lo) at
// point O the net downward rate is
//   n_u,O [A (1 - Ld) + B_ul Jb] - n_lo,O B_lu Jb - sum_r cpl_r n_u,c(r),
//   cpl_r = A (k_O / k_c) Ln_r,  k = h nu/4pi (n_lo B_lu - n_u B_ul) with the previous populations,
// so the system of all points is A = K + C with K the block diagonal of the points' own
// rate matrices and C the couplings.  It is solved by BiCGSTAB (van der Vorst 1992) on the
// block-Jacobi preconditioned system (I + K^-1 C) x = K^-1 b, starting from the uncoupled
// solution K^-1 b, with inner products weighted by 1 / n_tot^2 (fractional populations).
// Points of converged models are held fixed.  A model with a singular local matrix, or
// whose coupled solution has a population that is not positive and finite, takes the
// local (diagonal ALO) solve instead (Sec. 6.1); its couplings are left out of the
// coupled system, which is block diagonal over models.
//
// The solver runs on the device: three kernels per step, each of which sums the per-block
// partials of the inner products before it (every block the same numbers in the same order)
// and takes the step's scalars from them.  What ends the solve is written to BandState; kernels
// enqueued past that point return at once, so the host enqueues several steps and looks once.
// Updates of a vector whose product with the system follows are not a pass of their own: the
// product forms its operand from the old vectors where it reads it.
// Launches and their latency bound it for few points: with a synchronisation for each set of
// inner products and vector updates as kernels of their own, an iteration of the band ALO for a
// sphere of 3,001 points (4 steps) took 590 us, now 215, of which the formal solve takes 85 (132
// before its pairs were split over waves).  The solver's kernels keep 0.15 waves on a SIMD and
// read 0.3 TB/s: a chain of waits (the scalars' partial sums, then the couplings, then the factors).
#include <algorithm>

#include "rates.h"

namespace nlte {

namespace {

constexpr int kBandGroup = 4;          // lanes that share a point's rays
constexpr int kBandBlocks = 1024;      // most blocks of a solver kernel
constexpr int kBandSteps = 200;
constexpr double kBandTol = 1e-13;

// In-place LU factorisation with partial pivoting, rows swapped whole; entry i of the matrix is
// M[i * STRIDE], perm 4 bits per column (the row it was swapped with).  False: singular.
template <int STRIDE>
__device__ inline bool lu_factor(int n, double *M, unsigned long long &perm)
{
    perm = 0;
    for (int col = 0; col < n; ++col) {
        int p = col;
        for (int r = col + 1; r < n; ++r)
            if (fabs(M[(r * n + col) * STRIDE]) > fabs(M[(p * n + col) * STRIDE])) p = r;
        perm |= (unsigned long long)p << (4 * col);
        if (!(M[(p * n + col) * STRIDE] != 0.0)) return false;
        if (p != col)
            for (int c = 0; c < n; ++c) {
                const double t = M[(col * n + c) * STRIDE];
                M[(col * n + c) * STRIDE] = M[(p * n + c) * STRIDE];
                M[(p * n + c) * STRIDE] = t;
            }
        for (int r = col + 1; r < n; ++r) {
            const double f = M[(r * n + col) * STRIDE] / M[(col * n + col) * STRIDE];
            M[(r * n + col) * STRIDE] = f;
            for (int c = col + 1; c < n; ++c) M[(r * n + c) * STRIDE] -= f * M[(col * n + c) * STRIDE];
        }
    }
    return true;
}

// The columns' rows of a factorisation without swaps, 4 bits each.
__device__ inline unsigned long long identity_perm(int n)
{
    return 0xFEDCBA9876543210ull & (n < 16 ? (1ull << (4 * n)) - 1 : ~0ull);
}

// b := A^-1 b from the factors (the rows are swapped first: the factors' rows were swapped whole).
__device__ __forceinline__ void lu_solve_any(int n, const double *__restrict__ LU, unsigned long long perm, double *b)
{
    for (int col = 0; col < n; ++col) {
        const int p = (int)(perm >> (4 * col)) & 15;
        const double t = b[col];
        b[col] = b[p];
        b[p] = t;
    }
    for (int r = 1; r < n; ++r)
        for (int c = 0; c < r; ++c) b[r] -= LU[r * n + c] * b[c];
    for (int r = n - 1; r >= 0; --r) {
        for (int c = r + 1; c < n; ++c) b[r] -= LU[r * n + c] * b[c];
        b[r] /= LU[r * n + r];
    }
}

// The same with b in registers.
template <int N>
__device__ __forceinline__ void lu_solve(const double *__restrict__ LU, unsigned long long perm, double (&b)[N])
{
    if (perm != identity_perm(N)) {
#pragma unroll
        for (int col = 0; col < N - 1; ++col) {
            const int p = (int)(perm >> (4 * col)) & 15;
            const double was = b[col];
            double now = was;
#pragma unroll
            for (int r = col + 1; r < N; ++r) {
                now = p == r ? b[r] : now;
                b[r] = p == r ? was : b[r];
            }
            b[col] = now;
        }
    }
#pragma unroll
    for (int r = 1; r < N; ++r)
#pragma unroll
        for (int c = 0; c < r; ++c) b[r] -= LU[r * N + c] * b[c];
#pragma unroll
    for (int r = N - 1; r >= 0; --r) {
#pragma unroll
        for (int c = r + 1; c < N; ++c) b[r] -= LU[r * N + c] * b[c];
        b[r] /= LU[r * N + r];
    }
}

// Sums over the blocks' partials, the same in every lane of every block.
template <int K>
__device__ __forceinline__ void sum_partials(const double *__restrict__ part, int nb, double (&out)[K])
{
#pragma unroll
    for (int k = 0; k < K; ++k) out[k] = 0.0;
    for (int i = threadIdx.x & (kWave - 1); i < nb; i += kWave)
#pragma unroll
        for (int k = 0; k < K; ++k) out[k] += part[i * K + k];
    for (int o = 1; o < kWave; o <<= 1)
#pragma unroll
        for (int k = 0; k < K; ++k) out[k] += __shfl_xor(out[k], o);
}

// A block's sums of acc into its row of part.
template <int K>
__device__ __forceinline__ void block_partials(double (&acc)[K], double *__restrict__ part)
{
    __shared__ double red[4][K];
    for (int o = kWave / 2; o > 0; o >>= 1)
#pragma unroll
        for (int k = 0; k < K; ++k) acc[k] += __shfl_down(acc[k], o);
    const int wave = threadIdx.x / kWave, waves = blockDim.x / kWave;
    if (threadIdx.x % kWave == 0)
#pragma unroll
        for (int k = 0; k < K; ++k) red[wave][k] = acc[k];
    __syncthreads();
    if (threadIdx.x < K) {
        double s = red[0][threadIdx.x];
        for (int w = 1; w < waves; ++w) s += red[w][threadIdx.x];
        part[blockIdx.x * K + threadIdx.x] = s;
    }
}

// K^-1 C y at point p for the group's lanes, each of which takes every fourth ray; y(i) is
// element i of the operand.  All lanes of the group get the result.
template <int N, class Y>
__device__ __forceinline__ void coupling(const BandArgs &b, const SpeciesDev &sp, int64_t p, int g, Y &&y,
                                         double (&cv)[N > 0 ? N : kMaxLev])
{
    const int n = N > 0 ? N : sp.n_lev, nl = sp.n_lines, R = b.R;
#pragma unroll
    for (int i = 0; i < n; ++i) cv[i] = 0.0;
    for (int l = 0; l < nl; ++l) {
        const int u = sp.lu[l], lo = sp.ll[l];
        double v = 0.0;
#pragma unroll 4
        for (int r = g; r < R; r += kBandGroup) {
            const double k = b.cpl[(p * nl + l) * R + r];
            const int32_t c = b.first[p * R + r];
            const double yc = y((int64_t)max(c, 0) * n + u);
            v += k != 0.0 ? k * yc : 0.0;
        }
#pragma unroll
        for (int o = 1; o < kBandGroup; o <<= 1) v += __shfl_xor(v, o);
        if constexpr (N > 0) {
#pragma unroll
            for (int i = 1; i < n; ++i) cv[i] += i == u ? v : i == lo ? -v : 0.0;
        } else {
            if (u != 0) cv[u] += v;
            if (lo != 0) cv[lo] -= v;
        }
    }
    if constexpr (N > 0)
        lu_solve<N>(b.LU + p * N * N, b.perm[p], cv);
    else
        lu_solve_any(n, b.LU + p * n * n, b.perm[p], cv);
}

}  // namespace

// First cell of the walk from every point along every ray (-1 for an empty walk).
__global__ void k_first_cells(const int64_t *__restrict__ roff, const int32_t *__restrict__ rcells, int64_t n,
                              int32_t *__restrict__ first)
{
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q >= n) return;
    first[q] = roff[q + 1] > roff[q] ? rcells[roff[q]] : -1;
}

hipError_t launch_first_cells(const int64_t *roff, const int32_t *rcells, int64_t n, int32_t *first, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_first_cells, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, roff, rcells, n, first);
    return hipGetLastError();
}

// Per point: LU factors of its own rate matrix (with the band diagonal Ld and Jb) and the
// uncoupled solution x = K^-1 b.  One point per lane; LDS: the matrices of a wave side by side
// (N^2 * 512 bytes, up to 11 levels), else private memory.
template <bool LDS>
__global__ __launch_bounds__(kWave) void k_band_setup(BandArgs b, SpeciesDev sp, const CellRec *__restrict__ cell,
                                                      const double *__restrict__ nh2, const double *__restrict__ T,
                                                      const double *__restrict__ old)
{
    extern __shared__ double lds[];
    constexpr int S = LDS ? kWave : 1;
    const int64_t p = blockIdx.x * (int64_t)kWave + threadIdx.x;
    if (p >= b.P) return;
    const int n = sp.n_lev, nl = sp.n_lines;
    double priv[LDS ? 1 : kMaxLev * kMaxLev], rhs[kMaxLev];
    double *M = LDS ? lds + threadIdx.x : priv;
    const bool fixed = b.done != nullptr && b.done[b.model_of[p]];
    if (fixed) {
        for (int i = 0; i < n * n; ++i) M[i * S] = i % (n + 1) == 0 ? 1.0 : 0.0;
        for (int i = 0; i < n; ++i) rhs[i] = old[p * n + i];
    } else {
        rate_matrix<S>(sp, T[p], nh2[p], cell[p].ntot, b.Jb + p * nl, b.Ld + p * nl, true, M, rhs);
    }
    unsigned long long perm;
    if (!lu_factor<S>(n, M, perm)) {
        b.model_bad[b.model_of[p]] = 1;
        for (int i = 0; i < n * n; ++i) M[i * S] = i % (n + 1) == 0 ? 1.0 : 0.0;
        perm = identity_perm(n);
        for (int i = 0; i < n; ++i) rhs[i] = old[p * n + i];
    }
    for (int i = 0; i < n * n; ++i) b.LU[p * n * n + i] = M[i * S];
    b.perm[p] = perm;
    lu_solve_any(n, b.LU + p * n * n, perm, rhs);
    for (int i = 0; i < n; ++i) b.x[p * n + i] = rhs[i];
}

// The coupling coefficients to the first cells, one thread per (point, ray).  Couplings of the
// points of models that take the local solve are dropped, so their rows read x = K^-1 b and
// the coupled solve of the other models is unchanged.
__global__ __launch_bounds__(256) void k_band_couple(BandArgs b, SpeciesDev sp, const double *__restrict__ old)
{
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int n = sp.n_lev, nl = sp.n_lines, R = b.R;
    if (q >= b.P * R) return;
    const int64_t p = q / R;
    const int r = (int)(q - p * R), m = b.model_of[p];
    const int32_t c = b.first[q];
    const bool none = (b.done != nullptr && b.done[m]) || b.model_bad[m] || c < 0;
    for (int l = 0; l < nl; ++l) {
        double k = 0.0;
        if (!none) {
            const int u = sp.lu[l], lo = sp.ll[l];
            const double kO = sp.pre[l] * (old[p * n + lo] * sp.Blu[l] - old[p * n + u] * sp.Bul[l]);
            const double kc = sp.pre[l] * (old[(int64_t)c * n + lo] * sp.Blu[l] - old[(int64_t)c * n + u] * sp.Bul[l]);
            if (kO > 0.0 && kc > 0.0) k = sp.A[l] * (kO / kc) * b.Ln[(p * nl + l) * R + r];
        }
        b.cpl[(p * nl + l) * R + r] = k;
    }
}

// A step it = 0, 1, ... of BiCGSTAB is three kernels; with A = I + K^-1 C
//   P  p = r + beta (p - omega v), v = A p                       sum: (r0, v)
//   S  s = r - alpha v, t = A s                                  sums: (s, s), (t, s), (t, t)
//   X  x = x + alpha p + omega s, r = s - omega t                sums: (r0, r), (r, r), (x, x)
// after START (r = r0 = -K^-1 C x for x = K^-1 b, as step -1's X).  Kernel q of the solve
// (counted from 1) returns if the solve ended at one before it.  p and v alternate between
// two buffers, since neighbours read the old ones.  Inner products are weighted by 1 / n_tot^2.
enum { kBandStart, kBandP, kBandS };

template <int N, int KIND>
__global__ __launch_bounds__(256, 2) void k_band_product(BandArgs b, SpeciesDev sp, const CellRec *__restrict__ cell, int it)
{
    const int n = N > 0 ? N : sp.n_lev;
    BandState &st = *b.state;
    const int seq = KIND == kBandStart ? 1 : 3 * it + (KIND == kBandP ? 2 : 3);
    const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
    const int now = it & 1, was = now ^ 1;
    auto end = [&](int status, int iters) {
        if (lead) {
            st.status = status;
            st.iters = iters;
            st.ended = seq;
        }
    };
    if (KIND != kBandStart && st.ended != 0 && st.ended < seq) return;
    double alpha = 0.0, beta = 0.0, omega = 0.0;
    if constexpr (KIND == kBandP) {
        double d[3];   // (r0, r), (r, r), (x, x)
        sum_partials(b.part_x, b.nb, d);
        const bool conv = d[1] <= kBandTol * kBandTol * d[2];
        if (it > 0) {
            omega = st.omega[was];
            if (!(omega != 0.0)) return end(kBandFailed, it);
        }
        if (conv || (it == 0 && !(d[2] > 0.0))) return end(kBandConverged, it);
        if (it == kBandSteps) return end(kBandFailed, it);
        if (!(d[0] != 0.0) || !isfinite(d[0])) return end(kBandFailed, it + 1);
        if (it > 0) beta = (d[0] / st.rho[was]) * (st.alpha[was] / omega);
        if (lead) {
            st.rho[now] = d[0];
            st.xx = d[2];
            st.iters = it + 1;
        }
    }
    if constexpr (KIND == kBandS) {
        double d[1];   // (r0, v)
        sum_partials(b.part_p, b.nb, d);
        if (!(d[0] != 0.0) || !isfinite(d[0])) return end(kBandFailed, it + 1);
        alpha = st.rho[now] / d[0];
        if (lead) st.alpha[now] = alpha;
    }
    const double *x = b.x, *r = b.r, *po = b.p[was], *vo = b.v[was], *vn = b.v[now];
    const double bo = -beta * omega;
    auto y = [&](int64_t i) {
        if constexpr (KIND == kBandStart)
            return x[i];
        else if constexpr (KIND == kBandP)
            return it == 0 ? r[i] : (r[i] + beta * po[i]) + bo * vo[i];
        else
            return r[i] - alpha * vn[i];
    };
    double acc[KIND == kBandP ? 1 : 3] = {};
    const int g = threadIdx.x % kBandGroup, per_block = blockDim.x / kBandGroup;
    for (int64_t p0 = (int64_t)blockIdx.x * per_block; p0 < b.P; p0 += (int64_t)gridDim.x * per_block) {
        const int64_t p = p0 + threadIdx.x / kBandGroup;
        const int64_t q = p < b.P ? p : b.P - 1;   // (whole groups shuffle)
        double cv[N > 0 ? N : kMaxLev];
        coupling<N>(b, sp, q, g, y, cv);
        if (p >= b.P || g != 0) continue;
        const double wgt = 1.0 / (cell[p].ntot * cell[p].ntot);
        double s0 = 0.0, s1 = 0.0, s2 = 0.0;
#pragma unroll
        for (int i = 0; i < n; ++i) {
            const int64_t e = p * n + i;
            if constexpr (KIND == kBandStart) {
                const double r0 = -cv[i], xe = x[e];
                b.r[e] = r0;
                b.r0[e] = r0;
                s0 += r0 * r0;
                s2 += xe * xe;
            } else if constexpr (KIND == kBandP) {
                const double ye = y(e), w = ye + cv[i];
                b.p[now][e] = ye;
                b.v[now][e] = w;
                s0 += b.r0[e] * w;
            } else {
                const double ye = y(e), w = ye + cv[i];
                b.s[e] = ye;
                b.t[e] = w;
                s0 += ye * ye;
                s1 += w * ye;
                s2 += w * w;
            }
        }
        acc[0] += s0 * wgt;
        if constexpr (KIND != kBandP) {
            acc[1] += (KIND == kBandStart ? s0 : s1) * wgt;
            acc[2] += s2 * wgt;
        }
    }
    block_partials(acc, KIND == kBandStart ? b.part_x : KIND == kBandP ? b.part_p : b.part_s);
}

__global__ __launch_bounds__(256) void k_band_update(BandArgs b, const CellRec *__restrict__ cell, int n, int it)
{
    BandState &st = *b.state;
    const int seq = 3 * it + 4, now = it & 1;
    const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
    if (st.ended != 0 && st.ended < seq) return;
    double d[3];   // (s, s), (t, s), (t, t)
    sum_partials(b.part_s, b.nb, d);
    const double alpha = st.alpha[now], omega = d[1] / d[2];
    const bool conv = d[0] <= kBandTol * kBandTol * st.xx, fail = !conv && !(d[2] > 0.0);
    if (lead) {
        st.omega[now] = omega;
        if (conv || fail) {
            st.status = conv ? kBandConverged : kBandFailed;
            st.ended = seq;
        }
    }
    if (fail) return;
    double acc[3] = {};
    const double *pv = b.p[now];
    const int g = threadIdx.x % kBandGroup, per_block = blockDim.x / kBandGroup;
    for (int64_t p = (int64_t)blockIdx.x * per_block + threadIdx.x / kBandGroup; p < b.P;
         p += (int64_t)gridDim.x * per_block) {
        const double wgt = 1.0 / (cell[p].ntot * cell[p].ntot);
        double s0 = 0.0, s1 = 0.0, s2 = 0.0;
        for (int i = g; i < n; i += kBandGroup) {
            const int64_t e = p * n + i;
            if (conv) {
                b.x[e] += alpha * pv[e];
                continue;
            }
            const double s = b.s[e], x = (b.x[e] + alpha * pv[e]) + omega * s, r = s - omega * b.t[e];
            b.x[e] = x;
            b.r[e] = r;
            s0 += b.r0[e] * r;
            s1 += r * r;
            s2 += x * x;
        }
        acc[0] += s0 * wgt;
        acc[1] += s1 * wgt;
        acc[2] += s2 * wgt;
    }
    if (!conv) block_partials(acc, b.part_x);
}

// Models with a population that is not positive and finite.
__global__ void k_band_check_models(const double *__restrict__ x, int n, int64_t P,
                                    const int32_t *__restrict__ model_of, uint8_t *__restrict__ model_bad,
                                    const BandState *__restrict__ state)
{
    if (state->status != kBandConverged) return;
    const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (p >= P) return;
    bool ok = true;
    for (int i = 0; i < n; ++i) ok = ok && x[p * n + i] > 0.0 && isfinite(x[p * n + i]);
    if (!ok) model_bad[model_of[p]] = 1;
}

// New populations: the band's, or the local solve's for models marked in model_bad
// (local and model_bad nullable: every model takes the band's); change statistics and
// per-model changes as the local solve reports them.
__global__ __launch_bounds__(kWave) void k_band_finish(const double *__restrict__ x, const double *__restrict__ local,
                                                     const uint8_t *__restrict__ model_bad,
                                                     const double *__restrict__ old,
                                                     const CellRec *__restrict__ cell, int n, int64_t P,
                                                     double *__restrict__ pops_new, uint8_t *__restrict__ flags,
                                                     ConvPartial *partials, const uint8_t *__restrict__ done,
                                                     const int32_t *__restrict__ model_of,
                                                     unsigned long long *__restrict__ model_change)
{
    const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    double mx = 0.0, sum = 0.0;
    int64_t cnt = 0;
    if (p < P) {
        const bool fixed = done != nullptr && done[model_of[p]];
        const bool loc = model_bad != nullptr && model_bad[model_of[p]];
        const double *src = loc ? local : x;
        const double nt = cell[p].ntot;
        for (int i = 0; i < n; ++i) {
            const double v = fixed ? old[p * n + i] : src[p * n + i];
            pops_new[p * n + i] = v;
            if (!fixed && v / nt > 1e-10) {
                const double d = fabs(v - old[p * n + i]) / v;
                mx = fmax(mx, d);
                sum += d;
                ++cnt;
            }
        }
        if (flags && !loc) flags[p] = 0;   // the local solve has set its own
    }
    report_change(mx, sum, cnt, 0, 0, p, P, model_of, model_change, partials);
}

hipError_t launch_band_setup(const BandArgs &b, const SpeciesDev &sp, const CellRec *cell, const double *nh2,
                             const double *T, const double *old, hipStream_t s)
{
    if (b.P == 0) return hipSuccess;
    const dim3 grid((unsigned)((b.P + kWave - 1) / kWave));
    if (sp.n_lev <= 11)
        hipLaunchKernelGGL(k_band_setup<true>, grid, dim3(kWave), sizeof(double) * sp.n_lev * sp.n_lev * kWave, s, b, sp,
                           cell, nh2, T, old);
    else
        hipLaunchKernelGGL(k_band_setup<false>, grid, dim3(kWave), 0, s, b, sp, cell, nh2, T, old);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_band_couple, dim3((unsigned)((b.P * b.R + 255) / 256)), dim3(256), 0, s, b, sp, old);
    return hipGetLastError();
}

// Blocks of one wave (16 points) while that gives no more than kBandBlocks of them, so that few
// points still spread over the chip; else of four waves, each taking several points.
static int band_threads(int64_t P) { return P <= (int64_t)kBandBlocks * kWave / kBandGroup ? kWave : 256; }

int band_blocks(int64_t P)
{
    const int per_block = band_threads(P) / kBandGroup;
    return (int)std::min<int64_t>((P + per_block - 1) / per_block, kBandBlocks);
}

template <int N>
static hipError_t band_steps(const BandArgs &b, const SpeciesDev &sp, const CellRec *cell, int from, int to, hipStream_t s)
{
    if constexpr (N > 0) {
        if (sp.n_lev != N) return band_steps<N == 2 ? 0 : N - 1>(b, sp, cell, from, to, s);
    }
    const dim3 grid((unsigned)b.nb), block((unsigned)band_threads(b.P));
    if (from == 0) {
        hipLaunchKernelGGL((k_band_product<N, kBandStart>), grid, block, 0, s, b, sp, cell, 0);
        hipLaunchKernelGGL((k_band_product<N, kBandP>), grid, block, 0, s, b, sp, cell, 0);
    }
    // (a step's convergence is seen by the next one's P)
    for (int it = from; it < to && it < kBandSteps; ++it) {
        hipLaunchKernelGGL((k_band_product<N, kBandS>), grid, block, 0, s, b, sp, cell, it);
        hipLaunchKernelGGL(k_band_update, grid, block, 0, s, b, cell, sp.n_lev, it);
        hipLaunchKernelGGL((k_band_product<N, kBandP>), grid, block, 0, s, b, sp, cell, it + 1);
    }
    return hipGetLastError();
}

hipError_t launch_band_steps(const BandArgs &b, const SpeciesDev &sp, const CellRec *cell, int from, int to, hipStream_t s)
{
    if (b.P == 0) return hipSuccess;
    return band_steps<11>(b, sp, cell, from, to, s);
}

hipError_t launch_band_check_models(const double *x, int n, int64_t P, const int32_t *model_of, uint8_t *model_bad,
                                   const BandState *state, hipStream_t s)
{
    if (P == 0) return hipSuccess;
    hipLaunchKernelGGL(k_band_check_models, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, s, x, n, P, model_of,
                       model_bad, state);
    return hipGetLastError();
}

hipError_t launch_band_finish(const double *x, const double *local, const uint8_t *model_bad, const double *old,
                              const CellRec *cell, int n, int64_t P, double *pops_new, uint8_t *flags,
                              ConvPartial *partials, const uint8_t *done, const int32_t *model_of,
                              unsigned long long *model_change, hipStream_t s)
{
    if (P == 0) return hipSuccess;
    hipLaunchKernelGGL(k_band_finish, dim3((unsigned)stateq_blocks(P)), dim3(kWave), 0, s, x, local, model_bad, old,
                       cell, n, P, pops_new, flags, partials, done, model_of, model_change);
    return hipGetLastError();
}

}  // namespace nlte
