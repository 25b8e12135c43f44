// Statistical equilibrium per point and the convergence reduction.
#include "rates.h"

namespace nlte {

// Gaussian elimination with partial pivoting of one point's rate equations, the matrix in
// private memory (any number of levels).
__device__ int solve_point(const SpeciesDev &sp, double T, double nh2, double ntot,
                           const double *Jrow, const double *Lrow, bool with_L, double *x)
{
    const int n = sp.n_lev;
    double M[kMaxLev * kMaxLev];
    double rhs[kMaxLev];
    rate_matrix(sp, T, nh2, ntot, Jrow, Lrow, with_L, M, rhs);
    for (int col = 0; col < n; ++col) {
        int piv = col;
        for (int r = col + 1; r < n; ++r)
            if (fabs(M[r * n + col]) > fabs(M[piv * n + col])) piv = r;
        if (M[piv * n + col] == 0.0) return -1;
        if (piv != col) {
            for (int c = 0; c < n; ++c) {
                double t = M[col * n + c];
                M[col * n + c] = M[piv * n + c];
                M[piv * n + c] = t;
            }
            double t = rhs[col];
            rhs[col] = rhs[piv];
            rhs[piv] = t;
        }
        for (int r = col + 1; r < n; ++r) {
            double f = M[r * n + col] / M[col * n + col];
            for (int c = col; c < n; ++c) M[r * n + c] -= f * M[col * n + c];
            rhs[r] -= f * rhs[col];
        }
    }
    for (int r = n - 1; r >= 0; --r) {
        double s = rhs[r];
        for (int c = r + 1; c < n; ++c) s -= M[r * n + c] * x[c];
        x[r] = s / M[r * n + r];
    }
    return 0;
}

// The same elimination, operation for operation, of N levels in registers: every index is
// known when it is compiled, and rows change places by selects where some lane needs it
// (rarely: the conservation row is the largest of the first column, the diagonal of the
// others).
template <int N>
__device__ __forceinline__ int solve_registers(double (&M)[N][N], double ntot, double *x)
{
    double rhs[N];
#pragma unroll
    for (int r = 0; r < N; ++r) rhs[r] = r == 0 ? ntot : 0.0;
    int bad = 0;
#pragma unroll
    for (int col = 0; col < N; ++col) {
        int piv = col;
        double big = fabs(M[col][col]);
#pragma unroll
        for (int r = col + 1; r < N; ++r) {
            const double v = fabs(M[r][col]);
            if (v > big) {
                big = v;
                piv = r;
            }
        }
        if (__any(piv != col)) {
#pragma unroll
            for (int r = col + 1; r < N; ++r)
                if (piv == r) {
#pragma unroll
                    for (int c = col; c < N; ++c) {
                        const double t = M[col][c];
                        M[col][c] = M[r][c];
                        M[r][c] = t;
                    }
                    const double t = rhs[col];
                    rhs[col] = rhs[r];
                    rhs[r] = t;
                }
        }
        if (M[col][col] == 0.0) bad = -1;   // (the values computed from here on are not used)
#pragma unroll
        for (int r = col + 1; r < N; ++r) {
            const double f = M[r][col] / M[col][col];
#pragma unroll
            for (int c = col + 1; c < N; ++c) M[r][c] -= f * M[col][c];
            rhs[r] -= f * rhs[col];
        }
    }
#pragma unroll
    for (int r = N - 1; r >= 0; --r) {
        double s = rhs[r];
#pragma unroll
        for (int c = r + 1; c < N; ++c) s -= M[r][c] * x[c];
        x[r] = s / M[r][r];
    }
    return bad;
}

// One point's rate equations.  N > 0: the wave's matrices are assembled side by side in LDS
// (the levels of a transition are data, so the entries cannot be addressed in registers)
// and solved from registers.  N = 0: any number of levels, in private memory.
template <int N>
__device__ __forceinline__ int solve_rates(const SpeciesDev &sp, double T, double nh2, double ntot,
                                           const double *Jrow, const double *Lrow, bool with_L, double *lds, double *x)
{
    if constexpr (N == 0) {
        return solve_point(sp, T, nh2, ntot, Jrow, Lrow, with_L, x);
    } else {
        double *own = lds + threadIdx.x;
        rate_matrix<kWave>(sp, T, nh2, ntot, Jrow, Lrow, with_L, own, nullptr);
        double M[N][N];
#pragma unroll
        for (int r = 0; r < N; ++r)
#pragma unroll
            for (int c = 0; c < N; ++c) M[r][c] = own[(r * N + c) * kWave];
        return solve_registers<N>(M, ntot, x);
    }
}

__device__ __forceinline__ bool valid(int n, const double *x)
{
    for (int i = 0; i < n; ++i)
        if (!(x[i] > 0.0) || !isfinite(x[i])) return false;
    return true;
}

// Statistical equilibrium of every point and the change of its populations.  One wave per 64
// points, one point per lane.  The matrices are what bounds it: in private memory (256
// doubles a lane, whatever the number of levels) their traffic to scratch took 0.55 ms for
// 200,003 points of ten levels, two orders over the bytes of the call; N levels in registers,
// assembled in N^2 * 512 bytes of LDS, take 0.15 ms (one pass of the call 586 -> 157 us; 95 with the
// shorter collision rates of rate_matrix), most of it the assembly: three waves fit a CU and
// every transition updates four entries.  N stops at 11, whose
// matrices fill 62 of the 64 KB a launch may ask for as it is; more levels stay with N = 0.
template <int N>
__global__ __launch_bounds__(kWave) void k_stateq(SpeciesDev sp, const CellRec *__restrict__ cell,
                                                  const double *__restrict__ nh2, const double *__restrict__ Tg,
                                                  int64_t P, int use_alo, const double *__restrict__ pops_old,
                                                  const double *__restrict__ J, const double *__restrict__ Jeff,
                                                  const double *__restrict__ L, double *__restrict__ pops_new,
                                                  uint8_t *__restrict__ flags, ConvPartial *partials,
                                                  const uint8_t *__restrict__ model_done,
                                                  const int32_t *__restrict__ model_of,
                                                  unsigned long long *__restrict__ model_change)
{
    extern __shared__ double lds[];
    const int64_t p = blockIdx.x * (int64_t)kWave + threadIdx.x;
    const int n = N > 0 ? N : sp.n_lev, nl = sp.n_lines;
    double mx = 0.0, sum = 0.0;
    int64_t cnt = 0, fb = 0, kept = 0;
    const bool skip = p < P && model_done != nullptr && model_done[model_of[p]];
    bool todo = p < P && !skip;
    if (skip) {
        // converged model: populations stay as they are
        for (int i = 0; i < n; ++i) pops_new[p * n + i] = pops_old[p * n + i];
        if (flags) flags[p] = 0;
    }
    if (__any(todo)) {
        const int64_t q = p < P ? p : P - 1;   // lanes past the end repeat the last point
        const double T = Tg[q], nh = nh2[q], nt = cell[q].ntot;
        double x[N > 0 ? N : kMaxLev];
        uint8_t f = 2;
        // with the ALO; Sec. 6.1: redo without it, then keep the old populations
        for (int attempt = 0; attempt < 2; ++attempt) {
            const bool alo = attempt == 0 && use_alo != 0;
            double y[N > 0 ? N : kMaxLev];
            const bool ok = solve_rates<N>(sp, T, nh, nt, (alo ? Jeff : J) + q * nl, L + q * nl, alo, lds, y) == 0 &&
                            valid(n, y);
            if (ok && f == 2) {
                f = (uint8_t)attempt;
#pragma unroll
                for (int i = 0; i < (N > 0 ? N : kMaxLev); ++i)
                    if (N > 0 || i < n) x[i] = y[i];
            }
            if (!__any(todo && f == 2)) break;
        }
        if (todo) {
#pragma unroll
            for (int i = 0; i < (N > 0 ? N : kMaxLev); ++i) {
                if (N == 0 && i >= n) break;
                const double old = pops_old[p * n + i];
                if (f == 2) x[i] = old;
                pops_new[p * n + i] = x[i];
                if (x[i] / nt > 1e-10) {
                    double d = fabs(x[i] - old) / x[i];
                    mx = fmax(mx, d);
                    sum += d;
                    ++cnt;
                }
            }
            if (flags) flags[p] = f;
            fb = (f == 1);
            kept = (f == 2);
        }
    }
    report_change(mx, sum, cnt, fb, kept, p, P, model_of, model_change, partials);
}

int64_t stateq_blocks(int64_t P) { return (P + kWave - 1) / kWave; }

template <int N>
static hipError_t launch_stateq_n(const SpeciesDev &sp, const CellRec *cell, const double *nh2, const double *T,
                                  int64_t P, int use_alo, const double *pops_old, const double *J, const double *Jeff,
                                  const double *L, double *pops_new, uint8_t *flags, ConvPartial *partials,
                                  const uint8_t *model_done, const int32_t *model_of,
                                  unsigned long long *model_change, hipStream_t s)
{
    if constexpr (N > 0) {
        if (sp.n_lev != N)
            return launch_stateq_n<N - 1>(sp, cell, nh2, T, P, use_alo, pops_old, J, Jeff, L, pops_new, flags,
                                          partials, model_done, model_of, model_change, s);
    }
    hipLaunchKernelGGL(k_stateq<N>, dim3((unsigned)stateq_blocks(P)), dim3(kWave), sizeof(double) * N * N * kWave, s,
                       sp, cell, nh2, T, P, use_alo, pops_old, J, Jeff, L, pops_new, flags, partials, model_done,
                       model_of, model_change);
    return hipGetLastError();
}

hipError_t launch_stateq(const SpeciesDev &sp, const CellRec *cell, const double *nh2,
                         const double *T, int64_t P, int use_alo, const double *pops_old,
                         const double *J, const double *Jeff, const double *L, double *pops_new,
                         uint8_t *flags, ConvPartial *partials,
                         const uint8_t *model_done, const int32_t *model_of,
                         unsigned long long *model_change, hipStream_t s)
{
    if (P == 0) return hipSuccess;
    return launch_stateq_n<11>(sp, cell, nh2, T, P, use_alo, pops_old, J, Jeff, L, pops_new, flags, partials,
                               model_done, model_of, model_change, s);
}

// Per-model convergence after an iteration: a model still iterating counts one more
// iteration, records its maximum relative change and stops once it is below tol.
__global__ void k_model_update(int n_models, const unsigned long long *__restrict__ change,
                               uint8_t *__restrict__ done, int32_t *__restrict__ iters,
                               double *__restrict__ last, double tol, int32_t *active)
{
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= n_models || done[m]) return;
    iters[m] += 1;
    const double ch = __longlong_as_double((long long)change[m]);
    last[m] = ch;
    if (ch < tol)
        done[m] = 1;
    else
        atomicAdd(active, 1);
}

hipError_t launch_model_update(int n_models, unsigned long long *change, uint8_t *done, int32_t *iters,
                               double *last, double tol, int32_t *active, hipStream_t s)
{
    hipLaunchKernelGGL(k_model_update, dim3((n_models + 255) / 256), dim3(256), 0, s, n_models, change, done,
                       iters, last, tol, active);
    return hipGetLastError();
}

// Fill kernels (used instead of memset nodes so that the iteration can be captured).
__global__ void k_fill_u64(unsigned long long *p, int64_t n, unsigned long long v)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void k_fill_u8(uint8_t *p, int64_t n, uint8_t v)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

hipError_t launch_fill_u64(unsigned long long *p, int64_t n, unsigned long long v, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u64, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t launch_fill_u8(uint8_t *p, int64_t n, uint8_t v, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u8, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

// Deterministic final reduction of the per-block partials (one workgroup, fixed order).
__global__ __launch_bounds__(256) void k_conv_final(const ConvPartial *__restrict__ part, int64_t n,
                                                    ConvResult *out)
{
    __shared__ double s_max[256], s_sum[256];
    __shared__ int64_t s_cnt[256], s_fb[256], s_kept[256];
    const int t = threadIdx.x;
    double mx = 0.0, sum = 0.0;
    int64_t cnt = 0, fb = 0, kept = 0;
    for (int64_t i = t; i < n; i += 256) {
        mx = fmax(mx, part[i].max_change);
        sum += part[i].sum_change;
        cnt += part[i].count;
        fb += part[i].n_fallback;
        kept += part[i].n_kept;
    }
    s_max[t] = mx;
    s_sum[t] = sum;
    s_cnt[t] = cnt;
    s_fb[t] = fb;
    s_kept[t] = kept;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (t < w) {
            s_max[t] = fmax(s_max[t], s_max[t + w]);
            s_sum[t] += s_sum[t + w];
            s_cnt[t] += s_cnt[t + w];
            s_fb[t] += s_fb[t + w];
            s_kept[t] += s_kept[t + w];
        }
        __syncthreads();
    }
    if (t == 0) {
        ConvResult r;
        r.max_change = s_max[0];
        r.mean_change = s_cnt[0] ? s_sum[0] / (double)s_cnt[0] : 0.0;
        r.n_fallback = s_fb[0];
        r.n_kept = s_kept[0];
        *out = r;
    }
}

hipError_t launch_conv_final(const ConvPartial *partials, int64_t n, ConvResult *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_conv_final, dim3(1), dim3(256), 0, s, partials, n, out);
    return hipGetLastError();
}

}  // namespace nlte
