// Per-point setup, LTE populations and the neighbour-graph ray walk.
//
// Everything here is compiled with -ffp-contract=off: the walk's comparisons and the
// line-width speeds feed integer decisions (the next cell, the number of velocity
// sub-steps) that must not depend on fused rounding.
#include <hipcub/hipcub.hpp>

#include "nlte_internal.h"

namespace nlte {

// Sec. 2.2.1: v_th = sqrt(2kT/m); the line width is nu/c sqrt(v_th^2 + v_turb^2).
__global__ void k_setup_points(const double *__restrict__ pos, const double *__restrict__ vel,
                               const double *__restrict__ nh2, const double *__restrict__ T,
                               const double *__restrict__ vturb, const double *__restrict__ X,
                               double mass, int64_t P, CellRec *__restrict__ cell, double4 *__restrict__ pn)
{
    int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (p >= P) return;
    CellRec c;
    c.px = pos[3 * p];
    c.py = pos[3 * p + 1];
    c.pz = pos[3 * p + 2];
    c.vx = vel[3 * p];
    c.vy = vel[3 * p + 1];
    c.vz = vel[3 * p + 2];
    double vth2 = 2.0 * kKB * T[p] / mass;
    c.vw = sqrt(vth2 + vturb[p] * vturb[p]);
    c.ntot = X[p] * nh2[p];
    cell[p] = c;
    pn[p] = make_double4(c.px, c.py, c.pz, nh2[p]);
}

hipError_t launch_setup_points(const double *pos, const double *vel, const double *nh2,
                               const double *T, const double *vturb, const double *X,
                               double mass, int64_t P, CellRec *cell, double4 *pn, hipStream_t s)
{
    if (P == 0) return hipSuccess;
    int64_t blocks = (P + 255) / 256;
    hipLaunchKernelGGL(k_setup_points, dim3((unsigned)blocks), dim3(256), 0, s, pos, vel, nh2, T,
                       vturb, X, mass, P, cell, pn);
    return hipGetLastError();
}

// Boltzmann populations at the local temperature, normalised to the species density.
__global__ void k_lte(SpeciesDev sp, const CellRec *__restrict__ cell, const double *__restrict__ T,
                      int64_t P, double *__restrict__ pops)
{
    int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (p >= P) return;
    double kT = kKB * T[p];
    double Z = 0.0;
    for (int i = 0; i < sp.n_lev; ++i) Z += sp.g[i] * exp(-(sp.E[i] - sp.E[0]) / kT);
    double nt = cell[p].ntot;
    for (int i = 0; i < sp.n_lev; ++i)
        pops[p * sp.n_lev + i] = nt * sp.g[i] * exp(-(sp.E[i] - sp.E[0]) / kT) / Z;
}

hipError_t launch_lte(const SpeciesDev &sp, const CellRec *cell, const double *T, int64_t P,
                      double *pops, hipStream_t s)
{
    if (P == 0) return hipSuccess;
    hipLaunchKernelGGL(k_lte, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, s, sp, cell, T, P, pops);
    return hipGetLastError();
}

// ---------------------------------------------------------------- ray walk (Sec. 3.2)
//
// From the current cell the walk moves to the neighbour whose projection Z on the ray
// exceeds the current one and whose squared distance q to the line through the origin is
// smallest (ties: lower index), and stops when no neighbour lies farther along the ray or
// at a flagged boundary point.  Z strictly increases, so at most P steps are taken.
//
// These decisions are those of FP64 arithmetic in a fixed order (exact_step below).  What
// bounds the walk is reading every neighbour of every cell on the way: the gathers'
// transactions first (one per lane and 16 bytes when every lane follows its own ray), then
// the bytes.  So four lanes share a ray and read a cell's slots together, 64 contiguous
// bytes at a time, and a slot holds the neighbour's offset from the cell in FP32 (16 bytes
// with its index, where its FP64 position takes 32).  The FP32 evaluation decides where the
// best candidate is ahead of the second by more than the evaluation's error; otherwise the
// four lanes repeat the step in FP64.
//
// Error of the FP32 form, lengths in units of the model's extent R: with e the current
// cell's offset from the line (FP64, rounded once), d a neighbour's offset from the cell and
// n the direction, p = e + d - (d.n) n is off by less than 5e-7 (|e| + |d|) and q = |p|^2 by
// less than 2.4e-6 (e^2 + d^2); the FP64 values themselves are off by about 1e-15 R, less
// than 1e-7 |d| since cells with a neighbour nearer than 1e-8 R take the FP64 step.  Two
// values of q differ by more than 1e-5 (e^2 + max d^2), or the step is repeated.  A neighbour
// with |d.n| <= 2e-6 |d|, whose sign FP32 may miss, is never taken without the repeat, but asks
// for it only where its q rivals the best candidate's.  Across an axis ray of a lattice it does
// not: the walks of two axis rays through 30^3 points took 0.50 ms with a repeat wherever there
// is such a neighbour, 0.34 now, 0.43 in FP64 alone; 60^3 points 2.87, 1.13 and 4.02.
//
// A workgroup takes 64 points next to each other in Morton order and one direction, so that
// its walks cross the same cells and have similar lengths; an XCD takes a contiguous range
// of such groups, all directions of the same points after one another.
//
// Instruction issue bounds it now (vector instructions issued 85% of the time in the count, 91%
// in the fill, at 3.4 and 4.0 waves per SIMD; 0.3 and 1.1 TB/s).
// Measured on the outflow of 50,000 points with 48 rays (84 M steps): count 2.31 ms with the
// step counts, fill 1.83 ms (2.63 and 2.36 with branches on candidates and rivals in place of
// selects).  One lane per ray, one point's rays per wave and 32-byte FP64
// slots took 10.4 and 11.0 ms, and the step counts 1.6 ms more in a kernel of their own.

__device__ __forceinline__ float quad_xor1(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, true));
}
__device__ __forceinline__ float quad_xor2(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xF, 0xF, true));
}
__device__ __forceinline__ int quad_xor1(int v) { return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true); }
__device__ __forceinline__ int quad_xor2(int v) { return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true); }

// One step in FP64, the arithmetic that defines the walk.  The four lanes of a ray take
// every fourth slot each; all four return the same neighbour (-1: none).
__device__ __forceinline__ int32_t exact_step(const CellRec *__restrict__ cell, const NbrSlot *__restrict__ slots,
                                              int kp, int sub, double ox, double oy, double oz, double nx, double ny,
                                              double nz, double zcur)
{
    int32_t best = -1;
    double bq = 0.0;
    for (int s = sub; s < kp; s += 4) {
        const int32_t m = slots[s].m;
        if (m < 0) continue;
        const double dx = cell[m].px - ox, dy = cell[m].py - oy, dz = cell[m].pz - oz;
        const double Z = (dx * nx + dy * ny) + dz * nz;
        if (!(Z > zcur)) continue;
        const double qx = dx - Z * nx, qy = dy - Z * ny, qz = dz - Z * nz;
        const double qq = (qx * qx + qy * qy) + qz * qz;
        if (best < 0 || qq < bq || (qq == bq && m < best)) {
            best = m;
            bq = qq;
        }
    }
#pragma unroll
    for (int o = 1; o <= 2; o <<= 1) {
        const int32_t om = __shfl_xor(best, o);
        const double oq = __shfl_xor(bq, o);
        if (om >= 0 && (best < 0 || oq < bq || (oq == bq && om < best))) {
            best = om;
            bq = oq;
        }
    }
    return best;
}

// FILL false: every ray's length, and per origin point the elimination steps per frequency
// of its rays (their cells plus the velocity sub-steps of the segments between them, by the
// sweep's rule) added to cost.  FILL true: the cells.
template <bool FILL>
__global__ __launch_bounds__(256) void k_walk(WalkArgs a, int64_t *__restrict__ len_out,
                                              unsigned long long *__restrict__ cost, const int64_t *__restrict__ off,
                                              int32_t *__restrict__ cells_out)
{
    const int sub = threadIdx.x & 3, kp = a.kp;
    const int64_t n_groups = (a.P + 63) / 64 * a.n_rays;
    const int64_t per_xcd = (n_groups + 7) / 8;
    for (int64_t v = blockIdx.x; v < per_xcd * 8; v += gridDim.x) {   // (gridDim.x is a multiple of 8)
        const int64_t g = (v & 7) * per_xcd + (v >> 3);
        if (g >= n_groups) continue;
        const int64_t block = g / a.n_rays;
        const int r = (int)(g - block * a.n_rays);
        const int64_t rank = block * 64 + (threadIdx.x >> 2);
        if (rank >= a.P) continue;
        const int64_t O = a.order[rank];
        const int64_t q = O * a.n_rays + r;
        const double nx = a.dir[3 * r], ny = a.dir[3 * r + 1], nz = a.dir[3 * r + 2];
        const float fx = (float)nx, fy = (float)ny, fz = (float)nz;
        const double ox = a.cell[O].px, oy = a.cell[O].py, oz = a.cell[O].pz;
        const double ovx = a.cell[O].vx, ovy = a.cell[O].vy, ovz = a.cell[O].vz;
        int64_t cur = O, len = 0, base = FILL ? off[q] : 0;
        double zcur = 0.0, s_prev = 0.0, w_prev = a.cell[O].vw;
        float ex = 0.0f, ey = 0.0f, ez = 0.0f;   // offset of the current cell from the line / R
        unsigned long long n = 0;
        int32_t hold = 0;                         // FILL: this lane's cell of every four
        for (int64_t step = 0; step < a.P; ++step) {
            if (a.bnd != nullptr && cur != O && a.bnd[cur]) break;
            const NbrSlot *slots = a.tab + cur * kp;
            float bq = INFINITY, q2 = INFINITY, dmax = 0.0f;
            int32_t best = -1;
#pragma unroll 3
            for (int s = sub; s < kp; s += 4) {
                const NbrSlot e = slots[s];
                const float dn = fmaf(e.z, fz, fmaf(e.y, fy, e.x * fx));
                const float px = ex + fmaf(-dn, fx, e.x), py = ey + fmaf(-dn, fy, e.y), pz = ez + fmaf(-dn, fz, e.z);
                const float qq = fmaf(pz, pz, fmaf(py, py, px * px));
                const float d2 = fmaf(e.z, e.z, fmaf(e.y, e.y, e.x * e.x));
                // ahead for certain: a candidate; ahead or not: a rival (NaN: a cell that needs FP64)
                const bool sure = dn * dn > 4e-12f * d2;
                const float qc = e.m >= 0 && sure && dn > 0.0f ? qq : INFINITY;
                const float qr = e.m >= 0 && !sure ? (qq >= 0.0f ? qq : -1.0f) : INFINITY;
                dmax = fmaxf(dmax, d2);
                q2 = fminf(fminf(q2, qr), fmaxf(bq, qc));
                best = qc < bq ? e.m : best;
                bq = fminf(bq, qc);
            }
            {
                float oq = quad_xor1(bq);
                int om = quad_xor1(best);
                q2 = fminf(fminf(q2, quad_xor1(q2)), fmaxf(bq, oq));
                best = oq < bq ? om : best;
                bq = fminf(bq, oq);
                oq = quad_xor2(bq);
                om = quad_xor2(best);
                q2 = fminf(fminf(q2, quad_xor2(q2)), fmaxf(bq, oq));
                best = oq < bq ? om : best;
                bq = fminf(bq, oq);
                dmax = fmaxf(dmax, quad_xor1(dmax));
                dmax = fmaxf(dmax, quad_xor2(dmax));
            }
            if (q2 < INFINITY && !(q2 - bq > 1e-5f * (fmaf(ez, ez, fmaf(ey, ey, ex * ex)) + dmax)))
                best = exact_step(a.cell, slots, kp, sub, ox, oy, oz, nx, ny, nz, zcur);
            if (best < 0) break;
            if (FILL) {
                if ((int)(len & 3) == sub) hold = best;
                if ((len & 3) == 3) cells_out[base + (len & ~(int64_t)3) + sub] = hold;
            }
            ++len;
            cur = best;
            const CellRec c = a.cell[cur];
            const double dx = c.px - ox, dy = c.py - oy, dz = c.pz - oz;
            zcur = (dx * nx + dy * ny) + dz * nz;
            ex = (float)((dx - zcur * nx) * a.inv_extent);
            ey = (float)((dy - zcur * ny) * a.inv_extent);
            ez = (float)((dz - zcur * nz) * a.inv_extent);
            if (!FILL) {
                const double dvx = c.vx - ovx, dvy = c.vy - ovy, dvz = c.vz - ovz;
                const double sv = (dvx * nx + dvy * ny) + dvz * nz;
                const double ds = fabs(sv - s_prev), thr = a.f_sub * fmin(c.vw, w_prev);
                unsigned long long m = 1;
                if (ds > thr) {
                    const double mr = ceil(ds / thr);
                    m = mr < (double)kMaxSub ? (unsigned long long)mr : (unsigned long long)kMaxSub;
                }
                n += m;
                s_prev = sv;
                w_prev = c.vw;
            }
        }
        if (FILL) {
            if (sub < (int)(len & 3)) cells_out[base + (len & ~(int64_t)3) + sub] = hold;
        } else if (sub == 0) {
            len_out[q] = len;
            atomicAdd(&cost[O], n + 1);
        }
    }
}

// Neighbour slots for the walks: offsets in units of the extent, kp slots per cell (k rounded
// up to a multiple of four, the rest unused).  A cell with a neighbour nearer than 1e-8 of the
// extent gets a NaN in its first used slot, which sends its steps to FP64.
__global__ void k_nbr_slots(const CellRec *__restrict__ cell, const int32_t *__restrict__ nbr, int k, int kp,
                            int64_t P, double inv_extent, NbrSlot *__restrict__ tab)
{
    const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (p >= P) return;
    bool near = false;
    int first = -1;
    for (int s = 0; s < kp; ++s) {
        NbrSlot e{0.0f, 0.0f, 0.0f, -1};
        const int32_t m = s < k ? nbr[p * k + s] : -1;
        if (m >= 0) {
            const double dx = (cell[m].px - cell[p].px) * inv_extent, dy = (cell[m].py - cell[p].py) * inv_extent,
                         dz = (cell[m].pz - cell[p].pz) * inv_extent;
            e = NbrSlot{(float)dx, (float)dy, (float)dz, m};
            near = near || !((dx * dx + dy * dy) + dz * dz > 1e-16);
            if (first < 0) first = s;
        }
        tab[p * kp + s] = e;
    }
    if (near) tab[p * kp + first].x = NAN;
}

hipError_t launch_nbr_slots(const CellRec *cell, const int32_t *nbr, int k, int kp, int64_t P, double inv_extent,
                            NbrSlot *tab, hipStream_t s)
{
    if (P == 0) return hipSuccess;
    hipLaunchKernelGGL(k_nbr_slots, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, s, cell, nbr, k, kp, P,
                       inv_extent, tab);
    return hipGetLastError();
}

static unsigned walk_grid(const WalkArgs &a)
{
    const int64_t n = (a.P + 63) / 64 * a.n_rays;
    return (unsigned)(((n < (1 << 20) ? n : (1 << 20)) + 7) / 8 * 8);
}

hipError_t launch_walk_count(const WalkArgs &a, int64_t *len, unsigned long long *cost, hipStream_t s)
{
    if (a.P * a.n_rays == 0) return hipSuccess;
    hipLaunchKernelGGL(k_walk<false>, dim3(walk_grid(a)), dim3(256), 0, s, a, len, cost, nullptr, nullptr);
    return hipGetLastError();
}

hipError_t launch_walk_fill(const WalkArgs &a, const int64_t *off, int32_t *cells, hipStream_t s)
{
    if (a.P * a.n_rays == 0) return hipSuccess;
    hipLaunchKernelGGL(k_walk<true>, dim3(walk_grid(a)), dim3(256), 0, s, a, nullptr, nullptr, off, cells);
    return hipGetLastError();
}

// Longest ray and the sum of the points' costs (integers, order-independent): out[0] and
// out[1], zero before the call.
__global__ __launch_bounds__(256) void k_trace_sums(const int64_t *__restrict__ len, int64_t n,
                                                    const unsigned long long *__restrict__ cost, int64_t P,
                                                    unsigned long long *__restrict__ out)
{
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
    unsigned long long mx = 0, sum = 0;
    for (int64_t i = t; i < n; i += stride) mx = max(mx, (unsigned long long)len[i]);
    for (int64_t i = t; i < P; i += stride) sum += cost[i];
    for (int o = kWave / 2; o > 0; o >>= 1) {
        mx = max(mx, __shfl_xor(mx, o));
        sum += __shfl_xor(sum, o);
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        atomicMax(&out[0], mx);
        atomicAdd(&out[1], sum);
    }
}

hipError_t launch_trace_sums(const int64_t *len, int64_t n, const unsigned long long *cost, int64_t P,
                             unsigned long long *out, hipStream_t s)
{
    const int64_t blocks = (n + 255) / 256;
    hipLaunchKernelGGL(k_trace_sums, dim3((unsigned)(blocks < 512 ? (blocks > 0 ? blocks : 1) : 512)), dim3(256), 0, s,
                       len, n, cost, P, out);
    return hipGetLastError();
}

// In-place inclusive scan of lengths stored at [1..n] of an (n+1)-array whose [0] is 0,
// turning them into CSR offsets.  With tmp == nullptr only *tmp_bytes is set.
hipError_t scan_lengths(int64_t *arr, int64_t n, void *tmp, size_t *tmp_bytes, hipStream_t s)
{
    return hipcub::DeviceScan::InclusiveSum(tmp, *tmp_bytes, arr + 1, arr + 1, (int)n, s);
}

__global__ void k_iota(int32_t *__restrict__ v, int64_t n)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) v[i] = (int32_t)i;
}

// Order of the points by decreasing cost (stable: equal costs keep increasing index).
hipError_t sort_by_cost(unsigned long long *cost, int32_t *order, int64_t P, hipStream_t s)
{
    unsigned long long *keys_out = nullptr;
    int32_t *idx_in = nullptr;
    hipError_t e = hipMalloc((void **)&keys_out, sizeof(unsigned long long) * P);
    if (e == hipSuccess) e = hipMalloc((void **)&idx_in, sizeof(int32_t) * P);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_iota, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, s, idx_in, P);
        e = hipGetLastError();
    }
    size_t tmp_bytes = 0;
    if (e == hipSuccess)
        e = hipcub::DeviceRadixSort::SortPairsDescending(nullptr, tmp_bytes, cost, keys_out, idx_in, order, (int)P,
                                                         0, 64, s);
    void *tmp = nullptr;
    if (e == hipSuccess) e = hipMalloc(&tmp, tmp_bytes ? tmp_bytes : 1);
    if (e == hipSuccess)
        e = hipcub::DeviceRadixSort::SortPairsDescending(tmp, tmp_bytes, cost, keys_out, idx_in, order, (int)P, 0,
                                                         64, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (tmp) (void)hipFree(tmp);
    if (keys_out) (void)hipFree(keys_out);
    if (idx_in) (void)hipFree(idx_in);
    return e;
}

// Morton code of a point within its model's bounding box (box[m] = min x, y, z and
// extents): each coordinate quantised to q = floor((x - min) / extent * (2^21 - 1)) (0 for
// a flat extent), bits interleaved x, y, z from the most significant.
__global__ void k_morton(const CellRec *__restrict__ cell, const int32_t *__restrict__ model_of,
                         const double *__restrict__ box, int64_t P, unsigned long long *__restrict__ code)
{
    const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (p >= P) return;
    const double *b = box + 6 * model_of[p];
    const double x[3] = {cell[p].px, cell[p].py, cell[p].pz};
    unsigned long long q[3];
    for (int d = 0; d < 3; ++d) {
        const double ext = b[3 + d];
        q[d] = ext > 0.0 ? (unsigned long long)floor((x[d] - b[d]) / ext * 2097151.0) : 0ull;
    }
    unsigned long long c = 0;
    for (int bit = 0; bit < 21; ++bit)
        for (int d = 0; d < 3; ++d) c |= ((q[d] >> bit) & 1ull) << (3 * bit + 2 - d);
    code[p] = c;
}

// Points of each model (offsets on the device) in Morton order, equal codes by index
// (the radix sort is stable).  Synchronises the stream.
hipError_t morton_order(const CellRec *cell, const int32_t *model_of, const double *box, const int64_t *off,
                        int n_models, int64_t P, int32_t *order, hipStream_t s)
{
    if (P == 0) return hipSuccess;
    unsigned long long *codes = nullptr, *codes_out = nullptr;
    int32_t *idx = nullptr;
    void *tmp = nullptr;
    size_t tmp_bytes = 0;
    hipError_t e = hipMalloc((void **)&codes, sizeof(unsigned long long) * P);
    if (e == hipSuccess) e = hipMalloc((void **)&codes_out, sizeof(unsigned long long) * P);
    if (e == hipSuccess) e = hipMalloc((void **)&idx, sizeof(int32_t) * P);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_morton, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, s, cell, model_of, box, P, codes);
        hipLaunchKernelGGL(k_iota, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, s, idx, P);
        e = hipGetLastError();
    }
    if (e == hipSuccess)
        e = hipcub::DeviceSegmentedRadixSort::SortPairs(nullptr, tmp_bytes, codes, codes_out, idx, order, (int)P,
                                                         n_models, off, off + 1, 0, 63, s);
    if (e == hipSuccess) e = hipMalloc(&tmp, tmp_bytes ? tmp_bytes : 1);
    if (e == hipSuccess)
        e = hipcub::DeviceSegmentedRadixSort::SortPairs(tmp, tmp_bytes, codes, codes_out, idx, order, (int)P,
                                                         n_models, off, off + 1, 0, 63, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (tmp) (void)hipFree(tmp);
    if (codes) (void)hipFree(codes);
    if (codes_out) (void)hipFree(codes_out);
    if (idx) (void)hipFree(idx);
    return e;
}

}  // namespace nlte
