// Images of the model (Sec. 3.5): the intensity leaving the model along an image
// direction n at the far end of the ray pair through every point, at observer-frame
// channel velocities v.  The pixel of point O sits at O's projection on the plane
// orthogonal to n.
//
// Along the pair (the cached walk of the antipode from its far end to O, then the walk
// of n outward) the profile offset at node k is x_k = (v - n.v_k)/v_w,k.  The
// second-order system of the pair (Sec. 3.3) is eliminated from the upwind end to the
// emergent end E, which plays the part of the origin with an empty far side, so that
//   u_E = (h_E S_E + y + I_in) / (h_E + Q + 1),   I_out = 2 u_E - I_in
// (u = (I(n) + I(-n))/2 with the CMB entering at E).  The elimination uses the
// division-free scaled state of the formal solve (n, d, y~ with Q = n/(sqrt 2 d),
// y = y~/(sqrt 2 d), P = D_+/sqrt 2) in FP64; velocity sub-steps interpolate z, the
// Doppler coefficients, kappa and S linearly as in the formal solve.
//
// One wave per point and block of 64 channels, one channel per lane.  The wave stages up
// to 64 nodes of the pair at a time in LDS (gathered by the lanes together) and sweeps
// them with uniform control flow, two segments at a time where neither has sub-steps (their
// profiles are independent).  Inside a sub-step segment the offset is linear in the
// step index, so e^{-x^2} follows the multiplicative recurrence g <- g r, r <- r c with
// exact restarts after at most 16 widths of travel; cell nodes and short segments
// evaluate the exponential directly.  The state only grows; it is rescaled by a power of two
// once d passes 2^300, checked at least every fourth step.
// Instruction issue bounds it (5,000 vector instructions per wave, issued 99% of the time), so its
// time follows the clock: 64 channels of a disc of 40,009 points 301 us in a long series, 435
// within ten calls of an idle GPU; with an exponential of degree 11 and a rescaling at every
// node 353 and 505.
#include "nlte_internal.h"
#include "device_math.h"

namespace nlte {

namespace {

constexpr double kSqrt2i = 1.41421356237309504880;
constexpr double kInvSqrt2 = 0.70710678118654752440;

// Staged base node (sweep order): Doppler coefficients x = a x_O - b in O's frame, line
// coefficients, and the segment to the next node: optical-depth weight hz = (z_next - z) /
// (2 sqrt 2 m) of its m sub-intervals, over each of which the offset changes by da x_O - db,
// kappa hz by dkq and S by dS.
struct alignas(16) ImgNode {
    double kap, S, a, b, hz, da, db, dkq, dS, pad;
};

// Up to this many sub-steps the profile is evaluated directly: the recurrence takes two
// exponentials to start and saves one per inner sub-node and the end node's (the disc's
// image at 1, 2, 3, 5, 8: 486, 395, 389, 397, 403 us in one short series).
constexpr int kDirect = 3;

constexpr double kRescaleAbove = 2.0370359763344861e90;   // 2^300

__device__ __forceinline__ double profile(double x, const double *tab) { return exp_tab64(-(x * x), tab); }

struct Elim {
    double n, d, y, Pm;   // scaled elimination state and the previous step's P
};

// S is the source of the node that the step eliminates.
__device__ __forceinline__ void elim(Elim &e, double P, double S)
{
    const double t = e.Pm + P;
    e.n = fma(t, e.d, e.n);
    e.y = fma(S * t, e.d, e.y);
    e.d = fma(P, e.n, e.d);
    e.Pm = P;
}

__device__ __forceinline__ void rescale_if_big(Elim &e)
{
    if (e.d > kRescaleAbove) {
        const int ex = __builtin_amdgcn_frexp_exp(e.d);
        e.n = ldexp(e.n, -ex);
        e.d = ldexp(e.d, -ex);
        e.y = ldexp(e.y, -ex);
    }
}

}  // namespace

__global__ __launch_bounds__(64) void k_image(ImageArgs a)
{
    __shared__ ImgNode nd[kWave];
    __shared__ double tab[64];
    tab[threadIdx.x] = kExp2SixtyFourths[threadIdx.x];
    const int chunks = (a.n_ch + kWave - 1) / kWave;
    const int64_t O = blockIdx.x / chunks;
    const int lane = threadIdx.x;
    const int ch = (int)(blockIdx.x % chunks) * kWave + lane;
    if (O >= a.P) return;
    const bool act = ch < a.n_ch;
    const double nx = a.dir[3 * a.ray], ny = a.dir[3 * a.ray + 1], nz = a.dir[3 * a.ray + 2];
    const CellRec cO = a.cell[O];
    const double xO = act ? (a.v_ch[ch] - ((cO.vx * nx + cO.vy * ny) + cO.vz * nz)) / cO.vw : 0.0;
    double xmax = fabs(xO);
    for (int o = kWave / 2; o > 0; o >>= 1) xmax = fmax(xmax, __shfl_xor(xmax, o));
    const double2 *lc = reinterpret_cast<const double2 *>(a.lc);

    // base nodes in sweep order: the antipode's walk from its far end, O, the walk along n
    const int rb = a.anti[a.ray];
    const int64_t bb = a.roff[O * a.n_rays + rb], be = a.roff[O * a.n_rays + rb + 1];
    const int64_t fb = a.roff[O * a.n_rays + a.ray];
    const int nb = (int)(be - bb);
    const int Ls = nb + (int)(a.roff[O * a.n_rays + a.ray + 1] - fb);   // segments

    Elim e;
    e.n = kSqrt2i;
    e.d = 1.0;
    e.y = kSqrt2i * a.I_in;
    e.Pm = 0.0;
    // the current node's offset, profile, kappa and S
    double x_cur = 0.0, g_cur = 0.0, kap_cur = 0.0, S_cur = 0.0;
    float travel = 0.0f;   // bounds how far x moved (any lane) since g was last evaluated exactly
    for (int b0 = 0; b0 < Ls; b0 += kWave - 1) {
        __syncthreads();
        // ---- stage nodes b0 .. b0 + 63
        const int sidx = b0 + lane;
        const bool load = sidx <= Ls, seg = sidx < Ls && lane < kWave - 1;
        double z = 0.0, sv = 0.0, vw = 1.0, an = 0.0, bn = 0.0;
        double2 k = {0.0, 0.0};
        if (load) {
            const int64_t c = sidx < nb ? (int64_t)a.rcells[be - 1 - sidx]
                                        : (sidx == nb ? O : (int64_t)a.rcells[fb + (sidx - nb - 1)]);
            const CellRec cc = a.cell[c];
            k = lc[c * a.n_lines + a.line];
            const double dx = cc.px - cO.px, dy = cc.py - cO.py, dz = cc.pz - cO.pz;
            z = (dx * nx + dy * ny) + dz * nz;
            const double dvx = cc.vx - cO.vx, dvy = cc.vy - cO.vy, dvz = cc.vz - cO.vz;
            sv = (dvx * nx + dvy * ny) + dvz * nz;
            vw = cc.vw;
            an = cO.vw / vw;
            bn = sv / vw;
        }
        const double zn = __shfl_down(z, 1), sn = __shfl_down(sv, 1), vwn = __shfl_down(vw, 1);
        const double an1 = __shfl_down(an, 1), bn1 = __shfl_down(bn, 1);
        const double kn1 = __shfl_down(k.x, 1), Sn1 = __shfl_down(k.y, 1);
        int m_seg = 1, K_seg = 64;   // sub-intervals, and the restart interval of the recurrence (0: direct)
        float dx_seg = 0.0f;         // bound on |dx| over the block's channels
        if (load) {
            ImgNode v{};
            v.kap = k.x;
            v.S = k.y;
            v.a = an;
            v.b = bn;
            if (seg) {
                // velocity sub-steps (Sec. 3.2): split when the projected velocity changes by
                // more than f_sub of the smaller line-width speed
                const double ds = fabs(sn - sv);
                const double thr = a.f_sub * fmin(vw, vwn);
                if (ds > thr) {
                    const double mr = ceil(ds / thr);
                    m_seg = mr < (double)kMaxSub ? (int)mr : kMaxSub;
                }
                const double im = 1.0 / (double)m_seg;
                v.hz = 0.5 * kInvSqrt2 * (zn - z) * im;
                v.da = (an1 - an) * im;
                v.db = (bn1 - bn) * im;
                v.dkq = (kn1 - k.x) * im * v.hz;
                v.dS = (Sn1 - k.y) * im;
                const double maxdx = (fabs(an1 - an) * xmax + fabs(bn1 - bn)) * im;
                dx_seg = (float)maxdx * 1.0000002f;
                K_seg = maxdx > 4.0 ? 0 : (maxdx > 0.25 ? (int)(16.0 / maxdx) : 64);
            }
            nd[lane] = v;
        }
        const unsigned long long sub_mask = __ballot(m_seg > 1);
        __syncthreads();
        // ---- sweep the staged segments
        const int nseg = min(kWave - 1, Ls - b0);
        if (b0 == 0) {
            x_cur = fma(nd[0].a, xO, -nd[0].b);
            g_cur = profile(x_cur, tab);
            kap_cur = nd[0].kap;
            S_cur = nd[0].S;
        }
        for (int i = 0; i < nseg; ++i) {
            if (i + 1 < nseg && ((sub_mask >> i) & 3) == 0) {
                // a run of segments without sub-steps, two at a time (an odd last one takes the
                // general path)
                const unsigned long long ends = sub_mask >> i;
                const int left = nseg - i;
                for (int k2 = (ends ? min((int)__builtin_ctzll(ends), left) : left) >> 1; k2 > 0; --k2, i += 2) {
                    const ImgNode n1 = nd[i + 1], n2 = nd[i + 2];
                    const double h0 = nd[i].hz, h1 = n1.hz;
                    const double x1 = fma(n1.a, xO, -n1.b), x2 = fma(n2.a, xO, -n2.b);
                    const double g1 = profile(x1, tab), g2 = profile(x2, tab);
                    elim(e, fma(kap_cur, g_cur * h0, n1.kap * (g1 * h0)), S_cur);
                    elim(e, fma(n1.kap, g1 * h1, n2.kap * (g2 * h1)), n1.S);
                    rescale_if_big(e);
                    x_cur = x2;
                    g_cur = g2;
                    kap_cur = n2.kap;
                    S_cur = n2.S;
                }
                travel = 0.0f;
                --i;
                continue;
            }
            const ImgNode n0 = nd[i], n1 = nd[i + 1];
            const double xn = fma(n1.a, xO, -n1.b);
            const double hz = n0.hz;
            double q = kap_cur * (g_cur * hz);   // the last node's weight in this segment's steps
            double gn;
            const int m = __builtin_amdgcn_readlane(m_seg, i);
            if (m == 1) {
                gn = profile(xn, tab);
                travel = 0.0f;
            } else {
                const double dx = fma(n0.da, xO, -n0.db);
                const double kq0 = kap_cur * hz, S0 = S_cur;
                const int K = __builtin_amdgcn_readlane(K_seg, i);
                const float maxdx = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, dx_seg), i));
                auto step = [&](double qj, double Sj) {
                    elim(e, q + qj, S_cur);
                    q = qj;
                    S_cur = Sj;
                };
                if (K == 0 || m <= kDirect) {
                    for (int j = 1; j < m; ++j) {
                        const double fj = (double)j;
                        step(fma(fj, n0.dkq, kq0) * profile(fma(fj, dx, x_cur), tab), fma(fj, n0.dS, S0));
                        if ((j & 3) == 3) rescale_if_big(e);
                    }
                    gn = profile(xn, tab);
                    travel = 0.0f;
                } else {
                    // g_{j+1} = g_j r_j, r_{j+1} = r_j c with r_j = e^{-2 x_j dx - dx^2} and
                    // c = e^{-2 dx^2}; exact values again whenever x may have moved by more
                    // than 16 widths since the last exact one, so that an underflowed value
                    // (|x| > 27) cannot hide a profile above e^{-121}
                    const double u2 = 2.0 * dx * dx;
                    const double c = maxdx <= 0.5f ? exp_neg_small(u2) : exp_tab64(-u2, tab);
                    double g = g_cur;
                    double r = exp_tab64(fmin(-(2.0 * x_cur + dx) * dx, 700.0), tab);
                    double kq = kq0, St = S0;
                    int budget = K;
                    if (maxdx > 0.0f) budget = (int)fminf((16.0f - travel) * __builtin_amdgcn_rcpf(maxdx), (float)K);
                    if (budget < 1) {
                        g = profile(x_cur, tab);
                        travel = 0.0f;
                        budget = K;
                    }
                    auto recur = [&] {
                        g *= r;
                        r *= c;
                        kq += n0.dkq;
                        St += n0.dS;
                        step(kq * g, St);
                    };
                    int j = 0;
                    for (;;) {
                        const int jend = min(j + budget, m);
                        const int jint = min(jend, m - 1);
                        int jj = j;
                        for (; jj + 3 < jint; jj += 4) {
                            recur();
                            recur();
                            recur();
                            recur();
                            rescale_if_big(e);
                        }
                        // the last 0-3 steps (checked after the cell node's)
                        const int rem = jint - jj;
                        if (rem >= 2) {
                            recur();
                            recur();
                        }
                        if (rem & 1) recur();
                        travel += maxdx * (float)(jint - j);
                        j = jint;
                        if (jend == m) {
                            g *= r;   // the cell node at the end of the segment
                            travel += maxdx;
                            break;
                        }
                        rescale_if_big(e);
                        const double xj = fma((double)j, dx, x_cur);
                        g = profile(xj, tab);
                        r = exp_tab64(fmin(-(2.0 * xj + dx) * dx, 700.0), tab);
                        kq = fma((double)j, n0.dkq, kq0);
                        St = fma((double)j, n0.dS, S0);
                        travel = 0.0f;
                        budget = K;
                    }
                    gn = g;
                }
            }
            elim(e, fma(n1.kap, gn * hz, q), S_cur);
            rescale_if_big(e);
            x_cur = xn;
            g_cur = gn;
            kap_cur = n1.kap;
            S_cur = n1.S;
        }
    }
    // the last node is the emergent end: its far side is empty (Q = 1, y = I_in)
    const double id = 1.0 / e.d;
    const double u = (e.Pm * S_cur + e.y * id + kSqrt2i * a.I_in) / (e.Pm + e.n * id + kSqrt2i);
    if (act) a.I[O * a.n_ch + ch] = 2.0 * u - a.I_in;
}

// Image-plane coordinates (x . e1, x . e2) of every point.
__global__ void k_image_plane(const CellRec *__restrict__ cell, double3 e1, double3 e2, int64_t P,
                              double *__restrict__ xy)
{
    const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (p >= P) return;
    const CellRec c = cell[p];
    xy[2 * p] = (c.px * e1.x + c.py * e1.y) + c.pz * e1.z;
    xy[2 * p + 1] = (c.px * e2.x + c.py * e2.y) + c.pz * e2.z;
}

hipError_t launch_image(const ImageArgs &a, hipStream_t s)
{
    if (a.P == 0) return hipSuccess;
    const int64_t chunks = (a.n_ch + 63) / 64;
    hipLaunchKernelGGL(k_image, dim3((unsigned)(a.P * chunks)), dim3(64), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_image_plane(const CellRec *cell, double3 e1, double3 e2, int64_t P, double *xy, hipStream_t s)
{
    if (P == 0) return hipSuccess;
    hipLaunchKernelGGL(k_image_plane, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, s, cell, e1, e2, P, xy);
    return hipGetLastError();
}

}  // namespace nlte
