// Ray-pair formal solve (the ALI hot loop): device templates shared by the per-precision
// instantiation units fs_fp64.hip and fs_fp32.hip.  The discretisation and the
// elimination are described at the top of formal_solve.hip.
//
// Mapping: one workgroup = one wave = one origin point and up to 64 (line, frequency)
// items; lanes [0, n_q) take lines line0 .. line0+LPL-1 ("group" 0), lanes [n_q, 2 n_q)
// the next LPL lines (group 1), one frequency per lane.  The Doppler offset of a node
// depends on the frequency only (line widths are proportional to the line frequency), so
// the LPL lines of a lane share its profile evaluation and its recurrence; with up to
// five lines per lane a point's nine lines take a single wave, which stages each ray
// segment and evaluates each profile once.  All lanes walk the same nodes (uniform control
// flow).  The wave stages `ns` nodes of a ray at a time in LDS (Doppler coefficients, the
// length of their segment's sub-steps, kappa and S of its lines; see Node), the sub-step
// counts and what a segment needs of the wave as a whole in scalar registers.
#pragma once
#include <algorithm>
#include <type_traits>

#include "device_math.h"
#include "nlte_internal.h"

namespace nlte {

constexpr double kSqrt2 = 1.41421356237309504880;
constexpr double kInv2Sqrt2 = 0.35355339059327376220;  // 1 / (2 sqrt 2)
// The elimination state only grows (see elim_p); it is rescaled by a power of two once
// any line's D passes 2^300, checked at least every fifth step.  A step multiplies D by at most
// about D_+^2, so the FP64 range leaves room for steps with D_+ up to 2^70 (300 + 5 * 140 of
// 1023).
// Power-of-two rescaling is exact, so when it happens does not change any result.
constexpr double kRenormAbove = 2.0370359763344861e90;   // 2^300

template <bool F32>
struct Bulk {
    using T = double;
    using T2 = double2;
};
template <>
struct Bulk<true> {
    using T = float;
    using T2 = float2;
};

// A staged node of a half ray: one row of Node::kStride values in LDS.
//   (a, b)  the Doppler offset of a lane's frequency x_q at this node, x = a x_q - b;
//   the segment to the next node toward O has m sub-intervals (im = 1/m) of length
//   2 sqrt(2) dzq; per sub-interval x changes by da x_q - db (read by the FP32 form only);
//   kappa, S: line-centre opacity and source function of each line group's lines.
// Two ways to read a node (kRowValues chooses; the values and what is done with them are the same):
//   rows   lane e of every row of 16 lanes loads value e of its line group ([kappa][S] of the
//          group's lines, then the six values of the node), ONE load and one register per node, and
//          each value is broadcast over its row by a DPP move where it is used (all lanes of a row
//          belong to one group).  Between two cells kappa and S are linear, so a velocity sub-node
//          is the two nodes' values combined by one multiply-add for all lines.
//   values every lane loads every value (an LDS broadcast) and keeps its lines' in registers.
// Instruction issue and the number of waves bound the sweep.  Five lines by values kept both
// nodes' values, their differences and the running values in 80 FP64 registers and took an
// instruction for each line and sub-node; by rows a disc of 30,011 points and nine lines takes
// 77 ms (95.6 before), in FP32 one of 24,000 points 45.1 (51.8).  The FP64 long mode gains with two
// lines too (outflow of 20,011 points 4.42 ms by rows, 4.60 by values, 4.75 before); without
// the recurrence's registers, or with one line, the moves cost more than they save (a sphere of
// 30,000 points 1.65 ms by rows, 0.91 by values; that outflow in FP32 4.15 and 3.53).
template <bool F32, int LPL, bool LONG>
inline constexpr bool kRowValues = LPL >= 4 || (!F32 && LONG && LPL >= 2);

template <int LPL, bool ROWS>
struct Node {
    static constexpr int kCommon = 4 * LPL;              // a, b, dzq, im, da, db
    // (rows: odd, so that nodes start in different banks when they are written; otherwise
    // even, so that values are read in aligned pairs)
    static constexpr int kStride = 4 * LPL + 6 + (ROWS ? 1 : 0);
};

// The value that lane N of this lane's row of 16 holds.  FP64 by one 64-bit move: the compiler's
// builtin takes 32-bit values only, so its intrinsic is bound by name (a compiler without it stops
// at an undefined symbol).  Two 32-bit moves in its place: the disc of 30,011 points 76.8 -> 79.4 ms,
// the FP32 disc 44.8 -> 46.7, the outflow of 20,011 points 4.45 -> 4.60, its batched ALI 19.3 -> 20.2.
extern "C" __device__ __attribute__((const)) long nlte_update_dpp_i64(long, long, int, int, int, bool)
    __asm("llvm.amdgcn.update.dpp.i64");
template <int N>
__device__ __forceinline__ double row_value(double v)
{
    return __builtin_bit_cast(double, nlte_update_dpp_i64(0l, __builtin_bit_cast(long, v), 0x150 + N, 0xF, 0xF, true));
}
template <int N>
__device__ __forceinline__ float row_value(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x150 + N, 0xF, 0xF, true));
}

// f(0), f(1), .., f(N - 1) with the argument known when it is compiled (row_value needs that)
template <int N, int I = 0, class F>
__device__ __forceinline__ void unrolled(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        unrolled<N, I + 1>(f);
    }
}

// The kappa and S of a lane's lines at a node: by rows one value of the node per lane.
template <typename T, int LPL, bool ROWS>
struct NodeVals {
    T v[ROWS ? 1 : 2 * LPL];
    template <int L>
    __device__ __forceinline__ T kap() const
    {
        if constexpr (ROWS)
            return row_value<L>(v[0]);
        else
            return v[L];
    }
    template <int L>
    __device__ __forceinline__ T src() const
    {
        return kap<LPL + L>();
    }
    static constexpr int kN = ROWS ? 1 : 2 * LPL;
};

// The same values in FP64 (rows: one conversion for all lines).
template <int LPL, bool ROWS, typename T>
__device__ __forceinline__ NodeVals<double, LPL, ROWS> in_fp64(const NodeVals<T, LPL, ROWS> &v)
{
    NodeVals<double, LPL, ROWS> w;
#pragma unroll
    for (int k = 0; k < w.kN; ++k) w.v[k] = (double)v.v[k];
    return w;
}

// Reads of a staged node: `my` points at this lane's value of node 0 (rows) or at its line
// group's values there, `com` at the node's own values (not for rows).
template <typename T, int LPL, bool ROWS>
struct NodeReader {
    const T *my, *com;
    using Vals = NodeVals<T, LPL, ROWS>;
    typedef T Pair __attribute__((ext_vector_type(2)));
    __device__ __forceinline__ NodeReader(const T *rec, int grp, int lane)
    {
        const int e = lane & 15;
        my = rec + (!ROWS || e < 2 * LPL ? grp * 2 * LPL : 0);
        if constexpr (ROWS) my += e < 2 * LPL ? e : Node<LPL, ROWS>::kCommon + min(e - 2 * LPL, 5);
        com = rec + Node<LPL, ROWS>::kCommon;
    }
    __device__ __forceinline__ Vals values(int i) const
    {
        Vals w;
        if constexpr (ROWS) {
            w.v[0] = my[i * Node<LPL, ROWS>::kStride];
        } else {
#pragma unroll
            for (int k = 0; k < Vals::kN; k += 2) {
                const Pair p = *reinterpret_cast<const Pair *>(my + i * Node<LPL, ROWS>::kStride + k);
                w.v[k] = p.x;
                w.v[k + 1] = p.y;
            }
        }
        return w;
    }
    // value K of the node itself (0 a, 1 b, 2 dzq, 3 im, 4 da, 5 db), whose row values are in w
    template <int K>
    __device__ __forceinline__ T own(int i, const Vals &w) const
    {
        if constexpr (ROWS)
            return row_value<2 * LPL + K>(w.v[0]);
        else
            return (*reinterpret_cast<const Pair *>(com + i * Node<LPL, ROWS>::kStride + (K & ~1)))[K & 1];
    }
};

// Elimination state of a half sweep in homogeneous form: the Rybicki-Hummer quantities
// Q = N / (sqrt 2 D) and y = Y / (sqrt 2 D), and Hm = D_- / sqrt 2, the previous
// optical-depth step (see elim_p).
struct HalfState {
    double N, D, Y, Hm;
    double hd;   // weight h d of the last step (rescaled with the state): the share of the
    double Sl;   // last eliminated node's source Sl in Y (read by the band operator only)
};

// e^{-x^2}: FP64 by the table-driven exponential (tab: 2^{j/64} in LDS); FP32 on the
// hardware exp2, e^{-x^2} = 2^{-x^2 log2 e}.
__device__ __forceinline__ double profile(double x, const double *tab) { return exp_tab64(-(x * x), tab); }
__device__ __forceinline__ float profile(float x, const double *)
{
    return __builtin_amdgcn_exp2f(-(x * x) * 1.44269504088896340736f);
}

// Doppler offset a x_q - b.  (FP32 rounds the product, as it always has.)
template <bool F32>
__device__ __forceinline__ typename Bulk<F32>::T doppler(typename Bulk<F32>::T a, typename Bulk<F32>::T xq,
                                                         typename Bulk<F32>::T b)
{
    if constexpr (F32)
        return a * xq - b;
    else
        return fma(a, xq, -b);
}

template <bool TRACK>
__device__ __forceinline__ void rescale(HalfState &st)
{
    const int e = __builtin_amdgcn_frexp_exp(st.D);
    st.N = ldexp(st.N, -e);
    st.D = ldexp(st.D, -e);
    st.Y = ldexp(st.Y, -e);
    if (TRACK) st.hd = ldexp(st.hd, -e);
}

// One elimination step.  The Rybicki-Hummer update with h = (D_- + D_+)/2 (mean of the
// trapezoid optical depths D_-, D_+ on either side of the node)
//   T = h + Q,  E = 1/(1 + D_+ T),  Q' = T E,  y' = (S h + y) E
// becomes, for Q = N/D and y = Y/D,
//   N' = N + h D,  Y' = Y + S h D,  D' = D + D_+ N'
// (products and sums of non-negative numbers only).  The node coefficients a are
// chi dz / (2 sqrt 2), so Pp = a_prev + a_t = D_+ / sqrt 2, and the state is carried as
// n = sqrt 2 N, y~ = sqrt 2 Y, d = D, which turns the update into
//   n' = n + (P_- + P) d,  y~' = y~ + S (P_- + P) d,  d' = d + P n'
// with no constant factors; Q = n/(sqrt 2 d), y = y~/(sqrt 2 d), and the factor sqrt 2
// cancels in every quantity formed at the origin.  S_row is the source of the row being
// eliminated.  The weight t d is not formed (but for the band operator's record): with S t as a
// factor of its own the new n, y~ and d are two dependent multiply-adds from the old d.
template <bool TRACK = false>
__device__ __forceinline__ void elim_p(double Pp, double S_row, HalfState &st)
{
    const double t = st.Hm + Pp;
    if (TRACK) {
        st.hd = t * st.D;
        st.Sl = S_row;
    }
    st.N = fma(t, st.D, st.N);
    st.Y = fma(S_row * t, st.D, st.Y);
    st.D = fma(Pp, st.N, st.D);
    st.Hm = Pp;
}

// Per-line state of a lane during a half sweep.
template <int LPL>
struct LineState {
    HalfState st[LPL];
    int m_last;   // sub-intervals of the last segment (the one ending at O)
};

// A compiler barrier: values read after it are loaded again instead of being kept in
// registers across the code before it (it emits no instruction).
__device__ __forceinline__ void reload_fence() { __atomic_signal_fence(__ATOMIC_SEQ_CST); }

// Rescale the lanes whose state passed 2^300 (in any of their lines).
template <int LPL, bool TRACK>
__device__ __forceinline__ void rescale_if_big(LineState<LPL> &ls)
{
    bool big = false;
#pragma unroll
    for (int l = 0; l < LPL; ++l) big = big || ls.st[l].D > kRenormAbove;
    if (big) {
#pragma unroll
        for (int l = 0; l < LPL; ++l) rescale<TRACK>(ls.st[l]);
    }
}

// Whether a segment lies beyond the line's range at every frequency of the quadrature, so
// that the sweep may cross it in one step without opacity.  Along it the offset
// x = a x_q - b has |x| >= x_min = min|b| - max(a) max|x_q| (one sign of b at both ends), so
// its optical depth is at most tau = kappa_max dz e^{-x_min^2} and what it emits relative to
// the incoming background at most tau S_max / I_bdy.  Both below 2^-66 change Q = N/D and
// y = Y/D by less than FP64 rounding can show (2^-53), also where an optically thick cell has
// brought Q down by a few orders.  far: log2 of a cell's largest line-centre opacity and of
// its largest S / I_bdy (at least 0) over ALL lines of the species, so that the choice does
// not depend on how the lines are spread over waves; it does not depend on the staging
// window either, and crossing consecutive segments one by one gives the same state.  Where
// e^{-x^2} itself underflows (x^2 > 750 in FP64, 105 in FP32) the opacity is exactly 0
// whatever the populations.
// (|x_min| is about 8 at the densities here.  An outflow of 20,011 points executes 17.3% of
// its steps in FP64, 42.9% with the underflow alone as the bound; a disc of 30,011 points 79.5%
// against 99.7%.  With the lane-wise vote at every segment that this replaces, the outflow's
// iteration took 10.15 ms, now 4.49; the disc's, now also in the short mode, 208 and 95 ms.
// The test costs the staging lanes about 20 instructions per round, none per segment.)
template <bool F32>
__device__ __forceinline__ bool far_segment(bool in, double a0, double b0, double a1, double b1, double dz,
                                            double xq_max, short2 far)
{
    const short2 next = __builtin_bit_cast(short2, __shfl_down(__builtin_bit_cast(int, far), 1));
    const float lkr = (float)(max((int)far.x, (int)next.x) + max((int)far.y, (int)next.y));
    const float xm = (float)(fmin(fabs(b0), fabs(b1)) - fmax(a0, a1) * xq_max);
    const float x2 = xm * xm * 0.99999f;   // (rounded down: this is FP32)
    // (dz < 2^its exponent; in FP32 a length under 1e-38 would be 0 and far whatever its opacity)
    const float tau2 = lkr + (float)__builtin_amdgcn_frexp_exp(dz) - x2 * 1.44269504f;
    return in && b0 * b1 > 0.0 && xm > 0.0f && (tau2 < -66.0f || x2 > (F32 ? 105.0f : 750.0f));
}

// Half-sweep along ray `ray` from its far end to O for Doppler offset xq of this lane.
// The result is left in ls.st (one HalfState per line of the lane).  nexec counts the
// elimination steps the wave executes (a run of far-wing segments counts as one).
// LONG: the long-segment mode, whose sub-steps take the profile by recurrence (FP64 only: the
// FP32 exponential is one instruction).
//
// Carried from node to node: the node's values V (see Node), its offset x_cur and
// profile g_cur, and per line c: in FP64 kappa, with P = kappa_0 (g_0 dzq) + kappa_1 (g_1 dzq),
// which takes the two products with dzq once for all lines; in FP32 kappa g, whose
// P = (kappa_0 g_0) dzq + (kappa_1 g_1) dzq rounds every product (sub-nodes: kappa (g dzq)).
// Control flow is uniform, on masks and counts that the staging lanes left in scalar
// registers; the only branch on a vector result is the check for rescaling.
// Up to three lines leave registers for two profiles at a time, which hide each other's
// latency: a sphere of 30,000 points 0.91 ms against 1.02 one by one, the FP64 outflow 4.4
// against 5.0; with five lines it is the other way round (the disc 77 ms one by one, 89 with
// pairs of sub-nodes, 100 with pairs of segments too).  FP32's long mode, where most segments
// have sub-steps, is better without the pairs of segments (outflow 3.70 against 3.75 ms).
template <bool F32, int LPL, bool LONG, bool TRACK = false>
__device__ __forceinline__ void half_sweep(const SolveArgs &a, typename Bulk<F32>::T *rec, const double *tab, int64_t O,
                                          int ray, typename Bulk<F32>::T xq, int grp, int line0, int nlw,
                                          LineState<LPL> &ls, int64_t &nexec)
{
    using T = typename Bulk<F32>::T;
    using T2 = typename Bulk<F32>::T2;
    constexpr bool kRows = kRowValues<F32, LPL, LONG>, kPairs = LPL == 1 || (LPL <= 3 && !(F32 && LONG));
    using Nd = Node<LPL, kRows>;
    using Vals = NodeVals<T, LPL, kRows>;
    const T2 *lc = reinterpret_cast<const T2 *>(a.lc);
    const int lane = threadIdx.x;
    const int ns = a.ns;   // nodes staged per round (2..64)
    const NodeReader<T, LPL, kRows> node(rec, grp, lane);
#pragma unroll
    for (int l = 0; l < LPL; ++l) {
        // Q = 1, y = I_in at the far boundary (in the scaled state of elim_p)
        const int li = grp * LPL + l;
        ls.st[l].N = kSqrt2;
        ls.st[l].D = 1.0;
        ls.st[l].Y = kSqrt2 * a.ibdy[line0 + (li < nlw ? li : 0)];
        ls.st[l].Hm = 0.0;
        if (TRACK) {
            ls.st[l].hd = 0.0;
            ls.st[l].Sl = 0.0;
        }
    }
    if (TRACK) ls.m_last = 1;
    const int64_t base = O * a.n_rays + ray;
    const int64_t beg = a.roff[base];
    const int L = (int)(a.roff[base + 1] - beg);
    if (L == 0) return;
    T x_cur = 0, g_cur = 0, c[LPL];
    float travel = 0.0f;   // bounds how far x moved (any lane) since g was last evaluated exactly
    int pend = 0;          // steps since rescaling was last checked
    auto check = [&] {
        rescale_if_big<LPL, TRACK>(ls);
        pend = 0;
    };
    auto stepped = [&](int n) {
        pend += n;
        if (pend >= (LPL >= 4 ? 5 : 4)) check();   // (steps come singly, or at most two at a time)
    };
    for (int b0 = 0; b0 < L; b0 += ns - 1) {
        __syncthreads();
        // ---- stage nodes b0 .. b0+ns-1 in sweep order (far end first, O last)
        const int s = b0 + lane;
        double Zs = 0.0, sv = 0.0, vw = 1.0, an = 0.0, bn = 0.0;
        int64_t cidx = O;
        const bool load = lane < ns && s <= L;
        if (load) {
            cidx = (s < L) ? (int64_t)a.rcells[beg + (L - 1 - s)] : O;
            const CellRec cc = a.cell[cidx];
            // O's record and the ray's direction are read again for each staging round (from
            // the caches) rather than held in registers through the sweep
            reload_fence();
            const CellRec cO = a.cell[O];
            const double nx = a.dir[3 * ray], ny = a.dir[3 * ray + 1], nz = a.dir[3 * ray + 2];
            double dx = cc.px - cO.px, dy = cc.py - cO.py, dz = cc.pz - cO.pz;
            Zs = (dx * nx + dy * ny) + dz * nz;
            double dvx = cc.vx - cO.vx, dvy = cc.vy - cO.vy, dvz = cc.vz - cO.vz;
            sv = (dvx * nx + dvy * ny) + dvz * nz;
            vw = cc.vw;
            an = cO.vw / vw;
            bn = sv / vw;
        }
        const double Zn = __shfl_down(Zs, 1), sn = __shfl_down(sv, 1), vwn = __shfl_down(vw, 1);
        const double an1 = __shfl_down(an, 1), bn1 = __shfl_down(bn, 1);
        const bool seg = s < L && lane < ns - 1;   // this lane's node starts a segment of the round
        // segments of this round that every frequency crosses beyond the line's range
        const unsigned long long far_mask = __ballot(
            far_segment<F32>(seg, an, bn, an1, bn1, Zs - Zn, a.xq_max, load ? a.far[cidx] : short2{0, 0}));
        int m_seg = 1, K_seg = 64;   // sub-intervals, and the restart interval of the recurrence (0: direct)
        float dx_seg = 0.0f;         // bound on |dx| over every frequency
        if (load) {
            T *w = rec + lane * Nd::kStride;
#pragma unroll
            for (int l = 0; l < 2 * LPL; ++l) {
                const T2 cl = l < nlw ? lc[cidx * a.n_lines + line0 + l] : T2{0, 0};
                w[(l / LPL) * 2 * LPL + l % LPL] = cl.x;
                w[(l / LPL) * 2 * LPL + LPL + l % LPL] = cl.y;
            }
            double im = 1.0, dzq = 0.0;
            if (seg) {
                // velocity sub-steps (Sec. 3.2): split when the projected velocity changes
                // by more than f_sub of the smaller line-width speed
                const double ds = fabs(sn - sv);
                const double thr = a.f_sub * fmin(vw, vwn);
                if (ds > thr) {
                    const double mr = ceil(ds / thr);
                    m_seg = mr < (double)kMaxSub ? (int)mr : kMaxSub;
                }
                im = 1.0 / (double)m_seg;
                dzq = kInv2Sqrt2 * (Zs - Zn) * im;
                if (LONG && !F32) {
                    // the recurrence of the profile restarts after at most 16 widths of travel (and
                    // divides by dzq at the segment's end)
                    const double maxdx = (fabs(an1 - an) * a.xq_max + fabs(bn1 - bn)) * im;
                    dx_seg = (float)maxdx * 1.0000002f;
                    K_seg = maxdx > 4.0 || !(dzq > 1e-200) ? 0 : (maxdx > 0.25 ? (int)(16.0 / maxdx) : 64);
                }
            }
            w[Nd::kCommon] = (T)an;
            w[Nd::kCommon + 1] = (T)bn;
            w[Nd::kCommon + 2] = (T)dzq;
            w[Nd::kCommon + 3] = (T)im;
            w[Nd::kCommon + 4] = (T)((an1 - an) * im);
            w[Nd::kCommon + 5] = (T)((bn1 - bn) * im);
        }
        const unsigned long long sub_mask = __ballot(m_seg > 1);
        const int nseg = min(ns - 1, L - b0);
        __syncthreads();
        // ---- sweep the staged segments
        Vals V = node.values(0);
        if (b0 == 0) {
            x_cur = doppler<F32>(node.template own<0>(0, V), xq, node.template own<1>(0, V));
            g_cur = profile(x_cur, tab);
        }
        unrolled<LPL>([&](auto l) { c[l] = F32 ? V.template kap<l>() * g_cur : V.template kap<l>(); });
        Vals V1;
        if (kRows) V1 = node.values(1);   // the next node, read one ahead
        for (int i = 0; i < nseg; ++i) {
            if ((far_mask >> i) & 1) {
                // a run of far-wing segments, eliminated in one step (see far_segment; the
                // segment that ends at O, whose step the band operator records, is never one:
                // O's own offsets lie within the quadrature)
                i += (int)__builtin_ctzll(~(far_mask >> i));
                unrolled<LPL>([&](auto l) { elim_p<false>(0.0, (double)V.template src<l>(), ls.st[l]); });
                stepped(1);
                V = node.values(i);
                x_cur = doppler<F32>(node.template own<0>(i, V), xq, node.template own<1>(i, V));
                g_cur = profile(x_cur, tab);
                unrolled<LPL>([&](auto l) { c[l] = F32 ? V.template kap<l>() * g_cur : V.template kap<l>(); });
                travel = 0.0f;
                ++nexec;
                if (i >= nseg) break;
                if (kRows) V1 = node.values(i + 1);
            }
            if (!kRows) V1 = node.values(i + 1);
            if (kPairs && i + 1 < nseg && (((far_mask | sub_mask) >> i) & 3) == 0) {
                // a run of segments without sub-steps, two at a time: both profiles first, which do
                // not depend on the eliminations (an odd last one takes the general path)
                const unsigned long long ends = (far_mask | sub_mask) >> i;
                const int left = nseg - i, run = kRows ? 2 : (ends ? min((int)__builtin_ctzll(ends), left) : left) & ~1;
                nexec += run;
                for (int k = run; k > 0; k -= 2, i += 2) {
                    if (!kRows && k < run) V1 = node.values(i + 1);
                    const Vals V2 = node.values(i + 2);
                    const T dz0 = node.template own<2>(i, V), dz1 = node.template own<2>(i + 1, V1);
                    const T x1 = doppler<F32>(node.template own<0>(i + 1, V1), xq, node.template own<1>(i + 1, V1));
                    const T x2 = doppler<F32>(node.template own<0>(i + 2, V2), xq, node.template own<1>(i + 2, V2));
                    const T g1 = profile(x1, tab), g2 = profile(x2, tab);
                    const T G00 = g_cur * dz0, G01 = g1 * dz0, G10 = g1 * dz1, G11 = g2 * dz1;
                    unrolled<LPL>([&](auto l) {
                        const T k1 = V1.template kap<l>(), k2 = V2.template kap<l>();
                        const double S0 = (double)V.template src<l>(), S1 = (double)V1.template src<l>();
                        if constexpr (F32) {
                            const T u1 = k1 * g1, u2 = k2 * g2;
                            elim_p<TRACK>((double)(c[l] * dz0 + u1 * dz0), S0, ls.st[l]);
                            elim_p<TRACK>((double)(u1 * dz1 + u2 * dz1), S1, ls.st[l]);
                            c[l] = u2;
                        } else {
                            elim_p<TRACK>(fma(c[l], G00, k1 * G01), S0, ls.st[l]);
                            elim_p<TRACK>(fma(k1, G10, k2 * G11), S1, ls.st[l]);
                            c[l] = k2;
                        }
                    });
                    stepped(2);
                    g_cur = g2;
                    x_cur = x2;
                    V = V2;
                    if (kRows) V1 = node.values(min(i + 3, ns - 1));
                }
                travel = 0.0f;
                if (TRACK) ls.m_last = 1;
                --i;
                continue;
            }
            const T dzq = node.template own<2>(i, V);
            const T xn = doppler<F32>(node.template own<0>(i + 1, V1), xq, node.template own<1>(i + 1, V1));
            // the segment's first node: G = g dzq (FP64), or every line's kappa g dzq (FP32)
            T G = g_cur * dzq, gn = 0;
            Vals Vr = V;   // the values of the row to be eliminated next
            if (F32) unrolled<LPL>([&](auto l) { c[l] = c[l] * dzq; });
            int m = 1;
            bool have_gn = false;
            if ((sub_mask >> i) & 1) {
                m = __builtin_amdgcn_readlane(m_seg, i);
                const T im = node.template own<3>(i, V);
                const T dx = F32 ? node.template own<4>(i, V) * xq - node.template own<5>(i, V) : (xn - x_cur) * im;
                Vals dV;
#pragma unroll
                for (int k = 0; k < Vals::kN; ++k) dV.v[k] = (V1.v[k] - V.v[k]) * im;
                // the values of sub-node j, and its step with G = g dzq there
                auto at = [&](T t) {
                    Vals w;
#pragma unroll
                    for (int k = 0; k < Vals::kN; ++k) w.v[k] = fma(t, dV.v[k], V.v[k]);
                    return w;
                };
                auto sub_node = [&](const Vals &w, T G1) {
                    const NodeVals<double, LPL, kRows> Sr = in_fp64<LPL, kRows>(Vr);
                    unrolled<LPL>([&](auto l) {
                        const T k = w.template kap<l>();
                        if constexpr (F32) {
                            const T a1 = k * G1;
                            elim_p<TRACK>((double)(c[l] + a1), Sr.template src<l>(), ls.st[l]);
                            c[l] = a1;
                        } else {
                            elim_p<TRACK>(fma(c[l], G, k * G1), Sr.template src<l>(), ls.st[l]);
                            c[l] = k;
                        }
                    });
                    G = G1;
                    Vr = w;
                };
                const int K = LONG && !F32 ? __builtin_amdgcn_readlane(K_seg, i) : 0;
                if (F32 || !LONG || K == 0 || m <= 2) {
                    // direct evaluation: the only form of the short mode, and where the recurrence
                    // would not pay for its two exponentials or cannot be used
                    int j = 1;
                    if constexpr (LPL <= 3)
                        for (; j + 1 < m; j += 2) {
                            const T t1 = (T)j, t2 = (T)(j + 1);
                            const T G1 = profile(fma(t1, dx, x_cur), tab) * dzq;
                            const T G2 = profile(fma(t2, dx, x_cur), tab) * dzq;
                            sub_node(at(t1), G1);
                            sub_node(at(t2), G2);
                            stepped(2);
                        }
                    for (; j < m; ++j) {
                        const T t = (T)j;
                        sub_node(at(t), profile(fma(t, dx, x_cur), tab) * dzq);
                        stepped(1);
                    }
                } else if constexpr (LONG && !F32) {
                    // x is linear in the sub-step index j, so g_j = e^{-x_j^2} obeys
                    // g_{j+1} = g_j r_j, r_{j+1} = r_j q with r_j = e^{-2 x_j dx - dx^2} and
                    // q = e^{-2 dx^2}.  Values are recomputed exactly whenever x may have
                    // moved by more than 16 widths since the last exact value, so one that
                    // underflowed (|x| > 27) cannot hide a profile above e^{-121}.
                    const float mdx = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, dx_seg), i));
                    const double u2 = 2.0 * dx * dx;
                    const double q = mdx <= 0.5f ? exp_neg_small(u2) : exp_tab64(-u2, tab);
                    double r = exp_tab64(fmin(-(2.0 * x_cur + dx) * dx, 700.0), tab);
                    double Gj = G;
                    Vals w = V;
                    int budget = K;
                    if (mdx > 0.0f) budget = (int)fminf((16.0f - travel) * __builtin_amdgcn_rcpf(mdx), (float)K);
                    if (budget < 1) {
                        Gj = profile(x_cur, tab) * dzq;
                        travel = 0.0f;
                        budget = K;
                    }
                    if (pend > 0) check();
                    int j = 0;
                    for (;;) {
                        const int jend = min(j + budget, m);
                        const int jint = min(jend, m - 1);
                        auto recur = [&] {
                            Gj *= r;
                            r *= q;
#pragma unroll
                            for (int v = 0; v < Vals::kN; ++v) w.v[v] += dV.v[v];
                            sub_node(w, Gj);
                        };
                        int k = j;
                        for (; k + 3 < jint; k += 4) {
                            recur();
                            recur();
                            recur();
                            recur();
                            check();
                        }
                        // the last 0-3 steps in straight-line code
                        if (jint - k >= 2) {
                            recur();
                            recur();
                        }
                        if ((jint - k) & 1) recur();
                        pend = jint - k;
                        travel += mdx * (float)(jint - j);
                        j = jint;
                        if (jend == m) {
                            gn = Gj * r;     // the cell at the end of the segment (times dzq)
                            have_gn = true;
                            travel += mdx;
                            break;
                        }
                        if (pend > 0) check();
                        const double xj = fma((double)j, dx, x_cur);
                        Gj = exp_tab64(-(xj * xj), tab) * dzq;
                        r = exp_tab64(fmin(-(2.0 * xj + dx) * dx, 700.0), tab);
                        w = at((double)j);
                        travel = 0.0f;
                        budget = K;
                    }
                }
            }
            nexec += m;
            // the cell node at the end of the segment
            T G1;
            if (LONG && !F32 && have_gn) {
                G1 = gn;
                g_cur = gn * rcp_refined(dzq);
            } else {
                g_cur = profile(xn, tab);
                G1 = g_cur * dzq;
                travel = 0.0f;
            }
            Vals Vn;
            if (kRows) Vn = node.values(min(i + 2, ns - 1));
            {
                const NodeVals<double, LPL, kRows> Sr = in_fp64<LPL, kRows>(Vr);
                unrolled<LPL>([&](auto l) {
                    const T k = V1.template kap<l>();
                    if constexpr (F32) {
                        const T u = k * g_cur;
                        elim_p<TRACK>((double)(c[l] + u * dzq), Sr.template src<l>(), ls.st[l]);
                        c[l] = u;
                    } else {
                        elim_p<TRACK>(fma(c[l], G, k * G1), Sr.template src<l>(), ls.st[l]);
                        c[l] = k;
                    }
                });
            }
            stepped(1);
            x_cur = xn;
            V = V1;
            if (kRows) V1 = Vn;
            if (TRACK) ls.m_last = m;
        }
    }
}

// All (line, frequency) work of one wave for origin point O and line block w over ray pairs
// p_beg .. p_end - 1, accumulated over them and written to J, L*, Jeff (or, where the point's
// pairs are split over several waves, left per pair in a.part).  Points of models that already
// converged are skipped (their outputs are not needed).
// Lanes: with two groups, group g takes lanes 32 g .. 32 g + n_q - 1 (one frequency each)
// and lines line0 + g LPL ...; with one group, lanes 0..63 take frequencies c 64 + lane of
// chunk c.
// After both half sweeps the lanes write their contributions to J, L* and Jeff of each line to
// LDS rows [3][LPL][64] (in the staged nodes' place), and lane q LPL + l of each group sums row
// (q, l) over the group's frequencies in index order and adds it to its one accumulator (one
// register, not three per line).
template <bool F32, int LPL, bool LONG, bool BAND = false>
__device__ __forceinline__ void solve_item(const SolveArgs &a, int64_t O, int w, int p_beg, int p_end,
                                           double *smem, const double *tab)
{
    using T = typename Bulk<F32>::T;
    using T2 = typename Bulk<F32>::T2;
    using Acc = typename Bulk<F32>::T;
    const int lane = threadIdx.x;
    if (a.model_done != nullptr && a.model_done[a.model_of[O]]) return;
    // lane -> (group, frequency); a wave owns lines line0 .. line0 + nlw - 1
    const int ngrp = a.ngrp;
    const int width = ngrp == 2 ? 32 : kWave;    // lanes per group
    const int line0 = w * a.lines_per_wave;
    const int nlw = min(a.lines_per_wave, a.n_lines - line0);
    const int grp = ngrp == 2 ? lane >> 5 : 0;
    const int sub = lane & (width - 1);           // lane within its group
    const T2 *lc = reinterpret_cast<const T2 *>(a.lc);
    bool lact[LPL];
#pragma unroll
    for (int l = 0; l < LPL; ++l) lact[l] = grp * LPL + l < nlw;
    const int nfq = ngrp == 2 ? a.n_q : min(kWave, a.n_q);   // frequencies of a group (per chunk)
    const int col0 = grp * width;                             // first lane of the group
    // lane col0 + q LPL + l (q < 3) accumulates quantity q (J, L*, Jeff) of line l; with
    // BAND lanes col0 + 3 LPL + q LPL + l (q < 2) accumulate Jb and Ld
    constexpr int kSums = BAND ? 5 : 3;
    Acc acc = 0;
    const int rq = sub / LPL, rl = sub - rq * LPL;   // the row this lane sums
    // LDS: the staged nodes during the sweeps, the rows of contributions after them
    T *rec = reinterpret_cast<T *>(smem);
    auto red = reinterpret_cast<double (*)[LPL][kWave]>(smem);
    LineState<LPL> ls;
    unsigned long long my_exec = 0;   // executed node-frequency steps of this lane
    for (int p = p_beg; p < p_end; ++p) {
        const int r = a.pair_r[p], rb = a.anti[r];
        for (int c = 0; c < a.fchunks; ++c) {
            const int nidx = (a.fchunks == 1) ? sub : c * kWave + lane;
            const bool act = nidx < a.n_q;
            const double xq = act ? a.qx[nidx] : 0.0;
            const double wq = act ? a.qw[nidx] : 0.0;
            // u pairs I(n, x) with I(-n, -x): the antipode sweeps at the mirrored offset
            int64_t nex = 0;
            double Q0[LPL], y0[LPL], H0[LPL];   // the first half's Q, y and last optical-depth step / sqrt 2
            double hdf[LPL], Sf[LPL];
            int mf = 1;
            // the two halves (unrolled: measured faster than one compiled sweep in a loop)
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                half_sweep<F32, LPL, LONG, BAND>(a, rec, tab, O, half ? rb : r, (T)(half ? -xq : xq), grp,
                                                     line0, nlw, ls, nex);
                if (half) break;
                if (BAND) mf = ls.m_last;
#pragma unroll
                for (int l = 0; l < LPL; ++l) {
                    const double id = rcp_refined(ls.st[l].D);
                    Q0[l] = ls.st[l].N * id;
                    y0[l] = ls.st[l].Y * id;
                    H0[l] = ls.st[l].Hm;
                    if (BAND) {
                        hdf[l] = ls.st[l].hd * id;
                        Sf[l] = ls.st[l].Sl;
                    }
                }
            }
            if (a.exec_steps != nullptr && act) {
                int nact = 0;
#pragma unroll
                for (int l = 0; l < LPL; ++l) nact += lact[l] ? 1 : 0;
                my_exec += (unsigned long long)nex * (unsigned long long)nact;
            }
            double vB[LPL], vD[LPL], nbf[LPL], nbb[LPL];
            double vJ[LPL], vL[LPL], vE[LPL];
#pragma unroll
            for (int l = 0; l < LPL; ++l) {
                const int li = grp * LPL + l;
                const double S_O = (double)lc[O * a.n_lines + line0 + (li < nlw ? li : 0)].y;
                const double id = rcp_refined(ls.st[l].D);
                const double h = H0[l] + ls.st[l].Hm;
                const double inv = rcp_refined(h + fma(ls.st[l].N, id, Q0[l]));
                const double yy = fma(ls.st[l].Y, id, y0[l]);
                const bool on = act && lact[l];
                vJ[l] = on ? wq * (fma(h, S_O, yy) * inv) : 0.0;
                vL[l] = on ? wq * (h * inv) : 0.0;
                vE[l] = on ? wq * (yy * inv) : 0.0;
                if (BAND) {
                    // (T^-1)_{O, neighbour} on either side: the neighbour's share of y
                    // over the combine's denominator; a neighbour at fraction 1/m of the
                    // segment toward the first cell interpolates O's own source by 1 - 1/m
                    const double tf = hdf[l] * inv, tb = ls.st[l].hd * id * inv;
                    const double imf = 1.0 / (double)mf, imb = 1.0 / (double)ls.m_last;
                    vB[l] = on ? wq * (yy * inv - tf * Sf[l] - tb * ls.st[l].Sl) : 0.0;
                    vD[l] = on ? wq * (h * inv + (1.0 - imf) * tf + (1.0 - imb) * tb) : 0.0;
                    nbf[l] = on ? wq * tf * imf : 0.0;
                    nbb[l] = on ? wq * tb * imb : 0.0;
                }
            }
            // sums over the group's frequencies
            __syncthreads();
#pragma unroll
            for (int l = 0; l < LPL; ++l) {
                red[0][l][lane] = vJ[l];
                red[1][l][lane] = vL[l];
                red[2][l][lane] = vE[l];
            }
            __syncthreads();
            // (where another wave has the point's other pairs, k_pair_sums adds them in order)
            Acc *part = nullptr;
            if (a.split > 1) {
                const int64_t row = ((O * a.groups + w) * a.n_pairs + p) * a.fchunks + c;
                part = static_cast<Acc *>(a.part) + (row * ngrp + grp) * (kSums * LPL) + sub;
            }
            auto add = [&](Acc sum) {
                if (part != nullptr)
                    *part = sum;
                else
                    acc += sum;
            };
            if (sub < 3 * LPL) {
                Acc sum = 0;
                for (int i = 0; i < nfq; ++i) sum += (Acc)red[rq][rl][col0 + i];
                add(sum);
            }
            if (BAND) {
                __syncthreads();
#pragma unroll
                for (int l = 0; l < LPL; ++l) {
                    red[0][l][lane] = vB[l];
                    red[1][l][lane] = vD[l];
                }
                __syncthreads();
                if (sub >= 3 * LPL && sub < 5 * LPL) {
                    const int q = (sub - 3 * LPL) / LPL, l = sub - 3 * LPL - q * LPL;
                    double sum = 0.0;
                    for (int i = 0; i < nfq; ++i) sum += red[q][l][col0 + i];
                    add((Acc)sum);
                }
                // couplings to the first cells along r and rb, per line summed over this
                // group's frequencies (fixed order)
                __syncthreads();
#pragma unroll
                for (int l = 0; l < LPL; ++l) {
                    red[0][l][lane] = nbf[l];
                    red[1][l][lane] = nbb[l];
                }
                __syncthreads();
                if (sub < 2 * LPL) {
                    const int q = sub / LPL, l = sub - q * LPL;
                    if (lact[l]) {
                        double sum = 0.0;
                        for (int i = 0; i < nfq; ++i) sum += red[q][l][col0 + i];
                        const int64_t o = (O * a.n_lines + line0 + grp * LPL + l) * a.n_rays + (q ? rb : r);
                        if (c == 0)
                            a.Ln[o] = a.norm * sum;
                        else
                            a.Ln[o] += a.norm * sum;
                    }
                }
            }
        }
    }
    if (a.exec_steps != nullptr) {
        for (int o = kWave / 2; o > 0; o >>= 1) my_exec += __shfl_xor(my_exec, o);
        if (lane == 0) atomicAdd(a.exec_steps, my_exec);
    }
    if (a.split > 1) return;
    if (sub < kSums * LPL && rl < LPL) {
        const int q = sub / LPL, l = sub - q * LPL, li = grp * LPL + l;
        if (li < nlw) {
            const int64_t o = O * a.n_lines + line0 + li;
            double *out = q == 0 ? a.J : q == 1 ? a.L : q == 2 ? a.Jeff : q == 3 ? a.Jb : a.Ld;
            out[o] = a.norm * (double)acc;
        }
    }
}

// Dynamic LDS of a formal-solve workgroup: ns staged nodes, or the rows [3][LPL][64] (FP64)
// that take their place.
template <bool F32, int LPL>
constexpr size_t fs_lds_bytes(int ns)
{
    const size_t rows = sizeof(double) * 3 * LPL * kWave;
    const size_t nodes = (size_t)ns * Node<LPL, true>::kStride * sizeof(typename Bulk<F32>::T);
    return rows > nodes ? rows : nodes;
}

// Work items are (point, line block), or with a.split > 1 the split parts of its ray pairs; a
// workgroup takes a.tile consecutive items.  Grid form: points in index order, consecutive
// hardware workgroups go round-robin to the 8 XCDs and each XCD gets a contiguous range of
// origin points, so that the cells their rays share stay in that XCD's L2.  Ordered form
// (a.persistent): points in the order a.order gives (by decreasing cached step count), one
// tile after the next in the order of the workgroups, which the hardware starts as room comes
// free: the longest items start first and the tail is short.  (A fixed grid of workgroups that
// took their items from an atomic counter did the same at a few ns per item and a launch to
// clear the counter: spheres of 12,000 and 60,000 points 413 and 2402 us against 363 and 2340,
// the outflow of 20,011 points 4.94 ms against 4.75, FP32 3.61 against 3.47; only five FP64
// lines per lane, whose workgroups also set up spill space, gained 1% from it.)
// W: waves per SIMD the register budget is built for (up to two FP32 lines need so few that the
// three-wave form is held to four: 3.53 ms for the FP32 outflow against 3.76).
template <bool F32, int LPL, int W, bool LONG>
__global__ __launch_bounds__(64, F32 && LPL <= 2 && W == 3 ? 4 : W) void k_formal_solve(SolveArgs a)
{
    extern __shared__ double fs_smem[];
    __shared__ double tab[64];
    if (!F32) {
        tab[threadIdx.x] = kExp2SixtyFourths[threadIdx.x];
        __syncthreads();
    }
    // (one call site for both forms: the sweep is compiled once)
    const int64_t tile = a.tile;
    const int64_t n_tiles = (a.n_blocks + tile - 1) / tile;
    const int64_t nb8 = (n_tiles + 7) / 8, n_points = a.n_blocks / a.split;   // (times line blocks)
    for (int64_t v = blockIdx.x; v < nb8 * 8; v += gridDim.x) {   // (gridDim.x is a multiple of 8)
        const int64_t first = (a.persistent ? v : (v & 7) * nb8 + (v >> 3)) * tile;
        const int64_t last = first + tile < a.n_blocks ? first + tile : a.n_blocks;
        for (int64_t item = first; item < last; ++item) {
            // part by part: consecutive workgroups, which go to the XCDs in turn, have different
            // points and like costs (the parts of a point side by side gave an XCD the same part
            // of every point where 8 is a multiple of their number: up to twice the time)
            const int part = (int)(item / n_points);
            const int64_t block = item - part * n_points;
            const int64_t rank = block / a.groups;
            const int64_t O = a.persistent ? (int64_t)a.order[rank] : rank;
            solve_item<F32, LPL, LONG>(a, O, (int)(block - rank * a.groups), part * a.n_pairs / a.split,
                                           (part + 1) * a.n_pairs / a.split, fs_smem, tab);
        }
    }
}

// J, L* and Jeff (Q = 5: also Jb and Ld) from the per-pair sums of a split launch, added in the order in which one
// wave would have met the pairs (the same bits).  One thread per (point, line block, lane
// group, sum).
template <bool F32, int LPL, int Q>
__global__ __launch_bounds__(256) void k_pair_sums(SolveArgs a)
{
    using Acc = typename Bulk<F32>::T;
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int slots = a.ngrp * Q * LPL;
    if (t >= a.P * a.groups * slots) return;
    const int64_t block = t / slots;
    const int slot = (int)(t - block * slots);
    const int64_t O = block / a.groups;
    const int w = (int)(block - O * a.groups);
    if (a.model_done != nullptr && a.model_done[a.model_of[O]]) return;
    const int grp = slot / (Q * LPL), q = (slot - grp * Q * LPL) / LPL;
    const int li = grp * LPL + (slot - grp * Q * LPL - q * LPL);
    const int line = w * a.lines_per_wave + li;
    if (li >= a.lines_per_wave || line >= a.n_lines) return;
    const int rows = a.n_pairs * a.fchunks;
    const Acc *part = static_cast<const Acc *>(a.part) + block * rows * slots + slot;
    Acc acc = 0;
#pragma unroll 8
    for (int i = 0; i < rows; ++i) acc += part[(int64_t)i * slots];
    double *out = q == 0 ? a.J : q == 1 ? a.L : q == 2 ? a.Jeff : q == 3 ? a.Jb : a.Ld;
    out[O * a.n_lines + line] = a.norm * (double)acc;
}

template <bool F32, int LPL, int Q>
hipError_t launch_pair_sums(const SolveArgs &a, hipStream_t s)
{
    const int64_t n = a.P * a.groups * a.ngrp * Q * LPL;
    hipLaunchKernelGGL((k_pair_sums<F32, LPL, Q>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

template <bool F32, int LPL, int W, bool LONG>
hipError_t launch_fs_variant(const SolveArgs &a, hipStream_t s)
{
    const size_t lds = fs_lds_bytes<F32, LPL>(a.ns);
    const int64_t n_tiles = (a.n_blocks + a.tile - 1) / a.tile;
    // one workgroup per tile (bounded: a launch counts its threads in 32 bits)
    const unsigned grid = (unsigned)(std::min<int64_t>((n_tiles + 7) / 8, 1 << 22) * 8);
    hipLaunchKernelGGL((k_formal_solve<F32, LPL, W, LONG>), dim3(grid), dim3(kWave), lds, s, a);
    if (a.split > 1) {
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        return launch_pair_sums<F32, LPL, 3>(a, s);
    }
    return hipGetLastError();
}

template <bool F32, int LPL, int W>
hipError_t launch_fs_waves(const SolveArgs &a, hipStream_t s)
{
    if constexpr (fs_has_modes(F32, LPL)) {
        if (a.long_mode) return launch_fs_variant<F32, LPL, W, true>(a, s);
    }
    return launch_fs_variant<F32, LPL, W, false>(a, s);
}

template <bool F32, int LPL>
hipError_t launch_fs_lpl(const SolveArgs &a, hipStream_t s)
{
    if (a.waves == 3) return launch_fs_waves<F32, LPL, 3>(a, s);
    if (a.waves == 1) return launch_fs_waves<F32, LPL, 1>(a, s);
    return launch_fs_waves<F32, LPL, 2>(a, s);
}

template <bool F32>
hipError_t launch_fs_prec(const SolveArgs &a, hipStream_t s)
{
    switch (a.lines_per_wave / a.ngrp) {
    case 1: return launch_fs_lpl<F32, 1>(a, s);
    case 2: return launch_fs_lpl<F32, 2>(a, s);
    case 3: return launch_fs_lpl<F32, 3>(a, s);
    case 4: return launch_fs_lpl<F32, 4>(a, s);
    case 5: return launch_fs_lpl<F32, 5>(a, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace nlte
