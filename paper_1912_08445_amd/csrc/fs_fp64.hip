// FP64 formal-solve kernels: the line solve in every launch shape (formal_solve_kernels.h)
// and its band-operator variant.
#include "formal_solve_kernels.h"

namespace nlte {

hipError_t launch_formal_solve_f64(const SolveArgs &a, hipStream_t s)
{
    return launch_fs_prec<false>(a, s);
}

size_t formal_solve_lds_f64(int lpl, int ns)
{
    switch (lpl) {
    case 1: return fs_lds_bytes<false, 1>(ns);
    case 2: return fs_lds_bytes<false, 2>(ns);
    case 3: return fs_lds_bytes<false, 3>(ns);
    case 4: return fs_lds_bytes<false, 4>(ns);
    default: return fs_lds_bytes<false, 5>(ns);
    }
}

// Band-operator variant of the grid kernel: also the entries of the inverse system matrix
// between O and its neighbour nodes (Jb, Ld, Ln of SolveArgs), from the last step of each half
// sweep (the segment that ends at O is never crossed as a far-wing one).  LONG: the long-segment
// mode.
template <int LPL, bool LONG>
__global__ __launch_bounds__(64, 2) void k_formal_solve_band(SolveArgs a)
{
    extern __shared__ double fs_smem[];
    __shared__ double tab[64];
    tab[threadIdx.x] = kExp2SixtyFourths[threadIdx.x];
    __syncthreads();
    if (a.split > 1) {   // the parts of a point's pairs, points in decreasing cost (see k_formal_solve)
        if (blockIdx.x >= a.n_blocks) return;
        const int64_t n_points = a.n_blocks / a.split;
        const int part = (int)(blockIdx.x / n_points);
        const int64_t block = blockIdx.x - part * n_points, rank = block / a.groups;
        solve_item<false, LPL, LONG, true>(a, a.order[rank], (int)(block - rank * a.groups), part * a.n_pairs / a.split,
                                           (part + 1) * a.n_pairs / a.split, fs_smem, tab);
        return;
    }
    const int64_t nb8 = (a.n_blocks + 7) / 8;
    const int64_t lb = (int64_t)(blockIdx.x & 7) * nb8 + (blockIdx.x >> 3);
    if (lb >= a.n_blocks) return;
    const int64_t O = lb / a.groups;
    solve_item<false, LPL, LONG, true>(a, O, (int)(lb - O * a.groups), 0, a.n_pairs, fs_smem, tab);
}

hipError_t launch_formal_solve_band(const SolveArgs &a, hipStream_t s)
{
    if (a.n_blocks == 0) return hipSuccess;
    const int lpl = a.lines_per_wave / a.ngrp;
    const int64_t nb8 = (a.n_blocks + 7) / 8;
    const dim3 grid((unsigned)(nb8 * 8));
    if (lpl == 1 && a.long_mode)
        hipLaunchKernelGGL((k_formal_solve_band<1, true>), grid, dim3(kWave), (fs_lds_bytes<false, 1>(a.ns)), s, a);
    else if (lpl == 1)
        hipLaunchKernelGGL((k_formal_solve_band<1, false>), grid, dim3(kWave), (fs_lds_bytes<false, 1>(a.ns)), s, a);
    else if (lpl == 2 && a.long_mode)
        hipLaunchKernelGGL((k_formal_solve_band<2, true>), grid, dim3(kWave), (fs_lds_bytes<false, 2>(a.ns)), s, a);
    else if (lpl == 2)
        hipLaunchKernelGGL((k_formal_solve_band<2, false>), grid, dim3(kWave), (fs_lds_bytes<false, 2>(a.ns)), s, a);
    else
        return hipErrorInvalidValue;
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.split <= 1) return e;
    return lpl == 1 ? launch_pair_sums<false, 1, 5>(a, s) : launch_pair_sums<false, 2, 5>(a, s);
}

}  // namespace nlte
