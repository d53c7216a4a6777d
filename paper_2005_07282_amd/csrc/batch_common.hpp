// Helpers shared by the batched-solve kernels: the per-system view of the
// concatenated matrix copy and of its dots.
#pragma once

#include "reduce.hpp"
#include "sell_spmv.hpp"

namespace rpcg {

// The sliced-ELL view of system S (local rows and columns).
__device__ __forceinline__ SellMat<double> batch_mat(const BatchArgs &a, const BatchSys &S)
{
    SellMat<double> M;
    M.n = S.n;
    M.nslices = a.ds ? (S.nslices + 1) / 2 : S.nslices;
    M.off = a.off + S.slice0;
    M.val = a.val;
    M.col = a.col;
    M.row_ptr = S.row_ptr;
    M.len8 = a.len8 ? a.len8 + S.row0 : nullptr;
    M.col16 = a.col16;
    M.cfirst = a.cfirst ? a.cfirst + S.slice0 : nullptr;
    M.val64 = nullptr;
    M.ds = a.ds ? a.ds + S.slice0 / 2 : nullptr;
    M.de = a.de;
    return M;
}

// The slices of wavefront `wave` of W in a run (whose bounds are 64-row slices,
// even with diagonal-aligned slices but for a system's end).
template <int LAY>
__device__ __forceinline__ SliceRange batch_slices(const BatchRun &R, int wave, int W)
{
    const int s0 = __builtin_amdgcn_readfirstlane(R.s0), s1 = __builtin_amdgcn_readfirstlane(R.s1);
    if constexpr (LAY == LAY_DIAG) return {s0 / 2 + wave, (s1 + 1) / 2, W};
    else return {s0 + wave, s1, W};
}

// Dot d of system S, and the copies of its accumulators (uniform).
__device__ __forceinline__ int batch_dot_copies(const BatchSys &S) { return __builtin_amdgcn_readfirstlane((int)S.copies); }
__device__ __forceinline__ DotWs batch_dot(const BatchArgs &a, const BatchSys &S, int d)
{
    DotWs w{};
    w.acc = a.acc + S.acc0 + (long long)d * batch_dot_copies(S) * DOT_PITCH;
    w.part = a.part + (long long)d * a.part_cap + S.slot0;
    return w;
}

} // namespace rpcg
