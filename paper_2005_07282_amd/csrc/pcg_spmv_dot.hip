// Jacobi-PCG iteration, first kernel: SpMV fused with the first dot (S1, S2),
// for binary64 (T = double) and the binary32 inner solver (T = float).
#include "reduce.hpp"
#include "sell_spmv.hpp"

namespace rpcg {

// K1: w = A d (S1; Section 4.3: per row a sequential fma chain in storage
// order from +0) and the workgroup partial of <d, w> (S2).
// Wavefront -> slice mapping: see wave_slices.
template <int MODE, int P, int LAY, typename T>
__global__ void __launch_bounds__(MAX_BLOCK)
k_pcg_spmv_dot(SellMat<T> A, PcgVecs<T> v, PcgState *st, DotWs wd, DotWs wb, DotWs wt, bool ee, bool capture,
               int xcd_parts)
{
    __shared__ RedShared sh;
    if (st->done) return;
    long long *acc = sh.acc[0];
    zero_acc(acc);
    if (MODE != MODE_PLAIN && blockIdx.x == 0) { // the direction kernel has read them
        clear_dot(wb);
        clear_dot(wt);
    }
    __syncthreads();
    LaneDot<MODE, P> L;
    L.init();
    const int lane = lane_id();
    const T *__restrict__ d = v.d;
    for_slices<T, LAY, false>(A, wave_slices(A.nslices, xcd_parts), lane, [&](long long i, auto &&rows) {
        constexpr int R = lane_rows<LAY>();
        T sum[R], di[R];
        rows(d, sum, nullptr, nullptr);
        load_rows<R>(di, d, i, A.n);
        store_rows(v.w, sum, i, A.n);
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (i + r < A.n) L.add(di[r], sum[r], acc, ee, capture);
    });
    block_publish<MODE, P, 1, false>({&L}, {acc}, {&wd}, blockIdx.x, ee, capture, &st->flags, sh);
}

template <typename T>
hipError_t launch_pcg_spmv_dot(int mode, const SellMat<T> &A, const PcgVecs<T> &v, PcgState *st,
                               const DotWs *ws3, const LaunchCfg &c)
{
    const int want = c.xcd_parts ? c.xcd_parts : (A.ds ? NUM_XCDS : 1);
    const int parts = c.grid >= 64 ? want : 1;
    dispatch(mode, c.fpe_size, [&](auto m, auto p) {
        constexpr int M = decltype(m)::value, PP = decltype(p)::value;
        dispatch_layout(A.layout(), [&](auto lay) {
            k_pcg_spmv_dot<M, PP, decltype(lay)::value, T><<<c.grid, c.block, 0, c.stream>>>(A, v, st, ws3[0], ws3[1], ws3[2],
                                                                                             c.early_exit, c.fallback, parts);
        });
    });
    return hipGetLastError();
}

// Built once per value type (the library compiles this file with
// -DRPCG_VALUE_TYPE=double and with -DRPCG_VALUE_TYPE=float).
#ifndef RPCG_VALUE_TYPE
#error "define RPCG_VALUE_TYPE (double or float)"
#endif
template hipError_t launch_pcg_spmv_dot<RPCG_VALUE_TYPE>(int, const SellMat<RPCG_VALUE_TYPE> &, const PcgVecs<RPCG_VALUE_TYPE> &, PcgState *,
                                                const DotWs *, const LaunchCfg &);

} // namespace rpcg
