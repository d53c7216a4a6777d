// Jacobi-PCG setup kernels: preconditioner, initial residual and dots
// (Fig. 1/Fig. 2 initialisation; Section 4.3 Jacobi: inverse diagonal once).
// T = double is the paper's solver; T = float the binary32 inner solver of
// the mixed-precision refinement (same steps, every rounding in binary32).
#include "reduce.hpp"
#include "sell_spmv.hpp"

namespace rpcg {

// The setup runs once per solve: its three block partials go through
// out-of-line calls, which keeps the number of inlined copies (and the
// compile time over all mode and length variants) down.
template <int MODE, int P>
__device__ __noinline__ void setup_publish(LaneDot<MODE, P> &L, long long *acc, const DotWs &w, bool ee, bool capture,
                                           int *gflags, RedShared &sh)
{
    block_publish<MODE, P, 1, false>({&L}, {acc}, {&w}, blockIdx.x, ee, capture, gflags, sh);
}

// State of a new solve; the dots' accumulators emptied (one workgroup).
static __global__ void k_state_init(PcgState *st, int maxit, DotWs w0, DotWs w1, DotWs w2)
{
    clear_dot(w0);
    clear_dot(w1);
    clear_dot(w2);
    if (threadIdx.x != 0) return;
    PcgState z = {};
    z.maxit = maxit;
    z.ended = 0x7FFFFFFF;
    *st = z;
}

// dinv = RN(1/a_ii), r = RN(b - A x0), z = RN(dinv r), d = z, and the
// workgroup partials of <z,r>, <r,r>, <b,b>. One wavefront per slice of the
// matrix copy, as in the iteration's SpMV.
template <int MODE, int P, int LAY, typename T>
__global__ void __launch_bounds__(MAX_BLOCK)
k_pcg_setup(SellMat<T> A, PcgVecs<T> v, PcgState *st, DotWs w0, DotWs w1, DotWs w2, bool ee, bool capture)
{
    __shared__ RedShared sh;
    zero_acc(sh.acc[0]); zero_acc(sh.acc[1]); zero_acc(sh.acc[2]);
    __syncthreads();
    LaneDot<MODE, P> Lb, Lt, Lbb;
    Lb.init(); Lt.init(); Lbb.init();
    int flags = 0;
    const int lane = lane_id();
    for_slices<T, LAY, true>(A, wave_slices(A.nslices, 1), lane, [&](long long i, auto &&rows) {
        constexpr int R = lane_rows<LAY>();
        T acc[R], aii[R], bi[R], xi[R], di[R], ri[R], zi[R];
        bool found[R];
#pragma unroll
        for (int r = 0; r < R; ++r) { aii[r] = T(0); found[r] = false; }
        rows(v.x, acc, aii, found);
        load_rows<R>(bi, v.b, i, A.n);
        load_rows<R>(xi, v.x, i, A.n);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            di[r] = T(1) / aii[r];
            ri[r] = bi[r] - acc[r];
            zi[r] = di[r] * ri[r];
            if (i + r < A.n) {
                if (!found[r] || !(aii[r] > T(0))) flags |= FLAG_NOT_SPD;
                if (!is_finite_bits((double)bi[r]) || !is_finite_bits((double)xi[r])) flags |= FLAG_NONFINITE;
                Lb.add(zi[r], ri[r], sh.acc[0], ee, capture);
                Lt.add(ri[r], ri[r], sh.acc[1], ee, capture);
                Lbb.add(bi[r], bi[r], sh.acc[2], ee, capture);
            }
        }
        store_rows(v.dinv, di, i, A.n);
        store_rows(v.r, ri, i, A.n);
        store_rows(v.z, zi, i, A.n);
        store_rows(v.d, zi, i, A.n);
    });
    if (flags) atomicOr(&st->flags, flags);
    setup_publish<MODE, P>(Lb, sh.acc[0], w0, ee, capture, &st->flags, sh);
    setup_publish<MODE, P>(Lt, sh.acc[1], w1, ee, capture, &st->flags, sh);
    setup_publish<MODE, P>(Lbb, sh.acc[2], w2, ee, capture, &st->flags, sh);
}

// One workgroup of FIN_BLOCK threads, a dot per wavefront: beta0, tau0, <b,b>; thr = RN(RN(tol*tol)
// <b,b>) in T with tol rounded to T; stopping test. Leaves the accumulators empty.
constexpr int FIN_BLOCK = 256;
template <int MODE, typename T>
__global__ void __launch_bounds__(FIN_BLOCK)
k_pcg_fin_setup(int G, PcgVecs<T> v, PcgState *st, DotWs w0, DotWs w1, DotWs w2, double tol, bool capture)
{
    __shared__ RedShared sh;
    const int wv = wave_id();
    if (wv < 3) {
        long long esc;
        const T d = wave_merge<MODE, T>(wv == 0 ? w0 : (wv == 1 ? w1 : w2), G, &esc);
        if (lane_id() == 0) {
            sh.val[wv] = d;
            sh.red_ll[wv] = esc;
        }
    }
    __syncthreads();
    if (MODE != MODE_PLAIN) {
        clear_dot(w0);
        clear_dot(w1);
        clear_dot(w2);
    }
    const T beta = (T)sh.val[0], tau = (T)sh.val[1], bb = (T)sh.val[2];
    const long long e0 = sh.red_ll[0], e1 = sh.red_ll[1], e2 = sh.red_ll[2];
    if (threadIdx.x == 0) {
        st->escapes += e0 + e1 + e2;
        if (capture) st->fallbacks += (e0 > 0) + (e1 > 0) + (e2 > 0);
        int f = st->flags;
        v.beta_hist[0] = beta;
        st->beta = beta;
        st->tau = tau;
        st->tau0 = tau;
        st->bb = bb;
        const T tolt = (T)tol;
        const T thr = (tolt * tolt) * bb;
        st->thr = thr;
        if (v.hist) v.hist[0] = tau;
        st->iter = 0;
        if (f & FLAG_NOT_SPD) { st->status = -4; st->done = 1; }
        else if ((f & FLAG_NONFINITE) || !is_finite_bits((double)tau) || !is_finite_bits((double)bb)) {
            st->status = -6;
            st->done = 1;
        } else st->done = (tau <= thr || st->maxit <= 0) ? 1 : 0;
        if (st->done) st->ended = 0;
    }
}

template <typename T>
hipError_t launch_pcg_setup(int mode, const SellMat<T> &A, const PcgVecs<T> &v, PcgState *st, const DotWs *ws3,
                            double tol, int maxit, const LaunchCfg &c)
{
    hipLaunchKernelGGL(k_state_init, dim3(1), dim3(256), 0, c.stream, st, maxit, ws3[0], ws3[1], ws3[2]);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    dispatch(mode, c.fpe_size, [&](auto m, auto p) {
        constexpr int M = decltype(m)::value, PP = decltype(p)::value;
        dispatch_layout(A.layout(), [&](auto lay) {
            k_pcg_setup<M, PP, decltype(lay)::value, T><<<c.grid, c.block, 0, c.stream>>>(A, v, st, ws3[0], ws3[1], ws3[2],
                                                                                          c.early_exit, c.fallback);
        });
        k_pcg_fin_setup<M, T><<<1, FIN_BLOCK, 0, c.stream>>>(c.grid, v, st, ws3[0], ws3[1], ws3[2], tol, c.fallback);
    });
    return hipGetLastError();
}

// Built once per value type (the library compiles this file with
// -DRPCG_VALUE_TYPE=double and with -DRPCG_VALUE_TYPE=float).
#ifndef RPCG_VALUE_TYPE
#error "define RPCG_VALUE_TYPE (double or float)"
#endif
template hipError_t launch_pcg_setup<RPCG_VALUE_TYPE>(int, const SellMat<RPCG_VALUE_TYPE> &, const PcgVecs<RPCG_VALUE_TYPE> &, PcgState *,
                                             const DotWs *, double, int, const LaunchCfg &);

} // namespace rpcg
