// Jacobi-PCG iteration, second and third kernels.
//
// K2 starts by merging the SpMV kernel's partials of <d, w> (every workgroup
// alike) into delta and rho = beta / delta (S2), then applies the residual
// update and the Jacobi preconditioner (S4, S5) and forms the partials of
// beta = <z, r> and tau = <r, r> (S6, S8).
// K3 starts by merging those into beta, tau and gamma = beta / beta_old, runs
// the stopping test of Fig. 1, and updates the iterate (S3, with the rho of
// K2) and, unless the solve stops, the search direction (S7). S3 sits in K3
// because K3 loads d anyway: K2 then reads neither d nor x.
//
// The iteration number l is a launch argument, so the beta and tau histories
// one kernel writes for later iterations are never read by another
// workgroup of the same kernel. A workgroup of K3 that starts after the
// first one has run the stopping test must still apply the iteration's S3:
// it returns early only when the solve ended before this iteration's S3 was
// owed (PcgState::ended <= l), which the stopping test of the same launch
// never sets.
#include "reduce.hpp"
#include "sell_spmv.hpp"

namespace rpcg {

// What a workgroup's first wavefronts read and merge at the start, handed to
// every thread through LDS. All loads of the kernel's head (state, both accumulators,
// the first elements) are issued before any of them is waited for.
template <int MODE, int P, typename T>
__global__ void __launch_bounds__(MAX_BLOCK)
k_pcg_update(int l, int n, PcgVecs<T> v, PcgState *st, DotWs wd, int Gd, DotWs wb, DotWs wt, bool ee, bool capture)
{
    __shared__ RedShared sh;
    // software-pipelined grid-stride loop: the operands of the thread's next
    // element are loaded before the current one is computed, so the loads
    // are in flight while the two exact dots of the current element run (the
    // first ones while delta is merged)
    const long long stride = (long long)gridDim.x * blockDim.x;
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    T wn = T(0), rn = T(0), qn = T(0);
    if (i < n) { wn = v.w[i]; rn = v.r[i]; qn = v.dinv[i]; }
    const T beta = (T)v.beta_hist[l];
    if (wave_id() == 0) {
        const int done = coherent_int(&st->done), flags = coherent_int(&st->flags);
        long long esc;
        const T d = wave_merge<MODE, T>(wd, Gd, &esc);
        if (lane_id() == 0) {
            sh.flag = done;
            sh.rng[0] = flags;
            sh.val[0] = d;
            sh.red_ll[0] = esc;
        }
    }
    zero_acc(sh.acc[0]);
    zero_acc(sh.acc[1]);
    __syncthreads();
    if (sh.flag) return;
    // S2: delta = <d, w> rounded once; rho = beta_l / delta
    const T delta = (T)sh.val[0];
    const bool bad = (sh.rng[0] & FLAG_NONFINITE) || !is_finite_bits((double)delta);
    const bool breakdown = !(delta > T(0));
    const T rho = beta / delta;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const long long esc_d = sh.red_ll[0];
        if (esc_d) st->escapes += esc_d;
        if (capture && esc_d > 0) st->fallbacks += 1;
        st->delta = delta;
        if (bad) { st->status = -6; st->done = 1; st->ended = l; }
        else if (breakdown) { st->status = -5; st->done = 1; st->ended = l; }
        else st->rho = rho;
    }
    if (bad || breakdown) return;
    LaneDot<MODE, P> Lb, Lt;
    Lb.init();
    Lt.init();
    for (; i < n; i += stride) {
        const T wi = wn, r0 = rn, qi = qn;
        const long long inext = i + stride;
        if (inext < n) { wn = v.w[inext]; rn = v.r[inext]; qn = v.dinv[inext]; }
        const T ri = fma_t(-rho, wi, r0);                 // S4
        const T zi = qi * ri;                             // S5
        v.r[i] = ri;
        v.z[i] = zi;
        Lb.add(zi, ri, sh.acc[0], ee, capture);           // S6
        Lt.add(ri, ri, sh.acc[1], ee, capture);           // S8
    }
    block_publish<MODE, P, 2, false>({&Lb, &Lt}, {sh.acc[0], sh.acc[1]}, {&wb, &wt}, blockIdx.x, ee, capture, &st->flags, sh);
}

// Elements per thread whose operands K3 loads before merging the dots, so
// the loads are in flight while the merge runs.
constexpr int DIR_PREFETCH = 8;

// S3: with S3 set (the Jacobi solver) this kernel also applies the iterate
// update x = fma(rho, d, x) of iteration l; the factored solver's update
// kernel applies it itself.
template <int MODE, typename T, bool S3>
__global__ void __launch_bounds__(MAX_BLOCK)
k_pcg_direction(int l, int n, PcgVecs<T> v, PcgState *st, DotWs wb, DotWs wt, DotWs wd, int G, bool capture)
{
    __shared__ RedShared sh;
    const long long i0 = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long stride = (long long)gridDim.x * blockDim.x;
    T dv[DIR_PREFETCH], zv[DIR_PREFETCH], xv[DIR_PREFETCH];
#pragma unroll
    for (int j = 0; j < DIR_PREFETCH; ++j) {
        const long long i = i0 + j * stride;
        dv[j] = i < n ? v.d[i] : T(0);
        zv[j] = i < n ? v.z[i] : T(0);
        if constexpr (S3) xv[j] = i < n ? v.x[i] : T(0);
    }
    const T beta_old = (T)v.beta_hist[l];
    const T rho = (T)st->rho; // K2's rho of iteration l
    const double thr = st->thr;
    const int maxit = st->maxit;
    // beta by the first wavefront, tau by the second (by the first when it is alone)
    const int wv = wave_id();
    if (wv == 0) {
        // the first iteration whose S3 is not owed, or whether the solve has ended
        const int ended = S3 ? coherent_int(&st->ended) <= l : coherent_int(&st->done);
        const int flags = coherent_int(&st->flags);
        long long esc;
        const T b = wave_merge<MODE, T>(wb, G, &esc);
        if (lane_id() == 0) {
            sh.flag = ended;
            sh.rng[0] = flags;
            sh.val[0] = b;
            sh.red_ll[0] = esc;
        }
    }
    if (wv == (num_waves() > 1 ? 1 : 0)) {
        long long esc;
        const T t = wave_merge<MODE, T>(wt, G, &esc);
        if (lane_id() == 0) {
            sh.val[1] = t;
            sh.red_ll[1] = esc;
        }
    }
    __syncthreads();
    if (sh.flag) return;
    const T beta = (T)sh.val[0], tau = (T)sh.val[1];
    const bool bad = (sh.rng[0] & FLAG_NONFINITE) || !is_finite_bits((double)beta) || !is_finite_bits((double)tau);
    const int it = l + 1;
    const bool stop = bad || (double)tau <= thr || it >= maxit;
    const T gamma = beta / beta_old;
    if (MODE != MODE_PLAIN && blockIdx.x == 0) clear_dot(wd); // K2 has read it
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const long long eb = sh.red_ll[0], et = sh.red_ll[1];
        if (eb + et) st->escapes += eb + et;
        if (capture && eb + et) st->fallbacks += (eb > 0) + (et > 0);
        if (bad) {
            st->status = -6;
        } else {
            v.beta_hist[it] = beta;
            st->beta = beta;
            st->tau = tau;
            st->iter = it;
            if (v.hist) v.hist[it] = tau;
        }
        if (stop) {
            st->done = 1;
            if constexpr (S3) st->ended = it;
        } else {
            st->gamma = gamma;
        }
    }
    if (!S3 && stop) return;
#pragma unroll
    for (int j = 0; j < DIR_PREFETCH; ++j) {
        const long long i = i0 + j * stride;
        if (i < n) {
            if constexpr (S3) v.x[i] = fma_t(rho, dv[j], xv[j]);   // S3
            if (!stop) v.d[i] = fma_t(gamma, dv[j], zv[j]);        // S7
        }
    }
    for (long long i = i0 + DIR_PREFETCH * stride; i < n; i += stride) {
        const T di = v.d[i];
        if constexpr (S3) v.x[i] = fma_t(rho, di, v.x[i]);
        if (!stop) v.d[i] = fma_t(gamma, di, v.z[i]);
    }
}

template <typename T>
hipError_t launch_pcg_update(int mode, int l, int n, const PcgVecs<T> &v, PcgState *st, const DotWs *ws3, int Gd,
                             const LaunchCfg &c)
{
    dispatch(mode, c.fpe_size, [&](auto m, auto p) {
        constexpr int M = decltype(m)::value, PP = decltype(p)::value;
        k_pcg_update<M, PP, T><<<c.grid, c.block, 0, c.stream>>>(l, n, v, st, ws3[0], Gd, ws3[1], ws3[2], c.early_exit,
                                                                 c.fallback);
    });
    return hipGetLastError();
}

template <typename T>
hipError_t launch_pcg_direction(int mode, int l, int n, const PcgVecs<T> &v, PcgState *st, const DotWs *ws3, int G,
                                const LaunchCfg &c, bool s3)
{
    dispatch_mode(mode, [&](auto m) {
        constexpr int M = decltype(m)::value;
        if (s3) k_pcg_direction<M, T, true><<<c.grid, c.block, 0, c.stream>>>(l, n, v, st, ws3[1], ws3[2], ws3[0], G, c.fallback);
        else k_pcg_direction<M, T, false><<<c.grid, c.block, 0, c.stream>>>(l, n, v, st, ws3[1], ws3[2], ws3[0], G, c.fallback);
    });
    return hipGetLastError();
}

// Built once per value type (the library compiles this file with
// -DRPCG_VALUE_TYPE=double and with -DRPCG_VALUE_TYPE=float).
#ifndef RPCG_VALUE_TYPE
#error "define RPCG_VALUE_TYPE (double or float)"
#endif
template hipError_t launch_pcg_update<RPCG_VALUE_TYPE>(int, int, int, const PcgVecs<RPCG_VALUE_TYPE> &, PcgState *, const DotWs *,
                                              int, const LaunchCfg &);
template hipError_t launch_pcg_direction<RPCG_VALUE_TYPE>(int, int, int, const PcgVecs<RPCG_VALUE_TYPE> &, PcgState *,
                                                 const DotWs *, int, const LaunchCfg &, bool);

} // namespace rpcg
