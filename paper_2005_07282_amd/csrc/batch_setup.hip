// Batched Jacobi-PCG setup (Fig. 1 initialisation, Section 4.3 Jacobi) of
// every system of a batch: state, then dinv, r, z, d and the partials of
// <z,r>, <r,r>, <b,b> per run, then one workgroup per system to merge them.
#include "batch_common.hpp"

namespace rpcg {

// State of every system; its dots emptied (one workgroup per system).
__global__ void __launch_bounds__(256) k_batch_state_init(BatchArgs a, int maxit)
{
    const int sys = blockIdx.x;
    const BatchSys S = a.sys[sys];
    for (int d = 0; d < 3; ++d) clear_dot(batch_dot(a, S, d), batch_dot_copies(S));
    if (threadIdx.x != 0) return;
    if (sys == 0) *a.active = a.nsys;
    PcgState z = {};
    z.maxit = maxit;
    z.ended = 0x7FFFFFFF;
    a.st[sys] = z;
}

// The setup runs once per solve: its block partials go through an
// out-of-line call, which keeps the inlined copies (and compile time) down.
template <int MODE, int P>
__device__ __noinline__ void batch_setup_publish(LaneDot<MODE, P> &L, long long *acc, const DotWs &w, int g, bool ee,
                                                 bool capture, int *gflags, RedShared &sh, int copies)
{
    block_publish<MODE, P, 1, false>({&L}, {acc}, {&w}, g, ee, capture, gflags, sh, copies);
}

template <int MODE, int P, int LAY>
__global__ void __launch_bounds__(MAX_BLOCK)
k_batch_setup(BatchArgs a, bool ee, bool capture)
{
    __shared__ RedShared sh;
    const int lane = lane_id();
    const int W = num_waves();
    const int wave = __builtin_amdgcn_readfirstlane(wave_id());
    for (int ri = a.wg_run[blockIdx.x]; ri < a.wg_run[blockIdx.x + 1]; ++ri) {
        const BatchRun R = a.runs[ri];
        const BatchSys S = a.sys[R.sys];
        const SellMat<double> M = batch_mat(a, S);
        const long long r0 = S.row0;
        __syncthreads();
        zero_acc(sh.acc[0]);
        zero_acc(sh.acc[1]);
        zero_acc(sh.acc[2]);
        __syncthreads();
        LaneDot<MODE, P> Lb, Lt, Lbb;
        Lb.init();
        Lt.init();
        Lbb.init();
        int flags = 0;
        for_slices<double, LAY, true>(M, batch_slices<LAY>(R, wave, W), lane, [&](long long i, auto &&rows) {
            constexpr int NR = lane_rows<LAY>();
            double acc[NR], aii[NR], bi[NR], xi[NR], di[NR], ri[NR], zi[NR];
            bool found[NR];
#pragma unroll
            for (int r = 0; r < NR; ++r) { aii[r] = 0.0; found[r] = false; }
            rows(a.x + r0, acc, aii, found);
            load_rows<NR>(bi, a.b + r0, i, M.n);
            load_rows<NR>(xi, (const double *)a.x + r0, i, M.n);
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                di[r] = 1.0 / aii[r];
                ri[r] = bi[r] - acc[r];
                zi[r] = di[r] * ri[r];
                if (i + r < M.n) {
                    if (!found[r] || !(aii[r] > 0.0)) flags |= FLAG_NOT_SPD;
                    if (!is_finite_bits(bi[r]) || !is_finite_bits(xi[r])) flags |= FLAG_NONFINITE;
                    Lb.add(zi[r], ri[r], sh.acc[0], ee, capture);
                    Lt.add(ri[r], ri[r], sh.acc[1], ee, capture);
                    Lbb.add(bi[r], bi[r], sh.acc[2], ee, capture);
                }
            }
            store_rows(a.dinv + r0, di, i, M.n);
            store_rows(a.r + r0, ri, i, M.n);
            store_rows(a.z + r0, zi, i, M.n);
            store_rows(a.d + r0, zi, i, M.n);
        });
        if (flags) atomicOr(&a.st[R.sys].flags, flags);
        int *gf = &a.st[R.sys].flags;
        const int g = R.slot - S.slot0, copies = batch_dot_copies(S);
        batch_setup_publish<MODE, P>(Lb, sh.acc[0], batch_dot(a, S, 0), g, ee, capture, gf, sh, copies);
        batch_setup_publish<MODE, P>(Lt, sh.acc[1], batch_dot(a, S, 1), g, ee, capture, gf, sh, copies);
        batch_setup_publish<MODE, P>(Lbb, sh.acc[2], batch_dot(a, S, 2), g, ee, capture, gf, sh, copies);
    }
}

// One workgroup per system, a dot per wavefront: beta0, tau0, <b,b>, thr =
// RN(RN(tol*tol) <b,b>), stopping test. Leaves the dots empty.
template <int MODE>
__global__ void __launch_bounds__(256) k_batch_fin_setup(BatchArgs a, double tol, bool capture)
{
    __shared__ RedShared sh;
    const int sys = blockIdx.x;
    PcgState *st = a.st + sys;
    const BatchSys S = a.sys[sys];
    const int wv = wave_id();
    if (wv < 3) {
        long long esc;
        const double d = wave_merge<MODE>(batch_dot(a, S, wv), S.slot1 - S.slot0, &esc, batch_dot_copies(S));
        if (lane_id() == 0) {
            sh.val[wv] = d;
            sh.red_ll[wv] = esc;
        }
    }
    __syncthreads();
    for (int d = 0; d < 3; ++d) clear_dot(batch_dot(a, S, d), batch_dot_copies(S));
    const double beta = sh.val[0], tau = sh.val[1], bb = sh.val[2];
    const long long e0 = sh.red_ll[0], e1 = sh.red_ll[1], e2 = sh.red_ll[2];
    if (threadIdx.x == 0) {
        st->escapes += e0 + e1 + e2;
        if (capture) st->fallbacks += (e0 > 0) + (e1 > 0) + (e2 > 0);
        const int f = coherent_int(&st->flags);
        st->beta = beta;
        st->beta_par[0] = beta;
        st->tau = tau;
        st->tau0 = tau;
        st->bb = bb;
        const double thr = (tol * tol) * bb;
        st->thr = thr;
        if (a.hist && a.hist[sys]) a.hist[sys][0] = tau;
        st->iter = 0;
        st->it_cur = 0;
        int done;
        if (f & FLAG_NOT_SPD) { st->status = -4; done = 1; }
        else if ((f & FLAG_NONFINITE) || !is_finite_bits(tau) || !is_finite_bits(bb)) { st->status = -6; done = 1; }
        else done = (tau <= thr || st->maxit <= 0) ? 1 : 0;
        st->done = done;
        if (done) {
            st->ended = 0;
            atomicSub(a.active, 1);
        }
    }
}

hipError_t launch_batch_setup(int mode, int layout, const BatchArgs &a, int grid, int block, double tol, int maxit,
                              const LaunchCfg &c)
{
    k_batch_state_init<<<a.nsys, 256, 0, c.stream>>>(a, maxit);
    dispatch(mode, c.fpe_size, [&](auto m, auto p) {
        constexpr int M = decltype(m)::value, PP = decltype(p)::value;
        dispatch_layout(layout, [&](auto lay) {
            k_batch_setup<M, PP, decltype(lay)::value><<<grid, block, 0, c.stream>>>(a, c.early_exit, c.fallback);
        });
        k_batch_fin_setup<M><<<a.nsys, 256, 0, c.stream>>>(a, tol, c.fallback);
    });
    return hipGetLastError();
}

} // namespace rpcg
