// Setup of the PCG with a factored preconditioner M^-1 = G G^T + eps I
// (Fig. 1 initialisation with the preconditioner step t = G^T r,
// z = G t + eps r). Runs once per solve: its partials and merges go through
// out-of-line calls, which keeps compile time down.
#include "pcg_factored.hpp"

namespace rpcg {

template <int MODE, int P>
__device__ __noinline__ void fac_publish(LaneDot<MODE, P> &L, long long *acc, const DotWs &w, bool ee, bool capture,
                                         int *gflags, RedShared &sh)
{
    block_publish<MODE, P, 1, false>({&L}, {acc}, {&w}, blockIdx.x, ee, capture, gflags, sh);
}

static __global__ void k_fac_state_init(PcgState *st, int maxit, DotWs w0, DotWs w1, DotWs w2)
{
    clear_dot(w0);
    clear_dot(w1);
    clear_dot(w2);
    if (threadIdx.x != 0) return;
    PcgState z = {};
    z.maxit = maxit;
    *st = z;
}

// r = b - A x0 over the sliced-ELL copy; partials of <r,r> and <b,b>.
template <int MODE, int P, int LAY>
__global__ void __launch_bounds__(MAX_BLOCK)
k_fac_setup_r(SellMat<double> A, PcgVecs<double> v, PcgState *st, DotWs wt, DotWs wbb, bool ee, bool capture)
{
    __shared__ RedShared sh;
    zero_acc(sh.acc[1]);
    zero_acc(sh.acc[2]);
    __syncthreads();
    LaneDot<MODE, P> Lt, Lbb;
    Lt.init();
    Lbb.init();
    int flags = 0;
    const int lane = lane_id();
    for_slices<double, LAY, false>(A, wave_slices(A.nslices, 1), lane, [&](long long i, auto &&rows) {
        constexpr int R = lane_rows<LAY>();
        double acc[R], bi[R], xi[R], ri[R];
        rows(v.x, acc, nullptr, nullptr);
        load_rows<R>(bi, v.b, i, A.n);
        load_rows<R>(xi, v.x, i, A.n);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            ri[r] = bi[r] - acc[r];
            if (i + r < A.n) {
                if (!is_finite_bits(bi[r]) || !is_finite_bits(xi[r])) flags |= FLAG_NONFINITE;
                Lt.add(ri[r], ri[r], sh.acc[1], ee, capture);
                Lbb.add(bi[r], bi[r], sh.acc[2], ee, capture);
            }
        }
        store_rows(v.r, ri, i, A.n);
    });
    if (flags) atomicOr(&st->flags, flags);
    fac_publish<MODE, P>(Lt, sh.acc[1], wt, ee, capture, &st->flags, sh);
    fac_publish<MODE, P>(Lbb, sh.acc[2], wbb, ee, capture, &st->flags, sh);
}

// One workgroup of FIN_BLOCK threads, a dot per wavefront: beta0, tau0, <b,b>,
// threshold, stopping test. Leaves the accumulators empty.
constexpr int FIN_BLOCK = 256;
template <int MODE>
__global__ void __launch_bounds__(FIN_BLOCK)
k_fac_fin_setup(int G, PcgVecs<double> v, PcgState *st, DotWs w0, DotWs w1, DotWs w2, double tol, bool capture)
{
    __shared__ RedShared sh;
    const int wv = wave_id();
    if (wv < 3) {
        long long esc;
        const double d = wave_merge<MODE>(wv == 0 ? w0 : (wv == 1 ? w1 : w2), G, &esc);
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
    const double beta = sh.val[0], tau = sh.val[1], bb = sh.val[2];
    const long long e0 = sh.red_ll[0], e1 = sh.red_ll[1], e2 = sh.red_ll[2];
    if (threadIdx.x == 0) {
        st->escapes += e0 + e1 + e2;
        if (capture) st->fallbacks += (e0 > 0) + (e1 > 0) + (e2 > 0);
        const int f = __hip_atomic_load(&st->flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        v.beta_hist[0] = beta;
        st->beta = beta;
        st->tau = tau;
        st->tau0 = tau;
        st->bb = bb;
        const double thr = (tol * tol) * bb;
        st->thr = thr;
        if (v.hist) v.hist[0] = tau;
        st->iter = 0;
        if ((f & FLAG_NONFINITE) || !is_finite_bits(tau) || !is_finite_bits(bb) || !is_finite_bits(beta)) {
            st->status = -6;
            st->done = 1;
        } else {
            st->done = (tau <= thr || st->maxit <= 0) ? 1 : 0;
        }
    }
}

hipError_t launch_fac_setup(int mode, const SellMat<double> &A, const FacPre &Pr, const PcgVecs<double> &v, double *t,
                            PcgState *st, const DotWs *ws3, double tol, int maxit, const LaunchCfg &c)
{
    const DotWs &s0 = ws3[0], &s1 = ws3[1], &s2 = ws3[2];
    k_fac_state_init<<<1, 256, 0, c.stream>>>(st, maxit, s0, s1, s2);
    dispatch(mode, c.fpe_size, [&](auto m, auto p) {
        constexpr int M = decltype(m)::value, PP = decltype(p)::value;
        dispatch_layout(A.layout(), [&](auto lay) {
            k_fac_setup_r<M, PP, decltype(lay)::value><<<c.grid, c.block, 0, c.stream>>>(A, v, st, s1, s2, c.early_exit,
                                                                                         c.fallback);
        });
        k_fac_gt<<<c.grid, c.block, 0, c.stream>>>(A.n, Pr, v.r, t, st);
        k_fac_z<M, PP, true><<<c.grid, c.block, 0, c.stream>>>(A.n, Pr, v, t, st, s0, c.early_exit, c.fallback);
        k_fac_fin_setup<M><<<1, FIN_BLOCK, 0, c.stream>>>(c.grid, v, st, s0, s1, s2, tol, c.fallback);
    });
    return hipGetLastError();
}

} // namespace rpcg
