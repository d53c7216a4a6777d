// Batched Jacobi-PCG: one iteration of every system of a batch that is not
// done, in three streaming kernels over runs (slice ranges of one system),
// cut at the two global reductions of Fig. 2 as in the single solver:
//   K1 SpMV and the partials of <d, w>;
//   K2 merge of that system's <d, w> partials (every run alike), rho, the
//      residual and Jacobi updates and the partials of <z, r>, <r, r>;
//   K3 merge of those, the stopping test, gamma, the iterate update (S3)
//      and the direction update (S7).
// Each merge sums the integer partials of the run's own system and rounds
// once, so every scalar of a system is the rounded exact value of that
// system's data alone: the results do not depend on the other systems, on
// their order or on the run schedule.
//
// The scalars of a system are written by its lead run (the run holding its
// first slice) and read by every run of the system in later kernels, never
// in the same one: beta alternates between two entries by the parity of the
// iteration, K3 records the new iteration count in iter, and K1 commits it
// to it_cur, which K2 and K3 read. A K3 run returns early only if the system
// ended before its x update of this iteration was owed (ended <= it_cur),
// which the stopping test of the same launch never sets. Nothing depends on
// a launch argument, so a captured sequence of iterations replays unchanged.
#include "batch_common.hpp"

namespace rpcg {

// K1: S1 + partial of S2 (as k_pcg_spmv_dot, per run).
template <int MODE, int P, int LAY>
__global__ void __launch_bounds__(MAX_BLOCK) k_batch_spmv_dot(BatchArgs a, bool ee, bool capture)
{
    __shared__ RedShared sh;
    const int lane = lane_id();
    const int W = num_waves();
    const int wave = __builtin_amdgcn_readfirstlane(wave_id());
    for (int ri = a.wg_run[blockIdx.x]; ri < a.wg_run[blockIdx.x + 1]; ++ri) {
        const BatchRun R = a.runs[ri];
        PcgState *st = a.st + R.sys;
        // the lead run commits the iteration count K3 recorded (no workgroup of
        // this kernel reads it_cur; done is not written during this kernel)
        if (R.s0 == 0 && threadIdx.x == 0) st->it_cur = st->iter;
        if (st->done) continue;
        const BatchSys S = a.sys[R.sys];
        const int copies = batch_dot_copies(S);
        const SellMat<double> M = batch_mat(a, S);
        const double *__restrict__ d = a.d + S.row0;
        double *__restrict__ w = a.w + S.row0;
        const DotWs wd = batch_dot(a, S, 0);
        if (MODE != MODE_PLAIN && R.s0 == 0) { // the direction kernel has read them
            clear_dot(batch_dot(a, S, 1), copies);
            clear_dot(batch_dot(a, S, 2), copies);
        }
        __syncthreads(); // the previous run's accumulator has been published before it is reused
        zero_acc(sh.acc[0]);
        __syncthreads();
        LaneDot<MODE, P> L;
        L.init();
        for_slices<double, LAY, false>(M, batch_slices<LAY>(R, wave, W), lane, [&](long long i, auto &&rows) {
            constexpr int NR = lane_rows<LAY>();
            double sum[NR], di[NR];
            rows(d, sum, nullptr, nullptr);
            load_rows<NR>(di, d, i, M.n);
            store_rows(w, sum, i, M.n);
#pragma unroll
            for (int r = 0; r < NR; ++r)
                if (i + r < M.n) L.add(di[r], sum[r], sh.acc[0], ee, capture);
        });
        block_publish<MODE, P, 1, false>({&L}, {sh.acc[0]}, {&wd}, R.slot - S.slot0, ee, capture, &st->flags, sh, copies);
    }
}

// K2: delta = <d, w> of the run's system merged (every run alike, by its first
// wavefront), rho = beta / delta; S4, S5 and the partials of S6, S8. Two rows per
// thread and step (16-byte accesses), the next two loaded ahead.
template <int MODE, int P>
__global__ void __launch_bounds__(MAX_BLOCK) k_batch_update(BatchArgs a, bool ee, bool capture)
{
    __shared__ RedShared sh;
    for (int ri = a.wg_run[blockIdx.x]; ri < a.wg_run[blockIdx.x + 1]; ++ri) {
        const BatchRun R = a.runs[ri];
        PcgState *st = a.st + R.sys;
        const BatchSys S = a.sys[R.sys];
        const int copies = batch_dot_copies(S);
        const bool lead = R.s0 == 0;
        const int i1 = (int)min((long long)R.s1 * 64, (long long)S.n);
        long long i = (long long)R.s0 * 64 + 2 * threadIdx.x;
        const double *__restrict__ wp = a.w + S.row0, *__restrict__ qp = a.dinv + S.row0;
        double *__restrict__ rp = a.r + S.row0, *__restrict__ zp = a.z + S.row0;
        double wn[2], rn[2], qn[2];
        load_rows<2>(wn, wp, i, i1);
        load_rows<2>(rn, (const double *)rp, i, i1);
        load_rows<2>(qn, qp, i, i1);
        const int it = st->it_cur;
        const double beta = st->beta_par[it & 1];
        __syncthreads(); // the previous run has read sh
        if (wave_id() == 0) {
            const int done = coherent_int(&st->done), flags = coherent_int(&st->flags);
            long long esc;
            const double d = wave_merge<MODE>(batch_dot(a, S, 0), S.slot1 - S.slot0, &esc, copies);
            if (lane_id() == 0) {
                sh.flag = done; // set in this kernel only by a breakdown every run sees
                sh.rng[0] = flags;
                sh.val[0] = d;
                sh.red_ll[0] = esc;
            }
        }
        zero_acc(sh.acc[0]);
        zero_acc(sh.acc[1]);
        __syncthreads();
        if (sh.flag) continue;
        const double delta = sh.val[0];
        const bool bad = (sh.rng[0] & FLAG_NONFINITE) || !is_finite_bits(delta);
        const bool breakdown = !(delta > 0.0);
        const double rho = beta / delta;
        if (lead && threadIdx.x == 0) {
            const long long esc = sh.red_ll[0];
            if (esc) st->escapes += esc;
            if (capture && esc > 0) st->fallbacks += 1;
            st->delta = delta;
            if (bad || breakdown) {
                st->status = bad ? -6 : -5;
                st->ended = it;
                st->done = 1;
                atomicSub(a.active, 1);
            } else {
                st->rho = rho;
            }
        }
        if (bad || breakdown) continue;
        LaneDot<MODE, P> Lb, Lt;
        Lb.init();
        Lt.init();
        while (i < i1) {
            const long long cur = i;
            double ri[2], zi[2];
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                ri[r] = __builtin_fma(-rho, wn[r], rn[r]);                 // S4
                zi[r] = qn[r] * ri[r];                                     // S5
            }
            i += 2 * blockDim.x;
            load_rows<2>(wn, wp, i, i1);
            load_rows<2>(rn, (const double *)rp, i, i1);
            load_rows<2>(qn, qp, i, i1);
            store_rows(rp, ri, cur, i1);
            store_rows(zp, zi, cur, i1);
#pragma unroll
            for (int r = 0; r < 2; ++r)
                if (cur + r < i1) {
                    Lb.add(zi[r], ri[r], sh.acc[0], ee, capture);          // S6
                    Lt.add(ri[r], ri[r], sh.acc[1], ee, capture);          // S8
                }
        }
        const DotWs wb = batch_dot(a, S, 1), wt = batch_dot(a, S, 2);
        block_publish<MODE, P, 2, false>({&Lb, &Lt}, {sh.acc[0], sh.acc[1]}, {&wb, &wt}, R.slot - S.slot0, ee, capture,
                                         &st->flags, sh, copies);
    }
}

// K3: beta, tau of the run's system merged (by its first two wavefronts);
// stopping test of Fig. 1; gamma = beta / beta_old; S3 and (unless the system
// stops) S7, BATCH_DIR row pairs per thread loaded at a time, the first while
// the dots are merged.
constexpr int BATCH_DIR = 4;
template <int MODE>
__global__ void __launch_bounds__(MAX_BLOCK) k_batch_direction(BatchArgs a, bool capture)
{
    __shared__ RedShared sh;
    for (int ri = a.wg_run[blockIdx.x]; ri < a.wg_run[blockIdx.x + 1]; ++ri) {
        const BatchRun R = a.runs[ri];
        PcgState *st = a.st + R.sys;
        const BatchSys S = a.sys[R.sys];
        const int copies = batch_dot_copies(S);
        const bool lead = R.s0 == 0;
        const int i1 = (int)min((long long)R.s1 * 64, (long long)S.n);
        const long long step = 2 * blockDim.x;
        long long i = (long long)R.s0 * 64 + 2 * threadIdx.x;
        double *__restrict__ dp = a.d + S.row0, *__restrict__ xp = a.x + S.row0;
        const double *__restrict__ zp = a.z + S.row0;
        double dv[BATCH_DIR][2], zv[BATCH_DIR][2], xv[BATCH_DIR][2];
        auto load = [&](long long at) {
#pragma unroll
            for (int j = 0; j < BATCH_DIR; ++j) {
                load_rows<2>(dv[j], (const double *)dp, at + j * step, i1);
                load_rows<2>(zv[j], zp, at + j * step, i1);
                load_rows<2>(xv[j], (const double *)xp, at + j * step, i1);
            }
        };
        load(i);
        const int it = st->it_cur, maxit = st->maxit;
        const double beta_old = st->beta_par[it & 1], thr = st->thr;
        const double rho = st->rho; // K2's rho of this iteration
        const int G = S.slot1 - S.slot0;
        __syncthreads(); // the previous run has read sh
        const int wv = wave_id();
        if (wv == 0) {
            const int ended = coherent_int(&st->ended) <= it, flags = coherent_int(&st->flags);
            long long esc;
            const double b = wave_merge<MODE>(batch_dot(a, S, 1), G, &esc, copies);
            if (lane_id() == 0) {
                sh.flag = ended;
                sh.rng[0] = flags;
                sh.val[0] = b;
                sh.red_ll[0] = esc;
            }
        }
        if (wv == (num_waves() > 1 ? 1 : 0)) {
            long long esc;
            const double t = wave_merge<MODE>(batch_dot(a, S, 2), G, &esc, copies);
            if (lane_id() == 0) {
                sh.val[1] = t;
                sh.red_ll[1] = esc;
            }
        }
        __syncthreads();
        if (sh.flag) continue;
        const double beta = sh.val[0], tau = sh.val[1];
        const bool bad = (sh.rng[0] & FLAG_NONFINITE) || !is_finite_bits(beta) || !is_finite_bits(tau);
        const bool stop = bad || tau <= thr || it + 1 >= maxit;
        const double gamma = beta / beta_old;
        if (MODE != MODE_PLAIN && lead) clear_dot(batch_dot(a, S, 0), copies); // K2 has read it
        if (lead && threadIdx.x == 0) {
            const long long eb = sh.red_ll[0], et = sh.red_ll[1];
            if (eb + et) st->escapes += eb + et;
            if (capture && eb + et) st->fallbacks += (eb > 0) + (et > 0);
            if (bad) {
                st->status = -6;
            } else {
                st->gamma = gamma;
                st->beta = beta;
                st->beta_par[(it + 1) & 1] = beta;
                st->tau = tau;
                st->iter = it + 1;
                if (a.hist && a.hist[R.sys]) a.hist[R.sys][it + 1] = tau;
            }
            if (stop) {
                st->ended = it + 1;
                st->done = 1;
                atomicSub(a.active, 1);
            }
        }
        while (i < i1) {
#pragma unroll
            for (int j = 0; j < BATCH_DIR; ++j) {
                const long long c = i + j * step;
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    xv[j][r] = __builtin_fma(rho, dv[j][r], xv[j][r]);      // S3
                    dv[j][r] = __builtin_fma(gamma, dv[j][r], zv[j][r]);    // S7
                }
                store_rows(xp, xv[j], c, i1);
                if (!stop) store_rows(dp, dv[j], c, i1);
            }
            i += BATCH_DIR * step;
            if (i < i1) load(i);
        }
    }
}

hipError_t launch_batch_iteration(int mode, int layout, const BatchArgs &a, int grid, int block, const LaunchCfg &c)
{
    dispatch(mode, c.fpe_size, [&](auto m, auto p) {
        constexpr int M = decltype(m)::value, PP = decltype(p)::value;
        dispatch_layout(layout, [&](auto lay) {
            k_batch_spmv_dot<M, PP, decltype(lay)::value><<<grid, block, 0, c.stream>>>(a, c.early_exit, c.fallback);
        });
        k_batch_update<M, PP><<<grid, block, 0, c.stream>>>(a, c.early_exit, c.fallback);
        k_batch_direction<M><<<grid, block, 0, c.stream>>>(a, c.fallback);
    });
    return hipGetLastError();
}

} // namespace rpcg
