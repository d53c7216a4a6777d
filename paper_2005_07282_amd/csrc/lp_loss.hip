// Learned preconditioner: the training loss and its gradient with respect to
// the network outputs, for every (instance k, probe vector m) pair of a batch
// in a handful of launches.
//
// For pair p = k nu + m with probe u = u_p and the factor G = G_k:
//   v = A u,  y = G^T v,  r = (G y + eps v) - u,  q = G^T r,
//   loss = scale sum_p <r_p, r_p> / <u_p, u_p>,
//   dL/dG_ij = (2 scale / <u, u>) (r_i y_j + v_i q_j) summed over the m of k,
// chained onto the outputs o through G's definition. The products run over
// every instance at once: a matrix row is read once for all nu vectors of its
// instance. <u, u> and <r, r> are exact dots (long accumulator, correctly
// rounded), and every sum over m and over the pairs runs in a fixed order, so
// the loss and the gradient are bit-reproducible.
#include "lp_factor.hpp"
#include "reduce.hpp"

namespace rpcg {

constexpr int LPL_BLOCK = 256;
constexpr int LPL_MG = 8;     // vectors per pass of the generic (any nu) path
typedef double v4d __attribute__((ext_vector_type(4)));

// The loss's own vectors (v, y, r, q) are interleaved: entry i of the vector
// of pair p = k nu + m sits at X + (k n + i) nu + m, so a neighbour's nu values
// come in one run (one 32-byte load for nu = 4, the training case). NU > 0 is
// that many vectors; NU = 0 handles any nu. The probes u_p stay where the caller
// keeps them (a pointer per pair). Every product is one fma chain per
// row and vector, in storage order from zero.
//
// G and G^T are not stored: an entry is a product of two of the five float32
// values of a cell (20 bytes, against 52 a row of stored values and columns), so
// these kernels, bound by memory, move little beside the vectors (8 instances of 64^3
// cells, four vectors: G^T x 54 -> 44 us, residual and dots 75 + 39 -> 88 us, dL/do
// 76 -> 55 us, and the 69 us that stored G and G^T are gone).

// V = M_k U for the nu vectors of instance k = blockIdx.y, any nu.
__global__ void __launch_bounds__(LPL_BLOCK) k_lp_mv(long long n, int nu, const LpMat *__restrict__ mats,
                                                     const double *const *__restrict__ utab, double *__restrict__ vbase)
{
    const int k = blockIdx.y;
    const LpMat M = mats[k];
    const double *const *__restrict__ ut = utab + (long long)k * nu;
    double *__restrict__ vk = vbase + (long long)k * n * nu;
    for (long long i = (long long)blockIdx.x * LPL_BLOCK + threadIdx.x; i < n; i += (long long)gridDim.x * LPL_BLOCK) {
        const int b = M.rp[i], len = M.rp[i + 1] - b;
        for (int m0 = 0; m0 < nu; m0 += LPL_MG) {
            const int mg = min(LPL_MG, nu - m0);
            double acc[LPL_MG] = {};
            for (int j = 0; j < len; ++j) {
                const double aj = M.val[b + j];
                const long long cj = M.col[b + j];
#pragma unroll
                for (int m = 0; m < LPL_MG; ++m)
                    if (m < mg) acc[m] = __builtin_fma(aj, ut[m0 + m][cj], acc[m]);
            }
#pragma unroll
            for (int m = 0; m < LPL_MG; ++m)
                if (m < mg) vk[i * nu + m0 + m] = acc[m];
        }
    }
}

// Row i of G^T (STEP = 1: diagonal, +x, +y, +z) or of G (STEP = -1: -z, -y, -x,
// diagonal): entries and column offsets in storage order, absent ones with
// offset 0 and in[j] false.
struct LpRow {
    double a[4];
    long long off[4];
    bool in[4];
};
template <int STEP>
__device__ __forceinline__ LpRow lp_row(const LpGrid &grid, long long i, const float *__restrict__ o, const float *__restrict__ s)
{
    const int N = grid.N;
    int c[3];
    grid.cell((int)i, c[0], c[1], c[2]); // i < n <= 2^30
    const long long st[3] = {1, N, (long long)N * N};
    LpRow r;
    const float si = s[i];
    const v4f oi = *(const v4f *)(o + i * 4);
    constexpr int DIAG = STEP > 0 ? 0 : 3;
    r.a[DIAG] = lp_g_diag(si, oi[0]);
    r.off[DIAG] = 0;
    r.in[DIAG] = true;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int j = STEP > 0 ? 1 + d : 2 - d;
        r.in[j] = STEP > 0 ? c[d] < N - 1 : c[d] > 0;
        r.off[j] = r.in[j] ? STEP * st[d] : 0;
        if constexpr (STEP > 0) { // entry G_{i + off, i}
            const long long e = i + r.off[j];
            r.a[j] = lp_g_off(s[e], o[e * 4 + 1 + d]);
        } else {
            r.a[j] = lp_g_off(si, oi[1 + d]);
        }
    }
    return r;
}

// Y = G_k^T X for the nu vectors of instance k = blockIdx.y.
template <int NU>
__global__ void __launch_bounds__(LPL_BLOCK) k_lp_gt(LpGrid grid, int nu, const float *__restrict__ o,
                                                     const float *__restrict__ s, const double *__restrict__ x,
                                                     double *__restrict__ y)
{
    const long long n = (long long)grid.N * grid.N * grid.N;
    const int k = blockIdx.y;
    o += (long long)k * n * 4;
    s += (long long)k * n;
    x += (long long)k * n * nu;
    y += (long long)k * n * nu;
    for (long long i = (long long)blockIdx.x * LPL_BLOCK + threadIdx.x; i < n; i += (long long)gridDim.x * LPL_BLOCK) {
        const LpRow r = lp_row<1>(grid, i, o, s);
        if constexpr (NU > 0) {
            typedef double vnd __attribute__((ext_vector_type(NU)));
            vnd xv[4], acc = 0.0;
#pragma unroll
            for (int j = 0; j < 4; ++j) xv[j] = *(const vnd *)(x + (i + r.off[j]) * NU);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int m = 0; m < NU; ++m) {
                    const double t = __builtin_fma(r.a[j], xv[j][m], acc[m]);
                    acc[m] = r.in[j] ? t : acc[m];
                }
            *(vnd *)(y + i * NU) = acc;
        } else {
            for (int m = 0; m < nu; ++m) {
                double acc = 0.0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const double t = __builtin_fma(r.a[j], x[(i + r.off[j]) * nu + m], acc);
                    acc = r.in[j] ? t : acc;
                }
                y[i * nu + m] = acc;
            }
        }
    }
}

// Entry t = i nu + m of R = (G_k Y + eps V) - U: the row's chain, then one rounding per operation.
__device__ __forceinline__ double lp_resid(const LpRow &g, long long t, int nu, double eps, const double *__restrict__ y,
                                           const double *__restrict__ v, double u)
{
    double w = 0.0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const double f = __builtin_fma(g.a[j], y[t + g.off[j] * nu], w);
        w = g.in[j] ? f : w;
    }
    return (w + eps * v[t]) - u;
}

// R of instance k = blockIdx.y, any nu.
__global__ void __launch_bounds__(LPL_BLOCK) k_lp_resid(LpGrid grid, int nu, double eps, const float *__restrict__ o,
                                                        const float *__restrict__ s,
                                                        const double *const *__restrict__ utab,
                                                        const double *__restrict__ y, const double *__restrict__ v,
                                                        double *__restrict__ r)
{
    const long long n = (long long)grid.N * grid.N * grid.N;
    const int k = blockIdx.y;
    const long long off = (long long)k * n * nu;
    o += (long long)k * n * 4;
    s += (long long)k * n;
    for (long long i = (long long)blockIdx.x * LPL_BLOCK + threadIdx.x; i < n; i += (long long)gridDim.x * LPL_BLOCK) {
        const LpRow g = lp_row<-1>(grid, i, o, s);
        for (int m = 0; m < nu; ++m)
            r[off + i * nu + m] = lp_resid(g, i * nu + m, nu, eps, y + off, v + off, utab[(long long)k * nu + m][i]);
    }
}

// The exact-dot partials of <u_p, u_p> and <r_p, r_p> into slots p chunks +
// blockIdx.x (grid: chunks x pairs); r_p read from the interleaved R.
template <int P>
__global__ void __launch_bounds__(LPL_BLOCK) k_lp_dots(long long n, int nu, const double *const *__restrict__ utab,
                                                       const double *__restrict__ rbase, SlotView su, SlotView sr,
                                                       int *flags)
{
    __shared__ RedShared sh;
    const int p = blockIdx.y, k = p / nu, m = p % nu;
    const double *__restrict__ u = utab[p];
    const double *__restrict__ r = rbase + (long long)k * n * nu + m;
    zero_acc(sh.acc[0]);
    zero_acc(sh.acc[1]);
    __syncthreads();
    LaneDot<MODE_EXBLAS, P> Lu, Lr;
    Lu.init();
    Lr.init();
    for (long long i = (long long)blockIdx.x * LPL_BLOCK + threadIdx.x; i < n;
         i += (long long)gridDim.x * LPL_BLOCK) {
        const double ui = u[i], ri = r[i * nu];
        Lu.add(ui, ui, sh.acc[0], true, true);
        Lr.add(ri, ri, sh.acc[1], true, true);
    }
    block_finish_pair<P>(Lu, sh.acc[0], su, Lr, sh.acc[1], sr, p * gridDim.x + blockIdx.x, flags, sh);
}

// R and those partials in one pass, NU = 1, 2 or 4: a lane takes one vector of
// a cell (entry t = i NU + m, so a wavefront reads runs of 512 bytes) and holds
// the expansions of that vector's two dots. At the end the lanes' expansions
// go through LDS, so that each wavefront sums lanes of one vector (NU sums
// a wavefront, most lanes empty, would cost NU times the flushes).
template <int NU, int P>
__global__ void __launch_bounds__(LPL_BLOCK) k_lp_resid_dots(LpGrid grid, double eps, const float *__restrict__ o,
                                                             const float *__restrict__ s,
                                                             const double *const *__restrict__ utab,
                                                             const double *__restrict__ y, const double *__restrict__ v,
                                                             double *__restrict__ r, SlotView su, SlotView sr,
                                                             int *flags)
{
    __shared__ long long acc[NU][2][ACC_DIGITS];
    __shared__ double ex[2 * P][LPL_BLOCK];
    __shared__ int rng[NU][2][2];
    const long long nt = (long long)grid.N * grid.N * grid.N * NU;
    const int k = blockIdx.y, tid = threadIdx.x, m = tid % NU;
    for (int q = tid; q < NU * 2 * ACC_DIGITS; q += LPL_BLOCK) (&acc[0][0][0])[q] = 0;
    for (int q = tid; q < NU * 4; q += LPL_BLOCK) (&rng[0][0][0])[q] = (q & 1) ? -1 : ACC_DIGITS;
    __syncthreads();
    o += (long long)k * nt / NU * 4;
    s += (long long)k * nt / NU;
    y += (long long)k * nt;
    v += (long long)k * nt;
    r += (long long)k * nt;
    const double *__restrict__ u = utab[(long long)k * NU + m];
    LaneDot<MODE_EXBLAS, P> Lu, Lr;
    Lu.init();
    Lr.init();
    for (long long t = (long long)blockIdx.x * LPL_BLOCK + tid; t < nt; t += (long long)gridDim.x * LPL_BLOCK) {
        const long long i = t / NU;
        const double ui = u[i];
        const double ri = lp_resid(lp_row<-1>(grid, i, o, s), t, NU, eps, y, v, ui);
        r[t] = ri;
        Lu.add(ui, ui, acc[m][0], true, true);
        Lr.add(ri, ri, acc[m][1], true, true);
    }
#pragma unroll
    for (int j = 0; j < P; ++j) {
        ex[j][tid] = Lu.a[j];
        ex[P + j][tid] = Lr.a[j];
    }
    __syncthreads();
    // lanes 64 w / NU .. of vector w % NU
    const int w = wave_id(), mm = w % NU, from = (lane_id() + 64 * (w / NU)) * NU + mm;
#pragma unroll
    for (int j = 0; j < P; ++j) {
        Lu.a[j] = ex[j][from];
        Lr.a[j] = ex[P + j][from];
    }
    wave_flush_exact2<P>(Lu.a, acc[mm][0], Lu.flags, Lr.a, acc[mm][1], Lr.flags);
    __syncthreads();
    for (int q = tid; q < NU * 2 * ACC_DIGITS; q += LPL_BLOCK) {
        const int c = q % ACC_DIGITS, d = q / ACC_DIGITS % 2, p = q / (2 * ACC_DIGITS);
        const SlotView &sv = d ? sr : su;
        const int g = (k * NU + p) * gridDim.x + blockIdx.x;
        const long long out = carried_word(acc[p][d], c);
        sv.ws.digits[(long long)c * sv.stride + g] = out;
        if (out != 0) {
            atomicMin(&rng[p][d][0], c);
            atomicMax(&rng[p][d][1], c);
        }
    }
    __syncthreads();
    if (tid < NU * 4) {
        const int e = tid & 1, d = tid >> 1 & 1, p = tid >> 2;
        (d ? sr : su).ws.range[2 * ((k * NU + p) * gridDim.x + blockIdx.x) + e] = rng[p][d][e];
    }
    const int fl = Lu.flags | Lr.flags;
    if (fl) atomicOr(flags, fl);
}

// Slots [g0, ...) of a workspace seen as slots [0, ...).
__device__ __forceinline__ SlotView slots_from(const SlotView &v, int g0)
{
    SlotView o = v;
    o.ws.digits += g0;
    o.ws.range += 2 * g0;
    return o;
}

// dots[2p] = <u_p, u_p>, dots[2p + 1] = <r_p, r_p> from the slots of pair p
// (one workgroup per pair).
__global__ void __launch_bounds__(LPL_BLOCK) k_lp_dots_merge(int chunks, SlotView su, SlotView sr, double *dots)
{
    __shared__ RedShared sh;
    const int p = blockIdx.x;
    const double uu = merge_slots(slots_from(su, p * chunks), chunks, sh.acc[0], sh, 0);
    const double rr = merge_slots(slots_from(sr, p * chunks), chunks, sh.acc[1], sh, 1);
    if (threadIdx.x == 0) {
        dots[2 * p] = uu;
        dots[2 * p + 1] = rr;
    }
}

// dL/do of instance k = blockIdx.y (summed over its nu pairs in order m = 0,
// 1, ...), rounded to bfloat16 into dob and, if do64 is given, written in
// binary64 there; the loss (pairs in order) by one thread. R, Y, V, Q are
// interleaved.
template <int NU>
__global__ void __launch_bounds__(LPL_BLOCK) k_lp_dodg(LpGrid grid, int nu_rt, int npairs, double scale,
                                                       const double *__restrict__ dots, const float *__restrict__ o,
                                                       const float *__restrict__ s,
                                                       const double *__restrict__ rbase,
                                                       const double *__restrict__ ybase,
                                                       const double *__restrict__ vbase,
                                                       const double *__restrict__ qbase, double *__restrict__ do64,
                                                       bf16_t *__restrict__ dob, double *loss)
{
    const int nu = NU ? NU : nu_rt;
    const long long N = grid.N, NN = N * N, n = NN * N;
    const int k = blockIdx.y;
    if (k == 0 && blockIdx.x == 0 && threadIdx.x == 0) {
        double L = 0.0;
        for (int p = 0; p < npairs; ++p) L += scale * dots[2 * p + 1] / dots[2 * p];
        loss[0] = L;
    }
    o += (long long)k * n * 4;
    s += (long long)k * n;
    if (do64) do64 += (long long)k * n * 4;
    dob += (long long)k * n * 4;
    const long long off = (long long)k * n * nu;
    const double *__restrict__ R = rbase + off, *__restrict__ Y = ybase + off;
    const double *__restrict__ V = vbase + off, *__restrict__ Q = qbase + off;
    for (long long i = (long long)blockIdx.x * LPL_BLOCK + threadIdx.x; i < n; i += (long long)gridDim.x * LPL_BLOCK) {
        int x, yy, z;
        grid.cell((int)i, x, yy, z);
        const double si = s[i];
        const double gdiag = lp_g_diag(s[i], o[i * 4]);
        const long long nbr[3] = {x > 0 ? i - 1 : -1, yy > 0 ? i - N : -1, z > 0 ? i - NN : -1};
        double g[4] = {0.0, 0.0, 0.0, 0.0};
        if constexpr (NU == 4) {
            const v4d r4 = *(const v4d *)(R + i * 4), v4 = *(const v4d *)(V + i * 4);
            const v4d y4 = *(const v4d *)(Y + i * 4), q4 = *(const v4d *)(Q + i * 4);
            v4d yn[3], qn[3];
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const long long j = nbr[d] >= 0 ? nbr[d] : i;
                yn[d] = *(const v4d *)(Y + j * 4);
                qn[d] = *(const v4d *)(Q + j * 4);
            }
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const double c = scale * 2.0 / dots[2 * ((long long)k * 4 + m)];
                g[0] += c * (r4[m] * y4[m] + v4[m] * q4[m]) * gdiag;
#pragma unroll
                for (int d = 0; d < 3; ++d)
                    if (nbr[d] >= 0) g[1 + d] += c * (r4[m] * yn[d][m] + v4[m] * qn[d][m]) * si;
            }
        } else {
            for (int m = 0; m < nu; ++m) {
                const double c = scale * 2.0 / dots[2 * ((long long)k * nu + m)];
                const double ri = R[i * nu + m], vi = V[i * nu + m];
                g[0] += c * (ri * Y[i * nu + m] + vi * Q[i * nu + m]) * gdiag;
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    const long long j = nbr[d];
                    if (j >= 0) g[1 + d] += c * (ri * Y[j * nu + m] + vi * Q[j * nu + m]) * si;
                }
            }
        }
        if (!(fabsf(o[i * 4]) < LP_OCLAMP)) g[0] = 0.0; // clamped: no gradient through the diagonal output
        if (do64) *(v4d *)(do64 + i * 4) = (v4d){g[0], g[1], g[2], g[3]};
        *(v4s *)(dob + i * 4) = (v4s){(short)f32_to_bf16((float)g[0]), (short)f32_to_bf16((float)g[1]),
                                      (short)f32_to_bf16((float)g[2]), (short)f32_to_bf16((float)g[3])};
    }
}

static unsigned lpl_grid(long long n) { return (unsigned)std::min<long long>(std::max<long long>((n + LPL_BLOCK - 1) / LPL_BLOCK, 1), 2048); }

hipError_t launch_lp_mv(long long n, int nb, int nu, const LpMat *mats, const double *const *utab, double *v,
                        hipStream_t st)
{
    k_lp_mv<<<dim3(lpl_grid(n), nb), LPL_BLOCK, 0, st>>>(n, nu, mats, utab, v);
    return hipGetLastError();
}

hipError_t launch_lp_gt(int N, int nb, int nu, const float *o, const float *s, const double *x, double *y,
                        hipStream_t st)
{
    const dim3 g(lpl_grid((long long)N * N * N), nb);
    if (nu == 4) k_lp_gt<4><<<g, LPL_BLOCK, 0, st>>>(LpGrid(N), nu, o, s, x, y);
    else if (nu == 2) k_lp_gt<2><<<g, LPL_BLOCK, 0, st>>>(LpGrid(N), nu, o, s, x, y);
    else k_lp_gt<0><<<g, LPL_BLOCK, 0, st>>>(LpGrid(N), nu, o, s, x, y);
    return hipGetLastError();
}

hipError_t launch_lp_resid_dots(int N, int nb, int nu, double eps, const float *o, const float *s,
                                const double *const *utab, const double *y, const double *v, double *r,
                                const SlotWs &wu, const SlotWs &wr, int stride, int *flags, int *chunks, hipStream_t st)
{
    SlotView su{wu, stride}, sr{wr, stride};
    const long long n = (long long)N * N * N;
    // four entries a lane at least: each workgroup's partials cost its flush and the merge a slot
    const long long per = (lp_fused_nu(nu) ? n * nu : n) / (4 * LPL_BLOCK);
    *chunks = (int)std::min<long long>(std::max<long long>(per, 1), LP_DOT_CHUNKS);
    const dim3 g(*chunks, nb);
    if (nu == 1) {
        k_lp_resid_dots<1, LP_DOT_P><<<g, LPL_BLOCK, 0, st>>>(LpGrid(N), eps, o, s, utab, y, v, r, su, sr, flags);
    } else if (nu == 2) {
        k_lp_resid_dots<2, LP_DOT_P><<<g, LPL_BLOCK, 0, st>>>(LpGrid(N), eps, o, s, utab, y, v, r, su, sr, flags);
    } else if (nu == 4) {
        k_lp_resid_dots<4, LP_DOT_P><<<g, LPL_BLOCK, 0, st>>>(LpGrid(N), eps, o, s, utab, y, v, r, su, sr, flags);
    } else {
        k_lp_resid<<<dim3(lpl_grid(n), nb), LPL_BLOCK, 0, st>>>(LpGrid(N), nu, eps, o, s, utab, y, v, r);
        k_lp_dots<LP_DOT_P><<<dim3(*chunks, nb * nu), LPL_BLOCK, 0, st>>>(n, nu, utab, r, su, sr, flags);
    }
    return hipGetLastError();
}

hipError_t launch_lp_dots_merge(int npairs, int chunks, const SlotWs &wu, const SlotWs &wr, int stride, double *dots,
                                hipStream_t st)
{
    SlotView su{wu, stride}, sr{wr, stride};
    hipLaunchKernelGGL(k_lp_dots_merge, dim3(npairs), dim3(LPL_BLOCK), 0, st, chunks, su, sr, dots);
    return hipGetLastError();
}

hipError_t launch_lp_dodg_all(int N, int nb, int nu, double scale, const double *dots, const float *o, const float *s,
                              const double *r, const double *y, const double *v, const double *q, double *do64,
                              bf16_t *dob, double *loss, hipStream_t st)
{
    const long long n = (long long)N * N * N;
    if (nu == 4)
        hipLaunchKernelGGL(k_lp_dodg<4>, dim3(lpl_grid(n), nb), dim3(LPL_BLOCK), 0, st, LpGrid(N), nu, nb * nu, scale, dots, o,
                           s, r, y, v, q, do64, dob, loss);
    else
        hipLaunchKernelGGL(k_lp_dodg<0>, dim3(lpl_grid(n), nb), dim3(LPL_BLOCK), 0, st, LpGrid(N), nu, nb * nu, scale, dots, o,
                           s, r, y, v, q, do64, dob, loss);
    return hipGetLastError();
}

} // namespace rpcg
