// Learned preconditioner: per-cell input features from the matrix and the
// factor G (and G^T) from the network outputs.
//
// G sits on the lower-triangle pattern of a 7-point operator on an N^3 grid:
// row i holds the -z, -y, -x neighbours and the diagonal (ascending columns);
// G^T row j the diagonal and the +x, +y, +z neighbours. With
// s_i = RN32(1 / sqrt(a_ii)) (in binary64, rounded once):
//   G_ii = RN32(s_i exp(clamp(o_i0, -4, 4))),  G_i,j(k) = RN32(s_i o_ik),
// k = 1, 2, 3 for the -x, -y, -z neighbour, widened to binary64 for the solve.
#include "lp_common.hpp"
#include "lp_factor.hpp"

namespace rpcg {

// features: ln(|a_ij| / a_ii) of the -x, -y, -z neighbours (LP_ABSENT if
// missing), (number of absent neighbours) / 6; and s_i. A non-positive or
// missing diagonal stores gen into *bad. System k = blockIdx.y. NU > 0: also
// v = A u of its NU probe vectors (interleaved), one fma chain per row and
// vector in storage order from zero.
//
// Bound by memory: the matrix is the largest operand, so one pass over it serves
// the features and the products, and a workgroup's rows, which lie one after
// the other, are staged in LDS with coalesced loads (rows of seven entries read by
// a lane each take seven partly used lines; 8 systems of 64^3 rows and four vectors:
// features 73 us and products 124 us -> 100 us together; larger batches of gathers
// cost wavefronts in flight: eight entries at once 110 us).
constexpr int LPF_BLOCK = 256;
constexpr int LPF_PER = 8;                      // entries staged per thread
constexpr int LPF_CAP = LPF_BLOCK * LPF_PER;    // entries a workgroup stages; longer blocks are read in place
constexpr int LPF_BATCH = 4;                    // entries whose operands are loaded together

// One row: len entries at (val, col).
template <int NU>
__device__ __forceinline__ void lp_feature_row(const LpGrid &grid, long long i, int len, const double *val, const int *col,
                                               const double *const (&u)[NU ? NU : 1], bf16_t *__restrict__ feat,
                                               float *__restrict__ s, double *__restrict__ v, int *bad, int gen)
{
    const int N = grid.N, ii = (int)i; // i < n <= 2^30
    int x, y, z;
    grid.cell(ii, x, y, z);
    const int nb[3] = {x > 0 ? ii - 1 : -1, y > 0 ? ii - N : -1, z > 0 ? ii - N * N : -1};
    double aii = 0.0, a[3] = {0.0, 0.0, 0.0}, acc[NU ? NU : 1];
#pragma unroll
    for (int m = 0; m < NU; ++m) acc[m] = 0.0;
    auto entry = [&](int c, double w) {
        if (c == ii) aii = w;
#pragma unroll
        for (int d = 0; d < 3; ++d)
            if (c == nb[d]) a[d] = w;
    };
    for (int j0 = 0; j0 < len; j0 += LPF_BATCH) {
        int c[LPF_BATCH], at[LPF_BATCH];
        double w[LPF_BATCH], g[LPF_BATCH][NU ? NU : 1];
#pragma unroll
        for (int j = 0; j < LPF_BATCH; ++j) {
            const int e = j0 + j < len ? j0 + j : 0;
            c[j] = col[e];
            w[j] = val[e];
            // the diagonal check of the same pass has not refused the matrix yet: nothing is read past a probe
            at[j] = (unsigned)c[j] < (unsigned)(N * N * N) ? c[j] : 0;
        }
#pragma unroll
        for (int j = 0; j < LPF_BATCH; ++j)
#pragma unroll
            for (int m = 0; m < NU; ++m) g[j][m] = u[m][at[j]];
#pragma unroll
        for (int j = 0; j < LPF_BATCH; ++j)
            if (j0 + j < len) {
                entry(c[j], w[j]);
#pragma unroll
                for (int m = 0; m < NU; ++m) acc[m] = __builtin_fma(w[j], g[j][m], acc[m]);
            }
    }
    if (!(aii > 0.0)) *bad = gen;
    bf16_t f[4];
#pragma unroll
    for (int d = 0; d < 3; ++d)
        f[d] = f32_to_bf16((nb[d] >= 0 && a[d] != 0.0) ? (float)log(fabs(a[d]) / aii) : LP_ABSENT);
    f[3] = f32_to_bf16((float)((7 - len) / 6.0));
    *(v4s *)&feat[i * 4] = (v4s){(short)f[0], (short)f[1], (short)f[2], (short)f[3]};
    s[i] = (float)(1.0 / sqrt(aii));
    if constexpr (NU > 0) {
        typedef double vnd __attribute__((ext_vector_type(NU)));
        vnd o;
#pragma unroll
        for (int m = 0; m < NU; ++m) o[m] = acc[m];
        *(vnd *)(v + i * NU) = o;
    }
}

template <int NU>
__global__ void __launch_bounds__(LPF_BLOCK) k_lp_features(LpGrid grid, LpMatSet set, bf16_t *__restrict__ feat,
                                                           float *__restrict__ s, int *bad, int gen,
                                                           const double *const *__restrict__ utab,
                                                           double *__restrict__ v)
{
    __shared__ double sval[LPF_CAP];
    __shared__ int scol[LPF_CAP];
    const long long n = (long long)grid.N * grid.N * grid.N;
    const int k = blockIdx.y;
    const int *__restrict__ rp = set.m[k].rp;
    const int *__restrict__ col = set.m[k].col;
    const double *__restrict__ val = set.m[k].val;
    feat += (long long)k * n * 4;
    s += (long long)k * n;
    v += (long long)k * n * NU;
    const double *u[NU ? NU : 1] = {};
#pragma unroll
    for (int m = 0; m < NU; ++m) u[m] = utab[(long long)k * NU + m];
    for (long long i0 = (long long)blockIdx.x * LPF_BLOCK; i0 < n; i0 += (long long)gridDim.x * LPF_BLOCK) { // workgroup-uniform
        const long long i = i0 + threadIdx.x;
        const int b0 = rp[i0], cnt = rp[min(i0 + LPF_BLOCK, n)] - b0;
        const int b = i < n ? rp[i] : b0, len = i < n ? rp[i + 1] - b : 0;
        const bool staged = cnt <= LPF_CAP; // workgroup-uniform
        if (staged) {
            double w[LPF_PER];
            int c[LPF_PER];
#pragma unroll
            for (int t = 0; t < LPF_PER; ++t) {
                const int q = threadIdx.x + t * LPF_BLOCK;
                w[t] = q < cnt ? val[b0 + q] : 0.0;
                c[t] = q < cnt ? col[b0 + q] : 0;
            }
            __syncthreads(); // the previous rows' readers are done
#pragma unroll
            for (int t = 0; t < LPF_PER; ++t) {
                const int q = threadIdx.x + t * LPF_BLOCK;
                sval[q] = w[t];
                scol[q] = c[t];
            }
            __syncthreads();
            if (i < n) lp_feature_row<NU>(grid, i, len, sval + (b - b0), scol + (b - b0), u, feat, s, v, bad, gen);
        } else if (i < n) {
            lp_feature_row<NU>(grid, i, len, val + b, col + b, u, feat, s, v, bad, gen);
        }
    }
}

// G and G^T values at the positions of the structure (lp_pattern); instance
// k = blockIdx.y reads o, s and writes g_val, gt_val at k times their strides.
__global__ void k_lp_factor(int N, const float *__restrict__ o, const float *__restrict__ s,
                            const int *__restrict__ g_rp, const int *__restrict__ gt_rp, double *__restrict__ g_val,
                            double *__restrict__ gt_val, long long val_stride)
{
    const long long n = (long long)N * N * N, NN = (long long)N * N;
    const int k = blockIdx.y;
    o += (long long)k * n * 4;
    s += (long long)k * n;
    g_val += (long long)k * val_stride;
    gt_val += (long long)k * val_stride;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
        const int x = (int)(i % N), y = (int)((i / N) % N), z = (int)(i / NN);
        const float si = s[i];
        // row i of G: -z, -y, -x, diagonal
        int p = g_rp[i];
        if (z > 0) g_val[p++] = lp_g_off(si, o[i * 4 + 3]);
        if (y > 0) g_val[p++] = lp_g_off(si, o[i * 4 + 2]);
        if (x > 0) g_val[p++] = lp_g_off(si, o[i * 4 + 1]);
        g_val[p] = lp_g_diag(si, o[i * 4]);
        // row i of G^T: diagonal, +x, +y, +z (entries G_{i+off, i})
        int q = gt_rp[i];
        gt_val[q++] = lp_g_diag(si, o[i * 4]);
        if (x < N - 1) gt_val[q++] = lp_g_off(s[i + 1], o[(i + 1) * 4 + 1]);
        if (y < N - 1) gt_val[q++] = lp_g_off(s[i + N], o[(i + N) * 4 + 2]);
        if (z < N - 1) gt_val[q] = lp_g_off(s[i + NN], o[(i + NN) * 4 + 3]);
    }
}

__global__ void k_lp_to_bf16(long long n, const double *__restrict__ a, bf16_t *__restrict__ b)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
        b[i] = f32_to_bf16((float)a[i]);
}

static int lp_grid(long long n) { return (int)std::min<long long>(std::max<long long>((n + 255) / 256, 1), 4096); }

hipError_t launch_lp_features(int N, int nb, const LpMatSet &set, bf16_t *feat, float *s, int *bad, int gen,
                              int nu, const double *const *utab, double *v, hipStream_t st)
{
    const long long n = (long long)N * N * N;
    if (nb < 1 || nb > LP_MAT_ARGS || (utab && !lp_fused_nu(nu))) return hipErrorInvalidValue;
    const dim3 g(lp_grid(n), nb);
    if (!utab) k_lp_features<0><<<g, LPF_BLOCK, 0, st>>>(LpGrid(N), set, feat, s, bad, gen, nullptr, nullptr);
    else if (nu == 1) k_lp_features<1><<<g, LPF_BLOCK, 0, st>>>(LpGrid(N), set, feat, s, bad, gen, utab, v);
    else if (nu == 2) k_lp_features<2><<<g, LPF_BLOCK, 0, st>>>(LpGrid(N), set, feat, s, bad, gen, utab, v);
    else k_lp_features<4><<<g, LPF_BLOCK, 0, st>>>(LpGrid(N), set, feat, s, bad, gen, utab, v);
    return hipGetLastError();
}

hipError_t launch_lp_factor(int N, int nb, const float *o, const float *s, const int *g_rp, const int *gt_rp,
                            double *g_val, double *gt_val, long long val_stride, hipStream_t st)
{
    const long long n = (long long)N * N * N;
    k_lp_factor<<<dim3(lp_grid(n), nb), 256, 0, st>>>(N, o, s, g_rp, gt_rp, g_val, gt_val, val_stride);
    return hipGetLastError();
}

hipError_t launch_lp_to_bf16(long long n, const double *a, bf16_t *b, hipStream_t st)
{
    k_lp_to_bf16<<<lp_grid(n), 256, 0, st>>>(n, a, b);
    return hipGetLastError();
}

} // namespace rpcg
