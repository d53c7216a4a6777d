// Learned preconditioner: launchers of the feature, factor and loss kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.hpp"
#include "lp_common.hpp"

namespace rpcg {

constexpr float LP_ABSENT = -4.0f; // feature of an absent neighbour
constexpr float LP_OCLAMP = 4.0f;  // clamp of the diagonal output

// The entries of G, widened to binary64 (clamped diagonal output).
__device__ __forceinline__ float lp_clamp(float v) { return fminf(fmaxf(v, -LP_OCLAMP), LP_OCLAMP); }
__device__ __forceinline__ double lp_g_diag(float s, float o0) { return (double)(s * expf(lp_clamp(o0))); }
__device__ __forceinline__ double lp_g_off(float s, float o) { return (double)(s * o); }

// The grid's edge N >= 2 with its reciprocal: cell numbers are below 2^30, so a
// quotient is the upper half of one product (exact: the reciprocal
// 2^(31 + l) / N, rounded up, with 2^l >= N, is off by less than 2^l).
struct LpGrid {
    int N;
    unsigned mul;
    int shift;
    explicit LpGrid(int n) : N(n), mul(0), shift(0)
    {
        int l = 1;
        while ((1 << l) < n) ++l;
        mul = (unsigned)(((1ull << (31 + l)) + n - 1) / n);
        shift = l - 1;
    }
    __device__ __forceinline__ int div(int i) const { return (int)(__umulhi((unsigned)i, mul) >> shift); }
    __device__ __forceinline__ void cell(int i, int &x, int &y, int &z) const
    {
        const int q = div(i);
        z = div(q);
        x = i - q * N;
        y = q - z * N;
    }
};

// A CSR matrix in device memory (32-bit row pointers and column indices).
struct LpMat {
    const int *rp;
    const int *col;
    const double *val;
};
// Up to LP_MAT_ARGS matrices passed by value to one launch.
constexpr int LP_MAT_ARGS = 16;
struct LpMatSet {
    LpMat m[LP_MAT_ARGS];
};

// Numbers of probe vectors whose products v = A u the feature kernel forms
// in the same pass over A (others: launch_lp_mv).
inline bool lp_fused_nu(int nu) { return nu == 1 || nu == 2 || nu == 4; }

// Features and s of nb <= LP_MAT_ARGS systems (grid.y = system; feat and s of
// system k at k n 4 and k n). A missing or non-positive diagonal stores gen
// into *bad (host-visible memory; plain stores of one value). With utab (one
// pointer per pair, lp_fused_nu(nu)) also v = A u, interleaved as below.
hipError_t launch_lp_features(int N, int nb, const LpMatSet &set, bf16_t *feat, float *s, int *bad, int gen,
                              int nu, const double *const *utab, double *v, hipStream_t st);
// G, G^T values of nb instances (grid.y = instance): o, s, g_val, gt_val of
// instance k at k times the given strides (in elements).
hipError_t launch_lp_factor(int N, int nb, const float *o, const float *s, const int *g_rp, const int *gt_rp,
                            double *g_val, double *gt_val, long long val_stride, hipStream_t st);
hipError_t launch_lp_to_bf16(long long n, const double *a, bf16_t *b, hipStream_t st);

// ---- loss over a batch of (instance, probe) pairs (lp_loss.hip) ----
constexpr int LP_DOT_P = 3;         // lane expansion length of the exact dots
constexpr int LP_DOT_CHUNKS = 128;  // most workgroups (slots) per pair and dot
// The loss's vectors v, y, r, q are interleaved per instance: entry i of the
// vector of pair p = k nu + m at base + (k n + i) nu + m; the probes u_p are
// read through the pointer table utab. G and G^T are formed from the network's
// outputs o and s where they are needed.
// V_k = M_k U_k (mats[k], k < nb) for the nu vectors of each instance.
hipError_t launch_lp_mv(long long n, int nb, int nu, const LpMat *mats, const double *const *utab, double *v,
                        hipStream_t st);
// Y_k = G_k^T X_k for the nu vectors of each instance.
hipError_t launch_lp_gt(int N, int nb, int nu, const float *o, const float *s, const double *x, double *y,
                        hipStream_t st);
// R = (G_k Y + eps V) - U (interleaved; U through utab) and the partials of
// <u_p, u_p>, <r_p, r_p> in slots p * *chunks + c of wu, wr (capacity
// stride >= nb nu LP_DOT_CHUNKS).
hipError_t launch_lp_resid_dots(int N, int nb, int nu, double eps, const float *o, const float *s,
                                const double *const *utab, const double *y, const double *v, double *r,
                                const SlotWs &wu, const SlotWs &wr, int stride, int *flags, int *chunks, hipStream_t st);
// dots[2p] = <u_p, u_p>, dots[2p + 1] = <r_p, r_p>, each correctly rounded.
hipError_t launch_lp_dots_merge(int npairs, int chunks, const SlotWs &wu, const SlotWs &wr, int stride, double *dots,
                                hipStream_t st);
// dL/do of every instance (bfloat16 into dob; binary64 into do64 unless null)
// and the loss, from the interleaved R, Y, V, Q.
hipError_t launch_lp_dodg_all(int N, int nb, int nu, double scale, const double *dots, const float *o, const float *s,
                              const double *r, const double *y, const double *v, const double *q, double *do64,
                              bf16_t *dob, double *loss, hipStream_t st);

} // namespace rpcg
