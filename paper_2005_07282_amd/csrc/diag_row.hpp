// Row loop over diagonal-aligned slices (layout described with DiagSlice):
// lane j of a wavefront computes the rows 128 s + 2 j and 128 s + 2 j + 1 of
// A x, each as the sequential fma chain over the row's stored entries in their
// original order (Section 4.3).
//
// What bounds it: with constant slices no matrix data is read per row, and the
// gathers through the vector L1 set the time; otherwise the 8 bytes per entry of
// values from HBM do. The texture path takes about 16 cycles for a wavefront's load
// whether its lanes ask for 8 or 16 bytes (measured: 8-byte gathers kept it busy 15 cycles
// each), hence two rows per lane and 16-byte gathers. Records in runs of three
// neighbouring offsets (DIAG_TRI: every 27-point row, odd bands) share them: four
// consecutive elements serve the six products of the lane's two rows.
// The records are the same for the whole wavefront and come through scalar
// loads; their lane masks go to the execution mask, so a masked product costs
// one fma instead of an fma and two selects.
// Measured (SpMV + dot of the solver): 160^3 27-point 235 us in the general layout
// (1.29 GB), 70 us with one row per lane, 30.5 us now; binary32 200^3 249 us and 40.4 us;
// 64 variable-coefficient 7-point systems together 313 us and 168 us (stored values).
#pragma once

#include "kernels.hpp"

namespace rpcg {

// Uniform read-only data through the scalar cache.
template <typename T>
using cptr = const T __attribute__((address_space(4))) *;
template <typename T>
__device__ __forceinline__ cptr<T> as_const(const T *p) { return (cptr<T>)p; }

// Two neighbouring elements, aligned as one.
template <typename T> struct Pair;
template <> struct Pair<double> { typedef double t __attribute__((ext_vector_type(2), aligned(8))); };
template <> struct Pair<float> { typedef float t __attribute__((ext_vector_type(2), aligned(4))); };
template <typename T>
using pair_t = typename Pair<T>::t;

// sum[r] = fma(a[u][r], g[u][r], sum[r]) in the lanes of mask m[u][r], for records
// u = 0, .. in order and the lane's two rows r; every lane of the wavefront is
// active here (the loops over slices are uniform). The execution mask is set for
// each product and restored once per block: scalar instructions are the
// largest part of a constant slice's, and a restore after every product took
// one in four of them (SpMV + dot, 27 points: binary32 200^3 45.8 -> 40.4 us, binary64 160^3
// 31.6 -> 30.5 us). The block is volatile so that it is not moved under a
// condition. S: the factors, one for both rows, are in scalar registers.
#define RPCG_MFMA(BITS, M, R, A, G) "s_mov_b64 exec, %" #M "\n\tv_fmac_f" #BITS " %" #R ", %" #A ", %" #G "\n\t"
#define RPCG_MFMA_END "s_mov_b64 exec, -1"
template <bool S, int K, typename T>
__device__ __forceinline__ void masked_fma(T (&sum)[2], const T (*a)[2], const T (*g)[2], const unsigned long long (*m)[2])
{
    static_assert(K == 1 || K == 3, "records per block");
#define RPCG_SUMS "+&v"(sum[0]), "+&v"(sum[1])
#define RPCG_REC(u) "v"(g[u][0]), "v"(g[u][1]), "s"(m[u][0]), "s"(m[u][1])
    if constexpr (S && K == 1) {
#define RPCG_BODY(B) RPCG_MFMA(B, 4, 0, 6, 2) RPCG_MFMA(B, 5, 1, 6, 3) RPCG_MFMA_END
        if constexpr (sizeof(T) == 8) asm volatile(RPCG_BODY(64) : RPCG_SUMS : RPCG_REC(0), "s"(a[0][0]));
        else asm volatile(RPCG_BODY(32) : RPCG_SUMS : RPCG_REC(0), "s"(a[0][0]));
#undef RPCG_BODY
    } else if constexpr (S) {
#define RPCG_BODY(B) RPCG_MFMA(B, 4, 0, 14, 2) RPCG_MFMA(B, 5, 1, 14, 3) RPCG_MFMA(B, 8, 0, 15, 6) RPCG_MFMA(B, 9, 1, 15, 7) \
    RPCG_MFMA(B, 12, 0, 16, 10) RPCG_MFMA(B, 13, 1, 16, 11) RPCG_MFMA_END
        if constexpr (sizeof(T) == 8)
            asm volatile(RPCG_BODY(64) : RPCG_SUMS : RPCG_REC(0), RPCG_REC(1), RPCG_REC(2), "s"(a[0][0]), "s"(a[1][0]), "s"(a[2][0]));
        else
            asm volatile(RPCG_BODY(32) : RPCG_SUMS : RPCG_REC(0), RPCG_REC(1), RPCG_REC(2), "s"(a[0][0]), "s"(a[1][0]), "s"(a[2][0]));
#undef RPCG_BODY
    } else if constexpr (K == 1) {
#define RPCG_BODY(B) RPCG_MFMA(B, 4, 0, 6, 2) RPCG_MFMA(B, 5, 1, 7, 3) RPCG_MFMA_END
        if constexpr (sizeof(T) == 8) asm volatile(RPCG_BODY(64) : RPCG_SUMS : RPCG_REC(0), "v"(a[0][0]), "v"(a[0][1]));
        else asm volatile(RPCG_BODY(32) : RPCG_SUMS : RPCG_REC(0), "v"(a[0][0]), "v"(a[0][1]));
#undef RPCG_BODY
    } else {
#define RPCG_BODY(B) RPCG_MFMA(B, 4, 0, 14, 2) RPCG_MFMA(B, 5, 1, 15, 3) RPCG_MFMA(B, 8, 0, 16, 6) RPCG_MFMA(B, 9, 1, 17, 7) \
    RPCG_MFMA(B, 12, 0, 18, 10) RPCG_MFMA(B, 13, 1, 19, 11) RPCG_MFMA_END
#define RPCG_FACTORS "v"(a[0][0]), "v"(a[0][1]), "v"(a[1][0]), "v"(a[1][1]), "v"(a[2][0]), "v"(a[2][1])
        if constexpr (sizeof(T) == 8) asm volatile(RPCG_BODY(64) : RPCG_SUMS : RPCG_REC(0), RPCG_REC(1), RPCG_REC(2), RPCG_FACTORS);
        else asm volatile(RPCG_BODY(32) : RPCG_SUMS : RPCG_REC(0), RPCG_REC(1), RPCG_REC(2), RPCG_FACTORS);
#undef RPCG_FACTORS
#undef RPCG_BODY
    }
#undef RPCG_SUMS
#undef RPCG_REC
}
#undef RPCG_MFMA
#undef RPCG_MFMA_END

template <typename T>
__device__ __forceinline__ T rec_value(cptr<DiagEnt> e)
{
    if constexpr (sizeof(T) == 8) return e->v;
    else return e->vf;
}

// R consecutive records from k0: all loads, then the two chains. xs = x + 128 s;
// CONSTV: values from the records, else at v; TRI: records 3 q, 3 q + 1, 3 q + 2 at
// neighbouring offsets; CLAMP: entries of masked-out lanes may point outside x.
template <typename T, bool DIAG, bool CONSTV, bool TRI, bool CLAMP, int R>
__device__ __forceinline__ void diag_batch(cptr<DiagEnt> e, int k0, int width, const T *__restrict__ v,
                                           const T *__restrict__ xs, long long s128, int n, unsigned lane, T (&sum)[2],
                                           T *aii, bool *found)
{
    T a[R][2], g[R][2];
    if constexpr (!CONSTV) {
#pragma unroll
        for (int u = 0; u < R; ++u) {
            // the records past the width repeat the last one's values (already in cache; masked out)
            const int k = k0 + u < width ? k0 + u : width - 1;
            const pair_t<T> p = __builtin_nontemporal_load((const pair_t<T> *)(v + 128ll * k + 2 * lane));
            a[u][0] = p.x;
            a[u][1] = p.y;
        }
    }
    if constexpr (CLAMP) {
#pragma unroll
        for (int u = 0; u < R; ++u)
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const long long c = 2 * (long long)lane + r + e[k0 + u].off, lo = -s128, hi = n - 1 - s128;
                g[u][r] = xs[c < lo ? lo : (c > hi ? hi : c)];
            }
    } else if constexpr (TRI) {
#pragma unroll
        for (int u = 0; u < R; u += 3) {
            const T *p = xs + e[k0 + u].off;
            const pair_t<T> q0 = *(const pair_t<T> *)(p + 2 * lane), q1 = *(const pair_t<T> *)(p + 2 * lane + 2);
            g[u][0] = q0.x;
            g[u][1] = g[u + 1][0] = q0.y;
            g[u + 1][1] = g[u + 2][0] = q1.x;
            g[u + 2][1] = q1.y;
        }
    } else {
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const pair_t<T> q = *(const pair_t<T> *)(xs + e[k0 + u].off + 2 * lane);
            g[u][0] = q.x;
            g[u][1] = q.y;
        }
    }
    // the records' values and masks, as many at a time as scalar registers hold
    constexpr int H = R > DIAG_TRI_BATCH ? R / 2 : R;
#pragma unroll
    for (int u0 = 0; u0 < R; u0 += H) {
        unsigned long long m[H][2];
        T c[H][2];
        int o[H];
#pragma unroll
        for (int u = 0; u < H; ++u) {
            m[u][0] = e[k0 + u0 + u].mask[0];
            m[u][1] = e[k0 + u0 + u].mask[1];
            if constexpr (CONSTV) c[u][0] = c[u][1] = rec_value<T>(e + k0 + u0 + u);
            if constexpr (DIAG) o[u] = e[k0 + u0 + u].off;
        }
        constexpr int K = H % 3 == 0 ? 3 : 1;
#pragma unroll
        for (int u = 0; u < H; u += K) masked_fma<CONSTV, K>(sum, CONSTV ? c + u : a + u0 + u, g + u0 + u, m + u);
        if constexpr (DIAG) {
#pragma unroll
            for (int u = 0; u < H; ++u)
#pragma unroll
                for (int r = 0; r < 2; ++r)
                    if (o[u] == 0 && ((m[u][r] >> lane) & 1ull)) {
                        aii[r] = CONSTV ? c[u][r] : a[u0 + u][r];
                        found[r] = true;
                    }
        }
    }
}

template <typename T, bool DIAG, bool CONSTV, bool TRI, bool CLAMP>
__device__ __forceinline__ void diag_chain(cptr<DiagEnt> e, int width, const T *__restrict__ v,
                                           const T *__restrict__ x, long long s128, int n, unsigned lane, T (&sum)[2],
                                           T *aii, bool *found)
{
    constexpr int B = TRI ? DIAG_TRI_BATCH : DIAG_BATCH;
    const T *__restrict__ xs = x + s128;
    sum[0] = sum[1] = T(0);
    int k = 0;
    if constexpr (CONSTV && !CLAMP) { // one batch more in flight while the registers allow it
        for (; k + B < width; k += 2 * B)
            diag_batch<T, DIAG, CONSTV, TRI, CLAMP, 2 * B>(e, k, width, v, xs, s128, n, lane, sum, aii, found);
    }
    for (; k < width; k += B)
        diag_batch<T, DIAG, CONSTV, TRI, CLAMP, B>(e, k, width, v, xs, s128, n, lane, sum, aii, found);
}

// A slice's record in scalar registers. It is loaded one slice ahead through
// the vector unit (in-order return) and made scalar when its slice is due: a
// scalar load there would have to return before the entry records' first wait.
struct DiagRec {
    long long mpos, vpos;
    int width, flags;
};
__device__ __forceinline__ DiagRec diag_scalar(const DiagSlice &v)
{
    auto u32 = [](unsigned q) { return (unsigned)__builtin_amdgcn_readfirstlane((int)q); };
    auto u64 = [&](long long q) {
        return (long long)(((unsigned long long)u32((unsigned)((unsigned long long)q >> 32)) << 32) | u32((unsigned)q));
    };
    return {u64(v.mpos), u64(v.vpos), (int)u32((unsigned)v.width), (int)u32((unsigned)v.flags)};
}

// Rows 128 s + 2 lane + {0, 1} of A x (s uniform, S its record). With DIAG,
// aii[] receives the value stored in the row's own column (the last such
// entry) and found[] whether there is one. Rows past the last one give 0.
template <typename T, bool DIAG>
__device__ __forceinline__ void diag_rows(const SellMat<T> &A, const DiagRec &S, long long s, unsigned lane,
                                          const T *__restrict__ x, T (&sum)[2], T *aii, bool *found)
{
    const cptr<DiagEnt> e = as_const(A.de) + S.mpos;
    const T *v = A.val + S.vpos;
    const long long s128 = s * DIAG_ROWS;
    if (S.flags & DIAG_CONST) {
        if (S.flags & DIAG_CLAMP) diag_chain<T, DIAG, true, false, true>(e, S.width, v, x, s128, A.n, lane, sum, aii, found);
        else if (S.flags & DIAG_TRI) diag_chain<T, DIAG, true, true, false>(e, S.width, v, x, s128, A.n, lane, sum, aii, found);
        else diag_chain<T, DIAG, true, false, false>(e, S.width, v, x, s128, A.n, lane, sum, aii, found);
    } else {
        if (S.flags & DIAG_CLAMP) diag_chain<T, DIAG, false, false, true>(e, S.width, v, x, s128, A.n, lane, sum, aii, found);
        else if (S.flags & DIAG_TRI) diag_chain<T, DIAG, false, true, false>(e, S.width, v, x, s128, A.n, lane, sum, aii, found);
        else diag_chain<T, DIAG, false, false, false>(e, S.width, v, x, s128, A.n, lane, sum, aii, found);
    }
}

} // namespace rpcg
