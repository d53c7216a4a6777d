// Diagonal-aligned slices: the matrix copy of the solvers for operators whose
// rows share their column offsets (stencils, bands). Layout with DiagSlice.
//
// A slice's 128 rows are merged by column offset (column - row): each step
// takes the smallest head offset over the rows and emits one entry record for
// every row whose next entry sits there, so a row's entries keep their storage
// order whatever that order is. The merge gives up on a matrix whose rows do
// not line up (more records in a slice than the longest rows of its two halves
// together, plus 8); the caller then builds the general sliced-ELL copy.
//
// What bounds the merge and the pass before it is what its wavefronts say to
// the whole device: a device-scope atomic on one address takes about 10 ns however many
// CUs wait for it. So a workgroup adds its totals once, as many workgroups as fit walk all slices, and a
// wavefront claims a record list's table slot only where it has not just seen it claimed
// (1 M rows of three entries: widths 62 -> 7 us, merge 288 -> 53 us; 512 k rows of 27
// 60 -> 4 and 174 -> 76 us).
#include "kernels.hpp"

#include <algorithm>

namespace rpcg {

// The matrix of slice s (wavefront-uniform; UNIT: 64-row slices per slice of s): of
// several the last that starts at or before it.
template <int UNIT, typename TIN>
__device__ __forceinline__ DiagCsr<TIN> matrix_of(const DiagCsr<TIN> &one, const DiagCsr<TIN> *__restrict__ mats, int nmats,
                                                  long long s)
{
    if (nmats <= 1) return one;
    int lo = 0, hi = nmats - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (mats[mid].slice0 <= UNIT * s) lo = mid;
        else hi = mid - 1;
    }
    return mats[lo];
}

// Pass 1: slice widths (longest row), the longest row of the matrix, and the
// check of row_ptr (0 at the start, nnz at the end, non-decreasing), over the slices of one
// matrix or of all systems of a batch (mats in device memory). The merge's table is
// emptied on the way. SAMPLE: info->varying counts the slices in which first entries at one
// offset differ, so that a matrix of few slices whose values plainly vary is not tried
// at all (a failed try costs 20 to 40 us).
template <typename TIN, bool SAMPLE>
__global__ void __launch_bounds__(256) k_row_widths(DiagCsr<TIN> one, const DiagCsr<TIN> *__restrict__ mats, int nmats,
                                                    int nslices, int *__restrict__ w, int *__restrict__ table, DotInfo *info)
{
    __shared__ int top, vary;
    if (blockIdx.x == 0)
        for (int k = threadIdx.x; k < DIAG_TABLE; k += blockDim.x) table[k] = -1;
    const int lane = threadIdx.x & 63;
    const long long nwaves = ((long long)gridDim.x * blockDim.x) >> 6;
    int wmax = 0, differ = 0;
    bool ok = true;
    if (threadIdx.x == 0) top = vary = 0;
    __syncthreads();
    for (long long s = __builtin_amdgcn_readfirstlane((int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6)); s < nslices;
         s += nwaves) {
        const DiagCsr<TIN> M = matrix_of<1>(one, mats, nmats, s);
        const long long i = (s - M.slice0) * 64 + lane;
        int a = 0, b = 0;
        bool good = true;
        if (i < M.n) {
            a = M.rp[i];
            b = M.rp[i + 1];
            good = a >= 0 && a <= b && b <= M.nnz;
            ok = ok && good && (i != 0 || a == 0) && (i != M.n - 1 || b == M.nnz);
        }
        if constexpr (SAMPLE) {
            const bool has = good && b > a;
            const unsigned off = has ? (unsigned)M.col[a] - (unsigned)i : 0u;
            const unsigned long long v = has ? __builtin_bit_cast(unsigned long long, (double)M.val[a]) : 0ull;
            const unsigned long long m = __ballot(has);
            if (m) {
                const int f = (int)__builtin_ctzll(m);
                const unsigned of = __builtin_amdgcn_readlane(off, f);
                const unsigned v0 = __builtin_amdgcn_readlane((unsigned)v, f), v1 = __builtin_amdgcn_readlane((unsigned)(v >> 32), f);
                differ += __ballot(has && off == of && v != (((unsigned long long)v1 << 32) | v0)) != 0;
            }
        }
        int len = max(0, b - a);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) len = max(len, __shfl_xor(len, o, 64));
        if (lane == 0) w[s] = len;
        wmax = max(wmax, len);
    }
    if (__ballot(!ok) != 0 && lane == 0) atomicOr(&info->flags, 1);
    if (lane == 0) {
        atomicMax(&top, wmax);
        if (SAMPLE && differ) atomicAdd(&vary, differ);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (__hip_atomic_load(&info->max_len, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < top) atomicMax(&info->max_len, top);
        if (SAMPLE && vary) atomicAdd(&info->varying, vary);
    }
}

// out[j * stride] = 64 sum(len[0..j)) for j < m, and out[m * stride] too when
// `total` is set. Each workgroup sums what lies before its tile itself (a few
// hundred KB at most at the largest sizes), so one launch does it.
constexpr int SCAN_TILE = 4096;
__global__ void __launch_bounds__(1024) k_scan_len(const int *__restrict__ len, int m, long long *__restrict__ out,
                                                   int stride, bool total)
{
    __shared__ long long part[1024];
    const int t = threadIdx.x;
    const int t0 = blockIdx.x * SCAN_TILE;
    long long before = 0;
    for (int j = t; j < t0; j += 1024) before += len[j];
    int v[4];
    long long own = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int j = t0 + 4 * t + q;
        v[q] = j < m ? len[j] : 0;
        own += v[q];
    }
    part[t] = before;
    __syncthreads();
    for (int d = 512; d > 0; d >>= 1) {
        if (t < d) part[t] += part[t + d];
        __syncthreads();
    }
    const long long start = part[0];
    __syncthreads();
    part[t] = own;
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {
        const long long p = t >= d ? part[t - d] : 0;
        __syncthreads();
        part[t] += p;
        __syncthreads();
    }
    long long run = start + part[t] - own;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int j = t0 + 4 * t + q;
        if (j < m) out[(long long)j * stride] = 64 * run;
        run += v[q];
        if (total && j == m - 1) out[(long long)m * stride] = 64 * run;
    }
}

// Minimum of an int over the wavefront, in every lane (DPP steps).
__device__ __forceinline__ int wave_min_i32(int v)
{
    constexpr int ID = 2147483647;
    v = min(v, __builtin_amdgcn_update_dpp(ID, v, 0x111, 0xF, 0xF, false));
    v = min(v, __builtin_amdgcn_update_dpp(ID, v, 0x112, 0xF, 0xF, false));
    v = min(v, __builtin_amdgcn_update_dpp(ID, v, 0x114, 0xF, 0xF, false));
    v = min(v, __builtin_amdgcn_update_dpp(ID, v, 0x118, 0xF, 0xF, false));
    v = min(v, __builtin_amdgcn_update_dpp(ID, v, 0x142, 0xA, 0xF, false));
    v = min(v, __builtin_amdgcn_update_dpp(ID, v, 0x143, 0xC, 0xF, false));
    return __builtin_amdgcn_readlane(v, 63);
}

constexpr int DW_WIN = 16;   // entries of every row staged in LDS at a time
constexpr int DW_PITCH = 17; // row pitch: the rows' heads fall in different banks
constexpr int DW_WAVES = 2;  // slices (wavefronts) per workgroup

// Stage the next DW_WIN entries of every row of the slice: 16 consecutive
// lanes read 16 consecutive entries of a row, with HALF of the loads in
// flight at a time. at[r]: next entry of the lane's row r, rem[r]: entries left.
template <typename TV, typename F>
__device__ __forceinline__ void stage_rows(TV *win, const TV *__restrict__ src, const int (&at)[2], const int (&rem)[2],
                                           int lane, F &&check)
{
    constexpr int HALF = 16;
    const int kk = lane & 15, sub = lane >> 4;
    __builtin_amdgcn_wave_barrier(); // one wavefront owns the window: LDS order is program order
#pragma unroll
    for (int r = 0; r < 2; ++r) { // rows 2 j + r of four lanes j at a time
        TV q[HALF];
        bool in[HALF];
#pragma unroll
        for (int g = 0; g < HALF; ++g) {
            const int j = 4 * g + sub;
            const int ar = __shfl(at[r], j, 64), lr = __shfl(rem[r], j, 64);
            in[g] = kk < lr;
            q[g] = in[g] ? src[(long long)ar + kk] : TV(0);
        }
#pragma unroll
        for (int g = 0; g < HALF; ++g)
            if (in[g]) {
                check(q[g]);
                win[(2 * (4 * g + sub) + r) * DW_PITCH + kk] = q[g];
            }
    }
    __builtin_amdgcn_wave_barrier();
}

// Pass 2: the merge, one wavefront per 128-row slice (grid-stride). Writes the
// entry records and DiagSlice (vpos excepted), ulen[s] (records whose values
// must be stored: 0 for a constant slice), the column check, and the totals of
// the matrix. Once a slice has failed, or more than max_stored of all slices
// need stored values, the others stop.
template <typename TIN>
__global__ void __launch_bounds__(64 * DW_WAVES)
k_diag_align(DiagCsr<TIN> one, const DiagCsr<TIN> *__restrict__ mats, int nmats, int nslices,
             const long long *__restrict__ off, DiagEnt *__restrict__ de, DiagSlice *__restrict__ ds,
             int *__restrict__ ulen, int *__restrict__ table, DotInfo *info, int max_stored)
{
    __shared__ int cwin[DW_WAVES][DIAG_ROWS * DW_PITCH];
    __shared__ TIN vwin[DW_WAVES][DIAG_ROWS * DW_PITCH];
    __shared__ unsigned long long sums[2]; // records, and those whose values must be stored
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (threadIdx.x < 2) sums[threadIdx.x] = 0;
    __syncthreads();
    int *cw = cwin[wv] + 2 * lane * DW_PITCH; // this lane's two rows
    TIN *vw = vwin[wv] + 2 * lane * DW_PITCH;
    unsigned long long tot = 0, totv = 0;
    bool failed = false, cbad = false;
    const bool few = max_stored != DIAG_ANY; // slices that need stored values are counted as they are met
    auto given_up = [&]() {
        return __builtin_amdgcn_readfirstlane(__hip_atomic_load(&info->diag_fail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) != 0;
    };
    int claimed = -1, seen = 0; // the table slot last found claimed; slices since the last look at the others
    const long long step = (long long)gridDim.x * DW_WAVES;
    for (long long s = (long long)blockIdx.x * DW_WAVES + wv; s < nslices; s += step) {
        if (++seen == 4) {
            seen = 0;
            if (given_up()) break;
        }
        const DiagCsr<TIN> M = matrix_of<2>(one, mats, nmats, s);
        const int n = M.n;
        const int *__restrict__ rp = M.rp, *__restrict__ col = M.col;
        const TIN *__restrict__ val = M.val;
        const long long s128 = (s - M.slice0 / 2) * DIAG_ROWS;
        const long long i = s128 + 2 * lane;
        int a[2], rem[2], p[2] = {0, 0}; // rem: entries from the window's start, p: consumed within the window
        a[0] = i < n ? rp[i] : 0;
        a[1] = i + 1 < n ? rp[i + 1] : 0;
        rem[0] = i < n ? rp[i + 1] - a[0] : 0;
        rem[1] = i + 1 < n ? rp[i + 2] - a[1] : 0;
        const long long W = off[2 * s];
        const int limit = (int)((off[2 * s + 2] - W) >> 6) + 8;
        const long long mpos = diag_mpos(W, s);
        int u = 0, omin = 0, omax = 0, oprev = 0;
        bool cst = true, tri = true;
        unsigned long long h = 0, hv = 0; // hashes of the offsets and masks, and of the values
        auto range = [&](int c) { if (c < 0 || c >= n) cbad = true; };
        auto none = [](TIN) {};
        stage_rows(cwin[wv], col, a, rem, lane, range);
        // values are staged only while the slice may be constant: the first
        // entries decide most matrices
        const TIN v0[2] = {rem[0] > 0 ? val[a[0]] : TIN(0), rem[1] > 0 ? val[a[1]] : TIN(0)};
        bool staged = false;
        while (true) {
            const bool has[2] = {p[0] < rem[0], p[1] < rem[1]};
            const int o[2] = {has[0] ? cw[p[0]] - (int)i : 2147483647,
                              has[1] ? cw[DW_PITCH + p[1]] - (int)(i + 1) : 2147483647};
            const int om = wave_min_i32(min(o[0], o[1]));
            if (__ballot(has[0] || has[1]) == 0) break;
            if (u == limit) { failed = true; break; }
            const bool in[2] = {has[0] && o[0] == om, has[1] && o[1] == om};
            const unsigned long long m[2] = {__ballot(in[0]), __ballot(in[1])};
            double vv = 0.0;
            if (cst) {
                if (!staged && u > 0) { stage_rows(vwin[wv], val, a, rem, lane, none); staged = true; }
                double mine[2];
#pragma unroll
                for (int r = 0; r < 2; ++r)
                    mine[r] = u == 0 ? (double)v0[r] : (in[r] ? (double)vw[r * DW_PITCH + p[r]] : 0.0);
                const unsigned long long b0 = __builtin_bit_cast(unsigned long long, mine[0]);
                const unsigned long long b1 = __builtin_bit_cast(unsigned long long, mine[1]);
                const unsigned long long mine_first = in[0] ? b0 : b1;
                const int f = (int)__builtin_ctzll(m[0] | m[1]);
                const unsigned lo = __builtin_amdgcn_readlane((unsigned)mine_first, f);
                const unsigned hi = __builtin_amdgcn_readlane((unsigned)(mine_first >> 32), f);
                const unsigned long long fb = ((unsigned long long)hi << 32) | lo;
                vv = __builtin_bit_cast(double, fb);
                if (__ballot((in[0] && b0 != fb) || (in[1] && b1 != fb)) != 0) {
                    cst = false;
                    if (few) {
                        int before = 0;
                        if (lane == 0) before = atomicAdd(&info->diag_stored, 1);
                        if (__builtin_amdgcn_readfirstlane(before) >= max_stored) { failed = true; break; }
                    }
                }
            }
            if (lane == 0) de[mpos + u] = DiagEnt{vv, {m[0], m[1]}, om, (float)vv};
            h = (h ^ (unsigned)om ^ (m[0] * 0x9E3779B97F4A7C15ull)) * 0xBF58476D1CE4E5B9ull;
            h = (h ^ (h >> 29) ^ m[1]) * 0xD6E8FEB86659FD93ull;
            hv = (hv ^ __builtin_bit_cast(unsigned long long, vv)) * 0x94D049BB133111EBull;
            hv ^= hv >> 31;
            if (u % 3 != 0 && om != oprev + 1) tri = false;
            oprev = om;
            omin = min(omin, om);
            omax = max(omax, om);
            ++u;
            if (in[0]) ++p[0];
            if (in[1]) ++p[1];
            if (__ballot((p[0] == DW_WIN && p[0] < rem[0]) || (p[1] == DW_WIN && p[1] < rem[1])) != 0) {
#pragma unroll
                for (int r = 0; r < 2; ++r) { a[r] += p[r]; rem[r] -= p[r]; p[r] = 0; }
                if (few && given_up()) { failed = true; break; }
                stage_rows(cwin[wv], col, a, rem, lane, range);
                staged = false; // the value window follows when it is next needed
            }
        }
        if (failed) break;
        if (cst) h ^= hv;
        const int slot = (int)((h ^ (h >> 32)) & (DIAG_TABLE - 1)); // wavefront-uniform
        if (slot != claimed) { // the first slice of a slot represents it
            if (lane == 0 && __hip_atomic_load(&table[slot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == -1)
                atomicCAS(&table[slot], -1, (int)s);
            claimed = slot;
        }
        if (lane < DIAG_PAD) de[mpos + u + lane] = DiagEnt{0.0, {0ull, 0ull}, 0, 0.0f};
        if (lane == 0) {
            // the loops read up to two elements past a record's rows
            const bool clamp = s128 + omin < 0 || s128 + DIAG_ROWS + 2 + omax >= n;
            ds[s].vpos = slot; // until the values are placed
            ds[s].mpos = mpos;
            ds[s].width = u;
            ds[s].flags = (cst ? DIAG_CONST : 0) | (clamp ? DIAG_CLAMP : 0) | (tri && u % 3 == 0 ? DIAG_TRI : 0);
            ulen[s] = cst ? 0 : 2 * u; // in 64-row units
        }
        tot += u;
        totv += cst ? 0 : u;
    }
    if (__ballot(cbad) != 0 && lane == 0) atomicOr(&info->flags, 1);
    if (lane == 0) {
        if (failed) atomicOr(&info->diag_fail, 1);
        if (tot) atomicAdd(&sums[0], tot);
        if (totv) atomicAdd(&sums[1], totv);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (sums[0]) atomicAdd(&info->diag_total, sums[0]);
        if (sums[1]) atomicAdd(&info->diag_values, sums[1]);
    }
}

// Pass 3: slices with the same records as their table slot's representative
// share its copy (most slices of a grid operator do), so the records a wavefront
// reads stay in the scalar cache. Without it every slice's 0.7 KB of records
// missed to HBM in dependent steps (160^3 27-point product, at one row per
// lane: 82 us against 70 us). A slot's representative keeps its own records (its slot holds itself).
__global__ void __launch_bounds__(256) k_diag_share(int nslices, const DiagEnt *__restrict__ de, DiagSlice *ds,
                                                    const int *__restrict__ table)
{
    const int lane = threadIdx.x & 63;
    const long long nwaves = ((long long)gridDim.x * blockDim.x) >> 6;
    for (long long s = ((long long)blockIdx.x * blockDim.x + threadIdx.x) >> 6; s < nslices; s += nwaves) {
        const int rep = table[ds[s].vpos];
        if (rep < 0 || rep == s) continue;
        const long long ma = ds[s].mpos, mb = ds[rep].mpos;
        const int width = ds[s].width;
        const bool cst = ds[s].flags & DIAG_CONST;
        bool same = ds[rep].width == width && (ds[rep].flags & DIAG_CONST) == (ds[s].flags & DIAG_CONST);
        for (int k = lane; same && k < width; k += 64) {
            const DiagEnt a = de[ma + k], b = de[mb + k];
            same = a.off == b.off && a.mask[0] == b.mask[0] && a.mask[1] == b.mask[1] &&
                   (!cst || __builtin_bit_cast(unsigned long long, a.v) == __builtin_bit_cast(unsigned long long, b.v));
        }
        if (__ballot(!same) == 0 && lane == 0) ds[s].mpos = mb;
    }
}

// Pass 4: the values of the slices that are not constant, in record order
// (lanes without the entry store 0; they are masked out of the chain).
template <typename TIN>
__global__ void __launch_bounds__(64 * DW_WAVES)
k_diag_fill(DiagCsr<TIN> one, const DiagCsr<TIN> *__restrict__ mats, int nmats, int nslices, const DiagEnt *__restrict__ de, const DiagSlice *__restrict__ ds, double *__restrict__ sval64,
            float *__restrict__ sval32)
{
    __shared__ TIN vwin[DW_WAVES][DIAG_ROWS * DW_PITCH];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const TIN *vw = vwin[wv] + 2 * lane * DW_PITCH;
    const long long step = (long long)gridDim.x * DW_WAVES;
    auto none = [](TIN) {};
    for (long long s = (long long)blockIdx.x * DW_WAVES + wv; s < nslices; s += step) {
        const DiagSlice S = ds[s];
        if (S.flags & DIAG_CONST) continue;
        const int width = __builtin_amdgcn_readfirstlane(S.width);
        const DiagCsr<TIN> M = matrix_of<2>(one, mats, nmats, s);
        const int n = M.n;
        const int *__restrict__ rp = M.rp;
        const TIN *__restrict__ val = M.val;
        const long long i = (s - M.slice0 / 2) * DIAG_ROWS + 2 * lane;
        int a[2], rem[2], p[2] = {0, 0};
        a[0] = i < n ? rp[i] : 0;
        a[1] = i + 1 < n ? rp[i + 1] : 0;
        rem[0] = i < n ? rp[i + 1] - a[0] : 0;
        rem[1] = i + 1 < n ? rp[i + 2] - a[1] : 0;
        stage_rows(vwin[wv], val, a, rem, lane, none);
        for (int u = 0; u < width; ++u) {
            double v[2];
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const bool in = (de[S.mpos + u].mask[r] >> lane) & 1ull;
                v[r] = in ? (double)vw[r * DW_PITCH + p[r]] : 0.0;
                if (in) ++p[r];
            }
            const long long at = S.vpos + (long long)DIAG_ROWS * u + 2 * lane;
            if (sval64) *(double2 *)(sval64 + at) = make_double2(v[0], v[1]);
            if (sval32) *(float2 *)(sval32 + at) = make_float2((float)v[0], (float)v[1]);
            if (__ballot((p[0] == DW_WIN && p[0] < rem[0]) || (p[1] == DW_WIN && p[1] < rem[1])) != 0) {
#pragma unroll
                for (int r = 0; r < 2; ++r) { a[r] += p[r]; rem[r] -= p[r]; p[r] = 0; }
                stage_rows(vwin[wv], val, a, rem, lane, none);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Launch functions

template <typename TIN>
hipError_t launch_row_widths(const DiagCsr<TIN> &one, const DiagCsr<TIN> *mats, int nmats, int nslices, bool sample, int *w,
                             int *table, DotInfo *info, hipStream_t s)
{
    if (nslices == 0) return hipSuccess;
    const int grid = (int)std::min<long long>(((long long)nslices + 3) / 4, 1024);
    if (sample) k_row_widths<TIN, true><<<grid, 256, 0, s>>>(one, mats, nmats, nslices, w, table, info);
    else k_row_widths<TIN, false><<<grid, 256, 0, s>>>(one, mats, nmats, nslices, w, table, info);
    return hipGetLastError();
}
hipError_t launch_scan_len(const int *len, int m, long long *out, int stride, bool total, hipStream_t s)
{
    if (m == 0) return hipSuccess;
    k_scan_len<<<(m + SCAN_TILE - 1) / SCAN_TILE, 1024, 0, s>>>(len, m, out, stride, total);
    return hipGetLastError();
}

template <typename TIN>
hipError_t launch_diag_align(const DiagCsr<TIN> &one, const DiagCsr<TIN> *mats, int nmats, int nslices, const long long *off,
                             DiagEnt *de, DiagSlice *ds, int *ulen, int *table, DotInfo *info, int max_stored, int num_cus,
                             hipStream_t s)
{
    if (nslices == 0) return hipSuccess;
    // three workgroups a CU: what their windows leave room for
    const int grid = (int)std::min<long long>(((long long)nslices + DW_WAVES - 1) / DW_WAVES, 3ll * num_cus);
    k_diag_align<TIN><<<grid, 64 * DW_WAVES, 0, s>>>(one, mats, nmats, nslices, off, de, ds, ulen, table, info, max_stored);
    return hipGetLastError();
}

hipError_t launch_diag_share(int nslices, const DiagEnt *de, DiagSlice *ds, const int *table, hipStream_t s)
{
    if (nslices == 0) return hipSuccess;
    k_diag_share<<<(int)std::min<long long>(((long long)nslices + 3) / 4, 4096), 256, 0, s>>>(nslices, de, ds, table);
    return hipGetLastError();
}

template <typename TIN>
hipError_t launch_diag_fill(const DiagCsr<TIN> &one, const DiagCsr<TIN> *mats, int nmats, int nslices, const DiagEnt *de,
                            const DiagSlice *ds, double *sval64, float *sval32, hipStream_t s)
{
    if (nslices == 0) return hipSuccess;
    const int grid = (int)std::min<long long>(((long long)nslices + DW_WAVES - 1) / DW_WAVES, 8192);
    k_diag_fill<TIN><<<grid, 64 * DW_WAVES, 0, s>>>(one, mats, nmats, nslices, de, ds, sval64, sval32);
    return hipGetLastError();
}

#define RPCG_DIAG_LAUNCHERS(TIN)                                                                                            \
    template hipError_t launch_row_widths<TIN>(const DiagCsr<TIN> &, const DiagCsr<TIN> *, int, int, bool, int *, int *,    \
                                               DotInfo *, hipStream_t);                                                     \
    template hipError_t launch_diag_align<TIN>(const DiagCsr<TIN> &, const DiagCsr<TIN> *, int, int, const long long *,     \
                                               DiagEnt *, DiagSlice *, int *, int *, DotInfo *, int, int, hipStream_t);     \
    template hipError_t launch_diag_fill<TIN>(const DiagCsr<TIN> &, const DiagCsr<TIN> *, int, int, const DiagEnt *,        \
                                              const DiagSlice *, double *, float *, hipStream_t);
RPCG_DIAG_LAUNCHERS(double)
RPCG_DIAG_LAUNCHERS(float)
#undef RPCG_DIAG_LAUNCHERS

} // namespace rpcg
