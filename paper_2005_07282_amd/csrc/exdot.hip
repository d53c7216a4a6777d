// Standalone dot product kernels (exact, expansion-based and plain), the
// rounding of a long accumulator, and the CSR SpMV.
#include "reduce.hpp"
#include "sell_spmv.hpp"

#include <algorithm>

namespace rpcg {

// ---------------------------------------------------------------------------
// Standalone dot product in one launch. Each workgroup adds the words of its
// exact partial into one of DOT_COPIES accumulators with device-scope integer
// atomics and takes a ticket once they are complete; the workgroup that takes
// the last one sums the copies, rounds and leaves the block empty for the next
// call. Nothing but those atomics, and loads and stores at their level, passes
// between workgroups, so no fence writes back a cache (a device-scope fence
// before each ticket had cost 2 to 14 times the whole dot). The tickets are in two levels: a thousand
// workgroups that end together would otherwise queue on one address.
// A call on one workgroup needs neither atomics nor tickets.
// What bounds it: HBM from about 2^26 pairs on in the exact mode, for narrow and
// wide exponents alike (2^26 pairs 188 and 222 -> 185 and 189 us, 5.7 TB/s), and in FPE mode
// for narrow ones (198 -> 172 us, 6.2 TB/s); FPE over +-200 binades is bound by
// its expansions and the LDS adds of what escapes them (285 -> 258 us, 4.2 TB/s; 2^28 pairs 890 -> 880 us,
// 4.9 TB/s). The next pairs are prefetched and the streamed loads marked non-temporal
// (2^26 narrow 199 us without the mark). Short calls are latency: 10007 pairs took a memset, two
// kernels of 8.3 and 7.2 us and a copy, and take one kernel of 9.6 us.

constexpr int EX_COPIES = 4;
constexpr int EX_PITCH = ACC_DIGITS; // 136 dwords: copies 8 banks apart
constexpr int EX_ONE_LEVEL = 64;     // workgroups up to which the tickets take one level (one round trip less)
// 16-byte pairs of each vector a thread loads together. FPE: one, as its two
// expansions and two pairs (with the next two in flight) took 76 registers and left one 1024-thread
// workgroup a CU (four terms, 59 registers now; us for narrow, +-30 and +-200 binades: 2^24 pairs
// 61, 95, 134 -> 48, 76, 125, 2^28 pairs 772, 928, 976 -> 705, 856, 902).
template <int MODE>
constexpr int ex_unroll() { return MODE == MODE_FPE ? 1 : 2; }

__device__ __forceinline__ long long coherent_ll(const long long *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Every vector memory operation of this wavefront, atomics included, has completed.
__device__ __forceinline__ void wait_vmem() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// EXBLAS mode: spread (in binades) of the products' exponents over a wavefront's
// first loads above which its lanes start in the direct mode, as the
// expansions of the default length would soon overflow. There it moves work
// between two exact paths that nobody can tell apart. In FPE mode what goes direct counts as
// escaped, so a lane goes direct only once its own expansions have kept overflowing.
constexpr int EX_WIDE = 128;

__device__ __forceinline__ void exponent_span(double x, double y, int &lo, int &hi)
{
    const int ex = (int)((__builtin_bit_cast(unsigned long long, x) >> 52) & 0x7FF);
    const int ey = (int)((__builtin_bit_cast(unsigned long long, y) >> 52) & 0x7FF);
    if (ex && ey) {
        lo = min(lo, ex + ey);
        hi = max(hi, ex + ey);
    }
}

// blk: DOT_COPIES x DOT_PITCH words, empty (words 68 and 69: tickets, 70:
// escapes, 71: flags); part: [gridDim.x] (plain). Writes *out, or with
// digits_out the exact sum as normalized words; rec (may be null): rec[0]
// the escapes, then rec[1] = seq << 32 | flags, at system scope, as the last action of the call.
template <int MODE, int P>
__global__ void __launch_bounds__(MAX_BLOCK)
k_exdot(long long n, const double *__restrict__ x, const double *__restrict__ y, long long *blk, double *part,
        double *out, long long *digits_out, unsigned long long *rec, unsigned seq, bool ee, bool capture)
{
    __shared__ RedShared sh;
    // lanes add into one of EX_COPIES copies of the long accumulator by
    // lane & (EX_COPIES - 1), so lanes that hit the same word in the same
    // instruction mostly hit different addresses (copies EX_PITCH words
    // apart start in different LDS banks); summed into copy 0 at the end
    __shared__ long long accx[EX_COPIES - 1][EX_PITCH];
    long long *acc = sh.acc[0];
    const long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long stride = (long long)gridDim.x * blockDim.x;
    constexpr int EX_UNROLL = ex_unroll<MODE>();
    typedef pair_t<double> pr; // 16-byte loads at any 8-byte alignment
    const long long n2 = n >> 1;
    pr a[EX_UNROLL], b[EX_UNROLL];
    // past the end nothing is loaded and the pair keeps what it held (it is not used)
    auto load = [&](long long i) {
#pragma unroll
        for (int u = 0; u < EX_UNROLL; ++u) {
            const long long j = i + u * stride;
            if (j < n2) {
                a[u] = __builtin_nontemporal_load((const pr *)(x + 2 * j));
                b[u] = __builtin_nontemporal_load((const pr *)(y + 2 * j));
            }
        }
    };
    long long i = tid;
    load(i);
    zero_acc(acc);
    for (int q = threadIdx.x; q < (EX_COPIES - 1) * EX_PITCH; q += blockDim.x) (&accx[0][0])[q] = 0;
    __syncthreads();
    const int cp = threadIdx.x & (EX_COPIES - 1);
    long long *accl = cp ? accx[cp - 1] : acc;

    LaneDot<MODE, P, MODE != MODE_PLAIN> L;
    L.init();
    if constexpr (MODE == MODE_EXBLAS) {
        int lo = 1 << 20, hi = -1;
        if (i < n2) {
            exponent_span(a[0].x, b[0].x, lo, hi);
            exponent_span(a[0].y, b[0].y, lo, hi);
        }
        if (wave_minmax_i32_all<true>(hi) - wave_minmax_i32_all<false>(lo) > EX_WIDE) L.direct = ADAPT_DIRECT;
    }
    while (i < n2) {
        pr ca[EX_UNROLL], cb[EX_UNROLL];
#pragma unroll
        for (int u = 0; u < EX_UNROLL; ++u) { ca[u] = a[u]; cb[u] = b[u]; }
        const long long i0 = i;
        i += EX_UNROLL * stride;
        load(i); // in flight while the current pairs are accumulated
#pragma unroll
        for (int u = 0; u < EX_UNROLL; ++u)
            if (u == 0 || i0 + u * stride < n2) {
                L.add(ca[u].x, cb[u].x, accl, ee, capture);
                L.add(ca[u].y, cb[u].y, accl, ee, capture);
            }
    }
    if ((n & 1) && tid == 0) L.add(x[n - 1], y[n - 1], accl, ee, capture);

    // the workgroup's partial
    const bool alone = gridDim.x == 1;
    if constexpr (MODE == MODE_PLAIN) {
        const double t = block_sum_d(L.s, sh);
        if (threadIdx.x == 0) {
            if (alone) sh.val[0] = t;
            else __hip_atomic_store(&part[blockIdx.x], t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    } else {
        if constexpr (MODE == MODE_EXBLAS) {
            wave_flush_exact<P>(L.a, accl, L.flags);
        } else {
            L.esc += fpe_sum_capture<P>(L.a, L.e, ee, capture, accl, L.flags);
            wave_fpe_finish<P>(L.a, L.esc, ee, capture, accl, L.flags);
        }
        if (threadIdx.x == 0) { sh.flag = 0; sh.red_ll[0] = 0; }
        __syncthreads();
        if (L.flags) atomicOr(&sh.flag, L.flags);
        if constexpr (MODE == MODE_FPE) {
            const long long esc = wave_sum_i64_all(L.esc);
            if (lane_id() == 0 && esc) atomicAdd((unsigned long long *)&sh.red_ll[0], (unsigned long long)esc);
        }
        for (int q = threadIdx.x; q < ACC_DIGITS; q += blockDim.x) {
            long long v = acc[q];
#pragma unroll
            for (int c = 0; c < EX_COPIES - 1; ++c) v += accx[c][q];
            acc[q] = v;
        }
        __syncthreads();
        if (!alone) {
            long long *copy = blk + (blockIdx.x % DOT_COPIES) * DOT_PITCH;
            auto add = [](long long *p, long long v) {
                __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            };
            for (int k = threadIdx.x; k < ACC_DIGITS; k += blockDim.x) {
                // one carry step keeps every word below 2^33 in magnitude, so the
                // integer sum over the workgroups cannot overflow
                const long long v = acc[k], cin = k ? (acc[k - 1] >> 32) : 0;
                const long long o = (k == ACC_DIGITS - 1) ? v + cin : (v & 0xFFFFFFFFll) + cin;
                if (o != 0) add(&copy[k], o);
            }
            if (threadIdx.x == 0) {
                if (sh.red_ll[0]) add(&blk[DOT_ESC], sh.red_ll[0]);
                if (sh.flag) __hip_atomic_fetch_or(&blk[DOT_ESC + 1], (long long)sh.flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
    if (!alone) {
        wait_vmem();
        __syncthreads();
        if (threadIdx.x == 0) {
            const int G = gridDim.x, g = blockIdx.x % DOT_COPIES;
            auto ticket = [](long long *p) { return __hip_atomic_fetch_add(p, 1ll, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
            bool last = true;
            if (G > EX_ONE_LEVEL) last = ticket(&blk[g * DOT_PITCH + ACC_DIGITS]) == (G - g + DOT_COPIES - 1) / DOT_COPIES - 1;
            if (last) last = ticket(&blk[ACC_DIGITS + 1]) == (G > EX_ONE_LEVEL ? DOT_COPIES : G) - 1;
            sh.rng[0] = last;
        }
        __syncthreads();
        if (!sh.rng[0]) return;
    } else {
        __syncthreads();
    }
    if (wave_id() != 0) return;

    // the finishing wavefront
    const int l = lane_id();
    long long da = 0, db = 0, esc = 0;
    int flags = 0;
    double r = 0.0;
    if constexpr (MODE == MODE_PLAIN) {
        if (alone) {
            r = sh.val[0];
        } else { // fixed order: lane-strided sums of the workgroups, then the tree
            const int G = gridDim.x;
            double s[4] = {0.0, 0.0, 0.0, 0.0};
            auto at = [&](int g) { return __hip_atomic_load(&part[g], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
            int g = l;
            for (; g + 3 * 64 < G; g += 4 * 64) {
#pragma unroll
                for (int j = 0; j < 4; ++j) s[j] += at(g + 64 * j);
            }
            for (; g < G; g += 64) s[0] += at(g);
            r = __shfl(wave_sum_down((s[0] + s[1]) + (s[2] + s[3])), 0, 64);
        }
    } else {
        if (alone) {
            if (2 * l < ACC_DIGITS) { da = acc[2 * l]; db = acc[2 * l + 1]; }
            esc = sh.red_ll[0];
            flags = sh.flag;
        } else if (l < DOT_PITCH / 2) {
            long long q[DOT_COPIES][2];
#pragma unroll
            for (int c = 0; c < DOT_COPIES; ++c) {
                q[c][0] = coherent_ll(&blk[c * DOT_PITCH + 2 * l]);
                q[c][1] = coherent_ll(&blk[c * DOT_PITCH + 2 * l + 1]);
            }
#pragma unroll
            for (int c = 0; c < DOT_COPIES; ++c) { da += q[c][0]; db += q[c][1]; }
        }
        if (!alone) {
            esc = wave_i64_of(da, DOT_ESC / 2);
            flags = (int)wave_i64_of(db, DOT_ESC / 2);
            if (l > TOP_LANE) da = db = 0;
        }
        if (digits_out) {
            wave_normalize(da, db);
            if (2 * l < ACC_DIGITS) {
                digits_out[2 * l] = da;
                digits_out[2 * l + 1] = db;
            }
        } else {
            r = wave_round<double>(da, db);
        }
    }
    if (!alone) { // empty the block again
        for (int k = l; k < DOT_COPIES * DOT_PITCH; k += 64)
            __hip_atomic_store(&blk[k], 0ll, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (l == 0 && out)
        __hip_atomic_store(out, (flags & FLAG_NONFINITE) ? __builtin_nan("") : r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (rec) {
        if (l == 0) __hip_atomic_store(&rec[0], (unsigned long long)esc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        wait_vmem(); // the result and the empty block are in place before the caller may go on
        if (l == 0)
            __hip_atomic_store(&rec[1], ((unsigned long long)seq << 32) | (unsigned)flags, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

__global__ void k_acc_round(const long long *digits, double *out)
{
    __shared__ long long acc[ACC_DIGITS];
    for (int k = threadIdx.x; k < ACC_DIGITS; k += blockDim.x) acc[k] = digits[k];
    __syncthreads();
    double r = wave_acc_round(acc);
    if (threadIdx.x == 0) *out = r;
}

// ---------------------------------------------------------------------------
// SpMV on CSR (Section 4.3): y_i = fold over the stored entries of row i, in
// storage order, of acc = fma(a_ik, x[col_k], acc), acc from +0.
//
// A workgroup owns R consecutive rows (one per thread); their entries
// form one contiguous range of the CSR arrays. The range is staged through
// LDS in chunks of E entries: consecutive threads load consecutive
// values and columns (coalesced, streamed once) and gather the x entries;
// then every thread continues its own row's fma chain over the part of the
// row inside the chunk, reading LDS. The accumulator stays in the row's
// thread across chunks, so a row of any length is one sequential chain in
// storage order, exactly as the definition reads.
// The next chunk's values and columns are loaded under the current chunk's
// chains and its x entries gathered right after them, so rows longer than a
// chunk's share no longer leave the memory idle while their chains run.

constexpr int SPMV_E = 2048; // chunk of entries staged at a time

template <int R, int E>
__global__ void __launch_bounds__(R)
k_spmv_csr(int n, const int *__restrict__ rp, const int *__restrict__ col, const double *__restrict__ val,
           const double *__restrict__ x, double *__restrict__ y)
{
    constexpr int PER = E / R; // entries each thread stages per chunk
    static_assert(E % R == 0, "chunk shape");
    __shared__ double2 st[E]; // (a_k, x[col_k]) of the chunk's entries
    const int t = threadIdx.x;
    for (long long r0 = (long long)blockIdx.x * R; r0 < n; r0 += (long long)gridDim.x * R) {
        const long long r1 = r0 + R < n ? r0 + R : n;
        const long long i = r0 + t;
        const long long b0 = rp[r0], b1 = rp[r1];
        long long rs = b1, re = b1;
        if (i < r1) { rs = rp[i]; re = rp[i + 1]; }
        double acc = 0.0;
        double a[PER], g[PER];
        int c[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const long long k = b0 + j * R + t;
            const bool in = k < b1;
            a[j] = in ? __builtin_nontemporal_load(val + k) : 0.0;
            c[j] = in ? __builtin_nontemporal_load(col + k) : 0;
        }
#pragma unroll
        for (int j = 0; j < PER; ++j) g[j] = x[c[j]];
        for (long long k0 = b0; k0 < b1; k0 += E) {
            if (k0 != b0) __syncthreads(); // the previous chunk has been read
#pragma unroll
            for (int j = 0; j < PER; ++j) st[j * R + t] = make_double2(a[j], g[j]);
            __syncthreads();
            const long long k1 = k0 + E;
            if (k1 < b1) { // the next chunk's values and columns, loaded under this chunk's chains
#pragma unroll
                for (int j = 0; j < PER; ++j) {
                    const long long k = k1 + j * R + t;
                    const bool in = k < b1;
                    a[j] = in ? __builtin_nontemporal_load(val + k) : 0.0;
                    c[j] = in ? __builtin_nontemporal_load(col + k) : 0;
                }
            }
            const int lo = (int)((rs > k0 ? rs : k0) - k0);
            const int hi = (int)((re < k0 + E ? re : k0 + E) - k0);
            int k = lo;
            for (; k + 4 <= hi; k += 4) {
                const double2 e0 = st[k], e1 = st[k + 1], e2 = st[k + 2], e3 = st[k + 3];
                acc = __builtin_fma(e0.x, e0.y, acc);
                acc = __builtin_fma(e1.x, e1.y, acc);
                acc = __builtin_fma(e2.x, e2.y, acc);
                acc = __builtin_fma(e3.x, e3.y, acc);
            }
            for (; k < hi; ++k) acc = __builtin_fma(st[k].x, st[k].y, acc);
            if (k1 < b1) {
#pragma unroll
                for (int j = 0; j < PER; ++j) g[j] = x[c[j]];
            }
        }
        if (i < r1) y[i] = acc;
        __syncthreads(); // the next block's first chunk overwrites st
    }
}

// ---------------------------------------------------------------------------
// Launch functions

hipError_t launch_exdot(int mode, long long n, const double *x, const double *y, double *out, const ExdotWs &w,
                        const LaunchCfg &c)
{
    dispatch(mode, c.fpe_size, [&](auto m, auto p) {
        constexpr int M = decltype(m)::value, PP = decltype(p)::value;
        k_exdot<M, PP><<<c.grid, c.block, 0, c.stream>>>(n, x, y, w.blk, w.part, out, nullptr, w.rec, w.seq, c.early_exit,
                                                         c.fallback);
    });
    return hipGetLastError();
}

hipError_t launch_exdot_partial(long long n, const double *x, const double *y, long long *digits, const ExdotWs &w,
                                const LaunchCfg &c)
{
    k_exdot<MODE_EXBLAS, 4><<<c.grid, c.block, 0, c.stream>>>(n, x, y, w.blk, w.part, nullptr, digits, nullptr, 0, true, true);
    return hipGetLastError();
}

hipError_t launch_acc_round(const long long *digits, double *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_acc_round, dim3(1), dim3(64), 0, s, digits, out);
    return hipGetLastError();
}

hipError_t launch_spmv_csr(int n, long long nnz, const int *row_ptr, const int *col, const double *val,
                           const double *x, double *y, int num_cus, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    auto run = [&](auto rows) {
        constexpr int R = decltype(rows)::value;
        const unsigned g = (unsigned)std::min<long long>(((long long)n + R - 1) / R, 65536);
        // short rows (under 32 entries on average) fill a chunk with many rows:
        // half-size chunks keep more workgroups per CU (measured 160^3: 0.58
        // against 0.56 of 8 TB/s); long rows need the full chunk
        if (nnz < 32ll * n)
            hipLaunchKernelGGL((k_spmv_csr<R, SPMV_E / 2>), dim3(g), dim3(R), 0, s, n, row_ptr, col, val, x, y);
        else
            hipLaunchKernelGGL((k_spmv_csr<R, SPMV_E>), dim3(g), dim3(R), 0, s, n, row_ptr, col, val, x, y);
    };
    // Rows per workgroup: the most that leave enough workgroups for every CU. A
    // workgroup's entries come chunk after chunk, each behind the last one's
    // latency, so a matrix that is cut into few workgroups waits on them with the
    // memory idle (us with 512 rows everywhere, and now: 201-wide band of 20 k rows 203
    // and 41, of 100 k 188 and 72, of 200 k 204 and 131; 27 points on 22 k rows 15.0 and 6.4,
    // on 64 k 16.4 and 7.7, on 216 k 20.1 and 16.7). Large matrices keep 512: 4.1 M
    // rows of 27 points 272 us against 282 us with 256, the band of 1 M rows 504 and 524 us.
    if (n >= 512ll * 3 * num_cus) run(std::integral_constant<int, 512>{});
    else if (n >= 256ll * 2 * num_cus) run(std::integral_constant<int, 256>{});
    else if (n >= 128ll * 2 * num_cus) run(std::integral_constant<int, 128>{});
    else run(std::integral_constant<int, 64>{});
    return hipGetLastError();
}

// Smallest and largest binary exponent (floor(log2 |v|)) over the nonzero
// finite entries of v; *emin / *emax are lowered / raised atomically.
__global__ void k_exp_range(long long n, const double *__restrict__ v, int *emin, int *emax)
{
    int lo = 1 << 20, hi = -(1 << 20);
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
        const unsigned long long b = __builtin_bit_cast(unsigned long long, v[i]) & 0x7FFFFFFFFFFFFFFFull;
        if (b == 0 || (b >> 52) == 0x7FF) continue;
        const int be = (int)(b >> 52);
        const int e = be ? be - 1023 : (63 - __builtin_clzll(b)) - 1074;
        lo = min(lo, e);
        hi = max(hi, e);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        lo = min(lo, __shfl_xor(lo, off, 64));
        hi = max(hi, __shfl_xor(hi, off, 64));
    }
    if ((threadIdx.x & 63) == 0) {
        atomicMin(emin, lo);
        atomicMax(emax, hi);
    }
}

hipError_t launch_exp_range(long long n, const double *v, int *emin, int *emax, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const int grid = (int)std::min<long long>((n + 255) / 256, 2048);
    hipLaunchKernelGGL(k_exp_range, dim3(grid), dim3(256), 0, s, n, v, emin, emax);
    return hipGetLastError();
}

} // namespace rpcg
