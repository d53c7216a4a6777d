// Host-side context of the C-ABI (private to the library): device
// workspace owned by an rpcg_ctx, and the small helpers every entry point uses.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cstdint>
#include <map>
#include <vector>

#include "rpcg.h"
#include "kernels.hpp"

namespace rpcg_host {

struct Buffer {
    void *p = nullptr;
    size_t bytes = 0;
    hipError_t ensure(size_t need)
    {
        if (need <= bytes) return hipSuccess;
        if (p) { hipError_t e = hipFree(p); if (e != hipSuccess) return e; p = nullptr; bytes = 0; }
        hipError_t e = hipMalloc(&p, need);
        if (e == hipSuccess) bytes = need;
        return e;
    }
    void release()
    {
        if (p) (void)hipFree(p); // teardown: nothing to report to
        p = nullptr;
        bytes = 0;
    }
};

// Accumulator blocks of the standalone dot that the calls on a context take in turn.
constexpr unsigned DOT_BLOCKS = 16;

} // namespace rpcg_host

struct rpcg_ctx {
    int device = 0;
    int num_cus = 256;
    int ws_groups = 0;        // capacity of the dot workspaces, in workgroups
    rpcg_host::Buffer ws_mem; // 3 dot workspaces, the refinement's slots
    rpcg::DotWs ws[3];
    rpcg::SlotWs slots{};
    rpcg_host::Buffer scalars; // DotInfo + PcgState + IrState
    rpcg::DotInfo *info = nullptr;
    rpcg::PcgState *st = nullptr;
    rpcg::IrState *ist = nullptr;
    rpcg_host::Buffer sell_off, sell_val, sell_val32, sell_col, sell_cfirst, sell_len, diag_ds, diag_de;
    rpcg_host::Buffer widths;  // construction scratch: table of record lists, then one int per slice
    rpcg_host::Buffer vecs;    // r, z, d, w, dinv of the solver
    rpcg_host::Buffer ir_vecs; // refinement: r (binary64), rf and c (binary32)
    rpcg_host::Buffer beta_hist; // beta of every iteration
    int *host_done = nullptr;  // pinned: polled flags
    rpcg::PcgState *host_state = nullptr;
    rpcg::IrState *host_ir = nullptr;
    rpcg_host::Buffer dot_blocks; // DOT_BLOCKS accumulator blocks of the standalone dot, empty between calls
    unsigned long long *host_dot = nullptr; // pinned: a record of two words per block
    unsigned dot_seq = 0;
    rpcg::DotInfo *host_info = nullptr; // and, behind it, one long long (construction total)
    std::vector<hipEvent_t> events;
    std::vector<hipEvent_t> ir_events;
    hipEvent_t poll_ev[2] = {nullptr, nullptr};
    std::map<uint64_t, rpcg_batch_tuning> batch_tunings; // autotuner results by batch signature
};

static_assert(sizeof(rpcg::DotInfo) <= 256 && sizeof(rpcg::PcgState) <= 256 && sizeof(rpcg::IrState) <= 256,
              "scalar layout");

namespace rpcg_host {

inline int hip_status(hipError_t e)
{
    if (e == hipSuccess) return RPCG_OK;
    if (e == hipErrorOutOfMemory) return RPCG_ERR_OOM;
    return RPCG_ERR_HIP;
}

#define RPCG_TRY(expr)                                          \
    do {                                                        \
        hipError_t _e = (expr);                                 \
        if (_e != hipSuccess) return rpcg_host::hip_status(_e); \
    } while (0)

inline bool valid_opts(const rpcg_opts &o)
{
    using rpcg::MAX_BLOCK;
    using rpcg::MAX_FPE;
    if (!(o.tol >= 0.0) || o.maxit < 0) return false;
    if (o.fpe_size < 0 || o.fpe_size > MAX_FPE) return false;
    if (o.block_size != 0 && (o.block_size < 64 || o.block_size > MAX_BLOCK || o.block_size % 64)) return false;
    if (o.grid_size < 0 || o.grid_size > 65536) return false;
    if (o.xcd_parts < 0 || o.xcd_parts > 64) return false;
    if (o.spmv_block_size != 0 && (o.spmv_block_size < 64 || o.spmv_block_size > MAX_BLOCK || o.spmv_block_size % 64))
        return false;
    if (o.spmv_grid_size < 0 || o.spmv_grid_size > 65536) return false;
    if (o.timing < 0 || o.timing > 65) return false;
    return true;
}

inline bool valid_csr(const rpcg_csr *A)
{
    if (!A || A->n < 0 || A->nnz < 0) return false;
    if (A->n > 0 && (!A->row_ptr || (A->nnz > 0 && (!A->col_idx || !A->val)))) return false;
    return true;
}

// Expansion length: 0 = auto. FPE mode: 4. EXBLAS mode: 3 (its results do
// not depend on the length; 3 was the fastest on the 27-point workload).
inline int resolve_fpe_size(int p, int mode)
{
    if (p) return p;
    return mode == rpcg::MODE_EXBLAS ? 3 : 4;
}

// Workgroups (of `block` threads) of a standalone dot. Plain: eight elements a
// thread, at most eight workgroups per CU. The exact modes: one workgroup up to
// EXDOT_ALONE elements (it needs no atomics and no tickets); then four elements
// a thread up to one workgroup per CU, as each costs the accumulator's setup and
// partial (2^20 pairs: 11.9 us on 256 workgroups, 13.9 us on 128, 14.3 us on 512). More per
// CU from so many elements a thread on (us for narrow, +-30 and +-200 binades):
// EXBLAS two from 32 (2^24 pairs 49, 76, 51 on 256, 53, 69, 52 on 512), three from 512 (2^27 pairs
// 359, 504, 371 on 512, 364, 469, 368 on 768; 2^28 720, 1017, 728 and 712, 950, 724; the next pairs
// are prefetched). FPE two from 512, as every workgroup pays the merges of its wavefronts'
// expansions and every lane its first measurement window (2^22 pairs 19, 34, 46 on 256, 23,
// 42, 57 on 512; 2^26 168, 235, 255 and 184, 227, 281; 2^27 332, 454, 514 and 352, 435, 453), four from
// 1024 (2^28 pairs 705, 856, 902 on 512, 761, 845, 866 on 1024).
constexpr int64_t EXDOT_ALONE = 8192;
inline int exdot_grid(int mode, int64_t n, int block, int cus)
{
    if (mode == rpcg::MODE_PLAIN)
        return (int)std::max<int64_t>(1, std::min<int64_t>((n + 8ll * block - 1) / (8ll * block), 8ll * cus));
    if (n <= EXDOT_ALONE) return 1;
    const int64_t each = n / ((int64_t)cus * block); // elements a thread, with one workgroup per CU
    const int64_t per_cu = mode == rpcg::MODE_FPE ? (each >= 1024 ? 4 : (each >= 512 ? 2 : 1))
                                                  : (each >= 512 ? 3 : (each >= 32 ? 2 : 1));
    return (int)std::max<int64_t>(1, std::min<int64_t>((n + 4ll * block - 1) / (4ll * block), per_cu * cus));
}

// A standalone dot's result record from the kernel's two words.
inline void exdot_result(unsigned long long rec0, unsigned long long rec1, int mode, const rpcg::LaunchCfg &cfg,
                         rpcg_result *res)
{
    const unsigned flags = (unsigned)rec1;
    res->fpe_escapes = (int64_t)rec0;
    res->fallbacks = mode == rpcg::MODE_FPE && rec0 > 0 && cfg.fallback ? 1 : 0;
    res->grid_size = cfg.grid;
    res->block_size = cfg.block;
    if (flags & rpcg::FLAG_NONFINITE) res->status = RPCG_ERR_NONFINITE;
    else if (flags & rpcg::FLAG_INEXACT) res->status = RPCG_WARN_FPE_INEXACT;
    else if (mode == rpcg::MODE_FPE && rec0 > 0 && !cfg.fallback) res->status = RPCG_WARN_FPE_INEXACT;
    else res->status = RPCG_OK;
}

// Timing events between solver kernels. They carry no system-scope fence:
// the kernels' results stay on the device, and a fence per event would write
// back the caches between kernels and slow the timed loop.
inline int ensure_events(std::vector<hipEvent_t> &evs, size_t need)
{
    while (evs.size() < need) {
        hipEvent_t e;
        RPCG_TRY(hipEventCreateWithFlags(&e, hipEventDisableSystemFence));
        evs.push_back(e);
    }
    return RPCG_OK;
}

inline double ms_since(std::chrono::steady_clock::time_point t)
{
    return std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t).count();
}

} // namespace rpcg_host
