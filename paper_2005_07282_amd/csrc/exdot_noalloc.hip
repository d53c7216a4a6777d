// rpcg_exdot_noalloc: the dot product of rpcg_exdot for callers that cannot
// allocate device memory. The accumulator block, the workgroup sums of the plain
// mode and the call's record live in a file-scope device array instead of a
// context workspace; the kernel is that of rpcg_exdot.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>

#include "rpcg.h"
#include "context.hpp"
#include "kernels.hpp"

namespace {

using namespace rpcg;

constexpr int NA_GROUPS = RPCG_NOALLOC_MAX_GROUPS;
constexpr size_t NA_REC_BYTES = 256; // the record
constexpr int NA_WORDS = DOT_COPIES * DOT_PITCH;
constexpr size_t NA_BYTES = NA_REC_BYTES + NA_WORDS * sizeof(long long) + (size_t)NA_GROUPS * sizeof(double);

// One copy per GPU, held until the process ends. In host code this name is
// only a handle for hipGetSymbolAddress: kernels receive the address that
// call returns.
static __device__ __align__(256) unsigned char scratch[NA_BYTES];

constexpr int NA_MAX_DEVICES = 64;
struct DevScratch {
    std::once_flag once;
    hipError_t err = hipSuccess;
    unsigned char *ptr = nullptr; // device address of this GPU's copy of scratch
    int num_cus = 256;
};
DevScratch g_dev[NA_MAX_DEVICES];

// Address of the current device's array (looked up once per device, with the
// device current) and its compute-unit count.
hipError_t device_scratch(int dev, unsigned char **ptr, int *cus)
{
    DevScratch &d = g_dev[dev];
    std::call_once(d.once, [&d, dev]() {
        void *p = nullptr;
        d.err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (d.err == hipSuccess) d.ptr = (unsigned char *)p;
        int c = 0;
        if (hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && c > 0)
            d.num_cus = c;
    });
    *ptr = d.ptr;
    *cus = d.num_cus;
    return d.err;
}

// The accumulators must start at zero, whatever calls that overlapped have left
// behind; a fill kernel rather than a memset node, so that a captured graph
// replays it correctly.
__global__ void k_zero_words(unsigned long long *p, int words)
{
    for (int i = threadIdx.x; i < words; i += blockDim.x) p[i] = 0ull;
}

} // namespace

extern "C" int rpcg_exdot_noalloc(rpcg_mode mode_in, int64_t n, const double *x, const double *y, double *out,
                                  const rpcg_opts *opts, rpcg_result *res, void *stream)
{
    using namespace rpcg_host;
    const int mode = (int)mode_in;
    if (n < 0 || (n > 0 && (!x || !y)) || !out) return RPCG_ERR_INVALID;
    if (mode != MODE_PLAIN && mode != MODE_FPE && mode != MODE_EXBLAS) return RPCG_ERR_INVALID;
    rpcg_opts o;
    rpcg_opts_default(&o);
    if (opts) o = *opts;
    if (!valid_opts(o)) return RPCG_ERR_INVALID;
    if (o.grid_size > NA_GROUPS) return RPCG_ERR_INVALID; // more slots than the static array holds
    o.fpe_size = resolve_fpe_size(o.fpe_size, mode);
    int dev = 0;
    RPCG_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= NA_MAX_DEVICES) return RPCG_ERR_INVALID;
    unsigned char *base = nullptr;
    int cus = 256;
    RPCG_TRY(device_scratch(dev, &base, &cus));
    hipStream_t s = (hipStream_t)stream;

    // launch shape of rpcg_exdot, with the grid capped by the array
    LaunchCfg cfg;
    cfg.block = o.block_size ? o.block_size : 1024;
    cfg.grid = o.grid_size ? o.grid_size : exdot_grid(mode, n, cfg.block, cus);
    cfg.grid = std::min(cfg.grid, NA_GROUPS);
    cfg.early_exit = o.early_exit != 0;
    cfg.fpe_size = o.fpe_size;
    cfg.fallback = o.fpe_fallback != 0;
    cfg.xcd_parts = 1;
    cfg.stream = s;

    // layout of the array: record, accumulators, workgroup sums
    ExdotWs w;
    w.rec = res ? (unsigned long long *)base : nullptr;
    w.blk = (long long *)(base + NA_REC_BYTES);
    w.part = (double *)(base + NA_REC_BYTES + NA_WORDS * sizeof(long long));
    w.seq = 1;
    hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(256), 0, s, (unsigned long long *)w.blk, NA_WORDS);
    RPCG_TRY(hipGetLastError());
    RPCG_TRY(launch_exdot(mode, n, x, y, out, w, cfg));
    if (res) {
        std::memset(res, 0, sizeof(*res));
        unsigned long long rec[2];
        RPCG_TRY(hipMemcpyAsync(rec, w.rec, sizeof rec, hipMemcpyDeviceToHost, s));
        RPCG_TRY(hipStreamSynchronize(s));
        exdot_result(rec[0], rec[1], mode, cfg, res);
        return res->status;
    }
    return RPCG_OK;
}
