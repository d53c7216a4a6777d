// Schedules of the batched solver's streaming kernels: the default and the
// autotuner's candidates. Host code without device or runtime headers.
#pragma once

#include <vector>

#include "rpcg.h"

namespace rpcg_host {

// A batch of nsys systems with `slices` slices of 64 rows in all. Two workgroups of 512
// threads a CU where they have work for it (64 systems of 16^3 to 96^3: 115 ms;
// 121 ms with 256 threads; 4 of 60^3 to 70^3: 13.0 ms against 14.7 ms with one), one
// for small batches (60 of 16^3 to 30^3: 4.9 ms against 5.3 ms). Small systems take a workgroup
// each, one wavefront or two, as many as a CU holds: in a larger one most wavefronts have
// no slice and the systems queue (us an iteration with 512 threads and with this: 4096 systems of 4^3 179 and 38,
// 4096 of 6^3 133 and 60, 3000 of 8^3 112 and 64, 1024 of 10^3 62 and 48, 512 of 14^3 60 and 59).
inline rpcg_batch_tuning default_tuning(int num_cus, long long slices, int nsys)
{
    rpcg_batch_tuning t{};
    t.policy = 0;
    t.tile_slices = 16;
    t.graph_iterations = 8;
    if (slices <= 8ll * nsys) {
        t.block_size = 64;
        t.grid_size = 16 * num_cus;
    } else if (slices < 48ll * nsys) {
        t.block_size = 128;
        t.grid_size = 4 * num_cus;
    } else {
        t.block_size = 512;
        t.grid_size = (slices >= 32ll * 2 * num_cus ? 2 : 1) * num_cus;
    }
    return t;
}

// What the autotuner tries: the default first, so that tuning never keeps less.
inline std::vector<rpcg_batch_tuning> tuning_candidates(const rpcg_batch_tuning &dflt, int num_cus, int graph_iterations)
{
    std::vector<rpcg_batch_tuning> cand;
    auto mk = [&](int policy, int tile, int grid, int block) {
        for (const rpcg_batch_tuning &c : cand)
            if (c.policy == policy && c.grid_size == grid && c.block_size == block && (policy == 0 || c.tile_slices == tile))
                return;
        rpcg_batch_tuning t{};
        t.policy = policy;
        t.tile_slices = tile;
        t.grid_size = grid;
        t.block_size = block;
        t.graph_iterations = graph_iterations;
        cand.push_back(t);
    };
    mk(dflt.policy, dflt.tile_slices, dflt.grid_size, dflt.block_size);
    mk(0, 16, num_cus, 256);
    mk(0, 16, 2 * num_cus, 256);
    mk(0, 16, 4 * num_cus, 256);
    mk(0, 16, 2 * num_cus, 512);
    mk(0, 16, num_cus, 1024);
    mk(1, 16, 2 * num_cus, 256);
    mk(1, 64, 2 * num_cus, 256);
    mk(1, 256, num_cus, 512);
    return cand;
}

} // namespace rpcg_host
