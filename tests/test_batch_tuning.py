"""The autotuner tries the schedule that a batch gets without it, whatever the
sizes (host code, compiled here): otherwise tuning could keep a slower one."""

import os
import subprocess


ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = r"""
#include "batch_tuning.hpp"
#include <cstdio>
using namespace rpcg_host;
int main()
{
    for (int cus : {32, 256, 304})
        for (int nsys : {1, 4, 60, 64, 512, 4096, 100000})
            for (long long per : {1ll, 2ll, 8ll, 9ll, 47ll, 48ll, 64ll, 3000ll, 100000ll}) {
                const long long slices = per * nsys;
                const rpcg_batch_tuning d = default_tuning(cus, slices, nsys);
                const auto cand = tuning_candidates(d, cus, 5);
                int same = 0, twice = 0, valid = 1;
                for (size_t a = 0; a < cand.size(); ++a) {
                    const rpcg_batch_tuning &c = cand[a];
                    same += c.policy == d.policy && c.grid_size == d.grid_size && c.block_size == d.block_size;
                    for (size_t b = 0; b < a; ++b)
                        twice += c.policy == cand[b].policy && c.tile_slices == cand[b].tile_slices &&
                                 c.grid_size == cand[b].grid_size && c.block_size == cand[b].block_size;
                    valid = valid && c.graph_iterations == 5 && c.grid_size >= 1 && c.grid_size <= 65536 && c.tile_slices >= 1 &&
                            c.block_size >= 64 && c.block_size <= 1024 && c.block_size % 64 == 0;
                }
                std::printf("%d %lld %d %d %d %d\n", cus, slices, nsys, same, twice, valid);
            }
}
"""


def test_the_default_is_a_candidate(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(MAIN)
    r = subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"), "-I",
                        os.path.join(ROOT, "paper_2005_07282_amd", "csrc"), str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    lines = subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split("\n")[:-1]
    assert len(lines) == 3 * 7 * 9
    for line in lines:
        cus, slices, nsys, same, twice, valid = map(int, line.split())
        assert same == 1 and twice == 0 and valid == 1, line


def test_small_systems_get_a_workgroup_each(tmp_path):
    """Workgroups of one or two wavefronts where a system has no slices for more."""
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(r"""
#include "batch_tuning.hpp"
#include <cstdio>
int main()
{
    for (long long per : {1ll, 2ll, 8ll, 16ll, 43ll, 64ll, 1000ll}) {
        const rpcg_batch_tuning d = rpcg_host::default_tuning(256, per * 4096, 4096);
        std::printf("%lld %d %d\n", per, d.block_size, d.grid_size);
    }
}
""")
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2005_07282_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    got = [tuple(map(int, x.split())) for x in subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split("\n")[:-1]]
    for per, block, grid in got:
        assert block // 64 <= max(1, per) and block * grid >= 256 * 512, (per, block, grid)
