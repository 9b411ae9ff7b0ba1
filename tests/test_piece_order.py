"""The order in which the workgroups of a grid take the pieces of a call (csrc/piece_order.hpp), compiled for the host:
every piece is taken exactly once, whatever the grid, and a round's XCD takes consecutive pieces; and the launches of a call
that is too large for one cover it without a gap."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = r"""
#include <cstdio>
#include <vector>
#include "piece_order.hpp"

int main()
{
    std::vector<uint32_t> grids;
    for (uint32_t g = 0; g <= 2600; ++g) grids.push_back(g);
    for (uint32_t g : {65535u, 65536u, 65537u, 1000003u}) grids.push_back(g);
    for (uint32_t g : grids) {
        std::vector<unsigned char> taken(g, 0);
        for (uint32_t b = 0; b < g; ++b) {
            const uint32_t p = ccf::piece_in_runs(b, g);
            if (p >= g || taken[p]++) { printf("grid %u: workgroup %u takes %u\n", g, b, p); return 1; }
        }
        for (uint32_t b = 0; b < g; ++b) {                       // runs of 32
            const uint32_t p = ccf::piece_in_runs<5>(b, g);
            if (p >= g || taken[p]++ != 1) { printf("grid %u, runs of 32: workgroup %u takes %u\n", g, b, p); return 1; }
        }
    }
    for (uint32_t x = 0; x < 8; ++x)                             // one XCD's workgroups b = x, x + 8, ... of the second round
        for (uint32_t k = 0; k < 64; ++k)
            if (ccf::piece_in_runs(512 + 8 * k + x, 1024) != 512 + 64 * x + k) { printf("XCD %u, %u\n", x, k); return 1; }
    const uint32_t most = 0x7fffffffu;                           // the largest grid a launch may have
    if (ccf::piece_in_runs(most - 1, most) != most - 1 || ccf::piece_in_runs(0, most) != 0) { printf("largest grid\n"); return 1; }
    for (uint64_t most : {1ull << 34, 512ull, 1024ull})
        for (uint64_t numel : {0ull, 1ull, 511ull, 512ull, 513ull, 1024ull, 1025ull, (1ull << 34) - 1, 1ull << 34, (1ull << 34) + 8, 1ull << 35, (1ull << 36) + 7}) {
            if (numel / most > 100000) continue;
            uint64_t next = 0;
            bool ok = true;
            ccf::in_launches(numel, most, [&](uint64_t at, uint64_t count) {
                const uint64_t threads = (count + 511) / 512 * 64;
                ok = ok && at == next && at % 512 == 0 && count > 0 && count <= most && threads < 1ull << 32;
                next = at + count;
            });
            if (!ok || next != numel) { printf("launches of %llu elements\n", (unsigned long long)numel); return 1; }
        }
    return 0;
}
"""


def test_every_piece_is_taken_once(tmp_path):
    src, exe = tmp_path / "order.cpp", tmp_path / "order"
    src.write_text(MAIN)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I", os.path.join(ROOT, "paper_2105_05720_amd", "csrc"),
                           "-o", str(exe), str(src)])
    done = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert done.returncode == 0, done.stdout
