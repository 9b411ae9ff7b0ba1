"""How many workgroups of the fused Adam kernels a compute unit holds on shards bound by HBM (csrc/occupancy.hpp), compiled for
the host: the bounds that the header states, at and beside each of them."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MIB = 1 << 20

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "occupancy.hpp"

int main(int, char **argv)
{
    if (argv[5][0] == 'p') return printf("%d\n", ccf::flat_beyond_small(strtoull(argv[1], nullptr, 10), atoi(argv[2]), atoi(argv[3]) != 0) ? 10000 : 20000) < 0;
    const auto rule = argv[5][0] == 'l' ? ccf::list_lds : ccf::flat_lds;
    printf("%u\n", rule(strtoull(argv[1], nullptr, 10), atoi(argv[2]), atoi(argv[3]) != 0, atoi(argv[4]) != 0));
    return 0;
}
"""


@pytest.fixture(scope="module")
def per_cu(tmp_path_factory):
    """Workgroups per compute unit of 160 KiB LDS."""
    d = tmp_path_factory.mktemp("occupancy")
    (d / "rules.cpp").write_text(MAIN)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I", os.path.join(ROOT, "paper_2105_05720_amd", "csrc"),
                           "-I", os.path.join(ROOT, "include"), "-o", str(d / "rules"), str(d / "rules.cpp")])

    def ask(*args, rule="list"):
        lds = int(subprocess.run([str(d / "rules")] + [str(int(x)) for x in args] + [rule], capture_output=True, text=True, timeout=60, check=True).stdout)
        assert 0 < lds < 64 * 1024                                       # what a launch may ask for without an attribute
        return 160 * 1024 // lds
    return ask


def test_lists(per_cu):
    large = -(-288 * MIB // 14)                                          # from here on the stores are non-temporal
    for R, f32, n in [(1, 0, 6), (8, 0, 6), (9, 0, 4), (16, 0, 4), (4, 1, 6), (5, 1, 4), (8, 1, 4), (9, 1, 3), (16, 1, 3)]:
        assert [per_cu(k, R, f32, nt) for k, nt in ((large - 1, 1), (large, 1), (1 << 26, 1))] == [6, n, n], (R, f32)
        assert per_cu(large, R, f32, 0) == 6                             # written through because the caller asked for it


@pytest.mark.parametrize("R,f32,through,streamed", [(1, 0, 16, 16), (2, 0, 15, 15), (4, 0, 13, 13), (6, 0, 12, 11), (8, 0, 12, 10), (12, 0, 12, 10),
                                                    (13, 0, 10, 10), (16, 0, 10, 10), (4, 1, 10, 10), (16, 1, 10, 10)])
def test_one_tensor(per_cu, R, f32, through, streamed):
    at = -(-300 * MIB // ((4 if f32 else 2) * R + 26))
    assert [per_cu(n, R, f32, nt, rule="flat") for nt in (0, 1) for n in (at - 1, at, 1 << 26)] == [16, through, through, 16, streamed, streamed]


@pytest.mark.parametrize("R,f32,sizes", [(1, 0, [0, 1, 1, 0, 0, 0, 0, 0]), (2, 0, [0, 1, 1, 1, 1, 0, 0, 0]), (10, 0, [0, 1, 1, 1, 1, 0, 0, 0]),
                                         (11, 0, [0] * 8), (16, 0, [0] * 8), (1, 1, [0, 1, 1, 1, 1, 0, 0, 0]), (3, 1, [0, 1, 1, 1, 1, 0, 0, 0]),
                                         (4, 1, [0, 1, 1, 1, 1, 1, 1, 0]), (16, 1, [0, 1, 1, 1, 1, 1, 1, 0])])
def test_pieces_on_one_large_tensor(per_cu, R, f32, sizes):
    """Only where the measured pairs show a gain: not from eleven fp16 slices on, and up to 144 Mi elements with one."""
    at = ((64 << 20) - 1, 64 << 20, (144 << 20) - 1, 144 << 20, (192 << 20) - 1, 192 << 20, 1 << 33, (1 << 33) + 1)
    assert [per_cu(n, R, f32, 0, rule="pieces") == 16 for n in at] == [bool(k) for k in sizes]
