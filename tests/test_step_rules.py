"""Which lists' Adam steps run single-wave pieces, which LAMB steps keep small chunks (csrc/occupancy.hpp) and where LAMB's sums are added
up (csrc/meeting.hpp), compiled for the host: one element or chunk below and at each bound that the headers state."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
M = 1 << 20
LINE = -(-(288 << 20) // 14)                    # elements from which a step stores too much to write through

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "meeting.hpp"
#include "occupancy.hpp"

int main(int argc, char **argv)
{
    const auto n = [&](int k) { return strtoull(argv[k], nullptr, 10); };
    if (argc == 5) return printf("%d\n", ccf::lamb_keeps_small_chunks(n(1), (int)n(2), n(3) != 0, n(4) != 0)) < 0;
    if (argc == 4) return printf("%d\n", n(1) ? ccf::lamb_one_group_each((int64_t)n(2), (uint32_t)n(3)) : ccf::lamb_tallies((int64_t)n(2), (uint32_t)n(3))) < 0;
    printf("%d\n", ccf::list_in_pieces(n(1), n(2), (int)n(3), n(4) != 0, n(5) != 0));
    return 0;
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(MAIN)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I", os.path.join(ROOT, "paper_2105_05720_amd", "csrc"),
                           "-I", os.path.join(ROOT, "include"), "-o", str(d / "rules"), str(d / "rules.cpp")])
    return lambda *a: bool(int(subprocess.run([str(d / "rules")] + [str(int(x)) for x in a], capture_output=True, text=True, timeout=60, check=True).stdout))


@pytest.mark.parametrize("R,f32,small,beyond", [(1, 0, True, 128 * M), (8, 0, True, 128 * M), (9, 0, True, 0), (10, 0, True, 0), (11, 0, False, 0),
                                                (1, 1, True, 256 * M), (8, 1, True, 256 * M), (9, 1, False, 0)])
def test_lists_in_pieces(rule, R, f32, small, beyond):
    ask = lambda numel, missing=0, nothing_asked=True: rule(numel, -(-(numel + missing) // 1024), R, f32, nothing_asked)
    assert [ask(LINE - 1), ask(LINE), ask(64 * M - 1), ask(64 * M - 1, nothing_asked=False)] == [False, small, small, small]
    assert [ask(64 * M), ask((beyond or 65 * M) - 1), ask(beyond or 128 * M)] == [bool(beyond), bool(beyond), False]
    assert not ask(64 * M, nothing_asked=False) and not ask(100 * M, nothing_asked=False)
    assert [ask(32 * M, 4 * M), ask(32 * M, 4 * M + 1)] == [small, False]           # one chunk in eight short


@pytest.mark.parametrize("R,f32,list_to,tensor_to", [(1, 0, 88, 72), (2, 0, 88, 72), (3, 0, 80, 0), (7, 0, 80, 0), (8, 0, 0, 0), (16, 0, 0, 0),
                                                     (1, 1, 88, 72), (2, 1, 80, 0), (3, 1, 80, 0), (4, 1, 0, 0)])
def test_lamb_keeps_small_chunks(rule, R, f32, list_to, tensor_to):
    for one_tensor, to in ((0, list_to), (1, tensor_to)):
        assert [rule(n, R, f32, one_tensor) for n in (64 * M, (to or 65) * M - 1, (to or 65) * M)] == [to > 0, to > 0, False]


def test_where_lamb_adds_up(rule):
    tallies, one_group = (lambda chunks, most: rule(0, chunks, most)), (lambda chunks, most: rule(1, chunks, most))
    assert [tallies(*x) for x in ((599, 599), (600, 600), (600, 513), (600, 512), (32768, 32768), (32769, 32769))] == [False, True, True, False, True, False]
    assert [one_group(*x) for x in ((0, 0), (1, 1), (64, 64), (65, 65), (65, 64), (8192, 64), (8193, 64))] == [False, True, True, False, True, True, False]
