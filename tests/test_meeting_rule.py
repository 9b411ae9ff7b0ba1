"""Which LAMB steps are one launch, and which workgroups make room (csrc/meeting.hpp), compiled for the host."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "meeting.hpp"

int main(int argc, char **argv)
{
    if (argv[1][0] == 's') { for (int b = 0; b < atoi(argv[2]); ++b) putchar('0' + ccf::meeting_stays((uint32_t)b)); return 0; }
    for (int i = 2; i + 4 < argc; i += 5)
        printf("%d ", ccf::lamb_meets(atoll(argv[i]), (uint32_t)atoi(argv[i + 1]), atoi(argv[i + 2]), atoi(argv[i + 3]), atoi(argv[i + 4]) != 0));
    return 0;
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("meeting")
    (d / "rule.cpp").write_text(MAIN)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I", os.path.join(ROOT, "paper_2105_05720_amd", "csrc"),
                           "-I", os.path.join(ROOT, "include"), "-o", str(d / "rule"), str(d / "rule.cpp")])
    return lambda *a: subprocess.run([str(d / "rule")] + [str(int(x)) if not isinstance(x, str) else x for x in a], capture_output=True, text=True, timeout=60).stdout


@pytest.mark.parametrize("R,f32,most", [(1, 0, 512), (4, 0, 512), (5, 0, 384), (7, 0, 384), (8, 0, 256), (16, 0, 256),
                                        (1, 1, 512), (8, 1, 512), (9, 1, 384), (12, 1, 384), (13, 1, 256), (16, 1, 256)])
def test_four_such_steps_fit_the_device(rule, R, f32, most):
    """At most a quarter of the workgroups that the device holds at a time: 256 compute units, and a partition of 32."""
    ask = lambda *cases: [int(x) for x in rule("r", *[v for c in cases for v in c]).split()]
    assert ask((0, 0, 256, R, f32), (1, 1, 256, R, f32), (most, 8, 256, R, f32), (most + 1, 9, 256, R, f32)) == [0, 1, 1, 0]
    assert ask((most // 8, 1, 32, R, f32), (most // 8 + 1, 2, 32, R, f32)) == [1, 0]
    assert ask((64, 64, 256, R, f32), (65, 65, 256, R, f32)) == [1, 0]


def test_on_every_part_of_the_device_some_make_room(rule):
    """Workgroups are dealt out in turn to XCDs, shader engines and compute units: of any eight in a row, or 2^k apart, three to five stay."""
    stays = [int(c) for c in rule("s", 512)]
    for step in (1, 2, 4, 8, 16, 32):
        for first in range(512 - 7 * step):
            assert 3 <= sum(stays[first + i * step] for i in range(8)) <= 5
