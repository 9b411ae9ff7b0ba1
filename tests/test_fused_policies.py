"""What the fused steps' launches use where AUTO says RESIDENT (fused_policies in csrc/cache_rules.hpp), compiled for the host: one element
below and at each bound that the header states."""
import os
import subprocess

import pytest

from paper_2105_05720_amd import binding as cc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
AUTO, RESIDENT, THROUGH, KEPT = cc.CC_CACHE_AUTO, cc.CC_CACHE_RESIDENT, cc.CC_CACHE_WRITE_THROUGH, 16
MIB = 1 << 20

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "cache_rules.hpp"
#include "tuning.hpp"

int main(int argc, char **argv)
{
    if (argc == 2) {                     // how many candidates choose nothing at all
        const std::vector<ccf::TuningLayout> layouts = {{1024, 5, true, false}, {4096, 2, false, true}, {16384, 1, false, false}};
        int n = 0;
        for (const auto &c : ccf::tuning_candidates(layouts, 4096, atoi(argv[1]), 256))
            n += c.chunk_elems == 0 && c.schedule == CC_SCHEDULE_AUTO && c.workgroups == 0 && c.cache == CC_CACHE_AUTO;
        return printf("%d\n", n) < 0;
    }
    const int asked = atoi(argv[1]), R = atoi(argv[3]);
    const uint64_t numel = strtoull(argv[2], nullptr, 10);
    const bool f32 = atoi(argv[4]) != 0, one_sweep = atoi(argv[5]) != 0;
    const ccf::CachePolicies c = ccf::fused_policies(ccf::cache_policies(asked, numel, R, f32, one_sweep), asked, numel, R, f32, one_sweep);
    if (argc > 6) return printf("%d\n", c.slices_plain) < 0;
    return printf("%d %d %d\n", c.adam, c.lamb1, c.lamb) < 0;
}
"""


@pytest.fixture(scope="module")
def policies(tmp_path_factory):
    d = tmp_path_factory.mktemp("fused")
    (d / "rules.cpp").write_text(MAIN)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I", os.path.join(ROOT, "paper_2105_05720_amd", "csrc"),
                           "-I", os.path.join(ROOT, "include"), "-o", str(d / "rules"), str(d / "rules.cpp")])

    def ask(asked, numel=None, R=None, f32=None, one_sweep=True, more=()):
        out = subprocess.run([str(d / "rules")] + [str(int(x)) for x in ((asked,) if numel is None else (asked, numel, R, f32, one_sweep, *more))], capture_output=True, text=True, timeout=60, check=True)
        return tuple(int(x) for x in out.stdout.split())
    return ask


@pytest.mark.parametrize("R,f32", [(1, False), (8, False), (16, False), (4, True), (16, True)])
def test_from_80_to_200_mib(policies, R, f32):
    per = (4 if f32 else 2) * R + 26
    at, end = -(-80 * MIB // per), -(-200 * MIB // per)
    again = -(-32 * MIB // 12)                                   # elements whose w, m' and v' fill the L2s
    assert policies(AUTO, at - 1, R, f32) == (RESIDENT,) * 3
    for n in {at, end - 1, again - 1, again}:
        if at <= n < end:
            assert policies(AUTO, n, R, f32) == (THROUGH, KEPT, RESIDENT if n < again else THROUGH)
    assert policies(AUTO, end, R, f32) == (THROUGH,) * 3
    assert policies(AUTO, end - 1, R, f32, one_sweep=False) == (RESIDENT,) * 3
    for asked in (cc.CC_CACHE_STREAMING, RESIDENT, THROUGH):
        assert policies(asked, end - 1, R, f32) == (asked,) * 3


@pytest.mark.parametrize("R,f32,kept", [(1, False, True), (2, False, True), (3, False, False), (8, False, False), (1, True, True), (2, True, False)])
def test_few_slices_are_read_plainly_up_to_144_mib(policies, R, f32, kept):
    per = (4 if f32 else 2) * R + 26
    at, end = -(-80 * MIB // per), -(-144 * MIB // per)
    ask = lambda asked, n, **kw: bool(policies(asked, n, R, f32, more=(1,), **kw)[0])
    assert [ask(AUTO, n) for n in (at - 1, at, end - 1, end)] == [False, kept, kept, False]
    assert not ask(AUTO, at, one_sweep=False) and not any(ask(p, at) for p in (cc.CC_CACHE_STREAMING, RESIDENT, THROUGH))


@pytest.mark.parametrize("optimizer", [0, 1])
def test_the_tuner_tries_a_plan_for_which_nothing_is_chosen(policies, optimizer):
    """No policy that is asked for reads few slices plainly and the state not: of the tuner's candidates only this one does."""
    assert policies(optimizer) == (1,)
