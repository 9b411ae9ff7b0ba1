"""Which cache policy each kernel family of a plan uses (csrc/cache_rules.hpp) and what the tuner tries (csrc/tuning.hpp),
compiled for the host: the bounds that the header states, one element below and at each of them."""
import os
import subprocess

import pytest

from paper_2105_05720_amd import binding as cc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
AUTO, STREAM, RESIDENT, THROUGH = cc.CC_CACHE_AUTO, cc.CC_CACHE_STREAMING, cc.CC_CACHE_RESIDENT, cc.CC_CACHE_WRITE_THROUGH
MIB = 1 << 20

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "cache_rules.hpp"

int main(int argc, char **argv)
{
    for (int i = 1; i + 4 < argc; i += 5) {
        const ccf::CachePolicies c = ccf::cache_policies(atoi(argv[i]), strtoull(argv[i + 1], nullptr, 10), atoi(argv[i + 2]), atoi(argv[i + 3]) != 0, atoi(argv[i + 4]) != 0);
        printf("%d %d %d\n", c.adam, c.lamb1, c.lamb);
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def policies(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(MAIN)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I", os.path.join(ROOT, "paper_2105_05720_amd", "csrc"),
                           "-I", os.path.join(ROOT, "include"), "-o", str(d / "rules"), str(d / "rules.cpp")])

    def ask(asked, numel, R, f32, one_sweep=True):
        out = subprocess.run([str(d / "rules")] + [str(int(x)) for x in (asked, numel, R, f32, one_sweep)], capture_output=True, text=True, timeout=60)
        return tuple(int(x) for x in out.stdout.split())
    return ask


def below_and_at(nbytes, per_element):
    n = -(-nbytes // per_element)
    return n - 1, n


@pytest.mark.parametrize("R,f32", [(1, False), (8, False), (16, False), (4, True)])
def test_automatic_policies_at_their_bounds(policies, R, f32):
    per = (4 if f32 else 2) * R + 26
    below, at = below_and_at(4 * MIB, per)
    assert policies(AUTO, below, R, f32) == (STREAM,) * 3
    assert policies(AUTO, at, R, f32) == (RESIDENT,) * 3
    below, at = below_and_at(200 * MIB, per)
    assert policies(AUTO, below, R, f32) == (RESIDENT,) * 3
    assert policies(AUTO, at, R, f32) == (THROUGH,) * 3
    below, at = below_and_at(288 * MIB, 14)                   # the Adam step's own stores, for a list as for one tensor
    assert [policies(AUTO, n, R, f32)[0] for n in (below, at)] == [THROUGH, STREAM]
    # LAMB writes both sweeps through until its first one stores 288 MiB, then the first only
    below, at = below_and_at(288 * MIB, 8)
    assert [policies(AUTO, n, R, f32)[1:] for n in (below, at)] == [(THROUGH, THROUGH), (THROUGH, STREAM)]
    assert policies(AUTO, 1 << 30, R, f32)[1:] == (THROUGH, STREAM)


@pytest.mark.parametrize("R,f32", [(1, False), (8, False), (16, False), (4, True)])
def test_the_unfused_pipelines(policies, R, f32):
    """Adam's goes by the 14 bytes per element that its update stores and changes at 20.6 Mi elements; what follows the reduce in
    LAMB's is written through at every size from 200 MiB of buffers on."""
    below, at = below_and_at(288 * MIB, 14)
    assert [policies(AUTO, n, R, f32)[:2] for n in (below, at)] == [(THROUGH, THROUGH), (STREAM, THROUGH)]
    below, at = below_and_at(288 * MIB, 8)
    assert [policies(AUTO, n, R, f32)[:2] for n in (below, at)] == [(STREAM, THROUGH), (STREAM, THROUGH)]


@pytest.mark.parametrize("R,f32", [(1, False), (8, False), (4, True)])
def test_chunks_of_several_sweeps_go_by_what_a_launch_stores(policies, R, f32):
    """Small chunks above 1024 elements: both of LAMB's sweeps alike."""
    below, at = below_and_at(288 * MIB, 14)
    assert [policies(AUTO, n, R, f32, False)[0] for n in (below, at)] == [THROUGH, STREAM]
    below, at = below_and_at(288 * MIB, 8)
    assert [policies(AUTO, n, R, f32, False)[1:] for n in (below, at)] == [(THROUGH, THROUGH), (STREAM, STREAM)]
    below, at = below_and_at(200 * MIB, (4 if f32 else 2) * R + 26)
    assert policies(AUTO, below, R, f32, False) == (RESIDENT,) * 3


def test_a_policy_that_was_asked_for_holds_everywhere(policies):
    for p in (STREAM, RESIDENT, THROUGH):
        for n in (100, 1 << 22, 1 << 25):
            assert policies(p, n, 8, False) == (p,) * 3


TUNER = r"""
#include <cstdio>
#include "cache_rules.hpp"
#include "tuning.hpp"

// Whatever AUTO gives an untuned plan's small chunks, some candidate gives them too.
int main()
{
    const std::vector<ccf::TuningLayout> layouts = {{1024, 5, true, false}, {4096, 2, false, true}, {16384, 1, false, false}};
    for (int optimizer : {0, 1})
        for (int32_t current : {1024, 4096, 16384}) {
            const auto cand = ccf::tuning_candidates(layouts, current, optimizer, 256);
            if (cand.empty() || cand[0].chunk_elems != current || cand[0].schedule != CC_SCHEDULE_PER_CHUNK || cand[0].cache != CC_CACHE_STREAMING) return 1;
            for (uint64_t numel : {1ull << 10, 1ull << 17, 1ull << 20, 5300000ull, 1ull << 23, 14000000ull, 1ull << 25, 42000000ull, 60000000ull})
                for (int R : {1, 8, 16}) {
                    const ccf::CachePolicies a = ccf::cache_policies(CC_CACHE_AUTO, numel, R, false, true);
                    int found = 0;
                    for (const auto &c : cand) {
                        const ccf::CachePolicies q = ccf::cache_policies(c.cache, numel, R, false, true);
                        if (c.chunk_elems != 1024 || c.schedule != CC_SCHEDULE_PER_CHUNK) continue;
                        found += optimizer == 0 ? q.adam == a.adam : q.lamb1 == a.lamb1 && q.lamb == a.lamb;
                    }
                    if (!found) { printf("optimizer %d, %llu elements, R = %d\n", optimizer, (unsigned long long)numel, R); return 2; }
                }
            int ordered = 0;
            for (const auto &c : cand) {
                if (c.schedule != CC_SCHEDULE_ORDERED) continue;
                ++ordered;
                if (c.chunk_elems != 4096 || (c.workgroups != 128 && c.workgroups != 256 && c.workgroups != 512)) return 3;
            }
            if (ordered != 3) return 4;
        }
    return 0;
}
"""


def test_the_tuner_tries_what_auto_would_choose(tmp_path):
    (tmp_path / "tuner.cpp").write_text(TUNER)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I", os.path.join(ROOT, "paper_2105_05720_amd", "csrc"),
                           "-I", os.path.join(ROOT, "include"), "-o", str(tmp_path / "tuner"), str(tmp_path / "tuner.cpp")])
    done = subprocess.run([str(tmp_path / "tuner")], capture_output=True, text=True, timeout=60)
    assert done.returncode == 0, "%d %s" % (done.returncode, done.stdout)
