"""How a launch's waves agree on the overflow flag (csrc/flag_word.hpp), compiled for the host: the last arrival and up to two waves
that report, before or after their stores, in every order of their accesses to the two words.  The kernels' FlagCount runs these two functions; a
wave that has lost words of LAMB's tally reports through the second one as well."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <vector>
#include <ucontext.h>
#include "flag_word.hpp"

// Coroutines that hand over in front of every access.
static unsigned long long state;
static int flag, running;
static ucontext_t home, self[3];
static char stacks[3][65536];
static bool done[3];
static std::function<void()> body[3];
static void step() { swapcontext(&self[running], &home); }
struct Words {
    unsigned long long read() const { step(); return state; }
    unsigned long long exchange(unsigned long long x) const { step(); const unsigned long long was = state; state = x; return was; }
    bool replace(unsigned long long &cur, unsigned long long x) const { step(); if (state != cur) { cur = state; return false; } state = x; return true; }
    void raise() const { step(); flag = 1; }
};
static void enter() { body[running](); done[running] = true; swapcontext(&self[running], &home); }

int main(int, char **argv)
{
    const int reporters = atoi(argv[1]), plain = atoi(argv[2]);
    const uint32_t tag = 7;
    body[0] = [&] { step(); flag = 0; ccf::flag_cleared(Words{}, tag); };
    for (int r = 1; r <= reporters; ++r) body[r] = [&] { if (plain) Words{}.raise(); else ccf::flag_report(Words{}, tag); };
    long orders = 0, wrong = 0;
    for (unsigned long long before : {0ull, ccf::state_of(tag - 1, ccf::kStateCleared), ccf::state_of(tag - 1, ccf::kStateBad)})
        for (int held = 0; held < 2; ++held) {
            std::vector<int> choice;                                    // whose turn, depth first over all of them
            do {
                state = before; flag = held;
                for (int p = 0; p <= reporters; ++p) {
                    done[p] = false;
                    getcontext(&self[p]);
                    self[p].uc_stack.ss_sp = stacks[p]; self[p].uc_stack.ss_size = sizeof(stacks[p]); self[p].uc_link = nullptr;
                    makecontext(&self[p], enter, 0);
                }
                for (size_t at = 0;; ++at) {
                    if (at == choice.size()) choice.push_back(0);
                    while (choice[at] <= reporters && done[choice[at]]) ++choice[at];
                    if (choice[at] > reporters) { choice.resize(at); break; }
                    running = choice[at];
                    swapcontext(&home, &self[running]);
                }
                bool all = true;
                for (int p = 0; p <= reporters; ++p) all = all && done[p];
                orders += all;                                          // (else nobody was left for the last turn that was tried)
                wrong += all && flag != (reporters > 0);
                while (!choice.empty()) {                               // the next order that differs
                    if (++choice.back() <= reporters) break;
                    choice.pop_back();
                }
            } while (!choice.empty());
        }
    return printf("%ld %ld\n", orders, wrong) < 0;
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    d = tmp_path_factory.mktemp("flag_word")
    (d / "walk.cpp").write_text(MAIN)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I", os.path.join(ROOT, "paper_2105_05720_amd", "csrc"), "-o", str(d / "walk"), str(d / "walk.cpp")])
    return lambda *a: [int(x) for x in subprocess.run([str(d / "walk")] + [str(x) for x in a], capture_output=True, text=True, timeout=60, check=True).stdout.split()]


@pytest.mark.parametrize("reporters,least", [(0, 1), (1, 20), (2, 500)])
def test_the_flag_is_one_exactly_if_somebody_reports(walk, reporters, least):
    orders, wrong = walk(reporters, 0)
    assert orders >= 6 * least and wrong == 0


def test_a_plain_store_would_be_lost(walk):
    assert walk(1, 1)[1] > 0


def test_the_tally_does_not_store_into_the_flag():
    """Whoever adds up a group has no way to the flag but FlagCount's."""
    with open(os.path.join(ROOT, "paper_2105_05720_amd", "csrc", "kernels.hip.h")) as f:
        text = f.read()
    body = text[text.index("bool tally_group("):]
    assert "flag" not in body[:body.index("\n}\n")]
    assert "!tally_group(ty, wh, tag) && fc.counting_lane()) fc.report(fs, flag);" in text
