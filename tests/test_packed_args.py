"""Kernel arguments in 96 bytes: what is taken comes out as it went in, what does not fit is refused."""
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "packed_args.hpp"
using namespace ccf;
static int epilogue(const uint64_t *v, int n)
{
    uint64_t base;
    uint32_t at[16];
    if (!pack_epilogue(v, n, &base, at)) return printf("-\n");
    for (int k = 0; k < n; ++k) printf("%llu ", (unsigned long long)unpack_address(base, at[k]));
    return printf("\n");
}
int main()
{
    char what;
    int R;
    while (scanf(" %c %d", &what, &R) == 2) {
        uint64_t v[32];
        const int n = what == 'a' ? 10 + R : 3 + R;
        for (int k = 0; k < n; ++k) { unsigned long long x; if (scanf("%llu", &x) != 1) return 1; v[k] = x; }
        if (what == 'e') {
            epilogue(v, n);
            continue;
        }
        // a: w_in .. w16, flag, scratch, numel, slices
        const uint64_t address[8] = {v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[10]};
        PackedAdam a;
        if (!pack_adam(address, v + 10, R, v[7], v[8], v[9], &a)) { printf("-\n"); continue; }
        for (int k = 0; k < 7; ++k) printf("%llu ", (unsigned long long)packed_at(a, k));
        printf("%llu %llu %llu ", (unsigned long long)packed_flag(a), (unsigned long long)a.scratch, (unsigned long long)a.numel);
        for (int r = 0; r < R; ++r) printf("%llu ", (unsigned long long)packed_slice(a, r));
        printf("\n");
    }
}
"""


@pytest.fixture(scope="module")
def pack(tmp_path_factory):
    d = tmp_path_factory.mktemp("packed")
    (d / "main.cpp").write_text(MAIN)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Wno-pedantic", "-I", os.path.join(ROOT, "paper_2105_05720_amd", "csrc"),
                           "-I", os.path.join(ROOT, "include"), "-o", str(d / "main"), str(d / "main.cpp")])

    def run(cases):
        text = "\n".join("%s %d %s" % (w, R, " ".join(map(str, v))) for w, R, v in cases)
        out = subprocess.run([str(d / "main")], input=text, capture_output=True, text=True, timeout=60, check=True).stdout.splitlines()
        assert len(out) == len(cases)
        return [None if line == "-" else [int(x) for x in line.split()] for line in out]
    return run


FAR = 16 * (2**32 - 1)                  # the furthest a buffer may lie above the lowest, 64 GiB - 16


def test_adam(pack):
    rng, cases, want = random.Random(5), [], []
    for R in (1, 2, 3, 8, 16):
        for _ in range(40):
            base = rng.randrange(1, 1 << 43) * 16
            state = [base + rng.randrange(FAR // 16 + 1) * 16 for _ in range(7)]
            lowest, stride = min(state), 16 * rng.randrange(-(1 << 20), 1 << 20)
            slices = [lowest + (1 << 28) + 16 * 7 + r * stride for r in range(R)]
            flag = lowest + rng.randrange(0, 1 << 36, 4)
            v = state + [flag, rng.randrange(1 << 47), rng.randrange(1, 1 << 26)] + slices
            cases.append(("a", R, v))
            want.append(v)
    assert pack(cases) == want


def test_adam_at_the_edges(pack):
    b = 1 << 40
    good = [b + 16 * k for k in range(7)] + [b + 160, 1, 5, b + 1024, b + 2048, b + 3072]
    def but(**kw):
        v = list(good)
        for k, x in kw.items():
            v[int(k[1:])] = x
        return ("a", 3, v)
    cases = [but(), but(_0=b + FAR), but(_0=b + 16 + FAR, _7=b + FAR + 12), but(_7=b + 4), but(_7=b - 4), but(_9=2**32 - 2**16),
             but(_11=b + 1024, _12=b + 1024), but(_10=b + (1 << 36) - 1024, _11=b + (1 << 35), _12=b + 1024)]
    got = pack(cases)
    assert got[0] == good and [x is not None for x in got] == [True, True, True, True, True, True, True, True]
    assert all(x == c[2] for x, c in zip(got, cases))
    assert pack([but(_0=b + FAR + 32), but(_7=b + FAR + 16), but(_7=b - 4, _0=b + FAR), but(_9=2**32 - 2**16 + 1), but(_12=b + 3088), but(_11=b + 2048 + 16),
                 but(_11=b + 1024 + 2**31 * 16, _12=b + 1024 + 2**32 * 16)]) == [None] * 7


def test_epilogue(pack):
    rng, cases = random.Random(6), []
    for R in (1, 8, 9):
        for _ in range(40):
            base = rng.randrange(1 << 43) * 16
            cases.append(("e", R, [base] + [base + rng.randrange(FAR // 16 + 1) * 16 for _ in range(R + 2)]))
    assert pack(cases) == [v for _, _, v in cases]
    b = 1 << 40
    assert pack([("e", 8, [b] * 10 + [b + FAR]), ("e", 8, [b] * 10 + [b + FAR + 16]), ("e", 1, [b + FAR + 16, b, b, b])])[1:] == [None] * 2
