"""LAMB's per-tensor sums added up in its two sweeps, from 600 to 32768 chunks, against the launch of their own that adds them up for the
unfused pipeline: the same additions in the same order, so the same bits."""
import numpy as np
import pytest
import torch

from paper_2105_05720_amd import binding as cc
from paper_2105_05720_amd.launches import launches
from paper_2105_05720_amd.shard import Shard

pytestmark = pytest.mark.gpu
K = 1024


def _filled(numels, R, **kw):
    shard = Shard(numels, [0.01] * len(numels), R, align_elems=8, unfused=True, **kw)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(len(numels) + R)
    shard.w[0].normal_(0, 0.02, generator=gen)
    shard.m[0].normal_(0, 1e-3, generator=gen)
    shard.v[0].uniform_(0, 1e-6, generator=gen)
    for g in shard.grads:
        g.copy_(torch.empty(g.numel(), device="cuda").normal_(0, 1e-3, generator=gen))
    return shard


@pytest.mark.parametrize("numels,tallied,kw", [
    ([600 * K], True, {}),                                        # the smallest: ten groups, the last of 24 chunks
    ([600 * K - K], False, {}),                                   # one chunk less
    ([K * K], True, {}),                                          # one row of 1024 chunks, sixteen whole groups
    ([K * K + 1], True, {}),                                      # a second row of one chunk
    ([3 * K * K + 70 * K + 5], True, {}),                         # a group of four rows, one of three and a part, others of three
    ([5 * K * K + 3], True, {}),                                  # a block of four rows and one
    ([32768 * K], True, {}),                                      # the largest
    ([32768 * K + 1], False, {}),                                 # one chunk more
    ([1000 * K, 7, 64 * K, 65 * K + 1] + [3] * 700, True, {}),    # groups of one tensor only, tensors of one chunk
    ([0, 1100 * K, 0], False, {}),                                # tensors without a chunk, whose sums are zero
    ([3 * K * K], True, {"chunk_elems": 2048}),
    ([2 * K * K + 9, 700], True, {"grad_dtype": torch.float32}),
    ([9 * K * K + 333], True, {}),                                # non-temporal loads, runs
])
def test_sums_are_those_of_the_launch_of_its_own(numels, tallied, kw):
    shard = _filled(numels, 2, **kw)
    plan = shard.plans[0]
    hp = cc.Hyper(step=3)
    ran = [x.kernel for x in launches(lambda: cc.cc_fused_lamb_step(plan, hp, shard.flag))]
    assert ran == ["lamb_phase1_kernel"] + ["lamb_norms_kernel"] * (not tallied) + ["lamb_phase2_kernel"]
    cc.cc_unfused_lamb_step(plan, hp, shard.flag)
    want = np.asarray(cc.cc_lamb_norms_read(plan, len(numels)))
    assert [bool(x) for x in want[:, 0]] == [n > 0 for n in numels]
    w_want, w16_want = shard.w[1].clone(), shard.w16[1].clone()
    for _ in range(3):                                      # the counts go on from launch to launch
        cc.cc_fused_adam_step(plan, hp, shard.flag)         # other launches that count arrivals, and overwrite the moments
        cc.cc_fused_lamb_step(plan, hp, shard.flag)
        got = np.asarray(cc.cc_lamb_norms_read(plan, len(numels)))
        assert np.array_equal(got, want)
    cc.cc_fused_lamb_step(plan, hp, shard.flag)
    assert int(shard.flag.item()) == 0
    for k in range(len(numels)):
        assert torch.equal(shard.view(shard.w[1], k), shard.view(w_want, k)) and torch.equal(shard.view(shard.w16[1], k), shard.view(w16_want, k))
    shard.view(shard.grads[1], 0 if numels[0] else 1)[-1] = float("inf")
    shard.w[1].fill_(7.0)
    cc.cc_fused_lamb_step(plan, hp, shard.flag)             # nothing of w is written when the last element overflows
    assert int(shard.flag.item()) == 1 and bool((shard.w[1] == 7.0).all())
    shard.destroy()


@pytest.mark.parametrize("numels,own,kw", [
    ([1], True, {}),
    ([64 * K], True, {}),                                         # one whole group
    ([64 * K + 1], False, {}),                                    # two
    ([5, 63 * K + 7, K, 64 * K, 1] * 40, True, {}),
    ([3] * 8192, True, {}),                                       # the most
    ([3] * 8193, False, {}),
    ([70 * K, 0, 9], False, {}),
    ([30 * K, 0, 9], False, {}),                                  # an empty tensor's zeros are written by the launch
    ([128 * K], True, {"chunk_elems": 2048}),
    ([4 * K + 3, 50], False, {"chunk_elems": 4096}),              # workgroups of 512 threads
])
def test_sums_of_the_first_phase_call(numels, own, kw):
    shard = _filled(numels, 3, **kw)
    plan, hp = shard.plans[0], cc.Hyper(step=3)

    def phases():
        cc.cc_fused_lamb_phase1(plan, hp, shard.flag)
        cc.cc_fused_lamb_phase2(plan, hp, shard.flag)
    assert [x.kernel for x in launches(phases)] == ["lamb_phase1_kernel"] + ["lamb_norms_kernel"] * (not own) + ["lamb_phase2_kernel"]
    cc.cc_unfused_lamb_step(plan, hp, shard.flag)
    want, w_want = np.asarray(cc.cc_lamb_norms_read(plan, len(numels))), shard.w[1].clone()
    for _ in range(2):
        cc.cc_fused_adam_step(plan, hp, shard.flag)
        cc.cc_fused_lamb_phase1(plan, hp, shard.flag)
        assert np.array_equal(np.asarray(cc.cc_lamb_norms_read(plan, len(numels))), want)
        cc.cc_fused_lamb_phase2(plan, hp, shard.flag)
        assert torch.equal(shard.w[1], w_want) and int(shard.flag.item()) == 0
    shard.destroy()


@pytest.mark.parametrize("numels,phases", [([700 * K + 1], False), ([64 * K, 5, 2 * K], True)])
def test_replays_of_a_captured_step(numels, phases):
    """A graph of two steps, replayed with other work and eager steps in between: each replay's result is the eager one."""
    shard = _filled(numels, 2)
    plan, hp = shard.plans[0], cc.Hyper(step=3)

    def step():
        if not phases:
            return cc.cc_fused_lamb_step(plan, hp, shard.flag)
        cc.cc_fused_lamb_phase1(plan, hp, shard.flag)
        cc.cc_fused_lamb_phase2(plan, hp, shard.flag)
    step()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        step()
        step()
    for k in range(5):
        shard.grads[0].mul_(1.25)
        shard.w[1].fill_(7.0)
        step()
        want = shard.w[1].clone()
        sums = np.asarray(cc.cc_lamb_norms_read(plan, len(numels)))
        shard.w[1].fill_(7.0)
        graph.replay()
        assert torch.equal(shard.w[1], want) and int(shard.flag.item()) == 0
        assert np.array_equal(np.asarray(cc.cc_lamb_norms_read(plan, len(numels))), sums)
    shard.destroy()
