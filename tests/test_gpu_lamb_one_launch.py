"""LAMB steps of few chunks (256 to 512, by what the kernel's registers leave room for) run as one launch in which the workgroups
wait for each other's norms.

Against the two phase calls (separate launches, same additions in the same order): sums, state and flag bit for bit, with
every wave patient and with none (a limit of 0 polls: whoever does not find all norms at once leaves its part of w to the last
workgroup that started) and with some of both, with and without an overflow, and against the oracle.  Sizes at the edges: one element, less than a
pack, around a chunk, 64 and 65 chunks (sums by
chunk and by group of 64), 256, 384 and 512 (the most, by the slices) and one more, lists with empty, tiny and ragged tensors, 64 groups (the most) and 65."""
import statistics

import numpy as np
import pytest
import torch

import oracle
from paper_2105_05720_amd import binding as cc
from paper_2105_05720_amd.launches import launches
from paper_2105_05720_amd.shard import Shard
from parity import OracleState, compare_committed, hyper_pair, seeded_grads, seeded_state

pytestmark = pytest.mark.gpu

LISTS = [[1], [3], [1023], [1024], [1027], [10007], [64 * 1024], [64 * 1024 + 1],
         [5, 0, 1024, 4099, 1, 2048, 7], [1] * 64, [20 * 1024 + 2, 42 * 1024 + 1, 1],
         [129 * 1024 - 3], [1 << 18], [(1 << 18) + 1], [1 << 19], [(1 << 19) + 1], [5, 0, 100 * 1024 + 3, 1, 64 * 1024, 300001], [1] * 61 + [192 * 1024], [1] * 62 + [192 * 1024]]


def _phases(plan, hp, flag, stream=None):
    cc.cc_fused_lamb_phase1(plan, hp, flag, stream)
    cc.cc_fused_lamb_phase2(plan, hp, flag, stream)


FORMS = [(8, torch.float16, cc.CC_CACHE_AUTO), (1, torch.float32, cc.CC_CACHE_AUTO),
         (3, torch.float16, cc.CC_CACHE_WRITE_THROUGH), (16, torch.float32, cc.CC_CACHE_RESIDENT)]


def _name(n):
    return "x".join(map(str, n[:4])) + ("_%d" % len(n))


@pytest.mark.parametrize("limit", [None, 0])
@pytest.mark.parametrize("numels", LISTS, ids=_name)
@pytest.mark.parametrize("R,dtype,policy", FORMS)
def test_one_launch_gives_the_bits_of_the_two_phases(numels, R, dtype, policy, limit):
    _compare_with_phases(numels, R, dtype, policy, limit)


@pytest.mark.parametrize("limit", [1, 3, 6, 12])
@pytest.mark.parametrize("numels", [[10007], [64 * 1024], [20 * 1024 + 2, 42 * 1024 + 1, 1], [1 << 18], [5, 0, 100 * 1024 + 3, 1, 64 * 1024]], ids=_name)
@pytest.mark.parametrize("R,dtype,policy", [FORMS[0], FORMS[1]])
def test_some_leave_and_some_stay(numels, R, dtype, policy, limit):
    """About as many looks as a wave needs anyway: some waves write their own part, some leave, some that stay take those over."""
    _compare_with_phases(numels, R, dtype, policy, limit)


def _compare_with_phases(numels, R, dtype, policy, limit):
    wds = [0.01 * (k % 2) for k in range(len(numels))]
    results = []
    for fn in (cc.cc_fused_lamb_step, _phases):
        shard = Shard(numels, wds, R, align_elems=8, grad_dtype=dtype, cache_policy=policy)
        if limit is not None:
            for p in shard.plans:
                cc.cc_plan_set_meeting_limit(p, limit)
        seeded_state(shard, 31)
        for c in (shard.w, shard.w16):
            c[1].fill_(7.0)                                     # what a skipped step has to leave alone
        seen = []
        for t in range(1, 9):
            seeded_grads(shard, 310 + t, 1e-2)
            if t in (3, 6):                                     # first and last element of the shard
                k = 0 if t == 3 else max(i for i, n in enumerate(numels) if n)
                shard.grad_of(R - 1, k)[0 if t == 3 else -1] = float("inf")
            plan, out = shard.plans[shard.cur], 1 - shard.cur
            before = shard.w[out].clone(), shard.w16[out].clone()
            shard.run(fn, cc.Hyper(step=t))
            sums = np.asarray(cc.cc_lamb_norms_read(plan, len(numels)))
            flag = int(shard.flag.item())
            assert flag == (t in (3, 6))
            if flag:
                assert torch.equal(before[0], shard.w[out]) and torch.equal(before[1], shard.w16[out])
            else:
                shard.commit()
            ints = [shard.m[out].view(torch.int32), shard.v[out].view(torch.int32), shard.w[out].view(torch.int32), shard.w16[out].view(torch.int16)]
            seen.append([x.cpu().clone() for x in ints])
            seen[-1].append(torch.from_numpy(sums.view(np.int64).copy()) if not flag else None)
        results.append(seen)
        shard.destroy()
    for t, (a, b) in enumerate(zip(*results)):
        for k, (x, y) in enumerate(zip(a, b)):
            assert x is None or torch.equal(x, y), "step %d, output %d" % (t + 1, k)


@pytest.mark.parametrize("numels", [[10007, 3, 20 * 1024 + 2], [129 * 1024 - 3, 5, 64 * 1024 + 1]], ids=_name)
def test_one_launch_matches_the_oracle(numels):
    shard = Shard(numels, [0.01, 0.0, 0.01], 4, align_elems=8)
    seeded_state(shard, 5)
    ost = OracleState(shard, range(3))
    for t in (1, 2):
        seeded_grads(shard, 50 + t, 1e-2)
        ghp, ohp = hyper_pair(step=t)
        ots = ost.tensors(shard)
        oracle.lamb_step(ots, ohp)
        assert shard.step(cc.cc_fused_lamb_step, ghp) == 0
        ost.adopt(ots)
        compare_committed(shard, ost, "lamb in one launch, step %d" % t)
    shard.destroy()


@pytest.mark.parametrize("limit", [None, 2])
@pytest.mark.parametrize("numels", [[10007, 3, 20 * 1024 + 2], [129 * 1024 - 3, 5, 64 * 1024 + 1]], ids=_name)
def test_one_launch_replayed_from_a_graph(numels, limit):
    """The words of earlier replays stay where they are; every replay has to tell its own from theirs."""
    R = 4
    shards = [Shard(numels, [0.01, 0.0, 0.01], R, align_elems=8) for _ in range(2)]
    for s in shards:
        seeded_state(s, 6)
        seeded_grads(s, 60, 1e-2)
    eager, graphed = shards
    if limit is not None:
        for p in graphed.plans:
            cc.cc_plan_set_meeting_limit(p, limit)

    def two_steps(s):                    # ping -> pong -> ping: the committed copy is the same buffer afterwards
        for t in (1, 2):
            s.run(cc.cc_fused_lamb_step, cc.Hyper(step=t))
            s.commit()
    two_steps(eager)
    two_steps(graphed)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        two_steps(graphed)
    for rep in range(5):
        for s in shards:
            seeded_grads(s, 61 + rep, 1e-2)
            if rep == 2:                 # an overflow: neither copy of w changes, and the next replays go on from them
                s.grad_of(1, 2)[-1] = float("inf")
        _ = shards[0].w[0].sum().item()  # eager work and a synchronization in between
        two_steps(eager)
        g.replay()
        torch.cuda.synchronize()
        assert int(graphed.flag.item()) == int(eager.flag.item()) == (rep == 2)
        for name in ("w", "m", "v", "w16"):
            for a, b in zip(getattr(eager, name), getattr(graphed, name)):
                bits = torch.int16 if name == "w16" else torch.int32
                assert torch.equal(a.view(bits), b.view(bits)), "replay %d, %s" % (rep, name)
    for s in shards:
        s.destroy()


@pytest.mark.parametrize("R,numel", [(8, 1 << 19), (8, 1 << 18), (16, 1 << 18), (4, 1 << 19), (8, 1 << 16)])
def test_steps_on_several_streams_do_not_keep_each_other_out(R, numel):
    """Four plans on four streams, released together: same bits as one after the other, and not much more time than as phases.  (Where
    more workgroups waited than the device holds at a time, two such steps took 3.3 ms where the phases take 24 us.)"""
    plans = [Shard([numel], [0.01], R, unfused=False) for _ in range(4)]
    streams, gate = [torch.cuda.Stream() for _ in plans], torch.cuda.Stream()
    want = []
    for k, s in enumerate(plans):
        seeded_state(s, 70 + k)
        seeded_grads(s, 700 + k, 1e-2)
        s.run(_phases, cc.Hyper(step=1))
        want.append([x[1].view(torch.int32).clone() for x in (s.w, s.m, s.v)])
    torch.cuda.synchronize()

    def together(fn):
        for s in plans:
            s.w[1].zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(gate):
            torch.cuda._sleep(400000)                           # until everything has been enqueued
            start = torch.cuda.Event(enable_timing=True)
            start.record()
        ends = [torch.cuda.Event(enable_timing=True) for _ in plans]
        for s, st, e in zip(plans, streams, ends):
            st.wait_event(start)
            with torch.cuda.stream(st):
                s.run(fn, cc.Hyper(step=1))
                e.record()
        torch.cuda.synchronize()
        assert all(int(s.flag.item()) == 0 for s in plans)
        for s, bits in zip(plans, want):
            for x, y in zip((s.w, s.m, s.v), bits):
                assert torch.equal(x[1].view(torch.int32), y)
        return max(start.elapsed_time(e) for e in ends)

    together(_phases)
    phases = statistics.median(together(_phases) for _ in range(5))
    one = statistics.median(together(cc.cc_fused_lamb_step) for _ in range(5))
    assert one < 5 * phases, "%.3f ms against %.3f ms" % (one, phases)
    for s in plans:
        s.destroy()


@pytest.mark.parametrize("policy,mem", [(cc.CC_CACHE_STREAMING, "9Streaming"), (cc.CC_CACHE_RESIDENT, "8Resident"), (cc.CC_CACHE_WRITE_THROUGH, "12WriteThrough")])
@pytest.mark.parametrize("numel", [10007, 65 * 1024])
def test_the_policy_asked_for_is_the_one_that_runs(numel, policy, mem):
    for R, dtype in ((2, torch.float16), (2, torch.float32)):
        shard = Shard([numel], [0.01], R, grad_dtype=dtype, cache_policy=policy)
        assert cc.cc_plan_layout(shard.plans[0])[2] == policy
        what = launches(lambda: shard.run(cc.cc_fused_lamb_step, cc.Hyper(step=1)))
        assert [x.kernel for x in what] == ["lamb_one_launch_kernel"] and mem in what[0].symbol
        shard.destroy()
