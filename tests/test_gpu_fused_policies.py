"""Shards whose step's buffers total 80 to 200 MiB: what AUTO launches, and that it gives the bits of the policy that is reported
(which a caller can ask for).  One tensor and a list with short and empty tensors, either side of the second sweep's line."""
import pytest
import torch

from paper_2105_05720_amd import binding as cc
from paper_2105_05720_amd.launches import launches
from paper_2105_05720_amd.shard import Shard
from parity import seeded_grads, seeded_state

pytestmark = pytest.mark.gpu


def _phases(plan, hp, flag, stream=None):
    cc.cc_fused_lamb_phase1(plan, hp, flag, stream)
    cc.cc_fused_lamb_phase2(plan, hp, flag, stream)


def _bits(shard):
    return [x.view(torch.int16 if x.dtype == torch.float16 else torch.int32).clone() for a in (shard.w, shard.m, shard.v, shard.w16) for x in a]


@pytest.mark.parametrize("numels,R,dtype", [([(80 << 20) // 42 + 1], 8, torch.float16), ([(80 << 20) // 42 - 1], 8, torch.float16), ([1500007], 16, torch.float16),
                                            ([3000001], 2, torch.float16), ([1000003], 16, torch.float32),
                                            ([5, 0, 700001, 1023, 1024, 1300000, 2], 8, torch.float16), ([1025, 2900000, 3], 3, torch.float32)],
                         ids=lambda x: "x".join(map(str, x[:3])) if isinstance(x, list) else str(x))
@pytest.mark.parametrize("fn", [cc.cc_fused_adam_step, cc.cc_fused_lamb_step, _phases], ids=["adam", "lamb", "lamb phases"])
def test_auto_launches_other_loads_and_gives_the_same_bits(numels, R, dtype, fn):
    n = sum(numels)
    beyond = n * ((2 if dtype == torch.float16 else 4) * R + 26) >= 80 << 20
    results = []
    for policy in (cc.CC_CACHE_AUTO, cc.CC_CACHE_RESIDENT):
        shard = Shard(numels, [0.01 * (k % 2) for k in range(len(numels))], R, align_elems=8, grad_dtype=dtype, cache_policy=policy, unfused=False)
        assert cc.cc_plan_layout(shard.plans[0]) == (1024, 128, cc.CC_CACHE_RESIDENT)
        what = launches(lambda: shard.run(fn, cc.Hyper(step=1)))
        other = beyond and policy == cc.CC_CACHE_AUTO
        first = "12WriteThrough" if fn is cc.cc_fused_adam_step else "11WeightsKept"
        assert (first if other else "8Resident") in what[0].symbol
        if fn is cc.cc_fused_adam_step and len(numels) == 1:
            assert (what[0].grid, what[0].block) == ((-(-n // 256), 64) if other else (-(-n // 1024), 128))
        elif fn is not cc.cc_fused_adam_step:
            assert ("8Resident" if not other or 12 * n < 32 << 20 else "12WriteThrough") in what[-1].symbol
        seeded_state(shard, 3)
        seen = []
        for t in (1, 2, 3):
            seeded_grads(shard, 30 + t, 1e-2)
            if t == 2:
                shard.grad_of(R - 1, len(numels) - 1)[-1] = float("inf")
            shard.run(fn, cc.Hyper(step=t))
            seen.append(_bits(shard) + [shard.flag.clone()])
            assert int(shard.flag.item()) == (t == 2)
            if t != 2:
                shard.commit()
        results.append(seen)
        shard.destroy()
    for a, b in zip(*results):
        assert all(torch.equal(x, y) for x, y in zip(a, b))


def test_the_static_step_takes_the_same_line():
    for n in ((80 << 20) // 42 - 1, (80 << 20) // 42 + 1):
        shard = Shard([n], [0.01], 8, align_elems=8, unfused=False)
        t = cc.Tensor(numel=n, w_in=shard.w[0], m_in=shard.m[0], v_in=shard.v[0], w_out=shard.w[1], m_out=shard.m[1], v_out=shard.v[1], w16_out=shard.w16[1],
                      grad=shard.grads, weight_decay=0.01)
        of_plan = launches(lambda: shard.run(cc.cc_fused_adam_step, cc.Hyper(step=1)))
        assert launches(lambda: cc.cc_fused_adam_step_static(t, 8, cc.Hyper(step=1), shard.flag)) == of_plan
        shard.destroy()


@pytest.mark.parametrize("numels,R,dtype,kept", [([3000001], 1, torch.float16, True), ([(144 << 20) // 30 - 7], 2, torch.float16, True), ([(144 << 20) // 30 + 9], 2, torch.float16, False),
                                                 ([7, 0, 1500003, 1025, 1600000], 1, torch.float16, True), ([2900000, 3], 1, torch.float32, True),
                                                 ([255, 2000001, 2900000], 2, torch.float16, True), ([255, 2900001, 2900000], 2, torch.float16, False)],
                         ids=lambda x: "x".join(map(str, x[:3])) if isinstance(x, list) else str(x))
@pytest.mark.parametrize("mode", [{}, {"adam_mode": 0, "skip_mode": 1}], ids=["default", "l2 guard"])
def test_few_slices_are_read_plainly(numels, R, dtype, kept, mode):
    """The slices by plain loads up to 144 MiB, with the bits of the policy that reads everything that way; slices that a step before has seen are not kept."""
    results = []
    for policy in (cc.CC_CACHE_AUTO, cc.CC_CACHE_RESIDENT):
        shard = Shard(numels, [0.01 * (k % 2) for k in range(len(numels))], R, align_elems=8, grad_dtype=dtype, cache_policy=policy, unfused=False)
        step = lambda t: shard.run(cc.cc_fused_adam_step, cc.Hyper(step=t, **mode))
        assert ("12WriteThroughELb1E" in launches(lambda: step(1))[0].symbol) == (kept and policy == cc.CC_CACHE_AUTO)
        seeded_state(shard, 3)
        for t in (1, 2):
            seeded_grads(shard, 30 + t, 1e-2)
            step(t)
            assert int(shard.flag.item()) == 0
            shard.commit()
        shard.grad_of(R - 1, len(numels) - 1)[-1] = float("inf")
        step(3)
        results.append(_bits(shard) + [shard.flag.clone()])
        assert int(shard.flag.item()) == 1
        if len(numels) == 1 and dtype == torch.float16:
            shard.flag.zero_()
            cc.cc_fused_adam_step_static(cc.Tensor(numel=numels[0], w_in=shard.w[0], m_in=shard.m[0], v_in=shard.v[0], w_out=shard.w[1], m_out=shard.m[1], v_out=shard.v[1],
                                                   w16_out=shard.w16[1], grad=shard.grads, weight_decay=0.0), R, cc.Hyper(step=3, **mode), shard.flag)
            results[-1] += _bits(shard) + [shard.flag.clone()]
        shard.destroy()
    assert all(torch.equal(x, y) for x, y in zip(*results))
