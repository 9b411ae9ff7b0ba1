"""The fused LAMB step just beyond 64 Mi elements, which keeps chunks of 1024 elements: the kernels, the same bits as with those chunks
chosen, in one call and in two, and the unfused pipeline beside it as it was."""
import numpy as np
import pytest
import torch

from paper_2105_05720_amd import binding as cc
from paper_2105_05720_amd.launches import launches
from paper_2105_05720_amd.shard import Shard

pytestmark = pytest.mark.gpu
M = 1 << 20


@pytest.mark.parametrize("numels,R,dtype,small", [
    ([64 * M - 3, 5], 1, torch.float16, True),
    ([88 * M - 1030, 1029], 2, torch.float16, True),
    ([88 * M], 1, torch.float16, False),
    ([130001] * 600, 1, torch.float16, True),              # no tensor of more than 512 chunks: the second sweep adds up the norms
    ([65 * M + 7], 1, torch.float32, True),
    ([66 * M, 4099], 7, torch.float16, True),
    ([66 * M, 4099], 8, torch.float16, False),             # more slices
    ([66 * M + 5], 3, torch.float16, False),
])
def test_beyond_64_mi_elements(numels, R, dtype, small):
    shard = Shard(numels, [0.01] * len(numels), R, align_elems=8, grad_dtype=dtype, unfused=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(R)
    shard.w[0].normal_(0, 0.02, generator=gen)
    shard.m[0].normal_(0, 1e-3, generator=gen)
    shard.v[0].uniform_(0, 1e-6, generator=gen)
    for g in shard.grads:
        g.copy_(torch.empty(g.numel(), device="cuda").normal_(0, 1e-2, generator=gen))
    plan, hp, out = shard.plans[0], cc.Hyper(step=2), (shard.w[1], shard.m[1], shard.v[1], shard.w16[1])

    def one():
        cc.cc_fused_lamb_step(plan, hp, shard.flag)

    def two():
        cc.cc_fused_lamb_phase1(plan, hp, shard.flag)
        cc.cc_fused_lamb_phase2(plan, hp, shard.flag)
    ran = launches(one)
    chunks = sum(-(-n // 1024) for n in numels)
    if small:
        norms = [] if max(numels) <= 512 * 1024 else ["lamb_norms_kernel"]
        assert [x.kernel for x in ran] == ["lamb_phase1_kernel"] + norms + ["lamb_phase2_kernel" if norms else "lamb_phase2_with_norms_kernel"]
        assert (ran[0].grid, ran[0].block) == (ran[-1].grid, ran[-1].block) == (chunks, 128)
    else:
        assert [x.kernel for x in ran] == ["lamb_phase1_ordered_kernel", "lamb_norms_kernel", "lamb_phase2_ordered_kernel"]
    assert [x.kernel for x in launches(lambda: cc.cc_unfused_lamb_step(plan, hp, shard.flag))][:2] == ["reduce_ordered_kernel", "lamb_phase1_from_sum_ordered_kernel"]
    results = []
    for step, chosen in ((one, 0), (two, 0), (one, 1024 if small else 4096)):
        cc.cc_plan_set_chunk_elems(plan, chosen)
        for x in out:
            x.fill_(7.0)
        step()
        assert int(shard.flag.item()) == 0
        results.append(([x.clone() for x in out], np.asarray(cc.cc_lamb_norms_read(plan, len(numels)))))
    for got, sums in results[:2]:
        assert all(torch.equal(a, b) for a, b in zip(got, results[2][0])) and np.array_equal(sums, results[2][1])
    cc.cc_plan_set_chunk_elems(plan, 0)
    cc.cc_unfused_lamb_step(plan, hp, shard.flag)
    assert np.allclose(np.asarray(cc.cc_lamb_norms_read(plan, len(numels))), results[0][1], rtol=1e-5)
    shard.grad_of(0, len(numels) - 1)[-1] = float("nan")
    shard.w[1].fill_(7.0)
    one()
    assert int(shard.flag.item()) == 1 and bool((shard.w[1] == 7.0).all())
    shard.destroy()
