"""A list bound by HBM whose fused Adam step runs single-wave pieces, against one workgroup of 512 threads per chunk: the same bits, the
same flag, and nothing written between the tensors."""
import pytest
import torch

from paper_2105_05720_amd import binding as cc
from paper_2105_05720_amd.launches import launches
from paper_2105_05720_amd.shard import Shard

pytestmark = pytest.mark.gpu
M = 1 << 20
LINE = -(-(288 << 20) // 14)                    # elements from which a step stores too much to write through
RAGGED = [1, 3, 4, 255, 256, 257, 511, 767, 769, 1023, 1024, 1025, 4099]


@pytest.mark.parametrize("numels,R,dtype,pieces,hyper", [
    ([LINE - 9, 9], 2, torch.float16, True, {}),                                  # the smallest
    ([LINE - 10, 9], 2, torch.float16, False, {}),
    (RAGGED + [LINE] + RAGGED, 1, torch.float16, True, {}),
    (RAGGED + [LINE // 2] * 2 + RAGGED, 10, torch.float16, True, {"grad_average": 1, "loss_scale": 8.0}),
    ([LINE, 5], 11, torch.float16, False, {}),                                    # more slices
    ([LINE] + RAGGED, 8, torch.float32, True, {"adam_mode": 0}),
    ([LINE, 7], 9, torch.float32, False, {}),
    ([LINE] + [1] * 3000, 1, torch.float16, False, {}),                           # too many short chunks
    ([LINE, 0, 5001], 3, torch.float16, True, {"skip_mode": 1}),
    ([64 * M, 1027], 1, torch.float16, True, {}),                                 # instead of the ordered schedule
    ([64 * M, 1027], 9, torch.float16, False, {}),
    ([128 * M - 4, 4], 1, torch.float16, False, {}),
    ([128 * M, 1027], 2, torch.float32, True, {}),                                # fp32 slices: further up
    ([64 * M, 1027], 9, torch.float32, False, {}),
])
def test_pieces_give_the_bits_of_chunks(numels, R, dtype, pieces, hyper):
    guard = hyper.get("skip_mode") == 1
    shard = Shard(numels, [0.01, 0.0] * (len(numels) // 2) + [0.01] * (len(numels) % 2), R, align_elems=8, grad_dtype=dtype, unfused=False)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(R)
    shard.w[0].normal_(0, 0.02, generator=gen)
    shard.m[0].normal_(0, 1e-3, generator=gen)
    shard.v[0].uniform_(0, 1e-6, generator=gen)
    for g in shard.grads:
        for part in g.split(64 * M):
            part.copy_(torch.empty(part.numel(), device="cuda").normal_(0, 1e-2, generator=gen))
    plan, hp, out = shard.plans[0], cc.Hyper(step=2, **hyper), (shard.w[1], shard.m[1], shard.v[1], shard.w16[1])
    step = lambda: cc.cc_fused_adam_step(plan, hp, shard.flag)
    ran = launches(step)
    assert [x.kernel == "fused_adam_piece_kernel" for x in ran] == [pieces]
    if pieces:
        assert (ran[0].grid, ran[0].block) == (4 * sum(-(-n // 1024) for n in numels), 64)
    last = max(k for k, n in enumerate(numels) if n > 0)
    for bad in (False, True):
        if bad:
            shard.grad_of(R - 1, last)[-1] = float("inf")
        results = []
        for chosen in (0, 4096):
            cc.cc_plan_set_chunk_elems(plan, chosen)
            cc.cc_plan_set_schedule(plan, cc.CC_SCHEDULE_PER_CHUNK if chosen else cc.CC_SCHEDULE_AUTO)
            for x in out:
                x.fill_(7.0)
            step()
            assert int(shard.flag.item()) == int(bad)
            results.append([x.clone() for x in out])
            cc.cc_plan_set_schedule(plan, cc.CC_SCHEDULE_AUTO)
        cc.cc_plan_set_chunk_elems(plan, 0)
        # a step that overflowed is not adopted, and what it has written then may differ: with the guard it is defined
        if not bad or guard:
            for a, b in zip(*results):
                assert torch.equal(a, b)
    shard.destroy()


@pytest.mark.parametrize("numels,chunk,policy,pieces", [
    ([LINE, 5], 1024, cc.CC_CACHE_AUTO, True),
    ([64 * M - 9, 8], 1024, cc.CC_CACHE_STREAMING, True),
    ([64 * M, 1027], 1024, cc.CC_CACHE_AUTO, False),                              # chunks of 1024 elements get a workgroup each
    ([64 * M, 1027], 1024, cc.CC_CACHE_STREAMING, False),
    ([64 * M, 1027], 0, cc.CC_CACHE_STREAMING, False),                            # the ordered schedule
])
def test_what_is_asked_for_beyond_64_mi_elements_runs(numels, chunk, policy, pieces):
    shard = Shard(numels, [0.01, 0.0], 1, align_elems=8, unfused=False)
    plan = shard.plans[0]
    cc.cc_plan_set_chunk_elems(plan, chunk)
    cc.cc_plan_set_cache_policy(plan, policy)
    ran = launches(lambda: cc.cc_fused_adam_step(plan, cc.Hyper(step=2), shard.flag))
    assert [x.kernel for x in ran] == ["fused_adam_piece_kernel" if pieces else "fused_adam_kernel" if chunk else "fused_adam_ordered_kernel"]
    if chunk and not pieces:
        assert (ran[0].grid, ran[0].block) == (sum(-(-n // 1024) for n in numels), 128)
    shard.destroy()
