"""Which kernels the step calls launch on either side of their dispatch rules, read from captured graphs: without this, a rule that
always took the general path would pass every comparison with it."""
import importlib.util
import os

import pytest
import torch

from paper_2105_05720_amd import binding as cc
from paper_2105_05720_amd.launches import launches
from paper_2105_05720_amd.shard import Shard

pytestmark = pytest.mark.gpu
ONE, TWO = ["lamb_one_launch_kernel"], ["lamb_phase1_kernel", "lamb_phase2_with_norms_kernel"]
THREE = ["lamb_phase1_kernel", "lamb_norms_kernel", "lamb_phase2_kernel"]


def _kernels(numels, R, dtype, fn, **kw):
    shard = Shard(numels, [0.01] * len(numels), R, align_elems=8, grad_dtype=dtype, unfused=False, **kw)
    what = launches(lambda: shard.run(fn, cc.Hyper(step=1)))
    shard.destroy()
    return [x.kernel for x in what], what


@pytest.mark.parametrize("R,dtype,most", [(4, torch.float16, 512), (7, torch.float16, 384), (8, torch.float16, 256), (8, torch.float32, 512), (12, torch.float32, 384)])
def test_lamb_at_the_edge_of_one_launch(R, dtype, most):
    """The lines of a whole device (a partition has its own: tests/test_meeting_rule.py)."""
    if cc.cc_device_info()[0] != 256:
        pytest.skip("the lines are drawn by the device's compute units")
    for numels, kernels in (([most * 1024], ONE), ([most * 1024 + 1], TWO if most < 512 else THREE), ([1] * 64, ONE), ([1] * 65, TWO)):
        got, what = _kernels(numels, R, dtype, cc.cc_fused_lamb_step)
        assert got == kernels, numels[:2]
        assert what[0].grid == sum(-(-n // 1024) for n in numels) and what[0].block == 128
    assert _kernels([most * 1024], R, dtype, cc.cc_fused_lamb_step, chunk_elems=2048)[0] == TWO


@pytest.mark.parametrize("numel,R,pieces", [((64 << 20) + 5, 2, True), (144 << 20, 1, False), (64 << 20, 11, False)])
def test_adam_on_one_large_tensor(numel, R, pieces):
    want = [("fused_adam_flat_kernel", -(-numel // 256), 64)] if pieces else [("fused_adam_ordered_kernel", cc.cc_device_info()[0], 512)]
    assert [(x.kernel, x.grid, x.block) for x in _kernels([numel], R, torch.float16, cc.cc_fused_adam_step)[1]] == want
    for chosen in (dict(schedule=cc.CC_SCHEDULE_ORDERED), dict(chunk_elems=4096)):
        assert _kernels([numel], R, torch.float16, cc.cc_fused_adam_step, **chosen)[0] == ["fused_adam_ordered_kernel"]


def test_the_benchmark_names_the_kernels_that_it_times():
    spec = importlib.util.spec_from_file_location("bench", os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    for numels, optimizer, kernel, schedule in (
            ([64 << 20], "adam", "fused_adam_flat_kernel<R=2, 64 threads>", "262144 workgroups of 64 threads, one per piece of 256 elements"),
            ([10007], "lamb", "lamb_one_launch_kernel<R=2, 128 threads>", "one workgroup of 128 threads per chunk"),
            ([600000, 5], "lamb", "lamb_phase1_kernel<R=2, 128 threads> + lamb_norms_kernel<1024 threads> + lamb_phase2_kernel<128 threads>", "one workgroup of 128 threads per chunk"),
            ([192 << 20, 8], "adam", "fused_adam_ordered_kernel<R=2, 512 threads>", "ordered: %d persistent workgroups take the chunks in table order" % cc.cc_device_info()[0])):
        shard = Shard(numels, [0.01] * len(numels), 2, unfused=False)
        told = bench.describe(cc, shard, 2, optimizer, False)
        assert (told["kernel"], told["schedule"]) == (kernel, schedule)
        shard.destroy()
