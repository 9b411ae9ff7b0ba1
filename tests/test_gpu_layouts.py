"""What a plan may vary without changing results: chunk size, cache policy; and what the unfused pipelines need first.

Adam is independent per element, so every chunk size and both cache policies must give the same bits.  LAMB adds its
per-chunk partial sums in double in a fixed order per chunk size; another chunk size groups them differently, so its
results move within rounding of the norms (checked against the oracle at the parity bar) while the cache policy leaves
the bits alone."""
import pytest
import torch

import oracle
from paper_2105_05720_amd import binding as cc
from paper_2105_05720_amd.shard import Shard
from parity import OracleState, hyper_pair, run_steps, seeded_grads, seeded_state

pytestmark = pytest.mark.gpu

LIST = [16384 * 2 + 4097, 0, 1, 4096 * 3, 1024 * 9 + 1023, 8192, 777, 16384]


def wds_for(numels, wd=0.01):
    return [wd if (i % 3) else 0.0 for i in range(len(numels))]


def bits_of(sh):
    c = sh.cur
    return [sh.w[c].view(torch.int32).clone(), sh.m[c].view(torch.int32).clone(), sh.v[c].view(torch.int32).clone(),
            sh.w16[c].view(torch.int16).clone()]


def run_shape(fn, ofn, chunk, policy, R=4, grad_dtype=torch.float16, steps=2, numels=LIST):
    sh = Shard(numels, wds_for(numels), R, align_elems=8, grad_dtype=grad_dtype)
    for p in sh.plans:
        cc.cc_plan_set_chunk_elems(p, chunk)
        cc.cc_plan_set_cache_policy(p, policy)
        assert cc.cc_plan_layout(p)[0] == chunk
        want = policy if chunk < 4096 else cc.CC_CACHE_STREAMING
        assert cc.cc_plan_layout(p)[2] == want
    seeded_state(sh, 5)
    ost = OracleState(sh, range(len(numels)))
    run_steps(sh, ost, fn, ofn, [hyper_pair(step=t) for t in range(1, steps + 1)], "chunk %d policy %d" % (chunk, policy),
              lambda i: seeded_grads(sh, 500 + i, 1e-2), expect_flags=[0] * steps)
    out = bits_of(sh)
    sh.destroy()
    return out


@pytest.mark.parametrize("fn,ofn", [(cc.cc_fused_adam_step, oracle.adam_step), (cc.cc_unfused_adam_step, oracle.adam_step)])
def test_adam_bits_do_not_depend_on_chunk_size_or_cache_policy(fn, ofn):
    ref = run_shape(fn, ofn, 1024, cc.CC_CACHE_STREAMING)
    for chunk, policy in ((1024, cc.CC_CACHE_RESIDENT), (1024, cc.CC_CACHE_WRITE_THROUGH), (4096, cc.CC_CACHE_STREAMING),
                          (16384, cc.CC_CACHE_STREAMING), (4096, cc.CC_CACHE_RESIDENT)):
        got = run_shape(fn, ofn, chunk, policy)
        assert all(torch.equal(a, b) for a, b in zip(ref, got)), "chunk %d policy %d changes Adam's bits" % (chunk, policy)


@pytest.mark.parametrize("fn", [cc.cc_fused_lamb_step, cc.cc_unfused_lamb_step])
def test_lamb_every_chunk_size_and_policy_against_oracle(fn):
    per_chunk = {}
    for chunk, policy in ((1024, cc.CC_CACHE_STREAMING), (1024, cc.CC_CACHE_RESIDENT), (1024, cc.CC_CACHE_WRITE_THROUGH),
                          (4096, cc.CC_CACHE_STREAMING), (16384, cc.CC_CACHE_STREAMING)):
        got = run_shape(fn, oracle.lamb_step, chunk, policy)
        if chunk in per_chunk:          # same chunk size, other cache policy: the same bits
            assert all(torch.equal(a, b) for a, b in zip(per_chunk[chunk], got))
        per_chunk[chunk] = got


@pytest.mark.parametrize("R", [1, 8, 16])
def test_resident_policy_every_kind_of_R_and_fp32_slices(R):
    for gd in (torch.float16, torch.float32):
        a = run_shape(cc.cc_fused_adam_step, oracle.adam_step, 1024, cc.CC_CACHE_RESIDENT, R=R, grad_dtype=gd, steps=1)
        b = run_shape(cc.cc_fused_adam_step, oracle.adam_step, 1024, cc.CC_CACHE_STREAMING, R=R, grad_dtype=gd, steps=1)
        c = run_shape(cc.cc_fused_adam_step, oracle.adam_step, 1024, cc.CC_CACHE_WRITE_THROUGH, R=R, grad_dtype=gd, steps=1)
        assert all(torch.equal(x, y) and torch.equal(x, z) for x, y, z in zip(a, b, c))


def test_in_place_guard_mode_under_every_cache_policy():
    """skip_mode 1 reads and writes the same buffers; the written-through stores go through inline assembly, so the guard's
    "keep the input" case and the ordinary case are checked against the oracle under each policy, with an inf, a NaN made
    of opposite infinities and a NaN in a ragged tail planted in the first step, and the policies must agree bit for bit."""
    outs = []
    for policy in (cc.CC_CACHE_STREAMING, cc.CC_CACHE_RESIDENT, cc.CC_CACHE_WRITE_THROUGH):
        numels = [1024 * 9 + 1023, 100, 4096]
        sh = Shard(numels, [0.01, 0.0, 0.01], 4, in_place=True, align_elems=8, chunk_elems=1024, cache_policy=policy)
        assert cc.cc_plan_layout(sh.plans[0]) == (1024, 128, policy)
        seeded_state(sh, 6)
        ost = OracleState(sh, range(3))

        def fill(i):
            seeded_grads(sh, 60 + i, 1e-2)
            if i == 0:
                for r, t, e, bits in ((0, 0, 4100, 0x7C00), (3, 0, 4100, 0xFC00), (2, 0, 1024 * 9 + 1000, 0x7C00), (1, 1, 99, 0x7D55)):
                    sh.grad_of(r, t).view(torch.int16)[e] = bits - 0x10000 if bits >= 0x8000 else bits
        hps = [hyper_pair(step=1, skip_mode=1), hyper_pair(step=2, skip_mode=1), hyper_pair(step=3, skip_mode=1, adam_mode=0, grad_average=1)]
        run_steps(sh, ost, cc.cc_fused_adam_step, oracle.adam_step, hps, "guard, policy %d" % policy, fill, expect_flags=[1, 0, 0])
        outs.append(bits_of(sh))
        sh.destroy()
    for other in outs[1:]:
        assert all(torch.equal(a, b) for a, b in zip(outs[0], other))


def test_single_tensor_plan_resident_and_streaming():
    """One tensor: the table-free kernel, both policies, against the oracle (2^17 + a ragged end)."""
    for policy in (cc.CC_CACHE_RESIDENT, cc.CC_CACHE_STREAMING, cc.CC_CACHE_WRITE_THROUGH):
        run_shape(cc.cc_fused_adam_step, oracle.adam_step, 1024, policy, numels=[(1 << 17) + 5], steps=2)


def test_auto_policy_and_layout_rules():
    small = Shard([1 << 20], [0.0], 4, align_elems=8)                                  # 36 MB of buffers
    assert cc.cc_plan_layout(small.plans[0]) == (1024, 128, cc.CC_CACHE_RESIDENT)
    cc.cc_plan_set_cache_policy(small.plans[0], cc.CC_CACHE_STREAMING)
    assert cc.cc_plan_layout(small.plans[0])[2] == cc.CC_CACHE_STREAMING
    cc.cc_plan_set_cache_policy(small.plans[0], cc.CC_CACHE_RESIDENT)
    cc.cc_plan_set_chunk_elems(small.plans[0], 4096)
    assert cc.cc_plan_layout(small.plans[0]) == (4096, 512, cc.CC_CACHE_STREAMING)     # resident exists for 128-thread workgroups only
    with pytest.raises(cc.CcError) as e:
        cc.cc_plan_set_chunk_elems(small.plans[0], 2048)
    assert e.value.code == cc.CC_ERR_ARG
    with pytest.raises(cc.CcError):
        cc.cc_plan_set_cache_policy(small.plans[0], 9)
    cc.cc_plan_set_chunk_elems(small.plans[0], 0)
    assert cc.cc_plan_layout(small.plans[0]) == (1024, 128, cc.CC_CACHE_RESIDENT)
    cc.cc_plan_set_cache_policy(small.plans[0], cc.CC_CACHE_STREAMING)
    cc.cc_plan_set_cache_policy(small.plans[0], cc.CC_CACHE_AUTO)
    assert cc.cc_plan_layout(small.plans[0])[2] == cc.CC_CACHE_RESIDENT
    small.destroy()
    mid = Shard([1 << 22], [0.0], 8, align_elems=8, unfused=False)                      # 176 MB of buffers: still inside the Infinity Cache
    assert cc.cc_plan_layout(mid.plans[0]) == (1024, 128, cc.CC_CACHE_RESIDENT)
    mid.destroy()
    big = Shard([1 << 23], [0.0], 8, align_elems=8, unfused=False)                      # 352 MB: streams in, writes through
    assert cc.cc_plan_layout(big.plans[0]) == (1024, 128, cc.CC_CACHE_WRITE_THROUGH)
    big.destroy()
    tiny = Shard([1 << 16], [0.0], 8, align_elems=8, unfused=False)                     # 2.75 MB: launch-bound, streams
    assert cc.cc_plan_layout(tiny.plans[0]) == (1024, 128, cc.CC_CACHE_STREAMING)
    tiny.destroy()
    for mi, want in ((20, cc.CC_CACHE_WRITE_THROUGH), (21, cc.CC_CACHE_STREAMING)):     # 14 B stored per element against 288 MiB
        edge = Shard([mi << 20], [0.0], 2, align_elems=8, unfused=False)
        assert cc.cc_plan_layout(edge.plans[0]) == (1024, 128, want)
        edge.destroy()
    fixed = Shard([1 << 16], [0.0], 2, chunk_elems=2048, align_elems=8)                 # a caller's own chunk size: that one only
    assert cc.cc_plan_layout(fixed.plans[0])[:2] == (2048, 128)
    with pytest.raises(cc.CcError):
        cc.cc_plan_set_chunk_elems(fixed.plans[0], 4096)
    fixed.destroy()


def test_unfused_steps_need_the_reserved_buffer_and_never_allocate():
    sh = Shard([5000, 3], [0.01, 0.0], 2, align_elems=8, unfused=False)
    seeded_state(sh, 3)
    seeded_grads(sh, 30, 1e-2)
    before = bits_of(sh)
    for fn in (cc.cc_unfused_adam_step, cc.cc_unfused_lamb_step):
        with pytest.raises(cc.CcError) as e:
            sh.run(fn, cc.Hyper())
        assert e.value.code == cc.CC_ERR_ARG and "cc_plan_reserve_unfused" in cc.cc_last_error()
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(before, bits_of(sh)))
    sh.reserve_unfused()
    sh.reserve_unfused()                                   # a second call does nothing
    # the very first unfused call can be captured into a graph: nothing is allocated or copied by a step call
    ref = Shard([5000, 3], [0.01, 0.0], 2, align_elems=8, unfused=True)
    seeded_state(ref, 3)
    seeded_grads(ref, 30, 1e-2)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        sh.run(cc.cc_unfused_adam_step, cc.Hyper())
    g.replay()
    ref.run(cc.cc_unfused_adam_step, cc.Hyper())
    torch.cuda.synchronize()
    sh.commit(); ref.commit()
    assert all(torch.equal(a, b) for a, b in zip(bits_of(sh), bits_of(ref)))
    sh.destroy(); ref.destroy()


@pytest.mark.parametrize("log2n,R,policy", [(21, 8, cc.CC_CACHE_RESIDENT), (23, 2, cc.CC_CACHE_WRITE_THROUGH), (23, 8, cc.CC_CACHE_WRITE_THROUGH)])
@pytest.mark.parametrize("fn,ofn", [(cc.cc_fused_adam_step, oracle.adam_step), (cc.cc_fused_lamb_step, oracle.lamb_step)])
def test_mid_size_shard_under_the_automatic_cache_policy(fn, ofn, log2n, R, policy):
    """2^21 elements with R = 8 (88 MB of buffers: AUTO keeps the shard on chip) and 2^23 elements with R = 2 and 8 (252 and
    352 MB, of which a launch stores 117 MB: AUTO writes through); two steps, every element against the oracle."""
    n = 1 << log2n
    sh = Shard([n - 4096 * 100 - 3, 4096 * 100 + 3], [0.01, 0.0], R, unfused=False)
    assert cc.cc_plan_layout(sh.plans[0]) == (1024, 128, policy)
    seeded_state(sh, 8)
    ost = OracleState(sh, [0, 1])
    run_steps(sh, ost, fn, ofn, [hyper_pair(step=t) for t in (1, 2)], "2^%d policy %d" % (log2n, policy),
              lambda i: seeded_grads(sh, 800 + i, 1e-3), expect_flags=[0, 0])
    sh.destroy()


@pytest.mark.parametrize("fn,ofn,numels,R,why", [
    (cc.cc_fused_adam_step, oracle.adam_step, [1024 * 3584 - 7, 3, 9], 16, "just over 200 MiB: written through, 14 rounds of runs and two workgroups behind them"),
    (cc.cc_fused_adam_step, oracle.adam_step, [1024 * 5000 + 1, 17, 1024 * 503], 16, "over 300 MiB: still written through"),
    (cc.cc_fused_adam_step, oracle.adam_step, [1024 * 21070 - 7, 5], 1, "288 MiB stored and more: non-temporal stores"),
    (cc.cc_fused_adam_step, oracle.adam_step, [1024 * 21070 - 5, 3], 9, "... and four workgroups per compute unit"),
    (cc.cc_fused_lamb_step, oracle.lamb_step, [1024 * 5001, 1024 * 7900 + 5, 11], 1, "both sweeps write through"),
    (cc.cc_fused_lamb_step, oracle.lamb_step, [1024 * 5001, 1024 * 31870 + 5, 11], 1, "288 MiB of moments and more: the second sweep stores non-temporally"),
    (cc.cc_fused_lamb_step, oracle.lamb_step, [1024 * 512, 1024 * 511 + 3, 1024 * 512, 17, 1024 * 512, 1024 * 500 + 1, 1024 * 512, 1024 * 509 + 1023, 1024 * 20], 16,
     "no tensor above 512 chunks: the second sweep adds up the norms itself, in runs from the end of the table"),
])
def test_chunks_in_runs(fn, ofn, numels, R, why):
    """Shards that do not fit the Infinity Cache: each XCD takes runs of 32 chunks and what is left behind the last full
    round goes in table order.  Every element against the oracle."""
    sh = Shard(numels, wds_for(numels), R, align_elems=8, unfused=False)
    assert cc.cc_plan_layout(sh.plans[0])[:2] == (1024, 128)
    seeded_state(sh, 12)
    ost = OracleState(sh, range(len(numels)))
    run_steps(sh, ost, fn, ofn, [hyper_pair(step=3)], why, lambda i: seeded_grads(sh, 120 + i, 1e-3), expect_flags=[0])
    sh.destroy()


@pytest.mark.parametrize("fn,ofn", [(cc.cc_fused_adam_step, oracle.adam_step), (cc.cc_fused_lamb_step, oracle.lamb_step)])
@pytest.mark.parametrize("numels", [[1, 2, 3, 4, 5, 7, 8, 511, 512, 513, 515, 516, 1023, 1024, 1025, 1026, 1028, 2047], [1], [3], [6], [1022]])
def test_short_chunks(fn, ofn, numels):
    """Chunks shorter than a sweep: no whole pack of four, lanes and whole groups past the end, one to three elements
    behind the last pack; as a list and as one tensor, every element against the oracle."""
    run_shape(fn, ofn, 1024, cc.CC_CACHE_STREAMING, numels=numels, steps=2)


@pytest.mark.parametrize("n,R,grad_dtype,policy", [
    (3615780 + 256, 16, torch.float16, cc.CC_CACHE_AUTO),              # just over 200 MiB of buffers: written through, the short-launch shape
    (5423671 + 255, 16, torch.float16, cc.CC_CACHE_AUTO),              # just over 300 MiB, a piece that is one element short of full
    (1024 * 7000 + 1, 1, torch.float32, cc.CC_CACHE_STREAMING),        # fp32 slices, non-temporal stores, a last piece of one element
])
def test_one_tensor_in_single_wave_pieces(n, R, grad_dtype, policy):
    """One tensor beyond the Infinity Cache runs in 64-thread workgroups of 256 elements; its bits are those of the
    512-thread workgroups on the same plan, under both overflow modes' arithmetic (guard in place, whole-step skip)."""
    for in_place in (False, True):
        sh = Shard([n], [0.01], R, align_elems=8, unfused=False, grad_dtype=grad_dtype, cache_policy=policy, in_place=in_place)
        assert cc.cc_plan_layout(sh.plans[0])[0] == 1024
        outs = []
        for chunk in (0, 4096):
            cc.cc_plan_set_chunk_elems(sh.plans[0], chunk)
            seeded_state(sh, 6)
            seeded_grads(sh, 60, 1e-3)
            sh.grads[0][n - 1] = float("inf")
            sh.run(cc.cc_fused_adam_step, cc.Hyper(step=5, skip_mode=1 if in_place else 0))
            torch.cuda.synchronize()
            assert int(sh.flag.item()) == 1
            i = sh.out_index
            outs.append([x[i].clone() for x in (sh.w, sh.m, sh.v, sh.w16)])
        for a, b in zip(*outs):
            assert torch.equal(a.view(torch.int16), b.view(torch.int16))
        sh.destroy()


@pytest.mark.parametrize("fn,ofn", [(cc.cc_fused_adam_step, oracle.adam_step), (cc.cc_fused_lamb_step, oracle.lamb_step),
                                    (cc.cc_unfused_adam_step, oracle.adam_step)])
def test_both_forms_of_the_chunk_table(fn, ofn):
    """Layouts of up to 2048 chunks give the kernels one copy of the tensor's descriptor per chunk, larger ones a chunk
    entry that points at the descriptor.  A list of exactly 2048 chunks and the same list with one more one-element
    tensor (2049 chunks) are each checked against the oracle, every element, two steps."""
    shared = [1024 * 700 + 5, 1024 * 1300, 17, 1024 * 44 + 1000, 1]            # 701 + 1300 + 1 + 45 + 1 = 2048 chunks
    for numels in (shared, shared + [1]):
        sh = Shard(numels, wds_for(numels), 3, align_elems=8, chunk_elems=1024, unfused=True)
        assert cc.cc_plan_info(sh.plans[0])[1] == len(numels) - 5 + 2048
        seeded_state(sh, 31)
        ost = OracleState(sh, range(len(numels)))
        run_steps(sh, ost, fn, ofn, [hyper_pair(step=t) for t in (1, 2)], "%d chunks" % (len(numels) - 5 + 2048),
                  lambda i: seeded_grads(sh, 310 + i, 1e-2), expect_flags=[0, 0])
        sh.destroy()


@pytest.mark.parametrize("R,dtype,in_place", [(2, torch.float16, False), (2, torch.float16, True), (5, torch.float32, False)])
def test_one_large_tensor_in_pieces_gives_the_bits_of_the_ordered_schedule(R, dtype, in_place):
    """One tensor of 64 Mi elements and more for which nothing was chosen: the fused Adam step runs single-wave pieces of 256
    elements instead of the ordered schedule.  With a ragged end, an overflow in the last element, and without."""
    numel = (64 << 20) + 4096 * 3 + 257 + 2
    outs = []
    for schedule in (cc.CC_SCHEDULE_AUTO, cc.CC_SCHEDULE_ORDERED):
        shard = Shard([numel], [0.01], R, schedule=schedule, in_place=in_place, grad_dtype=dtype, unfused=False)
        seeded_state(shard, 41)
        flags = []
        for t in (1, 2):
            seeded_grads(shard, 410 + t, 1e-2)
            if t == 2:
                shard.grad_of(R - 1, 0)[-1] = float("inf")
            flags.append(shard.step(cc.cc_fused_adam_step, cc.Hyper(step=t, skip_mode=int(in_place), adam_mode=int(in_place))))
        assert flags == [0, 1]
        outs.append([x.clone() for a in (shard.w, shard.m, shard.v) for x in a] + [x.view(torch.int16).clone() for x in shard.w16])
        shard.destroy()
    for a, b in zip(*outs):
        a, b = (x if x.dtype == torch.int16 else x.view(torch.int32) for x in (a, b))
        assert torch.equal(a, b)
