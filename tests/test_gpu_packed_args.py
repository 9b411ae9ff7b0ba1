"""Small calls whose kernel arguments fit 96 bytes and the same calls where they do not (slices that are not the same distance apart):
the kernels, and the same bits."""
import pytest
import torch

from paper_2105_05720_amd import binding as cc
from paper_2105_05720_amd.launches import launches

pytestmark = pytest.mark.gpu


class Arena:
    """Tensors out of one allocation: separate ones may lie more than 64 GiB apart, which does not fit the packed arguments."""

    def __init__(self, nbytes):
        self.bytes, self.used = torch.zeros(nbytes, dtype=torch.uint8, device="cuda"), 0

    def __call__(self, n, dtype):
        first, self.used = self.used, self.used + -(-n * dtype.itemsize // 256) * 256
        return self.bytes[first:first + n * dtype.itemsize].view(dtype)


def _slices(arena, R, n, dtype, even):
    """R slices one after the other from the last to the first, or with one of them further away."""
    pitch = -(-n // 64) * 64
    arena = arena((R + 1) * pitch, dtype)
    where = list(range(R))[::-1]
    if not even:
        where[-1] = R
    return [arena[k * pitch:k * pitch + n] for k in where]


@pytest.mark.parametrize("hyper", [{}, {"adam_mode": 0, "grad_average": 1, "loss_scale": 8.0, "skip_mode": 1}])
@pytest.mark.parametrize("numel,R,dtype", [(1, 1, torch.float16), (1023, 2, torch.float16), (1025, 3, torch.float16), (4099, 4, torch.float16), (70001, 16, torch.float16),
                                           (131072, 8, torch.float32), (300001, 5, torch.float32), (1 << 20, 8, torch.float16)])
def test_adam(numel, R, dtype, hyper):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(numel + R)
    arena = Arena(numel * (26 + (2 * R + 2) * dtype.itemsize) + (4 << 10) * (R + 12))
    w, m, v, *out = [arena(numel, torch.float32) for _ in range(6)] + [arena(numel, torch.float16)]
    w.normal_(0, 0.02, generator=gen)
    m.normal_(0, 1e-3, generator=gen)
    v.uniform_(0, 1e-6, generator=gen)
    values = torch.empty(R, numel, device="cuda").normal_(0, 1e-2, generator=gen).to(dtype)
    flag, hp, results = arena(2, torch.int32), cc.Hyper(step=3, **hyper), []
    for even in (True, False):
        grads = _slices(arena, R, numel, dtype, even)
        for g, x in zip(grads, values):
            g.copy_(x)
        for bad in (False, True):
            if bad:
                grads[-1][-1] = float("inf")
            t = cc.Tensor(numel, w, m, v, *out, grads, 0.01)
            plan = cc.cc_plan_create_ex([t], R, 0, cc.CC_GRAD_F16 if dtype == torch.float16 else cc.CC_GRAD_F32)
            calls = [lambda: cc.cc_fused_adam_step(plan, hp, flag[1:])]             # a flag that is not 16-byte aligned
            if dtype == torch.float16:
                calls.append(lambda: cc.cc_fused_adam_step_static(t, R, hp, flag[1:]))
            for call in calls:
                packed = even or R <= 2
                assert [x.kernel for x in launches(call)] == ["fused_adam_packed_kernel" if packed else "fused_adam_flat_kernel"]
                for _ in range(2):
                    for x in out:
                        x.fill_(7.0)
                    call()
                    assert flag.tolist() == [0, int(bad)]
                if not bad or hp.skip_mode == 1:
                    results.append((bad, [x.clone() for x in out]))
            plan.destroy()
    for bad, got in results:
        want = next(x for b, x in results if b == bad)
        assert all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("numel,R", [(8, 1), (513, 2), (40303, 9), (646352, 8), (838856, 8)])
def test_epilogue(numel, R):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(numel + R)
    arena = Arena(2 * numel * (R + 4) + (1 << 16))

    def half(n, std):
        return arena(n, torch.float16).copy_(torch.empty(n, device="cuda").normal_(0, std, generator=gen))
    values, bias, residual = [half(numel, 0.3) for _ in range(R)], half(3072, 0.1), half(numel, 1.0)
    for first in (1 << 33, 0):
        partials = values
        out = arena(numel, torch.float16).fill_(7.0)
        call = lambda: cc.cc_fused_epilogue(partials, bias, residual, out, first, 3072, 0.1, 12345678901)
        small = numel * (2 * R + 4) < 16 << 20
        assert [x.kernel for x in launches(call)] == ["fused_epilogue_packed_kernel" if small else "fused_epilogue_kernel"]
        call()
        scratch, unfused = torch.empty(numel + 8, device="cuda"), torch.empty_like(residual)
        cc.cc_unfused_epilogue(values, bias, residual, unfused, scratch, first, 3072, 0.1, 12345678901)
        assert torch.equal(out, unfused)
