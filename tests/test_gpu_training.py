"""GPU tests of the differentiable layer's batch path: one call over a
contiguous batch gives, bit for bit, what per-image calls of the plan give,
also when saved tensors are moved by hooks, when the gradient or the input is
not contiguous, and when two calls share a plan before either's backward."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

dp = pytest.importorskip("paper_2511_04261_amd")


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _by_image(plan, x, masks, gy):
    frames, y, gx = [x[i] for i in range(len(x))], torch.empty_like(x), torch.empty_like(x)
    clip, store = plan.clip_buffers(), plan.new_store()
    plan.plan(masks, store=store)
    plan.forward(frames, out=[y[i] for i in range(len(x))], clip=clip, store=store)
    plan.backward([gy[i] for i in range(len(x))], [gx[i] for i in range(len(x))], clip, store=store)
    return y, gx


@pytest.mark.parametrize("shape,b,sb", [((3, 3, 29, 31), 8, 4), ((1, 1, 16, 16), 16, 16), ((2, 4, 33, 70), 12, 3),
                                        ((5, 3, 64, 64), 16, 8)])
@pytest.mark.parametrize("how", ["plain", "hooks", "strided", "no masks"])
def test_batch_call_equals_image_calls(dev, shape, b, sb, how):
    print("case: batch call", shape, b, sb, how, file=sys.stderr, flush=True)
    g = torch.Generator(device=dev)
    g.manual_seed(sum(shape) + b)
    B, C, H, W = shape
    x = torch.rand(shape, generator=g, device=dev) * 255.0
    gy = torch.randn(shape, generator=g, device=dev)
    masks = None if how == "no masks" else [(torch.rand(H, W, generator=g, device=dev) < 0.03).to(torch.uint8)
                                            for _ in range(B)]
    layer = dp.DPPixLayer(b, sb, 8, 1.0, 0.5, 1, seed=3)
    want_y, want_gx = _by_image(layer.plan_for(x), x, masks, gy)
    leaf = x.clone()
    if how == "strided":
        leaf = torch.empty((B, C, W, H), device=dev).transpose(2, 3).copy_(x)
        gy = torch.empty((B, H, W, C), device=dev).permute(0, 3, 1, 2).copy_(gy)
    leaf.requires_grad_(True)

    def step():
        y = layer(leaf, masks)
        other = None if masks is None else [1 - m for m in masks]
        z = layer(leaf, other)     # another call of the plan before the first one's backward
        gx, = torch.autograd.grad(y, leaf, gy)
        del z
        return y, gx

    if how == "hooks":
        with torch.autograd.graph.save_on_cpu():
            y, gx = step()
    else:
        y, gx = step()
    torch.cuda.synchronize()
    assert torch.equal(y, want_y) and torch.equal(gx, want_gx)


def test_plans_that_no_batch_holds(dev):
    """Frames of unequal geometry, or of a wider pitch, go image by image, and
    are refused or accepted as they were."""
    fps = [dp.FrameParams(16, 16, 3, dp.F32_CHW, b=8, pitch=p) for p in (16, 20)]
    for f in (fps, fps[1:]):
        plan = dp.Plan(f, device=dev)
        x = torch.zeros((len(f), 3, 16, 16), device=dev, requires_grad=True)
        assert not plan._holds_batch(x)
        with pytest.raises(ValueError):
            dp.DPPixFn.apply(x, plan, None)
    plan = dp.Plan(fps[:1], device=dev)
    with pytest.raises(ValueError):
        dp.DPPixFn.apply(torch.zeros((2, 3, 16, 16), device=dev), plan, None)
    with pytest.raises(ValueError):
        dp.DPPixFn.apply(torch.zeros((1, 3, 16, 16), device=dev, dtype=torch.float64), plan, None)
