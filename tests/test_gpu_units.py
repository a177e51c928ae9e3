"""GPU tests of the kernels that find their unit's frame by a search over the
batch's frames (label masks, plans from labels, metrics, the adjoint's mirror
pass): batches around the search's steps of 64 and 4096 frames, with frames of
several sizes and channel counts, against the oracle.  Tolerances are those of
the other parity tests."""
import sys

import numpy as np
import pytest

import oracle
from tests.helpers import chw_to_hwc, hwc_to_chw, oracle_params

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

dp = pytest.importorskip("paper_2511_04261_amd")

SIZES = [(9, 10), (7, 23), (12, 8), (30, 200), (8, 7)]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _views(arrays, dev):
    """GPU tensors of the arrays, slices of one buffer (one upload)."""
    flat = torch.from_numpy(np.concatenate([a.reshape(-1) for a in arrays])).to(dev)
    out, at = [], 0
    for a in arrays:
        out.append(flat[at:at + a.size].view(a.shape))
        at += a.size
    return flat, out


@pytest.mark.parametrize("n", [1, 63, 64, 65, 129, 4096, 4161])
def test_byte_units(dev, n):
    print("case: byte units", n, file=sys.stderr, flush=True)
    r = np.random.Generator(np.random.PCG64(n))
    fps, xs, ys = [], [], []
    for i in range(n):
        h, w = SIZES[int(r.integers(len(SIZES)))] if i % 97 else (70, 333)
        c = int(r.integers(1, 5)) if n % 2 else 3
        fps.append(dp.FrameParams(h, w, c, dp.U8_HWC, b=4, sb=2, m=8, tau=2, frame_index=i))
        xs.append((r.integers(0, 256, (h, w, c)) // (1 + 9 * (r.random((h, w, 1)) < 0.7))).astype(np.uint8))
        ys.append(np.clip(xs[-1] // 3 + r.integers(0, 90, (h, w, c)), 0, 255).astype(np.uint8))
    _, ti = _views(xs, dev)
    _, to = _views(ys, dev)
    plan = dp.Plan(fps, device=dev)
    masks = plan.edge_masks(ti, 60)
    one, two = plan.new_store(), plan.new_store()
    plan.plan(masks, store=two)
    plan.plan_labels(ti, 60, store=one)
    got = plan.metrics(ti, to).cpu().numpy()
    assert torch.equal(one.flags, two.flags) and torch.equal(one.counts, two.counts)
    flat = torch.cat([m.reshape(-1) for m in masks]).cpu().numpy()
    assert np.array_equal(flat, np.concatenate([oracle.edge_mask(x, 60, 0).reshape(-1) for x in xs]))
    for i in range(n):
        want = oracle.metrics(xs[i], ys[i])
        assert abs(got[i, 0] - want[0]) <= 1e-12 * want[0] and abs(got[i, 1] - want[1]) <= 1e-9, i
    plan.close()


@pytest.mark.parametrize("n,pad", [(1, 0), (64, 1), (65, 0), (130, 2), (4100, 0)])
def test_mirror_units(dev, n, pad):
    print("case: mirror units", n, pad, file=sys.stderr, flush=True)
    r = np.random.Generator(np.random.PCG64(10 * n + pad))
    fps, xs, gs, ms = [], [], [], []
    for i in range(n):
        h, w = SIZES[int(r.integers(len(SIZES)))] if i % 97 else (41, 333)
        fps.append(dp.FrameParams(h, w, 1 + i % 3, dp.F32_CHW, b=8 if i % 5 else 64, sb=4, m=8, eps_bg=1.0, eps_fg=0.5, tau=1,
                                  pad_mode=pad, seed=4, frame_index=i))
        xs.append((r.random((1 + i % 3, h, w)) * 255.0).astype(np.float32))
        gs.append(r.standard_normal((1 + i % 3, h, w)).astype(np.float32))
        ms.append((r.random((h, w)) < 0.02).astype(np.uint8))
    _, ti = _views(xs, dev)
    _, tg = _views(gs, dev)
    _, tm = _views(ms, dev)
    flat, tx = _views([np.zeros_like(x) for x in xs], dev)
    plan = dp.Plan(fps, device=dev)
    clip = plan.clip_buffers()
    plan.plan(tm)
    plan.forward(ti, clip=clip)
    plan.backward(tg, tx, clip)
    host, at = flat.cpu().numpy(), 0
    for i in range(n):
        gw = oracle.backward(chw_to_hwc(xs[i]), ms[i], chw_to_hwc(gs[i]), oracle_params(fps[i]))
        got = host[at:at + xs[i].size].reshape(xs[i].shape)
        at += xs[i].size
        assert np.abs(got - hwc_to_chw(gw)).max() <= 1e-5 * max(1.0, np.abs(gw).max()), i
    plan.close()


@pytest.mark.parametrize("c", [1, 2, 3, 4])
@pytest.mark.parametrize("narrow", [True, False])
def test_metrics_of_narrow_and_wide_units(dev, c, narrow):
    """Widths around the edges of both kinds of metrics units (a wave's and a
    workgroup's lanes), in a batch whose frames take the one kind, or, with a
    frame that outweighs them, the other: MSE exact, SSIM within 1e-9."""
    print("case: metrics units", c, narrow, file=sys.stderr, flush=True)
    r = np.random.Generator(np.random.PCG64(40 + c))
    small, wide = 64 // c // 16 * 16, 512 // c // 16 * 16
    widths = [7, 15, 16, 17, 23] + [w + d for w in (small, 2 * small, wide) for d in (-1, 0, 1, 6, 7)]
    shapes = [((7, 8, 14, 21, 30, 33)[i % 6], max(w, 7)) for i, w in enumerate(widths)]
    if not narrow:
        shapes.append((400, 4 * wide))
    xs = [r.integers(0, 256, (h, w, c)) for h, w in shapes]
    ys = [np.clip(x // 3 + r.integers(0, 90, x.shape), 0, 255).astype(np.uint8) for x in xs]
    xs = [x.astype(np.uint8) for x in xs]
    _, ti = _views(xs, dev)
    _, to = _views(ys, dev)
    plan = dp.Plan([dp.FrameParams(h, w, c, dp.U8_HWC, b=8) for h, w in shapes], device=dev)
    got = plan.metrics(ti, to).cpu().numpy()
    for i in range(len(shapes)):
        mse, ssim = oracle.metrics(xs[i], ys[i])
        assert abs(got[i, 0] - mse) <= 1e-12 * mse and abs(got[i, 1] - ssim) <= 1e-9, (shapes[i], got[i], ssim)
    plan.close()


@pytest.mark.parametrize("n", [2, 66])
def test_frames_of_as_many_units(dev, n):
    """Batches in which every frame has as many units (the unit's frame then
    comes from a division), also of one channel count only."""
    print("case: equal frames", n, file=sys.stderr, flush=True)
    r = np.random.Generator(np.random.PCG64(n))
    cs = [3] * n if n == 2 else [1 + i % 4 for i in range(n)]
    xs = [(r.integers(0, 256, (50, 190, c)) // (1 + 9 * (r.random((50, 190, 1)) < 0.7))).astype(np.uint8) for c in cs]
    ys = [np.clip(x // 3 + r.integers(0, 90, x.shape), 0, 255).astype(np.uint8) for x in xs]
    _, ti = _views(xs, dev)
    _, to = _views(ys, dev)
    plan = dp.Plan([dp.FrameParams(50, 190, c, dp.U8_HWC, b=8, sb=4, m=8, tau=2) for c in cs], device=dev)
    masks = plan.edge_masks(ti, 60)
    one, two = plan.new_store(), plan.new_store()
    plan.plan(masks, store=two)
    plan.plan_labels(ti, 60, store=one)
    got = plan.metrics(ti, to).cpu().numpy()
    assert torch.equal(one.flags, two.flags) and torch.equal(one.counts, two.counts)
    for i in range(n):
        assert np.array_equal(masks[i].cpu().numpy(), oracle.edge_mask(xs[i], 60, 0)), i
        want = oracle.metrics(xs[i], ys[i])
        assert abs(got[i, 0] - want[0]) <= 1e-12 * want[0] and abs(got[i, 1] - want[1]) <= 1e-9, i
    plan.close()
