"""GPU tests of fp32 frames that hold NaN or infinite pixels: a statistic whose
sum is NaN is released, stored, rebuilt and trained through as NaN, an infinite
one is clipped, both as the oracle has them; no other statistic changes.
Tolerances are those of the other parity tests (statistics within 1e-3,
gradients within 1e-5)."""
import sys

import numpy as np
import pytest

import oracle
from tests.helpers import STAT_TOL, chw_to_hwc, hwc_to_chw, oracle_params

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

dp = pytest.importorskip("paper_2511_04261_amd")

INF = float("inf")
# (row, column, channel, value) on a 45 x 61 frame of 8 x 8 cells, subcells of 4
PIXELS = [(2, 3, 0, np.nan), (2, 12, 1, INF), (3, 20, 2, -INF), (1, 27, 0, INF), (6, 30, 0, -INF),
          (19, 9, 1, np.nan), (17, 18, 0, INF), (18, 19, 0, -INF), (21, 30, 2, -INF),
          (43, 5, 0, np.nan), (10, 59, 2, np.nan), (44, 60, 1, INF)]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _inputs(seed):
    r = np.random.Generator(np.random.PCG64(seed))
    x = (r.random((45, 61, 3)) * 255.0).astype(np.float32)
    for row, col, ch, v in PIXELS:
        x[row, col, ch] = v
    mask = np.zeros((45, 61), np.uint8)
    mask[16:24] = 1                       # the third band of cells is complex
    return r, x, mask


def _params(pad, eps):
    return dp.FrameParams(45, 61, 3, dp.F32_CHW, b=8, sb=4, m=8, eps_bg=eps, eps_fg=eps / 2, tau=1, pad_mode=pad, seed=3,
                          frame_index=5)


@pytest.mark.parametrize("pad", [0, 1, 2])
@pytest.mark.parametrize("eps", [1.0, INF])
def test_nonfinite_pixels_as_the_oracle_has_them(dev, pad, eps):
    print("case: nonfinite pixels", pad, eps, file=sys.stderr, flush=True)
    _, x, mask = _inputs(7 + pad)
    fp = _params(pad, eps)
    want = oracle.forward(x, mask, oracle_params(fp))
    assert np.isnan(want["bg"]).any() and np.isnan(want["fg"]).any()
    plan = dp.Plan([fp], device=dev)
    ti = torch.from_numpy(hwc_to_chw(x)).to(dev)
    fused, rebuilt = torch.empty_like(ti), torch.empty_like(ti)
    clip = plan.clip_buffers()
    plan.plan([torch.from_numpy(mask).to(dev)])
    plan.forward([ti], out=[fused], clip=clip)
    plan.reconstruct([rebuilt])
    torch.cuda.synchronize()
    st = plan.store_host()[0]
    for k in ("bg", "fg"):
        np.testing.assert_allclose(st[k], want[k], rtol=0, atol=STAT_TOL, equal_nan=True)
    for got in (fused, rebuilt):
        np.testing.assert_allclose(chw_to_hwc(got.cpu().numpy()), want["recon_f32"], rtol=0, atol=STAT_TOL,
                                   equal_nan=True)
    nb, nf = want["pass_bg"].size, want["pass_fg"].size
    assert np.array_equal(clip[0].cpu().numpy()[:nb], want["pass_bg"].reshape(-1))
    assert np.array_equal(clip[1].cpu().numpy()[:nf], want["pass_fg"].reshape(-1))
    plan.close()


def test_layer_shows_a_diverged_input(dev):
    print("case: layer on nonfinite pixels", file=sys.stderr, flush=True)
    r, x, mask = _inputs(11)
    layer = dp.DPPixLayer(8, 4, 8, 1.0, 0.5, 1, seed=3, first_frame_index=5)
    gy = r.standard_normal(x.shape).astype(np.float32)
    leaf = torch.from_numpy(hwc_to_chw(x)).to(dev)[None].requires_grad_(True)
    y = layer(leaf, [torch.from_numpy(mask).to(dev)])
    gx, = torch.autograd.grad(y, leaf, torch.from_numpy(hwc_to_chw(gy)).to(dev)[None])
    p = oracle_params(_params(0, 1.0))
    want = oracle.forward(x, mask, p)["recon_f32"]
    np.testing.assert_allclose(chw_to_hwc(y[0].detach().cpu().numpy()), want, rtol=0, atol=STAT_TOL, equal_nan=True)
    gw = oracle.backward(x, mask, gy, p)
    assert np.abs(chw_to_hwc(gx[0].cpu().numpy()) - gw).max() <= 1e-5 * max(1.0, np.abs(gw).max())
