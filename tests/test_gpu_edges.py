"""GPU parity at the edges of the vector paths: rows that start at any byte
(or float), a last strip moved back to end with the real columns, padded
columns copied from the sums of the columns they mirror, and tiles too narrow
for either (fewer real columns than one strip, or than the padding mirrors).
Every frame against the oracle; bytes past each row's end keep their sentinel.

Tolerances are those of the other parity tests: flags and counts exact,
statistics within 1e-3, bytes within one level, gradients within 1e-5.
"""
import sys

import numpy as np
import pytest

import oracle
from tests.helpers import chw_to_hwc, compare_frame, hwc_to_chw, oracle_params

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

dp = pytest.importorskip("paper_2511_04261_amd")


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


# width, b, s_b, channels, tile_cells: the last tile holds 1 to 17 real
# columns, fewer or more than its padding, on and off the strip grid
WIDTHS = [(16, 16, 4, 1, 0), (17, 16, 4, 1, 1), (31, 16, 8, 1, 1), (33, 8, 2, 3, 2), (65, 16, 4, 3, 4),
          (47, 5, 5, 3, 3), (63, 32, 8, 1, 1), (49, 48, 16, 2, 1), (70, 32, 4, 4, 2), (101, 20, 10, 3, 0),
          (1, 4, 2, 3, 0), (5, 64, 16, 3, 0), (23, 3, 1, 1, 4), (257, 256, 32, 1, 1), (130, 24, 3, 3, 0)]


def _frames(layout, pad, width_pad):
    fps = []
    for i, (w, b, s, c, k) in enumerate(WIDTHS):
        h = (b + 1, 2 * b - 1, 2 * b, 7)[i % 4]
        pitch = (w + width_pad) if layout == dp.F32_CHW else (w * c + width_pad)
        fps.append(dp.FrameParams(h, w, c, layout, b=b, sb=s, m=8, eps_bg=1.0, eps_fg=0.5, tau=1 + i % 2, pad_mode=pad,
                                  seed=9, frame_index=i, pitch=pitch, tile_cells=k))
    return fps


def _strided(fp, dev, offset, fill):
    """(buffer, frame view) with the view's first element `offset` into the buffer."""
    if fp.layout == dp.F32_CHW:
        shape, stride = (fp.channels, fp.height, fp.width), (fp.height * fp.pitch, fp.pitch, 1)
        n, dtype = fp.channels * fp.height * fp.pitch, torch.float32
    else:
        shape, stride = (fp.height, fp.width, fp.channels), (fp.pitch, fp.channels, 1)
        n, dtype = fp.height * fp.pitch, torch.uint8
    buf = torch.full((n + 2 * offset,), fill, dtype=dtype, device=dev)
    return buf, buf.as_strided(shape, stride, offset)


def _untouched(buf, view, fill):
    """Every element of the buffer outside the view still holds `fill`."""
    rest = torch.ones_like(buf, dtype=torch.bool)
    rest.as_strided(view.shape, view.stride(), view.storage_offset()).fill_(False)
    return bool((buf[rest] == fill).all())


@pytest.mark.parametrize("pad", [0, 1, 2])
@pytest.mark.parametrize("offset,width_pad", [(0, 0), (1, 3), (16, 16)])
def test_u8_rows_at_any_byte(dev, pad, offset, width_pad):
    say("case: u8 edges", pad, offset, width_pad)
    r = np.random.Generator(np.random.PCG64(100 * pad + offset))
    fps = _frames(dp.U8_HWC, pad, width_pad)
    xs = [r.integers(0, 256, (f.height, f.width, f.channels)).astype(np.uint8) for f in fps]
    ms = [(r.random((f.height, f.width)) < 0.02).astype(np.uint8) * 3 for f in fps]
    ins = [_strided(f, dev, offset, 0) for f in fps]
    for (_, v), x in zip(ins, xs):
        v.copy_(torch.from_numpy(x).to(dev))
    fused, rebuilt = ([_strided(f, dev, offset, 77) for f in fps] for _ in range(2))
    plan = dp.Plan(fps, device=dev)
    plan.plan([torch.from_numpy(m).to(dev) for m in ms])
    plan.forward([v for _, v in ins], out=[v for _, v in fused])
    plan.reconstruct([v for _, v in rebuilt])
    torch.cuda.synchronize()
    store = plan.store_host()
    for i, f in enumerate(fps):
        want = oracle.forward(xs[i], ms[i], oracle_params(f))
        for buf, v in (fused[i], rebuilt[i]):
            compare_frame(store[i], want, v.cpu().numpy(), "frame %d" % i)
            assert _untouched(buf, v, 77), i
    plan.close()


@pytest.mark.parametrize("pad", [0, 1, 2])
@pytest.mark.parametrize("offset,width_pad", [(0, 0), (1, 1), (4, 4)])
def test_f32_rows_at_any_float(dev, pad, offset, width_pad):
    say("case: f32 edges", pad, offset, width_pad)
    r = np.random.Generator(np.random.PCG64(1000 + 100 * pad + offset))
    fps = _frames(dp.F32_CHW, pad, width_pad)
    xs = [(r.random((f.channels, f.height, f.width)) * 255.0).astype(np.float32) for f in fps]
    gs = [r.standard_normal((f.channels, f.height, f.width)).astype(np.float32) for f in fps]
    ms = [(r.random((f.height, f.width)) < 0.02).astype(np.uint8) for f in fps]
    ins, gos = ([_strided(f, dev, offset, 0.0) for f in fps] for _ in range(2))
    for (_, v), (_, g), x, gx in zip(ins, gos, xs, gs):
        v.copy_(torch.from_numpy(x).to(dev))
        g.copy_(torch.from_numpy(gx).to(dev))
    fused, rebuilt, gis = ([_strided(f, dev, offset, -7.0) for f in fps] for _ in range(3))
    plan = dp.Plan(fps, device=dev)
    clip = plan.clip_buffers()
    plan.plan([torch.from_numpy(m).to(dev) for m in ms])
    plan.forward([v for _, v in ins], out=[v for _, v in fused], clip=clip)
    plan.reconstruct([v for _, v in rebuilt])
    plan.backward([v for _, v in gos], [v for _, v in gis], clip)
    torch.cuda.synchronize()
    store = plan.store_host()
    for i, f in enumerate(fps):
        want = oracle.forward(chw_to_hwc(xs[i]), ms[i], oracle_params(f))
        for buf, v in (fused[i], rebuilt[i]):
            compare_frame(store[i], want, chw_to_hwc(v.cpu().numpy()), "frame %d" % i)
            assert _untouched(buf, v, -7.0), i
        gw = oracle.backward(chw_to_hwc(xs[i]).astype(np.float64), ms[i], chw_to_hwc(gs[i]).astype(np.float64),
                             oracle_params(f))
        got = chw_to_hwc(gis[i][1].cpu().numpy())
        assert np.abs(got - gw).max() <= 1e-5 * max(1.0, np.abs(gw).max()), i
        assert _untouched(gis[i][0], gis[i][1], -7.0), i
    plan.close()


@pytest.mark.parametrize("offset,width_pad", [(0, 0), (1, 5), (16, 16)])
def test_metrics_at_unit_edges(dev, offset, width_pad):
    """Frames around the metrics kernel's pixel groups, units of columns and
    blocks of rows, for every channel count: MSE exact, SSIM within 1e-9."""
    say("case: metrics edges", offset, width_pad)
    r = np.random.Generator(np.random.PCG64(500 + offset))
    shapes = [(7, 7, 3), (8, 13, 1), (14, 16, 2), (13, 17, 4), (15, 31, 3), (7, 165, 3), (21, 166, 3), (9, 167, 3),
              (64, 128, 4), (16, 133, 4), (70, 135, 4), (20, 262, 2), (71, 257, 2), (65, 518, 1), (10, 519, 1),
              (77, 320, 3), (6, 200, 3), (40, 6, 3), (1, 1, 1), (133, 337, 3)]
    fps, xs, ys = [], [], []
    for i, (h, w, c) in enumerate(shapes):
        fps.append(dp.FrameParams(h, w, c, dp.U8_HWC, b=(8, 16, 5)[i % 3], pitch=w * c + width_pad))
        x = r.integers(0, 256, (h, w, c))
        xs.append(x.astype(np.uint8))
        ys.append(np.clip(x // 3 + r.integers(0, 90, (h, w, c)), 0, 255).astype(np.uint8))
    ti, to = ([_strided(f, dev, offset, 255)[1] for f in fps] for _ in range(2))
    for i in range(len(shapes)):
        ti[i].copy_(torch.from_numpy(xs[i]).to(dev))
        to[i].copy_(torch.from_numpy(ys[i]).to(dev))
    plan = dp.Plan(fps, device=dev)
    got = plan.metrics(ti, to).cpu().numpy()
    for i, (h, w, c) in enumerate(shapes):
        assert got[i, 0] == pytest.approx(((xs[i].astype(float) - ys[i].astype(float)) ** 2).mean(), rel=1e-15, abs=0), i
        ssim = oracle.metrics(xs[i], ys[i])[1] if h >= 7 and w >= 7 else 0.0
        assert abs(got[i, 1] - ssim) <= 1e-9, (i, got[i, 1], ssim)
    plan.close()


@pytest.mark.parametrize("pad", [0, 1, 2])
@pytest.mark.parametrize("offset,width_pad", [(0, 0), (3, 2)])
def test_labels_at_group_edges(dev, pad, offset, width_pad):
    """Widths around the label kernels' 16-pixel groups, four-column lanes and
    walks of 992 columns, bands of every parity: the masks equal the oracle's,
    nothing beside them is written, and the fused plan equals the two-step one."""
    say("case: label edges", pad, offset, width_pad)
    r = np.random.Generator(np.random.PCG64(700 + 10 * pad + offset))
    shapes = [(9, 1, 3, 4, 0), (5, 15, 1, 4, 1), (33, 16, 3, 16, 0), (18, 17, 2, 5, 2), (31, 31, 3, 32, 0),
              (14, 33, 4, 7, 3), (257, 47, 1, 256, 0), (20, 64, 3, 3, 9), (35, 130, 3, 129, 0), (8, 991, 1, 8, 0),
              (19, 992, 3, 16, 0), (7, 993, 1, 2, 0), (34, 1010, 3, 32, 0), (6, 1999, 2, 12, 100), (300, 21, 3, 150, 1)]
    fps, xs = [], []
    for i, (h, w, c, b, k) in enumerate(shapes):
        fps.append(dp.FrameParams(h, w, c, dp.U8_HWC, b=b, sb=b, m=8, tau=1 + i % 3, pad_mode=pad, pitch=w * c + width_pad,
                                  tile_cells=k))
        xs.append(r.integers(0, 256, (h, w, c)).astype(np.uint8) // (1 + 9 * (r.random((h, w, 1)) < 0.7)).astype(np.uint8))
    ti = [_strided(f, dev, offset, 255)[1] for f in fps]
    for v, x in zip(ti, xs):
        v.copy_(torch.from_numpy(x).to(dev))
    bufs = [torch.full((f.height * f.width + 2 * offset,), 9, dtype=torch.uint8, device=dev) for f in fps]
    masks = [t[offset:offset + f.height * f.width].view(f.height, f.width) for t, f in zip(bufs, fps)]
    plan = dp.Plan(fps, device=dev)
    one, two = plan.new_store(), plan.new_store()
    plan.edge_masks(ti, 90, out=masks)
    plan.plan(masks, store=two)
    plan.plan_labels(ti, 90, store=one)
    torch.cuda.synchronize()
    for i, x in enumerate(xs):
        assert np.array_equal(masks[i].cpu().numpy(), oracle.edge_mask(x, 90, pad)), i
        assert _untouched(bufs[i], masks[i], 9), i
    assert torch.equal(one.flags, two.flags) and torch.equal(one.counts, two.counts)
    plan.close()


@pytest.mark.parametrize("b", [1, 2, 3, 4, 8, 12, 16, 20, 24, 48])
@pytest.mark.parametrize("pad", [0, 2])
def test_mask_counts_of_every_cell_size(dev, b, pad):
    """Cell sizes on each path of the mask count (whole short bands, four
    columns a dword, column by column), rows of whole strips and not, bands
    past the frame, mask bytes of any nonzero value: flags equal the oracle's."""
    say("case: mask counts", b, pad)
    r = np.random.Generator(np.random.PCG64(900 + b + pad))
    shapes = [(5 * b, 96, 0), (8 * b + 1, 192, 0), (16 * b - 1, 208, 0), (3, 64, 0), (40, 250, 0), (4 * b, 16 * b, 3)]
    fps, ms = [], []
    for i, (h, w, k) in enumerate(shapes):
        fps.append(dp.FrameParams(h, w, 1, dp.U8_HWC, b=b, sb=b, m=8, tau=(1, 2, 0)[i % 3] if b > 1 else 1, pad_mode=pad,
                                  tile_cells=k))
        ms.append((r.random((h, w)) < (0.3, 0.05, 0.6)[i % 3]) * r.choice([1, 2, 127, 128, 255], (h, w)))
    ms = [m.astype(np.uint8) for m in ms]
    plan = dp.Plan(fps, device=dev)
    plan.plan([torch.from_numpy(m).to(dev) for m in ms])
    store = plan.store_host()
    for i, f in enumerate(fps):
        x = np.zeros((f.height, f.width, 1), np.uint8)
        want = oracle.forward(x, ms[i], oracle_params(f))
        assert np.array_equal(store[i]["flags"], want["flags"]), i
        assert tuple(store[i]["counts"]) == tuple(want["counts"]), i
    plan.close()


# frames, height, width, b, s_b, layout: every workgroup size of forward and
# reconstruction (few tiles: 128, 256, 512 lanes; many: 128 or 256, the
# reconstruction of large tiles in a large batch 512), and batches of several
BATCHES = [[(1, 64, 16, 16, 4, dp.U8_HWC)], [(1, 64, 200, 16, 4, dp.U8_HWC)], [(2, 96, 700, 32, 4, dp.U8_HWC)],
           [(60, 90, 333, 16, 4, dp.U8_HWC)], [(60, 120, 640, 16, 4, dp.U8_HWC)], [(70, 1024, 640, 32, 8, dp.U8_HWC)],
           [(70, 1024, 640, 32, 8, dp.U8_HWC), (5, 61, 100, 8, 4, dp.U8_HWC), (3, 77, 300, 16, 8, dp.F32_CHW)],
           [(40, 61, 50, 8, 4, dp.F32_CHW), (2, 130, 512, 16, 2, dp.F32_CHW)]]


@pytest.mark.parametrize("batch", BATCHES, ids=range(len(BATCHES)))
def test_workgroup_sizes_give_equal_results(batch, dev):
    """The sizes chosen per launch group against one fixed size: equal bytes."""
    fps, images = [], []
    rng = np.random.default_rng(17)
    for n, h, w, b, s, layout in batch:
        x = rng.integers(0, 256, (h, w, 3), dtype=np.uint8)
        if layout == dp.F32_CHW:
            x = hwc_to_chw(x).astype(np.float32)
        x = torch.from_numpy(x).to(dev)
        for _ in range(n):
            fps.append(dp.FrameParams(h, w, 3, layout, b=b, sb=s, m=8, eps_bg=1.0, eps_fg=0.5, tau=1, seed=9,
                                      frame_index=len(fps)))
            images.append(x)
    masks = [torch.from_numpy(rng.integers(0, 40, (f.height, f.width), dtype=np.uint8) // 39).to(dev) for f in fps]
    got = []
    for threads in (0, 256):
        plan = dp.Plan(fps, device=dev, threads=threads)
        plan.plan(masks)
        fused = [torch.empty_like(x) for x in images]
        plan.forward(images, out=fused)
        rebuilt = [torch.empty_like(x) for x in images]
        plan.reconstruct(rebuilt)
        torch.cuda.synchronize()
        got.append((fused, rebuilt))
    for i in range(len(fps)):
        for k in range(2):
            assert torch.equal(got[0][k][i], got[1][k][i]), (i, k)


# frames of the batch: (count, height, width, channels, b, s_b, tile_cells); one C and n or several, 1 to 513
# frames, tiles of a frame around 8, 2048 and 4096 of the scan's rounds, prefixes that end inside a 16-byte group
SCANS = [[(1, 64, 64, 3, 2, 1, 1)], [(3, 128, 128, 1, 2, 1, 1), (2, 5, 5, 3, 5, 1, 0)],
         [(1, 7, 5, 1, 1, 1, 1), (1, 90, 91, 2, 2, 1, 1), (1, 3, 3, 4, 1, 1, 1), (1, 91, 91, 3, 2, 2, 1)],
         [(511, 6, 9, 3, 4, 2, 1), (1, 9, 9, 1, 4, 1, 0)], [(512, 6, 9, 3, 4, 2, 1), (1, 9, 9, 1, 4, 1, 0)],
         [(40, 33, 65, 3, 16, 4, 1), (40, 47, 31, 1, 8, 4, 1)], [(90, 40, 60, 3, 4, 2, 1), (3, 16, 16, 3, 16, 4, 0)],
         [(2, 128, 300, 3, 2, 1, 1)], [(1, 256, 64, 1, 2, 1, 1), (7, 17, 19, 3, 4, 4, 1)]]


@pytest.mark.parametrize("batch", SCANS, ids=range(len(SCANS)))
def test_store_offsets_of_any_batch(batch, dev):
    """Counts and offsets of every frame against sums over its flags; the statistics end up where they say."""
    fps, masks, images = [], [], []
    rng = np.random.default_rng(23)
    for n, h, w, c, b, s, k in batch:
        for _ in range(n):
            fps.append(dp.FrameParams(h, w, c, b=b, sb=s, m=8, eps_bg=float("inf"), eps_fg=float("inf"), tau=1, seed=9,
                                      frame_index=len(fps), tile_cells=k))
    order = rng.permutation(len(fps))
    fps = [fps[i] for i in order]
    for f in fps:
        masks.append(torch.from_numpy((rng.random((f.height, f.width)) < 0.2).astype(np.uint8)).to(dev))
        images.append(torch.from_numpy(rng.integers(0, 256, (f.height, f.width, f.channels), dtype=np.uint8)).to(dev))
    plan = dp.Plan(fps, device=dev)
    plan.plan(masks)
    fused = [torch.empty_like(x) for x in images]
    plan.forward(images, out=fused)
    rebuilt = [torch.empty_like(x) for x in images]
    plan.reconstruct(rebuilt)
    torch.cuda.synchronize()
    counts = plan.store.counts.cpu().numpy().view(np.uint64).reshape(len(fps), 4)
    bg = fg = 0
    for i, (f, st) in enumerate(zip(fps, plan.store_host())):
        n2 = (f.b // f.sb) ** 2
        nf = int((st["flags"] != 0).sum())
        nb = st["flags"].size - nf
        assert counts[i].tolist() == [nb, nf, bg, fg], i
        bg += nb * f.channels
        fg += nf * n2 * f.channels
        assert torch.equal(fused[i], rebuilt[i]), i


@pytest.mark.parametrize("b", [10, 12])
@pytest.mark.parametrize("persistent", [0, 1])
def test_paced_reconstruction_gives_equal_bytes(dev, b, persistent):
    """Batches whose reconstruction paces its stores (RGB, two subgrid rows of
    five or six), of whole and ragged tiles and rows at any byte: the bytes of
    the fused forward, and of a batch in which another frame keeps the group
    from pacing."""
    say("case: paced reconstruction", b, persistent)
    r = np.random.Generator(np.random.PCG64(b))
    shapes = [(60, 768), (61, 767), (b, 5 * b), (7, 30), (b + 1, 400), (3, 3)]
    fps = [dp.FrameParams(h, w, 3, dp.U8_HWC, b=b, sb=b // 2, m=8, tau=1, seed=2, frame_index=i, pitch=3 * w + i % 3)
           for i, (h, w) in enumerate(shapes)]
    other = dp.FrameParams(50, 300, 3, dp.U8_HWC, b=16, sb=4, m=8, tau=1, seed=2, frame_index=99, pitch=900)
    xs = [r.integers(0, 256, (f.height, f.width, 3)).astype(np.uint8) for f in fps + [other]]
    ms = [torch.from_numpy((r.random((f.height, f.width)) < 0.02).astype(np.uint8)).to(dev) for f in fps + [other]]
    got = []
    for frames in (fps, fps + [other]):
        ins, fused, rebuilt = ([_strided(f, dev, 1, fill) for f in frames] for fill in (0, 77, 77))
        for (_, v), x in zip(ins, xs):
            v.copy_(torch.from_numpy(x).to(dev))
        plan = dp.Plan(frames, device=dev, persistent=persistent)
        plan.plan(ms[:len(frames)])
        plan.forward([v for _, v in ins], out=[v for _, v in fused])
        plan.reconstruct([v for _, v in rebuilt])
        torch.cuda.synchronize()
        for i in range(len(frames)):
            assert torch.equal(fused[i][0], rebuilt[i][0]), i
            assert _untouched(rebuilt[i][0], rebuilt[i][1], 77), i
        got.append([buf for buf, _ in rebuilt])
        plan.close()
    for i in range(len(fps)):
        assert torch.equal(got[0][i], got[1][i]), i
