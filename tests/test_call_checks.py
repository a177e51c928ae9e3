"""Host checks of a call's tensors: the short comparison that most tensors
pass on accepts only what the full check accepts, and what it does not accept
is decided by the full check, over shapes, strides, types and devices."""
import itertools

import pytest

torch = pytest.importorskip("torch")

import paper_2511_04261_amd as dp  # noqa: E402


class OnGpu:
    """A CPU tensor's geometry, said to live on a GPU."""

    def __init__(self, t, index=0):
        self.t, self.index = t, index
        self.shape, self.dtype, self.is_cuda = t.shape, t.dtype, index is not None
        self.device = torch.device("cuda", index) if index is not None else torch.device("cpu")

    def stride(self, *a):
        return self.t.stride(*a)

    def dim(self):
        return self.t.dim()

    def numel(self):
        return self.t.numel()

    def element_size(self):
        return self.t.element_size()

    def data_ptr(self):
        return self.t.data_ptr()

    def get_device(self):
        return -1 if self.index is None else self.index


def _plan(fp, index):
    plan = dp.Plan.__new__(dp.Plan)
    plan.frames = [fp]
    plan.device = torch.device("cuda") if index is None else torch.device("cuda", index)
    plan._expect = [dp._expected(fp.desc())]
    return plan


def _forms(h, w, c, dtype):
    """Tensors of the frame's elements in every order, with gaps, and of other sizes."""
    flat = torch.zeros(8 * h * w * c + 64, dtype=dtype)
    for dims in itertools.permutations((h, w, c)):
        base = flat[:h * w * c].view(dims)
        for p in itertools.permutations(range(3)):
            yield base.permute(p)
    yield flat[:h * w].view(h, w)
    yield flat[:w * h].view(w, h).t()
    for pad in (1, 5):
        yield flat.as_strided((h, w, c), ((w + pad) * c, c, 1))
        yield flat.as_strided((c, h, w), ((w + pad) * h, w + pad, 1))
        yield flat.as_strided((c, h, w), ((w + pad) * (h + 1), w + pad, 1))
        yield flat.as_strided((h, w), (w + pad, 1))
        yield flat.as_strided((h, w, c), ((w + pad) * c, 2 * c, 2))
    yield flat.as_strided((h, w, c), (0, 0, 0))
    yield flat[:(h + 1) * w * c].view(h + 1, w, c)
    yield flat[:h * w * c].view(1, h, w, c)


@pytest.mark.parametrize("h,w,c", [(6, 5, 3), (5, 7, 1), (1, 4, 2), (4, 1, 4), (1, 1, 1)])
@pytest.mark.parametrize("layout", [dp.U8_HWC, dp.F32_CHW])
@pytest.mark.parametrize("pad", [0, 1])
def test_short_check_agrees_with_the_full_one(h, w, c, layout, pad):
    pitch = (w + pad) * (c if layout == dp.U8_HWC else 1)
    fp = dp.FrameParams(h, w, c, layout, b=4, pitch=pitch)
    seen = set()
    for dtype in (torch.uint8, torch.float32, torch.int8):
        for t in _forms(h, w, c, dtype):
            for index, where in ((None, 0), (0, 0), (0, 1), (1, 1), (0, None)):
                plan, x = _plan(fp, index), OnGpu(t, where)
                try:
                    plan._check_images([x], "images")
                    want = None
                except ValueError as e:
                    want = str(e)
                try:
                    got = plan._addresses([x], "images")
                    assert want is None and got == (t.data_ptr(),), (t.shape, t.stride(), dtype, want)
                    span = dp._span(x)
                    assert plan._expect[0][3] == span[1] - span[0]
                except ValueError as e:
                    assert str(e) == want, (t.shape, t.stride(), dtype, want)
                seen.add(want is None)
    assert seen == {True, False}
    with pytest.raises(ValueError, match="need one tensor per frame"):
        _plan(fp, 0)._addresses([], "images")


def test_overlap_by_addresses_agrees_with_the_spans():
    fp = dp.FrameParams(4, 5, 3, dp.U8_HWC, b=4, pitch=20)
    plan, flat = _plan(fp, 0), torch.zeros(400, dtype=torch.uint8)
    for d in range(-80, 81):
        a, b = (OnGpu(flat.as_strided((4, 5, 3), (20, 3, 1), 160 + o)) for o in (0, d))
        want = None
        try:
            dp.check_no_alias([a], [b])
        except ValueError as e:
            want = str(e)
        try:
            plan._no_alias(plan._addresses([a], "images"), plan._addresses([b], "out"))
            assert want is None, d
        except ValueError as e:
            assert str(e) == want, d


class _Evicting(dict):
    """A table cache that another thread empties after every look at it."""

    def __contains__(self, key):
        found = super().__contains__(key)
        self.clear()
        return found or True

    def move_to_end(self, key):
        pass

    def popitem(self, last=True):
        raise AssertionError("nothing to evict")


@pytest.mark.parametrize("n", [1, 3])
def test_batch_table_holds_every_image_when_it_was_evicted(n):
    """A batch's pointer table has one address per frame, also where the table
    of its base address goes away between two looks at the cache (the kernels
    read an entry per frame)."""
    plan = dp.Plan.__new__(dp.Plan)
    plan.frames, plan.device, plan._tables = [None] * n, torch.device("cpu"), _Evicting()
    x = torch.zeros((n, 3, 4, 5))
    for _ in range(2):
        assert plan._batch_table(x).tolist() == [x[i].data_ptr() for i in range(n)]
        plan._tables.clear()


@pytest.mark.parametrize("pad", [0, 3])
def test_gray_frames_pass_the_short_check_in_both_forms(pad):
    """(H, W) and (H, W, 1) tensors of a gray frame are accepted without the
    full check; the same with a gap between pixels are not."""
    fp = dp.FrameParams(6, 5, 1, dp.U8_HWC, b=4, pitch=5 + pad)
    plan = _plan(fp, 0)
    full = []
    plan._check_images = lambda tensors, what, frames=None: full.append(tensors)
    flat = torch.zeros(200, dtype=torch.uint8)
    for shape, stride, short in (((6, 5, 1), (5 + pad, 1, 1), True), ((6, 5), (5 + pad, 1), True), ((6, 5), (5 + pad, 2), False),
                                 ((5, 6), (5 + pad, 1), False), ((6, 5), (6 + pad, 1), False)):
        x = OnGpu(flat.as_strided(shape, stride))
        assert plan._addresses([x], "images") == (flat.data_ptr(),)
        assert (not full) == short, (shape, stride)
        full.clear()
