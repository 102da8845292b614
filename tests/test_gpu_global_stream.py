"""GPU parity of the streaming global operators where their loops turn:
lanes that count more pixels than a byte counter holds, rows narrower than a
wave, images of fewer chunks than a group has threads."""
import numpy as np
import pytest

import oracle.globalops as G
import paper_2008_11476_amd as hvx
from tests.gpu_util import log

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = hvx.hvx_context_create(0)
    yield c
    hvx.hvx_context_release(c)


def _image(ctx, arr):
    import torch
    h, w = arr.shape
    buf, view = hvx.alloc_image(h, w, hvx.HVX_DF_U8)
    buf.fill_(0xA5)  # padding
    view.copy_(torch.from_numpy(arr))
    return hvx.image_from_tensor(ctx, view, hvx.HVX_DF_U8), buf, view


def _pixels(w, h, kind):
    if kind == "flat":
        a = np.full((h, w), 201, np.uint8)
        a[h // 2, w // 2] = 7
        return a
    return np.random.default_rng(w + h).integers(3, 250, (h, w), dtype=np.uint8)


@pytest.mark.parametrize("kind", ["flat", "noise"])
@pytest.mark.parametrize("w,h", [(8192, 8192), (10007, 2503), (40, 65535), (1, 60001), (16, 64), (1025, 3)])
def test_histogram_extremes_and_equalize(ctx, w, h, kind):
    import torch
    log("global stream %dx%d %s" % (w, h, kind))
    arr = _pixels(w, h, kind)
    im, buf, view = _image(ctx, arr)
    hist = np.bincount(arr.ravel(), minlength=256)
    out = torch.full((256,), -1, dtype=torch.int32, device="cuda")
    hvx.hvx_histogram(ctx, im, 256, 0, 256, out.data_ptr())
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), hist)
    hvx.hvx_histogram(ctx, im, 10, 5, 200, out.data_ptr())
    torch.cuda.synchronize()
    assert np.array_equal(out[:10].cpu().numpy(), hist[5:205].reshape(10, 20).sum(1))
    res = torch.full((1032,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    hvx.hvx_min_max_count(ctx, im, res.data_ptr())
    lo, hi = int(arr.min()), int(arr.max())
    torch.cuda.synchronize()
    assert res[:4].cpu().tolist() == [lo, hi, int(hist[lo]), int(hist[hi])]
    eb, ev = hvx.alloc_image(h, w, hvx.HVX_DF_U8)
    eo = hvx.image_from_tensor(ctx, ev, hvx.HVX_DF_U8)
    tab = torch.zeros(160, dtype=torch.int64, device="cuda")
    hvx.hvx_equalize_hist(ctx, im, eo, tab.data_ptr())
    torch.cuda.synchronize()
    assert np.array_equal(ev.cpu().numpy(), G.equalize_hist(arr))
    hvx.hvx_release_image(im)
    hvx.hvx_release_image(eo)
