"""GPU: min_max_count of images far smaller than its 256 counting keys.  The
result is exact, and no call takes much longer on the device than min_max, which
reads the same bytes (the keys that no work-group owns are set side by side)."""
import time

import numpy as np
import pytest

import oracle.globalops as G
import paper_2008_11476_amd as hvx
import synth
from tests.gpu_util import device_image, log

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = hvx.hvx_context_create(0)
    yield c
    hvx.hvx_context_release(c)


def _device_us(call):
    """Device time of a call: the best of several replays of 50 captured ones."""
    import torch
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        call(s.cuda_stream)
        torch.cuda.synchronize()
        with torch.cuda.graph(g, stream=s):
            for _ in range(50):
                call(torch.cuda.current_stream().cuda_stream)
    best = 1e9
    for _ in range(20):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        g.replay()
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t0) / 50 * 1e6)
    return best


@pytest.mark.parametrize("dtype", [np.uint8, np.int16])
@pytest.mark.parametrize("w,h", [(1, 1), (17, 2), (64, 64), (300, 200)])
def test_min_max_count_of_small_images(ctx, w, h, dtype):
    import torch
    img = synth.uniform_u8(w, h, seed=w) if dtype == np.uint8 else synth.uniform_s16(w, h, seed=w)
    im, keep = device_image(ctx, img, hvx.HVX_DF_U8 if dtype == np.uint8 else hvx.HVX_DF_S16)
    out = torch.full((4128,), 0x5A, dtype=torch.uint8, device="cuda")
    log("small %dx%d" % (w, h))
    for _ in range(2):
        hvx.hvx_min_max_count(ctx, im, out.data_ptr())
    torch.cuda.synchronize()
    assert tuple(out.cpu().numpy().view(np.int32)[:4].tolist()) == tuple(G.min_max_count(img))
    counted = _device_us(lambda s: hvx.hvx_min_max_count(ctx, im, out.data_ptr(), s))
    plain = _device_us(lambda s: hvx.hvx_min_max(ctx, im, out.data_ptr(), s))
    log("  min_max_count %.2f us, min_max %.2f us" % (counted, plain))
    assert counted < 2 * plain
