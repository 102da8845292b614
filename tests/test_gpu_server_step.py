"""A server step of more images than one launch carries, and waiting for the
server from several threads: every result equals the oracle's."""
import threading

import numpy as np
import pytest

import paper_2008_11476_amd as hvx
from tests.gpu_util import compare, log
from tests.test_gpu_batch_serve import _build, _host_frames

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = hvx.hvx_context_create(0)
    yield c
    hvx.hvx_context_release(c)


@pytest.mark.parametrize("kinds", [("sobel_edge",), ("harris", "uyvy_gauss5", "sobel_edge")])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 33])
def test_steps_of_many_images(ctx, kinds, n):
    """The first request (a pageable 4K frame, milliseconds of copying) holds
    the one stream while the others queue; they then go in one step, sixteen
    images to a launch."""
    import torch
    s = hvx.hvx_server_create(ctx, hvx.HVX_SERVER_CONTINUOUS, 1 << 28, 64, 1)
    held, reqs, graphs = [], {}, []
    big, spec = _host_frames("sobel_edge", 3840, 2160, seed=5)
    g, outs, keep, imgs = _build(ctx, spec)
    graphs.append(g)
    held.append((outs, keep))
    src, dst = torch.from_numpy(np.ascontiguousarray(big)), torch.full((2160, 3840), 7, dtype=torch.uint8)
    plans = []
    for tag in range(n):
        kind = kinds[tag % len(kinds)]
        w, h = (64, 48) if tag % 2 else (322, 101)
        f, sp = _host_frames(kind, w, h, seed=300 + tag)
        gt, outs, keep, imgs = _build(ctx, sp)
        graphs.append(gt)
        held.append((outs, keep))
        buf, view = hvx.alloc_image(h, w, hvx.HVX_DF_UYVY if kind == "uyvy_gauss5" else hvx.HVX_DF_U8)
        view.copy_(torch.from_numpy(np.ascontiguousarray(f)))
        ob, out = hvx.alloc_image(h, w, hvx.HVX_DF_U8)
        out.fill_(7)
        reqs[tag] = (kind, sp, out)
        (iname,), (oname,) = sp.inputs, sp.outputs
        plans.append((gt, [(imgs[iname], view.data_ptr(), view.stride(0)), (imgs[oname], out.data_ptr(), out.stride(0))]))
        held.append((buf, view, ob))
    torch.cuda.synchronize()
    log("steps %s n=%d" % (",".join(kinds), n))
    hvx.hvx_server_submit(s, g, src.data_ptr(), src.stride(0), dst.data_ptr(), dst.stride(0), 1000, ctx=ctx)
    for tag, (gt, bind) in enumerate(plans):
        hvx.hvx_server_submit_bound(s, gt, bind, hvx.HVX_MEMORY_DEVICE, tag, ctx=ctx)
    waits = [threading.Thread(target=hvx.hvx_server_drain, args=(s,)) for _ in range(3)]
    for t in waits:
        t.start()
    hvx.hvx_server_drain(s, ctx=ctx)
    done = hvx.hvx_server_poll(s, 1000, ctx=ctx)
    for t in waits:
        t.join(30)
        assert not t.is_alive()
    assert sorted(t for t, _, _ in done) == list(range(n)) + [1000]
    assert all(st == 0 for _, st, _ in done)
    hvx.hvx_server_drain(s, ctx=ctx)  # nothing in flight: returns at once
    compare(spec, {"out": dst.numpy()}, spec.run_oracle())
    for tag, (kind, sp, out) in reqs.items():
        compare(sp, {next(iter(sp.outputs)): out.cpu().numpy()}, sp.run_oracle(), corner=(kind == "harris"))
    hvx.hvx_release_server(s)
    for gr in graphs:
        hvx.hvx_release_graph(gr)
