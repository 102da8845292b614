"""GPU parity of streamed kernels on images hardly taller than the rows their
operators reach: single frames at and around the heights where the rows
before the tail band fit one band, and such images in one launch with large
ones, whose bands are tall; and on images narrower than a lane, which go row
by row in bands.  Bit for bit the tile interpreter's results."""
import numpy as np
import pytest

import oracle
import paper_2008_11476_amd as hvx
import synth
from tests import graphspec as gs
from tests.gpu_util import compare, log, run_spec
from tests.test_gpu_codegen import _fchain, _tomasi
from tests.test_gpu_custom import unsharp_spec
from tests.test_gpu_global_graph import _check_buffers
from tests.test_gpu_slide import _read_again
from tests.test_gpu_stream import _response, _thin, _two_inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = hvx.hvx_context_create(0)
    yield c
    hvx.hvx_context_release(c)


def _chain(img, ops, border):
    names = ["in"] + ["v%d" % i for i in range(1, len(ops))] + ["out"]
    return gs.Spec([gs.N(op, [names[i]], [names[i + 1]], *border) for i, op in enumerate(ops)], {"in": img},
                   {"out": np.uint8})


# operators that reach 6, 8 and 8 rows in all
CHAINS = {"three5": ["gaussian5x5"] * 3, "four5": ["gaussian5x5"] * 4,
          "eight3": ["gaussian3x3", "median3x3", "box3x3", "dilate3x3", "gaussian3x3", "erode3x3", "box3x3", "median3x3"]}


def _streamed(g):
    return hvx.hvx_graph_query(g, hvx.HVX_QUERY_GEN_TILE) & 0xFFFF == 4


@pytest.mark.parametrize("border", [("replicate", 0), ("mirror", 0), ("constant", 77)], ids=lambda b: b[0])
@pytest.mark.parametrize("chain", list(CHAINS))
def test_short_frames(ctx, chain, border):
    for h in range(14, 25):
        for w in (65, 640, 1003):
            spec = _chain(synth.edge_image(w, h, seed=h), CHAINS[chain], border)
            log("short %s %s %dx%d" % (chain, border[0], w, h))
            got, g = run_spec(spec, ctx, specialize=False)
            assert _streamed(g)
            ref, _ = run_spec(spec, ctx, specialize=False, codegen=False)
            assert np.array_equal(got["out"], ref["out"]), "differs from the interpreter at %dx%d" % (w, h)
            compare(spec, got, spec.run_oracle())


@pytest.mark.parametrize("h", [16, 17, 18, 19, 20])
def test_short_frames_reduced(ctx, h):
    """Every pixel counted once."""
    ops = [gs.N("gaussian5x5", ["in"], ["a"], "mirror"), gs.N("gaussian5x5", ["a"], ["b"], "mirror"),
           gs.N("gaussian5x5", ["b"], ["c"], "mirror"), gs.N("histogram", ["c"], ["bins"], params={"bins": 256}),
           gs.N("mean_std_dev", ["c"], ["sums"])]
    spec = gs.Spec(ops, {"in": synth.edge_image(1201, h, seed=h)}, {}, buffers={"bins": 1024, "sums": 64})
    log("short reduced 1201x%d" % h)
    got, g = run_spec(spec, ctx)
    assert _streamed(g)
    _check_buffers(spec, got, spec.run_oracle())


GRAPHS = {"unsharp": unsharp_spec, "tomasi": _tomasi, "fchain": lambda img: _fchain(img, ("mirror", 0))}


@pytest.mark.parametrize("big,frames", [((3840, 2160), 2), ((7936, 3000), 10)], ids=["two4k", "ten8k"])
@pytest.mark.parametrize("graph", list(GRAPHS))
def test_short_images_beside_large_ones(ctx, graph, big, frames):
    """Heights 5 to 37 in one launch whose bands are chosen for the large
    frames (8 to 16 rows, and the most a band takes)."""
    import torch
    make = GRAPHS[graph]
    graphs, small, held = [], [], []
    frame = synth.uniform_u8(big[0], big[1], seed=1)
    for i in range(frames):
        held.append({})
        _, g = run_spec(make(frame), ctx, specialize=False, keep=held[-1])
        assert _streamed(g)
        graphs.append(g)
    for h in range(5, 38):
        w = 60 + 17 * (h % 5) + (500 if h % 3 == 0 else 0)
        spec = make(synth.edge_image(w, h, seed=h))
        keep = {}
        ref, _ = run_spec(spec, ctx, specialize=False, codegen=False)
        _, g = run_spec(spec, ctx, specialize=False, keep=keep)
        for (t, _, _) in keep["outputs"].values():
            t.zero_()
        graphs.append(g)
        small.append((w, h, keep, ref))
    b = hvx.hvx_batch_create(ctx, graphs)
    log("short beside large %s %dx%dx%d" % (graph, big[0], big[1], frames))
    assert hvx.hvx_batch_query(b, hvx.HVX_QUERY_NUM_KERNELS) == 1
    hvx.hvx_batch_schedule(b, torch.cuda.current_stream().cuda_stream, ctx=ctx)
    torch.cuda.synchronize()
    for w, h, keep, ref in small:
        for name, (t, ww, dt) in keep["outputs"].items():
            assert np.array_equal(t.cpu().numpy().view(dt)[:, :ww], ref[name]), "%s differs at %dx%d" % (name, w, h)
    hvx.hvx_release_batch(b)
    for g in graphs:
        hvx.hvx_release_graph(g)


ROW_BY_ROW = {"thin": _thin, "response": _response, "two_inputs": _two_inputs, "fchain": _fchain, "read_again": _read_again,
              "four5": lambda img, border: _chain(img, CHAINS["four5"], border)}


@pytest.mark.parametrize("border", [("replicate", 0), ("mirror", 0), ("constant", 77), ("undefined", 0)], ids=lambda b: b[0])
@pytest.mark.parametrize("graph", list(ROW_BY_ROW))
def test_bands_of_single_rows(ctx, graph, border):
    """Narrow images of several bands, and low ones of one to three."""
    sizes = [(1, 75), (2, 501), (3, 38), (5, 130), (7, 1026)] + [(w, h) for h in range(1, 14) for w in (8, 1003)]
    for w, h in sizes:
        spec = ROW_BY_ROW[graph](synth.edge_image(w, h, seed=w + h), border)
        log("row by row %s %s %dx%d" % (graph, border[0], w, h))
        got, g = run_spec(spec, ctx, specialize=False)
        assert _streamed(g)
        ref, _ = run_spec(spec, ctx, specialize=False, codegen=False)
        valid = oracle.valid_masks(spec.oracle_graph(), spec.shapes())
        for out in spec.outputs:
            a, b = got[out], ref[out]
            if a.dtype == np.float32:
                a, b = a.view(np.uint32), b.view(np.uint32)
            bad = (a != b) & valid[out]
            assert not bad.any(), "%s differs at %dx%d, first at (y, x) = %s" % (
                out, w, h, tuple(int(i[0]) for i in np.nonzero(bad)))


@pytest.mark.parametrize("w,h", [(1, 65536), (2, 40000), (3, 65535), (7, 9435), (7, 20000), (8, 20000)])
def test_sums_of_bright_narrow_images(ctx, w, h):
    """Sums of squares past 32 bits in one column of lanes: 65025 a pixel."""
    spec = gs.Spec([gs.N("gaussian3x3", ["in"], ["g"]), gs.N("mean_std_dev", ["g"], ["sums"]),
                    gs.N("histogram", ["g"], ["bins"], params={"bins": 256})],
                   {"in": np.full((h, w), 255, np.uint8)}, {}, buffers={"sums": 64, "bins": 1024})
    log("bright %dx%d" % (w, h))
    got, g = run_spec(spec, ctx)
    assert _streamed(g)
    s1, s2 = got["sums"].view(np.uint64)[:2].tolist()
    assert (s1, s2) == (255 * w * h, 65025 * w * h)
    mean, std = got["sums"].view(np.float32)[4:6].tolist()
    assert (mean, std) == (255.0, 0.0)
    assert got["bins"].view(np.uint32)[:256].tolist() == [0] * 255 + [w * h]
