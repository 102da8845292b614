"""GPU: the two square roots that rest on what the hardware's root returns,
compared for every argument (the rounded magnitude of bounded gradients) or
for every float of whole binades (the root of bounded numbers in F32 user
kernels)."""
import glob

import numpy as np
import pytest

import paper_2008_11476_amd as hvx
from tests import graphspec as gs
from tests.gpu_util import log, run_spec

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = hvx.hvx_context_create(0)
    yield c
    hvx.hvx_context_release(c)


def _written(path):
    return "".join(open(f).read() for f in glob.glob(str(path / "hvx_gen_*.hip")))


def test_magnitude_of_every_pair_of_sobel_gradients(ctx, tmp_path, monkeypatch):
    """All (gx, gy) of [-1020, 1020]^2, the range that Sobel3x3 of a U8 image
    has: two user kernels clamp S16 images to it, and the extremes make the
    group a streamed one."""
    monkeypatch.setenv("HVX_GEN_DUMP", str(tmp_path))
    r = np.arange(-1020, 1021, dtype=np.int16)
    gy, gx = np.meshgrid(r, r, indexing="ij")
    clamp = {"expr": "clamp(a, -1020, 1020)", "out_dtype": np.int16}
    spec = gs.Spec([gs.N("custom_point", ["x"], ["cx"], params=clamp), gs.N("custom_point", ["y"], ["cy"], params=clamp),
                    gs.N("magnitude", ["cx", "cy"], ["m"]), gs.N("min_max", ["m"], ["ends"])],
                   {"x": np.ascontiguousarray(gx), "y": np.ascontiguousarray(gy)}, {"m": np.int16}, buffers={"ends": 8})
    log("magnitude of every pair")
    got, g = run_spec(spec, ctx)
    assert hvx.hvx_graph_query(g, hvx.HVX_QUERY_GEN_TILE) & 0xFFFF == 4
    assert "row_magnitude<true>" in _written(tmp_path)
    s = gx.astype(np.int64) ** 2 + gy.astype(np.int64) ** 2
    q = np.floor(np.sqrt(s.astype(np.float64))).astype(np.int64)
    assert ((q * q <= s) & (s < (q + 1) ** 2)).all()
    want = q + (s - q * q > q)
    bad = got["m"] != want
    assert not bad.any(), "%d differ, first for the sum %d" % (bad.sum(), s[bad][0])
    assert got["ends"].view(np.int32).tolist() == [0, 1442]


# 2^k times every whole number below 2^24: all floats of the binades
# [2^(23 + k), 2^(24 + k)), zero, and the numbers of few bits below them
@pytest.mark.parametrize("k", [-96, -95, 0, 1, 97, 98])
def test_root_of_every_float_of_a_binade(ctx, tmp_path, monkeypatch, k):
    monkeypatch.setenv("HVX_GEN_DUMP", str(tmp_path))
    hi, lo = np.meshgrid(np.arange(16384, dtype=np.int16), np.arange(1024, dtype=np.int16), indexing="ij")
    expr = "sqrt(max(a * 1024 + b, 0) * %r)" % (2.0 ** k)
    spec = gs.Spec([gs.N("custom_point", ["h", "l"], ["r"], params={"expr": expr, "out_dtype": np.float32})],
                   {"h": np.ascontiguousarray(hi), "l": np.ascontiguousarray(lo)}, {"r": np.float32})
    log("roots, 2^%d" % k)
    got, _ = run_spec(spec, ctx)
    assert "sqrt_bounded(" in _written(tmp_path)
    x = (hi.astype(np.int64) * 1024 + lo).astype(np.float32) * np.float32(2.0 ** k)
    want = np.sqrt(x)
    bad = got["r"].view(np.uint32) != want.view(np.uint32)
    assert not bad.any(), "%d differ, first the root of %r" % (bad.sum(), x[bad][0])
