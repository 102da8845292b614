"""Sliding box sums of products in streamed kernels, and square roots without
scaling: bit for bit the interpreter's results, for the graphs that take these
forms and their neighbours that must not (another border rule per product, a
factor or product with other readers, a constant border, sums read by a local
operator, roots of numbers on no known grid)."""
import numpy as np
import pytest

import oracle
import paper_2008_11476_amd as hvx
import synth
from tests import graphspec as gs
from tests.gpu_util import log, run_spec

pytestmark = pytest.mark.gpu

F32 = np.float32


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = hvx.hvx_context_create(0)
    yield c
    hvx.hvx_context_release(c)


def _point(ins, out, expr, dtype=F32):
    return gs.N("custom_point", ins, [out], params={"expr": expr, "out_dtype": dtype})


def _products(b0, b1):
    return [gs.N("sobel3x3", ["in"], ["gx", "gy"], *b0),
            gs.N("multiply_f32", ["gx", "gx"], ["pxx"]), gs.N("multiply_f32", ["gx", "gy"], ["pxy"]),
            gs.N("box5x5_f32", ["pxx"], ["sxx"], *b1), gs.N("box5x5_f32", ["pxy"], ["sxy"], *b1)]


def _plain(img, b):
    return gs.Spec(_products(b, b), {"in": img}, {"sxx": F32, "sxy": F32})


def _read_again(img, b):
    """The sums have rows of their own to spare: a local kernel reads them."""
    return gs.Spec(_products(("constant", 200), b) + [
        gs.N("custom_local", ["sxx"], ["l"], *b, params={"expr": "a[-1, 2] / 4 - a[1, -2]", "out_dtype": F32}),
        gs.N("box5x5_f32", ["sxy"], ["m"], *b)], {"in": img}, {"l": F32, "m": F32})


def _two_rules(img, b):
    nodes = _products(b, b)
    nodes[-1] = gs.N("box5x5_f32", ["pxy"], ["sxy"], *(("replicate", 0) if b[0] == "mirror" else ("mirror", 0)))
    return gs.Spec(nodes, {"in": img}, {"sxx": F32, "sxy": F32})


def _other_readers(img, b):
    return gs.Spec(_products(b, b) + [gs.N("magnitude", ["gx", "gy"], ["m"]),
                                      gs.N("box5x5_f32", ["pxx"], ["again"], *b), _point(["again", "sxx"], "d", "a - b")],
                   {"in": img}, {"m": np.int16, "sxy": F32, "d": F32, "pxy": F32})


def _of_values(img, b):
    """Products of S16 values of any size, and of one with a gradient."""
    return gs.Spec([gs.N("gaussian3x3", ["in"], ["g"], *b),
                    gs.N("custom_point", ["in", "g"], ["w"], params={"expr": "(a - b) * 100", "out_dtype": np.int16}),
                    gs.N("sobel3x3", ["g"], ["x", "y"], *b), gs.N("multiply_f32", ["x", "w"], ["q"]),
                    gs.N("multiply_f32", ["w", "w"], ["p"]), gs.N("multiply_f32", ["y", "y"], ["t"]),
                    gs.N("box5x5_f32", ["q"], ["r"], *b), gs.N("box5x5_f32", ["p"], ["s"], *b),
                    gs.N("box5x5_f32", ["t"], ["u"], *b)], {"in": img}, {"r": F32, "s": F32, "u": F32})


def _roots(img, b):
    """Grids that are known (0, -2, -31) and that are not."""
    return gs.Spec(_products(b, b) + [
        _point(["sxx", "sxy"], "r0", "sqrt((a - b) * (a - b) / 4 + b * b)"),
        _point(["sxx", "sxy"], "r1", "sqrt(max(a, abs(b)) * 0.000030517578125 / 65536)"),
        _point(["sxx", "sxy"], "r2", "sqrt(a / 3) - sqrt(abs(b) * 0.1)"),
        _point(["r0", "sxx"], "r3", "sqrt(a) + sqrt(sel(gt(b, 1000), -b, b))"),
        _point(["sxx", "r0"], "r4", "sqrt(a * b / (a + b)) + sqrt(clamp(a, 0, 7) / 1048576 / 1048576)")],
        {"in": img}, {"r%d" % i: F32 for i in range(5)})


def _scaled(img, b):
    """Scalings by powers of two inside sums, exact or not provably so."""
    return gs.Spec(_products(b, b) + [
        _point(["sxx", "sxy"], "r0", "a / 4 - b * 0.125 + sqrt(abs(a) * 0.5 + 1)"),
        _point(["sxx", "sxy"], "r1", "(a - b) * (a - b) / 8 - b / 2 - (b - a * 0.25)"),
        _point(["r1", "sxy"], "r2", "sqrt(a * a / 65536 + b * b) / 2 + a * 4"),
        _point(["sxx", "sxy"], "r3", "sqrt(a * b * a * b) - sqrt(a * a * a * a) / 2"),
        _point(["r2", "r3"], "r4", "a / 1048576 + b / 1048576 / 1048576 / 1048576 / 1048576 - a")],
        {"in": img}, {"r%d" % i: F32 for i in range(5)})


GRAPHS = {"plain": _plain, "read_again": _read_again, "two_rules": _two_rules, "other_readers": _other_readers,
          "of_values": _of_values, "roots": _roots, "scaled": _scaled}
BORDERS = [("replicate", 0), ("mirror", 0), ("constant", 0), ("constant", 3)]
SIZES = [(248, 40), (993, 209), (1, 40), (2, 2), (64, 1031), (500, 67)]


@pytest.mark.parametrize("border", BORDERS, ids=lambda b: "%s%d" % b)
@pytest.mark.parametrize("graph", list(GRAPHS))
def test_equals_interpreter(ctx, graph, border):
    for w, h in SIZES:
        img = synth.corner_image(w, h, seed=w)
        img[h // 3:h // 2] = 0  # flat: sums of zero
        img[h // 2:, ::2] = 255
        img[h // 2:, 1::2] = 0  # the steepest gradients
        spec = GRAPHS[graph](img, border)
        log("slide %s %s %dx%d" % (graph, border, w, h))
        got, g = run_spec(spec, ctx, specialize=False)
        assert hvx.hvx_graph_query(g, hvx.HVX_QUERY_GEN_TILE) & 0xFFFF == 4 or graph == "two_rules", "not streamed"
        ref, _ = run_spec(spec, ctx, specialize=False, codegen=False)
        valid = oracle.valid_masks(spec.oracle_graph(), spec.shapes())
        for out in spec.outputs:
            a, b = got[out], ref[out]
            if a.dtype == F32:
                nan = np.isnan(a) & np.isnan(b)
                a, b = a.view(np.uint32), b.view(np.uint32)
            else:
                nan = np.zeros(a.shape, bool)
            bad = (a != b) & valid[out] & ~nan
            assert not bad.any(), "%s: %d differ, first at (y, x) = %s" % (
                out, bad.sum(), tuple(int(i[0]) for i in np.nonzero(bad)))
