"""GPU parity of the streamed form of generated kernels: each graph runs
streamed and in the tile interpreter, compared bit for bit, and
against the oracle.  Widths lie at and around whole strips of 496 and 248
columns, heights at and around whole bands; images smaller than a lane or a
window are among them."""
import numpy as np
import pytest

import oracle
import paper_2008_11476_amd as hvx
import synth
from tests import graphspec as gs
from tests.gpu_util import compare, log, run_spec
from tests.test_gpu_codegen import (BORDERS, SEPARABLE3, _edge_phase, _fchain, _laplace_float, _morph, _s16_local,
                                    _separable, _tomasi, _uyvy)
from tests.test_gpu_custom import unsharp_spec

pytestmark = pytest.mark.gpu

SIZES = [(992, 212), (993, 209), (1487, 103), (2046, 97), (1241, 311), (64, 1570), (3131, 32), (1, 40), (2, 2), (500, 67), (3, 1), (9, 3)]


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = hvx.hvx_context_create(0)
    yield c
    hvx.hvx_context_release(c)


def _thin(img, border):
    return gs.Spec([gs.N("median3x3", ["in"], ["m"], *border), gs.N("sobel3x3", ["m"], ["gx", "gy"], *border),
                    gs.N("magnitude", ["gx", "gy"], ["mag"]),
                    gs.N("nonmax", ["mag"], ["out"], *border, params={"win": 3})], {"in": img}, {"out": np.int16})


def _response(img, border):
    spec = gs.corner_spec(img, b0=border, b1=border)
    return gs.Spec(spec.nodes[:-1], {"in": img}, {"r": np.float32, "sxy": np.float32})


def _two_inputs(a, border):
    """A second input read by a point operator only, an S16 input read by a
    local one, saturating and wrapping sums, selections and divisions."""
    b = synth.uniform_s16(a.shape[1], a.shape[0], seed=3)
    b.flat[::5] = 32767
    b.flat[1::7] = -32768
    return gs.Spec([gs.N("custom_local", ["b"], ["l"], *border,
                         params={"expr": "max(a[-2, 1], a[1, -1]) / 4 - a[0, 2] / 8", "out_dtype": np.int16}),
                    gs.N("gaussian3x3", ["a"], ["g"], *border),
                    gs.N("custom_point", ["l", "g", "a"], ["p"],
                         params={"expr": "sel(gt(a, b), clamp(b - c, -20, 90) * 3, abs(a / 16) - c)",
                                 "out_dtype": np.int16}),
                    gs.N("add", ["p", "b"], ["s"], params={"policy": "saturate", "out_dtype": "s16"}),
                    gs.N("add", ["s", "g"], ["w"], params={"policy": "wrap", "out_dtype": "s16"}),
                    gs.N("threshold", ["w"], ["out"], params={"thresh": -7.5, "true_v": 3, "false_v": 250}),
                    gs.N("box3x3", ["g"], ["x"], *border)],
                   {"a": a, "b": b}, {"l": np.int16, "w": np.int16, "out": np.uint8, "x": np.uint8})


def _cases():
    out = []
    n = 0

    def add(name, make, border=None, uyvy=False):
        nonlocal n
        for k in range(3):
            w, h = SIZES[(n + 4 * k) % len(SIZES)]
            out.append(("%s-%s-%dx%d" % (name, "-".join(map(str, border or ("", ))), w, h), make, border, w, h))
        n += 1

    add("unsharp", lambda w, h, b: unsharp_spec(synth.edge_image(w, h, seed=1)))
    add("tomasi", lambda w, h, b: _tomasi(synth.corner_image(w, h, seed=w)))
    for b in BORDERS:
        add("fchain", lambda w, h, b: _fchain(synth.edge_image(w, h, seed=2), b), b)
        add("separable3", lambda w, h, b: _separable(synth.edge_image(w, h, seed=3), b, SEPARABLE3), b)
        add("morph", lambda w, h, b: _morph(synth.edge_image(w, h, seed=4), b), b)
        add("laplace_float", lambda w, h, b: _laplace_float(synth.edge_image(w, h, seed=5), b), b)
        add("s16_local", lambda w, h, b: _s16_local(synth.edge_image(w, h, seed=6), b), b)
        add("edge_phase", lambda w, h, b: _edge_phase(synth.edge_image(w, h, seed=7), b, b), b)
        add("thin", lambda w, h, b: _thin(synth.edge_image(w, h, seed=8), b), b)
        add("response", lambda w, h, b: _response(synth.corner_image(w, h, seed=9), b), b)
        add("two_inputs", lambda w, h, b: _two_inputs(synth.edge_image(w, h, seed=10), b), b)
        add("uyvy", lambda w, h, b: _uyvy(synth.uyvy_image((w + 1) // 2 * 2, h, seed=11), b), b)
    return out


CASES = _cases()


@pytest.mark.parametrize("case", range(len(CASES)), ids=[c[0] for c in CASES])
def test_streamed_equals_interpreter_and_oracle(ctx, case):
    name, make, border, w, h = CASES[case]
    spec = make(w, h, border)
    log("stream %s" % name)
    got, g = run_spec(spec, ctx, specialize=False)
    tile = hvx.hvx_graph_query(g, hvx.HVX_QUERY_GEN_TILE)
    assert tile & 0xFFFF == 4 and (tile >> 16) % 4 == 0, "not streamed: tile %dx%d" % (tile >> 16, tile & 0xFFFF)
    ref, _ = run_spec(spec, ctx, specialize=False, codegen=False)
    valid = oracle.valid_masks(spec.oracle_graph(), spec.shapes())
    for out in spec.outputs:
        m = valid[out]
        a, b = got[out], ref[out]
        if a.dtype == np.float32:
            a, b = a.view(np.uint32), b.view(np.uint32)
        bad = (a != b) & m
        assert not bad.any(), "%s: %d pixels differ from the interpreter, first at (y, x) = %s" % (
            out, bad.sum(), tuple(int(i[0]) for i in np.nonzero(bad)))
    whole = {o: d for o, d in spec.outputs.items() if np.dtype(d) != np.float32}
    if name.startswith("laplace_float"):  # the threshold of an F32 value
        whole.pop("out")
    if name.startswith("tomasi"):
        whole = {}
    if whole:
        compare(gs.Spec(spec.nodes, spec.inputs, whole, uyvy=spec.uyvy), got, spec.run_oracle(), phase_names=("ph",))


def test_streamed_batch_of_tall_bands(ctx):
    """A batch of images of several sizes in one launch (bands of many rows,
    the last of an image ragged): the same pixels as each image alone."""
    import torch
    rng = np.random.default_rng(5)
    sizes = [(1990 + 7 * i, 1001 + 3 * i) for i in range(24)]
    graphs, outs, alone = [], [], []
    for w, h in sizes:
        keep = {}
        img = rng.integers(0, 256, (h, w), dtype=np.uint8)
        got, g = run_spec(_fchain(img, ("mirror", 0)), ctx, specialize=False, keep=keep)
        graphs.append(g)
        outs.append(keep)
        alone.append(got)
    for keep in outs:
        for (t, w, dt) in keep["outputs"].values():
            t.zero_()
    b = hvx.hvx_batch_create(ctx, graphs)
    log("stream batch")
    assert hvx.hvx_batch_query(b, hvx.HVX_QUERY_NUM_KERNELS) == 1
    hvx.hvx_batch_schedule(b, torch.cuda.current_stream().cuda_stream, ctx=ctx)
    torch.cuda.synchronize()
    for keep, got in zip(outs, alone):
        for name, (t, w, dt) in keep["outputs"].items():
            assert np.array_equal(t.cpu().numpy().view(dt)[:, :w], got[name]), name
    hvx.hvx_release_batch(b)


# pairs of global operators fused into streamed producers: U8 and S16 inputs
# of the reduction, bins that do and do not divide their interval
REDUCTIONS = {
    "hist+sums": ([("histogram", "g", {"bins": 256}), ("mean_std_dev", "g", {})], {"bins": 1024, "r1": 64}),
    "hist10+counts": ([("histogram", "g", {"bins": 10, "offset": 5, "range": 201}), ("min_max_loc", "g", {})],
                      {"bins": 1024, "r1": 4128}),
    "s16": ([("min_max", "gx", {}), ("min_max_loc", "gy", {})], {"bins": 8, "r1": 4128}),
    "point": ([("histogram", "t", {"bins": 3, "range": 256}), ("mean_std_dev", "t", {})], {"bins": 1024, "r1": 64}),
}


@pytest.mark.parametrize("which", list(REDUCTIONS))
@pytest.mark.parametrize("w,h,border", [(3001, 2003, "replicate"), (497, 61, "mirror"), (3, 2, "constant"),
                                        (1, 1, "replicate"), (64, 3000, "undefined")])
def test_streamed_reductions(ctx, which, w, h, border):
    """One to many items per wave, ragged last columns and bands; a second run
    over the same buffers starts afresh."""
    import torch
    from tests.test_gpu_global_graph import _check_buffers
    ops, bufs = REDUCTIONS[which]
    b = ("replicate", 0) if border == "undefined" else (border, 9)
    nodes = [gs.N("gaussian3x3", ["in"], ["g"], *b), gs.N("sobel3x3", ["g"], ["gx", "gy"], *b),
             gs.N("threshold", ["in"], ["t"], params={"thresh": 99.0, "true_v": 200, "false_v": 90})]
    used = {src for (_, src, _) in ops}
    nodes = [n for n in nodes if used & set(n.outs) or (n.outs == ["g"] and "gx" in used)]
    nodes += [gs.N(op, [src], [buf], params=dict(p)) for (op, src, p), buf in zip(ops, bufs)]
    spec = gs.Spec(nodes, {"in": synth.edge_image(w, h, seed=w)}, {}, buffers=bufs)
    log("stream reductions %s %dx%d" % (which, w, h))
    keep = {}
    got, g = run_spec(spec, ctx, keep=keep)
    assert hvx.hvx_graph_query(g, hvx.HVX_QUERY_NUM_KERNELS) == 1
    env = spec.run_oracle()
    _check_buffers(spec, got, env)
    hvx.hvx_graph_process(g, ctx=ctx)
    torch.cuda.synchronize()
    _check_buffers(spec, {n: t.cpu().numpy() for n, t in keep["buffers"].items()}, env)
