"""GPU parity of global operators reduced by generated tile kernels: groups
that cannot be streamed, against the oracle; and the tiles that the plan tuner
tries for a group that can, whose results must equal the streamed kernel's."""
import numpy as np
import pytest

import paper_2008_11476_amd as hvx
import synth
from tests import graphspec as gs
from tests.gpu_util import log, run_spec
from tests.test_gpu_global_graph import _check_buffers

pytestmark = pytest.mark.gpu

N = gs.N


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = hvx.hvx_context_create(0)
    yield c
    hvx.hvx_context_release(c)


CROSS = [[0, 1, 0], [1, 1, 1], [0, 1, 0]]
PRODUCERS = {
    "repeat": [N("gaussian3x3", ["in"], ["v"], "repeat")],
    "two_rules": [N("gaussian3x3", ["in"], ["p"], "replicate"), N("box3x3", ["in"], ["q"], "mirror"),
                  N("custom_point", ["p", "q"], ["v"], params={"expr": "max(a, b)", "out_dtype": np.uint8})],
    "nonlinear": [N("nonlinear", ["in"], ["v"], params={"func": "median", "mask": CROSS})],
    "table": [N("equalize_hist", ["in"], ["e"]), N("gaussian3x3", ["e"], ["v"])],
}
REDUCTIONS = {
    "sums+hist": [N("mean_std_dev", ["v"], ["r0"]), N("histogram", ["v"], ["r1"], params={"bins": 256})],
    "hist10+counts": [N("histogram", ["v"], ["r0"], params={"bins": 10, "offset": 5, "range": 201}),
                      N("min_max_loc", ["v"], ["r1"])],
    "extremes": [N("min_max", ["v"], ["r0"]), N("mean_std_dev", ["v"], ["r1"])],
}


@pytest.mark.parametrize("reduction", list(REDUCTIONS))
@pytest.mark.parametrize("producer", list(PRODUCERS))
def test_tile_reductions(ctx, producer, reduction):
    for w, h in ((1, 1), (5, 3), (129, 17), (641, 363), (2003, 1501)):
        spec = gs.Spec(PRODUCERS[producer] + REDUCTIONS[reduction], {"in": synth.edge_image(w, h, seed=w)}, {},
                       buffers={"r0": 8192, "r1": 8192})
        log("tile reductions %s %s %dx%d" % (producer, reduction, w, h))
        got, g = run_spec(spec, ctx)
        assert hvx.hvx_graph_query(g, hvx.HVX_QUERY_NUM_GENERATED) == 1
        assert hvx.hvx_graph_query(g, hvx.HVX_QUERY_GEN_TILE) & 0xFFFF == 16
        _check_buffers(spec, got, spec.run_oracle())


def test_tuned_tiles_of_a_reducing_group(ctx):
    spec = gs.Spec([N("gaussian3x3", ["in"], ["v"], "mirror")] + REDUCTIONS["sums+hist"],
                   {"in": synth.edge_image(641, 363, seed=2)}, {}, buffers={"r0": 8192, "r1": 8192})
    log("tuned tiles")
    got, _ = run_spec(spec, ctx, autotune=True)
    _check_buffers(spec, got, spec.run_oracle())
