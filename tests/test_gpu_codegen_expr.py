"""GPU parity of long user kernels in streamed kernels: bit for bit the tile
interpreter's results, and the oracle's."""
import numpy as np
import pytest

import paper_2008_11476_amd as hvx
import synth
from tests import graphspec as gs
from tests.expr_cases import long_expressions
from tests.gpu_util import compare, log, run_spec

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = hvx.hvx_context_create(0)
    yield c
    hvx.hvx_context_release(c)


@pytest.mark.parametrize("terms", [10, 11, 12, 13])
def test_long_user_kernels(ctx, terms):
    for k, expr in enumerate(long_expressions(terms)):
        spec = gs.Spec([gs.N("gaussian3x3", ["in"], ["v"], "mirror"),
                        gs.N("custom_local", ["v"], ["out"], "mirror", params={"expr": expr, "out_dtype": np.uint8})],
                       {"in": synth.edge_image(1003, 211, seed=terms + k)}, {"out": np.uint8})
        log("long user kernel %d.%d" % (terms, k))
        got, g = run_spec(spec, ctx)
        assert hvx.hvx_graph_query(g, hvx.HVX_QUERY_NUM_GENERATED) == 1
        ref, _ = run_spec(spec, ctx, codegen=False)
        assert np.array_equal(got["out"], ref["out"]), expr
        compare(spec, got, spec.run_oracle())
