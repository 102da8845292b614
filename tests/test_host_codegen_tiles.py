"""Host-side tests of generated kernels in the tile form: reducing groups that
cannot be streamed (a periodic border, two border rules on one value,
NonLinearFilter, the EqualizeHist table) are generated, as the others are.
Verification writes and compiles them; no compute call is made."""
import pytest

import paper_2008_11476_amd as hvx

FAKE = 0x7f0000000000  # 16-byte aligned, never dereferenced here


@pytest.fixture(scope="module")
def lib():
    import os
    if not os.path.exists(hvx.LIB_PATH):
        from paper_2008_11476_amd import build
        build.build()
    return hvx.lib()


@pytest.fixture
def ctx(lib):
    c = hvx.hvx_context_create(0)
    yield c
    hvx.hvx_context_release(c)


def _q(g, attr):
    return hvx.hvx_graph_query(g, attr)


def _repeat(g, a, v):
    """Gaussian3x3 under the periodic border."""
    hvx.hvx_node_set_border(hvx.hvx_gaussian3x3_node(g, a, v[0]), hvx.HVX_BORDER_REPEAT, 0)
    return v[0]


def _two_rules(g, a, v):
    """One image read under two border rules."""
    hvx.hvx_gaussian3x3_node(g, a, v[0])
    hvx.hvx_node_set_border(hvx.hvx_box3x3_node(g, a, v[1]), hvx.HVX_BORDER_MIRROR, 0)
    hvx.hvx_custom_point_node(g, "max(a, b)", [v[0], v[1]], hvx.HVX_DF_U8, v[2])
    return v[2]


def _nonlinear(g, a, v):
    hvx.hvx_nonlinear_filter_node(g, hvx.HVX_NONLINEAR_MEDIAN, a, [[0, 1, 0], [1, 1, 1], [0, 1, 0]], v[0])
    return v[0]


def _table(g, a, v):
    """The EqualizeHist table applied, then a local operator, in one group."""
    hvx.hvx_equalize_hist_node(g, a, v[0])
    hvx.hvx_gaussian3x3_node(g, v[0], v[1])
    return v[1]


PRODUCERS = {"repeat": _repeat, "two_rules": _two_rules, "nonlinear": _nonlinear, "table": _table}
REDUCTIONS = {
    "histogram": lambda g, v, b: hvx.hvx_histogram_node(g, v, 100, 0, 256, b[0]),
    "min_max": lambda g, v, b: hvx.hvx_min_max_node(g, v, b[0]),
    "min_max_count": lambda g, v, b: hvx.hvx_min_max_loc_node(g, v, b[0], None, 0),
    "mean_std_dev": lambda g, v, b: hvx.hvx_mean_std_dev_node(g, v, b[0]),
    "two": lambda g, v, b: (hvx.hvx_mean_std_dev_node(g, v, b[0]), hvx.hvx_histogram_node(g, v, 256, 0, 256, b[1])),
}


@pytest.mark.parametrize("reduction", list(REDUCTIONS))
@pytest.mark.parametrize("producer", list(PRODUCERS))
def test_reductions_that_cannot_stream_are_generated(ctx, producer, reduction):
    g = hvx.hvx_graph_create(ctx)
    a = hvx.hvx_image_from_ptr(ctx, 640, 480, hvx.HVX_DF_U8, FAKE, 640)
    v = [hvx.hvx_image_create_virtual(g) for _ in range(3)]
    bufs = [hvx.hvx_buffer_from_ptr(ctx, FAKE + (1 << 40) + (k << 20), 8192) for k in range(2)]
    REDUCTIONS[reduction](g, PRODUCERS[producer](g, a, v), bufs)
    hvx.hvx_graph_verify(g)
    # the histogram of EqualizeHist is a kernel of its own
    assert _q(g, hvx.HVX_QUERY_NUM_KERNELS) == (2 if producer == "table" else 1)
    assert _q(g, hvx.HVX_QUERY_NUM_GENERATED) == 1
    assert _q(g, hvx.HVX_QUERY_GEN_TILE) & 0xFFFF == 16  # tiles of 16 rows
    hvx.hvx_release_graph(g)
