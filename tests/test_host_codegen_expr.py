"""Host-side test: user kernels of every length up to the longest are
generated.  The expression written for two 16-bit pixels at a time names a
window pixel in 14 characters and repeats the argument of abs(), so the longest
ones pass several hundred characters."""
import os

import pytest

import paper_2008_11476_amd as hvx
from tests.expr_cases import long_expressions

FAKE = 0x7f0000000000  # 16-byte aligned, never dereferenced here


@pytest.fixture(scope="module")
def ctx():
    if not os.path.exists(hvx.LIB_PATH):
        from paper_2008_11476_amd import build
        build.build()
    c = hvx.hvx_context_create(0)
    yield c
    hvx.hvx_context_release(c)


@pytest.mark.parametrize("terms", range(8, 14))
def test_long_user_kernels_are_generated(ctx, terms):
    for expr in long_expressions(terms):
        g = hvx.hvx_graph_create(ctx)
        a, o = (hvx.hvx_image_from_ptr(ctx, 640, 480, hvx.HVX_DF_U8, FAKE + k * (1 << 28), 640) for k in range(2))
        v = hvx.hvx_image_create_virtual(g)
        hvx.hvx_gaussian3x3_node(g, a, v)
        hvx.hvx_custom_local_node(g, expr, v, hvx.HVX_DF_U8, o)
        hvx.hvx_graph_verify(g)
        assert hvx.hvx_graph_query(g, hvx.HVX_QUERY_NUM_GENERATED) == 1, expr
        hvx.hvx_release_graph(g)


def _assembly(ctx, tmp_path, monkeypatch, expr):
    """The source and the assembly of an F32 point kernel of one U8 image."""
    import glob
    import subprocess
    from paper_2008_11476_amd import build
    monkeypatch.setenv("HVX_GEN_DUMP", str(tmp_path))
    g = hvx.hvx_graph_create(ctx)
    a = hvx.hvx_image_from_ptr(ctx, 640, 480, hvx.HVX_DF_U8, FAKE, 640)
    o = hvx.hvx_image_from_ptr(ctx, 640, 480, hvx.HVX_DF_F32, FAKE + (1 << 28), 2560)
    hvx.hvx_custom_point_node(g, expr, [a], hvx.HVX_DF_F32, o)
    hvx.hvx_graph_verify(g)
    src, = glob.glob(str(tmp_path / "hvx_gen_*.hip"))
    text = open(src).read()
    (tmp_path / "k.hip").write_text(text.replace("namespace __hip_internal {}\nusing namespace __hip_internal;\n", ""))
    csrc = os.path.join(os.path.dirname(build.__file__), "csrc")
    r = subprocess.run([build._hipcc(), "-x", "hip", "-O3", "-std=c++17", "--offload-arch=gfx950", "--cuda-device-only",
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-w", "-S", "-I", csrc,
                        str(tmp_path / "k.hip"), "-o", "-"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return text, r.stdout


@pytest.mark.parametrize("expr,roots", [("a * sqrt(2) + sqrt(abs(-7) * 3)", 2), ("sel(gt(0, sqrt(a * 3)), a * 5, a - 1)", 1)],
                         ids=["literal", "comparison"])
def test_roots_that_the_compiler_can_spare(ctx, tmp_path, monkeypatch, expr, roots):
    """Roots of bounded numbers are formed from the hardware's reciprocal root;
    that of a literal is a constant all the same, and one that is only compared
    with what it cannot be under is not formed."""
    text, asm = _assembly(ctx, tmp_path, monkeypatch, expr)
    assert text.count("sqrt_bounded(") == roots
    assert "v_rsq" not in asm and "v_sqrt" not in asm
