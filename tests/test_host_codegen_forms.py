"""Host-side test: the source of a group that can take both forms of generated
kernels holds each under its own macro, so that a kernel of one form (a tile
that the plan tuner tries, say) is compiled without the other."""
import glob
import os
import subprocess

import pytest

import paper_2008_11476_amd as hvx
from paper_2008_11476_amd import build

FAKE = 0x7f0000000000  # 16-byte aligned, never dereferenced here


@pytest.mark.parametrize("macro,form,other", [("HVX_GEN_TILES", "void hvx_gen(", "void hvx_gen_stream("),
                                              ("HVX_GEN_STREAM_ONLY", "void hvx_gen_stream(", "void hvx_gen(")])
def test_a_kernel_is_compiled_without_the_other_form(tmp_path, monkeypatch, macro, form, other):
    if not os.path.exists(hvx.LIB_PATH):
        build.build()
    monkeypatch.setenv("HVX_GEN_DUMP", str(tmp_path))
    ctx = hvx.hvx_context_create(0)
    g = hvx.hvx_graph_create(ctx)
    a, o = (hvx.hvx_image_from_ptr(ctx, 640, 480, hvx.HVX_DF_U8, FAKE + k * (1 << 28), 640) for k in range(2))
    v = hvx.hvx_image_create_virtual(g)
    hvx.hvx_erode3x3_node(g, a, v)
    # a source that no other test writes
    hvx.hvx_custom_point_node(g, "a - b * %d / 11" % len(macro), [a, v], hvx.HVX_DF_U8, o)
    hvx.hvx_graph_verify(g)
    src, = glob.glob(str(tmp_path / "hvx_gen_*.hip"))
    text = open(src).read().replace("namespace __hip_internal {}\nusing namespace __hip_internal;\n", "")
    main = tmp_path / "main.hip"
    main.write_text("\n".join(ln for ln in text.split("\n") if not ln.startswith("#include")))
    r = subprocess.run([build._hipcc(), "-E", "-P", "-x", "c++", "-D" + macro, str(main)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    assert form in r.stdout and other not in r.stdout
    hvx.hvx_context_release(ctx)
