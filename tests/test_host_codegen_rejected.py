"""Host-side test: a group whose source the compiler rejects is left to the
interpreter, and the compiler is not asked again for the same program."""
import os
import subprocess
import sys

import pytest

from paper_2008_11476_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# In a process of its own, whose hipRTC is given an option that fails every
# compilation.  A compilation writes the source to the dump folder first.
PROGRAM = """
import os, sys
import paper_2008_11476_amd as hvx
ctx = hvx.hvx_context_create(0)
FAKE = 0x7f0000000000

def verify(w):
    g = hvx.hvx_graph_create(ctx)
    a, o = (hvx.hvx_image_from_ptr(ctx, w, 480, hvx.HVX_DF_U8, FAKE + k * (1 << 28), w) for k in range(2))
    v = hvx.hvx_image_create_virtual(g)
    hvx.hvx_gaussian3x3_node(g, a, v)
    hvx.hvx_box3x3_node(g, v, o)
    hvx.hvx_graph_verify(g)
    names = os.listdir(os.environ["HVX_GEN_DUMP"])
    for n in names:
        os.remove(os.path.join(os.environ["HVX_GEN_DUMP"], n))
    print(hvx.hvx_graph_query(g, hvx.HVX_QUERY_NUM_GENERATED), len(names))

verify(640)
verify(640)
verify(1280)
"""


def test_a_rejected_source_is_compiled_once(tmp_path):
    if not os.path.exists(build.LIB):
        build.build()
    env = dict(os.environ, HVX_GEN_DUMP=str(tmp_path), HIPRTC_COMPILE_OPTIONS_APPEND="-include not_there.h",
               PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", PROGRAM], capture_output=True, text=True, env=env, cwd=ROOT)
    assert r.returncode == 0, r.stderr[-2000:]
    lines = [ln for ln in r.stdout.splitlines() if ln]
    if lines[0].startswith("1 "):
        pytest.skip("this hipRTC takes no options from the environment")
    assert lines == ["0 1", "0 0", "0 0"]
