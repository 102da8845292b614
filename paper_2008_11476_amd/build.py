"""Build libhvx.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree.

Usage: python -m paper_2008_11476_amd.build   (or call build()).
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT_DIR = os.path.join(os.path.dirname(HERE), "_build")
LIB = os.path.join(HERE, "libhvx.so")

SOURCES = ["api.cpp", "verify.cpp", "runtime.cpp", "server.cpp", "expr.cpp", "codegen.cpp", "codegen_stream.cpp", "kernels.hip", "global.hip"]
# device headers compiled again, with the generated kernels, by hipRTC at run time
RTC_HEADERS = ["hvx_desc.h", "gen_abi.h", "dev_phase.hpp", "dev_reduce.hpp", "dev_generic.hpp", "dev_stream.hpp"]

ARCH = os.environ.get("HVX_OFFLOAD_ARCH", "gfx950")
COMMON = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=" + ARCH,
    # no packed FP32 instructions anywhere (hipcc flag; the host pass warns)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unused-variable", "-Wno-unused-result",
    "-DHVX_ARCH=\"" + ARCH + "\"",
]


def _hipcc():
    for c in (os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc"), "hipcc"):
        if os.path.sep not in c or os.path.exists(c):
            return c
    return "hipcc"


def _embed_headers() -> str:
    """Write a source file holding the text of RTC_HEADERS as string constants."""
    delim = "hvx_rtc"
    out = ["// generated by build.py: device headers for run-time compilation", "namespace hvx {",
           "extern const int kRtcHeaderCount = %d;" % len(RTC_HEADERS),
           "extern const char* const kRtcHeaderNames[] = {%s};" % ", ".join('"%s"' % h for h in RTC_HEADERS),
           "extern const char* const kRtcHeaderTexts[] = {"]
    for h in RTC_HEADERS:
        with open(os.path.join(CSRC, h)) as f:
            text = f.read()
        if ")" + delim + '"' in text:
            raise RuntimeError("%s holds the raw-string delimiter" % h)
        out.append('R"%s(%s)%s",' % (delim, text, delim))
    out += ["};", "}  // namespace hvx", ""]
    path = os.path.join(OUT_DIR, "rtc_headers.cpp")
    with open(path, "w") as f:
        f.write("\n".join(out))
    return path


def _compile(src: str) -> str:
    obj = os.path.join(OUT_DIR, os.path.basename(src) + ".o")
    path = src if os.path.isabs(src) else os.path.join(CSRC, src)
    cmd = [_hipcc(), "-x", "hip", *COMMON, "-c", path, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (src, " ".join(cmd), r.stderr[-6000:]))
    return obj


def build(verbose: bool = False) -> str:
    """Compile every source and link libhvx.so.  Always rebuilds."""
    os.makedirs(OUT_DIR, exist_ok=True)
    sources = SOURCES + [_embed_headers()]
    with cf.ThreadPoolExecutor(max_workers=min(8, len(sources))) as ex:
        objs = list(ex.map(_compile, sources))
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [_hipcc(), "-shared", "-fPIC", "--offload-arch=" + ARCH, "-o", tmp, *objs, "-lhiprtc", "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s\n%s" % (" ".join(cmd), r.stderr[-4000:]))
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
