"""Host-side test of how a streamed kernel divides an image's rows (gen_abi.h,
the code that the kernels and the host both run): every band holds whole loop
iterations, only the first reads rows above the image and only the last below
it, and the bands count every row once; images that cannot be divided so go
row by row, in bands of no more rows than asked for."""
import os
import shutil
import subprocess

import pytest

from paper_2008_11476_amd import build

SOURCE = r"""
#define __host__
#define __device__
#include "gen_abi.h"
#include <cstdio>
#include <vector>
using namespace hvx;
int main() {
  int bad = 0, several = 0;
  auto fail = [&](int h, int ext, int rows, int band, const char* what) {
    if (++bad <= 20) printf("h %d ext %d rows %d band %d: %s\n", h, ext, rows, band, what);
  };
  for (int ext = 0; ext <= 8; ++ext)
    for (int h = 1; h <= 140; ++h) {
      const int tail = stream_tail(ext);
      if (tail < ext || tail > ext + 3 || tail % kStreamUnroll) fail(h, ext, 0, 0, "tail");
      for (int rows = 1; rows <= 64; ++rows) {
        for (int w : {1, 7}) {  // narrow images: row by row, in bands all the same
          const StreamBands b = stream_bands(w, h, rows, ext);
          if (b.whole || b.n != (h + rows - 1) / rows) fail(h, ext, rows, b.n, "a narrow image");
        }
        const StreamBands b = stream_bands(8, h, rows, ext);
        if (b.n < 1) fail(h, ext, rows, 0, "no band");
        if (!b.whole) {
          for (int k = 0, y = 0; k < b.n; ++k) {
            const StreamBand q = stream_band(b, k);
            if (q.last || q.y0 != y || q.y1 <= y || q.y1 > y + rows || q.own != q.y1 || (k + 1 == b.n) != (q.y1 == h))
              fail(h, ext, rows, k, "a band of single rows");
            y = q.y1;
          }
          continue;
        }
        ++several;
        std::vector<int> counted(h, 0);
        for (int k = 0; k < b.n; ++k) {
          const StreamBand q = stream_band(b, k);
          if (q.last != (tail > 0 && k + 1 == b.n)) fail(h, ext, rows, k, "last");
          if (q.y0 < 0 || q.y1 < q.y0 || (q.y1 == q.y0) != q.last) fail(h, ext, rows, k, "empty");
          if ((q.y1 - q.y0) % kStreamUnroll) fail(h, ext, rows, k, "not whole iterations");
          if (k > 0 && q.y0 < ext) fail(h, ext, rows, k, "reads rows above the image");
          if (q.last ? q.y0 + tail != h : q.y1 + ext > h) fail(h, ext, rows, k, "reads rows below the image");
          const int end = q.last ? h : q.own;
          if (end < q.y0 || end > (q.last ? h : q.y1)) fail(h, ext, rows, k, "counts rows it does not compute");
          for (int y = q.y0; y < end && y < h; ++y) ++counted[y];
        }
        for (int y = 0; y < h; ++y)
          if (counted[y] != 1) {
            fail(h, ext, rows, counted[y], "a row not counted once");
            break;
          }
      }
    }
  printf("%d divided, %d bad\n", several, bad);
  return bad || several < 5000;
}
"""


def test_bands_hold_whole_iterations_inside_the_image(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "bands.cpp", tmp_path / "bands"
    src.write_text(SOURCE)
    csrc = os.path.join(os.path.dirname(build.__file__), "csrc")
    r = subprocess.run([cxx, "-std=c++17", "-O1", "-I", csrc, str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout[-3000:]
