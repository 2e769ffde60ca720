"""Addresses of the segment kernel's stem in LDS, on the host: the header's own
functions compiled into a small program that walks every image of a group and
every element a window row can start at."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include "gevo_cnn_fused.h"
using namespace gevo;
int main() {
  long seen = 0;
  for (int H = 3; H <= 33; ++H)
    for (int W = 3; W <= 32; ++W)
      for (int C = 1; C <= 4; ++C) {
        const int pitch = seg_pitch(H, W, C), real = (H + 2) * (W + 2) * C, im = 4096, im2 = im + 16 * pitch + 64;
        if (pitch < real || pitch > real + 1) return printf("pitch %dx%dx%d\n", H, W, C), 1;
        for (int img = 0; img < 8; ++img)
          for (int y = 0; y < H + 2; ++y)
            for (int x = 0; x < W; ++x) {
              const int e = (y * (W + 2) + x) * C, at = 2 * img * pitch + seg_window(im, im2, e);
              // a dword, and the place where the element was stored
              const int i = img * pitch + e, stored = (e & 1) ? im2 + 2 * (i + 1) : im + 2 * i;
              if (at % 4 || at != stored) return printf("%dx%dx%d image %d element %d at %d\n", H, W, C, img, e, at), 1;
              ++seen;
            }
      }
  return printf("%ld\n", seen), 0;
}
"""


def test_every_window_row_of_the_stem_starts_on_a_dword(tmp_path):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no g++")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "paper_2310_10211_amd", "csrc"), "-o", str(exe), str(src)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0 and int(res.stdout) > 10 ** 6, res.stdout
