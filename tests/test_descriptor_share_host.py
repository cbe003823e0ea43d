"""When the waves of a descriptor work-group share a keypoint: the number of keypoints
up to which they do follows what a window is cut into and how many sizes each pixel is
binned for (compiled for the host)."""
import subprocess
from pathlib import Path

ROOT = Path(__file__).resolve().parents[1]

PROG = r"""
#include <cstdio>
#include <cstring>
#include "sift_internal.h"
using namespace sift;
static int fails = 0;
static void check(int n_dsp, float largest, int want) {
  DevParams p;
  std::memset(&p, 0, sizeof p);
  p.desc_magnif = 3.0f;
  p.sigma0 = 1.6f;
  p.n_dsp = n_dsp;
  p.dsp[0] = largest;
  const int got = desc_share_limit(desc_largest_window(p), p.n_dsp);
  if (got != want) { std::printf("FAIL %d sizes up to %g: %d\n", n_dsp, largest, got); ++fails; }
}
int main() {
  check(1, 1.0f, 4);
  check(1, 8.0f, 4);
  check(2, 4.0f / 3, 4);
  check(5, 2.0f, 4);
  check(5, 4.0f / 3, 3);
  check(10, 4.0f / 3, 2);
  check(10, 2.0f, 4);
  check(16, 1.0f, 1);
  check(16, 4.0f, 4);
  return fails;
}
"""


def test_limit_follows_the_settings(tmp_path):
    src = tmp_path / "share.cpp"
    src.write_text(PROG)
    exe = tmp_path / "share"
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", str(ROOT / "paper_2605_17869_amd" / "csrc"),
                    "-I", str(ROOT / "include"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
