"""The LDS rows that the node phase of the 2D strip kernels reads (csrc/ilh_strip.h), compiled for the CPU:
for every order, strip length, node-group width and wave count they lie within the 64 rows a wave
writes, and within the strip's own elements, and lanes that hold a node read the elements that share it."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_16424_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "ilh_strip.h"
int main() {
  int bad = 0;
  for (int K = 1; K <= 4; ++K) {
    const int Q1D = 2 * K, EPW = 64 / Q1D, NS = K * EPW + 1, GS = NS <= 32 ? 32 : 64;
    for (int W = 1; W <= 2; ++W)
      for (int E = 1; E <= EPW; ++E) {
        if (ilh::strip_last_row(K, Q1D, GS, W, E) >= 64 * (W - 1) + E * Q1D) {
          std::printf("K %d W %d E %d: row %d\n", K, W, E, ilh::strip_last_row(K, Q1D, GS, W, E));
          ++bad;
        }
        for (int tn = 0; tn <= K * E; ++tn) {
          if (tn < K * E && ilh::strip_element(tn, K, E) != tn / K) ++bad;
          if (tn % K == 0 && tn > 0 && ilh::strip_left(tn, K, E) != tn / K - 1) ++bad;
        }
      }
  }
  return bad != 0;
}
"""


def test_rows_stay_in_the_strip(tmp_path):
    (tmp_path / "strip.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(tmp_path / "strip.cpp"), "-o",
                    str(tmp_path / "strip")], check=True)
    r = subprocess.run([str(tmp_path / "strip")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
