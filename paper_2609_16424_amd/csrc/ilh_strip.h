// Index arithmetic of the 2D strip kernels.  Plain C++ (constexpr functions are compiled for the device
// too).  A strip is E consecutive elements of a row; node column tn holds entry tn - K z of element z.
#pragma once

namespace ilh {

// The element that node column tn starts or lies in, and the one before, whose last column it may be.
// Lanes past the strip take the last element: they read its rows of LDS and drop them.
constexpr int strip_element(int tn, int K, int E) { return tn / K < E ? tn / K : E - 1; }
constexpr int strip_left(int tn, int K, int E) {
  const int l = tn / K > 0 ? tn / K - 1 : 0;
  return l < E ? l : E - 1;
}

// The last of the per-lane LDS rows (Q1D lanes an element, 64 a wave) that the node phase of W waves with
// GS lanes a node row reads
constexpr int strip_last_row(int K, int Q1D, int GS, int W, int E) {
  int last = 0;
  for (int tn = 0; tn < GS; ++tn) {
    const int e = strip_element(tn, K, E), l = strip_left(tn, K, E), m = e > l ? e : l;
    if (m > last) last = m;
  }
  return 64 * (W - 1) + last * Q1D + Q1D - 1;
}

}  // namespace ilh
