// Index maps of the symmetric extension of a line of n samples to a period of P.
#pragma once

#include <hip/hip_runtime.h>

namespace scat {

// Sample that position i of the period shows: the margin's first half mirrors the right edge, the
// rest the left edge of the next period; reflections repeat with period 2n.
__device__ __forceinline__ int pad_source(int i, int n, int P) {
  const int h = (P - n + 1) / 2;
  int v = i < n + h ? i : i - P;
  v %= 2 * n;
  if (v < 0) v += 2 * n;
  return v < n ? v : 2 * n - 1 - v;
}

// Positions of the period-P extension that mirror sample r of n (see pad_source): virtual
// positions v = r + 2 n t and v = 2 n - 1 - r + 2 n t inside [-(P - n - h), n + h), stored
// at v (v >= 0) or v + P.  Calls f(position) for each.
template <class Fn>
__device__ __forceinline__ void for_each_image(int r, int n, int P, Fn f) {
  const int h = (P - n + 1) / 2, lo = P - n - h;
  const int reps = P / (2 * n) + 1;
  for (int t = -reps; t <= reps; ++t) {
    const int v0 = r + 2 * n * t, v1 = 2 * n - 1 - r + 2 * n * t;
    if (v0 >= -lo && v0 < n + h) f(v0 >= 0 ? v0 : v0 + P);
    if (v1 >= -lo && v1 < n + h) f(v1 >= 0 ? v1 : v1 + P);
  }
}

}  // namespace scat
