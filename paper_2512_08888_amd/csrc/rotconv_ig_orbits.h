// The k x k positions of a filter as orbits of four that a quarter turn permutes (and the centre), the order in which the
// one-contraction kernels (rotconv_ig_*.hip) use and store a filter's taps.
#pragma once

#include <hip/hip_runtime.h>

namespace rotconv {

// Position (i, j) of the k x k window after a quarter turn of the filter: (k - 1 - j, i).
struct Orbit { int i, j; };
__device__ __host__ __forceinline__ Orbit orbit_rep(int o, int k) { return Orbit{o / (k / 2), o % (k / 2)}; }
__device__ __host__ __forceinline__ Orbit turn(Orbit t, int k) { return Orbit{k - 1 - t.j, t.i}; }

// The tap that tile t of a block of turning filters holds: the orbits one after the other, then the centre.
__device__ __host__ __forceinline__ int packed_tap(int t, int k) {
  if ((k & 1) && t == k * k - 1) return k * k / 2;
  Orbit at = orbit_rep(t / 4, k);
  for (int m = 0; m < t % 4; ++m) at = turn(at, k);
  return at.i * k + at.j;
}

}  // namespace rotconv
