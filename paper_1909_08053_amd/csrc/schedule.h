// Host arithmetic of launches that hold the tiles of two problems.
#pragma once

namespace mlm {

// End of `units` units working through n0 items of c0 and then n1 of c1 (microseconds), each taking the next item when it is done.
inline double two_batches(int units, int n0, double c0, int n1, double c1) {
  const double t0 = (double)(n0 / units) * c0;
  const int busy = n0 % units;                        // units that are done with the first batch c0 later than the others
  double lo = busy ? t0 + c0 : t0, hi = t0 + c0 + c1 * (n1 / units + 2);
  auto done = [&](double t) {
    const double late = t - t0 - c0;
    return (double)(units - busy) * (long)((t - t0) / c1 + 1e-6) + (late > 0 ? (double)busy * (long)(late / c1 + 1e-6) : 0.0) >= n1;
  };
  if (done(lo)) return lo;
  for (int i = 0; i < 24; ++i) {
    const double mid = 0.5 * (lo + hi);
    if (done(mid)) hi = mid; else lo = mid;
  }
  return hi;
}

}  // namespace mlm
