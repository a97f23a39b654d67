// Host arithmetic of launches: two problems in one, and threads of the pass that forms the gradients of the logits.
#pragma once

namespace mlm {

// Vectors of a row of logits (nv in all) that a thread takes: four, one workgroup a row, up to 1024 vectors and from two rows a compute
// unit on (8192 x 6400 bf16 37.2 -> 33.0 us, where every fourth workgroup had an eighth of its threads at work; 1000 x 2056 7.0 -> 5.0);
// fewer rows leave units idle in that form (40 x 6400 2.7 / 3.2, 300 x 6400 4.9 / 5.3), and of longer rows it gains nothing (8192 x 51200
// in fours 266 -> 279).
inline int dlogits_vectors(int rows, int nv, int cus) { return nv <= 1024 && rows >= 2 * cus ? 4 : 1; }

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
