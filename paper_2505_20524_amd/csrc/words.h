// How a workgroup of THREADS threads reads the words that a scale comes from.  (No device types: the walk also runs on the host.)
#pragma once

// take(i, p[i]) for words i = tid, + THREADS, ... of `n` but never of word `skip` (none if negative), which another workgroup may be
// storing: p[skip] is not read at all.  In batches of four independent loads; in a plain loop each waits for the one before it.
template <int THREADS, typename P, typename F>
FOG_DEVICE void for_words(P p, int n, int skip, int tid, F take) {
  for (int base = 0; base < n; base += 4 * THREADS) {
    decltype(+p[0]) v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = base + k * THREADS + tid;
      v[k] = {};
      if (i < n && i != skip) v[k] = p[i];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = base + k * THREADS + tid;
      if (i < n && i != skip) take(i, v[k]);
    }
  }
}
