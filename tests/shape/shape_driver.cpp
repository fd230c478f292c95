// Prints the launch shape the library chooses for scan descriptors read from
// standard input, one "complex in_dtype batch seqlen dim dstate chunk" per
// line: tokens per chunk, chunks, threads, waves on the fullest SIMD, expected
// ns with and without readout, those of one pass, and the workspace's chunks.
// Host code only; test infrastructure.
#include <cstdio>

#include "scan_shape.h"

int main() {
  int complex, in;
  long long b, l, d, n, c;
  while (std::scanf("%d %d %lld %lld %lld %lld %lld", &complex, &in, &b, &l, &d, &n, &c) == 7) {
    precog_scan_desc x{};
    x.batch = b;
    x.seqlen = l;
    x.dim = d;
    x.dstate = n;
    x.chunk = c;
    x.in_dtype = in ? PRECOG_BF16 : PRECOG_F32;
    const precog::ScanShape s = precog::scan_shape(&x, complex != 0);
    const int64_t chunks = precog::ceil_div(l, s.chunk);
    const precog::ScanTime t = precog::scan_time(&x, complex != 0, s.chunk, chunks, s.threads);
    const precog::ScanTime one = precog::scan_time(&x, complex != 0, l, 1, precog::pick_threads(&x, 1));
    std::printf("%lld %lld %lld %lld %.0f %.0f %.0f %.0f %lld\n", (long long)s.chunk, (long long)chunks,
                (long long)s.threads, (long long)precog::simd_waves(&x, s.threads, chunks), t.readout, t.states,
                one.readout, one.states, (long long)precog::workspace_chunks(&x));
  }
  return 0;
}
