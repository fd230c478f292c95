// How a scan is launched: tokens per time chunk and threads per workgroup,
// chosen from its descriptor alone.  Host code without HIP, internal to the
// library.
#pragma once

#include <stdint.h>

#include <cmath>
#include <initializer_list>

#include "precog.h"

namespace precog {

constexpr int64_t kShapeBlock = 512;     // threads of the larger workgroup
constexpr int64_t kShapeHalf = 256;      // and of the smaller one
constexpr int64_t kShapeCus = 256;       // compute units of the MI355X
constexpr int64_t kTargetWaves = 2048;   // 2 waves per SIMD on 256 CUs
constexpr int64_t kMinAutoChunk = 8;

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Longest chunk whose per-token streams stay addressable with the kernels'
// 32-bit buffer offsets: x, dt, z, y take D elements per token and B, C take
// N, at most 4 bytes each, so chunk * max(D, N) * 4 < 2^31.
inline int64_t max_chunk(const precog_scan_desc* d) {
  const int64_t w = d->dim > d->dstate ? d->dim : d->dstate;
  const int64_t row = (w > 0 ? w : 1) * 4;
  return ((1LL << 31) - 1) / row;
}

inline int64_t lanes_per_row(const precog_scan_desc* d) {
  return d->dim * (d->dstate > 16 ? d->dstate / 16 : 1);
}
inline int64_t waves_per_row(const precog_scan_desc* d) { return ceil_div(lanes_per_row(d), 64); }

struct ScanShape {
  int64_t chunk, threads;
};

// Time of a token in ns with one and with two waves on the fullest SIMD, of the
// pass with the readout and of the summary pass.  Measured, one pass of 1024
// tokens over 1024 and 2048 waves.  Three waves take 1.5 times two, four 1.9-2:
// every further wave counts half of two.
struct ScanRate {
  double one, two, sum_one, sum_two;
};
inline ScanRate scan_rate(const precog_scan_desc* d, bool complex) {
  const bool wide = d->in_dtype == PRECOG_F32;
  if (complex) return d->dstate == 16 ? ScanRate{555, 920, 485, 808} : ScanRate{490, 590, 390, 450};
  if (d->dstate > 16) return wide ? ScanRate{314, 420, 222, 295} : ScanRate{318, 405, 210, 270};
  if (d->dstate == 16) return wide ? ScanRate{318, 474, 213, 320} : ScanRate{289, 414, 208, 285};
  return wide ? ScanRate{276, 414, 153, 218} : ScanRate{266, 336, 123, 183};  // N = 8; fewer states less
}

// Threads of a workgroup: whole rows of up to four waves (a workgroup with
// waves past the last channel puts its live ones on the same SIMDs as the
// next: 2048 rows of 64 channels 726 ns a token with 512 threads, 442 with
// 64), else `large` or half of it.
inline int64_t group_threads(const precog_scan_desc* d, bool large) {
  const int64_t w = waves_per_row(d);
  return w > 0 && w <= 4 ? 64 * w : large ? kShapeBlock : kShapeHalf;
}

// Waves on the fullest SIMD when `chunks` chunks of every row run side by side.
// Workgroups of one wave spread over a CU's SIMDs (1024 rows of 64 channels 279
// ns a token), two of two waves do not (512 rows of 128 channels 387, 256 rows
// 265).
inline int64_t simd_waves(const precog_scan_desc* d, int64_t threads, int64_t chunks) {
  const int64_t groups = d->batch * ceil_div(lanes_per_row(d), threads) * chunks;
  const int64_t per_cu = ceil_div(groups, kShapeCus);
  const int64_t w = ceil_div(per_cu * (threads / 64), 4);
  return threads == 128 && per_cu > 1 && w < 2 ? 2 : w;
}

// The smaller workgroup where it leaves the fullest SIMD less to do (up to
// 1024 waves, one per SIMD: 365 -> 275 ns a token; 2304 waves 661 -> 554),
// the larger one, whose waves are balanced in pairs, where both are equal
// (1280 waves 368 against 393) and in launches of more than one round.
inline int64_t pick_threads(const precog_scan_desc* d, int64_t chunks) {
  const int64_t half = group_threads(d, false), block = group_threads(d, true);
  const int64_t groups = d->batch * ceil_div(lanes_per_row(d), half) * chunks;
  return groups <= 4 * kShapeCus && simd_waves(d, half, chunks) < simd_waves(d, block, chunks) ? half : block;
}

// Chunks for which a descriptor's workspace is sized: time may be cut when
// batch x channel waves alone do not fill two waves on every SIMD, into at
// most as many chunks as do.
inline int64_t reserve_chunks(const precog_scan_desc* d) {
  const int64_t L = d->seqlen;
  const int64_t waves = d->batch * waves_per_row(d);
  if (waves >= kTargetWaves || L <= 2 * kMinAutoChunk) return 1;
  int64_t nch = ceil_div(kTargetWaves, waves > 0 ? waves : 1);
  const int64_t max_nch = L / kMinAutoChunk;
  if (nch > max_nch) nch = max_nch;
  return nch < 1 ? 1 : nch;
}

// Pass 2 as a scan over the chunks' maps within one wave instead of a fold
// (real A; the kernels' launch takes the same test).
constexpr int64_t kCarryScanMaxChunks = 64;
constexpr int64_t kCarryScanMaxLanes = 8192;  // (b, d, n) lanes: waves of strided loads
inline bool carry_scan(int64_t chunks, int64_t lanes) {
  return chunks > 8 && chunks <= kCarryScanMaxChunks && lanes <= kCarryScanMaxLanes;
}

// Expected time in ns of a scan in `chunks` chunks of `chunk` tokens, with the
// readout and without.  A cut adds a summary pass over all chunks but the
// last, two launches (8.5 us), four trips of the states between the chunks at
// 4 TB/s, and the fold over the chunks (90 ns each, complex A 260).
struct ScanTime {
  double readout, states;
};
inline ScanTime scan_time(const precog_scan_desc* d, bool complex, int64_t chunk, int64_t chunks, int64_t threads) {
  const ScanRate r = scan_rate(d, complex);
  auto at = [&](int64_t n, double one, double two) {
    const int64_t w = simd_waves(d, threads, n);
    return static_cast<double>(chunk) * (w <= 1 ? one * static_cast<double>(w) : 0.5 * two * static_cast<double>(w));
  };
  const double sum = at(chunks, r.sum_one, r.sum_two);
  ScanTime t{at(chunks, r.one, r.two), sum};
  if (chunks > 1) {
    const int64_t lanes = d->batch * d->dim * d->dstate;
    const double n = static_cast<double>(chunks);
    double cut = 8500.0 + at(chunks - 1, r.sum_one, r.sum_two);
    cut += 4e-3 * n * static_cast<double>(lanes) * (complex ? 2.0 : 1.0);
    if (complex || !carry_scan(chunks, lanes)) cut += n * (complex ? 260.0 : 90.0);
    t.readout += cut;
    t.states += cut;
  }
  return t;
}

// Auto policy: of one pass, the cuts that put one or two waves on every SIMD
// with the one or the other workgroup size, and the fewer chunks at which the
// fold is still shorter than what further cuts save, the one expected to be
// over first.  Filling to just past a whole number of workgroups per CU is
// what this avoids: 5 x 1237 x 1000 in 26 chunks is 260 workgroups (60.5 us),
// in 25 it is 250 (48.8 us).  The shape is the descriptor's alone, so that
// scans with and without a readout or a trajectory give the same final
// states: it has the smallest sum of both expected times.
inline ScanShape auto_shape(const precog_scan_desc* d, bool complex) {
  const int64_t L = d->seqlen;
  const int64_t most = reserve_chunks(d);
  ScanShape best{L, pick_threads(d, 1)};
  if (most <= 1) return best;
  const ScanTime one = scan_time(d, complex, L, 1, best.threads);
  double best_ns = one.readout + one.states;
  const ScanRate r = scan_rate(d, complex);
  const double fold = std::sqrt(static_cast<double>(L) * (r.one + r.sum_one) / (complex ? 260.0 : 90.0));
  for (const bool large : {true, false}) {
    const int64_t threads = group_threads(d, large);
    const int64_t row_groups = d->batch * ceil_div(lanes_per_row(d), threads);
    const int64_t rows = row_groups > 0 ? row_groups : 1;
    // workgroups on a CU with two waves and with one on a SIMD, and one
    const int64_t two = kShapeCus * (512 / threads) / rows, one_each = kShapeCus * (256 / threads) / rows;
    for (int64_t n : {two, one_each, kShapeCus / rows, static_cast<int64_t>(fold), kCarryScanMaxChunks}) {
      if (n > two) n = two;
      if (n > most) n = most;
      if (n < 2) continue;
      const int64_t chunk = ceil_div(L, n);
      const ScanTime t = scan_time(d, complex, chunk, ceil_div(L, chunk), threads);
      if (t.readout + t.states < best_ns) {
        best_ns = t.readout + t.states;
        best = ScanShape{chunk, threads};
      }
    }
  }
  return best;
}

// Chunk length and workgroup size used for a descriptor (after validation).
inline ScanShape scan_shape(const precog_scan_desc* d, bool complex) {
  const int64_t L = d->seqlen;
  if (L <= 0) return ScanShape{1, kShapeBlock};
  const int64_t cap = max_chunk(d);
  ScanShape s{d->chunk, kShapeBlock};
  if (d->chunk <= 0) s = auto_shape(d, complex);
  if (s.chunk > L) s.chunk = L;
  const bool cut = s.chunk > cap;
  if (cut) s.chunk = cap;
  if (d->chunk > 0 || cut) s.threads = pick_threads(d, ceil_div(L, s.chunk));
  return s;
}

// Chunks the workspace of a descriptor is sized for: those an automatic cut may
// take at most (auto_shape stays within reserve_chunks), or those requested.
inline int64_t workspace_chunks(const precog_scan_desc* d) {
  const int64_t L = d->seqlen;
  if (L <= 0) return 1;
  const int64_t cap = max_chunk(d);
  int64_t chunk = d->chunk > 0 ? d->chunk : ceil_div(L, reserve_chunks(d));
  if (chunk > L) chunk = L;
  if (chunk > cap) chunk = cap;
  return ceil_div(L, chunk);
}

}  // namespace precog
