// Rows of the zero-padded input that a band of consecutive reduction indices of
// the backward-weights convolution touches, at most over the bands of a layer.
// Host arithmetic only (no HIP), so that a test can compile it by itself.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <numeric>

namespace dfp {

struct BandRows {
  int64_t T, P, Q;      // reduction length N*P*Q, output height and width
  int64_t Hpad, sh, R;  // padded input rows per image, row stride, filter rows
  int64_t band;         // indices per band (a multiple of 32)
};

// Rows from the first one index ta reads to the last one index tb reads.
inline int64_t band_rows(const BandRows& g, int64_t ta, int64_t tb) {
  const int64_t PQ = g.P * g.Q;
  const int64_t za = (ta / PQ) * g.Hpad + ((ta % PQ) / g.Q) * g.sh;
  const int64_t zb = (tb / PQ) * g.Hpad + ((tb % PQ) / g.Q) * g.sh + g.R - 1;
  return zb - za + 1;
}

// The maximum over all bands: segments of seg_len indices, each in bands from
// its own (32-aligned) start.
//
// Where segments are whole bands, band i starts at index band * i, and a few
// bands stand for all of them (a plan scans them on every call: 64 images of
// 111 x 111 are 6160 bands, 54 us one by one and under 3 us so):
//   - a band inside one image touches a number of rows that only grows with its
//     first column, and the columns band * i mod Q repeat after Q / gcd(Q, band)
//     bands;
//   - what a band across an image's end touches depends on where in it the end
//     lies, n P Q mod band for image n, which repeats after band / gcd(P Q, band)
//     images.  (It touches no fewer rows than a band inside an image with the same
//     first column as long as an image's end skips no rows backwards.)
// Images of less than a band, and strides that leave the last rows unread,
// scan one period of the bands instead.
inline int64_t band_rows_max(const BandRows& g, int64_t seg_len) {
  const int64_t B = g.band, PQ = g.P * g.Q, nbands = (g.T + B - 1) / B;
  int64_t rows = 0;
  auto at = [&](int64_t i) { rows = std::max(rows, band_rows(g, i * B, std::min((i + 1) * B, g.T) - 1)); };
  if (seg_len % B == 0 || seg_len >= g.T) {
    if (PQ < B || g.Hpad < g.P * g.sh) {
      const int64_t period = PQ / std::gcd(PQ, B);
      for (int64_t i = 0; i < std::min(nbands, period); ++i) at(i);
      return rows;
    }
    const int64_t columns = g.Q / std::gcd(g.Q, B), ends = B / std::gcd(PQ, B), images = g.T / PQ;
    for (int64_t i = 0; i < std::min(nbands, columns); ++i) at(i);
    for (int64_t n = 1; n <= std::min(images - 1, ends); ++n) at((n * PQ - 1) / B);
    return rows;
  }
  for (int64_t t0 = 0; t0 < g.T; t0 += seg_len) {
    const int64_t t1 = std::min(t0 + seg_len, g.T);
    for (int64_t sb = t0 / 32; sb < (t1 + 31) / 32; sb += B / 32)
      rows = std::max(rows, band_rows(g, std::max(sb * 32, t0), std::min(sb * 32 + B, t1) - 1));
  }
  return rows;
}

}  // namespace dfp
