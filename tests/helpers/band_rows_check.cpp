// Compares band_rows_max with a scan of every band over a grid and random layers,
// and times it on the layers whose scan was long.
#include <chrono>
#include <cstdio>
#include <random>

#include "band_rows.h"

static int64_t scan(const dfp::BandRows& g, int64_t seg_len) {
  int64_t rows = 0;
  for (int64_t t0 = 0; t0 < g.T; t0 += seg_len) {
    const int64_t t1 = std::min(t0 + seg_len, g.T);
    for (int64_t sb = t0 / 32; sb < (t1 + 31) / 32; sb += g.band / 32)
      rows = std::max(rows, dfp::band_rows(g, std::max(sb * 32, t0), std::min(sb * 32 + g.band, t1) - 1));
  }
  return rows;
}

int main() {
  std::mt19937 rng(1);
  long checked = 0;
  auto check = [&](int64_t n, int64_t h, int64_t w, int64_t r, int64_t s, int64_t sh, int64_t sw, int64_t ph, int64_t pw,
                   int64_t seg_len) {
    if (h + 2 * ph < r || w + 2 * pw < s) return true;
    const int64_t p = (h + 2 * ph - r) / sh + 1, q = (w + 2 * pw - s) / sw + 1;
    const dfp::BandRows g{n * p * q, p, q, h + 2 * ph, sh, r, 128};
    const int64_t got = dfp::band_rows_max(g, seg_len), want = scan(g, seg_len);
    ++checked;
    if (got == want) return true;
    std::printf("n %ld h %ld w %ld r %ld s %ld stride %ld %ld pad %ld %ld seg %ld: %ld, scan %ld\n", (long)n, (long)h,
                (long)w, (long)r, (long)s, (long)sh, (long)sw, (long)ph, (long)pw, (long)seg_len, (long)got, (long)want);
    return false;
  };
  for (int64_t h = 1; h <= 40; ++h)
    for (int64_t w = 1; w <= 140; ++w)
      for (int64_t st = 1; st <= 3; ++st)
        if (!check(1 + (h * w) % 5, h, w, 1 + (w % 3), 1 + (h % 3), st, st, w % 2, h % 2, 4096)) return 1;
  const int64_t segs[] = {64, 96, 128, 256, 1000, 1024, 4096, 8192, 1 << 30};
  for (int i = 0; i < 200000; ++i) {
    auto u = [&](int64_t a, int64_t b) { return a + (int64_t)(rng() % (uint32_t)(b - a + 1)); };
    const int64_t big = i % 50 == 0;
    if (!check(u(1, big ? 64 : 6), u(1, big ? 130 : 30), u(1, big ? 400 : 60), u(1, 7), u(1, 7), u(1, 5), u(1, 5), u(0, 3),
               u(0, 3), segs[u(0, 8)]))
      return 1;
  }
  std::printf("%ld layers agree\n", checked);
  for (int64_t hw : {63, 111, 113}) {
    const dfp::BandRows g{64 * hw * hw, hw, hw, hw + 2, 1, 3, 128};
    volatile int64_t sink = 0;
    const auto t0 = std::chrono::steady_clock::now();
    for (int i = 0; i < 2000; ++i) sink = sink + dfp::band_rows_max(g, 4096);
    const double us = std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count() / 2000;
    std::printf("%ld x %ld: %.2f us\n", (long)hw, (long)hw, us);
    if (us > 10) return 1;  // (the scan of every band: 20 to 60)
  }
  return 0;
}
