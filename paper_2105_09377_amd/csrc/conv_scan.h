// Host: how many patch rows the tiles of a convolution need.  Plain C++, so that a test can hold it against a
// count over every tile without a GPU.
#pragma once
#include <stdint.h>

#include <numeric>

namespace gs {

// Most patch rows that any tile of `tp` consecutive ones of `m` positions needs, (rows between its first and last
// output row) * sh + kh for every image that it touches, or -1 if a tile touches more than `max_images`.
// What a tile needs follows from where in an image it starts, and tiles start hwo / gcd(hwo, tp) different ways
// before they repeat; the last tile, cut short, is looked at by itself.  *looked: tiles looked at.
inline int scan_patch_rows(int64_t m, int64_t hwo, int64_t wo, int64_t sh, int64_t kh, int64_t tp, int max_images,
                           int64_t* looked = nullptr) {
  const int64_t whole = m / tp, period = hwo / std::gcd(hwo, tp), n = whole < period ? whole : period;
  if (looked) *looked = n + (m % tp ? 1 : 0);
  int64_t most = 0;
  for (int64_t i = 0; i <= n; ++i) {
    const int64_t first = (i < n ? i : whole) * tp, end = i < n || first + tp < m ? first + tp : m;
    if (first >= end) break;                              // no tile is cut short
    const int64_t n0 = first / hwo, n1 = (end - 1) / hwo, p0 = first - n0 * hwo, p1 = end - 1 - n1 * hwo;
    if (n1 - n0 + 1 > max_images) return -1;
    const int64_t r0 = p0 / wo, r1 = p1 / wo, last = hwo / wo - 1;    // output rows of the first and the last position
    const int64_t rows = n0 == n1 ? r1 - r0 : (last - r0) + (n1 - n0 - 1) * last + r1;
    const int64_t need = rows * sh + (n1 - n0 + 1) * kh;
    if (need > most) most = need;
  }
  return int(most);
}

}  // namespace gs
