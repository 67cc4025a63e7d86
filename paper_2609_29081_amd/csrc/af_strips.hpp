// af_strips.hpp -- how the 2D strip kernel (af_strip2d.hip) cuts a grid: host
// arithmetic alone, without HIP.
#pragma once

#include <algorithm>

namespace afi {

constexpr int kStripColumns = 60;  // cell columns of a strip

// Strips of a grid: nx along x, ny ranges of H rows; for one instance, and for
// the instances of a batch, which are launched together
struct StripShape {
  int nx, ny, H;
};

// the strips of a grid of n1x columns and n2y rows of points in ranges of H rows
inline StripShape strips_with(int n1x, int n2y, int H) {
  return StripShape{(n1x + kStripColumns - 1) / kStripColumns, (n2y + H - 1) / H, H};
}

// The strips of a single grid.  One workgroup fills a CU (its LDS), so a launch
// runs in ceil(nx ny / cus) rounds of H + 5 row steps each (a row is finished
// three rows behind the march, which starts two rows early): the H with the
// fewest steps in all, and of those the largest, with at most 8 rounds and `most`
// strips beside one range.  Of the row counts that fit a number of rounds the one
// with the most ranges has the lowest strips, so it alone is looked at: this is
// asked for at every launch, and a look at every count took 4 us at 400 x 200 and
// 35 at 57 x 2000.
inline StripShape strip_shape(int n1x, int n2y, int cus, long most) {
  StripShape b = strips_with(n1x, n2y, n2y);
  auto steps = [cus](const StripShape& t) {
    return ((long)t.nx * t.ny + cus - 1) / cus * (t.H + 5);
  };
  long best = steps(b);
  most = std::min(most, 8L * cus);
  for (long q = 1;; ++q) {
    const long fit = std::min(q * cus, most) / b.nx, ny = std::min(fit, (long)n2y);
    if (ny > 1) {
      const StripShape t = strips_with(n1x, n2y, (int)((n2y + ny - 1) / ny));
      if (steps(t) < best) {
        b = t;
        best = steps(t);
      }
    }
    if (q * cus >= most || fit >= n2y) return b;
  }
}

}  // namespace afi
