// The cut of an expert's rows into dense items (kernels.h), over every row count.
#include <cstdio>

#include "kernels.h"

int main() {
  using namespace oled;
  for (const int R : {kDenseRowsSmall, kDenseRowsLarge})
    for (int rows = 1; rows <= 65535; ++rows) {
      const int m = dense_items(rows, R);
      int next = 0, least = R, most = 0;
      for (int i = 0; i < m; ++i) {
        const DenseItem d = dense_item(rows, R, i);
        if (d.first != next || d.rows <= 0 || d.rows > R || d.first % 32) {
          std::printf("R %d rows %d item %d: first %d rows %d\n", R, rows, i, d.first, d.rows);
          return 1;
        }
        next += d.rows;
        const int groups = (d.rows + 31) / 32;   // the last one may be partly filled
        least = groups < least ? groups : least;
        most = groups > most ? groups : most;
      }
      if (next != rows || most - least > 1) {
        std::printf("R %d rows %d: %d covered, items of %d to %d groups\n", R, rows, next, least, most);
        return 1;
      }
      // a tile's cost in the split over the XCDs is within its declared bounds
      const int cost = m * kDenseCostBase + (rows + 31) / 32;
      if (rows >= kDenseMinRows && (cost / m < kDenseCostMin || (cost + m - 1) / m > dense_cost_max(R))) {
        std::printf("R %d rows %d: cost %d of %d items\n", R, rows, cost, m);
        return 1;
      }
    }
  std::puts("ALL OK");
  return 0;
}
