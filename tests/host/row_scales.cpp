// Row-scale bytes that the tiles of a batch request, against the buffer that
// holds them, for batches whose pair count is right and for miscounted ones
// (n_pairs below the ids' own count: the library reports those, so they may
// not read out of range either).  Tiles are listed here as the routing scan's
// rules state it: an expert's rows padded to the alignment, tiles of m rows
// each, a tile listed when its rows lie inside the grouped rows.
#include "common.h"

#include <cstdio>
#include <cstdlib>
#include <vector>

using namespace cep;

static int checked = 0, last_group = 0;

static void check(const std::vector<int> &cnt, int max_mpad, int align, int m) {
  const int groups = max_mpad / 128;  // groups per K step in the scale buffers
  int pad = 0;
  for (const int c : cnt) {
    for (int q = 0; q * m < c; ++q) {
      const int row0 = pad + q * m, rows = c - q * m < m ? c - q * m : m;
      if (row0 + rows > max_mpad) break;
      const int n = mx_row_groups(row0, rows);
      // the last K step's load starts at group row0 / 128 and ends n groups on
      if (row0 / 128 + n > groups || n * 128 < row0 % 128 + rows || n < 1 || n > (m + 254) / 128) {
        std::printf("tile at row %d of %d (%d rows, tiles of %d): %d groups, buffer of %d\n",
                    row0, max_mpad, rows, m, n, groups);
        std::exit(1);
      }
      ++checked;
      last_group += row0 / 128 == groups - 1;
    }
    pad += (c + align - 1) / align * align;
  }
}

int main() {
  // counted by hand: 2000 declared pairs of 8 experts, 3552 real ones; the tile
  // at row 4224 lies in the last of 34 groups
  const int mpad = (int)align_up(2000, kMaxAlign) + kMaxAlign * 9;
  check({160, 160, 160, 160, 160, 400, 400, 1952}, mpad, kFp8TileM, kRowsMidM);
  if (mpad != 4352 || last_group != 1) return std::printf("example: %d %d\n", mpad, last_group), 1;
  unsigned long long s = 1;
  auto rnd = [&](int n) {
    s = s * 6364136223846793005ull + 1442695040888963407ull;
    return (int)((s >> 33) % (unsigned)n);
  };
  for (int it = 0; it < 200000; ++it) {
    const int E = 1 + rnd(16), P = 1 + rnd(3000);
    std::vector<int> c(E, 0);
    const int real = rnd(3) ? 1 + rnd(2 * P + 600) : P;  // declared: P
    for (int left = real; left > 0;) {
      const int n = 1 + rnd(left < 400 ? left : 400);
      c[rnd(E)] += n;
      left -= n;
    }
    for (const int m : {kRowsSmallM, kRowsMidM}) {
      check(c, (int)align_up((size_t)P, kMaxAlign) + kMaxAlign * (E + 1), kFp8TileM, m);
      check(c, (int)align_up((size_t)P + (size_t)E * kFp8TileM, kMaxAlign), kFp8TileM, m);
    }
  }
  if (last_group < 1000) return std::printf("only %d tiles in the last group\n", last_group), 1;
  std::printf("%d tiles, %d in the last group\n", checked, last_group);
  return 0;
}
