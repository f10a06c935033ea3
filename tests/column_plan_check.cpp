// Replays the LDS indices of the column kernel for every split that the library
// plans: see test_column_plan_cpu.py.  Prints the number of tiles it went
// through; any violation ends the program with status 1.
#include <cstdio>
#include <cstdlib>
#include <set>
#include <tuple>
#include <utility>
#include <vector>

#include "internal.hpp"

using namespace lbm;

static long tiles = 0;

static void fail(const char* what, int Q, int nx, int rows, int nsub, int ny, int tile) {
  std::printf("%s: Q %d nx %d rows %d nsub %d ny %d tile %d\n", what, Q, nx, rows, nsub, ny, tile);
  std::exit(1);
}

// One tile of a plate of ny rows.
template <class L>
static void replay(int nx, int es, int rows, int nsub, int ny, int tile) {
  constexpr int Q = L::Q, R = L::R, cap = kColumnCells;
  auto bad = [&](const char* what) { fail(what, Q, nx, rows, nsub, ny, tile); };
  const int y0 = tile * rows, y1 = y0 + rows < ny ? y0 + rows : ny;
  const int ylo = y0 - R * nsub, region = rows + 2 * R * nsub;
  const int ys = column_stride(region, nx, es);
  if (region * nx > cap || ys < region || ys * nx > cap) bad("the planes do not fit");
  // columns of the reflections of one cell differ by the velocity only, so
  // rows suffice: which (velocity, row) behind a wall is written
  std::vector<int> written(Q * region, 0);
  for (int row = 0; row < region; ++row) {
    const int y = ylo + row;
    if (y < 0 || y >= ny) continue;
    for (int q = 0; q < Q; ++q)
      for (int x : {0, nx - 1}) {
        int g = -1;
        if (y < L::vy[q]) g = row_behind_moving(row, y, region);
        else if (ny - 1 - y < -L::vy[q]) g = row_behind_far(row, ny - 1 - y, region);
        else continue;
        if (g == -1) continue;
        // inside the plane and column of the velocity, on no lattice row
        const int at = q * cap + x * ys + g;
        if (at < q * cap || at >= (q + 1) * cap) bad("a reflection leaves its plane");
        if (g < 0 || g >= region) bad("a reflection leaves its column");
        if (ylo + g >= 0 && ylo + g < ny) bad("a reflection lands on a lattice row");
        if (x == 0) ++written[q * region + g];
      }
  }
  // every pull of a cell that a step updates (the first one updates most) comes
  // from a row of the region that holds a lattice row, or one reflection
  const int more = R * (nsub - 1);
  for (int row = 0; row < region; ++row) {
    const int y = ylo + row;
    if (y < 0 || y >= ny || y < y0 - more || y >= y1 + more) continue;
    for (int q = 0; q < Q; ++q) {
      const int from = row - L::vy[q], sy = ylo + from;
      if (from < 0 || from >= region) bad("a pull leaves the region");
      if ((sy < 0 || sy >= ny) && written[q * region + from] != 1)
        bad("a pull from behind a wall has no source");
    }
  }
  ++tiles;
}

template <class L>
static void check() {
  constexpr int Q = L::Q, R = L::R;
  for (int nx = 3; nx <= kColumnMaxNx; ++nx) {
    // every plan of lattices of this width: it depends on their lengths only
    // through the workgroups they take
    std::set<std::pair<int, int>> plans;
    for (bool f64 : {false, true}) {
      auto add = [&](const std::vector<int>& ny) {
        const ColumnPlan p = column_plan(Q, f64, nx, ny);
        if (p.rows < 1 || p.max_sub < 1 || (p.rows + 2 * R * p.max_sub) * nx > kColumnCells)
          fail("plan", Q, nx, p.rows, p.max_sub, ny[0], (int)ny.size());
        // a row's cells on a bank each, or nearly
        if (nx > 4 && column_stride(p.rows + 2 * R * p.max_sub, nx, f64 ? 8 : 4) % (f64 ? 16 : 32) == 0)
          fail("columns on one bank", Q, nx, p.rows, p.max_sub, ny[0], (int)ny.size());
        plans.insert({p.rows, p.max_sub});
      };
      for (int groups = 1; groups < 70; ++groups) {
        add({groups * 40});
        add(std::vector<int>(groups, 4096));
      }
      for (int ny = 2000; ny < 20000; ny += 151) add({ny});
      for (int ny = 20000; ny < 4000000; ny += ny / 7) add({ny});
    }
    for (const auto& [rows, most] : plans) {
      std::set<int> subs;
      for (int n = 1; n <= 3 * most + 2; ++n)
        for (int k : odd_pieces(n, most)) subs.insert(k);
      for (int nsub : subs) {
        if (nsub < 1 || nsub > kColumnMaxSub || nsub % 2 == 0)
          fail("an even piece", Q, nx, rows, nsub, 0, 0);
        const ColumnShape sh = column_shape(Q, nx, rows, nsub);
        if (sh.threads > kColumnThreads || sh.threads - 64 < (rows + 2 * R * nsub) * nx)
          fail("threads", Q, nx, rows, nsub, 0, 0);
        // tiles in reach of a wall, the far one at every offset in its tile
        const int reach = (R * nsub + R) / rows + 2;
        for (int es : {4, 8}) {
          for (int tile = 0; tile < reach; ++tile)
            replay<L>(nx, es, rows, nsub, 4 * reach * rows, tile);
          for (int rest = 1; rest <= rows; ++rest) {
            const int ny = 2 * reach * rows + rest, last = (ny + rows - 1) / rows - 1;
            for (int tile = last; tile > last - reach; --tile) replay<L>(nx, es, rows, nsub, ny, tile);
          }
          // thin plates: both walls in one region
          for (int ny = R < 3 ? 3 : R; ny <= 2 * rows; ++ny)
            for (int tile = 0; tile * rows < ny; ++tile) replay<L>(nx, es, rows, nsub, ny, tile);
        }
      }
    }
  }
}

int main() {
  check<D2Q9>();
  check<D2Q37>();
  std::printf("%ld tiles\n", tiles);
  return 0;
}
