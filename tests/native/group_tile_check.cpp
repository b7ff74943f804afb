// Host check of the tile a launch of several GEMMs takes (csrc/kernels.hip), against the rule written
// out here.  Linked with the library; no GPU.  One line per failure; exit status 0 if none.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "kernels.hpp"

using namespace psc;

static int failures = 0;
static void check(bool ok, const char *what, int a, int b) {
  if (ok) return;
  ++failures;
  std::printf("%s: tile %d, %d\n", what, a, b);
}

struct Shape {
  int m, n;
};
constexpr Shape kTile[13] = {{0, 0},   {128, 128}, {64, 64}, {32, 32}, {128, 64}, {64, 128}, {64, 64},
                             {32, 64}, {64, 32},   {32, 32}, {16, 32}, {32, 16},  {16, 16}};

static std::vector<GemmArgs> gemms(int rows, int count, int n = 512, int k = 512) {
  GemmArgs a{};
  a.M = rows;
  a.N = n;
  a.K = k;
  return std::vector<GemmArgs>(size_t(count), a);
}
static std::vector<GemmArgs> operator+(std::vector<GemmArgs> a, const std::vector<GemmArgs> &b) {
  a.insert(a.end(), b.begin(), b.end());
  return a;
}
static long blocks(const std::vector<GemmArgs> &v, int t) {
  long n = 0;
  for (const GemmArgs &a : v) n += long((a.M + kTile[t].m - 1) / kTile[t].m) * ((a.N + kTile[t].n - 1) / kTile[t].n);
  return n;
}

int main() {
  for (int tile : {2, 6, 10, 12})
    for (int count : {2, 4, 8, 16, 40})
      for (int rows : {1, 16, 17, 33, 64, 100, 512, 1000}) {
        const std::vector<GemmArgs> v = gemms(rows, count);
        const int t = gemm_group_tile(v, tile);
        check(gemm_sum_order(t) == gemm_sum_order(tile), "another summation order", t, tile);
        // alike members: a tile at least twice as high as the rows is taken only as the last resort
        check(t == (tile == 2 ? 2 : 12) || kTile[t].m < 2 * std::max(rows, 16), "mostly padding", t, rows);
        // one short member beside them changes nothing where it is an eighth of the blocks at most
        const std::vector<GemmArgs> w = v + gemms(1, 1);
        const int s = gemm_group_tile(w, tile);
        check(gemm_sum_order(s) == gemm_sum_order(tile), "another summation order with a short member", s, tile);
        if (8 * blocks(gemms(1, 1), t) <= blocks(w, t) && blocks(v, t) >= 384)
          check(kTile[s].m * kTile[s].n >= kTile[t].m * kTile[t].n, "a short member sets a smaller tile", s, t);
        // and many short ones do not: their padding would be most of the work
        const std::vector<GemmArgs> x = gemms(rows, 1) + gemms(1, 400);
        const int u = gemm_group_tile(x, tile);
        if (rows <= 512) check(u == (tile == 2 ? 2 : 12) || kTile[u].m <= 16, "short members padded", u, rows);
      }
  std::printf("%d failures\n", failures);
  return failures != 0;
}
