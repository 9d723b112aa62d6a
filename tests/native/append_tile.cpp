// Tile choice of kv_append at the edges of its rules: a launch's grid must hold
// fewer than 2^32 threads, counted in whole tiles.
#include <cstdio>

#include "append_grid.h"

using hswa::append_groups;
using hswa::append_tile;

static int fails = 0;

static void expect(int want, bool single, int32_t ns, int32_t total, int32_t hkv) {
  const int tile = append_tile(single, ns, total, hkv);
  const long long threads = (long long)append_groups(tile, total, hkv) * hswa::kAppendThreads;
  if (tile == want && threads < (1ll << 32)) return;
  std::printf("ns %d, %d tokens, %d heads: tile %d (expected %d), %lld threads\n", ns, total, hkv, tile, want, threads);
  ++fails;
}

int main() {
  // the rules of the lengths
  expect(8, true, 100000, 100000, 8);
  expect(8, false, 1, 256, 8);
  expect(32, false, 1, 257, 8);
  expect(32, false, 4, 259, 8);  // 64 a sequence
  expect(8, false, 5, 300, 8);   // 60
  expect(8, false, 32, 512, 8);
  expect(16, false, 32, 513, 8);
  expect(8, false, 33, 527, 8);  // fewer than 16 a sequence
  expect(16, false, 20, 559, 8);
  expect(32, false, 20, 560, 8);  // 28
  // few heads: the workgroups of 8-token tiles count, not the tokens
  expect(8, false, 1, 2048, 1);
  expect(32, false, 1, 2049, 1);
  expect(8, false, 128, 2048, 2);
  expect(16, false, 128, 2049, 2);
  expect(8, false, 27, 540, 1);
  expect(8, false, 3, 240, 16);  // more than 8 heads: the tokens
  expect(32, false, 3, 257, 16);
  // the grid: 8-token tiles up to one workgroup fewer than 2^32 threads take
  const int32_t ns = 1 << 21;  // fewer than 16 tokens a sequence
  expect(8, false, ns, (1 << 24) - 8, 8);
  for (int d = 1; d < 8; ++d) expect(32, false, ns, (1 << 24) - d, 8);  // exactly 2^32 threads in 8-token tiles
  expect(32, false, ns, 1 << 24, 8);
  expect(8, false, 32760, 32760, 4096);
  for (int t = 32761; t <= 32769; ++t) expect(32, false, 32760, t, 4096);
  expect(32, false, 1, 1 << 25, 8);
  std::printf(fails ? "failed %d\n" : "ok\n", fails);
  return fails != 0;
}
