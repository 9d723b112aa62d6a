// Tile and grid of a kv_append launch (host arithmetic only).
#pragma once

#include <stdint.h>

namespace hswa {

// Tokens of a workgroup's tile. `single`: one token per sequence (decode step).
// A few tokens per sequence, or a few in all (or a few workgroups of 8-token
// tiles: few KV heads), are bound by the launch and a chain of loads: 8-token
// tiles, scattered, put them on more compute units with the rows' loads ahead of
// the slots. Longer sequences are written by runs of
// 32 positions: from 16-token tiles where the mean is short, since a tile's
// runs and scattered tokens follow each other, from 32-token ones otherwise,
// half of a long sequence's 16-token tiles having no run to write. The host
// knows no sequence's own length, so the mean decides; a long sequence among
// many single tokens then takes the 8-token tiles, which write eight tokens on
// aligned slots as wide as a run does. 8 heads, PG 64, us per call with tiles of
// 8 / 16 / 32 tokens:
//   16 sequences x 16, unaligned              4.2 /  5.0 /  7.1
//   32 x 12, unaligned                        5.2 /  6.7 /  8.1
//   10 x 30, unaligned                        4.7 /  5.9 /  5.9
//   512 + 16 x 8, aligned                     4.0 /  4.9 /  6.5
//   100 x 16, unaligned                      12.2 / 10.2 / 10.7
//   128 x 24, unaligned                      18.9 / 12.2 / 13.2
//   200 x 36, unaligned                         - / 18.8 / 19.0
//   200 x 36, unaligned, 2 heads                - /  9.9 /  9.3
//   800 x 36, unaligned                         - / 74.9 / 73.4
//   100 x 47, aligned                        26.6 / 13.1 / 12.1
//   8 x 1536, aligned                        20.5 / 21.5 / 16.6
//   8 x 1500, unaligned                      58.1 / 18.9 / 18.1
//   2048 aligned among 256 single ones       10.7 / 11.4 / 11.9
//   27 x 20, unaligned, 1 head                3.5 /  5.5 /  6.6
//   20 x 80, unaligned, 1 head                4.1 /    - /  5.7
//   20 x 40, unaligned, 4 heads               5.1 /    - /  5.6
//   150 x 20, aligned, 1 head                 5.4 /  4.5 /  5.4
// (16 heads need no fewer tokens than 8: 3 x 80 unaligned 4.3 in 8-token tiles,
// 5.1 by runs).
// A grid holds fewer than 2^32 threads, counted in whole tiles: calls that
// smaller tiles would take past that (from just under 2^27 token-heads on,
// 69 GB of input) take 32-token ones whatever their lengths.
constexpr int kAppendThreads = 256;
constexpr int64_t kAppendMaxGroups = (int64_t{1} << 32) / kAppendThreads - 1;

constexpr int64_t append_groups(int tile, int32_t total_tokens, int32_t hkv) {
  return ((int64_t)total_tokens + tile - 1) / tile * hkv;
}

constexpr int append_tile(bool single, int32_t ns, int32_t total_tokens, int32_t hkv) {
  const int64_t groups8 = append_groups(8, total_tokens, hkv);
  const int64_t n = groups8 < total_tokens ? groups8 : total_tokens;
  const bool runs = !single && ((n > 512 && total_tokens / 16 >= ns) || (n > 256 && total_tokens / 64 >= ns));
  const int tile = !runs ? 8 : total_tokens / 28 < ns ? 16 : 32;
  return append_groups(tile, total_tokens, hkv) <= kAppendMaxGroups ? tile : 32;
}

}  // namespace hswa
