// host_limits.h -- pure host-side size rules of libsieve (no HIP), so that a
// plain C++ compiler can check them without a GPU.
#pragma once

#include <math.h>
#include <stdint.h>
#include <stdlib.h>

#include <algorithm>

namespace sieve {

// The final merge groups the candidate pool by query with 64-bit per-query
// offsets (exclusive scan of the counts, scatter cursors, segment starts), so
// the limit on candidate slots is a sanity bound, 2^38, far more than device
// memory holds (the pool's allocation fails first).  knob: the value of an
// override (tests lower the limit to reach the error path without filling
// memory); null, empty or non-positive means no override.
inline int64_t pool_index_limit(const char* knob) {
  const int64_t hard = (int64_t)1 << 38;
  if (!knob || !*knob) return hard;
  const long long v = atoll(knob);
  return v > 0 && v < hard ? (int64_t)v : hard;
}

// Whether a search whose scans claimed `slots` pool slots can be merged.
inline bool pool_slots_fit(uint64_t slots, int64_t limit) {
  return limit >= 0 && slots <= (uint64_t)limit;
}

// Most tiles of a round: n_items items in groups of `group` per list, lists in
// chunks of `chunk` rows, sum_p ceil(c_p / group) ceil(len_p / chunk).
inline int64_t round_tile_bound(int64_t n_items, int64_t group, int64_t chunk, int64_t nlist,
                                int64_t n, int64_t max_list) {
  const int64_t max_ch = std::max<int64_t>((max_list + chunk - 1) / chunk, 1);
  const int64_t once = std::min(nlist + n / chunk, std::min(n_items, nlist) * max_ch);
  return n_items / group * max_ch + once;
}

// Rows per tile of a screened round.  `chunk` suits rounds that fill the chip;
// lists that make few tiles of it are split (by the average length) into twice
// as many equal parts, down to 128 rows, as long as nine tenths of the grid's
// work-groups hold the tiles: a second tile per work-group costs more than the
// shorter ones save (80 lists of 2,229 rows, fp32 128, loose threshold: 24 us
// in 160 tiles, 31 in 640).  25 lists of 2,145 rows at 768 dimensions, 124
// queries: 185 us in whole lists, 45 in 200 tiles; 20 of 1,517 at 96: 63 -> 26.
// A split is taken only where its tiles fit tile_cap for any lists.
inline int screen_rows_per_tile(int chunk, int64_t grid, int64_t n_items, int64_t group,
                                int64_t nlist, int64_t n, int64_t max_list, int64_t tile_cap) {
  const double per = (double)n_items / (double)std::max<int64_t>(nlist, 1);
  const double lists = std::max((double)nlist * (1.0 - exp(-per)), 1.0);  // that have items
  const int64_t groups = (int64_t)(lists * ceil((double)n_items / (lists * (double)group)));
  const int64_t avg = std::max<int64_t>(n / std::max<int64_t>(nlist, 1), 1);
  int64_t parts = (avg + chunk - 1) / chunk;
  while (groups * 2 * parts <= grid * 9 / 10 && avg / (2 * parts) >= 128) {
    parts *= 2;
    const int64_t rows = ((avg + parts - 1) / parts + 63) / 64 * 64;
    if (rows >= chunk) continue;  // the first split of lists just past a chunk
    if (round_tile_bound(n_items, group, rows, nlist, n, max_list) > tile_cap) break;
    chunk = (int)rows;
  }
  return chunk;
}

}  // namespace sieve
