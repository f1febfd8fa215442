// Which kernel, and in which form, a call goes to: rules on sizes and alignment alone (host-compilable: the CPU tests look at them).
#ifndef EJOIN_RULES_H
#define EJOIN_RULES_H

#include <stdint.h>
#include "tile_cursor.h"

constexpr int64_t EJ_MEMORY_SIDE_CACHE = 256ll << 20;  // bytes of it

// Norms alone, from the last point on: where the rows have just been written, more of them than the memory-side cache holds, the last ones are
// still in it.  Rows of which all are there are read in the order in which they were written: the XCD that wrote a row still has it in its L2.
// Converted and normed, first to last and last to first, us: d = 16, rows of 100 MB 37.9 and 41.2, 128 46.8 and 50.0, 230 89.7 and 94.2, 250 102.0
// and 101.3, 275 128.1 and 116.2, 350 166.4 and 157.4, 500 230.3 and 229.5; d = 48, 128 MB 71.8 and 71.8, 250 132.7 and 132.2, 350 220.5 and
// 196.3, 500 310.3 and 295.5; d = 128, 650 MB 456 and 453, 950 MB 664 and 663; d = 16, 800 MB 357 and 360.  (A little of the cache is others'.)
inline bool norms_from_the_end(int64_t n, int64_t ld) {
  const int64_t bytes = n * ld * 2;
  return bytes > EJ_MEMORY_SIDE_CACHE / 16 * 15 && bytes <= EJ_MEMORY_SIDE_CACHE * 3;
}

// Ingestion: threads side by side on a row of `chunks` (a power of two that divides them, 8 to 64).
inline uint32_t ingest_wide(int64_t chunks) {
  const int64_t two = chunks & -chunks;
  return (uint32_t)(two < 64 ? two : 64);
}
// Ingestion with four columns a thread.  Input that the memory-side cache cannot hold only; at few coordinates most of a row of the result is padding, and
// eight columns are the better ones.  (A grid has fewer than 2^32 threads.)
inline bool ingest_large(int64_t n, int32_t d, int64_t ld16) {
  return n * d * 4 > EJ_MEMORY_SIDE_CACHE && d > 32 && n * (ld16 / 8) < (1ll << 32);
}
// ... and past the caches: rows that are 16-byte aligned, where a line is rarely read twice.  A row is read in pieces of 16 * ingest_wide bytes by wavefronts that know
// nothing of each other; where there are several and the rows do not begin at lines, the pieces share their first and last ones, and past the caches a shared line
// is fetched twice.  Converted, and converted and normed, past the caches over eight columns through them:
// one piece a row (d = 48, 100, 200), 400 MB 0.87, 0.82, 0.86 and 0.86, 0.84, 0.84; 1,700 MB 0.91, 0.89, 0.93 and 0.98, 0.97, 1.00;
// whole lines (d = 192, 640, 960), 400 MB 0.86, 0.90, 0.88 and 0.83, 0.85, 0.84; 700 MB 0.98, 1.03, 0.99 and 0.94, 1.00, 0.99; 1,000 MB 0.98, 1.03, 1.00 and 0.98, 1.02, 1.01; 1,700 MB 0.99, 1.06,
// 1.02 and 1.01, 1.06, 1.03, d = 768 1.02 and 1.04; rows of a power of two (d = 512, 1,024, 2,048) 1,700 MB 0.97, 0.94, 0.92 and 1.01, 0.96, 0.99;
// shared lines, pieces of 256 bytes (d = 132, 300, 784), 330 MB 1.07, 1.07, 1.02 and 0.91, 0.95, 0.94; 520 MB 1.30, 1.15, 1.08 and 1.16, 1.08, 1.04; 700 MB 1.33, 1.27, 1.21 and 1.18, 1.17, 1.14; of 512
// (d = 324, 600), 460 MB 0.98, 0.97 and 0.97, 0.93; 520 MB 1.07, 1.03 and 1.01, 1.01; 700 MB 1.13, 1.16 and 1.07, 1.10; of 1 KB (d = 980, 1,000, 2,000), 550 MB 0.96, 0.96, 0.98 and 0.96, 0.96, 0.91;
// 600 MB 1.00, 1.01, 1.02 and 0.98, 0.98, 0.96.
inline bool ingest_past_the_caches(int64_t n, int32_t d, int64_t ld32, uint64_t address, int64_t ld16) {
  if (!ingest_large(n, d, ld16) || ld32 % 4 != 0 || address % 16 != 0) return false;
  const int64_t chunks = ld16 / 4;
  const uint32_t wide = ingest_wide(chunks);
  if (chunks == wide) return true;
  const bool whole_lines = ld32 % 32 == 0 && address % 128 == 0;
  if (whole_lines && (chunks & (chunks - 1)) == 0) return true;
  const int64_t eighths = whole_lines ? 24 : wide == 64 ? 18 : wide == 32 ? 15 : 0;  // of the cache
  return n * d * 4 <= EJ_MEMORY_SIDE_CACHE / 8 * eighths;
}

// Tiles of edge x edge points of a self-join of a points, or of a and b points.
inline int64_t tiles_of(int64_t edge, int64_t a, int64_t b, bool self) {
  const int64_t ta = (a + edge - 1) / edge, tb = (b + edge - 1) / edge;
  return self ? ta * (ta + 1) / 2 : ta * tb;
}

// Which tile k_join_once works a join of FP16 rows in, or 0: another kernel, its tiles do not all fit the CUs at once (three workgroups a CU).
// Counts: tiles of 64 while they do (1,984 points, d = 64, 384 and 960: 8.3, 10.1 and 14.0 us, in tiles of 128 9.1, 12.4 and 18.7; 2,400
// points 9.0, 11.4 and 17.5 against 9.3, 12.9 and 20.0; 3,000 x 1,000, d = 128, 10.4 against 10.6).  Lists pay some 13 ns a tile for their place in the result, tiles of 128 1.6 us and 0.19 us a
// k-block for their longer chain (tiles of 64 and of 128: 1,000 x 64 8.0 and 9.2 us; 1,984 points, d = 64, 384 and 960, 12.7, 14.6 and 18.4,
// 9.9, 13.4 and 20.0); with three of them on a CU tiles of 64 lose more (2,400 x 960 23.4 against 21.2).
// Tiles of 128 are copied in half lines and their norms multiplied once a tile: with three of them on a CU and many k-blocks k_prep and k_join_small are the better
// ones (time here over time there).  Counts, 30, 36, 40 and 48 k-blocks: 4,100 points 0.92, 0.97, 0.99, 1.03, 4,400 0.96, 0.97, 1.03, 1.07, 4,800 0.93, 0.96, 1.00, 1.06; of two sets, 24, 26, 30 and 36:
// 8,000 x 1,400 0.99, 1.00, 1.02, 1.03, 4,000 x 3,000 0.92, 0.97, 0.98, 1.02, 2,500 x 4,300 0.97, 1.01, 1.03.  Lists, 12, 16, 20, 24 and 30: 4,100 0.95, 0.94, 0.96, 0.96, 0.97, 4,400 0.98, 0.96, 0.98, 1.00, 1.00,
// 4,300 at 20 and 24 1.02, 1.04, 8,000 x 1,400 0.98, 0.97, 1.00, 1.03, 1.04.  With two up to 128 k-blocks not (3,900 points,
// d = 2,048 and 4,096: 59.8 and 97.7, 52.3 and 95.4; counts of 4,000 x 2,000, d = 4,096, 99 and 98).
constexpr int ONCE_SLOTS = 2048, ONCE_COUNTS = 1 << 17, ONCE_GROUPS_PER_CU = 3;
inline int once_tile_edge(int num_cu, int64_t a, int64_t b, bool self, int nkb, bool count) {
  const int64_t held = (int64_t)num_cu * ONCE_GROUPS_PER_CU, t64 = tiles_of(64, a, b, self), t128 = tiles_of(128, a, b, self);
  if (held >= 4096 || a + (self ? 0 : b) > ONCE_COUNTS || (a + 63) / 64 + (self ? 0 : (b + 63) / 64) > ONCE_SLOTS) return 0;
  if (count ? t64 <= held : t64 <= 2 * num_cu && t64 - t128 <= 123 + 15 * nkb) return 64;
  const int most_kb = count ? (self ? 36 : 24) : 16;
  return t128 <= (nkb <= most_kb ? held : nkb <= 128 ? 2 * num_cu : 0) ? 128 : 0;
}

// The dense block: workgroups in tiles of edge x edge, and whether in tiles of 128 (see k_dist2_tile) or of 64.
inline int64_t dense_groups(int edge, int64_t rows, int64_t cols) { return (tiles_of(edge, rows, cols, false) + EJ_NUM_XCD - 1) / EJ_NUM_XCD * EJ_NUM_XCD; }
inline bool dense_wide(int num_cu, int64_t rows, int64_t cols) { return 4 * dense_groups(128, rows, cols) >= 3 * num_cu; }
// Workgroups for the norms of n points in the launch of the block itself, or 0: a launch of their own.  One launch where there is about one workgroup a CU
// in all (a call among others, two launches and one, in us: 300 x 300 of 8,000 x 64 9.5 and 7.3; 600 x 600 of 8,000 x 384 10.6 and 9.6; 1,000 x 1,000 of 1,000 x 96 10.8 and 7.7).  Beyond, it is the slots that take long to
// read and what waits for them (300 x 300 of 20,000 x 384 11.6 both ways, of 120,000 x 64 11.1 and 21.4; 2,500 x 700 of 12,000 x 200 11.3, 12.3).
inline int64_t dense_norm_groups(int num_cu, int64_t n, int64_t rows, int64_t cols) {
  const bool wide = dense_wide(num_cu, rows, cols);
  const int64_t per = 16 * (wide ? 8 : 4), groups = ((n + per - 1) / per + EJ_NUM_XCD - 1) / EJ_NUM_XCD * EJ_NUM_XCD;
  return groups <= ONCE_SLOTS && 4 * (groups + dense_groups(wide ? 128 : 64, rows, cols)) <= 5 * num_cu ? groups : 0;
}

// A prepared set of n points against few query points: groups of 16 of them that k_join_few is built for (0: too many) ...
inline int few_groups_of(int64_t nq) { return nq <= 32 ? 2 : (nq <= 64 ? 4 : (nq <= 128 ? 8 : (nq <= 256 ? 16 : 0))); }
// ... and whether it is the better kernel, where the LDS holds them.  Every workgroup fills its LDS with them, 1 KB a group and k-block, and has one panel of 256
// points or a few: the more there is to fill, the more points it takes to have the CUs at work.  What it is measured against (time here over time there, sparse results, 4 and
// 14 % of all pairs; counts, lists) is k_prep and k_join_small.  Up to 300 tiles of 64 that works in those, on up to 300 workgroups: 60 queries, 6,000 points,
// d = 256 0.83, 0.82, 0.85; 0.78, 0.90, 1.04; d = 512 1.09, 1.06, 1.07; 1.09, 1.14, 1.24; 13,000 points 1.01, 0.90, 0.91; 1.01, 1.01, 1.11; d = 768, 18,500 points 1.14, 1.05, 1.07;
// 1.14, 1.17, 1.23; 30 queries, d = 512, 6,000 points 0.92, 0.91, 0.91; 0.93, 0.94, 0.96; d = 1,024, 13,000 1.17, 1.13, 1.13; 1.17, 1.15, 1.17; 120 queries, 6,000 points, d = 128
// 0.78, 0.89, 0.95; 0.78, 1.01, 1.37; d = 256 1.03, 1.04, 1.10; 1.01, 1.22, 1.46.  From there on in tiles of 128, and up to 128 queries it is the slower one: 60, 19,500 points,
// d = 768 0.91, 0.84, 0.84; 0.89, 0.83, 0.79; 120, 13,000 points, d = 480 0.97, 0.92, 0.93; 0.98, 0.98, 0.95; 30, 19,500 points, d = 2,100 0.80, 0.79, 0.79; 0.79, 0.78, 0.77.
// More than 128 queries it has in two columns of tiles and their registers leave k_join_few one workgroup a CU.  250 queries, counts: d = 64, 3,000 points 0.83, 1.08, 1.22; d = 128, 13,000 0.99,
// 0.96, 1.04; 16 neighbours a query, d = 180, 16,000 and 20,000 0.98, 0.92; d = 220, 16,000, 20,000 and 24,000 1.10, 1.02, 0.96; d = 250, 24,000, 33,000 and 38,000 1.08, 1.03, 0.90; lists, which every wavefront sorts out
// by itself: d = 64, 13,000 0.80, 1.16, 0.86; 24,000 0.75, 1.01, 0.57; d = 128 0.90, 1.13, 0.59; 4 %, 30,000 and 40,000 1.09, 0.94; d = 256 1.21, 1.06.
inline bool few_pays(int64_t n, int64_t nq, int groups, int nkb, bool count) {
  const int kb = groups * nkb;
  if (groups == 16) return n >= (count ? 9ll * kb * kb / 5 : 14000 + 300ll * kb);
  const bool other_in_64 = tiles_of(64, n, nq, false) <= 300;
  return !other_in_64 || n >= (groups == 4 ? 300ll : 600ll) * (kb - 32);
}

#endif  // EJOIN_RULES_H
