// Static tile schedule of the join kernel (host- and device-compilable: the CPU tests enumerate it).
#ifndef EJOIN_TILE_CURSOR_H
#define EJOIN_TILE_CURSOR_H

#include <math.h>
#include <stdint.h>

#if defined(__HIPCC__)
#define EJ_HD __host__ __device__
#else
#define EJ_HD
#endif
#if defined(__HIP_DEVICE_COMPILE__)
// every lane computes the same value; say so to the compiler (the values feed scalar operands)
#define EJ_UNIFORM(x) __builtin_amdgcn_readfirstlane(x)
#else
#define EJ_UNIFORM(x) (x)
#endif

constexpr uint32_t EJ_NUM_XCD = 8;  // accelerator complex dies of the MI355X, each with its own L2
constexpr int EJ_TILE = 256;        // edge of a tile
constexpr uint32_t EJ_SB = 16;      // rows of tiles by which a launch can be cut (one super-block row = two bands)
constexpr uint32_t EJ_BAND = 8;     // rows of tiles per band

// Work distribution (the counterpart of the paper's work queue that orders block tiles in small
// squares for L2 reuse, Section 3.3.1, re-derived for 8 XCDs with private 4 MB L2s):
//   * the rows of the tile grid (the upper triangle of the self-join, the whole grid otherwise) are cut into
//     bands of 8; the tiles of a band are numbered column by column, the bands one after the other.  32 consecutive
//     tiles are then 4 columns x 8 rows (5 where they start inside a column): 12 row and column panels;
//   * workgroup w runs on XCD w % 8 (hardware round-robin, verified on device).  In each pass of the 256 CUs
//     XCD x computes the x-th 32 of the next 256 tiles, one each.  So the 32 workgroups of an XCD share 12
//     panels through its own L2, all XCDs share the 8 row panels, and -- as long as the grid is a multiple of 64
//     workgroups -- a workgroup keeps its row panel to the end of the band;
//   * every workgroup computes the same number of tiles (+-1), whatever the shape of the grid.  That keeps the
//     workgroups of an XCD in step without any synchronisation or queue, which is what makes the panels they share
//     hit in L2: a schedule that lets workgroups skip empty tiles individually drifts apart by many tiles and the
//     L2 hit rate collapses (measured: 16 % instead of ~75 %).
// Before, each XCD owned the 8 x 4 rectangle of every 16 x 16 super-block whose position rotated with the block's number:
// the same 12 panels, but the partly empty rectangles of the diagonal and the edge were dealt out unevenly.  Largest number
// of tiles of a workgroup, with the ideal: 30,011 x 7,001 points 16 (12.9, now 13), 20,011 points 14 (12.3, now 13).
struct TileCursor {
  uint32_t xcd, wpx;     // this workgroup's XCD; workgroups per XCD
  uint32_t self, ntA, ntB;
  uint32_t stride;       // tiles per pass of all workgroups
  uint32_t band, band_end;
  uint32_t rem;          // position of this workgroup's next tile, counted from the first tile of the current band
  uint32_t fast_end;     // steps of the common kind may be taken while rem is below this (see next)
  uint32_t row, col;     // the tile handed out last
#ifdef EJOIN_ABL_ROWMAJOR_TILES
  uint32_t started;
#endif
  // self_join: upper triangle of an nt x nt grid (nt_a == nt_b); otherwise the whole nt_a x nt_b grid.
  // sb_row_begin .. sb_row_end - 1: the rows of super-blocks this launch covers (a join may be cut into several
  // launches by rows of super-blocks; 0 .. UINT32_MAX = everything)
  EJ_HD void init(uint32_t block, uint32_t nblocks, uint32_t self_join, uint32_t nt_a, uint32_t nt_b, uint32_t sb_row_begin = 0,
                  uint32_t sb_row_end = 0xFFFFFFFFu) {
    xcd = block % EJ_NUM_XCD;
    wpx = (nblocks - xcd + EJ_NUM_XCD - 1) / EJ_NUM_XCD;  // workgroups with this XCD id
    self = self_join;
    ntA = nt_a;
    ntB = nt_b;
    stride = nblocks;
    const uint32_t per_sb = EJ_SB / EJ_BAND, bands = (nt_a + EJ_BAND - 1) / EJ_BAND;
    band = sb_row_begin * per_sb;
    band_end = sb_row_end < (nt_a + EJ_SB - 1) / EJ_SB ? sb_row_end * per_sb : bands;
    const uint32_t per = nblocks / EJ_NUM_XCD, more = nblocks % EJ_NUM_XCD;  // the first `more` XCDs have one workgroup more
    rem = xcd * per + (xcd < more ? xcd : more) + block / EJ_NUM_XCD;
    fast_end = 0;
    row = col = 0;
#ifdef EJOIN_ABL_ROWMAJOR_TILES
    started = 0;
    rem = block;
#endif
  }
  // next tile of this workgroup; false when the work is exhausted
  EJ_HD bool next(uint32_t& I, uint32_t& J) {
#ifdef EJOIN_ABL_ROWMAJOR_TILES
    // tiles of the triangle (or grid) in row-major order, tile t to workgroup t % nblocks
    if (!started) {
      started = 1;
      row = 0;
      col = rem;
    } else {
      col += stride;
    }
    while (row < ntA && col >= ntB) {
      col -= ntB;
      ++row;
      if (self) col += row;  // row P of the triangle starts at column P
    }
    if (row >= ntA) return false;
    I = EJ_UNIFORM(row);
    J = EJ_UNIFORM(col);
    return true;
#endif
    // Everything here is uniform over the workgroup and meant to stay on the scalar unit.  All eight wavefronts of a
    // workgroup run it at the same time, between two tiles, with nothing else to overlap it: every instruction is paid
    // eight times on the one scalar unit.  So the common step comes first: inside a band, right of its diagonal block, a
    // grid of a multiple of 8 workgroups goes on in the same row, stride / 8 columns further.
#ifndef EJOIN_CURSOR_NO_FAST_PATH
    if (rem < fast_end) {
      rem += stride;
      col += stride / EJ_BAND;
      I = EJ_UNIFORM(row);
      J = EJ_UNIFORM(col);
      return true;
    }
#endif
    while (band < band_end) {
      const uint32_t first = band * EJ_BAND;  // first row
      const uint32_t h = ntA - first < EJ_BAND ? ntA - first : EJ_BAND;
      // the self-join's band starts with the triangle of its h columns on the diagonal
      const uint32_t tri = self ? h * (h + 1) / 2 : 0u, c0 = self ? first + h : 0u;
      const uint32_t size = tri + h * (ntB - c0);
      if (rem < size) {
        if (rem < tri) {
          uint32_t c = 0, r = rem;
          while (r > c) r -= ++c;  // column c of the triangle has rows 0 .. c
          row = first + r;
          col = first + c;
        } else if (h == EJ_BAND) {
          const uint32_t q = rem - tri;
          row = first + q % EJ_BAND;
          col = c0 + q / EJ_BAND;
        } else {
          const uint32_t q = rem - tri;
          row = first + q % h;
          col = c0 + q / h;
        }
        I = EJ_UNIFORM(row);
        J = EJ_UNIFORM(col);
        fast_end = rem >= tri && h == EJ_BAND && stride % EJ_BAND == 0 ? size : 0u;
        rem += stride;
        return true;
      }
      rem -= size;
      ++band;
    }
    fast_end = 0;
    return false;
  }
};

// The one tile of a workgroup of k_join_once: first the tiles on the diagonal (two sets: of the first column, then of the first row),
// whose workgroups others wait for, then the rest, column by column (row by row).
EJ_HD inline void once_tile(uint32_t block, uint32_t self_join, uint32_t nt_a, uint32_t nt_b, uint32_t& I, uint32_t& J) {
  if (block < nt_a) {
    I = block;
    J = self_join ? block : 0;
    return;
  }
  uint32_t r = block - nt_a;
  if (self_join) {
    J = 1;
    while (r >= J) r -= J++;  // column J has rows 0 .. J - 1 above the diagonal
    I = r;
  } else if (r < nt_b - 1) {
    I = 0;
    J = r + 1;
  } else {
    r -= nt_b - 1;
    I = 1 + r / (nt_b - 1);
    J = 1 + r % (nt_b - 1);
  }
}

// Work distribution of k_join_strip, whose workgroups hold a panel of 512 rows in registers and stream columns past it, 64 at a
// time (a stage): what counts is that a workgroup changes its rows as seldom as possible, that the workgroups of an XCD stream the
// same columns at the same time (through its L2), and that all have the same number of stages.
//   * The panels are cut into bands of 32 (the rest into bands of 16, 8, 4, 2, 1).  A band is worked on along 32 lines: line w has
//     panel w and goes through its columns from left to right (a band of h panels: 32 / h lines a panel, a part of its columns each).
//   * XCD x works on the x-th eighth of all bands' lengths, its workgroup y on line y.
//   * A self-join's band starts with the triangle on the diagonal, folded so that every line has (h + 1) / 2 of its squares of 512 x
//     512: a line of the upper half gives the end of its row of the triangle to line h - 1 - w, which has that much less of its own.
// So there are runs of consecutive stages in one panel, two for a band.
constexpr uint32_t EJ_STRIP_ROWS = 512, EJ_STRIP_COLS = 64, EJ_STRIP_LINES = 32;
struct StripCursor {
  uint32_t self, stages, row_end;  // stages in a row (columns / 64); panels this launch covers
  uint32_t line, step;             // this workgroup's line, workgroups of the XCD
  uint32_t start_row, start_at, last_row, last_at;  // the XCD's part: from position start_at of the band that starts at start_row ...
  uint32_t first, h_log2, reach, len;  // the current band: its first panel, log2 of its panels, stages of a panel, positions of a line
  uint32_t at, piece;              // this line's position in it, and which of its two runs comes next

  EJ_HD __attribute__((always_inline)) void enter(uint32_t f) {
    first = f;
    h_log2 = 0;
    while ((2u << h_log2) <= EJ_STRIP_LINES && (2u << h_log2) <= row_end - f) ++h_log2;
    const uint32_t h = 1u << h_log2, per = EJ_STRIP_ROWS / EJ_STRIP_COLS, diag_end = per * (f + h);
    reach = self ? per / 2 * (h + 1) + (stages > diag_end ? stages - diag_end : 0u) : stages;
    const uint32_t share = EJ_STRIP_LINES >> h_log2;  // lines of a panel
    len = (reach + share - 1) / share;
  }
  // panels_begin .. panels_end - 1: the panels of rows of this launch
  EJ_HD void init(uint32_t block, uint32_t nblocks, uint32_t self_join, uint32_t n_stages, uint32_t panels_begin, uint32_t panels_end) {
    self = self_join;
    stages = n_stages;
    row_end = panels_end;
    const uint32_t xcds = nblocks < EJ_NUM_XCD ? nblocks : EJ_NUM_XCD, xcd = block % xcds;
    step = (nblocks - xcd + xcds - 1) / xcds;
    line = block / xcds;
    uint64_t total = 0;
    for (uint32_t f = panels_begin; f < row_end; f += 1u << h_log2) {
      enter(f);
      total += len;
    }
    uint64_t from = total * xcd / xcds, to = total * (xcd + 1) / xcds;
    start_row = last_row = row_end;
    start_at = last_at = 0;
    first = row_end;
    at = piece = 0;
    if (from == to || line >= EJ_STRIP_LINES) {
      line = EJ_STRIP_LINES;
      return;
    }
    uint32_t f = panels_begin;
    for (enter(f); from >= len; enter(f)) {
      from -= len;
      to -= len;
      f += 1u << h_log2;
    }
    start_row = f;
    start_at = (uint32_t)from;
    for (; to > len; enter(f)) {
      to -= len;
      f += 1u << h_log2;
    }
    last_row = f;
    last_at = (uint32_t)to;
    enter(start_row);
    at = start_at;
  }
  // the next run: stages c .. c_end - 1 of panel I; false when the work is exhausted
  EJ_HD __attribute__((always_inline)) bool next(uint32_t& I, uint32_t& c, uint32_t& c_end) {
    while (line < EJ_STRIP_LINES) {
      const uint32_t h = 1u << h_log2, w = line & (h - 1), offset = (line >> h_log2) * len;
      const uint32_t per = EJ_STRIP_ROWS / EJ_STRIP_COLS;
      // positions of this line in the band that belong to the XCD's part, as stages of the panel
      const uint32_t lo = offset + at;
      uint32_t hi = offset + (first == last_row ? last_at : len);
      if (hi > reach) hi = reach;
      // its runs: [0, turn) of panel r0 from column c0 on, [turn, reach) of panel w from column c1 on
      uint32_t turn = 0, r0 = w, c0 = 0, c1 = 0;
      if (self) {
        if (w < h / 2) {
          turn = per / 2 * (h + 1);
          c0 = per * (first + w);
          c1 = per * (first + h);
        } else {
          turn = per * w + per / 2 - per / 2 * h;
          r0 = h - 1 - w;
          c0 = per * (first + r0) + per / 2 * (h + 1);
          c1 = per * (first + w);
        }
      }
      while (piece < 2) {
        const uint32_t a = piece ? (lo > turn ? lo : turn) : lo, b = piece ? hi : (hi < turn ? hi : turn);
        const uint32_t row = first + (piece ? w : r0);
        c = piece ? c1 + (a - turn) : c0 + a;
        c_end = piece ? c1 + (b - turn) : c0 + b;
        const bool some = a < b;
        ++piece;
        if (c_end > stages) c_end = stages;
        if (some && c < c_end) {
          I = EJ_UNIFORM(row);
          c = EJ_UNIFORM(c);
          c_end = EJ_UNIFORM(c_end);
          return true;
        }
      }
      piece = 0;
      at = 0;
      if (first != last_row) {
        enter(first + h);
      } else {  // (a grid of fewer workgroups than lines: the next of this one's lines)
        line += step;
        enter(start_row);
        at = start_at;
      }
    }
    return false;
  }
};

// Which joins k_join_strip takes, and with which set in its rows (`swapped`: the second of two).
//
// At eleven k-blocks 12 (pairs) and 21 (counts) of its registers are spilled, and what is read back at every stage waits for the copies
// just issued: d = 350, S = 16, 50,000 points 676 us of counts and 662 of pairs against 650 and 653 by k_join, 100,000 points 2.47 and
// 2.43 ms against 2.49 and 2.49; 30,000 x 7,000 130 us of counts against 123.
//
// Two sets: the way round that has fewer stages, where a panel of rows, which is read before its first stage starts, counts four
// (300,000 points x 300 queries, d = 128: 45 us with the queries in the rows, 47 with the points; x 700 71 and 65; 100,000 x 2,000
// 56 and 61).  More than two bands of panels are read anew by every XCD (the term of the cost: 50,000 x 600 lists, d = 200, 26 us by k_join,
// 29 here).  None of it depends on which set is the first (so long as the second's panels counted nothing, 700 x 100,000 counts,
// d = 320, took 82 us here, and 100,000 x 700 52 by k_join), but for counts, where hits in rows are added up in the LDS and hits in
// columns are mostly one atomic each, those on one address served one after the other.  The points of a small set have the more hits
// the more queries there are: they go into the rows where the queries are sixteen times as many (1,000 x 200,000, d = 60, four hits a
// query: 74 us, 177 the other way round; 700 x 300,000, d = 128, two hits a query: 231 with the queries in the rows, 188 by k_join).  Else, up
// to two bands, the queries do (3,000 x 20,000, d = 128, S = 32: 44 us, 62 the other way round); and columns of
// at most two panels are met by rows of at least 1.5 panels a CU only (600 .. 700 columns, d = 128, S = 16 and 64: 90,000 points 32 and
// 38 us by k_join, 32 and 44 here; 150,000 44 and 49, 42 and 50; 200,000 57 and 61, 51 and 58; 1,200 columns of 150,000: 64 and 70, 55 and 65).
// k_join computes a tile, twice a stage's pairs, in 2 `gain` times the time of a stage (150,000 points, d = 64, 128, 224,
// 320: 2.14, 2.85, 4.02, 5.33 ms against 1.93, 2.48, 3.60, 5.08), but needs no rows in place before it starts: where a workgroup has
// few stages it is the better one (18,000 points, d = 128 / 224 / 320: 189 / 203 / 223 us against 187 / 206 / 235; 26,000:
// 266 / 300 / 339 against 253 / 293 / 342; 100,000 x 700 points, d = 320: 54 against 62).  Counts of a set with itself, eight and nine
// k-blocks: the gain is less, the filter of blocks full of candidates being in the open (d = 256, S = 16, 64 and 300: 65,000 points 0.81,
// 0.90 and 1.19 ms by k_join, 0.81, 0.95 and 1.29 here; 100,000 1.88, 2.02 and 2.52, 1.81, 2.02 and 2.62; 200,000 7.37, 7.81 and 9.14,
// 7.01, 7.47 and 8.82).
constexpr int EJ_STRIP_KB_MAX = 10;
struct StripPlan {
  bool use, swapped;
};
inline int64_t strip_panels(int64_t n) { return (n + EJ_STRIP_ROWS - 1) / EJ_STRIP_ROWS; }
inline int64_t strip_stages(int64_t n) { return (n + EJ_STRIP_COLS - 1) / EJ_STRIP_COLS; }
inline StripPlan strip_plan(int num_cu, int64_t nA, int64_t nB, bool self, int nkb, bool count) {
  constexpr int64_t MANY = 2 * EJ_STRIP_LINES;
  const double cu = num_cu;
  const int64_t a = strip_panels(nA), b = strip_panels(nB), plain = a * strip_stages(nB), turned = b * strip_stages(nA);
  const int64_t rows_a = plain + 4 * a, rows_b = turned + 4 * b;
  StripPlan p{false, !self && (rows_b < rows_a || (rows_b == rows_a && b < a))};
  if (!self && count) p.swapped = nB < 16 * nA && (b <= MANY ? turned : rows_b) <= rows_a;
  if (nkb > EJ_STRIP_KB_MAX) return p;
  const double rows = p.swapped ? b : a, columns = p.swapped ? a : b;
  const double load = nkb <= 4 ? 1. : (nkb <= 7 ? 1.5 : 2.);
  double gain = nkb <= 2 ? 1.07 : (nkb <= 4 ? 1.13 : (nkb <= 7 ? 1.11 : 1.05));
  if (self && count && (nkb == 8 || nkb == 9)) gain -= 0.06 * fmin(1., 1e5 / (double)nA);
  const double cost = self ? ceil((double)a * (a + 1) * (EJ_STRIP_ROWS / EJ_STRIP_COLS / 2) / cu) + 1.5 * load
                           : ceil((p.swapped ? turned : plain) / cu) + load * (rows <= MANY ? 0.6 : 1.6 + 0.7 * rows / cu);
  const int64_t ta = (nA + EJ_TILE - 1) / EJ_TILE, tb = (nB + EJ_TILE - 1) / EJ_TILE;
  const double rounds = ceil((self ? (double)ta * (ta + 1) / 2 : (double)ta * tb) / cu);
  const bool contended = !self && count && columns <= 2 && rows > MANY && rows < 1.5 * cu;
  p.use = cost < 2 * gain * rounds && !contended;
  return p;
}

#endif  // EJOIN_TILE_CURSOR_H
