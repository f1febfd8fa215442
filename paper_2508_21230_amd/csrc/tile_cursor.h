// Static tile schedule of the join kernel (host- and device-compilable: the CPU tests enumerate it).
#ifndef EJOIN_TILE_CURSOR_H
#define EJOIN_TILE_CURSOR_H

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

#endif  // EJOIN_TILE_CURSOR_H
