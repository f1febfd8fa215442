// Host build of the join kernel's tile schedule for the CPU tests: enumerates, for every workgroup, the
// tiles it would compute, in order.  Compiled by tests/test_schedule.py with g++ (no GPU code involved).
#include <stdint.h>
#include "tile_cursor.h"

extern "C" {

// Writes up to `cap` (block, step, I, J) quadruples; returns the number of tiles of the whole schedule.
// sb_row_begin .. sb_row_end - 1: rows of super-blocks covered (0 .. UINT32_MAX = all).
int64_t ejoin_test_schedule_rows(uint32_t nblocks, uint32_t self_join, uint32_t nt_a, uint32_t nt_b, uint32_t sb_row_begin,
                                 uint32_t sb_row_end, uint32_t* out, int64_t cap) {
  int64_t m = 0;
  for (uint32_t b = 0; b < nblocks; ++b) {
    TileCursor tc;
    tc.init(b, nblocks, self_join, nt_a, nt_b, sb_row_begin, sb_row_end);
    uint32_t I = 0, J = 0, step = 0;
    while (tc.next(I, J)) {
      if (m < cap) {
        out[4 * m] = b;
        out[4 * m + 1] = step;
        out[4 * m + 2] = I;
        out[4 * m + 3] = J;
      }
      ++m;
      ++step;
    }
  }
  return m;
}

int64_t ejoin_test_schedule(uint32_t nblocks, uint32_t self_join, uint32_t nt_a, uint32_t nt_b, uint32_t* out, int64_t cap) {
  return ejoin_test_schedule_rows(nblocks, self_join, nt_a, nt_b, 0, 0xFFFFFFFFu, out, cap);
}

// The same of the schedule in panels of 512 rows and stages of 64 columns: (block, panel, first stage, end) per run.
int64_t ejoin_test_strips(uint32_t nblocks, uint32_t self_join, uint32_t stages, uint32_t panels_begin, uint32_t panels_end, uint32_t* out,
                          int64_t cap) {
  int64_t m = 0;
  for (uint32_t b = 0; b < nblocks; ++b) {
    StripCursor tc;
    tc.init(b, nblocks, self_join, stages, panels_begin, panels_end);
    uint32_t I = 0, c = 0, c_end = 0;
    while (tc.next(I, c, c_end)) {
      if (m < cap) {
        out[4 * m] = b;
        out[4 * m + 1] = I;
        out[4 * m + 2] = c;
        out[4 * m + 3] = c_end;
      }
      ++m;
    }
  }
  return m;
}

// The tiles of the one-launch join, two numbers each.
void ejoin_test_once(uint32_t blocks, uint32_t self_join, uint32_t nt_a, uint32_t nt_b, uint32_t* out) {
  for (uint32_t b = 0; b < blocks; ++b) once_tile(b, self_join, nt_a, nt_b, out[2 * b], out[2 * b + 1]);
}

// Which joins go to the kernel of few coordinates: 0, or 1, or 3: with the second of the two sets in its rows.
int32_t ejoin_test_strip_plan(int32_t num_cu, int64_t n_a, int64_t n_b, int32_t self_join, int32_t nkb, int32_t count) {
  const StripPlan p = strip_plan(num_cu, n_a, n_b, self_join != 0, nkb, count != 0);
  return p.use ? 1 + 2 * p.swapped : 0;
}
}
