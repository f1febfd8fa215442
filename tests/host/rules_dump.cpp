// Host build of the rules that choose a call's kernel, for the CPU tests.  Compiled by tests/test_rules.py with g++ (no GPU code involved).
#include <stdint.h>
#include "rules.h"

extern "C" {

int32_t ejoin_test_norms_from_the_end(int64_t n, int64_t ld) { return norms_from_the_end(n, ld); }
uint32_t ejoin_test_ingest_wide(int64_t chunks) { return ingest_wide(chunks); }
int32_t ejoin_test_ingest_past_the_caches(int64_t n, int32_t d, int64_t ld32, uint64_t address) { return ingest_past_the_caches(n, d, ld32, address, (d + 63) / 64 * 64); }
// (d: one k-block for every 32 coordinates)
int32_t ejoin_test_few_pays(int64_t n, int64_t nq, int32_t d, int32_t count) { return few_pays(n, nq, few_groups_of(nq), (d + 31) / 32, count != 0); }
int32_t ejoin_test_once_edge(int64_t a, int64_t b, int32_t d, int32_t count) { return once_tile_edge(256, a, b ? b : a, b == 0, (d + 31) / 32, count != 0); }
int64_t ejoin_test_dense_norm_groups(int64_t n, int64_t rows, int64_t cols) { return dense_norm_groups(256, n, rows, cols); }
int32_t ejoin_test_few_groups_of(int64_t nq) { return few_groups_of(nq); }
}
