// Host build of the rules that choose a call's kernel, for the CPU tests.  Compiled by tests/test_rules.py with g++ (no GPU code involved).
#include <stdint.h>
#include "rules.h"

extern "C" {

int32_t ejoin_test_norms_from_the_end(int64_t n, int64_t ld) { return norms_from_the_end(n, ld); }
}
