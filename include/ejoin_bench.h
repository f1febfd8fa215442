/*
 * ejoin_bench -- measurement hooks of libejoin.so, kept apart from the product interface (ejoin.h):
 * only benchmark programs call these.
 */
#ifndef EJOIN_BENCH_H
#define EJOIN_BENCH_H

#include "ejoin.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Kernel timing.  With profiling on, each join call records HIP events on the call's stream around its
 * preparation kernels (norms and re-layout, FP16 split of the norm terms) and around its Gram/epilogue
 * kernel (the roofline of the join is stated for that kernel: Step 2 of Section 3.1 is where the time
 * goes).  ejoin_last_kernel_ms waits for those events and returns the two durations in milliseconds
 * (host pointers, either may be NULL).  EJOIN_EINVAL if no call has been timed since profiling was set. */
int ejoin_set_profiling(ejoin_ctx* ctx, int on);
int ejoin_last_kernel_ms(ejoin_ctx* ctx, float* prep_ms, float* join_ms);

/* What the join kernel of a call executes: *tiles output tiles of *edge x *edge points (256; 128 or 64 for small problems), of a pair list of
 * rows (counts of a few thousand points may have the other of the two; for prepared sets see ejoin_join_kernel), *steps
 * matrix-core steps of 32 coordinates each, i.e. 2 * edge * edge * 32 * steps FLOP per tile (without the one step per tile that adds
 * the norms).  np points with themselves (nq = 0) or with nq query points; split != 0: the split-FP16 join of np FP32 rows.
 * (EJOIN_KERNEL_STRIP works in pieces of 512 x 64 points; they are counted as tiles of 256 all the same, which for 10^5 points with
 * themselves is 0.2 % less than it executes, for 10^6 the same.)
 * (ejoin_selfjoin_pairs_to_host takes tiles of 256 where it cuts the join into several launches.)  Host pointers; no device work. */
int ejoin_join_work(const ejoin_ctx* ctx, int64_t np, int64_t nq, int32_t d, int32_t split, int32_t* edge, int32_t* steps, int64_t* tiles);

/* Which kernel a call goes to, for a list (count = 0) or counts, of rows (split = 0), the split-FP16 join (1) or a prepared set of np points with nq query
 * points (2): the one of small problems, the general one in tiles of 256, the one that keeps 512 rows of few coordinates in registers, the join of rows in one launch, or
 * the one that holds the few query points of a prepared set in the LDS. */
#define EJOIN_KERNEL_SMALL 0
#define EJOIN_KERNEL_TILES 1
#define EJOIN_KERNEL_STRIP 2
#define EJOIN_KERNEL_ONCE 3
#define EJOIN_KERNEL_FEW 4
int ejoin_join_kernel(const ejoin_ctx* ctx, int64_t np, int64_t nq, int32_t d, int32_t split, int32_t count, int32_t* kernel);

#ifdef __cplusplus
}
#endif
#endif /* EJOIN_BENCH_H */
