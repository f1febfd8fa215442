// Brute-force Euclidean-distance epsilon self-join for gfx950 (MI355X): kernels and C ABI.
//
// Method (arXiv 2508.21230, Section 3.1): Step 1 norms s_i, Step 2 Gram products a_ij on the
// matrix cores with FP16 inputs / FP32 accumulation, Step 3 dist^2 = s_i + s_j - 2 a_ij, then
// the "<= epsilon" filter of Section 2.2.1.  The tiling below is designed for CDNA4 (64-wide
// wavefronts, v_mfma_f32_16x16x32_f16, 160 KB LDS with 64 banks, 8 XCDs with private L2s); the
// paper's A100 tiling (Section 3.2-3.3) is prior art, not the blueprint.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>
#include <math.h>
#include <new>
#include <type_traits>
#include <utility>

#include "ejoin.h"
#include "ejoin_bench.h"
#include "panel_layout.h"
#include "rules.h"
#include "tile_cursor.h"

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef float float4v __attribute__((ext_vector_type(4)));

#define EJ_LDS(p) ((__attribute__((address_space(3))) void*)(p))
#define EJ_GLB(p) ((const __attribute__((address_space(1))) void*)(p))

// ------------------------------------------------------------------------------------------
// Tiling constants
// ------------------------------------------------------------------------------------------
constexpr int TILE = EJ_TILE;  // a workgroup computes a TILE x TILE block of the distance matrix
constexpr int KPAD = 64;      // rows are padded with zeros to a multiple of KPAD coordinates (by the caller)
constexpr int KSLICE = 32;    // coordinates per LDS stage (64 B per row)
// Ablation builds (bench_ablation.py) take one design element out at a time; every variant computes the
// same results.  EJOIN_ABL_NSTAGE=3 (one LDS stage less), EJOIN_ABL_NOSWIZZLE (plain LDS rows),
// EJOIN_ABL_ROWMAJOR_TILES (tiles dealt round-robin in row-major order), EJOIN_ABL_NOALIGN (workgroups of
// an XCD never re-aligned), EJOIN_ABL_NOPREFILTER (every block goes through the exact path).
#if defined(EJOIN_ABL_NSTAGE) || defined(EJOIN_ABL_NOSWIZZLE) || defined(EJOIN_ABL_ROWMAJOR_TILES) || defined(EJOIN_ABL_NOALIGN) || \
    defined(EJOIN_ABL_NOPREFILTER) || defined(EJOIN_EXP_HOT_PANELS) || defined(EJOIN_EXP_NO_COPIES) || defined(EJOIN_EXP_CYCLE_MARKS)
#define EJOIN_ONLY_K_JOIN  // these builds are about k_join: problems of every size go to it (as in the tests' build of that kernel)
#endif
#ifndef EJOIN_ABL_NSTAGE
#define EJOIN_ABL_NSTAGE 4
#endif
// Three measurement builds whose RESULTS ARE MEANINGLESS (timing only, never loaded by the product path or the tests):
// EJOIN_EXP_HOT_PANELS: every global->LDS copy reads one of four panels, so that every copy hits in the L2 while
//   tiles, MFMAs, LDS traffic and operand values stay what they are -- what the memory-side fetch costs in clock.
// EJOIN_EXP_NO_COPIES: after the first NSTAGE slices and the first tile's augmentation operands no global->LDS copy is
//   issued at all, and the rare path is switched off: every later slice computes on what those copies left in the LDS --
//   the same MFMAs, LDS reads and barriers on real operand bits with the copy path, the L2 and the fabric idle: what
//   feeding the LDS costs in cycles and clock (compared with the full kernel at epsilon = 0).
// EJOIN_EXP_CYCLE_MARKS: s_memtime marks between the sections of a tile; the per-section sums of all wavefronts
//   are added into the last 16 u64 of the pair buffer (waves 0-3, then waves 4-7) -- where a tile's cycles go.
#ifdef EJOIN_EXP_HOT_PANELS
#define EJ_PANEL_A(I) ((I) & 1u)
#define EJ_PANEL_B(J) (2u + ((J) & 1u))
#else
#define EJ_PANEL_A(I) (I)
#define EJ_PANEL_B(J) (J)
#endif
constexpr int NSTAGE = EJOIN_ABL_NSTAGE;  // ring of LDS stages; NSTAGE-1 slices are in flight from L2/HBM
constexpr int DIST = NSTAGE - 1;
constexpr int THREADS = 512;  // 8 wavefronts: 2 (rows) x 4 (columns), wave tile 128 x 64
constexpr int SB = (int)EJ_SB;
constexpr int PANEL_BYTES = TILE * KSLICE * 2;  // 16 KB : one operand panel of one stage
constexpr int STAGE_BYTES = 2 * PANEL_BYTES;    // A panel + B panel
constexpr int DUMP_OFF = NSTAGE * STAGE_BYTES;  // 1 KB that absorbs the copies issued past the end of the work
// Operands of the augmentation step of the tile being computed: 16 bytes per row of the A panel (4 KB), 16 bytes per
// column of the B panel (4 KB), and the two constant chunks of that step (layout: panel_layout.h, "a tile's
// augmentation buffer")
constexpr int AUG_OFF = DUMP_OFF + 1024;
constexpr int AUG_PART_BYTES = EJ_AUG_PART;
constexpr int AUGC_OFF = AUG_OFF + EJ_AUG_CONST;
constexpr int AUG_REGION_STEP = EJ_AUG_REGION_STEP;
constexpr int STG_OFF = AUG_OFF + EJ_AUG_BYTES;  // per-wave result staging: STG_CAP entries of (i, j, d2)
constexpr int STG_CAP = 128;
constexpr int DENSE_LANES = 12;  // candidates in that many lanes of a region: each lane looks at its own (see the rare path)
constexpr int QUEUE_CAP = 16;    // per-wave queue of lanes that hold a candidate (see the rare path): 16 values and a tag each
constexpr int STG_WAVE_BYTES = STG_CAP * 12 + QUEUE_CAP * 68;
constexpr int LDS_BYTES = STG_OFF + 8 * STG_WAVE_BYTES;
constexpr int NUM_XCD = (int)EJ_NUM_XCD;
static_assert(LDS_BYTES <= 160 * 1024, "LDS budget of one CU");
static_assert(NSTAGE == 3 || NSTAGE == 4, "the slice pipeline reads one slice ahead: at least two slices in flight");

// Device status word written by k_aux, read by the other kernels.
constexpr uint32_t ST_OK = 0, ST_NORM_RANGE = 1, ST_NONFINITE = 2;

struct JoinArgs {
  // "points" (rows of the distance matrix) and "query points" (columns); the self-join passes the same set twice
  const uint4* XpA;        // packed copy of the points plus their augmentation block, see k_norms / k_aux
  const uint4* XpB;        // ... of the query points
  int64_t nA, nB;
  int self;                // 1: self-join (upper triangle, self pairs), 0: two different sets (full rectangle)
  int swapped;             // k_join_strip: its rows are the query points, its columns the points (XpA, nA, counts: of the rows)
  uint32_t* status;        // status block of the workspace (see k_reset)
  int nslices;  // k-blocks of data per panel = slices per tile (the augmentation block follows them)
  float thr;    // pass <=> acc' >= thr, thr = -eps^2 / 2
  uint32_t ntilesA, ntilesB;  // ceil(n / TILE)
  uint32_t sb_row_begin, sb_row_end;  // rows of super-blocks this launch covers (a join returned in batches is cut by them)
  // pair mode
  uint32_t* pairs;
  float* dist2;
  unsigned long long capacity;
  unsigned long long* n_pairs;
  // count mode
  uint32_t* counts;    // per point (self-join: per point of the one set)
  uint32_t* counts_b;  // per query point (two-set join only; may be null)
  unsigned long long* total;
  // XCD-wide alignment of the workgroups (performance hint, see xcd_align)
  uint32_t* xcd_bar;  // NUM_XCD counters, zeroed before the launch
  int sync_mode;      // 0: never; k > 0: at the start and then before every k-th tile
};

// ------------------------------------------------------------------------------------------
// Small kernels
// ------------------------------------------------------------------------------------------
// Status block of a workspace (64 words): [0] status word, [1] largest norm seen so far in the call (FP32 bits),
// [2..3] the constant C = { c, c, c, 0 } of the call's augmentation step (FP16 bits, written by k_aux),
// [8..15] alignment counters of the XCDs.  Between calls [1] and [8..15] are zero: k_aux clears the counters
// (and the result counter of the call), k_join clears the maximum.  k_reset restores that state after a call
// that did not get as far as its join kernel, and before every call of k_join on the shared static workspace.
// (Small problems and the dense-tile call use word [0] only.)
__global__ void k_reset(uint32_t* status_and_max) {
  if (threadIdx.x < 8) status_and_max[8 + threadIdx.x] = 0;
  if (threadIdx.x == 0) {
    status_and_max[0] = ST_OK;
    status_and_max[1] = 0;
  }
}

__global__ void k_fill_u32(uint32_t* p, int64_t n, uint32_t v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// The largest of the values of a workgroup's lanes (the same for all of them).
__device__ __forceinline__ uint32_t max_of_group(uint32_t bits) {
  __shared__ uint32_t wave_max[8];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) bits = max(bits, (uint32_t)__shfl_xor((int)bits, off));
  if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = bits;
  __syncthreads();
  for (uint32_t w = 0; w < blockDim.x / 64; ++w) bits = max(bits, wave_max[w]);
  return bits;
}
// ... and added to *max_bits with one atomic: those on one address are served one after the other, about 11 ns each.
__device__ __forceinline__ void merge_max(uint32_t bits, uint32_t* max_bits) {
  bits = max_of_group(bits);
  if (threadIdx.x == 0) atomicMax(max_bits, bits);
}

// The largest of n values (n > 0) into the first of them; one workgroup.
__global__ __launch_bounds__(512) void k_fold_max(uint32_t* values, uint32_t n) {
  uint32_t most = 0;
  for (uint32_t q = threadIdx.x; q < n; q += 512) most = max(most, values[q]);
  most = max_of_group(most);  // (every value has been read once this returns)
  if (threadIdx.x == 0) values[0] = most;
}

// ---- What the workgroups of the one-launch kernels tell each other, in memory of the context's that is all zero between calls:
// 64-bit words, [0] and [16 (1 + x)] of XCD x (bits 0 .. 39: pairs found; 40 .. 51: workgroups that were late; 52 .. 63: tickets), slots for the largest norms of
// parts of the points, once for each XCD, and counters.  A slot that has been filled has its top bit set (a norm has no sign).
// (ONCE_SLOTS, ONCE_COUNTS: capacities)
constexpr size_t ONCE_STATE_BYTES = 16 * 8 * (1 + EJ_NUM_XCD);
constexpr unsigned long long ONCE_FOUND = (1ull << 40) - 1, ONCE_TICKET = 1ull << 52;
// A workgroup's ticket, with what it adds to the fields below, XCD by XCD: an eighth of the atomics on each of the XCDs' words, then
// one each on [0].  (One thread.)  True for the last workgroup of all, whose `all` are the fields' sums; the state is zero again.
__device__ __forceinline__ unsigned long long* state_of_xcd(unsigned long long* state) { return state + 16 * (1 + blockIdx.x % EJ_NUM_XCD); }
__device__ __forceinline__ bool close_by_xcd(unsigned long long* state, uint32_t workgroups, unsigned long long in_xcd /* with the ticket */, unsigned long long& all) {
  const uint32_t xcd = blockIdx.x % EJ_NUM_XCD, xcds = min(workgroups, EJ_NUM_XCD);
  unsigned long long* own = state_of_xcd(state);
  if (in_xcd >> 52 != (workgroups - xcd + xcds - 1) / xcds) return false;
  *own = 0;
  const unsigned long long sum = ONCE_TICKET | (in_xcd & (ONCE_TICKET - 1));
  all = atomicAdd(state, sum) + sum;
  if (all >> 52 != xcds) return false;
  *state = 0;
  return true;
}
// Looks at empty slots, of a thread at all of its own together, before it gives up; each is a load past the L2.  Where the GPU is shared the slots may be filled
// only once others' work has ended, and a workgroup that waits keeps its LDS from them; what it does instead, the norms of the points of the empty slots, is not
// much longer (every workgroup without waiting, and with a third of the slots empty to it: 1,000 x 96 15 and 13 us a call, 3,900 x 960 228 and 158, 3,900 x 4,096 919 and
// 633; 95.8 with all slots seen).  (Builds for the tests: EJOIN_ONCE_SPINS=0 waits for nothing, EJOIN_ONCE_BLIND=m takes every m-th slot for empty.)
#ifndef EJOIN_ONCE_SPINS
#define EJOIN_ONCE_SPINS 256
#endif
constexpr uint32_t ONCE_FILLED = 0x80000000u;
constexpr int ONCE_EMPTY_WORDS = ONCE_SLOTS / 32;
// The largest norm in the slots, of what this thread reads of them, for threads of `threads`; missing: one of them is still empty
// after `spins` more looks.  empty (LDS, ONCE_EMPTY_WORDS words that are zero, may be null): a bit for each of those.
__device__ __forceinline__ uint32_t look_at_slots(const uint32_t* slot, uint32_t slots, uint32_t threads, int spins, bool& missing, uint32_t* empty = nullptr) {
  uint32_t most = 0;
  missing = false;
  slot += blockIdx.x % EJ_NUM_XCD * ONCE_SLOTS;
  for (uint32_t q = threadIdx.x; q < slots; q += threads) {
    uint32_t v = __hip_atomic_load(slot + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (; v == 0 && spins > 0; --spins) {
      __builtin_amdgcn_s_sleep(1);
      v = __hip_atomic_load(slot + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
#ifdef EJOIN_ONCE_BLIND
    if (empty && q % EJOIN_ONCE_BLIND == 1) v = 0;
#endif
    if (v == 0) {
      missing = true;
      if (empty) atomicOr(empty + q / 32, 1u << (q % 32));
    }
    most = max(most, v & ~ONCE_FILLED);
  }
  return most;
}
// f(q) for every empty slot q, by all threads of the workgroup.  (Behind a barrier.)
template <typename F>
__device__ __forceinline__ void for_empty_slots(const uint32_t* empty, uint32_t slots, F f) {
  for (uint32_t word = 0; word * 32 < slots; ++word)
    for (uint32_t bits = __builtin_amdgcn_readfirstlane(empty[word]); bits; bits &= bits - 1) f(word * 32 + (uint32_t)__builtin_ctz(bits));
}

// Diagonal of the 16 x 16 Gram block of points row0 .. row0 + 15, whose element (row, col) sits in lane col + 16 * (row / 4),
// register row % 4: stored to s for points below n.  Returns this lane's norm (0 in a lane that holds none).
template <bool SHARED = false>  // SHARED: for other workgroups of the launch
__device__ __forceinline__ float store_diagonal(const float4v& acc, int64_t row0, int64_t n, float* __restrict__ s) {
  const int lane = threadIdx.x & 63, c = lane & 15;
  if ((c >> 2) != (lane >> 4) || row0 + c >= n) return 0.f;
  const float lo = (c & 1) ? acc[1] : acc[0], hi = (c & 1) ? acc[3] : acc[2];
  const float v = (c & 2) ? hi : lo;
  if (SHARED) __hip_atomic_store(s + row0 + c, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else s[row0 + c] = v;
  return v;
}

// Step 1 (Section 3.1): s_i = sum_k x_ik^2.  One wavefront per 32 consecutive points; the 16 x 16
// Gram blocks of its two halves are accumulated with the same MFMA steps, in the same k order, as
// the join kernel uses, and their diagonals are stored.  That makes s_i bit-identical to a_ii, and
// to a_ij for a duplicate j of i, so duplicates come out at distance exactly 0.  (The paper
// matches its norm rounding to its tensor cores' for the same reason.)  Also tracks max_i s_i
// (as FP32 bits; s >= 0 so unsigned order is numeric order, and NaN/Inf sort above every finite value).
//
// PACK: the same pass also writes the packed copy of X for the join kernel.  A panel (256 points) is cut into
// k-blocks of 32 coordinates; a k-block holds, for each of the panel's rows, the 64 bytes of a row of the LDS
// panel, already arranged the way the LDS wants them (see place_of); points n .. npad-1 are zero.  A k-block is
// 16 KB of contiguous memory, so the global->LDS copies of the join are straight 1 KB block copies made of full
// 128-byte lines (in the row-major X a 32-coordinate slice of a row is half a line, and the L2 would be asked for
// every line twice), and the `blocks` k-blocks of a panel follow each other (packed_index).  The 16 bytes a lane
// loads as its part of the MFMA operand (point l%16, chunk l/16 of the k-block) are exactly one chunk of that layout, and
// the two halves of 32 points together fill 2 KB of it.
//
// Bound by memory; what it takes is enough loads in flight (four k-blocks of two halves per wavefront) and few atomics: with
// 16 points per wavefront and one atomic each it ran at 0.7 TB/s on 10^6 x 128 (725 us with k_aux, now 94 + 12: 5.4 TB/s) and
// at 1.9 TB/s on 3 10^5 x 384 (244 us, now 86).
// HALVES = 1: 16 points per wavefront.  That is better where there is neither a copy to write nor a largest norm to fold: no atomics
// to save, so more and smaller workgroups (of one wavefront), and two k-blocks (d <= 64) are loaded together.  With 32 points,
// one k-block after the other: 10^6 x 64 26.5 us, now 19.6 (16 points, workgroups of 256, one k-block after the other, as
// before: 23.8); 10^5 x 512 18.4, now 16.1 (17.9).
constexpr int NORM_POINTS = 32;  // points per wavefront
template <bool PACK, int HALVES = 2, bool SHARED = false>  // returns the pattern of this lane's largest norm
__device__ __forceinline__ uint32_t norms_of_wave(int64_t row0, const uint16_t* __restrict__ X, int64_t n, int64_t ld, int k32steps,
                                                  float* __restrict__ s, uint4* __restrict__ Xp, int blocks) {
  const int lane = threadIdx.x & 63;
  int64_t own[HALVES];
  const half8* p[HALVES];
  uint4* out[HALVES];
  bool valid[HALVES];
#pragma unroll
  for (int h = 0; h < HALVES; ++h) {
    own[h] = row0 + 16 * h + (lane & 15);
    valid[h] = own[h] < n;
    p[h] = reinterpret_cast<const half8*>(X + (valid[h] ? own[h] : n - 1) * ld) + (lane >> 4);
    if (PACK) out[h] = Xp + packed_index(place_of(own[h], lane >> 4), 0, blocks);
  }
  float4v acc[HALVES];
#pragma unroll
  for (int h = 0; h < HALVES; ++h) acc[h] = float4v{0.f, 0.f, 0.f, 0.f};
  auto steps = [&](int k0, auto count_c) {
    constexpr int K = decltype(count_c)::value;
    half8 a[HALVES][K];
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int h = 0; h < HALVES; ++h) a[h][k] = p[h][4 * (k0 + k)];
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int h = 0; h < HALVES; ++h) {
        acc[h] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[h][k], a[h][k], acc[h], 0, 0, 0);
        if (PACK) out[h][(int64_t)(k0 + k) * 1024] = valid[h] ? __builtin_bit_cast(uint4, a[h][k]) : make_uint4(0, 0, 0, 0);
      }
  };
  int k = 0;
  for (; k + 4 <= k32steps; k += 4) steps(k, std::integral_constant<int, 4>{});
  if (k + 2 <= k32steps) {
    steps(k, std::integral_constant<int, 2>{});
    k += 2;
  }
  if (k < k32steps) steps(k, std::integral_constant<int, 1>{});
  uint32_t most = 0;
#pragma unroll
  for (int h = 0; h < HALVES; ++h) most = max(most, __float_as_uint(store_diagonal<SHARED>(acc[h], row0 + 16 * h, n, s)));
  return most;
}

template <bool PACK, int HALVES = 2, bool FROM_THE_END = false>
__global__ __launch_bounds__(512) void k_norms(const uint16_t* __restrict__ X, int64_t n, int64_t npad, int64_t ld, int k32steps,
                                               float* __restrict__ s, uint32_t* __restrict__ max_bits, uint4* __restrict__ Xp,
                                               int blocks /* k-blocks per panel of Xp: k32steps + 1 */,
                                               uint32_t* __restrict__ maxima /* one per workgroup (may be null) */) {
  const uint32_t group = FROM_THE_END ? gridDim.x - 1 - blockIdx.x : blockIdx.x;
  const int64_t row0 = ((int64_t)group * (blockDim.x >> 6) + (threadIdx.x >> 6)) * (16 * HALVES);
  uint32_t most = 0;
  if (row0 < (PACK ? npad : n)) most = norms_of_wave<PACK, HALVES>(row0, X, n, ld, k32steps, s, Xp, blocks);
  if (max_bits) merge_max(most, max_bits);
  if (maxima) {
    most = max_of_group(most);
    if (threadIdx.x == 0) maxima[blockIdx.x] = most;
  }
}

// Rows past the end of the data set carry -60000 c in place of -s/2 (at least the largest norm of the
// data), so that none of their pairs passes the filter for any ordinary epsilon (the rare path masks
// them exactly) and nothing non-finite enters the matrix cores.
constexpr uint32_t P1_OUT_OF_RANGE = 0xFB53u;  // -60000 in FP16

// Augmentation rows.  Step 3 of Section 3.1 (dist^2 = s_i + s_j - 2 a_ij) is folded into the
// matrix-core accumulation: after the Gram steps one more MFMA step (16 wide) adds
// -s_i/2 - s_j/2 to a_ij, so the accumulator ends as acc' = -dist^2 / 2 and the filter becomes a
// sign-like test against -eps^2/2.  -s/2 is FP32; scaled by 2^-m it is split into three FP16 pieces
// p1 + p2 + p3, where m puts the largest norm of the data just below 2^16 (s_max / 2 < 2^15 2^m),
// within -14 <= m <= 15 so that c = 2^m is a normal FP16 value (the matrix cores align the products
// of a step by their exponent fields; a subnormal c would cost them low bits).  The split is exact
// for every point with s >= max(2^-16 s_max, 2^-14): the 24 mantissa bits of s / 2^(m+1) then lie
// above FP16's smallest subnormal.  A smaller norm is carried to 2^-25 2^m absolute.  With the pieces
// P_i = { p1, p2, p3, 0 } and C = { c, c, c, 0 } the extra step multiplies
// pieces by constants, c (p1 + p2 + p3)_i + c (q1 + q2 + q3)_j = -s_i/2 - s_j/2, every product exact in FP32.
// For the join the operands of the extra step are
// written, ready made, into one more k-block behind the data k-blocks of each panel of the packed set (`Xp`,
// null: a set that is not there; k-block `aug_kb` of `blocks`): 16 bytes per row for the panel as the A operand (chunk 0 of
// panel_layout.h, "the augmentation step": 256 x 16 B), then 16 bytes per row for the panel as the B operand
// (chunk 1); the rest of the 16 KB is not used.  The join kernel copies the 4 KB + 4 KB of a tile's two panels
// to the LDS once per tile; the constant chunks 2 and 3 it builds itself from C, which is left in the status block.
// The kernel also clears what the join kernel expects to find zero (the join kernel of the call before has
// finished by now): the XCD alignment counters, the call's result counter `counter` and, in count mode,
// the per-point counts `counts` (n entries; may be null).
struct NormScale {
  uint32_t st;  // status of the data
  int m;        // (only if st is OK)
  _Float16 c;
};
__device__ __forceinline__ uint32_t fp16_bits(_Float16 x) { return (uint32_t)__builtin_bit_cast(uint16_t, x); }
__device__ __forceinline__ NormScale norm_scale(uint32_t max_bits) {
  NormScale r;
  r.m = 0;
  r.st = ST_OK;
  if (max_bits >= 0x7f800000u) r.st = ST_NONFINITE;  // Inf or NaN among the norms
  else {
    const int e = (int)(max_bits >> 23) - 127;  // max s < 2^(e+1)
    r.m = e - 15 < -14 ? -14 : e - 15;
    if (r.m > 15) r.st = ST_NORM_RANGE;  // 2^m must be an FP16 value: needs max s < 2^31
  }
  r.c = (_Float16)ldexpf(1.f, r.m > 15 ? 15 : r.m);
  return r;
}
// The pieces of the point of norm s (or, where it lies past the end, the marker) as two 32-bit words { p1 | p2 << 16, p3 }.
__device__ __forceinline__ uint2 norm_pieces(float s, int m) {
  const float v = ldexpf(-0.5f * s, -m);
  const _Float16 p1 = (_Float16)v;
  const float r1 = v - (float)p1;
  const _Float16 p2 = (_Float16)r1;
  const _Float16 p3 = (_Float16)(r1 - (float)p2);
  return make_uint2(fp16_bits(p1) | (fp16_bits(p2) << 16), fp16_bits(p3));
}

struct AuxSet {
  const float* s;
  int64_t n, npad;
  uint4* Xp;
  uint32_t* counts;  // count mode: cleared on the way (n entries; may be null)
};
struct AuxArgs {
  AuxSet a, b;  // (b.npad = 0: one set)
  uint32_t* status_and_max;
  const uint32_t* set_max;  // largest norm of a prepared set, or null
  int aug_kb;               // k-block of the augmentation operands = data k-blocks of a panel
  unsigned long long* counter;
};
__global__ __launch_bounds__(256) void k_aux(const AuxArgs args) {
  const uint32_t groups_a = (uint32_t)(args.a.npad / 256);
  const bool second = blockIdx.x >= groups_a;
  const AuxSet& set = second ? args.b : args.a;
  const int64_t i = (int64_t)(blockIdx.x - (second ? groups_a : 0u)) * 256 + threadIdx.x, n = set.n;
  const float* s = set.s;
  uint32_t mb = args.status_and_max[1];
  if (args.set_max) mb = max(mb, *args.set_max);
  if (blockIdx.x == 0) {
    if (threadIdx.x < 8) args.status_and_max[8 + threadIdx.x] = 0;
    if (threadIdx.x == 8 && args.counter) *args.counter = 0;
  }
  if (set.counts && i < n) set.counts[i] = 0;
  const NormScale ns = norm_scale(mb);
  const uint32_t st = ns.st, c = fp16_bits(ns.c);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    args.status_and_max[0] = st;
    args.status_and_max[2] = c | (c << 16);
    args.status_and_max[3] = c;
  }
  auto pieces = [&](int64_t x) -> uint2 {
    if (x >= n) return make_uint2(P1_OUT_OF_RANGE, 0u);
    if (st != ST_OK) return make_uint2(0u, 0u);
    return norm_pieces(s[x], ns.m);
  };
  const int r = (int)(i & 31);
  const int64_t b = i - r;
  const int64_t xa = b + aug_row_point(r), xb = b + aug_col_point(r);
  const uint2 a0 = pieces(xa), a1 = pieces(xa + 4), b0 = pieces(xb), b1 = pieces(xb + 16);
  uint4* blk = set.Xp + packed_index((i >> 8) << 10, args.aug_kb, args.aug_kb + 1);  // the panel's augmentation block
  blk[aug_block_unit((int)(i & 255), 0)] = make_uint4(a0.x, a0.y, a1.x, a1.y);
  blk[aug_block_unit((int)(i & 255), 1)] = make_uint4(b0.x, b0.y, b1.x, b1.y);
}

__device__ __forceinline__ half8 as_half8(uint4 v) { return __builtin_bit_cast(half8, v); }
__device__ __forceinline__ float16v cat4(float4v a, float4v b, float4v c, float4v d) {
  return __builtin_shufflevector(__builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7), __builtin_shufflevector(c, d, 0, 1, 2, 3, 4, 5, 6, 7),
                                 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
}

// Four consecutive floats from an address that need not be a multiple of 16 bytes (one 16-byte load all the same).
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));

// Ingestion: FP32 rows -> FP16 rows in the layout the join expects (row stride ld16, a multiple of 64,
// columns d .. ld16-1 zero).  y = fp16_rne(fl32(scale * fl32(x - center_k))).
// Bound by memory.  A thread makes COLS output columns of CONVERT_ROWS rows: 16-byte loads, and one store per row, the
// loads of all its rows in flight together; `wide` consecutive threads (a power of two that divides the chunks of a row, 8 to 64)
// take consecutive chunks of a row: at least a full line of the result.  With one row per thread, eight 4-byte loads 32 bytes
// apart and a 64-bit division per chunk it took 346 us on 5 10^5 x 200 (1.9 TB/s), with eight columns and four rows 105 to 115 (two rows
// per thread 111, eight 117).
// Input that the memory-side cache (256 MB) cannot hold is read past the caches (NT), which leaves them to the result: what comes next,
// norms or a join, reads that.  Then it has to be four columns a thread, whose loads are whole lines: 5 10^5 x 200 100 us, with the
// norms after it 161 us, now 135; 10^6 x 128 176, now 148; eight columns (half lines) 151.  Smaller input may well be in that cache
// already (10^5 x 128 again and again, with the norms: 19.7 us, 20.3 past the caches; 2 10^5 x 200 57, 60), and keeps eight columns; so do rows whose lines would be fetched
// twice (ingest_past_the_caches: 256,233 x 668 with the norms 267 us, 297 past the caches).  Rows that
// are not 16-byte aligned have lines that two loads share: 4 10^5 x 333 158 us with eight columns, 184 past the caches with four,
// 146 through them.
constexpr int CONVERT_ROWS = 4;
template <int COLS, bool NT>
__global__ __launch_bounds__(256) void k_convert_f32(const float* __restrict__ X32, int64_t n, int32_t d, int64_t ld32,
                                                     const float* __restrict__ center, float scale, uint16_t* __restrict__ X16, int64_t ld16,
                                                     uint32_t wide_log2, uint32_t blocks_per_row) {
  typedef _Float16 halves __attribute__((ext_vector_type(COLS)));
  const uint32_t wide = 1u << wide_log2, step = 256u >> wide_log2;  // chunks side by side, rows at a time
  const uint32_t rows_block = blockIdx.x / blocks_per_row;
  const int64_t chunk = ((int64_t)(blockIdx.x - rows_block * blocks_per_row) << wide_log2) + (threadIdx.x & (wide - 1));
  const int64_t row0 = (int64_t)rows_block * (step * CONVERT_ROWS) + (threadIdx.x >> wide_log2);
  const int64_t k0 = chunk * COLS;
  float c[COLS];
#pragma unroll
  for (int k = 0; k < COLS; ++k) c[k] = center && k0 + k < d ? center[k0 + k] : 0.f;
  float x[CONVERT_ROWS][COLS];
#pragma unroll
  for (int r = 0; r < CONVERT_ROWS; ++r) {
    const int64_t i = row0 + r * step;
    const float* p = X32 + (i < n ? i : n - 1) * ld32 + k0;
    if (k0 + COLS <= d) {
#pragma unroll
      for (int q = 0; q < COLS; q += 4) {
        const float4u* at = reinterpret_cast<const float4u*>(p + q);
        const float4u four = NT ? __builtin_nontemporal_load(at) : *at;
#pragma unroll
        for (int k = 0; k < 4; ++k) x[r][q + k] = four[k];
      }
    } else {
#pragma unroll
      for (int k = 0; k < COLS; ++k) x[r][k] = k0 + k < d ? p[k] : 0.f;
    }
  }
#pragma unroll
  for (int r = 0; r < CONVERT_ROWS; ++r) {
    const int64_t i = row0 + r * step;
    halves h;
#pragma unroll
    for (int k = 0; k < COLS; ++k) {
      float t = x[r][k] - c[k];
      asm volatile("" : "+v"(t));  // keep the FP32 rounding of every step: no fused subtract-multiply-convert
      float y = k0 + k < d ? scale * t : 0.f;
      asm volatile("" : "+v"(y));
      h[k] = (_Float16)y;
    }
    if (i < n) *reinterpret_cast<halves*>(X16 + i * ld16 + k0) = h;
  }
}

// Split-FP16 variant (higher accuracy for FP32 inputs).  Each FP32 coordinate is cut into two FP16
// numbers, x ~ hi + lo with hi = fp16(x), lo = fp16(x - hi) (22 significant bits together), and the
// inner product is taken as hi.hi + lo.hi + hi.lo (the lo.lo term is below the 22 bits kept): an ordinary inner product of the
// 3d-dimensional rows A' = [hi | lo | hi] and B' = [hi | hi | lo].  The packed copy (the k-block layout of k_norms<true>) holds
// hi and lo once, nkb blocks each; the join kernels take the k-blocks of A' and B' from them (split_block_a, split_block_b).
//
// One pass over the FP32 rows writes both and accumulates the norms s_i = A'_i . B'_i with the MFMA steps, and in the order, in
// which the join accumulates a_ii; the second and third part of that order read the rows again, from the caches.  Bound by
// memory.  Before, two copies of three parts each were written, 32 bytes of FP32 per thread and chunk, and the norms read back
// from them with one atomic per 16 points: 122 us for 50,000 x 300, now 45.
constexpr int split_block_a(int ks, int nkb) { return ks >= 2 * nkb ? ks - 2 * nkb : ks; }
constexpr int split_block_b(int ks, int nkb) { return ks >= nkb ? ks - nkb : ks; }
struct SplitArgs {
  const float* X32;
  int64_t n, npad, ld32;
  int32_t d;
  int nkb;
  float* s;
  uint4* Xp;           // 2 nkb + 1 k-blocks per panel
  uint32_t* maxima;    // one per workgroup, or null:
  uint32_t* max_bits;  // ... the largest of all
  unsigned long long* counter;  // cleared, like the counts (may be null)
  uint32_t* counts;
};
__global__ __launch_bounds__(512) void k_split_prep(const SplitArgs a) {
  const int lane = threadIdx.x & 63;
  const int64_t row0 = ((int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * NORM_POINTS;
  if (blockIdx.x == 0 && threadIdx.x == 0 && a.counter) *a.counter = 0;
  uint32_t most = 0;
  if (row0 < a.npad) {
    if (a.counts && lane < NORM_POINTS && row0 + lane < a.n) a.counts[row0 + lane] = 0;
    const int c0 = (lane >> 4) * 8;  // first coordinate of this lane's chunk in a k-block
    const float* p[2];
    uint4* out[2];
    bool valid[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t own = row0 + 16 * h + (lane & 15);
      valid[h] = own < a.n;
      p[h] = a.X32 + (valid[h] ? own : a.n - 1) * a.ld32 + c0;
      out[h] = a.Xp + packed_index(place_of(own, lane >> 4), 0, 2 * a.nkb + 1);
    }
    auto load = [&](int h, int kb, half8& hi, half8& lo) {
      const int k0 = kb * KSLICE + c0;
      const float* q = p[h] + kb * KSLICE;
      float x[8];
      if (k0 + 8 <= a.d) {
        const float4u u = *reinterpret_cast<const float4u*>(q), v = *reinterpret_cast<const float4u*>(q + 4);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          x[k] = u[k];
          x[4 + k] = v[k];
        }
      } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) x[k] = k0 + k < a.d ? q[k] : 0.f;
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float y = valid[h] ? x[k] : 0.f;
        const _Float16 t = (_Float16)y;
        float rest = y - (float)t;
        asm volatile("" : "+v"(rest));  // the residual is an FP32 number: no fused subtract-convert
        hi[k] = t;
        lo[k] = (_Float16)rest;
      }
    };
    float4v acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    auto steps = [&](auto part_c, int kb0, auto count_c) {
      constexpr int PART = decltype(part_c)::value, K = decltype(count_c)::value;
      half8 hi[2][K], lo[2][K];
#pragma unroll
      for (int k = 0; k < K; ++k)
#pragma unroll
        for (int h = 0; h < 2; ++h) load(h, kb0 + k, hi[h][k], lo[h][k]);
#pragma unroll
      for (int k = 0; k < K; ++k)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          acc[h] = __builtin_amdgcn_mfma_f32_16x16x32_f16(PART == 1 ? lo[h][k] : hi[h][k], PART == 2 ? lo[h][k] : hi[h][k], acc[h], 0, 0, 0);
          if (PART == 0) {
            out[h][(int64_t)(kb0 + k) * 1024] = __builtin_bit_cast(uint4, hi[h][k]);
            out[h][(int64_t)(a.nkb + kb0 + k) * 1024] = __builtin_bit_cast(uint4, lo[h][k]);
          }
        }
    };
    auto part = [&](auto part_c) {
      int kb = 0;
      for (; kb + 2 <= a.nkb; kb += 2) steps(part_c, kb, std::integral_constant<int, 2>{});
      if (kb < a.nkb) steps(part_c, kb, std::integral_constant<int, 1>{});
    };
    part(std::integral_constant<int, 0>{});
    part(std::integral_constant<int, 1>{});
    part(std::integral_constant<int, 2>{});
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float v = store_diagonal(acc[h], row0 + 16 * h, a.n, a.s);
      most = max(most, v < 0.f ? 0u : __float_as_uint(v));  // (a sum that rounds below zero counts as zero; NaN stays NaN)
    }
  }
  most = max_of_group(most);
  if (threadIdx.x == 0) {
    if (a.max_bits) atomicMax(a.max_bits, most);
    else a.maxima[blockIdx.x] = most;
  }
}

// Workgroup barrier without the fences of __syncthreads(): those make the compiler wait for every
// outstanding global->LDS copy (vmcnt(0)) at each barrier, which would serialise the copy pipeline.
// The kernel orders its LDS traffic itself: copies are certified with counted vmcnt waits before the
// barrier, and fragment reads are complete once the MFMAs consuming them have issued.
__device__ __forceinline__ void wg_barrier() { asm volatile("s_barrier" ::: "memory"); }

// One global->LDS copy instruction: every lane moves 16 bytes from sbase + voff (sbase uniform) to
// LDS address lds_addr + LDS_IMM + 16 * lane (lds_addr uniform, goes through M0).  Written as inline
// assembly on purpose: for the builtin form the compiler assumes the instruction may also count on
// lgkmcnt, and from then on turns every LDS wait into lgkmcnt(0), which breaks the overlap of
// fragment reads with MFMAs.  The copies are tracked by hand with counted vmcnt waits.
template <int LDS_IMM>
__device__ __forceinline__ void copy16_to_lds(uint32_t lds_addr, const void* sbase, uint32_t voff) {
  asm volatile(
      "s_add_u32 m0, %0, %3\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %1, %2"
      :
      : "s"(lds_addr), "v"(voff), "s"(sbase), "n"(LDS_IMM)
      : "memory", "m0", "scc");
}
// The same from an address of each lane's own.
template <int LDS_IMM>
__device__ __forceinline__ void copy16_to_lds_from(uint32_t lds_addr, const void* p) {
  asm volatile(
      "s_add_u32 m0, %0, %2\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %1, off"
      :
      : "s"(lds_addr), "v"(p), "n"(LDS_IMM)
      : "memory", "m0", "scc");
}

// Dense block of squared distances with the join's arithmetic: a workgroup of 2 x 2 or 2 x 4 wavefronts per TS x TS tile of the block,
// every 32 x 32 region of it computed the way the join kernel computes a region of its wave tile: four 16 x 16 blocks
// accumulated with v_mfma_f32_16x16x32_f16, then one v_mfma_f32_32x32x16_f16 on the four blocks' registers side by side that
// adds -s_i/2 - s_j/2 (operand layout: see the augmentation step of k_join).
// Bound by how the operands reach the CUs and then by writing the block (4,000 x 5,000 at d = 384, 80 MB: 33.5 to 38 us a call over
// the cards, of which the norms of the 20,000 points take 6; some 28 without the stores).  The operands come from X as it is, 64 coordinates of a row (a whole
// line) at a time, straight to the LDS, STAGES - 1 slices ahead; the columns are the rows of the MFMAs, so that a lane stores sixteen
// bytes of a row; the operands of the augmentation step are worked out here, from the norms.  With slices through registers, four
// wavefronts, 4-byte stores and a launch of their own for the augmentation rows, both on one card: 53.8 us a call, now 37.8;
// 1,500 x 1,500 20.5, now 17.2; 2,000 x 3,000 at d = 960 47.2, now 33.7; 6,000 x 6,000 at d = 128 56.2, now 40.6.  Eight wavefronts for TS = 128, of which two workgroups fit a CU: with four of
// 64 x 64 each (another card) 41 us a call, with eight 37, with sixteen 38; 6,000 x 6,000 at d = 128 41, 37, 41.  (Tried: rows of
// 256 bytes stored by way of the LDS: the same; stores that pass the caches by: 68.)
// ONE: the norms are worked out in this launch, by workgroups that come before those of the tiles, which look for them before their
// first slice and, where they are not there yet, after the last (see k_join_once: slots, a bounded wait, tickets).
// TS = 128 needs half the operand traffic of TS = 64, which gives four times the workgroups: at 144 of the larger kind (1,500 x
// 1,500, d = 384) 15.2 us a call against 13.6, at 225 (1,800 x 1,800) 15.6 against 16.9, at 240 (700 x 5,001, d = 100) 13.2 against
// 14.6, at 289 the same, at 1,280 39 against 46: the line lies at three workgroups of the larger kind for four CUs.
struct DenseArgs {
  const uint16_t* X;
  const float* s;
  const uint32_t* maxima;  // largest norms, one per workgroup of k_norms
  uint32_t nmaxima;
  uint32_t* status;
  int64_t n, ld;
  int slices;  // of 64 coordinates
  int64_t i0, j0;
  int rows, cols;
  float* out;
};
struct NoArgs {};
struct DenseOneArgs {  // (ONE)
  // workgroups that work out the norms (a multiple of 8), their k-blocks, and of the context, all zero between calls:
  float* s_out;  // (s)
  uint32_t norm_groups;
  int nkb;
  unsigned long long* state;
  uint32_t* slot;
};
template <int TS>
constexpr int dense_stages() { return TS == 64 ? 3 : 2; }
template <int TS>
constexpr int dense_waves() { return TS == 64 ? 4 : 8; }
template <int TS>
constexpr int dense_lds_bytes() { return dense_stages<TS>() * 2 * TS * 128 + 2 * TS * 16 + 64; }
template <int TS, bool ONE>
__global__ __launch_bounds__(64 * dense_waves<TS>(), TS == 64 ? 3 : 4) void k_dist2_tile(const DenseArgs a, const std::conditional_t<ONE, DenseOneArgs, NoArgs> one) {
  constexpr int WAVES = dense_waves<TS>(), ACROSS = WAVES / 2;  // two rows of wavefronts
  constexpr int WR = TS / 2, WC = TS / ACROSS, MR = WR / 16, MC = WC / 16;  // wave tile, and its 16 x 16 blocks: rows, columns
  constexpr int COPIES = TS / 8 / WAVES;                  // copy instructions per wavefront, operand and slice
  constexpr int STAGES = dense_stages<TS>();
  constexpr int OP_BYTES = TS * 128, ST_BYTES = 2 * OP_BYTES;
  constexpr int AUG = STAGES * ST_BYTES, AUG_B = AUG + TS * 16, AUG_CONST = AUG_B + TS * 16;
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / ACROSS * WR, wn = wave % ACROSS * WC;
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
  // workgroup -> tile: a contiguous part of the tiles for every XCD, in bands of eight rows, column by column
  const uint32_t tr = (uint32_t)(a.rows + TS - 1) / TS, tc = (uint32_t)(a.cols + TS - 1) / TS, tiles = tr * tc;
  uint32_t block = blockIdx.x;
  if constexpr (ONE) block -= one.norm_groups;
  const uint32_t t = block % EJ_NUM_XCD * ((tiles + EJ_NUM_XCD - 1) / EJ_NUM_XCD) + block / EJ_NUM_XCD;
  unsigned long long in_xcd = 0;
  auto ticket = [&]() __attribute__((always_inline)) {  // (ONE) the slots are no longer needed
    if constexpr (ONE) {
      if (tid == 0) in_xcd = atomicAdd(state_of_xcd(one.state), ONCE_TICKET);
    }
  };
  auto leave = [&]() __attribute__((always_inline)) {  // the last workgroup of all clears them
    if constexpr (ONE) {
      if (wave != 0) return;
      unsigned long long all;
      const bool last = lane == 0 && close_by_xcd(one.state, gridDim.x, in_xcd + ONCE_TICKET, all);
      if (__ballot(last))
        for (uint32_t q = lane; q < one.norm_groups * EJ_NUM_XCD; q += 64) one.slot[q % EJ_NUM_XCD * ONCE_SLOTS + q / EJ_NUM_XCD] = 0;
    }
  };
  auto norms_from = [&](int64_t row0) __attribute__((always_inline)) -> uint32_t {
    if constexpr (!ONE) return 0u;
    else return row0 < a.n ? norms_of_wave<false, 1, true>(row0, a.X, a.n, a.ld, one.nkb, one.s_out, nullptr, 0) : 0u;
  };
  if constexpr (ONE) {
    if (blockIdx.x < one.norm_groups) {
      const uint32_t own = norms_from(((int64_t)blockIdx.x * WAVES + wave) * 16);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the norms are there before the slot says so
      const uint32_t most = max_of_group(own);
      if (tid < (int)EJ_NUM_XCD) __hip_atomic_store(one.slot + tid * ONCE_SLOTS + blockIdx.x, most | ONCE_FILLED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      ticket();
      leave();
      return;
    }
  }
  if (t >= tiles) {
    if constexpr (ONE) {
      ticket();
      leave();
    }
    return;
  }
  const uint32_t band = t / (EJ_BAND * tc), in_band = t - band * EJ_BAND * tc;
  const uint32_t h = tr - band * EJ_BAND < EJ_BAND ? tr - band * EJ_BAND : EJ_BAND;
  const int bi = (int)(band * EJ_BAND + in_band % h) * TS, bj = (int)(in_band / h) * TS;
  auto row_a = [&](int local) { const int64_t r = a.i0 + bi + local; return r >= a.n ? a.n - 1 : r; };
  auto row_b = [&](int local) { const int64_t r = a.j0 + bj + local; return r >= a.n ? a.n - 1 : r; };
  // A slice of an operand in the LDS: rows of 128 bytes (64 coordinates), chunk c of row r at position c ^ swizzle(r): the 16 lanes
  // that an LDS read serves together, rows r .. r + 15 at one chunk or half of them at the chunk beside it, hit all banks.  A copy
  // instruction fills eight rows.
  auto swizzle = [](int row) { return (row >> 1) & 7; };
  const char *ga[COPIES], *gb[COPIES];
#pragma unroll
  for (int q = 0; q < COPIES; ++q) {
    const int r = 8 * (WAVES * q + wave) + (lane >> 3), c = (lane & 7) ^ swizzle(r);
    ga[q] = reinterpret_cast<const char*>(a.X + row_a(r) * a.ld) + 16 * c;
    gb[q] = reinterpret_cast<const char*>(a.X + row_b(r) * a.ld) + 16 * c;
  }
  auto issue = [&](int stage) {  // the next slice
    const uint32_t at = __builtin_amdgcn_readfirstlane(lds0 + stage * ST_BYTES + wave * 1024);
    static_assert(COPIES == 2, "two copy instructions per wavefront and operand");
    copy16_to_lds_from<0>(at, ga[0]);
    copy16_to_lds_from<WAVES * 1024>(at, ga[1]);
    copy16_to_lds_from<OP_BYTES>(at, gb[0]);
    copy16_to_lds_from<OP_BYTES + WAVES * 1024>(at, gb[1]);
#pragma unroll
    for (int q = 0; q < COPIES; ++q) {
      ga[q] += 128;
      gb[q] += 128;
    }
  };
#pragma unroll
  for (int ks = 0; ks < STAGES - 1; ++ks)
    if (ks < a.slices) issue(ks);
  // ---- operands of the augmentation step from the norms: thread t row t of the tile's column points, then of its row points.  The
  // wave tile is accumulated with the columns as rows of the MFMA (a lane then holds four consecutive columns of a row of the block);
  // the step adds the rows' terms first all the same, as the joins do.
  float sx = 0.f, sy = 0.f;
  uint32_t mb = 0;
  auto read_norms = [&]() __attribute__((always_inline)) {
    if (tid < 2 * TS) {
      const bool row_part = tid >= TS;
      const int r = tid & (TS - 1), in = r & 31;
      const int x = (r & ~31) + (row_part ? aug_col_point(in) : aug_row_point(in)), y = x + (row_part ? 16 : 4);
      const int64_t ax = row_a(x), bx = row_b(x), ay = row_a(y), by = row_b(y);  // (a choice between the two before they are worked out puts the arguments into scratch memory)
      sx = __hip_atomic_load(a.s + (row_part ? ax : bx), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      sy = __hip_atomic_load(a.s + (row_part ? ay : by), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  };
  auto norm_operands = [&]() __attribute__((always_inline)) -> bool {  // false: data out of range
    const NormScale ns = norm_scale(max_of_group(mb));
    if (block == 0 && tid == 0) a.status[0] = ns.st;
    if (ns.st != ST_OK) return false;
    if (tid < 2 * TS) {
      const uint2 p = norm_pieces(sx, ns.m), q = norm_pieces(sy, ns.m);
      *reinterpret_cast<uint4*>(lds + AUG + tid * 16) = make_uint4(p.x, p.y, q.x, q.y);
    }
    if (tid < 4) {  // the constant chunks of the augmentation step (2 and 3)
      const uint32_t c = fp16_bits(ns.c), c0 = c | (c << 16);
      *reinterpret_cast<uint2*>(lds + AUG_CONST + tid * 8) = tid == 0 || tid == 3 ? make_uint2(c0, c) : make_uint2(0u, 0u);
    }
    return true;
  };
  bool there = true;  // the norms and their largest
  if constexpr (ONE) {
    bool missing;
    mb = look_at_slots(one.slot, one.norm_groups, 64 * WAVES, 0, missing);
    there = !__syncthreads_or(missing);
    if (there) {
      read_norms();
      ticket();
    }
  } else {  // (as in read_norms, which by itself makes these instances 20 instructions longer)
    if (tid < 2 * TS) {
      const bool row_part = tid >= TS;
      const int r = tid & (TS - 1), in = r & 31;
      const int x = (r & ~31) + (row_part ? aug_col_point(in) : aug_row_point(in)), y = x + (row_part ? 16 : 4);
      sx = a.s[row_part ? row_a(x) : row_b(x)];
      sy = a.s[row_part ? row_a(y) : row_b(y)];
    }
    for (uint32_t q = tid; q < a.nmaxima; q += 64 * WAVES) mb = max(mb, a.maxima[q]);
  }
  if (there && !norm_operands()) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the copies must land before the wave ends
    leave();
    return;
  }
  uint32_t off[2];  // k-block kb of the slice: row lane % 16, chunk 4 kb + lane / 16
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) off[kb] = (lane & 15) * 128 + (((4 * kb + (lane >> 4)) ^ swizzle(lane & 15)) << 4);
  float4v acc[MC][MR];  // [columns][rows]
#pragma unroll
  for (int x = 0; x < MC; ++x)
#pragma unroll
    for (int y = 0; y < MR; ++y) acc[x][y] = float4v{0.f, 0.f, 0.f, 0.f};
  int stage = 0;
  for (int ks = 0; ks < a.slices; ++ks) {
    // (as in k_join_small)
    if (STAGES == 3 && ks + 1 < a.slices) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(2 * COPIES) : "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    wg_barrier();  // slice ks is there for everybody, and everybody is done with slice ks - 1
    if (ks + STAGES - 1 < a.slices) issue(stage == 0 ? STAGES - 1 : stage - 1);
    const char* st = lds + stage * ST_BYTES;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      half8 fa[MR], fb[MC];
#pragma unroll
      for (int f = 0; f < MR; ++f) fa[f] = *reinterpret_cast<const half8*>(st + (wm + 16 * f) * 128 + off[kb]);
#pragma unroll
      for (int f = 0; f < MC; ++f) fb[f] = *reinterpret_cast<const half8*>(st + OP_BYTES + (wn + 16 * f) * 128 + off[kb]);
#pragma unroll
      for (int x = 0; x < MC; ++x)
#pragma unroll
        for (int y = 0; y < MR; ++y) acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fb[x], fa[y], acc[x][y], 0, 0, 0);
    }
    stage = stage == STAGES - 1 ? 0 : stage + 1;
  }
  if constexpr (ONE) {
    if (!there) {
      uint32_t* empty = reinterpret_cast<uint32_t*>(lds + AUG);
      if (tid < ONCE_EMPTY_WORDS) empty[tid] = 0;
      __syncthreads();
      bool missing;
      mb = look_at_slots(one.slot, one.norm_groups, 64 * WAVES, EJOIN_ONCE_SPINS, missing, empty);
      if (__syncthreads_or(missing)) {  // workgroups that have not been started: their norms by this one
        for_empty_slots(empty, one.norm_groups, [&](uint32_t q) { mb = max(mb, norms_from(((int64_t)q * WAVES + wave) * 16)); });
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
      }
      read_norms();
      ticket();
      if (!norm_operands()) {
        leave();
        return;
      }
      __syncthreads();
    }
  }
  const int m = lane & 31;
  const char* aug_c = lds + (lane < 32 ? AUG_CONST + 16 * ((lane >> 3) & 1) : AUG + 16 * (wn + m));
  const char* aug_r = lds + (lane < 32 ? AUG_B + 16 * (wm + m) : AUG_CONST + 16 * ((lane >> 4) & 1));
  const int step_c = lane < 32 ? 0 : 512, step_r = lane < 32 ? 512 : 0;
#pragma unroll
  for (int Rr = 0; Rr < MR / 2; ++Rr) {
    const half8 hr = *reinterpret_cast<const half8*>(aug_r + Rr * step_r);
#pragma unroll
    for (int Rc = 0; Rc < MC / 2; ++Rc) {
      const half8 hc = *reinterpret_cast<const half8*>(aug_c + Rc * step_c);
      const float16v res = __builtin_amdgcn_mfma_f32_32x32x16_f16(
          hc, hr, cat4(acc[2 * Rc][2 * Rr], acc[2 * Rc][2 * Rr + 1], acc[2 * Rc + 1][2 * Rr], acc[2 * Rc + 1][2 * Rr + 1]), 0, 0, 0);
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int b = 0; b < 2; ++b) {  // (region_pair with rows and columns exchanged)
          const int rr = bi + wm + 32 * Rr + 16 * c + (lane & 15), cc = bj + wn + 32 * Rc + 16 * b + 4 * (lane >> 4);
          if (rr >= a.rows || cc >= a.cols) continue;
          const int64_t self = a.i0 + rr - a.j0 - cc;  // column of the point itself, from cc
          float4u v;
#pragma unroll
          for (int q = 0; q < 4; ++q) v[q] = self == q ? 0.f : fmaxf(-2.f * res[8 * b + 4 * c + q], 0.f);
          float* to = a.out + (int64_t)rr * a.cols + cc;
          if (cc + 4 <= a.cols) *reinterpret_cast<float4u*>(to) = v;
          else
            for (int q = 0; q < a.cols - cc; ++q) to[q] = v[q];
        }
    }
  }
  leave();
}

// ------------------------------------------------------------------------------------------
// The join kernel
// ------------------------------------------------------------------------------------------
// Brings the workgroups of one XCD back in step: each adds one to its XCD's counter and waits until
// the counter reaches `expect` (workgroups per XCD x number of alignments so far).  Workgroups that
// share operand panels only hit each other's lines in the XCD's L2 while they are within a few slices
// of each other.  Purely a performance hint: the wait is bounded, so a grid that is not fully
// resident cannot hang, and nothing depends on the counter's value.  A workgroup that has run out of
// tiles adds 2^24, which satisfies every later expectation of the others.
__device__ __forceinline__ void xcd_align(uint32_t* bar, uint32_t expect) {
  if (threadIdx.x == 0) {
    __hip_atomic_fetch_add(bar, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int spin = 0; spin < 20000; ++spin) {
      if (__hip_atomic_load(bar, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= expect) break;
      __builtin_amdgcn_s_sleep(8);
    }
  }
  __syncthreads();
}

// ---- The sixteen values of a lane for a 32 x 32 region (register r: pair (i0 + 16 (r / 8) + r % 4, j0 + 16 (r / 4 % 2)) of the
// lane's register 0, see region_pair), looked at by the lane itself.
// Register r of v, r different from lane to lane.
__device__ __forceinline__ float pick(const float16v& v, uint32_t r) {
  const bool b0 = r & 1u, b1 = r & 2u, b2 = r & 4u, b3 = r & 8u;
  auto four = [&](float w, float x, float y, float z) {
    const float lo = b0 ? x : w, hi = b0 ? z : y;
    return b1 ? hi : lo;
  };
  const float q0 = four(v[0], v[1], v[2], v[3]), q1 = four(v[4], v[5], v[6], v[7]);
  const float q2 = four(v[8], v[9], v[10], v[11]), q3 = four(v[12], v[13], v[14], v[15]);
  const float lo = b2 ? q1 : q0, hi = b2 ? q3 : q2;
  return b3 ? hi : lo;
}
// The registers whose pairs are pairs of the result at all (bit r: register r).  Rows and columns past n carry a large negative
// marker, which a huge epsilon can still reach.
__device__ __forceinline__ uint32_t keep_mask(uint32_t i0, uint32_t j0, uint32_t nA, uint32_t nB, bool diag) {
  uint32_t keep = 0;
#pragma unroll 1
  for (int r = 15; r >= 0; --r) {
    const uint32_t i = i0 + 16 * (r >> 3) + (r & 3), j = j0 + 16 * ((r >> 2) & 1);
    keep = 2 * keep + (i < nA && j < nB && (!diag || i < j) ? 1u : 0u);
  }
  return keep;
}
// Adds the hits of a region to counters in the LDS: rows[0] is the lane's register 0's row, columns[0] its column.
__device__ __forceinline__ void add_region_counts(uint32_t hit, uint32_t* rows, uint32_t* columns) {
  const uint32_t c0 = __popc(hit & 0x0F0Fu), c1 = __popc(hit & 0xF0F0u);
  if (c0) atomicAdd(columns, c0);
  if (c1) atomicAdd(columns + 16, c1);
  uint32_t left = (hit | (hit >> 4)) & 0x0F0Fu;  // two registers share a row
  while (__ballot(left != 0)) {
    if (left) {
      const uint32_t r = (uint32_t)__builtin_ctz(left);
      atomicAdd(rows + 2 * (r & 8u) + (r & 3u), ((hit >> r) & 1u) + ((hit >> (r + 4)) & 1u));
      left &= left - 1;
    }
  }
}
// The counters of a wave tile (128 rows from i0, 64 columns from j0) to the result, one atomic per row and column; zero again after.
__device__ __forceinline__ void send_region_counts(uint32_t* counters, uint32_t lane, const JoinArgs& a, uint32_t i0, uint32_t j0) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  for (int q = 0; q < 3; ++q) {
    const uint32_t c = counters[64 * q + lane];
    if (c) {
      counters[64 * q + lane] = 0;
      if (q < 2) atomicAdd(&a.counts[i0 + 64 * q + lane], c);
      else if (a.self) atomicAdd(&a.counts[j0 + lane], c);
      else if (a.counts_b) atomicAdd(&a.counts_b[j0 + lane], c);
    }
  }
}
__device__ __forceinline__ uint32_t wave_sum(uint32_t x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += (uint32_t)__shfl_xor((int)x, off);
  return __builtin_amdgcn_readfirstlane(x);
}

// DENSE (count mode): the instance whose rare path also handles regions with candidates in many lanes lane by lane.
// SPLIT: the k-blocks of the slices are those of a split-FP16 set (see k_split_prep).
template <bool COUNT, bool DENSE, bool SPLIT>
__global__ __launch_bounds__(THREADS) void k_join(const JoinArgs a) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  // the largest norm of the call has been consumed by k_aux: cleared here for the next call
  if (blockIdx.x == 0 && threadIdx.x == 0) a.status[1] = 0;
  if (*a.status != ST_OK) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  const int nsl = a.nslices;       // slices per tile (at least 2)
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
  // the constant chunks of the augmentation step (made visible by the barrier of the prologue)
  if (tid < 8) {
    const uint32_t c0 = a.status[2], c1 = a.status[3];
    *reinterpret_cast<uint4*>(lds + AUGC_OFF + (tid >> 1) * AUG_REGION_STEP + (tid & 1) * 16) =
        (tid & 1) ? make_uint4(0u, 0u, c0, c1) : make_uint4(c0, c1, 0u, 0u);
  }

  // --- global->LDS copies.  One global_load_lds_dwordx4 moves 1 KB (64 lanes x 16 B) = 16 rows of a
  // panel; in the packed layout that is 1 KB of contiguous global memory.  Only waves 4..7 copy: wave
  // 4 + c moves blocks c, c + 4, c + 8, c + 12 of both 16 KB panels of a slice, 8 copy instructions per
  // slice, always (past the end of the work they are pointed at a dump area), so the number of their
  // outstanding copies is a constant.  The copy unit of the CU accepts the instructions one after the
  // other and a wave waits at the issue of its own until they are taken; waves 0..3, which share the
  // SIMDs with 4..7 one to one, issue none and keep the MFMA pipes busy meanwhile.
  const char* XbA = reinterpret_cast<const char*>(a.XpA);
  const char* XbB = reinterpret_cast<const char*>(a.XpB);
  // a panel's k-blocks (16 KB each) follow each other in memory: the data blocks, then the augmentation block
  const int third = SPLIT ? nsl / 3 : 0;
  const int data_blocks = SPLIT ? 2 * third : nsl;
  const int64_t panel_stride = (int64_t)(data_blocks + 1) * PANEL_BYTES;
  const int cw = wave & 3;
  const bool copier = wave >= 4;
  const uint32_t voff0 = lane * 16 + cw * 1024;
  // (a copy takes its base address in scalar registers; the addresses are uniform, which is said explicitly because the
  // compiler, when it keeps such a pointer in vector registers, does not always move it back by itself)
  auto uniform_ptr = [](const char* p) -> const char* {
    const uint64_t b = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b), hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return reinterpret_cast<const char*>(((uint64_t)hi << 32) | lo);
  };
  auto issue_slice = [&](const char* pa_, const char* pb_, uint32_t lds_stage /* LDS address of the stage + cw*1024 */) {
    const char* pa = uniform_ptr(pa_);
    const char* pb = uniform_ptr(pb_);
    copy16_to_lds<0>(lds_stage, pa, voff0);
    copy16_to_lds<4096>(lds_stage, pa, voff0 + 4096);
    copy16_to_lds<8192>(lds_stage, pa, voff0 + 8192);
    copy16_to_lds<12288>(lds_stage, pa, voff0 + 12288);
    copy16_to_lds<PANEL_BYTES>(lds_stage, pb, voff0);
    copy16_to_lds<PANEL_BYTES + 4096>(lds_stage, pb, voff0 + 4096);
    copy16_to_lds<PANEL_BYTES + 8192>(lds_stage, pb, voff0 + 8192);
    copy16_to_lds<PANEL_BYTES + 12288>(lds_stage, pb, voff0 + 12288);
  };
  constexpr int NCOPY = 8;  // copy instructions per slice and copying wave
  // The operands of a tile's augmentation step: 4 KB of panel I's augmentation block and 4 KB of panel J's, into a
  // buffer of their own: eight copy instructions per tile, issued in the tile's first slice (every wave has then left the
  // tile before and its reads of the buffer behind) and read in its last.  They are the job of
  // the four waves that do not copy slices, two each, behind their MFMAs of the first slice: they have nothing to do from
  // there to the next barrier, and their copies do not enter the counted waits of the copying waves; they wait for them
  // (nothing else of theirs is outstanding) before the barrier of the tile's last slice.
  // (Tried at four slices, where a slice always lands in the same stage: the row panel left in the LDS across the tiles that share
  // it, its copies left out.  Since the copying waves then have the operands' copies too, it is the slower one: self-joins of 8,200 to
  // 17,000 points, d = 128, S = 30, lists 31 .. 66 us, 30 .. 64 without; counts 38 .. 69, 37 .. 67.)
#ifdef EJOIN_EXP_NO_COPIES
  bool aug_copied = false;
#endif
  auto issue_aug = [&](uint32_t I, uint32_t J) {
#ifdef EJOIN_EXP_NO_COPIES
    if (aug_copied) return;
    aug_copied = true;
#endif
    const char* ga = uniform_ptr(XbA + (int64_t)EJ_PANEL_A(I) * panel_stride + (int64_t)data_blocks * PANEL_BYTES);
    const char* gb = uniform_ptr(XbB + (int64_t)EJ_PANEL_B(J) * panel_stride + (int64_t)data_blocks * PANEL_BYTES);
    copy16_to_lds<AUG_OFF>(lds0 + cw * 1024, ga, voff0);
    copy16_to_lds<AUG_OFF + AUG_PART_BYTES>(lds0 + cw * 1024, gb, voff0 + AUG_PART_BYTES);
  };

  // --- fragment read addressing (byte offsets inside a stage).  Operands of v_mfma_f32_16x16x32_f16:
  // lane l supplies point l%16 of the fragment, coordinates 8*(l/16) .. +7 of the 32-wide step; in the
  // panel layout (see stored_at) that is row l%32 of the fragment's group of 32 rows, chunk 2 h + l/32
  // for fragment t = 2 T + h.  Group T adds 32 rows = 2048 B (swz unchanged: 32 rows = 8 groups of 4).
  // (= fragment_offset(lane, h) of panel_layout.h on top of the wave's first row)
  uint32_t offA[2], offB[2];
  {
    const int rowA = wm * 128 + (lane & 31), rowB = wn * 64 + (lane & 31);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      offA[h] = lds0 + rowA * 64 + (((2 * h + (lane >> 5)) ^ swz(rowA)) << 4);
      offB[h] = lds0 + PANEL_BYTES + rowB * 64 + (((2 * h + (lane >> 5)) ^ swz(rowB)) << 4);
    }
  }
  // Operands of the augmentation step (one v_mfma_f32_32x32x16_f16 per 32 x 32 region, see there): lane l
  // supplies row (or column) m = l%32 of the region, k = 8*(l/32) .. +7, and finds its 16 bytes ready made in
  // the LDS (panel_layout.h, "the augmentation step"): the A operand in the A part of the tile's augmentation
  // buffer, row m (chunk 0, k = 0..7) or, for k = 8..15, the constant chunk chosen by bit 3 of m (chunk 2 or 3);
  // the B operand the constant chunk chosen by bit 4 of m (k = 0..7) or column m of the B part (chunk 1,
  // k = 8..15).  Region t adds 32 rows = AUG_REGION_STEP in either place.
  const uint32_t offA_aug = lds0 + AUG_OFF + aug_lds_offset_a(lane, wm * 128);
  const uint32_t offB_aug = lds0 + AUG_OFF + aug_lds_offset_b(lane, wn * 64);
  typedef const __attribute__((address_space(3))) char* lds_cptr;
  typedef const __attribute__((address_space(3))) half8* lds_h8ptr;
  // fragment t (points 16 t .. 16 t + 15 of the wave tile's rows or columns); off: offA or offB (+ stage offset)
  auto frag = [&](uint32_t stage_off, const uint32_t (&off)[2], int t) -> half8 {
    return *reinterpret_cast<lds_h8ptr>((lds_cptr)(uintptr_t)(off[t & 1] + stage_off) + (t >> 1) * 2048);
  };
  // augmentation operand of region t (points 32 t .. 32 t + 31); addr: offA_aug or offB_aug + stage offset
  auto aug_operand = [&](uint32_t addr, int t) -> half8 { return *reinterpret_cast<lds_h8ptr>((lds_cptr)(uintptr_t)addr + t * AUG_REGION_STEP); };

  // acc[mt][nt]: the 16 x 16 block at rows 16 mt, columns 16 nt of the wave tile
  float4v acc[8][4];
  // Four MFMAs: column block nt of half H of the wave tile (rows 64 H .. 64 H + 63); they share their B
  // operand.  (The 16x16x32 shape accumulates 32 products per accumulator access, against 16 for 32x32x16:
  // on operands that toggle, the chip's power limit allows it a 14 % higher rate.)
  auto mma4 = [&](auto first_c, auto h_c, auto nt_c, const half8 (&fa)[4], const half8& b) {
    constexpr bool FIRST = decltype(first_c)::value;
    constexpr int H = decltype(h_c)::value, NT = decltype(nt_c)::value;
    const float4v z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int t = (NT & 1) ? 3 - u : u;  // up, down, up, down: only one operand changes from one MFMA to the next
      acc[4 * H + t][NT] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa[t], b, FIRST ? z : acc[4 * H + t][NT], 0, 0, 0);
    }
  };
  // scheduling hints: one LDS read, then `M` MFMAs.  The reads of a half step are spread one by one between
  // its MFMAs (two reads in a row already cost 2-3 %: the MFMA pipe runs dry while the wave issues them).
  auto read_then_mfma = [&](auto m_c) {
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, decltype(m_c)::value, 0);
  };

  // --- per-wave result staging (pair mode): entries are appended in LDS and written out in bulk
  // with one atomic per flush (wavefront ballot + prefix ranks + one atomic per wavefront flush).
  uint32_t* stg = reinterpret_cast<uint32_t*>(lds + STG_OFF + wave * STG_WAVE_BYTES);
  uint32_t fill = 0;               // wave-uniform
  unsigned long long hits = 0;     // count mode: pairs found by this wave
  bool dirty = false;              // stores/atomics issued by the rare path of the current tile (see there)
  // What only storing results needs is read from the kernel's arguments again where it is needed (`a` lies at their start): kept
  // across the main loop it costs scalar registers, whose spills are read back at every tile.  Together with the fillings
  // of the queue after the first in code of their own (below): 10^6 points, d = 128, on operands that hardly toggle (no power
  // limit) 86.7 ms, now 84.0; 10^5 points, d = 128, S = 64 1.5 % less.
  auto arguments = []() {
    auto ka = (const __attribute__((address_space(4))) JoinArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(ka));
    return ka;
  };
  auto store_staged = [&](unsigned long long base) {  // the staged entries to places base .. of the result
    const auto ka = arguments();
    for (uint32_t e = lane; e < fill; e += 64) {
      const unsigned long long idx = base + e;
      if (idx < ka->capacity) {
        reinterpret_cast<uint2*>(ka->pairs)[idx] = make_uint2(stg[3 * e], stg[3 * e + 1]);
        if (ka->dist2) ka->dist2[idx] = __uint_as_float(stg[3 * e + 2]);
      }
    }
  };
  auto flush = [&]() {
    if (fill == 0) return;
    unsigned long long base = 0;
    const auto ka = arguments();
    if (lane == 0) base = atomicAdd(ka->n_pairs, (unsigned long long)fill);
    const uint32_t blo = __builtin_amdgcn_readfirstlane((uint32_t)base);
    const uint32_t bhi = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32));
    store_staged(((unsigned long long)bhi << 32) | blo);
    fill = 0;
    dirty = true;
  };
  if constexpr (COUNT)  // (count mode stages nothing: the area holds the counters of dense wave tiles, 128 rows and 64 columns)
    for (int q = 0; q < 3; ++q) stg[64 * q + lane] = 0;
  // appends one entry per lane of `mask` to the staging area
  auto append = [&](unsigned long long mask, bool pass, uint32_t i, uint32_t j, uint32_t d2_bits) {
    const uint32_t cnt = __popcll(mask);
    if (fill + cnt > STG_CAP) flush();
    const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
    if (pass) {
      const uint32_t e = fill + rank;
      stg[3 * e] = i;
      stg[3 * e + 1] = j;
      stg[3 * e + 2] = d2_bits;
    }
    fill += cnt;
  };
  // --- candidate queue of the rare path: entry e is the 16 registers of one lane for one 32 x 32 region (queue_v[16 e ..])
  // and where they belong: row offset | column offset << 16 inside the wave tile (queue_t[e])
  float* queue_v = reinterpret_cast<float*>(lds + STG_OFF + wave * STG_WAVE_BYTES + STG_CAP * 12);
  uint32_t* queue_t = reinterpret_cast<uint32_t*>(queue_v + 16 * QUEUE_CAP);

  // ---------------- prologue
  TileCursor tc;
  tc.init(blockIdx.x, gridDim.x, (uint32_t)a.self, a.ntilesA, a.ntilesB, a.sb_row_begin, a.sb_row_end);
  // the tile being computed and the two after it (the copies run up to two tiles ahead, see issue_one)
  uint32_t I = 0, J = 0, In = 0, Jn = 0, In2 = 0, Jn2 = 0;
  bool have = tc.next(I, J);
  // a workgroup that leaves (now, or after its last tile) releases every later alignment of its XCD
  auto xcd_leave = [&]() {
    if (a.sync_mode >= 1 && tid == 0) __hip_atomic_fetch_add(a.xcd_bar + tc.xcd, 1u << 24, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  if (!have) {
    xcd_leave();
    return;
  }
  bool have_next = tc.next(In, Jn);
  bool have_next2 = have_next && tc.next(In2, Jn2);
  uint32_t epoch = 0;
  // tiles until the next re-alignment of the XCD's workgroups (never: a count no workgroup reaches)
  uint32_t sync_left = a.sync_mode >= 1 ? (uint32_t)a.sync_mode : 0xFFFFFFFFu;
  if (a.sync_mode >= 1) xcd_align(a.xcd_bar + tc.xcd, tc.wpx * ++epoch);
  uint32_t G = 0;  // slices computed so far (stage = G % NSTAGE); slices issued so far = G + DIST
  // The issue cursor runs DIST slices ahead of the compute cursor: slice `iks` (0 .. nsl-1) of the tile
  // `ahead` tiles after the one being computed.  With nsl >= 2 and DIST <= 3 that is at most two tiles ahead
  // (two when a tile has no more slices than are in flight: d <= 96).  After the last tile it keeps issuing
  // copies of valid memory into the dump area.
  int iks = 0;
  int ahead = 0;
  bool issue_live = true;       // the issue cursor points at real work
  const char* pa = XbA + (int64_t)EJ_PANEL_A(I) * panel_stride;
  const char* pb = XbB + (int64_t)EJ_PANEL_B(J) * panel_stride;
  const uint32_t lds_w = lds0 + cw * 1024;
  auto issue_one = [&](uint32_t Gissue) {
    if (!copier) return;
#ifdef EJOIN_EXP_NO_COPIES
    if (Gissue >= (uint32_t)NSTAGE) return;
#endif
    if (issue_live) {
      issue_slice(pa, pb, lds_w + (Gissue % NSTAGE) * STAGE_BYTES);
    } else {
#pragma unroll
      for (int q = 0; q < NCOPY; ++q) copy16_to_lds<0>(lds0 + DUMP_OFF, XbA, lane * 16);
    }
    pa += PANEL_BYTES;
    pb += PANEL_BYTES;
    ++iks;
    if constexpr (SPLIT) {
      if (iks == third) pb -= (int64_t)third * PANEL_BYTES;           // B' = [hi | hi | lo]
      if (iks == 2 * third) pa -= (int64_t)(2 * third) * PANEL_BYTES;  // A' = [hi | lo | hi]
    }
    if (iks == nsl) {
      iks = 0;
      ++ahead;
      const bool first_after = ahead == 1;
      issue_live = first_after ? have_next : have_next2;
      const uint32_t ti = first_after ? In : In2, tj = first_after ? Jn : Jn2;
      pa = XbA + (int64_t)(issue_live ? EJ_PANEL_A(ti) : 0) * panel_stride;
      pb = XbB + (int64_t)(issue_live ? EJ_PANEL_B(tj) : 0) * panel_stride;
    }
  };
  for (int q = 0; q < DIST; ++q) issue_one(q);
  // slice 0 has landed when only the copies of the DIST-1 younger slices (NCOPY per slice and copying wave) are
  // outstanding (the waves that do not copy have nothing outstanding: their waits pass at once)
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NCOPY * (DIST - 1)) : "memory");
  __syncthreads();
  using T_ = std::true_type;
  using F_ = std::false_type;
  using I0_ = std::integral_constant<int, 0>;
  using I1_ = std::integral_constant<int, 1>;
  using I2_ = std::integral_constant<int, 2>;
  using I3_ = std::integral_constant<int, 3>;
  using I4_ = std::integral_constant<int, 4>;
  using I6_ = std::integral_constant<int, 6>;
  // Fragment registers: the A fragments of the two halves of the wave tile and the four B fragments.  A slice
  // starts with faL and fb[0..2] in registers (read under the slice before); fb[3] and faH follow under its first half.
  half8 faL[4], faH[4], fb[4];
  auto load_first = [&](uint32_t stage_off) {
#pragma unroll
    for (int t = 0; t < 4; ++t) faL[t] = frag(stage_off, offA, t);
#pragma unroll
    for (int t = 0; t < 3; ++t) fb[t] = frag(stage_off, offB, t);
  };
  load_first(0);

  // One slice (G-th of the stream) = one 32-wide step: 32 MFMAs, upper half of the wave tile then lower half, each
  // column block by column block.  A B fragment is dead after its four MFMAs of the lower half, and the fragment of
  // the next slice is read into its place right away; the A fragments of the upper half are re-read under the lower
  // half.  FIRST: first slice of a tile (accumulators start from zero).  oa, ob: lane addresses of this slice's
  // fragments, oa_n, ob_n: of the next slice's, which the barrier of this slice has certified.
  auto mma_slice = [&](auto first_c, auto last_c, uint32_t st_cur, uint32_t st_nxt) {
    constexpr bool LAST = decltype(last_c)::value;
    fb[3] = frag(st_cur, offB, 3);
#pragma unroll
    for (int t = 0; t < 4; ++t) faH[t] = frag(st_cur, offA, 4 + t);
    mma4(first_c, I0_{}, I0_{}, faL, fb[0]);
    mma4(first_c, I0_{}, I1_{}, faL, fb[1]);
    mma4(first_c, I0_{}, I2_{}, faL, fb[2]);
    mma4(first_c, I0_{}, I3_{}, faL, fb[3]);
    read_then_mfma(I3_{});
    read_then_mfma(I3_{});
    read_then_mfma(I3_{});
    read_then_mfma(I3_{});
    read_then_mfma(I4_{});
    __builtin_amdgcn_sched_barrier(0);  // keep the two halves apart: each has its own interleave pattern
    if constexpr (!LAST) {
      faL[0] = frag(st_nxt, offA, 0);
      faL[1] = frag(st_nxt, offA, 1);
      mma4(first_c, I1_{}, I0_{}, faH, fb[0]);
      fb[0] = frag(st_nxt, offB, 0);
      faL[2] = frag(st_nxt, offA, 2);
      mma4(first_c, I1_{}, I1_{}, faH, fb[1]);
      fb[1] = frag(st_nxt, offB, 1);
      faL[3] = frag(st_nxt, offA, 3);
      mma4(first_c, I1_{}, I2_{}, faH, fb[2]);
      fb[2] = frag(st_nxt, offB, 2);
      mma4(first_c, I1_{}, I3_{}, faH, fb[3]);
      read_then_mfma(I2_{});
      read_then_mfma(I2_{});
      read_then_mfma(I2_{});
      read_then_mfma(I2_{});
      read_then_mfma(I2_{});
      read_then_mfma(I2_{});
      read_then_mfma(I4_{});
    } else {
      // the augmentation step follows: its six operands go where the fragments would
      // (faL[t]: A operand of region t, fb[0], fb[1]: B operands)
      const uint32_t oa_n = offA_aug, ob_n = offB_aug;
      faL[0] = aug_operand(oa_n, 0);
      faL[1] = aug_operand(oa_n, 1);
      mma4(first_c, I1_{}, I0_{}, faH, fb[0]);
      fb[0] = aug_operand(ob_n, 0);
      faL[2] = aug_operand(oa_n, 2);
      mma4(first_c, I1_{}, I1_{}, faH, fb[1]);
      fb[1] = aug_operand(ob_n, 1);
      faL[3] = aug_operand(oa_n, 3);
      mma4(first_c, I1_{}, I2_{}, faH, fb[2]);
      mma4(first_c, I1_{}, I3_{}, faH, fb[3]);
      read_then_mfma(I2_{});
      read_then_mfma(I2_{});
      read_then_mfma(I2_{});
      read_then_mfma(I2_{});
      read_then_mfma(I2_{});
      read_then_mfma(I6_{});
    }
  };
  // One slice.  LAST: last slice of a tile (what is read ahead are the operands of the augmentation step).
  // COPIER: the instance the copying waves run; the other waves run one without any copy code in it
  // (the copy instructions are opaque to the scheduler and would break up the MFMA / LDS-read interleave for nothing).
  auto data_slice = [&](auto first_c, auto last_c, auto copier_c) {
    constexpr bool FIRST = decltype(first_c)::value;
    constexpr bool COPIER = decltype(copier_c)::value;
    const uint32_t st_cur = (G % NSTAGE) * STAGE_BYTES, st_nxt = ((G + 1) % NSTAGE) * STAGE_BYTES;
    // (a) this wave's copies of slice G+1 have landed once only those of slice G+2 are outstanding.
    //     The waves that do not copy slices have at most the tile's augmentation copies outstanding, which must have
    //     landed before the barrier of the last slice.
    constexpr bool LAST_ = decltype(last_c)::value;
    if constexpr (COPIER) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NCOPY * (DIST - 2)) : "memory");
    else if constexpr (LAST_) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    // (b) after the barrier slice G+1 is complete in LDS for everybody, and everybody is done with slice G-1
    wg_barrier();
    // (c) the copying waves refill the stage slice G-1 occupied with slice G+DIST, while the other wave of
    //     their SIMD starts on the MFMAs of the slice
    if constexpr (COPIER) issue_one(G + DIST);
    // (d) the MFMAs of slice G, overlapped with the LDS reads of what follows
    mma_slice(first_c, last_c, st_cur, st_nxt);
    if constexpr (!COPIER && FIRST) issue_aug(I, J);
    ++G;
  };

#ifdef EJOIN_EXP_CYCLE_MARKS
  // sections: 0 tile cursor, 1 first slice, 2 middle slices, 3 last slice, 4 augmentation MFMAs + filter + exact path,
  // 5 reads of the next tile's first fragments (a mark waits for them to arrive: the section is their latency),
  // 6 the periodic re-alignment of the XCD's workgroups, 7 the wait for all copies in flight before it
  unsigned long long mark_sum[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  unsigned long long mark_prev = __builtin_amdgcn_s_memtime();
#define EJ_MARK(k)                                                  \
  {                                                                 \
    const unsigned long long now_ = __builtin_amdgcn_s_memtime();   \
    mark_sum[k] += now_ - mark_prev;                                \
    mark_prev = now_;                                               \
  }
#else
#define EJ_MARK(k)
#endif
  while (have) {
    // ---------------- the nsl >= 2 slices of the tile
    EJ_MARK(0)
    if (copier) {
      data_slice(T_{}, F_{}, T_{});
      EJ_MARK(1)
      for (int ks = 1; ks < nsl - 1; ++ks) data_slice(F_{}, F_{}, T_{});
      EJ_MARK(2)
      data_slice(F_{}, T_{}, T_{});
    } else {
      data_slice(T_{}, F_{}, F_{});
      EJ_MARK(1)
      for (int ks = 1; ks < nsl - 1; ++ks) data_slice(F_{}, F_{}, F_{});
      EJ_MARK(2)
      data_slice(F_{}, T_{}, F_{});
    }
    EJ_MARK(3)
    // ---------------- the augmentation step, then the filter.
    // The step adds -s_i/2 - s_j/2 to every accumulator with eight v_mfma_f32_32x32x16_f16, one per 32 x 32
    // region of the wave tile, half the matrix-core time that 32 more 16x16x32 (with 26 of 32 products zero)
    // would take.  A region's accumulator is its four 16 x 16 blocks' registers side by side, R = (mt2, nt2):
    // register q = 8 a + 4 c + r of lane l holds the pair  i = 16 a + 4 (l/16) + r,  j = 16 c + l%16  of the
    // region, where the 32 x 32 MFMA puts its element  m = 8 (q/4) + 4 (l/32) + q%4,  n = l%32.  So the step
    // needs  D[m][n] = -s_i/2 - s_j/2  with  i = i(m; bit 4 of n),  j = j(n%16; bit 3 of m),  which is bilinear
    // in indicator columns:  row m of the A operand = { P(i(m;0)), P(i(m;1)), c [bit3(m)=0], c [bit3(m)=1] },
    // row n of the B operand = { c [bit4(n)=0], c [bit4(n)=1], P(j(n;0)), P(j(n;1)) }, where P(x) = {p1, p2, p3, 0}
    // are the pieces of -s_x/2 and c stands for {c, c, c, 0}.  Of the 16 products of an element 6 are non-zero
    // and each is exact, as in a plain { P, c } . { c, P } step.
    float16v R[4][2];
    {
#pragma unroll
      for (int mt2 = 0; mt2 < 4; ++mt2)
#pragma unroll
        for (int nt2 = 0; nt2 < 2; ++nt2)
          R[mt2][nt2] = __builtin_amdgcn_mfma_f32_32x32x16_f16(
              faL[mt2], fb[nt2], cat4(acc[2 * mt2][2 * nt2], acc[2 * mt2][2 * nt2 + 1], acc[2 * mt2 + 1][2 * nt2], acc[2 * mt2 + 1][2 * nt2 + 1]),
              0, 0, 0);
    }
    {
      // acc' = a_ij - s_i/2 - s_j/2 = -dist^2/2 ; register r of block (mt, nt) in lane l is the pair
      //   i = I*256 + wm*128 + mt*16 + 4*(l/16) + r ,  j = J*256 + wn*64 + nt*16 + l%16.
      const bool diag = a.self && (I == J);
      // a wave tile of a diagonal block that lies entirely below the diagonal holds no pair i <= j
      const bool skip = diag && (wm * 128 >= wn * 64 + 64);
      // cheap filter: which of the eight 32 x 32 regions of this wave tile (2 x 2 blocks each, bit mt2*2 + nt2)
      // hold a passing pair at all
      const uint32_t thr_bits = __float_as_uint(a.thr) | 0x80000000u;
      uint32_t blocks_hit = 0;
      uint32_t least[8];  // per lane: smallest of the region's sixteen patterns
      {
        // x >= thr for a threshold thr <= 0 reads, on the bit patterns taken as unsigned integers, bits(x) <=
        // bits(thr) with thr's sign bit set: a positive x has a smaller pattern than any negative number, and a
        // negative one passes iff its magnitude is at most |thr|.  (A NaN with a clear sign bit would be flagged;
        // the exact path below compares as floats and drops it.)  Integer minima need no NaN quieting, which
        // costs the float version two more instructions per region.
#pragma unroll
        for (int mt2 = 0; mt2 < 4; ++mt2) {
#pragma unroll
          for (int nt2 = 0; nt2 < 2; ++nt2) {
            const float16v& v = R[mt2][nt2];
            auto u = [&](int r) { return __float_as_uint(v[r]); };
            uint32_t m = min(min(u(0), u(1)), u(2));
#pragma unroll
            for (int r = 3; r < 15; r += 2) m = min(min(m, u(r)), u(r + 1));
            m = min(m, u(15));
            least[mt2 * 2 + nt2] = m;
            if (__ballot(m <= thr_bits)) blocks_hit |= 1u << (mt2 * 2 + nt2);
          }
        }
        // the filter of a region only needs that region's MFMA: let the VALU work of a region run
        // under the augmentation MFMAs of the regions after it
        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
#pragma unroll
        for (int b = 0; b < 6; ++b) {
          __builtin_amdgcn_sched_group_barrier(0x002, 9, 0);
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        }
      }
#ifdef EJOIN_ABL_NOPREFILTER
      blocks_hit = 0xFF;
#endif
#ifdef EJOIN_EXP_NO_COPIES
      blocks_hit = 0;  // (every tile holds the first tile's distances: keep the rare path out of the comparison)
#endif
      if (skip) blocks_hit = 0;
      // Rare path.  What bounds it is instruction issue: two wavefronts share a SIMD, both are here at the same time, and every
      // vector instruction costs them eight cycles together.  So no register is tested one by one where it lies: the lanes that
      // hold a candidate (in a flagged region usually one) queue the sixteen registers of their region in the LDS with four
      // 16-byte stores, and the queue is then looked at four entries at a time, one value per lane, by code that exists once.
      // A ballot and branch per register of a flagged region instead, as before: n = 10^5, d = 128, 43 hits per tile 1676 us
      // against 1430 now, n = 3 10^5, d = 384, 56 hits per tile 28.0 ms against 25.9.  (A bit mask per lane, one hit of every
      // lane per round picked out of the sixteen registers by selects: 1768 us on the first.)
      if (diag && !COUNT && wave < 4) {  // (i, i) belongs to the result by definition, whatever the arithmetic says
        const uint32_t i = I * TILE + tid;
        append(__ballot(i < (uint32_t)a.nA), i < (uint32_t)a.nA, i, i, 0u);
      }
      uint32_t l = lane;
      if constexpr (DENSE) asm volatile("" : "+v"(l));  // (this instance has no registers to keep what follows across the main loop)
      const uint32_t lr = l & 15u, lg = l >> 4;
      const uint32_t lane_tag = 4 * lg | (lr << 16);                                                  // region_pair(lane, 0)
      const uint32_t reg_tag = (16 * (lr >> 3) + (lr & 3)) | ((16 * ((lr >> 2) & 1)) << 16);  // ... of register lane % 16
      uint32_t todo = blocks_hit;  // regions not (completely) queued yet
      uint32_t taken = 0;          // lanes of the first of them that are
      uint32_t dense = 0;          // (DENSE) regions with candidates in many lanes
      // again_c: a filling after the first
      auto fill_queue = [&](auto again_c, uint32_t& todo, uint32_t& taken) -> uint32_t {
        uint32_t qfill = 0;
        uint32_t now = todo;
#pragma unroll
        for (int b = 0; b < 8; ++b) {
          if (!(now & (1u << b))) continue;
          const float16v& v = R[b >> 1][b & 1];
#ifdef EJOIN_ABL_NOPREFILTER
          const bool has = true;
#else
          bool has = least[b] <= thr_bits;
          if constexpr (decltype(again_c)::value) {
            uint32_t h = has;
            asm volatile("" : "+v"(h));  // (else what both fillings compute is moved ahead of the first, for all eight regions)
            has = h != 0;
          }
#endif
          const unsigned long long lanes = __ballot(has);
          if (DENSE && __popcll(lanes) >= DENSE_LANES) {
            dense |= 1u << b;
            todo &= ~(1u << b);
            continue;
          }
          const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(lanes >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)lanes, 0u));
          const uint32_t e = qfill + rank - taken;  // (a lane already taken: e wraps around or lies below qfill)
          if (has && rank >= taken && e < (uint32_t)QUEUE_CAP) {
            float4v* q = reinterpret_cast<float4v*>(queue_v + 16 * e);
            q[0] = __builtin_shufflevector(v, v, 0, 1, 2, 3);
            q[1] = __builtin_shufflevector(v, v, 4, 5, 6, 7);
            q[2] = __builtin_shufflevector(v, v, 8, 9, 10, 11);
            q[3] = __builtin_shufflevector(v, v, 12, 13, 14, 15);
            queue_t[e] = lane_tag + (uint32_t)(32 * (b >> 1) + ((32 * (b & 1)) << 16));
          }
          const uint32_t left = __popcll(lanes) - taken, room = QUEUE_CAP - qfill;
          if (left <= room) {
            qfill += left;
            taken = 0;
            todo &= ~(1u << b);
          } else {  // the queue is full: look at it, then go on with this region
            qfill = QUEUE_CAP;
            taken += room;
            now = 0;
          }
        }
        return qfill;
      };
      auto drain_queue = [&](uint32_t qfill, auto lds_c) {  // lds_c: (count mode) into the counters in the LDS
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        const uint32_t nnA = (uint32_t)a.nA, nnB = (uint32_t)a.nB;
        // tiles in which a value that passes may not be a result: on the diagonal, or with rows or columns past the end
        // (those carry a large negative marker, which a huge epsilon can still reach)
        const bool partial = diag || (I + 1) * TILE > nnA || (J + 1) * TILE > nnB;
#pragma unroll 1
        for (uint32_t q0 = 0; q0 < qfill; q0 += 4) {
          const float x = queue_v[16 * q0 + l];
          const uint32_t at = queue_t[q0 + lg] + reg_tag;
          const uint32_t i = I * TILE + wm * 128 + (at & 0xFFFFu), j = J * TILE + wn * 64 + (at >> 16);
          bool pass = x >= a.thr && l < 16 * (qfill - q0);
          if (partial) pass = pass && i < nnA && j < nnB && (!diag || i < j);
          const unsigned long long mask = __ballot(pass);
          if (!mask) continue;
          if (COUNT) {
            if constexpr (decltype(lds_c)::value) {
              if (pass) {
                atomicAdd(stg + (at & 0xFFFFu), 1u);
                atomicAdd(stg + 128 + (at >> 16), 1u);
              }
            } else {
              if (pass) {
                atomicAdd(&a.counts[i], 1u);
                if (a.self) atomicAdd(&a.counts[j], 1u);
                else if (a.counts_b) atomicAdd(&a.counts_b[j], 1u);
              }
              dirty = true;
            }
            hits += __popcll(mask);
          } else {
            append(mask, pass, i, j, __float_as_uint(fmaxf(-2.f * x, 0.f)));
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      };
      if constexpr (!DENSE) {
        if (todo) {
          uint32_t qfill = fill_queue(F_{}, todo, taken);
          if (!todo) {
            drain_queue(qfill, F_{});
          } else {
            // A dense wave tile: more candidates than the queue takes.  Counts: its hits share rows and columns, and one global atomic
            // per hit and side is what such counts are bound by (28 10^9 a second), so they are added up in the LDS first.  Against
            // global atomics (and, in brackets, the ballot per register before the queue): 33,000 points, d = 128, S = 1,500
            // 2,230 (1,980) us, now 700; S = 4,000 5.4 (4.6) ms, now 1.0; 200,000 x 600, d = 384, S = 5,000 1,100 (750) us, now 290.
            // Wave tiles whose candidates fit the queue go on as they did: 10^6 points, d = 128, S = 64 109 ms on both.
            for (;;) {
              drain_queue(qfill, std::integral_constant<bool, COUNT>{});
              if (!todo) break;
              qfill = fill_queue(T_{}, todo, taken);
            }
            if constexpr (COUNT) {
              send_region_counts(stg, l, a, I * TILE + wm * 128, J * TILE + wn * 64);
              dirty = true;
            }
          }
        }
      } else {
        while (todo) drain_queue(fill_queue(F_{}, todo, taken), F_{});
      }
      if (DENSE && dense) {
        // Every lane looks at its own registers: a bit mask of those that pass, whose numbers per row and column are added up in
        // the wavefront's part of the LDS; the tile's go out with one atomic per row and column.
        const uint32_t nnA = (uint32_t)a.nA, nnB = (uint32_t)a.nB;
        const bool partial = diag || (I + 1) * TILE > nnA || (J + 1) * TILE > nnB;
        do {
          const int b = __builtin_ctz(dense);
          dense &= dense - 1;
          float16v v;
          switch (b) {
            case 0: v = R[0][0]; break;
            case 1: v = R[0][1]; break;
            case 2: v = R[1][0]; break;
            case 3: v = R[1][1]; break;
            case 4: v = R[2][0]; break;
            case 5: v = R[2][1]; break;
            case 6: v = R[3][0]; break;
            default: v = R[3][1]; break;
          }
          asm volatile("" : "+v"(v));  // one copy of the region's registers, in one place
          uint32_t hit = 0;
#pragma unroll
          for (int r = 0; r < 16; ++r) hit |= v[r] >= a.thr ? 1u << r : 0u;
          const uint32_t il = 32 * (b >> 1) + 4 * lg, jl = 32 * (b & 1) + lr;  // register 0's place in the wave tile
          const uint32_t i0 = I * TILE + wm * 128 + il, j0 = J * TILE + wn * 64 + jl;
          if (partial) hit &= keep_mask(i0, j0, nnA, nnB, diag);
          hits += wave_sum(__popc(hit));
          add_region_counts(hit, stg + il, stg + 128 + jl);
        } while (dense);
        send_region_counts(stg, l, a, I * TILE + wm * 128, J * TILE + wn * 64);
        dirty = true;
      }
      // The stores and atomics of the path count on vmcnt like the copies, but complete in any order: the counted
      // waits of the slices hold only once they are all done.
      if (dirty) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        dirty = false;
      }
    }
    EJ_MARK(4)
    // first fragments of the next tile (slice G was certified by the barrier of the tile's last slice);
    // read after the filter to keep its registers free
    load_first((G % NSTAGE) * STAGE_BYTES);
    EJ_MARK(5)
    I = In;
    J = Jn;
    have = have_next;
    In = In2;
    Jn = Jn2;
    have_next = have_next2;
    --ahead;  // (at least 1 before: the issue cursor has left the tile that was just finished)
    if (have) {
      if (--sync_left == 0) {
        sync_left = (uint32_t)a.sync_mode;
        EJ_MARK(0)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        EJ_MARK(7)
        xcd_align(a.xcd_bar + tc.xcd, tc.wpx * ++epoch);
        EJ_MARK(6)
      }
      have_next2 = have_next && tc.next(In2, Jn2);
    }
  }
#ifdef EJOIN_EXP_CYCLE_MARKS
  if (lane == 0 && !COUNT && a.capacity >= 16) {
    unsigned long long* out = reinterpret_cast<unsigned long long*>(a.pairs) + (a.capacity - 16) + 8 * (wave >> 2);
    for (int k = 0; k < 8; ++k) atomicAdd(out + k, mark_sum[k]);
  }
#endif
  xcd_leave();
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the dump copies must land before the wave ends
  // What is left, with one atomic for the workgroup: those on one address are served one after the other, about 11 ns each,
  // and all workgroups end at about the same time (2048 of them, one per wavefront: 23 us).  Every copy to the LDS has landed.
  // Measured: 500 x 200,000 points, d = 384, count: 87.6 us, now 74.2; 4,096 points, d = 128, 64 k pairs: 29.4 us, now 21.1.
  __syncthreads();
  unsigned long long* sums = reinterpret_cast<unsigned long long*>(lds);
  if (lane == 0) sums[wave] = COUNT ? hits : (unsigned long long)fill;
  __syncthreads();
  if (tid == 0) {
    unsigned long long total = 0;
    for (int w = 0; w < THREADS / 64; ++w) {
      const unsigned long long v = sums[w];
      sums[w] = total;
      total += v;
    }
    if (COUNT && total) atomicAdd(a.total, total);
    if (!COUNT) sums[THREADS / 64] = total ? atomicAdd(a.n_pairs, total) : 0ull;
  }
  if (!COUNT) {
    __syncthreads();
    store_staged(sums[THREADS / 64] + sums[wave]);
  }
}


// ------------------------------------------------------------------------------------------
// The join of points with few coordinates
// ------------------------------------------------------------------------------------------
// A workgroup holds a panel of 512 rows in registers for as long as its part of the schedule stays in them (StripCursor): a
// wavefront all K k-blocks of its 64 rows (16 K registers).  Only the columns go through the LDS, 64 (32) of them with all their
// k-blocks at a time, and a block of 64 rows x 32 columns per wavefront is complete after K steps, with 32 accumulators.
// What bounds k_join at few coordinates is the boundary of a tile (a third of its time at four slices) and, in long launches, power.
// Here a block's filter runs under the next block's MFMAs, there is no barrier (progress counters, below), the L2 -> LDS copies are a
// quarter of k_join's (512 rows share them, and only columns are copied) and the LDS reads 64 B per clock and CU at MFMA peak instead
// of 96 (d = 128).  Measured (join kernel): 10^6 points, d = 128, S = 64, counts 105.5 ms, now 91.5; 10^5 points, pairs 1383 us, now 1170 (output
// left out 1160, now 900: MFMA pipe busy 0.76 of the cycles, at the clock that the power limit leaves); 40,000 points, d = 224,
// pairs 296 us, now 276.  From eight k-blocks on there are no registers for two buffers of accumulators, and the filter is in the open:
// 150,000 points, d = 320, 5.33 ms, now 5.08.
// Tried: a barrier per stage (candidates of one wavefront hold up all: 10^5 x 128 1680 us); 256 rows and 64 columns a workgroup,
// copies by four of the wavefronts (10^6 x 128 without candidates 94 ms, now 91); volatile progress counters (every LDS read
// waited for: 110).
template <class F, int... N>
__device__ __forceinline__ void for_each_index(F&& f, std::integer_sequence<int, N...>) {
  (f(std::integral_constant<int, N>{}), ...);
}
template <int K>
struct Strip {
  static constexpr bool TWO = K <= 7;             // two blocks of 32 columns a stage and two buffers of accumulators; else one of each
  static constexpr int BLOCKS = TWO ? 2 : 1, COLS = 32 * BLOCKS;
  static constexpr int KB = COLS * 64;            // bytes of a k-block of a stage
  static constexpr int DATA = K * KB;             // bytes of coordinates ...
  static constexpr int STAGE = DATA + COLS * 16;  // ... and of operands of the augmentation step
  static constexpr bool ROWS_LDS = K >= 8;        // the rows' operands of that step: in the LDS, or in registers
  static constexpr int DENSE = 5, FULL = 24;      // (counts) candidates in that many lanes of 32 x 32: each lane looks at its own, all at once
  static constexpr int QUEUE = 16;                // entries of the candidate queue: 16 values and the place of the first
  static constexpr int STG = 128;                 // staged results
  static constexpr int WAVE = STG * 12 + QUEUE * 72;
  static constexpr int TAIL = 640;                // constant chunks of the augmentation step (at 0 and 512), progress counters
  static constexpr int ROWS = ROWS_LDS ? 8192 : 0;
  static constexpr int FIT = (160 * 1024 - 8 * WAVE - TAIL - ROWS) / STAGE;
  static constexpr int STAGES = FIT < 8 ? FIT : 8;
  static constexpr int DEPTH = STAGES >= 8 ? 5 : (STAGES >= 5 ? 3 : 2);  // stages the copies are ahead
  static constexpr int LAG = STAGES - DEPTH;      // a stage is refilled that many stages after its own
  static constexpr int POST = DEPTH >= 4 ? 2 : 1; // at the start of stage g the copies of stage g + POST have landed
  static constexpr int COPIES = TWO ? K + 1 : (K + 2) / 2;  // copy instructions per copying wavefront and stage
  // fragments of the columns in registers (two at eight and nine k-blocks: 65,000 points, d = 240, S = 64 with eight 0.99 ms of counts and
  // 0.95 of pairs, with three 0.96 and 0.93, now 0.95 and 0.92)
  static constexpr int RING = K >= 10 ? 3 : (K >= 8 ? 2 : (K == 4 ? 8 : (K == 3 || K == 6 ? 6 : 4)));
  static constexpr int CONST_OFF = STAGES * STAGE;
  static constexpr int SYNC_OFF = CONST_OFF + 64;
  static constexpr int ROWS_OFF = CONST_OFF + TAIL;
  static constexpr int STG_OFF = ROWS_OFF + ROWS;
  static constexpr int LDS = STG_OFF + 8 * WAVE;
  static_assert(STAGES >= 3 && LAG >= 1 && DEPTH > POST && LDS <= 160 * 1024, "LDS budget of one CU");
  static_assert(RING <= 2 * K, "what is read ahead belongs to this block or the next");
};

template <bool COUNT, int K>
__global__ __launch_bounds__(THREADS) void k_join_strip(const JoinArgs a) {
  using L = Strip<K>;
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  // the largest norm of the call has been consumed by k_aux: cleared here for the next call
  if (blockIdx.x == 0 && threadIdx.x == 0) a.status[1] = 0;
  if (*a.status != ST_OK) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t turn = (uint32_t)wave >> 2;  // who copies: wavefronts 0 .. 3 the even stages, 4 .. 7 the odd ones
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
  const int64_t panel_stride = (int64_t)(K + 1) * PANEL_BYTES;
  const char* XbB = reinterpret_cast<const char*>(a.XpB);
  if (tid < 4) {
    const uint32_t c0 = a.status[2], c1 = a.status[3];
    *reinterpret_cast<uint4*>(lds + L::CONST_OFF + 512 * (tid >> 1) + 16 * (tid & 1)) = tid & 1 ? make_uint4(0u, 0u, c0, c1) : make_uint4(c0, c1, 0u, 0u);
  }

  auto uniform_ptr = [](const char* p) -> const char* {
    const uint64_t b = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b), hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return reinterpret_cast<const char*>(((uint64_t)hi << 32) | lo);
  };

  // ---- per-wavefront staging of results, and the queue of candidates (see k_join)
  uint32_t* stg = reinterpret_cast<uint32_t*>(lds + L::STG_OFF + wave * L::WAVE);
  float* queue_v = reinterpret_cast<float*>(lds + L::STG_OFF + wave * L::WAVE + L::STG * 12);
  uint2* queue_t = reinterpret_cast<uint2*>(queue_v + 16 * L::QUEUE);  // the pair of the entry's first value
  uint32_t fill = 0, qfill = 0;  // (uniform)
  unsigned long long hits = 0;   // (uniform)
  bool dirty = false;  // stores or atomics issued since the last wait for everything
  auto arguments = []() {  // (read again where only the rare path needs them, see k_join)
    auto ka = (const __attribute__((address_space(4))) JoinArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(ka));
    return ka;
  };
  // At the end of what runs now and then: nothing of it is outstanding on lgkmcnt (scalar loads return in any order: with one of them
  // perhaps in flight, the compiler could only wait for everything at the next LDS read of the main loop, every time)
  auto settle = []() { __builtin_amdgcn_s_waitcnt(0xC07F); };
  auto store_staged = [&](unsigned long long base) __attribute__((always_inline)) {
    const auto ka = arguments();
    for (uint32_t e = lane; e < fill; e += 64) {
      const unsigned long long idx = base + e;
      if (idx < ka->capacity) {
        reinterpret_cast<uint2*>(ka->pairs)[idx] = make_uint2(stg[3 * e], stg[3 * e + 1]);
        if (ka->dist2) ka->dist2[idx] = __uint_as_float(stg[3 * e + 2]);
      }
    }
  };
  auto flush = [&]() __attribute__((always_inline)) {
    unsigned long long base = 0;
    const auto ka = arguments();
    if (lane == 0) base = atomicAdd(ka->n_pairs, (unsigned long long)fill);
    const uint32_t blo = __builtin_amdgcn_readfirstlane((uint32_t)base), bhi = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32));
    store_staged(((unsigned long long)bhi << 32) | blo);
    fill = 0;
    dirty = true;
  };
  auto stage_entry = [&](unsigned long long mask, bool pass, uint32_t i, uint32_t j, uint32_t d2_bits) __attribute__((always_inline)) {
    const bool swapped = a.swapped;
    const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
    if (pass) {
      const uint32_t e = fill + rank;
      stg[3 * e] = swapped ? j : i;
      stg[3 * e + 1] = swapped ? i : j;
      stg[3 * e + 2] = d2_bits;
    }
    fill = __builtin_amdgcn_readfirstlane(fill + __popcll(mask));
  };
  // Count mode: the staging area holds counters instead, of the wavefront's 64 rows (kept until its row panel changes) and of the
  // 32 columns of a block.
  uint32_t* const row_counts = stg;
  uint32_t* const col_counts = stg + 64;
  uint32_t rows_at = 0;  // first row of the counters
  if constexpr (COUNT) {
    stg[lane] = 0;
    if (lane < 32) col_counts[lane] = 0;
  }
  auto send_rows = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    const uint32_t c = row_counts[lane];
    hits += wave_sum(c & 0xFFFFu) + ((unsigned long long)wave_sum(c >> 16) << 16);  // (every pair found is in one row's counter)
    if (c) {
      row_counts[lane] = 0;
      uint32_t* to = arguments()->counts;
      if (to) atomicAdd(to + rows_at + lane, c);
    }
    dirty = true;
  };
  auto drain = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    uint32_t l = lane;
    asm volatile("" : "+v"(l));  // (nothing of this is kept across the main loop)
    const uint32_t nnA = (uint32_t)a.nA, nnB = (uint32_t)a.nB, self = (uint32_t)a.self;
    const uint32_t lr = l & 15u, roff = 16 * (lr >> 3) + (lr & 3), coff = 16 * ((lr >> 2) & 1);  // region_pair(0, lane % 16)
    const float thr = a.thr;
    // four entries a pass, one value per lane; with registers to spare the reads of all passes are in flight together
    constexpr int AT_ONCE = K <= 6 ? L::QUEUE / 4 : 1;
#pragma unroll 1
    for (uint32_t p = 0; p < L::QUEUE / 4; p += AT_ONCE) {
      float x[AT_ONCE];
      uint2 at[AT_ONCE];
#pragma unroll
      for (int q = 0; q < AT_ONCE; ++q) {
        x[q] = queue_v[64 * (p + q) + l];
        at[q] = queue_t[4 * (p + q) + (l >> 4)];
      }
#pragma unroll
      for (int q = 0; q < AT_ONCE; ++q) {
        const uint32_t i = at[q].x + roff, j = at[q].y + coff;
        const bool pass = x[q] >= thr && l + 64 * (p + q) < 16 * qfill && i < nnA && j < nnB && (!self || i < j);
        const unsigned long long mask = __ballot(pass);
        if (!mask) continue;
        if constexpr (COUNT) {
          if (pass) {
            atomicAdd(row_counts + (i - rows_at), 1u);
            const auto ka = arguments();
            uint32_t* to = self ? ka->counts : ka->counts_b;
            if (to) atomicAdd(to + j, 1u);
          }
          dirty = true;
        } else {
          if (fill + __popcll(mask) > (uint32_t)L::STG) flush();
          stage_entry(mask, pass, i, j, __float_as_uint(fmaxf(-2.f * x[q], 0.f)));
        }
      }
    }
    settle();
    qfill = 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };

  // ---- schedule.  The cursor is the copies', DEPTH stages ahead of what is computed; which stage a place of the ring holds (panel of
  // rows, 64 columns) is kept in one lane of two registers per place.
  StripCursor tc;
  tc.init(blockIdx.x, gridDim.x, (uint32_t)a.self, (uint32_t)((a.nB + EJ_STRIP_COLS - 1) / EJ_STRIP_COLS), a.sb_row_begin, a.sb_row_end);
  uint32_t run_i = 0, run_c = 0, run_end = 0;
  auto next_run = [&]() __attribute__((always_inline)) -> bool {
    constexpr uint32_t PER = EJ_STRIP_COLS / L::COLS;
    const bool some = tc.next(run_i, run_c, run_end);
    run_c *= PER;
    run_end *= PER;
    return some;
  };
  bool live = next_run();
  auto xcd_leave = [&]() {
    const auto ka = arguments();
    if (ka->sync_mode >= 1 && tid == 0)
      __hip_atomic_fetch_add(ka->xcd_bar + blockIdx.x % NUM_XCD, 1u << 24, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  if (!live) {
    xcd_leave();
    return;
  }
  uint32_t epoch = 0;
  uint32_t sync_left = a.sync_mode >= 1 ? (uint32_t)a.sync_mode : 0xFFFFFFFFu;
  if (a.sync_mode >= 1) xcd_align(a.xcd_bar + blockIdx.x % NUM_XCD, tc.step * ++epoch);
  constexpr uint32_t NO_STAGE = 0xFFFFFFFFu;
  uint32_t places = 0;             // lane p: the columns of place p, lane 32 + p: its panel of rows
  uint32_t slot_in = 0, slot = 0;  // where the next stage goes; the stage being computed
  uint32_t g = 0, g_in = 0;        // their numbers
  const uint32_t quarter = wave & 3;
  const uint32_t voff = lane * 16 + (L::TWO ? quarter * 1024 : (quarter & 1) * 1024 + (quarter >> 1) * PANEL_BYTES);
  // The next stage.  64 columns: wavefront q of the four copies the q-th KB of every 4 KB (one k-block) and a quarter of the
  // augmentation operands.  32 columns: the q-th KB of every two k-blocks, and what then lacks to the same number for all four.
  auto issue = [&]() __attribute__((always_inline)) {
    places = lane == (int)slot_in ? (live ? run_c : NO_STAGE) : places;
    if (__builtin_expect(live, 1)) {
      places = lane == (int)slot_in + 32 ? run_i : places;
      if ((g_in & 1) == turn) {
        constexpr uint32_t PER = TILE / L::COLS;  // stages of a panel of columns
        const char* panel = uniform_ptr(XbB + (int64_t)(run_c / PER) * panel_stride);
        const char* src = panel + (run_c % PER) * (uint32_t)(L::COLS * 64);
        const uint32_t at = __builtin_amdgcn_readfirstlane(lds0 + slot_in * (uint32_t)L::STAGE);
        const char* aug = panel + (int64_t)K * PANEL_BYTES + AUG_PART_BYTES + (run_c % PER) * (uint32_t)(L::COLS * 16);
        for_each_index([&](auto n_c) {
          constexpr int N = decltype(n_c)::value;
          copy16_to_lds<N * 4096>(at + quarter * 1024, uniform_ptr(src + (int64_t)N * (L::TWO ? 1 : 2) * PANEL_BYTES), voff);
        }, std::make_integer_sequence<int, L::TWO ? K : K / 2>{});
        if constexpr (L::TWO || K % 2 == 0) {  // a quarter of the augmentation operands
          if (lane < L::COLS / 4) copy16_to_lds<L::DATA>(at + quarter * (L::COLS * 4), uniform_ptr(aug + quarter * (L::COLS * 4)), lane * 16);
        } else if (quarter < 2) {  // the last k-block
          copy16_to_lds<K / 2 * 4096>(at + quarter * 1024, uniform_ptr(src + (int64_t)(K - 1) * PANEL_BYTES), voff);
        } else {  // half of the augmentation operands
          if (lane < L::COLS / 2) copy16_to_lds<L::DATA>(at + (quarter - 2) * (L::COLS * 8), uniform_ptr(aug + (quarter - 2) * (L::COLS * 8)), lane * 16);
        }
      }
      if (__builtin_expect(++run_c == run_end, 0)) live = next_run();
    }
    slot_in = slot_in == L::STAGES - 1 ? 0 : slot_in + 1;
    ++g_in;
  };
  // ---- Progress of the wavefronts, in the LDS: word w says that wavefront w's copies of all stages below it have landed, word
  // 8 + w how many stages wavefront w has read.  A wavefront reads a stage when all of it has landed, and its place is refilled when
  // all have read it.  (A barrier per stage instead makes all of them wait for the one that has candidates to look at.)
  // (volatile accesses would make the compiler wait for every LDS read in flight)
  typedef __attribute__((address_space(3))) uint32_t* lds_u32ptr;
  const uint32_t sync0 = lds0 + L::SYNC_OFF;
  uint32_t look_at = sync0 + 4 * (lane & 15);
  if constexpr (L::TWO) asm volatile("" : "+v"(look_at));  // (kept in a register where there is one)
  auto sync_word = [&](uint32_t w) { return (lds_u32ptr)(uintptr_t)(sync0 + 4 * w); };
  if (tid < 16) *sync_word(tid) = tid < 8 ? L::POST + (((tid >> 2) & 1) != (L::POST & 1)) : 0;
  // a lane's word plus `lead` must not lie below g + 2 when stage g + 1 is about to be read, and then the place of stage g + 1 - LAG refilled
  const uint32_t lead = lane < 8 ? 0u : (lane < 16 ? (uint32_t)L::LAG : 0x40000000u);
  uint32_t seen = 0;  // this lane's word, read a while ago
  auto look = [&]() {
    asm volatile("" ::: "memory");
    seen = *(lds_u32ptr)(uintptr_t)look_at;
  };
  auto proceed = [&]() {
    if (__builtin_expect(__ballot((int32_t)(seen + lead - (g + 2)) < 0) != 0, 0)) {
      do look();
      while (__ballot((int32_t)(seen + lead - (g + 2)) < 0));
      settle();
    }
    asm volatile("" ::: "memory");
  };
  auto post_read = [&]() {  // every read of stage g has been issued, and the LDS serves a wavefront's instructions in order
    asm volatile("" ::: "memory");
    if (lane == 0) *sync_word(8 + wave) = g + 1;
    asm volatile("" ::: "memory");
  };
  // Start of stage g: the copies of stage g + POST, if they were this wavefront's, have landed once only those of its younger stages are
  // outstanding.  (Stores and atomics count on vmcnt like the copies, but complete in any order: with some of them issued since, once
  // nothing at all is.  Waiting for them where they are issued instead holds up every block that has candidates, in counts of many
  // neighbours all of them: 33,000 points, d = 60, S = 100 225 us, now 200; 65,000, d = 96, S = 400 1.02 ms, now 0.88.)
  auto begin_stage = [&]() __attribute__((always_inline)) {
    if (((g + L::POST) & 1) == turn) {
      if (__builtin_expect(live && !dirty, 1)) {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(L::COPIES * ((L::DEPTH - 1 - L::POST) / 2)) : "memory");
      } else {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        dirty = false;
      }
      if (lane == 0) *sync_word(wave) = g + L::POST + 2;
    }
    issue();  // stage g + DEPTH
  };

  // ---- operands.  Fragment h of the columns of a stage's block P, k-block kb: stage + kb * KB + 2048 P + fragment_offset(lane, h)
  typedef const __attribute__((address_space(3))) char* lds_cptr;
  typedef const __attribute__((address_space(3))) half8* lds_h8ptr;
  auto at_lds = [&](uint32_t addr, int imm) -> half8 { return *reinterpret_cast<lds_h8ptr>((lds_cptr)(uintptr_t)addr + imm); };
  const uint32_t off0 = lds0 + fragment_offset(lane, 0);  // (fragment_offset(lane, 1): bit 5 the other way)
  // augmentation operand of the columns: their pieces in the stage (lanes 32 .. 63) or the constant chunk; of the rows: the
  // wavefront's part of the rows' area (lanes 0 .. 31) or the constant chunk, 512 bytes further on for the second 32 rows
  // (swapped: the two halves of the step the other way round, so that it adds the points' terms before the query points' as ever)
  const bool upper = (lane >= 32) != (a.swapped != 0);
  const uint32_t aug0 = lds0 + (upper ? L::DATA + 16 * (lane & 31) : L::CONST_OFF + 16 * ((lane >> 4) & 1));
  const uint32_t aug_step = upper ? ~0u : 0u;
  const uint32_t aug_rows = lds0 + (upper ? L::CONST_OFF + 16 * ((lane >> 3) & 1) : L::ROWS_OFF + 1024 * wave + 16 * (lane & 31));
  constexpr int RING = L::RING, FRAGS = 2 * K;
  half8 fa[K][4], ga[2], fb[RING];
  float16v R[L::BLOCKS][2];  // [buffer][32 rows]: a region's four 16 x 16 blocks side by side
  if constexpr (L::TWO)
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int q = 0; q < 16; ++q) R[L::BLOCKS - 1][r][q] = __uint_as_float(0xFFFFFFFFu);  // (above every threshold's pattern: nothing to look at before the first block)
  const uint32_t thr_bits = __float_as_uint(a.thr) | 0x80000000u;  // (x >= thr on the bit patterns, see k_join)
  uint32_t pend_i = 0, pend_j = 0;  // place of the block that the filter looks at next

  // Rare path: candidates of the block in buffer P.  The lanes that hold one queue their sixteen values (see k_join); the queue is
  // looked at when it is full.
  auto rare = [&](auto p_c, uint32_t least0, uint32_t least1) __attribute__((always_inline)) {
    constexpr int P = decltype(p_c)::value;
    if constexpr (COUNT) {
      if (rows_at != pend_i) {
        if (qfill) drain();
        send_rows();
        rows_at = pend_i;
        settle();
      }
    }
    uint32_t l = lane;
    asm volatile("" : "+v"(l));
    const uint32_t in_i = 4 * (l >> 4), in_j = pend_j + (l & 15u);
    uint32_t todo = 0;  // regions that did not fit
    bool columns = false;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const float16v& v = R[P][r];
      const bool has = (r ? least1 : least0) <= thr_bits;
      const unsigned long long lanes = __ballot(has);
      const uint32_t cnt = __popcll(lanes);
      if (cnt == 0) continue;
      if (COUNT && cnt >= (uint32_t)L::DENSE) {
        // many candidates: every lane looks at its own, and the numbers are added up in the LDS
        const uint32_t self = (uint32_t)a.self, i0 = pend_i + 32 * r + in_i;
        uint32_t hit = 0;
#pragma unroll
        for (int q = 0; q < 16; ++q) hit |= v[q] >= a.thr ? 1u << q : 0u;
        if ((self && pend_j < pend_i + 64) || pend_i + 64 > (uint32_t)a.nA || pend_j + 32 > (uint32_t)a.nB)
          hit &= keep_mask(i0, in_j, (uint32_t)a.nA, (uint32_t)a.nB, self != 0);
        if (cnt < (uint32_t)L::FULL) {  // a few hits a lane: one of each lane's per round
          while (__ballot(hit != 0)) {
            if (hit) {
              const uint32_t q = (uint32_t)__builtin_ctz(hit);
              atomicAdd(row_counts + 32 * r + in_i + 2 * (q & 8u) + (q & 3u), 1u);
              atomicAdd(col_counts + (l & 15u) + 4 * (q & 4u), 1u);
              hit &= hit - 1;
            }
          }
          columns = true;
          continue;
        }
        const uint32_t n0 = __popc(hit & 0x0F0Fu), n1 = __popc(hit & 0xF0F0u);
        if (n0) atomicAdd(col_counts + (l & 15u), n0);
        if (n1) atomicAdd(col_counts + 16 + (l & 15u), n1);
        // Rows: a byte per row (two registers of a lane share one), added up over the sixteen lanes that share four of them twice.  (An
        // atomic per lane and row, sixteen on one address: 32,000 points, d = 60, 500 neighbours, 342 us against 308.)
        auto spread = [](uint32_t four) { return __umul24(four, 0x204081u) & 0x01010101u; };  // bit q to byte q
        uint32_t rows[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          rows[h] = spread((hit >> (8 * h)) & 15u) + spread((hit >> (8 * h + 4)) & 15u);
          rows[h] += __builtin_amdgcn_update_dpp(0, rows[h], 0x128, 0xF, 0xF, false);  // rotations by 8, 4, 2, 1 within sixteen lanes
          rows[h] += __builtin_amdgcn_update_dpp(0, rows[h], 0x124, 0xF, 0xF, false);
          rows[h] += __builtin_amdgcn_update_dpp(0, rows[h], 0x122, 0xF, 0xF, false);
          rows[h] += __builtin_amdgcn_update_dpp(0, rows[h], 0x121, 0xF, 0xF, false);
        }
        const uint32_t mine = ((l & 4u ? rows[1] : rows[0]) >> (8 * (l & 3u))) & 0xFFu;
        if ((l & 8u) == 0 && mine) atomicAdd(row_counts + 32 * r + in_i + 4 * (l & 4u) + (l & 3u), mine);
        columns = true;
      } else if (qfill + cnt <= (uint32_t)L::QUEUE) {
        if (has) {
          const uint32_t e = qfill + __builtin_amdgcn_mbcnt_hi((uint32_t)(lanes >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)lanes, 0u));
          float4v* q = reinterpret_cast<float4v*>(queue_v + 16 * e);
          q[0] = __builtin_shufflevector(v, v, 0, 1, 2, 3);
          q[1] = __builtin_shufflevector(v, v, 4, 5, 6, 7);
          q[2] = __builtin_shufflevector(v, v, 8, 9, 10, 11);
          q[3] = __builtin_shufflevector(v, v, 12, 13, 14, 15);
          queue_t[e] = make_uint2(pend_i + 32 * r + in_i, in_j);
        }
        qfill = __builtin_amdgcn_readfirstlane(qfill + cnt);
      } else {
        todo |= 1u << r;
      }
    }
    uint32_t taken = 0;
#pragma unroll 1
    while (todo) {
      drain();
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        if (!(todo & (1u << r)) || qfill == (uint32_t)L::QUEUE) continue;
        const float16v& v = R[P][r];
        uint32_t least = r ? least1 : least0;
        asm volatile("" : "+v"(least));
        const bool has = least <= thr_bits;
        const unsigned long long lanes = __ballot(has);
        const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(lanes >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)lanes, 0u));
        const uint32_t e = qfill + rank - taken;
        if (has && rank >= taken && e < (uint32_t)L::QUEUE) {
          float4v* q = reinterpret_cast<float4v*>(queue_v + 16 * e);
          q[0] = __builtin_shufflevector(v, v, 0, 1, 2, 3);
          q[1] = __builtin_shufflevector(v, v, 4, 5, 6, 7);
          q[2] = __builtin_shufflevector(v, v, 8, 9, 10, 11);
          q[3] = __builtin_shufflevector(v, v, 12, 13, 14, 15);
          queue_t[e] = make_uint2(pend_i + 32 * r + in_i, in_j);
        }
        const uint32_t left = __popcll(lanes) - taken, room = L::QUEUE - qfill;
        if (left <= room) {
          qfill = __builtin_amdgcn_readfirstlane(qfill + left);
          taken = 0;
          todo &= ~(1u << r);
        } else {
          qfill = L::QUEUE;
          taken += room;
        }
      }
    }
    if constexpr (COUNT) {
      if (columns) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        if (l < 32) {
          const uint32_t c = col_counts[l];
          if (c) {
            col_counts[l] = 0;
            const auto ka = arguments();
            if (ka->self) atomicAdd(&ka->counts[pend_j + l], c);
            else if (ka->counts_b) atomicAdd(&ka->counts_b[pend_j + l], c);
          }
        }
        dirty = true;
        settle();
      }
    }
  };
  auto least_of = [&](const float16v& v) -> uint32_t {
    auto u = [&](int r) { return __float_as_uint(v[r]); };
    uint32_t m = min(min(u(0), u(1)), u(2));
#pragma unroll
    for (int r = 3; r < 15; r += 2) m = min(min(m, u(r)), u(r + 1));
    return min(m, u(15));
  };
  // One block of a stage: 64 rows x 32 columns, k in ascending order, then the augmentation step.  P: which block, and its buffer;
  // with two buffers the other one's block goes through the filter under the MFMAs of the second k-block.  cur, nxt: LDS offset of
  // this and of the next stage.
  auto block = [&](auto p_c, uint32_t cur, uint32_t nxt, uint32_t i, uint32_t j) __attribute__((always_inline)) {
    constexpr int P = decltype(p_c)::value, Q = L::TWO ? 1 - P : 0;
    constexpr bool LAST = P == L::BLOCKS - 1;
    constexpr int TURN = FRAGS - (RING - 1);  // from this fragment on what is read belongs to the next block
    float4v acc[4][2];
    uint32_t least0 = 0, least1 = 0;
    half8 gb;
    for_each_index([&](auto f_c) __attribute__((always_inline)) {
      constexpr int f = decltype(f_c)::value, kb = f / 2, c = f % 2;
      constexpr int EARLY = L::TWO ? 0 : TURN - 2;  // what is needed at the end of the block is read here
      if constexpr (LAST && f == TURN) {
        post_read();
        proceed();
      }
      if constexpr (f == EARLY) {
        gb = at_lds(aug0 + ((cur + P * 512) & aug_step), 0);
        if (LAST) look();
      }
      constexpr int read = f + RING - 1, then = read % FRAGS;
      fb[(P * FRAGS + read) % RING] = at_lds((off0 + (LAST && read >= FRAGS ? nxt : cur)) ^ (then % 2 * 32),
                                             then / 2 * L::KB + (read < FRAGS ? P : (LAST ? 0 : P + 1)) * 2048);
      if constexpr (L::TWO && f == 2) {
        least0 = least_of(R[Q][0]);
        least1 = least_of(R[Q][1]);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int t = c ? 3 - u : u;
        const float4v z = {0.f, 0.f, 0.f, 0.f};
        acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa[kb][t], fb[(P * FRAGS + f) % RING], kb == 0 ? z : acc[t][c], 0, 0, 0);
      }
      // one LDS read, then four MFMAs, the filter's instructions between them
      if constexpr (f == EARLY) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      if constexpr (f == EARLY && LAST) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if constexpr (L::TWO && kb == 1) __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
      }
      if constexpr (c) __builtin_amdgcn_sched_barrier(0);
      if constexpr (L::TWO && f == 3) {
        if (__ballot(min(least0, least1) <= thr_bits)) rare(std::integral_constant<int, Q>{}, least0, least1);
      }
    }, std::make_integer_sequence<int, FRAGS>{});
#pragma unroll
    for (int r = 1; r >= 0; --r)
      R[P][r] = __builtin_amdgcn_mfma_f32_32x32x16_f16(L::ROWS_LDS ? at_lds(aug_rows, r * 512) : ga[r], gb,
                                                       cat4(acc[2 * r][0], acc[2 * r][1], acc[2 * r + 1][0], acc[2 * r + 1][1]), 0, 0, 0);
    pend_i = i;
    pend_j = j;
    if constexpr (!L::TWO) {
      least0 = least_of(R[0][0]);
      least1 = least_of(R[0][1]);
      if (__ballot(min(least0, least1) <= thr_bits)) rare(std::integral_constant<int, 0>{}, least0, least1);
    }
  };

  uint32_t held = run_i;  // the row panel in the registers
  auto load_panel = [&](uint32_t I) __attribute__((always_inline)) {
    held = I;
    const auto ka = arguments();
    uint32_t panel = 2 * I + (wave >> 2);
    const bool none = panel >= ka->ntilesA;  // (an odd number of panels of 256)
    if (none) panel = 2 * I;
    const char* p = reinterpret_cast<const char*>(ka->XpA) + (int64_t)panel * panel_stride;
#pragma unroll
    for (int kb = 0; kb < K; ++kb)
#pragma unroll
      for (int t = 0; t < 4; ++t)
        fa[kb][t] = *reinterpret_cast<const half8*>(p + kb * PANEL_BYTES + quarter * 4096 + (t >> 1) * 2048 + fragment_offset(lane, t & 1));
    if constexpr (L::ROWS_LDS) {
      uint4 own = *reinterpret_cast<const uint4*>(p + (int64_t)K * PANEL_BYTES + (quarter * 64 + lane) * 16);
      if (none) own = make_uint4(P1_OUT_OF_RANGE, 0u, P1_OUT_OF_RANGE, 0u);
      *reinterpret_cast<uint4*>(lds + L::ROWS_OFF + 1024 * wave + 16 * lane) = own;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    } else {
      const uint32_t c0 = ka->status[2], c1 = ka->status[3];
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        uint4 own = *reinterpret_cast<const uint4*>(p + (int64_t)K * PANEL_BYTES + (quarter * 64 + r * 32 + (lane & 31)) * 16);
        if (none) own = make_uint4(P1_OUT_OF_RANGE, 0u, P1_OUT_OF_RANGE, 0u);
        const uint4 con = (lane >> 3) & 1 ? make_uint4(0u, 0u, c0, c1) : make_uint4(c0, c1, 0u, 0u);
        ga[r] = as_half8(upper ? con : own);
      }
    }
    settle();
  };

  // ---------------- prologue
  const uint32_t first_panel = run_i;
  for (int q = 0; q < L::DEPTH; ++q) issue();
  load_panel(first_panel);
  // stages 0 .. POST - 1
  if (live) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(L::COPIES * ((L::DEPTH - L::POST) / 2)) : "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
#pragma unroll
  for (int f = 0; f < RING - 1; ++f) fb[f] = at_lds(off0 ^ (f % 2 * 32), f / 2 * L::KB);
  for (;;) {
    const uint32_t c = __builtin_amdgcn_readlane(places, slot), I = __builtin_amdgcn_readlane(places, slot + 32);
    if (__builtin_expect(c == NO_STAGE, 0)) break;
    begin_stage();
    if (__builtin_expect(I != held, 0)) load_panel(I);
    if (!COUNT && __builtin_expect(a.self && c == I * (EJ_STRIP_ROWS / L::COLS) + wave * (64 / L::COLS), 0)) {  // (i, i) belongs to the result by definition, whatever the arithmetic says
      const uint32_t i = c * L::COLS + lane;
      if (fill + 64 > (uint32_t)L::STG) flush();
      stage_entry(__ballot(i < (uint32_t)a.nA), i < (uint32_t)a.nA, i, i, 0u);
      settle();
    }
    const uint32_t cur = slot * (uint32_t)L::STAGE;
    slot = slot == L::STAGES - 1 ? 0 : slot + 1;
    const uint32_t nxt = slot * (uint32_t)L::STAGE;
    const uint32_t i = I * EJ_STRIP_ROWS + wave * 64, j = c * L::COLS;
    block(std::integral_constant<int, 0>{}, cur, nxt, i, j);
    if constexpr (L::TWO) block(std::integral_constant<int, 1>{}, cur, nxt, i, j + 32);
    if constexpr (L::BLOCKS * FRAGS % RING != 0) {  // the next block's first fragments to the places where it looks for them
      half8 moved[RING - 1];
#pragma unroll
      for (int f = 0; f < RING - 1; ++f) moved[f] = fb[(L::BLOCKS * FRAGS + f) % RING];
#pragma unroll
      for (int f = 0; f < RING - 1; ++f) fb[f] = moved[f];
    }
    ++g;
    if (__builtin_expect(--sync_left == 0, 0)) {
      const auto ka = arguments();
      sync_left = (uint32_t)ka->sync_mode;
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      xcd_align(ka->xcd_bar + blockIdx.x % NUM_XCD, tc.step * ++epoch);
      settle();
    }
  }
  if constexpr (L::TWO) {
    const uint32_t least0 = least_of(R[1][0]), least1 = least_of(R[1][1]);
    if (__ballot(min(least0, least1) <= thr_bits)) rare(std::integral_constant<int, 1>{}, least0, least1);
  }
  if (qfill) drain();
  if constexpr (COUNT) send_rows();
  xcd_leave();
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  // what is left, with one atomic for the workgroup (see k_join)
  __syncthreads();
  unsigned long long* sums = reinterpret_cast<unsigned long long*>(lds);
  if (lane == 0) sums[wave] = COUNT ? hits : (unsigned long long)fill;
  __syncthreads();
  if (tid == 0) {
    unsigned long long total = 0;
    for (int w = 0; w < THREADS / 64; ++w) {
      const unsigned long long v = sums[w];
      sums[w] = total;
      total += v;
    }
    if (COUNT && total) atomicAdd(a.total, total);
    if (!COUNT) sums[THREADS / 64] = total ? atomicAdd(a.n_pairs, total) : 0ull;
  }
  if (!COUNT) {
    __syncthreads();
    store_staged(sums[THREADS / 64] + sums[wave]);
  }
}


// ------------------------------------------------------------------------------------------
// The join of small problems
// ------------------------------------------------------------------------------------------
// Two launches instead of three: k_prep (norms and packed copies of both sets, in one launch, and everything the call needs
// zero) and k_join_small, which works out the operands of the augmentation step from the norms by itself.  The largest norm
// passes from one to the other as one value per workgroup of k_prep: nothing has to be zero before or after.
struct PrepSet {
  const uint16_t* X;  // null: a set prepared before
  int64_t n, npad, ld;
  float* s;
  uint4* Xp;
  uint32_t groups;  // workgroups that work on it
};
struct PrepArgs {
  PrepSet a, b;
  int k32steps;
  uint32_t* maxima;    // one per workgroup, or null:
  uint32_t* max_bits;  // ... the largest of all
  unsigned long long* counter;  // cleared, like the counts (may be null)
  uint32_t* counts;  // count mode: cleared (may be null)
  int64_t ncounts;
  uint32_t* counts_b;
  int64_t ncounts_b;
};
__global__ __launch_bounds__(512) void k_prep(const PrepArgs a) {
  const int64_t at = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, all = (int64_t)gridDim.x * blockDim.x;
  if (at == 0 && a.counter) *a.counter = 0;
  if (a.counts)
    for (int64_t i = at; i < a.ncounts; i += all) a.counts[i] = 0;
  if (a.counts_b)
    for (int64_t i = at; i < a.ncounts_b; i += all) a.counts_b[i] = 0;
  const bool second = blockIdx.x >= a.a.groups;
  const PrepSet& set = second ? a.b : a.a;
  const int64_t row0 = ((int64_t)(blockIdx.x - (second ? a.a.groups : 0u)) * (blockDim.x >> 6) + (threadIdx.x >> 6)) * NORM_POINTS;
  uint32_t most = 0;
  if (row0 < set.npad) most = norms_of_wave<true>(row0, set.X, set.n, set.ld, a.k32steps, set.s, set.Xp, a.k32steps + 1);
  most = max_of_group(most);
  if (threadIdx.x == 0 && blockIdx.x < a.a.groups + a.b.groups) {  // (the others only clear counts)
    if (a.max_bits) atomicMax(a.max_bits, most);
    else a.maxima[blockIdx.x] = most;
  }
}

struct SmallArgs {
  JoinArgs j;  // (ntilesA, ntilesB in tiles of TS)
  const float* sA;
  const float* sB;
  const uint32_t* maxima;
  uint32_t nmaxima;
  const uint32_t* set_max;  // largest norm of a prepared set, or null
  int data_blocks;          // k-blocks of data per panel
  int nkb_split;            // split-FP16 set: k-blocks of each part (see k_split_prep); else 0x3FFFFFFF
};

// Tiles of TS x TS points, a workgroup of 2 x 2 wavefronts each (wave tile TS/2 x TS/2), several workgroups to a CU, which
// hide each other's latencies: no copying wavefronts, no augmentation copies, no alignment.  The arithmetic is k_join's, step
// by step (16 x 16 blocks over k in ascending order, one augmentation step per 32 x 32 region), and so are the results, bit
// for bit.  Count mode adds up a tile's counts in the LDS and sends one atomic per row and column: the small problems are the
// dense ones, hits per tile grow as 1/n.
//
// Workgroups on a CU and LDS stages: at TS = 128 three workgroups with two stages each (136 registers, 48 KB), not two with
// three: 768 tiles at a time instead of 512 (4,096 points, d = 128: 17.9 against 23.9 us a call; up to 512 tiles the deeper
// pipeline would be 5 to 10 % faster at d = 960).  Four workgroups leave the staging too small (10,000 points, d = 384, 64
// neighbours: join 98 against 64 us).
template <int TS>
constexpr int small_stages() { return TS == 64 ? 3 : 2; }
template <int TS>
constexpr int small_groups_per_cu() { return TS == 64 ? 4 : 3; }
constexpr int SMALL_STG_CAP = 256;
template <bool COUNT, int TS>
constexpr int small_lds_bytes() {
  return small_stages<TS>() * 2 * TS * 64 + 2 * TS * 16 + 64 + (COUNT ? 2 * TS * 4 : 4 * SMALL_STG_CAP * 12) + 64;
}
template <bool COUNT, int TS>
__global__ __launch_bounds__(256, small_groups_per_cu<TS>()) void k_join_small(const SmallArgs args) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  constexpr int W = TS / 2, MT = W / 16, NR = W / 32;
  constexpr int OP_BYTES = TS * 64, ST_BYTES = 2 * OP_BYTES;
  constexpr int COPIES = TS / 64;  // copy instructions per wavefront, operand and slice
  constexpr int STAGES = small_stages<TS>();
  constexpr int AUG = STAGES * ST_BYTES, AUG_B = AUG + TS * 16, AUG_CONST = AUG_B + TS * 16;
  constexpr int TAIL = AUG_CONST + 64;                                     // staging (pairs) or counters (counts)
  constexpr int SUMS = TAIL + (COUNT ? 2 * TS * 4 : 4 * SMALL_STG_CAP * 12);  // 64 bytes
  const JoinArgs& a = args.j;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave >> 1) * W, wn = (wave & 1) * W;
  const int r16 = lane & 15, g = lane >> 4;
  const int nsl = a.nslices;
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
  TileCursor tc;
  tc.init(blockIdx.x, gridDim.x, (uint32_t)a.self, a.ntilesA, a.ntilesB);
  uint32_t I = 0, J = 0;
  bool have = tc.next(I, J);
  if (!have) return;
  const int64_t panel_stride = (int64_t)(args.data_blocks + 1) * PANEL_BYTES;
  const uint32_t voff = lane * 16 + wave * 1024;
  const char *pa = nullptr, *pb = nullptr;
  auto uniform_ptr = [](const char* p) -> const char* {
    const uint64_t b = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b), hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return reinterpret_cast<const char*>(((uint64_t)hi << 32) | lo);
  };
  auto issue = [&](int ks, int stage) {  // slice ks of the tile at (pa, pb)
    const char* ga = uniform_ptr(pa + (int64_t)split_block_a(ks, args.nkb_split) * PANEL_BYTES);
    const char* gb = uniform_ptr(pb + (int64_t)split_block_b(ks, args.nkb_split) * PANEL_BYTES);
    const uint32_t at = __builtin_amdgcn_readfirstlane(lds0 + stage * ST_BYTES + wave * 1024);
    copy16_to_lds<0>(at, ga, voff);
    if constexpr (COPIES == 2) copy16_to_lds<4096>(at, ga, voff + 4096);
    copy16_to_lds<OP_BYTES>(at, gb, voff);
    if constexpr (COPIES == 2) copy16_to_lds<OP_BYTES + 4096>(at, gb, voff + 4096);
  };
  auto start_tile = [&]() {
    pa = reinterpret_cast<const char*>(a.XpA) + (int64_t)(I * TS / TILE) * panel_stride + (I * TS % TILE) * 64;
    pb = reinterpret_cast<const char*>(a.XpB) + (int64_t)(J * TS / TILE) * panel_stride + (J * TS % TILE) * 64;
#pragma unroll
    for (int ks = 0; ks < STAGES - 1; ++ks) issue(ks, ks);
  };
  start_tile();
  uint32_t mb = args.set_max ? *args.set_max : 0u;
  for (uint32_t q = tid; q < args.nmaxima; q += 256) mb = max(mb, args.maxima[q]);
  const NormScale ns = norm_scale(max_of_group(mb));
  if (blockIdx.x == 0 && tid == 0) a.status[0] = ns.st;
  if (ns.st != ST_OK) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the copies must land before the wave ends
    return;
  }
  if (tid < 4) {  // the constant chunks of the augmentation step (2 and 3)
    const uint32_t c = fp16_bits(ns.c), c0 = c | (c << 16);
    *reinterpret_cast<uint2*>(lds + AUG_CONST + tid * 8) = tid == 0 || tid == 3 ? make_uint2(c0, c) : make_uint2(0u, 0u);
  }
  uint32_t* cnt = reinterpret_cast<uint32_t*>(lds + TAIL);
  if (COUNT && tid < 2 * TS) cnt[tid] = 0;
  uint32_t* stg = reinterpret_cast<uint32_t*>(lds + TAIL + wave * (SMALL_STG_CAP * 12));
  uint32_t fill = 0;     // (pairs) entries staged, wave-uniform
  uint32_t hits = 0;     // (counts) of this lane
  bool dirty = false;
  auto store_staged = [&](unsigned long long base) {
    for (uint32_t e = lane; e < fill; e += 64) {
      const unsigned long long idx = base + e;
      if (idx < a.capacity) {
        reinterpret_cast<uint2*>(a.pairs)[idx] = make_uint2(stg[3 * e], stg[3 * e + 1]);
        if (a.dist2) a.dist2[idx] = __uint_as_float(stg[3 * e + 2]);
      }
    }
  };
  auto append = [&](unsigned long long mask, bool pass, uint32_t i, uint32_t j, uint32_t d2_bits) {
    const uint32_t more = __popcll(mask);
    if (fill + more > SMALL_STG_CAP) {
      unsigned long long base = 0;
      if (lane == 0) base = atomicAdd(a.n_pairs, (unsigned long long)fill);
      const uint32_t blo = __builtin_amdgcn_readfirstlane((uint32_t)base), bhi = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32));
      store_staged(((unsigned long long)bhi << 32) | blo);
      fill = 0;
      dirty = true;
    }
    const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
    if (pass) {
      const uint32_t e = fill + rank;
      stg[3 * e] = i;
      stg[3 * e + 1] = j;
      stg[3 * e + 2] = d2_bits;
    }
    fill += more;
  };
  // fragment and augmentation operand addresses (see k_join)
  const uint32_t frag0 = fragment_offset(lane, 0), frag1 = fragment_offset(lane, 1);
  const int ca = aug_chunk_a(lane), cb = aug_chunk_b(lane);
  const char* aug_a = lds + (ca == 0 ? AUG + 16 * (wm + (lane & 31)) : AUG_CONST + 16 * (ca - 2));
  const char* aug_b = lds + (cb == 1 ? AUG_B + 16 * (wn + (lane & 31)) : AUG_CONST + 16 * (cb - 2));
  const int step_a = ca == 0 ? 512 : 0, step_b = cb == 1 ? 512 : 0;
  const uint32_t nnA = (uint32_t)a.nA, nnB = (uint32_t)a.nB;

  while (have) {
    // ---- operands of the augmentation step: thread t row t of the tile's A panel, then of its B panel (panel_layout.h)
    if (tid < 2 * TS) {
      const bool col = tid >= TS;
      const int row = tid & (TS - 1), in = row & 31;
      const uint32_t x = (col ? J : I) * TS + (row & ~31) + (col ? aug_col_point(in) : aug_row_point(in));
      const uint32_t y = x + (col ? 16u : 4u), nn = col ? nnB : nnA;
      const float* s = col ? args.sB : args.sA;
      uint2 p = make_uint2(P1_OUT_OF_RANGE, 0u), q = p;
      if (x < nn) p = norm_pieces(s[x], ns.m);
      if (y < nn) q = norm_pieces(s[y], ns.m);
      *reinterpret_cast<uint4*>(lds + (col ? AUG_B : AUG) + row * 16) = make_uint4(p.x, p.y, q.x, q.y);
    }
    // ---- the slices: two ahead in flight
    float4v acc[MT][MT];
#pragma unroll
    for (int x = 0; x < MT; ++x)
#pragma unroll
      for (int y = 0; y < MT; ++y) acc[x][y] = float4v{0.f, 0.f, 0.f, 0.f};
    int stage = 0;
    for (int ks = 0; ks < nsl; ++ks) {
      // this wavefront's copies of slice ks have landed once only those of slice ks + 1 are outstanding; what else it has
      // written to the LDS must be there for the others too
      if (STAGES == 3 && ks + 1 < nsl) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(2 * COPIES) : "memory");
      else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
      wg_barrier();  // slice ks is there for everybody, and everybody is done with slice ks - 1
      if (ks + STAGES - 1 < nsl) issue(ks + STAGES - 1, stage == 0 ? STAGES - 1 : stage - 1);
      const char* st = lds + stage * ST_BYTES;
      half8 fa[MT], fb[MT];
#pragma unroll
      for (int f = 0; f < MT; ++f) {
        fa[f] = *reinterpret_cast<const half8*>(st + wm * 64 + (f >> 1) * 2048 + ((f & 1) ? frag1 : frag0));
        fb[f] = *reinterpret_cast<const half8*>(st + OP_BYTES + wn * 64 + (f >> 1) * 2048 + ((f & 1) ? frag1 : frag0));
      }
#pragma unroll
      for (int y = 0; y < MT; ++y)
#pragma unroll
        for (int u = 0; u < MT; ++u) {
          const int x = (y & 1) ? MT - 1 - u : u;
          acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa[x], fb[y], acc[x][y], 0, 0, 0);
        }
      stage = stage == STAGES - 1 ? 0 : stage + 1;
    }
    half8 ha[NR], hb[NR];
#pragma unroll
    for (int t = 0; t < NR; ++t) {
      ha[t] = *reinterpret_cast<const half8*>(aug_a + t * step_a);
      hb[t] = *reinterpret_cast<const half8*>(aug_b + t * step_b);
    }
    const uint32_t i_tile = I * TS, j_tile = J * TS;
    const bool diag = a.self && I == J;
    have = tc.next(I, J);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    wg_barrier();  // everybody has read the last slice and the augmentation operands
    if (have) start_tile();
    // ---- filter and rare path
    const bool partial = diag || i_tile + TS > nnA || j_tile + TS > nnB;
    if (diag && !COUNT && wave < TS / 64) {  // (i, i) belongs to the result by definition
      const uint32_t i = i_tile + tid;
      append(__ballot(i < nnA), i < nnA, i, i, 0u);
    }
#pragma unroll
    for (int Ra = 0; Ra < NR; ++Ra)
#pragma unroll
      for (int Rb = 0; Rb < NR; ++Rb) {
        const float16v v = __builtin_amdgcn_mfma_f32_32x32x16_f16(
            ha[Ra], hb[Rb], cat4(acc[2 * Ra][2 * Rb], acc[2 * Ra][2 * Rb + 1], acc[2 * Ra + 1][2 * Rb], acc[2 * Ra + 1][2 * Rb + 1]), 0, 0, 0);
        // bit r of hit: register r of this lane passes
        uint32_t hit = 0;
#pragma unroll
        for (int r = 0; r < 16; ++r) hit |= v[r] >= a.thr ? 1u << r : 0u;
        if (__ballot(hit != 0) == 0) continue;
        const uint32_t il = wm + 32 * Ra + 4 * g, jl = wn + 32 * Rb + r16;  // register 0's place in the tile (region_pair)
        if (partial) hit &= keep_mask(i_tile + il, j_tile + jl, nnA, nnB, diag);
        if constexpr (COUNT) {
          hits += __popc(hit);
          add_region_counts(hit, cnt + il, cnt + TS + jl);
        } else {
          // every round takes one hit of each lane that has any left
          for (unsigned long long mask = __ballot(hit != 0); mask; mask = __ballot(hit != 0)) {
            const uint32_t r = (uint32_t)__builtin_ctz(hit | 0x10000u);
            append(mask, hit != 0, i_tile + il + 2 * (r & 8u) + (r & 3u), j_tile + jl + 4 * (r & 4u),
                   __float_as_uint(fmaxf(-2.f * pick(v, r), 0.f)));
            hit &= hit - 1;
          }
        }
      }
    if constexpr (COUNT) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      wg_barrier();
      if (tid < 2 * TS) {
        const uint32_t v = cnt[tid];
        if (v) {
          cnt[tid] = 0;
          uint32_t* to = tid < TS ? a.counts : (a.self ? a.counts : a.counts_b);
          if (to) atomicAdd(to + (tid < TS ? i_tile + tid : j_tile + (tid - TS)), v);
        }
      }
      dirty = true;
    }
    // (stores and atomics count on vmcnt like the copies, but complete in any order)
    if (dirty) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      dirty = false;
    }
  }
  // ---- what is left, with one atomic for the workgroup (see k_join)
  unsigned long long* sums = reinterpret_cast<unsigned long long*>(lds + SUMS);
  if constexpr (COUNT) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) hits += (uint32_t)__shfl_xor((int)hits, off);
  }
  if (lane == 0) sums[wave] = COUNT ? hits : fill;
  __syncthreads();
  if (tid == 0) {
    unsigned long long total = 0;
    for (int w = 0; w < 4; ++w) {
      const unsigned long long v = sums[w];
      sums[w] = total;
      total += v;
    }
    if (COUNT && total) atomicAdd(a.total, total);
    if (!COUNT) sums[4] = total ? atomicAdd(a.n_pairs, total) : 0ull;
  }
  if (!COUNT) {
    __syncthreads();
    store_staged(sums[4] + sums[wave]);
  }
}

// ------------------------------------------------------------------------------------------
// The join of the smallest problems, in one launch
// ------------------------------------------------------------------------------------------
// Problems whose tiles all fit the CUs at once: a workgroup of k_join_once computes one tile from the rows of X as they are, and the
// norms of the tile's points beside it (two more MFMA chains per wavefront, the diagonals of 16 points' Gram blocks as in
// norms_of_wave).  What bounds them is launches and latency, on the host as much as on the GPU; by k_prep and k_join_small, a call
// (all on one card): counts of 1,000 x 96 11.5 us, now 8.3; 2,400 x 128 14.3, now 9.3; lists of 4,096 x 128 18.1, now 15.5 (counts
// 17.8, 11.6), of 2,800 x 384 20.9, now 14.7, 4,096 x 960 39.9, now 38.4; 25,000 points x 60 queries, d = 384, 26.5, now 15.1.
//   * The scale of the norm terms comes from the largest norm of all points.  The workgroups on the diagonal (two sets: of the first
//     row and column of tiles) put the largest norm of every 64 of their points into a slot each, and every workgroup reads all the
//     slots before its augmentation step.  It waits for them a bounded number of times only: workgroups that the GPU has not started
//     yet may be behind others that wait for this kernel's.  Past that it works out by itself what is missing (`late`).
//     The slots are there once for every XCD, so that no line has more than an eighth of the readers (4,096 x 128: one copy 18.3 us,
//     eight 16.4, thirty-two 16.9, without the wait 14.8).
//   * Counts are cleared by the workgroups that fill those rows' slots, before they do, so whoever has seen all slots may add to them.  A late
//     workgroup adds to counters of the context's instead, which the last workgroup of all adds to the result.
//   * The result's counter is the context's, with a ticket in its upper bits: one atomic per workgroup says where its pairs go and
//     which workgroup is the last; that one stores the total and leaves everything as it was found, all zero.  Those atomics are served
//     one after the other, 6 to 13 ns each: counts take theirs XCD by XCD from ONCE_STEPS tiles on (4,096 x 128 16.3 us, then 13.0).
//   * Eight wavefronts to a tile of 128: with four of 64 x 64 each 16.2 us for the lists of 4,096 x 128 and 13.0 for the counts, with
//     eight 15.5 and 11.6.  Three workgroups fit a CU.  Its slices are of 32 coordinates (half lines, two-way bank conflicts), so that three stages do.
// The arithmetic is k_join's, step by step, and the results its bits.
struct OnceArgs {
  JoinArgs j;  // (ntilesA, ntilesB in tiles of TS; no packed copies)
  const uint16_t* XA;
  const uint16_t* XB;
  int64_t ldA, ldB;
  float* sA;  // for the norms that a late workgroup works out (nobody reads them)
  float* sB;
  uint32_t tiles, slots_a, slots;  // slots: one per 64 points of the first set, then of the second
  // of the context, all zero between calls
  unsigned long long* state;
  uint32_t* slot;
  uint32_t* late_counts;  // of the points, then of the query points
};
constexpr uint32_t ONCE_STEPS = 256; // tiles from which on counts take their tickets XCD by XCD
template <int TS>
struct Once {
  static constexpr int WR = TS / 32, WC = 2, WAVES = WR * WC, THREADS = 64 * WAVES;  // wavefronts: of the rows, of the columns; 32 x TS / 2 each
  static constexpr int SC = TS == 64 ? 64 : 32;  // coordinates of a slice
  static constexpr int ROW = 2 * SC;             // bytes of a row of it
  static constexpr int OP = TS * ROW, STAGE = 2 * OP;
  static constexpr int STAGES = 3;
  static constexpr int COPIES = OP / (WAVES * 1024);  // copy instructions per wavefront, operand and slice
  // after the last slice, where the stages were: the norms, staged results or counters, the operands of the augmentation step
  static constexpr int TAIL = 2 * TS * 4, AUG = TAIL + WAVES * SMALL_STG_CAP * 12, AUG_B = AUG + TS * 16, AUG_CONST = AUG_B + TS * 16;
  static constexpr int SUMS = STAGES * STAGE, LDS = SUMS + 128;
  static_assert(ONCE_EMPTY_WORDS * 4 <= TS * 16 && ONCE_EMPTY_WORDS <= THREADS && AUG_CONST + 64 <= SUMS && LDS * ONCE_GROUPS_PER_CU <= 152 * 1024, "LDS budget");
};
template <bool COUNT, int TS>
__global__ __launch_bounds__(Once<TS>::THREADS, ONCE_GROUPS_PER_CU * Once<TS>::WAVES / 4) void k_join_once(const OnceArgs args) {
  using L = Once<TS>;
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  constexpr int MR = 2, MC = TS / 32, NC = MC / 2, KBS = L::SC / KSLICE;  // a wavefront's blocks of rows and columns, its regions
  const JoinArgs& a = args.j;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * (TS / 2);
  const int r16 = lane & 15, g = lane >> 4;
  const int nkb = a.nslices, nsl = (nkb + KBS - 1) / KBS;
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds, nnA = (uint32_t)a.nA, nnB = (uint32_t)a.nB;
  // The tiles whose workgroups fill slots come first.
  uint32_t I, J;
  once_tile(blockIdx.x, (uint32_t)a.self, a.ntilesA, a.ntilesB, I, J);
  const uint32_t i_tile = I * TS, j_tile = J * TS;
  const bool diag = a.self && I == J;

  // ---- this thread's point of the tile: row tid of its rows, then of its columns
  const bool col = tid >= TS;
  const uint32_t own = (col ? j_tile : i_tile) + (tid & (TS - 1));
  const bool exists = tid < 2 * TS && own < (col ? nnB : nnA);
  const bool fills = col ? !a.self && I == 0 : (a.self ? I == J : J == 0);  // (uniform over a wavefront)
  if (COUNT && fills && exists) {
    uint32_t* to = col ? a.counts_b : a.counts;
    if (to) __hip_atomic_store(to + own, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // ---- copies.  Rows of 128 bytes: chunk c of row r at position c ^ (r / 2 % 8), as in the dense block; of 64 bytes: c ^ (r / 4 % 4).
  // Rows past the end are the last one's again (they carry the marker in the norm term).
  constexpr int PER = 1024 / L::ROW, CH = L::ROW / 16;  // rows and chunks a row of a copy instruction
  auto swizzle = [](int r) { return TS == 64 ? (r >> 1) & 7 : (r >> 2) & 3; };
  const char *ga[L::COPIES], *gb[L::COPIES];
#pragma unroll
  for (int q = 0; q < L::COPIES; ++q) {
    const int r = PER * (L::WAVES * q + wave) + lane / CH, c = (lane % CH) ^ swizzle(r);
    ga[q] = reinterpret_cast<const char*>(args.XA + (int64_t)min(i_tile + r, nnA - 1) * args.ldA) + 16 * c;
    gb[q] = reinterpret_cast<const char*>(args.XB + (int64_t)min(j_tile + r, nnB - 1) * args.ldB) + 16 * c;
  }
  auto issue = [&](int stage) {  // the next slice
    const uint32_t at = __builtin_amdgcn_readfirstlane(lds0 + stage * L::STAGE + wave * 1024);
    copy16_to_lds_from<0>(at, ga[0]);
    if constexpr (L::COPIES == 2) copy16_to_lds_from<4096>(at, ga[1]);
    copy16_to_lds_from<L::OP>(at, gb[0]);
    if constexpr (L::COPIES == 2) copy16_to_lds_from<L::OP + 4096>(at, gb[1]);
#pragma unroll
    for (int q = 0; q < L::COPIES; ++q) {
      ga[q] += L::ROW;
      gb[q] += L::ROW;
    }
  };
#pragma unroll
  for (int ks = 0; ks < L::STAGES - 1; ++ks)
    if (ks < nsl) issue(ks);
  uint32_t off[KBS];  // k-block kb of a slice: row lane % 16, chunk 4 kb + lane / 16
#pragma unroll
  for (int kb = 0; kb < KBS; ++kb) off[kb] = r16 * L::ROW + (((4 * kb + g) ^ swizzle(r16)) << 4);

  // ---- the Gram products and the norms: every wavefront's one of its two blocks of rows and one of its WR blocks of columns, so that
  // the wavefronts that share them have them all
  const int norm_r = wm + 16 * (wave & 1), norm_c = wn + 16 * (wave >> 1);
  float4v acc[MR][MC], norm[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
  for (int x = 0; x < MR; ++x)
#pragma unroll
    for (int y = 0; y < MC; ++y) acc[x][y] = float4v{0.f, 0.f, 0.f, 0.f};
  int stage = 0;
  for (int ks = 0; ks < nsl; ++ks) {
    if (ks + 1 < nsl) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(2 * L::COPIES) : "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    wg_barrier();  // slice ks is there for everybody, and everybody is done with slice ks - 1
    if (ks + L::STAGES - 1 < nsl) issue(stage == 0 ? L::STAGES - 1 : stage - 1);
    const char* st = lds + stage * L::STAGE;
#pragma unroll
    for (int kb = 0; kb < KBS; ++kb) {
      if (KBS > 1 && ks * KBS + kb >= nkb) break;
      half8 fa[MR], fb[MC];
#pragma unroll
      for (int f = 0; f < MR; ++f) fa[f] = *reinterpret_cast<const half8*>(st + (wm + 16 * f) * L::ROW + off[kb]);
#pragma unroll
      for (int f = 0; f < MC; ++f) fb[f] = *reinterpret_cast<const half8*>(st + L::OP + (wn + 16 * f) * L::ROW + off[kb]);
      const half8 nr = *reinterpret_cast<const half8*>(st + norm_r * L::ROW + off[kb]), nc = *reinterpret_cast<const half8*>(st + L::OP + norm_c * L::ROW + off[kb]);
#pragma unroll
      for (int y = 0; y < MC; ++y)
#pragma unroll
        for (int u = 0; u < MR; ++u) {
          const int x = (y & 1) ? MR - 1 - u : u;
          acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa[x], fb[y], acc[x][y], 0, 0, 0);
        }
      norm[0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(nr, nr, norm[0], 0, 0, 0);
      norm[1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(nc, nc, norm[1], 0, 0, 0);
    }
    stage = stage == L::STAGES - 1 ? 0 : stage + 1;
  }
  __syncthreads();  // everybody has read the last slice
  float* norms = reinterpret_cast<float*>(lds);  // of the rows, then of the columns
  store_diagonal(norm[0], norm_r, 2 * TS, norms);
  store_diagonal(norm[1], TS + norm_c, 2 * TS, norms);
  if (COUNT) {
    uint32_t* cnt = reinterpret_cast<uint32_t*>(lds + L::TAIL);
    if (tid < 2 * TS) cnt[tid] = 0;
  }
  uint32_t* empty = reinterpret_cast<uint32_t*>(lds + L::AUG);
  if (tid < ONCE_EMPTY_WORDS) empty[tid] = 0;
  __syncthreads();

  // ---- the largest norm of all
  if (fills && tid < 2 * TS) {
    uint32_t most = exists ? __float_as_uint(norms[tid]) : 0u;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) most = max(most, (uint32_t)__shfl_xor((int)most, o));
    if (COUNT) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the counts are cleared
    const uint32_t first = own - lane;
    if (lane < NUM_XCD && first < (col ? nnB : nnA))
      __hip_atomic_store(args.slot + lane * ONCE_SLOTS + (col ? args.slots_a : 0u) + first / 64, most | ONCE_FILLED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // before the ticket, after which the slots are cleared (not every copy has a reader, and barriers do not wait for stores)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  bool missing;
  uint32_t mb = look_at_slots(args.slot, args.slots, L::THREADS, EJOIN_ONCE_SPINS, missing, empty);
  const bool late = __syncthreads_or(missing);
  if (late) {
    uint32_t half = 0;  // 32 points a wavefront, in turn
    for_empty_slots(empty, args.slots, [&](uint32_t q) {
      const bool second = q >= args.slots_a;
      const int64_t row0 = (int64_t)(second ? q - args.slots_a : q) * 64;
      for (int h = 0; h < 2; ++h)
        if (half++ % L::WAVES == (uint32_t)wave && row0 + 32 * h < (second ? a.nB : a.nA))
          mb = max(mb, norms_of_wave<false>(row0 + 32 * h, second ? args.XB : args.XA, second ? a.nB : a.nA, second ? args.ldB : args.ldA, nkb,
                                            second ? args.sB : args.sA, nullptr, 0));
    });
  }
  const NormScale ns = norm_scale(max_of_group(mb));
  if (blockIdx.x == 0 && tid == 0) a.status[0] = ns.st;

  // ---- the augmentation step and the filter.  Bit r of hit: register r of this lane's part of a region passes.
  float16v v[NC];
  uint32_t hit[NC] = {};
  if (ns.st == ST_OK) {
    if (tid < 2 * TS) {  // (as in k_join_small)
      const int row = tid & (TS - 1), in = row & 31;
      const uint32_t first = (uint32_t)((row & ~31) + (col ? aug_col_point(in) : aug_row_point(in)));
      const uint32_t x = (col ? j_tile : i_tile) + first, y = x + (col ? 16u : 4u), nn = col ? nnB : nnA;
      const float* s = norms + (col ? TS : 0) + first;
      uint2 p = make_uint2(P1_OUT_OF_RANGE, 0u), q = p;
      if (x < nn) p = norm_pieces(s[0], ns.m);
      if (y < nn) q = norm_pieces(s[col ? 16 : 4], ns.m);
      *reinterpret_cast<uint4*>(lds + (col ? L::AUG_B : L::AUG) + row * 16) = make_uint4(p.x, p.y, q.x, q.y);
    }
    if (tid < 4) {  // the constant chunks of the augmentation step (2 and 3)
      const uint32_t c = fp16_bits(ns.c), c0 = c | (c << 16);
      *reinterpret_cast<uint2*>(lds + L::AUG_CONST + tid * 8) = tid == 0 || tid == 3 ? make_uint2(c0, c) : make_uint2(0u, 0u);
    }
    __syncthreads();
    const int ca = aug_chunk_a(lane), cb = aug_chunk_b(lane);
    const char* aug_a = lds + (ca == 0 ? L::AUG + 16 * (wm + (lane & 31)) : L::AUG_CONST + 16 * (ca - 2));
    const char* aug_b = lds + (cb == 1 ? L::AUG_B + 16 * (wn + (lane & 31)) : L::AUG_CONST + 16 * (cb - 2));
    const int step_b = cb == 1 ? 512 : 0;
    const bool partial = diag || i_tile + TS > nnA || j_tile + TS > nnB;
    const half8 ha = *reinterpret_cast<const half8*>(aug_a);
#pragma unroll
    for (int R = 0; R < NC; ++R) {
      const half8 hb = *reinterpret_cast<const half8*>(aug_b + R * step_b);
      v[R] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ha, hb, cat4(acc[0][2 * R], acc[0][2 * R + 1], acc[1][2 * R], acc[1][2 * R + 1]), 0, 0, 0);
    }
#pragma unroll
    for (int R = 0; R < NC; ++R) {
      uint32_t h = 0;
#pragma unroll
      for (int r = 0; r < 16; ++r) h |= v[R][r] >= a.thr ? 1u << r : 0u;
      if (partial && __ballot(h != 0)) h &= keep_mask(i_tile + wm + 4 * g, j_tile + wn + 32 * R + r16, nnA, nnB, diag);
      hit[R] = h;
    }
  }

  // ---- results.  One atomic for the workgroup, with its ticket.
  unsigned long long* sums = reinterpret_cast<unsigned long long*>(lds + L::SUMS);
  const bool own_pairs = diag && !COUNT && wave < TS / 64 && ns.st == ST_OK;  // (i, i) belongs to the result by definition
  uint32_t found = own_pairs && i_tile + tid < nnA ? 1u : 0u;
#pragma unroll
  for (int R = 0; R < NC; ++R) found += __popc(hit[R]);
  found = wave_sum(found);
  if (lane == 0) sums[wave] = found;
  if constexpr (COUNT) {
    uint32_t* cnt = reinterpret_cast<uint32_t*>(lds + L::TAIL);
#pragma unroll
    for (int R = 0; R < NC; ++R)
      if (__ballot(hit[R] != 0)) add_region_counts(hit[R], cnt + wm + 4 * g, cnt + TS + wn + 32 * R + r16);
    __syncthreads();
    if (tid < 2 * TS) {
      const uint32_t c = cnt[tid];
      uint32_t* to = !col || a.self ? a.counts : a.counts_b;
      if (late) to = args.late_counts + (!col || a.self ? 0 : a.nA);
      if (c && to) atomicAdd(to + own, c);
      if (late) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // before the ticket
    }
    if (late) __syncthreads();
  } else {
    __syncthreads();
  }
  unsigned long long all = 0, total = 0;  // (of thread 0) the state with this workgroup's ticket; its pairs
  bool last = false;
  if (tid == 0) {
    for (int w = 0; w < L::WAVES; ++w) total += sums[w];
    const unsigned long long add = ONCE_TICKET | ((unsigned long long)late << 40) | total;
    if (COUNT && args.tiles > ONCE_STEPS) last = close_by_xcd(args.state, args.tiles, atomicAdd(state_of_xcd(args.state), add) + add, all);
    else all = atomicAdd(args.state, add) + add;
  }
  auto close = [&]() {  // (thread 0) the workgroup's place in the result, and whether it is the last of all
    if (!(COUNT && args.tiles > ONCE_STEPS)) {
      last = all >> 52 == args.tiles;
      if (last) *args.state = 0;
    }
    sums[8] = (all & ONCE_FOUND) - total;
    sums[9] = last ? 1 + ((all >> 40) & 0xFFFu) : 0;  // 1 + late workgroups
    if (last) *(COUNT ? a.total : a.n_pairs) = all & ONCE_FOUND;
  };
  if constexpr (COUNT) {
    if (tid == 0) close();
    __syncthreads();
  } else {
    // The hits are sorted out while the atomic is under way, unless there are more than fit the LDS.
    uint32_t* stg = reinterpret_cast<uint32_t*>(lds + L::TAIL + wave * (SMALL_STG_CAP * 12));
    uint32_t fill = 0;            // entries staged, wave-uniform
    unsigned long long base = 0;  // where they go
    bool many = false;
    for (int w = 0; w < L::WAVES; ++w) many |= sums[w] > SMALL_STG_CAP;
    auto place = [&]() {
      if (tid == 0) close();
      __syncthreads();
      base = sums[8];
      for (int w = 0; w < wave; ++w) base += sums[w];
    };
    auto store_staged = [&]() {
      for (uint32_t e = lane; e < fill; e += 64) {
        const unsigned long long idx = base + e;
        if (idx < a.capacity) {
          reinterpret_cast<uint2*>(a.pairs)[idx] = make_uint2(stg[3 * e], stg[3 * e + 1]);
          if (a.dist2) a.dist2[idx] = __uint_as_float(stg[3 * e + 2]);
        }
      }
      base += fill;
      fill = 0;
    };
    auto append = [&](unsigned long long mask, bool pass, uint32_t i, uint32_t j, uint32_t d2_bits) {
      const uint32_t more = __popcll(mask);
      if (fill + more > SMALL_STG_CAP) store_staged();
      const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
      if (pass) {
        const uint32_t e = fill + rank;
        stg[3 * e] = i;
        stg[3 * e + 1] = j;
        stg[3 * e + 2] = d2_bits;
      }
      fill += more;
    };
    if (many) place();
    if (own_pairs) {
      const uint32_t i = i_tile + tid;
      append(__ballot(i < nnA), i < nnA, i, i, 0u);
    }
#pragma unroll
    for (int R = 0; R < NC; ++R) {
      uint32_t h = hit[R];
      // every round takes one hit of each lane that has any left
      for (unsigned long long mask = __ballot(h != 0); mask; mask = __ballot(h != 0)) {
        const uint32_t r = (uint32_t)__builtin_ctz(h | 0x10000u);
        append(mask, h != 0, i_tile + wm + 4 * g + 2 * (r & 8u) + (r & 3u), j_tile + wn + 32 * R + r16 + 4 * (r & 4u),
               __float_as_uint(fmaxf(-2.f * pick(v[R], r), 0.f)));
        h &= h - 1;
      }
    }
    if (!many) place();
    store_staged();
  }
  if (sums[9]) {
    for (uint32_t q = tid; q < args.slots * NUM_XCD; q += L::THREADS) args.slot[q % NUM_XCD * ONCE_SLOTS + q / NUM_XCD] = 0;
    if (COUNT && sums[9] > 1)
      for (uint32_t q = tid; q < nnA + (a.self ? 0u : nnB); q += L::THREADS) {
        const uint32_t c = __hip_atomic_exchange(args.late_counts + q, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        uint32_t* to = q < nnA ? a.counts + q : (a.counts_b ? a.counts_b + (q - nnA) : nullptr);
        if (c && to) atomicAdd(to, c);
      }
  }
}

// ------------------------------------------------------------------------------------------
// The join of a prepared set with few query points
// ------------------------------------------------------------------------------------------
// A batch of up to 16 RF query points against a prepared set, in one launch.  Bound by reading the set's packed copy and, where that is
// little, by the launch.  The query points are the rows of the MFMAs, in the LDS of every workgroup; a wavefront streams 32 points
// with all their k-blocks through its registers at a time, as MFMA operands the way they lie in the packed copy, a chunk of
// few_chunk k-blocks ahead, with no barrier and no copy to the LDS.  Every workgroup works out the norms of the query points, the largest with that of the
// set, and the points' part of the augmentation step from their norms: nothing is waited for, and the set's augmentation block is neither
// read nor written.  A point's count is complete in its wavefront; those of the query points go through the context's counters, which
// the last workgroup copies (see k_join_once).
// A call (counts) in us, by k_prep, k_aux and k_join or k_join_strip, or by k_prep and k_join_small, and now: 8, 60, 120 and 250 queries against 100,000
// points of 128 coordinates 28.0, 29.7, 30.9 and 26.9, now 10.0, 11.6, 14.6 and 19.1 (floor 5.3); 60 against 20,000 x 32 15.5, now 10.0; 60 against
// 400,000 x 384 104.9, now 60.5 (floor 63); 8 against 400,000 x 960 194, now 133; 60 201, now 189.
// Up to 64 query points two workgroups a CU and chunks of two k-blocks (60 against 400,000 x 384: one workgroup and chunks of four 78, of eight 77); more take
// the registers of one.
// Lists: a wavefront stages its results.  Those of a panel that do not fit stay in registers, as hits and distances, until their place in the result is known, by one
// atomic for them and what is staged; of a wavefront's last panel that is the workgroup's, with its ticket.  One atomic for every 256 results cost dense
// lists more than the rest (they are served one after the other; all wavefronts are full at the same time).  Before that, with an atomic for as many as are
// staged, and now, us: 100,000 x 120, d = 300, 4, 14 and 76 % of all pairs 46.4, 43.7 and 38.0; 108, 96 and 61; 482, 467 and 89; 60,000 x 200, d = 128,
// 66, 31 and 24; 184, 95 and 33; 1,110, 461 and 55; 400,000 x 60, d = 384, 235, 95 and 88; 456, 222 and 159; 2,263, 958 and 197.
// The arithmetic is k_join_strip's with the sets exchanged, step by step, and the results its bits.
struct FewArgs {
  const uint4* Xp;
  const float* s;
  const uint32_t* set_max;
  int64_t n;
  int nkb;
  const uint16_t* Q;
  int64_t nq, ldq;
  float thr;
  uint32_t* status;
  uint32_t* pairs;
  float* dist2;
  unsigned long long capacity;
  unsigned long long* n_pairs;
  uint32_t staged;  // (pairs) results a wavefront stages
  uint32_t* counts_p;
  uint32_t* counts_q;  // may be null
  unsigned long long* total;
  // of the context, all zero between calls (see OnceArgs)
  unsigned long long* state;
  uint32_t* counters;
};
constexpr int FEW_LDS = 159 * 1024;  // (a little is the compiler's)
template <int RF>
constexpr int few_chunk() { return RF == 8 ? 4 : 2; }
constexpr int few_groups_per_cu(int rf, int lds_bytes) { return rf <= 4 && lds_bytes <= 79 * 1024 ? 2 : 1; }
constexpr int FEW_WAVES = 8;
// the query points, their norms, part of the augmentation step and counters, the constants of that step, staged results
template <bool COUNT>
constexpr int few_lds_bytes(int rows, int nkb, int staged) { return rows * (nkb * 64 + 4 + 16 + 4) + 64 + 64 + (COUNT ? 0 : FEW_WAVES * staged * 12); }
// Results that a wavefront stages: 256, or 64 or 128 fewer where the LDS for them would cost a workgroup of the CU or the place in LDS (at least 64, what one append
// adds).  Lists with 128 and with 256, us: 100,000 points x 120 queries, d = 300, 4 % of all pairs 47.0 and 38.0, 20,000 x 30, d = 300, 14 % 14.1 and 13.4; with a
// workgroup less 300,000 x 60, d = 512 61.3 and 72.3.
constexpr int few_staged(int rf, int nkb) {
  const int groups = few_groups_per_cu(rf, few_lds_bytes<false>(16 * rf, nkb, 128));
  int staged = 256;
  while (staged > 128 && (few_lds_bytes<false>(16 * rf, nkb, staged) > FEW_LDS || few_groups_per_cu(rf, few_lds_bytes<false>(16 * rf, nkb, staged)) < groups)) staged -= 64;
  return staged;
}
// (waves_per_eu: without the upper bound the instances of up to 64 query points save registers for a fifth wavefront, one operand in flight at a time: + 0.3 us)
template <bool COUNT, int RF>
__global__ __launch_bounds__(64 * FEW_WAVES) __attribute__((amdgpu_waves_per_eu(RF <= 4 ? 4 : 2, RF <= 4 ? 4 : 2))) void k_join_few(const FewArgs a) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  constexpr int ROWS = 16 * RF, NR = RF / 2, CHUNK = few_chunk<RF>();
  const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nkb = a.nkb;
  const uint32_t n = (uint32_t)a.n, nq = (uint32_t)a.nq;
  char* const aug = lds + ROWS * nkb * 64;
  char* const constants = aug + ROWS * 16;
  float* const norms = reinterpret_cast<float*>(constants + 64);
  uint32_t* const row_counts = reinterpret_cast<uint32_t*>(norms + ROWS);
  unsigned long long* const sums = reinterpret_cast<unsigned long long*>(row_counts + ROWS);
  uint32_t* const stg = reinterpret_cast<uint32_t*>(sums + 8) + wave * a.staged * 3;

  // ---- the points: a workgroup a panel of 256, each of its wavefronts 32 of them, and so on through the panels
  const uint32_t panels = (n + TILE - 1) / TILE, chunks = (uint32_t)(nkb + CHUNK - 1) / CHUNK;
  const int64_t panel_stride = (int64_t)(nkb + 1) * PANEL_BYTES;
  const char* const mine = reinterpret_cast<const char*>(a.Xp) + wave * 2048;
  const uint32_t at0 = fragment_offset(lane, 0), at1 = fragment_offset(lane, 1);
  half8 buf[2][CHUNK][2];
  float point_norm[2][2];
  auto load = [&](auto b_c, uint32_t panel, uint32_t chunk) __attribute__((always_inline)) {
    constexpr int B = decltype(b_c)::value;
    if (panel >= panels) return;
    const char* p = mine + panel * panel_stride + (int64_t)chunk * (CHUNK * PANEL_BYTES);
#pragma unroll
    for (int k = 0; k < CHUNK; ++k)
      if ((int)chunk * CHUNK + k < nkb) {
        buf[B][k][0] = *reinterpret_cast<const half8*>(p + k * PANEL_BYTES + at0);
        buf[B][k][1] = *reinterpret_cast<const half8*>(p + k * PANEL_BYTES + at1);
      }
    if (chunk + 1 == chunks) {
#pragma unroll
      for (int h = 0; h < 2; ++h) point_norm[B][h] = a.s[min(panel * TILE + wave * 32 + 16 * h + r16, n - 1)];
    }
  };
  uint32_t panel = blockIdx.x, chunk = 0;  // what is computed next
  load(std::integral_constant<int, 0>{}, panel, chunk);

  // ---- the query points, as operands: k-block k of rows 16 f .. 16 f + 15 at (f nkb + k) KB.  (Rows past the last are that one again.)
  for (int q = wave; q < RF * nkb; q += FEW_WAVES) {
    const int f = q / nkb, k = q - f * nkb;
    const uint32_t row = min((uint32_t)(16 * f + r16), nq - 1);
    *reinterpret_cast<half8*>(lds + q * 1024 + lane * 16) = *reinterpret_cast<const half8*>(a.Q + row * a.ldq + k * KSLICE + 8 * g);
  }
  if (tid < ROWS) row_counts[tid] = 0;
  __syncthreads();
  for (int f = wave; f < RF; f += FEW_WAVES) {
    float4v sq = {0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < nkb; ++k) {
      const half8 x = *reinterpret_cast<const half8*>(lds + (f * nkb + k) * 1024 + lane * 16);
      sq = __builtin_amdgcn_mfma_f32_16x16x32_f16(x, x, sq, 0, 0, 0);
    }
    store_diagonal(sq, 16 * f, ROWS, norms);
  }
  __syncthreads();
  const NormScale ns = norm_scale(max_of_group(max(*a.set_max, (uint32_t)tid < nq ? __float_as_uint(norms[tid]) : 0u)));
  if (blockIdx.x == 0 && tid == 0) a.status[0] = ns.st;
  if (tid < ROWS) {
    const uint32_t x = (uint32_t)((tid & ~31) + aug_row_point(tid & 31)), y = x + 4;
    uint2 p = make_uint2(P1_OUT_OF_RANGE, 0u), q = p;
    if (x < nq) p = norm_pieces(norms[x], ns.m);
    if (y < nq) q = norm_pieces(norms[y], ns.m);
    *reinterpret_cast<uint4*>(aug + tid * 16) = make_uint4(p.x, p.y, q.x, q.y);
  }
  if (tid < 4) {  // the constant chunks of the augmentation step (2 and 3)
    const uint32_t c = fp16_bits(ns.c), c0 = c | (c << 16);
    *reinterpret_cast<uint2*>(constants + tid * 8) = tid == 0 || tid == 3 ? make_uint2(c0, c) : make_uint2(0u, 0u);
  }
  __syncthreads();
  // operands of that step, the halves exchanged as in k_join_strip with the sets exchanged
  const char* const row_operand = lane < 32 ? constants + 16 * ((lane >> 3) & 1) : aug + 16 * (lane & 31);
  const int row_step = lane < 32 ? 0 : 512;
  const uint32_t edge_mask = keep_mask(4 * g, 0, nq % 32, 0xFFFFFFFFu, false);  // registers of the last region whose query point exists
  const uint4 column_constant = *reinterpret_cast<const uint4*>(constants + 16 * ((lane >> 4) & 1));

  uint32_t fill = 0;             // (pairs) staged, uniform
  unsigned long long base = 0;   // (pairs) where what is staged goes, once that is known
  uint32_t hits[(NR + 1) / 2];   // (pairs) of the last 32 points, those that are not staged: two regions a word
  uint32_t left = 0, left_j0 = 0;  // (pairs) how many of those wait for the workgroup's atomic, and the first of the points
  unsigned long long found = 0;  // (counts) of this lane
  const uint32_t thr_bits = __float_as_uint(a.thr) | 0x80000000u;  // (x >= thr on the bit patterns, see k_join)
  auto uniform = [](unsigned long long x) {
    return ((unsigned long long)__builtin_amdgcn_readfirstlane((uint32_t)(x >> 32)) << 32) | __builtin_amdgcn_readfirstlane((uint32_t)x);
  };
  auto store_staged = [&]() {
    for (uint32_t e = lane; e < fill; e += 64) {
      const unsigned long long idx = base + e;
      if (idx < a.capacity) {
        reinterpret_cast<uint2*>(a.pairs)[idx] = make_uint2(stg[3 * e], stg[3 * e + 1]);
        if (a.dist2) a.dist2[idx] = __uint_as_float(stg[3 * e + 2]);
      }
    }
    base += fill;
    fill = 0;
  };
  auto append = [&](unsigned long long mask, bool pass, uint32_t i, uint32_t j, uint32_t d2_bits) {
    const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
    if (pass) {
      const uint32_t e = fill + rank;
      stg[3 * e] = i;
      stg[3 * e + 1] = j;
      stg[3 * e + 2] = d2_bits;
    }
    fill += __popcll(mask);
  };
  // Data out of range: nothing is found.  (Lists: by the same code, in the first panel; a branch past it would have acc cleared twice, 0.3 us of a call.)
  const bool none = !COUNT && __builtin_amdgcn_readfirstlane(ns.st) != ST_OK;
  const uint32_t end = none ? 0u : panels, reach = none ? 0u : n;
  float4v acc[RF][2];
  auto clear = [&]() {
#pragma unroll
    for (int f = 0; f < RF; ++f)
#pragma unroll
      for (int c = 0; c < 2; ++c) acc[f][c] = float4v{0.f, 0.f, 0.f, 0.f};
  };
  clear();
  // (pairs) the results in `hits` and acc, of 32 points from j0 on; their place is known
  auto emit = [&](uint32_t j0) __attribute__((always_inline)) {
    uint32_t l = lane;
    asm volatile("" : "+v"(l));  // (nothing of this is worked out before the loop over the points)
    const uint32_t r16 = l & 15, g = l >> 4;
#pragma unroll
    for (int R = 0; R < NR; ++R) {
      uint32_t h = R & 1 ? hits[R / 2] >> 16 : hits[R / 2] & 0xFFFFu;
      for (unsigned long long mask = __ballot(h != 0); mask; mask = __ballot(h != 0)) {
        if (fill + __popcll(mask) > a.staged) store_staged();
        const uint32_t r = (uint32_t)__builtin_ctz(h | 0x10000u);
        append(mask, h != 0, j0 + r16 + 4 * (r & 4u), 32 * R + 4 * g + 2 * (r & 8u) + (r & 3u),
               __float_as_uint(fmaxf(-2.f * pick(cat4(acc[2 * R][0], acc[2 * R][1], acc[2 * R + 1][0], acc[2 * R + 1][1]), r), 0.f)));
        h &= h - 1;
      }
    }
  };
  // the products of 32 points from j0 on are complete: the norm terms, the filter, the results
  auto finish = [&](uint32_t j0, float s0, float s1, bool last) __attribute__((always_inline)) {
    const uint32_t j = j0 + r16;
    uint2 p = make_uint2(P1_OUT_OF_RANGE, 0u), q = p;
    if (j < n) p = norm_pieces(s0, ns.m);
    if (j + 16 < n) q = norm_pieces(s1, ns.m);
    const half8 gb = as_half8(lane < 32 ? make_uint4(p.x, p.y, q.x, q.y) : column_constant);
    uint32_t first = 0, second = 0;  // (counts) of points j and j + 16
    bool full = false;               // (pairs) the rest have to wait for their place
#pragma unroll
    for (int R = 0; R < NR; ++R) {
      if (!COUNT && R % 2 == 0) hits[R / 2] = 0;
      const half8 ga = *reinterpret_cast<const half8*>(row_operand + R * row_step);
      const float16v v = __builtin_amdgcn_mfma_f32_32x32x16_f16(ga, gb, cat4(acc[2 * R][0], acc[2 * R][1], acc[2 * R + 1][0], acc[2 * R + 1][1]), 0, 0, 0);
      if constexpr (!COUNT) {
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[2 * R + q / 2][q % 2] = float4v{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
      }
      auto u = [&](int r) { return __float_as_uint(v[r]); };
      uint32_t least = min(min(u(0), u(1)), u(2));
#pragma unroll
      for (int r = 3; r < 15; r += 2) least = min(min(least, u(r)), u(r + 1));
      if (__ballot(min(least, u(15)) <= thr_bits) == 0) continue;
      uint32_t h = 0;
#pragma unroll
      for (int r = 0; r < 16; ++r) h |= v[r] >= a.thr ? 1u << r : 0u;
      h &= (32 * R + 32 <= nq ? 0xFFFFu : (32 * R < nq ? edge_mask : 0u)) & ((j < reach ? 0x0F0Fu : 0u) | (j + 16 < reach ? 0xF0F0u : 0u));
      if constexpr (COUNT) {
        first += __popc(h & 0x0F0Fu);
        second += __popc(h & 0xF0F0u);
        while (__ballot(h != 0)) {
          if (h) {
            const uint32_t r = (uint32_t)__builtin_ctz(h);
            atomicAdd(row_counts + 32 * R + 4 * g + 2 * (r & 8u) + (r & 3u), 1u);
            h &= h - 1;
          }
        }
      } else {
        for (unsigned long long mask = __ballot(h != 0); mask && !full; mask = __ballot(h != 0)) {
          full = fill + __popcll(mask) > a.staged;
          if (full) break;
          const uint32_t r = (uint32_t)__builtin_ctz(h | 0x10000u);
          append(mask, h != 0, j + 4 * (r & 4u), 32 * R + 4 * g + 2 * (r & 8u) + (r & 3u), __float_as_uint(fmaxf(-2.f * pick(v, r), 0.f)));
          h &= h - 1;
        }
        hits[R / 2] |= R & 1 ? h << 16 : h;
      }
    }
    if constexpr (!COUNT) {
      if (!full) return;
      uint32_t own = 0, more = 0;  // of this lane (at most 16 a region), of the wavefront
#pragma unroll
      for (int q = 0; q < (NR + 1) / 2; ++q) own += __popc(hits[q]);
#pragma unroll
      for (int bit = 1; bit <= 16 * NR; bit *= 2) more += bit * __popcll(__ballot(own & bit));
      if (last) {  // the workgroup's one atomic is next
        left = more;
        left_j0 = j0;
        return;
      }
      unsigned long long place = 0;
      if (lane == 0) place = atomicAdd(a.state, (unsigned long long)(fill + more)) & ONCE_FOUND;
      base = uniform(place);
      emit(j0);
      store_staged();
    }
    if constexpr (COUNT) {
      found += first + second;
      if (__ballot(first + second != 0)) {  // the four lanes of a point
        first += __shfl_xor(first, 16);
        first += __shfl_xor(first, 32);
        second += __shfl_xor(second, 16);
        second += __shfl_xor(second, 32);
      }
      if (lane < 32 && j0 + lane < n) a.counts_p[j0 + lane] = lane < 16 ? first : second;
    }
  };
  auto step = [&](auto b_c) __attribute__((always_inline)) -> bool {
    constexpr int B = decltype(b_c)::value;
    const bool ends = chunk + 1 == chunks;
    const uint32_t next_panel = ends ? panel + gridDim.x : panel, next_chunk = ends ? 0 : chunk + 1;
    load(std::integral_constant<int, 1 - B>{}, next_panel, next_chunk);
#pragma unroll
    for (int k = 0; k < CHUNK; ++k) {
      const int kb = (int)chunk * CHUNK + k;
      if (kb >= nkb) break;
#pragma unroll
      for (int f = 0; f < RF; ++f) {
        const half8 x = *reinterpret_cast<const half8*>(lds + (f * nkb + kb) * 1024 + lane * 16);
        acc[f][0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(x, buf[B][k][0], acc[f][0], 0, 0, 0);
        acc[f][1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(x, buf[B][k][1], acc[f][1], 0, 0, 0);
      }
    }
    if (ends) {
      const bool last = next_panel >= end;
      if (panel * TILE + wave * 32 < n) finish(panel * TILE + wave * 32, point_norm[B][0], point_norm[B][1], last);
      if (COUNT || !last) clear();
    }
    panel = next_panel;
    chunk = next_chunk;
    return panel < end;
  };
  if (!COUNT || ns.st == ST_OK) {
    while (step(std::integral_constant<int, 0>{}) && step(std::integral_constant<int, 1>{})) {}
  } else {  // data out of range: nothing is found
    for (; panel < panels; panel += gridDim.x)
      if (tid < TILE && panel * TILE + tid < n) a.counts_p[panel * TILE + tid] = 0;
  }

  // ---- what is left, and the workgroup's ticket
  if constexpr (COUNT) {
    found = wave_sum((uint32_t)found) + ((unsigned long long)wave_sum((uint32_t)(found >> 32)) << 32);
  }
  if (lane == 0) sums[wave] = COUNT ? found : fill + left;
  __syncthreads();
  if constexpr (COUNT) {
    if ((uint32_t)tid < nq && tid < ROWS && row_counts[tid] && a.counts_q) atomicAdd(a.counters + tid, row_counts[tid]);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // before the ticket
  }
  __syncthreads();
  __shared__ unsigned long long group_base;
  __shared__ bool last;
  if (tid == 0) {
    unsigned long long sum = 0, all = 0;
    for (int w = 0; w < FEW_WAVES; ++w) {
      const unsigned long long v = sums[w];
      sums[w] = sum;
      sum += v;
    }
    if (!COUNT) group_base = sum ? atomicAdd(a.state, sum) & ONCE_FOUND : 0;
    if (!COUNT) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const unsigned long long add = ONCE_TICKET | (COUNT ? sum : 0);
    last = close_by_xcd(a.state, gridDim.x, atomicAdd(state_of_xcd(a.state), add) + add, all);
    if (last) *(COUNT ? a.total : a.n_pairs) = all & ONCE_FOUND;
  }
  __syncthreads();
  if constexpr (!COUNT) {
    base = uniform(group_base + sums[wave]);
    if (left) emit(left_j0);
    store_staged();
  }
  if (COUNT && last && a.counts_q && (uint32_t)tid < nq)
    a.counts_q[tid] = __hip_atomic_exchange(a.counters + tid, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace

// ------------------------------------------------------------------------------------------
// Host side
// ------------------------------------------------------------------------------------------

// Workspace of the allocation-free entry point (ejoin_selfjoin_pairs_noalloc): device memory that exists from
// the moment the library is loaded, one copy per GPU.  Host code never uses this name as an address; it asks
// the runtime for the device address once per context (ejoin_create) and passes that to the kernels.
static __device__ __align__(256) unsigned char scratch[EJOIN_STATIC_SCRATCH_BYTES];

namespace {

// Device memory one call works in: either the context's own (grown on demand) or a carving of the static scratch.
struct Workspace {
  uint32_t* status;  // status block, 64 words (see k_reset)
  float* s;          // norms (4 B per point)
  uint32_t* maxima;  // behind them, small problems and the dense-tile call: largest norms of the norm kernels' workgroups (at most one per NORM_POINTS points)
  uint4* Xp;         // packed copy of X plus the augmentation k-block
};

}  // namespace

struct ejoin_ctx {
  int device;
  int num_cu;
  Workspace ws;      // owned by the context
  int64_t s_cap;     // points ws.s holds
  int64_t xp_bytes;  // bytes of ws.Xp
  bool ws_dirty;     // a call on ws did not reach its join kernel: the status block may hold leftovers
  unsigned char* once;            // device: k_join_once's state, slots and late counts, all zero between calls
  unsigned char* static_scratch;  // device address of `scratch` on this context's device
  uint32_t* last_status;          // status block of the last join or dense-tile call, and the stream it ran on
  hipStream_t last_stream;
  int profiling;
  hipEvent_t ev[4];
  int ev_valid;
  // batched result return (ejoin_selfjoin_pairs_to_host): a stream for the device-to-host copies, one event per
  // batch and the pair counter's value after each batch (pinned host memory)
  hipStream_t copy_stream;
  hipEvent_t batch_ev[EJOIN_MAX_BATCHES];
  unsigned long long* batch_count;
  char hip_error[256];
};

// A point set prepared once for many joins: its packed copy (data k-blocks + room for the augmentation
// block, which depends on the other set of each join and is rewritten per call), norms and largest norm.
struct ejoin_set {
  ejoin_ctx* ctx;
  int64_t n, pad;
  int32_t d;
  uint4* Xp;
  float* s;
  uint32_t* max_bits;  // device: FP32 bits of the largest norm
};

namespace {

int fail_hip(ejoin_ctx* ctx, hipError_t e, const char* what) {
  if (ctx) snprintf(ctx->hip_error, sizeof(ctx->hip_error), "%s: %s", what, hipGetErrorString(e));
  (void)hipGetLastError();
  return EJOIN_EHIP;
}

#define EJ_TRY(call)                                     \
  do {                                                   \
    hipError_t e_ = (call);                              \
    if (e_ != hipSuccess) return fail_hip(ctx, e_, #call); \
  } while (0)
#define EJ_RC(call)                 \
  do {                              \
    const int rc_ = (call);         \
    if (rc_ != EJOIN_OK) return rc_; \
  } while (0)

int64_t pad_rows(int64_t n) { return (n + TILE - 1) / TILE * TILE; }
int64_t pad_dims(int32_t d) { return ((int64_t)d + KPAD - 1) / KPAD * KPAD; }
// 32-coordinate k-blocks = MFMA steps per inner product: as many as hold a coordinate, not what the row stride is padded to (the
// sum over a block of zeros adds nothing to any accumulator).  The join kernel needs two slices per tile.  Against
// roundup(d, 64) / 32 blocks: 30,011 x 7,001 points, d = 200, join kernel 96.6 us, now 90.5; 9,299 FP32 points split, d = 400, 93.7, now 90.1.
int k_blocks(int32_t d) { return d <= 2 * KSLICE ? 2 : (d + KSLICE - 1) / KSLICE; }

int check_common(const ejoin_ctx* ctx, const void* X, int64_t n, int32_t d, int64_t ld) {
  if (!ctx || !X) return EJOIN_EINVAL;
  if (n < 1 || n >= (int64_t)0xFFFFFFFFll - TILE) return EJOIN_EINVAL;
  if (d < 1 || d > 65536) return EJOIN_EINVAL;
  if (ld < pad_dims(d) || (ld % KPAD) != 0) return EJOIN_EINVAL;
  if ((reinterpret_cast<uintptr_t>(X) & 127) != 0) return EJOIN_EINVAL;
  return EJOIN_OK;
}

bool bad_eps(float eps) { return !(eps >= 0.f) || !isfinite(eps); }

// Bytes of packed copy for `rows` (padded) points of dpad coordinates: the data k-blocks plus the augmentation block.
int64_t packed_bytes(int64_t rows, int64_t dpad) { return rows * (dpad + KSLICE) * 2; }

// The context's own workspace for `rows` points in total (each set padded to a multiple of TILE).
// dpad = 0: only the per-point arrays (norms); dpad > 0: also the packed copies.
// Growing frees the old arrays, which first waits for the device to be idle.
int ensure_workspace(ejoin_ctx* ctx, int64_t rows, int64_t dpad) {
  Workspace& w = ctx->ws;
  if (rows > ctx->s_cap) {
    if (w.s) {
      EJ_TRY(hipDeviceSynchronize());
      EJ_TRY(hipFree(w.s));
      w.s = nullptr;
      ctx->s_cap = 0;
    }
    hipError_t e = hipMalloc(reinterpret_cast<void**>(&w.s), (size_t)(rows + rows / NORM_POINTS) * sizeof(float));  // (+ maxima)
    if (e != hipSuccess) {
      (void)hipGetLastError();
      w.s = nullptr;
      if (e == hipErrorOutOfMemory) return EJOIN_ENOMEM;
      return fail_hip(ctx, e, "hipMalloc(workspace)");
    }
    w.maxima = reinterpret_cast<uint32_t*>(w.s + rows);
    ctx->s_cap = rows;
  }
  const int64_t need = dpad > 0 ? packed_bytes(rows, dpad) : 0;
  if (need > ctx->xp_bytes) {
    if (w.Xp) {
      EJ_TRY(hipDeviceSynchronize());
      EJ_TRY(hipFree(w.Xp));
      w.Xp = nullptr;
      ctx->xp_bytes = 0;
    }
    hipError_t e = hipMalloc(reinterpret_cast<void**>(&w.Xp), (size_t)need);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      if (e == hipErrorOutOfMemory) return EJOIN_ENOMEM;
      return fail_hip(ctx, e, "hipMalloc(packed X)");
    }
    ctx->xp_bytes = need;
  }
  return EJOIN_OK;
}

// The static scratch cut up for a self-join of `pad` (padded) points of dpad coordinates; false if it does not fit.
// Every piece starts on a 256-byte boundary.  (The limit that ejoin.h states for it counts 20 bytes per point besides the packed copy:
// 4 for the norms, 16 at whose start the maxima lie.)
bool carve_static(unsigned char* base, int64_t pad, int64_t dpad, Workspace& w) {
  auto up = [](int64_t x) { return (x + 255) / 256 * 256; };
  const int64_t off_s = 256, off_max = off_s + up(pad * 4), off_Xp = off_max + up(pad * 16);
  const int64_t end = off_Xp + packed_bytes(pad, dpad);
  if (end > (int64_t)EJOIN_STATIC_SCRATCH_BYTES) return false;
  w.status = reinterpret_cast<uint32_t*>(base);
  w.s = reinterpret_cast<float*>(base + off_s);
  w.maxima = reinterpret_cast<uint32_t*>(base + off_max);
  w.Xp = reinterpret_cast<uint4*>(base + off_Xp);
  return true;
}

// Workgroup size of the norm kernels.  Large sets: eight wavefronts, so that the atomics of the workgroups (11 ns each) take
// less time than the data; small sets: one, so that they spread over the CUs.
int norm_threads(int64_t waves) { return waves >= 2048 ? 512 : (waves >= 512 ? 256 : 64); }

// Norms of X into s (and, with Xp given, the packed copy of X); max_bits may be null.
int launch_norms(ejoin_ctx* ctx, const uint16_t* X, int64_t n, int32_t d, int64_t ld, float* s, uint32_t* max_bits, uint4* Xp,
                 hipStream_t st, uint32_t* maxima = nullptr, uint32_t* nmaxima = nullptr) {
  const int64_t npad = pad_rows(n);
  if (!Xp && !max_bits && !maxima && n < (1ll << 30)) {  // norms alone (a grid has fewer than 2^32 threads)
    hipLaunchKernelGGL((norms_from_the_end(n, ld) ? k_norms<false, 1, true> : k_norms<false, 1>), dim3((unsigned)((n + 15) / 16)), dim3(64), 0, st, X, n, npad, ld,
                       k_blocks(d), s, max_bits, Xp, 0, maxima);
    EJ_TRY(hipGetLastError());
    return EJOIN_OK;
  }
  const int64_t waves = ((Xp ? npad : n) + NORM_POINTS - 1) / NORM_POINTS;
  const int threads = norm_threads(waves);
  const dim3 grid((unsigned)((waves * 64 + threads - 1) / threads));
  if (nmaxima) *nmaxima = grid.x;
  if (Xp) hipLaunchKernelGGL(k_norms<true>, grid, dim3(threads), 0, st, X, n, npad, ld, k_blocks(d), s, max_bits, Xp, k_blocks(d) + 1, maxima);
  else hipLaunchKernelGGL(k_norms<false>, grid, dim3(threads), 0, st, X, n, npad, ld, k_blocks(d), s, max_bits, Xp, 0, maxima);
  EJ_TRY(hipGetLastError());
  return EJOIN_OK;
}

// Norms and packed copies of both sets of a join in one launch (B.npad == 0: one set; X == nullptr: a set prepared before).  Sets
// the sets' numbers of workgroups.  p: where the maxima go and what is cleared.
int launch_prep(ejoin_ctx* ctx, PrepSet& A, PrepSet& B, int nkb, PrepArgs& p, hipStream_t st) {
  const int64_t wavesA = A.X ? A.npad / NORM_POINTS : 0, wavesB = B.X ? B.npad / NORM_POINTS : 0;
  const int threads = norm_threads(wavesA + wavesB), per = threads / 64;
  A.groups = (uint32_t)((wavesA + per - 1) / per);
  B.groups = (uint32_t)((wavesB + per - 1) / per);
  p.a = A;
  p.b = B;
  p.k32steps = nkb;
  // enough workgroups that none clears more than 16 counts per thread
  const uint32_t clearing = p.counts ? (uint32_t)((p.ncounts + 16 * threads - 1) / (16 * threads)) : 0u, norming = A.groups + B.groups;
  hipLaunchKernelGGL(k_prep, dim3(clearing > norming ? clearing : norming), dim3(threads), 0, st, p);
  EJ_TRY(hipGetLastError());
  return EJOIN_OK;
}

// What follows the norms of a k_join call, for both its sets in one launch (B.npad == 0: one set): the augmentation operands, from
// the norms and the largest norm of all (in the status block; set_max: that of a prepared set), and what the call needs zero.
int launch_aux(ejoin_ctx* ctx, uint32_t* status, const uint32_t* set_max, const AuxSet& A, const AuxSet& B, int data_blocks,
               unsigned long long* counter, hipStream_t st) {
  const AuxArgs a{A, B, status, set_max, data_blocks, counter};
  hipLaunchKernelGGL(k_aux, dim3((unsigned)((A.npad + B.npad) / 256)), dim3(256), 0, st, a);
  EJ_TRY(hipGetLastError());
  return EJOIN_OK;
}

struct DeviceGuard {
  int prev;
  bool ok;
  explicit DeviceGuard(int dev) : prev(-1), ok(false) {
    if (hipGetDevice(&prev) != hipSuccess) return;
    ok = (prev == dev) || (hipSetDevice(dev) == hipSuccess);
  }
  ~DeviceGuard() {
    int cur = -1;
    if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
  }
};

// Where a call's results go.
struct Results {
  uint32_t* pairs = nullptr;
  float* dist2 = nullptr;
  uint64_t capacity = 0;
  uint64_t* n_pairs = nullptr;
  uint32_t* counts = nullptr;
  uint32_t* counts_b = nullptr;
  uint64_t* total = nullptr;
  unsigned long long* counter(bool count) const { return reinterpret_cast<unsigned long long*>(count ? total : n_pairs); }
};

// One packed operand set of a join.
struct Operand {
  const uint4* Xp;
  int64_t n, pad;
};

// Opens a call on workspace w: first profiling event, and the status block brought to its between-calls state
// if it may not be in it (always for the static scratch, which every context of the device shares).
int begin_call(ejoin_ctx* ctx, const Workspace& w, bool own, hipStream_t st) {
  if (ctx->profiling) EJ_TRY(hipEventRecord(ctx->ev[0], st));
  if (!own || ctx->ws_dirty) {
    hipLaunchKernelGGL(k_reset, dim3(1), dim3(64), 0, st, w.status);
    EJ_TRY(hipGetLastError());
  }
  if (own) ctx->ws_dirty = true;  // until the join kernel, which leaves the block clean, has been launched
  ctx->last_status = w.status;
  ctx->last_stream = st;
  return EJOIN_OK;
}

// What the join kernels of every size take.
JoinArgs join_args(const Workspace& w, const Operand& A, const Operand& B, bool self, int nslices, float eps, const Results& r, int tile) {
  JoinArgs a;
  memset(&a, 0, sizeof(a));
  a.XpA = A.Xp;
  a.XpB = B.Xp;
  a.nA = A.n;
  a.nB = B.n;
  a.self = self ? 1 : 0;
  a.status = w.status;
  a.nslices = nslices;
  a.thr = -0.5f * (eps * eps);
  a.ntilesA = (uint32_t)((A.n + tile - 1) / tile);
  a.ntilesB = (uint32_t)((B.n + tile - 1) / tile);
  a.sb_row_end = 0xFFFFFFFFu;
  a.pairs = r.pairs;
  a.dist2 = r.dist2;
  a.capacity = r.capacity;
  a.n_pairs = reinterpret_cast<unsigned long long*>(r.n_pairs);
  a.counts = r.counts;
  a.counts_b = r.counts_b;
  a.total = reinterpret_cast<unsigned long long*>(r.total);
  return a;
}

// k_join_strip of nkb k-blocks (2 .. EJ_STRIP_KB_MAX), and its LDS
typedef void (*JoinKernel)(JoinArgs);
template <bool COUNT, int... N>
JoinKernel strip_kernel_of(int nkb, std::integer_sequence<int, N...>) {
  static const JoinKernel k[] = {&k_join_strip<COUNT, N + 2>...};
  return k[nkb - 2];
}
template <int... N>
int strip_lds_of(int nkb, std::integer_sequence<int, N...>) {
  static const int b[] = {Strip<N + 2>::LDS...};
  return b[nkb - 2];
}
template <bool COUNT>
JoinKernel strip_kernel(int nkb) { return strip_kernel_of<COUNT>(nkb, std::make_integer_sequence<int, EJ_STRIP_KB_MAX - 1>{}); }
int strip_lds(int nkb) { return strip_lds_of(nkb, std::make_integer_sequence<int, EJ_STRIP_KB_MAX - 1>{}); }

StripPlan plan_strip(const ejoin_ctx* ctx, int64_t nA, int64_t nB, bool self, int nkb, bool count) {
  StripPlan p = strip_plan(ctx->num_cu, nA, nB, self, nkb, count);
#ifdef EJOIN_ONLY_K_JOIN
  p.use = false;
#endif
#ifdef EJOIN_ONLY_K_JOIN_STRIP
  p.use = nkb <= EJ_STRIP_KB_MAX;
#endif
  return p;
}

// The join kernel on two packed operand sets whose augmentation blocks are in place.
template <bool COUNT>
int launch_join(ejoin_ctx* ctx, const Workspace& w, bool own, const Operand& A, const Operand& B, bool self, int nslices, float eps,
                const Results& r, hipStream_t st, bool split = false, uint32_t sb_row_begin = 0, uint32_t sb_row_end = 0xFFFFFFFFu) {
  JoinArgs a = join_args(w, A, B, self, nslices, eps, r, TILE);
  a.sb_row_begin = sb_row_begin;
  a.sb_row_end = sb_row_end;
  a.xcd_bar = w.status + 8;
  {
    // re-align the workgroups of each XCD every few hundred microseconds: about 512 slices
    // (measured on MI355X: +12..16 % over never aligning; every tile costs more than it gains)
    const int per = 512 / (a.nslices + 1);
    a.sync_mode = per < 8 ? 8 : (per > 128 ? 128 : per);
    // a launch that ends before the first re-alignment would come starts without one too: its workgroups begin within a microsecond
    // or two of each other, and the start's costs about three (30,011 x 7,001, d = 200: 95.8 us, now 93.1; 24,680 points,
    // d = 384: 186.8, now 183.2)
    const int64_t tiles = self ? (int64_t)a.ntilesA * (a.ntilesA + 1) / 2 : (int64_t)a.ntilesA * a.ntilesB;
    if (tiles <= (int64_t)a.sync_mode * ctx->num_cu) a.sync_mode = 0;
#ifdef EJOIN_ABL_NOALIGN
    a.sync_mode = 0;
#endif
  }
  if (ctx->profiling) {
    EJ_TRY(hipEventRecord(ctx->ev[1], st));
    EJ_TRY(hipEventRecord(ctx->ev[2], st));
  }
  // Counts of sets of up to 32,768 points go to the instance for dense tiles.  Points in random order have 65,536 S / n hits a tile
  // at S neighbours: the smaller the set, the fuller its regions.  It is the better one from a few hundred neighbours on and the
  // other one below (30,000 points, d = 384: S = 30 280 us against 275, S = 100 332 against 305, S = 512 406 against 451; 15,000:
  // 87 against 83, 122 against 96, 123 against 158); beyond 32,768 points few sets are that dense, and the other instance counts what
  // dense tiles there are in the LDS, from its queue (100,000 points, d = 128, stored cluster by cluster, S = 900: 4.4 ms without).
  constexpr int64_t DENSE_POINTS = 32768;
  const bool dense = COUNT && A.n <= DENSE_POINTS && B.n <= DENSE_POINTS;
  JoinKernel kernel = split ? (dense ? &k_join<COUNT, COUNT, true> : &k_join<COUNT, false, true>) : (dense ? &k_join<COUNT, COUNT, false> : &k_join<COUNT, false, false>);
  int lds_bytes = LDS_BYTES;
  const StripPlan strip = split ? StripPlan{false, false} : plan_strip(ctx, A.n, B.n, self, a.nslices, COUNT);
  if (strip.use) {
    kernel = strip_kernel<COUNT>(a.nslices);
    lds_bytes = strip_lds(a.nslices);
    if (strip.swapped) {
      a.swapped = 1;
      std::swap(a.XpA, a.XpB);
      std::swap(a.nA, a.nB);
      std::swap(a.ntilesA, a.ntilesB);
      std::swap(a.counts, a.counts_b);
    }
    const int64_t panels = strip_panels(a.nA), per = SB * TILE / EJ_STRIP_ROWS;
    a.sb_row_begin = (uint32_t)(sb_row_begin * per);
    a.sb_row_end = (uint32_t)(sb_row_end < (panels + per - 1) / per ? sb_row_end * per : panels);
    a.sync_mode = 1024 / a.nslices;  // stages between two alignments: about as long as 512 slices of k_join
    if (panels * strip_stages(a.nB) / (self ? 2 : 1) <= (int64_t)a.sync_mode * ctx->num_cu) a.sync_mode = 0;
  }
  hipLaunchKernelGGL(kernel, dim3(ctx->num_cu), dim3(THREADS), lds_bytes, st, a);
  EJ_TRY(hipGetLastError());
  if (own) ctx->ws_dirty = false;
  if (ctx->profiling) {
    EJ_TRY(hipEventRecord(ctx->ev[3], st));
    ctx->ev_valid = 1;
  }
  return EJOIN_OK;
}

// Which tile k_join_small should work a problem in that k_join_once does not take (or a prepared or split set), or 0: k_join.  In tiles of 64 up to 300 of them (1,000 points, 136 tiles:
// 13.0 us a call against 14.0 in tiles of 128 and 23.7 by k_join; 2,000 points, 528 tiles: 15.5, 14.2, 21.8).  In tiles of 128
// where the CUs, which hold 768 of them, need no more rounds for them than k_join for its 256 at a time (at d = 64, 384 and
// 960: one round 10 + 4.5, 7 + 10.5, 0 + 24 us, further ones 4.5, 10.5, 24; k_join 10.5 + 5, 11 + 11, 11 + 22), or one more
// where it is at least the fourth and a tile has few slices (9,000 points, d = 64: 30.8 us against 33.6; d = 960: 101 against
// 97).  Two sets: two rounds at most, the operands of a long thin grid are read once and k_join's copies keep ahead better
// (200,000 x 60, d = 384: 67 us against 60).
int small_tile(const ejoin_ctx* ctx, int64_t nA, int64_t nB, bool self, int nslices) {
  auto tiles = [&](int64_t t) {
    const int64_t a = (nA + t - 1) / t, b = (nB + t - 1) / t;
    return self ? a * (a + 1) / 2 : a * b;
  };
#if defined(EJOIN_ONLY_K_JOIN) || defined(EJOIN_ONLY_K_JOIN_STRIP)
  return 0;
#endif
  if (tiles(64) <= 300) return 64;
  const int64_t held = (int64_t)ctx->num_cu * small_groups_per_cu<128>();
  const int64_t rounds = (tiles(128) + held - 1) / held, other = (tiles(TILE) + ctx->num_cu - 1) / ctx->num_cu;
  if (!self) return rounds <= 2 && rounds <= other ? 128 : 0;
  return rounds <= other + (rounds >= 4 && nslices <= 12 ? 1 : 0) ? 128 : 0;
}

template <bool COUNT, int TS>
int launch_small(ejoin_ctx* ctx, const SmallArgs& a, hipStream_t st) {
  const int64_t tiles = a.j.self ? (int64_t)a.j.ntilesA * (a.j.ntilesA + 1) / 2 : (int64_t)a.j.ntilesA * a.j.ntilesB;
  const int64_t most = (int64_t)ctx->num_cu * small_groups_per_cu<TS>();  // what the CUs hold at a time
  const int64_t groups = (tiles + NUM_XCD - 1) / NUM_XCD * NUM_XCD;
  hipLaunchKernelGGL((k_join_small<COUNT, TS>), dim3((unsigned)(groups < most ? groups : most)), dim3(256), (small_lds_bytes<COUNT, TS>()), st, a);
  EJ_TRY(hipGetLastError());
  return EJOIN_OK;
}

// The preparation of a split-FP16 join; groups: its number of workgroups.
int launch_split_prep(ejoin_ctx* ctx, const SplitArgs& a, uint32_t& groups, hipStream_t st) {
  const int64_t waves = a.npad / NORM_POINTS;
  const int threads = norm_threads(waves);
  groups = (uint32_t)((waves * 64 + threads - 1) / threads);
  hipLaunchKernelGGL(k_split_prep, dim3(groups), dim3(threads), 0, st, a);
  EJ_TRY(hipGetLastError());
  return EJOIN_OK;
}

// A join by k_prep (split: k_split_prep) and k_join_small.  B.npad == 0: self-join of A.  A.X == nullptr: A is a prepared set (its largest norm: set_max).
// Neither kernel reads or leaves anything in the status block but the status word.
template <bool COUNT>
int run_small(ejoin_ctx* ctx, const Workspace& w, int tile, PrepSet A, PrepSet B, const uint32_t* set_max, int nkb, float eps, const Results& r,
              hipStream_t st, SplitArgs* split = nullptr) {
  const bool self = B.npad == 0;
  if (ctx->profiling) EJ_TRY(hipEventRecord(ctx->ev[0], st));
  ctx->last_status = w.status;
  ctx->last_stream = st;
  uint32_t* maxima = w.maxima;
  SmallArgs a;
  if (split) {
    split->maxima = maxima;
    split->counter = r.counter(COUNT);
    split->counts = r.counts;
    EJ_RC(launch_split_prep(ctx, *split, a.nmaxima, st));
  } else {
    PrepArgs p;
    memset(&p, 0, sizeof(p));
    p.maxima = maxima;
    p.counter = r.counter(COUNT);
    p.counts = r.counts;
    p.ncounts = A.n;
    p.counts_b = r.counts_b;
    p.ncounts_b = B.n;
    EJ_RC(launch_prep(ctx, A, B, nkb, p, st));
    a.nmaxima = A.groups + B.groups;
  }
  const Operand OA{A.Xp, A.n, A.npad}, OB{self ? A.Xp : B.Xp, self ? A.n : B.n, self ? A.npad : B.npad};
  const int nslices = split ? 3 * nkb : nkb;
  a.j = join_args(w, OA, OB, self, nslices, eps, r, tile);
  a.sA = A.s;
  a.sB = self ? A.s : B.s;
  a.maxima = maxima;
  a.set_max = set_max;
  a.data_blocks = split ? 2 * nkb : nkb;
  a.nkb_split = split ? nkb : 0x3FFFFFFF;
  if (ctx->profiling) {
    EJ_TRY(hipEventRecord(ctx->ev[1], st));
    EJ_TRY(hipEventRecord(ctx->ev[2], st));
  }
  EJ_RC(tile == 64 ? (launch_small<COUNT, 64>(ctx, a, st)) : (launch_small<COUNT, 128>(ctx, a, st)));
  if (ctx->profiling) {
    EJ_TRY(hipEventRecord(ctx->ev[3], st));
    ctx->ev_valid = 1;
  }
  return EJOIN_OK;
}

// Which tile k_join_once works a join of FP16 rows in, or 0: another kernel.
int once_edge(const ejoin_ctx* ctx, int64_t nA, int64_t nB, bool self, int nkb, bool count) {
#if defined(EJOIN_ONLY_K_JOIN) || defined(EJOIN_ONLY_K_JOIN_STRIP)
  return 0;
#endif
  return once_tile_edge(ctx->num_cu, nA, nB, self, nkb, count);
}
// A join by k_join_once.  XB == nullptr: self-join of XA.
template <bool COUNT>
int run_once(ejoin_ctx* ctx, const Workspace& w, int tile, const uint16_t* XA, int64_t nA, int64_t ldA, const uint16_t* XB, int64_t nB, int64_t ldB,
             int nkb, float eps, const Results& r, hipStream_t st) {
  const bool self = XB == nullptr;
  for (int e = 0; ctx->profiling && e < 3; ++e) EJ_TRY(hipEventRecord(ctx->ev[e], st));
  ctx->last_status = w.status;
  ctx->last_stream = st;
  OnceArgs a;
  a.j = join_args(w, Operand{nullptr, nA, 0}, Operand{nullptr, self ? nA : nB, 0}, self, nkb, eps, r, tile);
  a.XA = XA;
  a.XB = self ? XA : XB;
  a.ldA = ldA;
  a.ldB = self ? ldA : ldB;
  a.sA = w.s;
  a.sB = w.s + pad_rows(nA);
  a.tiles = self ? a.j.ntilesA * (a.j.ntilesA + 1) / 2 : a.j.ntilesA * a.j.ntilesB;
  a.slots_a = (uint32_t)((nA + 63) / 64);
  a.slots = a.slots_a + (self ? 0u : (uint32_t)((nB + 63) / 64));
  a.state = reinterpret_cast<unsigned long long*>(ctx->once);
  a.slot = reinterpret_cast<uint32_t*>(ctx->once + ONCE_STATE_BYTES);
  a.late_counts = a.slot + NUM_XCD * ONCE_SLOTS;
  hipLaunchKernelGGL((tile == 64 ? k_join_once<COUNT, 64> : k_join_once<COUNT, 128>), dim3(a.tiles), dim3(tile == 64 ? Once<64>::THREADS : Once<128>::THREADS),
                     (tile == 64 ? Once<64>::LDS : Once<128>::LDS), st, a);
  EJ_TRY(hipGetLastError());
  if (ctx->profiling) {
    EJ_TRY(hipEventRecord(ctx->ev[3], st));
    ctx->ev_valid = 1;
  }
  return EJOIN_OK;
}

// Norms, packed copies and augmentation operands of the sets of a k_join call, and its results cleared.
int prep_and_aux(ejoin_ctx* ctx, const Workspace& w, PrepSet A, PrepSet B, const uint32_t* set_max, int nkb, unsigned long long* counter, const Results& r,
                 hipStream_t st) {
  PrepArgs p;
  memset(&p, 0, sizeof(p));
  p.max_bits = w.status + 1;
  EJ_RC(launch_prep(ctx, A, B, nkb, p, st));
  return launch_aux(ctx, w.status, set_max, AuxSet{A.s, A.n, A.npad, A.Xp, r.counts}, AuxSet{B.s, B.n, B.npad, B.Xp, r.counts_b}, nkb, counter, st);
}

// Join of FP16 rows in workspace w (the context's own, or a carving of the static scratch).  XB == nullptr: self-join of XA.
// batch_rows (self-join, pair mode only): null, or nbatches + 1 ascending bounds in rows of super-blocks; the join kernel is
// then launched once per range, and after each launch the pair counter is copied to ctx->batch_count[b] and
// ctx->batch_ev[b] recorded (the counter runs on from launch to launch: the pairs of batch b are those between the
// counts of batch b - 1 and b).
template <bool COUNT>
int run_join(ejoin_ctx* ctx, const Workspace& w, bool own, const uint16_t* XA, int64_t nA, int64_t ldA, const uint16_t* XB, int64_t nB,
             int64_t ldB, int32_t d, float eps, const Results& r, hipStream_t st, const uint32_t* batch_rows = nullptr, int nbatches = 0) {
  const bool self = (XB == nullptr);
  const int64_t padA = pad_rows(nA), padB = self ? 0 : pad_rows(nB);
  const int nkb = k_blocks(d);
  PrepSet SA{XA, nA, padA, ldA, w.s, w.Xp, 0}, SB{XB, nB, padB, ldB, w.s + padA, w.Xp + padA * (int64_t)(nkb + 1) * 4, 0};
  uint4 *XpA = SA.Xp, *XpB = SB.Xp;
  auto batch_done = [&](int b) -> int {
    EJ_TRY(hipMemcpyAsync(ctx->batch_count + b, r.n_pairs, sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
    EJ_TRY(hipEventRecord(ctx->batch_ev[b], st));
    return EJOIN_OK;
  };
  // (one batch is the plain join: every self-join of up to 4,096 points, which one row of super-blocks covers)
  const bool plain = !batch_rows || nbatches == 1;
  const int once = plain ? once_edge(ctx, nA, self ? nA : nB, self, nkb, COUNT) : 0;
  const int small = plain && !once ? small_tile(ctx, nA, self ? nA : nB, self, nkb) : 0;
  if (once || small) {
    EJ_RC(once ? run_once<COUNT>(ctx, w, once, XA, nA, ldA, XB, nB, ldB, nkb, eps, r, st) : run_small<COUNT>(ctx, w, small, SA, SB, nullptr, nkb, eps, r, st));
    return batch_rows ? batch_done(0) : EJOIN_OK;
  }
  EJ_RC(begin_call(ctx, w, own, st));
  EJ_RC(prep_and_aux(ctx, w, SA, SB, nullptr, nkb, r.counter(COUNT), r, st));
  const Operand A{XpA, nA, padA}, B{self ? XpA : XpB, self ? nA : nB, self ? padA : padB};
  if (!batch_rows) return launch_join<COUNT>(ctx, w, own, A, B, self, nkb, eps, r, st);
  for (int b = 0; b < nbatches; ++b) {
    if (b > 0) {  // the XCD alignment counters start every launch from zero
      hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, st, w.status + 8, (int64_t)NUM_XCD, 0u);
      EJ_TRY(hipGetLastError());
    }
    EJ_RC(launch_join<COUNT>(ctx, w, own, A, B, self, nkb, eps, r, st, false, batch_rows[b], batch_rows[b + 1]));
    EJ_RC(batch_done(b));
  }
  return EJOIN_OK;
}

// Split-FP16 self-join of FP32 rows (see k_split_prep): the join kernels on 3 * nkb slices.
template <bool COUNT>
int run_join_split(ejoin_ctx* ctx, const float* X32, int64_t n, int32_t d, int64_t ld32, float eps, const Results& r, hipStream_t st) {
  const int64_t pad = pad_rows(n);
  EJ_RC(ensure_workspace(ctx, pad, 2 * pad_dims(d)));  // 2 * nkb data blocks + 1 augmentation block
  const Workspace& w = ctx->ws;
  const int nkb = (d + KSLICE - 1) / KSLICE;
  SplitArgs p{X32, n, pad, ld32, d, nkb, w.s, w.Xp, nullptr, nullptr, nullptr, nullptr};
  PrepSet S{nullptr, n, pad, 0, w.s, w.Xp, 0}, none{};
  if (const int tile = small_tile(ctx, n, n, true, 3 * nkb)) return run_small<COUNT>(ctx, w, tile, S, none, nullptr, nkb, eps, r, st, &p);
  EJ_RC(begin_call(ctx, w, true, st));
  p.max_bits = w.status + 1;
  uint32_t groups = 0;
  EJ_RC(launch_split_prep(ctx, p, groups, st));
  EJ_RC(launch_aux(ctx, w.status, nullptr, AuxSet{w.s, n, pad, w.Xp, r.counts}, AuxSet{}, 2 * nkb, r.counter(COUNT), st));
  const Operand A{w.Xp, n, pad};
  return launch_join<COUNT>(ctx, w, true, A, A, true, 3 * nkb, eps, r, st, true);
}

typedef void (*FewKernel)(FewArgs);
template <bool COUNT>
FewKernel few_kernel(int rf) { return rf == 2 ? &k_join_few<COUNT, 2> : rf == 4 ? &k_join_few<COUNT, 4> : rf == 8 ? &k_join_few<COUNT, 8> : &k_join_few<COUNT, 16>; }
int few_workgroups(const ejoin_ctx* ctx, int64_t n, int rf, int lds_bytes) {
  const int64_t panels = (n + TILE - 1) / TILE, most = (int64_t)ctx->num_cu * few_groups_per_cu(rf, lds_bytes), rounds = (panels + most - 1) / most;
  return (int)((panels + rounds - 1) / rounds);
}
// Groups of 16 query points that k_join_few should hold for nQ of them against a prepared set of n, or 0: another kernel.
int few_groups(int64_t n, int64_t nQ, int nkb, bool count) {
#if defined(EJOIN_ONLY_K_JOIN) || defined(EJOIN_ONLY_K_JOIN_STRIP)
  return 0;
#endif
  const int rf = few_groups_of(nQ);
  return rf && few_lds_bytes<false>(16 * rf, nkb, few_staged(rf, nkb)) <= FEW_LDS && few_pays(n, nQ, rf, nkb, count) ? rf : 0;
}
template <bool COUNT>
int run_few(ejoin_ctx* ctx, const Workspace& w, const ejoin_set* P, int rf, int nkb, const uint16_t* XQ, int64_t nQ, int64_t ldQ, float eps, const Results& r,
            hipStream_t st) {
  for (int e = 0; ctx->profiling && e < 3; ++e) EJ_TRY(hipEventRecord(ctx->ev[e], st));
  ctx->last_status = w.status;
  ctx->last_stream = st;
  const int staged = few_staged(rf, nkb), lds_bytes = few_lds_bytes<COUNT>(16 * rf, nkb, staged);
  const int groups = few_workgroups(ctx, P->n, rf, lds_bytes);
  const FewArgs a{P->Xp, P->s, P->max_bits, P->n, nkb, XQ, nQ, ldQ, -0.5f * (eps * eps), w.status, r.pairs, r.dist2, r.capacity,
                  reinterpret_cast<unsigned long long*>(r.n_pairs), (uint32_t)staged, r.counts, r.counts_b, reinterpret_cast<unsigned long long*>(r.total),
                  reinterpret_cast<unsigned long long*>(ctx->once), reinterpret_cast<uint32_t*>(ctx->once + ONCE_STATE_BYTES) + NUM_XCD * ONCE_SLOTS};
  hipLaunchKernelGGL(few_kernel<COUNT>(rf), dim3((unsigned)groups), dim3(64 * FEW_WAVES), lds_bytes, st, a);
  EJ_TRY(hipGetLastError());
  if (ctx->profiling) {
    EJ_TRY(hipEventRecord(ctx->ev[3], st));
    ctx->ev_valid = 1;
  }
  return EJOIN_OK;
}

// Two-set join of a prepared point set with query points given as FP16 rows.
template <bool COUNT>
int run_join_prepared(ejoin_ctx* ctx, const ejoin_set* P, const uint16_t* XQ, int64_t nQ, int64_t ldQ, float eps, const Results& r,
                      hipStream_t st) {
  const int32_t d = P->d;
  const int64_t padQ = pad_rows(nQ);
  EJ_RC(ensure_workspace(ctx, padQ, pad_dims(d)));
  const Workspace& w = ctx->ws;
  const int nkb = k_blocks(d);
  if (const int rf = few_groups(P->n, nQ, nkb, COUNT)) return run_few<COUNT>(ctx, w, P, rf, nkb, XQ, nQ, ldQ, eps, r, st);
  PrepSet SP{nullptr, P->n, P->pad, 0, P->s, P->Xp, 0}, SQ{XQ, nQ, padQ, ldQ, w.s, w.Xp, 0};
  if (const int tile = small_tile(ctx, P->n, nQ, false, nkb)) return run_small<COUNT>(ctx, w, tile, SP, SQ, P->max_bits, nkb, eps, r, st);
  EJ_RC(begin_call(ctx, w, true, st));
  // the augmentation rows of both sets are scaled to the largest norm of the two: those of the prepared set are rewritten
  EJ_RC(prep_and_aux(ctx, w, SP, SQ, P->max_bits, nkb, r.counter(COUNT), r, st));
  const Operand A{P->Xp, P->n, P->pad}, B{w.Xp, nQ, padQ};
  return launch_join<COUNT>(ctx, w, true, A, B, false, nkb, eps, r, st);
}

int check_f32(const ejoin_ctx* ctx, const float* X32, int64_t n, int32_t d, int64_t ld32) {
  if (!ctx || !X32) return EJOIN_EINVAL;
  if (n < 1 || n >= (int64_t)0xFFFFFFFFll - TILE || d < 1 || d > 65536 / 4 || ld32 < d) return EJOIN_EINVAL;
  if ((int64_t)pad_rows(n) * (pad_dims(d) / KSLICE) * 4 / 256 > 0x7FFFFFFFll) return EJOIN_EUNSUPPORTED;  // (beyond any device's memory)
  return EJOIN_OK;
}

// Arguments of a pair-list call / a count call that every entry point checks the same way.
int check_pairs_out(const uint32_t* pairs, uint64_t capacity, const uint64_t* n_pairs, float eps) {
  return (!n_pairs || (!pairs && capacity > 0) || bad_eps(eps)) ? EJOIN_EINVAL : EJOIN_OK;
}
int check_count_out(const uint32_t* counts, const uint64_t* total, float eps) {
  return (!counts || !total || bad_eps(eps)) ? EJOIN_EINVAL : EJOIN_OK;
}

Results pair_results(uint32_t* pairs, float* dist2, uint64_t capacity, uint64_t* n_pairs) {
  Results r;
  r.pairs = pairs;
  r.dist2 = dist2;
  r.capacity = capacity;
  r.n_pairs = n_pairs;
  return r;
}
Results count_results(uint32_t* counts, uint32_t* counts_b, uint64_t* total) {
  Results r;
  r.counts = counts;
  r.counts_b = counts_b;
  r.total = total;
  return r;
}

// FP16 join on the context's own workspace.
template <bool COUNT>
int join_on_ctx(ejoin_ctx* ctx, const uint16_t* XA, int64_t nA, int64_t ldA, const uint16_t* XB, int64_t nB, int64_t ldB, int32_t d,
                float eps, const Results& r, void* stream) {
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return EJOIN_EHIP;
  EJ_RC(ensure_workspace(ctx, pad_rows(nA) + (XB ? pad_rows(nB) : 0), pad_dims(d)));
  return run_join<COUNT>(ctx, ctx->ws, true, XA, nA, ldA, XB, nB, ldB, d, eps, r, static_cast<hipStream_t>(stream));
}

}  // namespace

extern "C" {

int ejoin_create(ejoin_ctx** out, int device) {
  if (!out) return EJOIN_EINVAL;
  *out = nullptr;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev) {
    (void)hipGetLastError();
    return EJOIN_EINVAL;
  }
  hipDeviceProp_t prop;
  if (hipGetDeviceProperties(&prop, device) != hipSuccess) {
    (void)hipGetLastError();
    return EJOIN_EHIP;
  }
  if (strncmp(prop.gcnArchName, "gfx950", 6) != 0) return EJOIN_EUNSUPPORTED;
  ejoin_ctx* ctx = new (std::nothrow) ejoin_ctx();
  if (!ctx) return EJOIN_ENOMEM;
  memset(ctx, 0, sizeof(*ctx));
  ctx->device = device;
  ctx->num_cu = prop.multiProcessorCount;
  DeviceGuard guard(device);
  if (!guard.ok) {
    delete ctx;
    return EJOIN_EHIP;
  }
  hipError_t e = hipMalloc(reinterpret_cast<void**>(&ctx->ws.status), 256);
  if (e == hipSuccess) e = hipMemset(ctx->ws.status, 0, 256);
  for (int rf : {2, 4, 8, 16})
    for (FewKernel kernel : {few_kernel<false>(rf), few_kernel<true>(rf)})
      if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, FEW_LDS);
  constexpr size_t ONCE_BYTES = ONCE_STATE_BYTES + (NUM_XCD * ONCE_SLOTS + ONCE_COUNTS) * sizeof(uint32_t);
  if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void**>(&ctx->once), ONCE_BYTES);
  if (e == hipSuccess) e = hipMemset(ctx->once, 0, ONCE_BYTES);
  // this device's copy of the static scratch (the device is current here)
  if (e == hipSuccess) e = hipGetSymbolAddress(reinterpret_cast<void**>(&ctx->static_scratch), HIP_SYMBOL(scratch));
  for (int i = 0; i < 4 && e == hipSuccess; ++i) e = hipEventCreate(&ctx->ev[i]);
  if (e == hipSuccess) e = hipStreamCreateWithFlags(&ctx->copy_stream, hipStreamNonBlocking);
  for (int i = 0; i < EJOIN_MAX_BATCHES && e == hipSuccess; ++i) e = hipEventCreateWithFlags(&ctx->batch_ev[i], hipEventDisableTiming);
  if (e == hipSuccess) e = hipHostMalloc(reinterpret_cast<void**>(&ctx->batch_count), EJOIN_MAX_BATCHES * sizeof(unsigned long long), hipHostMallocDefault);
  for (void (*kernel)(JoinArgs) :
       {&k_join<false, false, false>, &k_join<false, false, true>, &k_join<true, false, false>, &k_join<true, false, true>, &k_join<true, true, false>,
        &k_join<true, true, true>})
    if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
  for (const void* kernel : {reinterpret_cast<const void*>(&k_dist2_tile<128, false>), reinterpret_cast<const void*>(&k_dist2_tile<128, true>)})
    if (e == hipSuccess) e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, dense_lds_bytes<128>());
  for (int nkb = 2; nkb <= EJ_STRIP_KB_MAX; ++nkb)
    for (JoinKernel kernel : {strip_kernel<false>(nkb), strip_kernel<true>(nkb)})
      if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, strip_lds(nkb));
  if (e != hipSuccess) {
    (void)hipGetLastError();
    ejoin_destroy(ctx);
    return EJOIN_EHIP;
  }
  ctx->last_status = ctx->ws.status;
  *out = ctx;
  return EJOIN_OK;
}

int ejoin_destroy(ejoin_ctx* ctx) {
  if (!ctx) return EJOIN_EINVAL;
  DeviceGuard guard(ctx->device);
  if (ctx->ws.status) (void)hipFree(ctx->ws.status);
  if (ctx->once) (void)hipFree(ctx->once);
  if (ctx->ws.s) (void)hipFree(ctx->ws.s);
  if (ctx->ws.Xp) (void)hipFree(ctx->ws.Xp);
  for (int i = 0; i < 4; ++i)
    if (ctx->ev[i]) (void)hipEventDestroy(ctx->ev[i]);
  for (int i = 0; i < EJOIN_MAX_BATCHES; ++i)
    if (ctx->batch_ev[i]) (void)hipEventDestroy(ctx->batch_ev[i]);
  if (ctx->copy_stream) (void)hipStreamDestroy(ctx->copy_stream);
  if (ctx->batch_count) (void)hipHostFree(ctx->batch_count);
  delete ctx;
  return EJOIN_OK;
}

int ejoin_reserve(ejoin_ctx* ctx, int64_t n, int32_t d) {
  if (!ctx || n < 1 || d < 1 || d > 65536) return EJOIN_EINVAL;
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return EJOIN_EHIP;
  return ensure_workspace(ctx, pad_rows(n) + TILE, pad_dims(d));  // + TILE: a total split over two sets pads each of them
}

const char* ejoin_strerror(int code) {
  switch (code) {
    case EJOIN_OK: return "ok";
    case EJOIN_EINVAL: return "invalid argument (null pointer, size out of range, ld not a multiple of 64 or < roundup(d,64), X not 128-byte aligned)";
    case EJOIN_EUNSUPPORTED: return "unsupported device (gfx950 required) or problem size";
    case EJOIN_EHIP: return "HIP runtime error (see ejoin_last_hip_error)";
    case EJOIN_ENOMEM: return "out of device memory for the workspace (20 bytes per point plus a packed copy of X)";
    case EJOIN_ESCRATCH: return "problem too large for the static scratch of the allocation-free entry point (EJOIN_STATIC_SCRATCH_BYTES)";
    default: return "unknown error code";
  }
}

const char* ejoin_last_hip_error(const ejoin_ctx* ctx) { return ctx ? ctx->hip_error : ""; }

int ejoin_norms(ejoin_ctx* ctx, const uint16_t* X, int64_t n, int32_t d, int64_t ld, float* s, void* stream) {
  EJ_RC(check_common(ctx, X, n, d, ld));
  if (!s) return EJOIN_EINVAL;
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return EJOIN_EHIP;
  return launch_norms(ctx, X, n, d, ld, s, nullptr, nullptr, static_cast<hipStream_t>(stream));
}

int ejoin_selfjoin_count(ejoin_ctx* ctx, const uint16_t* X, int64_t n, int32_t d, int64_t ld, float eps, uint32_t* counts,
                         uint64_t* total_pairs, void* stream) {
  EJ_RC(check_common(ctx, X, n, d, ld));
  EJ_RC(check_count_out(counts, total_pairs, eps));
  return join_on_ctx<true>(ctx, X, n, ld, nullptr, 0, 0, d, eps, count_results(counts, nullptr, total_pairs), stream);
}

int ejoin_selfjoin_pairs(ejoin_ctx* ctx, const uint16_t* X, int64_t n, int32_t d, int64_t ld, float eps, uint32_t* pairs,
                         float* dist2, uint64_t capacity, uint64_t* n_pairs, void* stream) {
  EJ_RC(check_common(ctx, X, n, d, ld));
  EJ_RC(check_pairs_out(pairs, capacity, n_pairs, eps));
  return join_on_ctx<false>(ctx, X, n, ld, nullptr, 0, 0, d, eps, pair_results(pairs, dist2, capacity, n_pairs), stream);
}

int ejoin_selfjoin_pairs_to_host(ejoin_ctx* ctx, const uint16_t* X, int64_t n, int32_t d, int64_t ld, float eps, uint32_t* pairs,
                                 float* dist2, uint64_t capacity, int32_t batches, uint32_t* host_pairs, float* host_dist2,
                                 uint64_t* host_n_pairs, void* stream) {
  EJ_RC(check_common(ctx, X, n, d, ld));
  if (!pairs || !host_pairs || !host_n_pairs || capacity == 0 || bad_eps(eps) || batches < 1 || (dist2 == nullptr) != (host_dist2 == nullptr))
    return EJOIN_EINVAL;
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return EJOIN_EHIP;
  hipStream_t st = static_cast<hipStream_t>(stream);
  // Ranges of super-block rows with about the same number of tiles each (row P of the triangle holds nsb - P super-blocks).
  const uint32_t nsb = (uint32_t)((pad_rows(n) / TILE + SB - 1) / SB);
  int nb = batches > EJOIN_MAX_BATCHES ? EJOIN_MAX_BATCHES : batches;
  if ((uint32_t)nb > nsb) nb = (int)nsb;
#ifdef EJOIN_ABL_ROWMAJOR_TILES
  nb = 1;  // (this ablation build deals the whole grid out in one launch)
#endif
  uint32_t bounds[EJOIN_MAX_BATCHES + 1];
  {
    const double total = 0.5 * nsb * (nsb + 1.0);
    double done = 0;
    uint32_t P = 0;
    bounds[0] = 0;
    for (int b = 1; b < nb; ++b) {
      while (P < nsb && done < total * b / nb) done += nsb - P++;
      if (P <= bounds[b - 1]) P = bounds[b - 1] + 1;  // every batch gets at least one row
      bounds[b] = P;
    }
    bounds[nb] = 0xFFFFFFFFu;
  }
  // the counter lives in the context's status block (the caller gets the final count in host memory)
  uint64_t* counter = reinterpret_cast<uint64_t*>(ctx->ws.status + 32);
  EJ_RC(ensure_workspace(ctx, pad_rows(n), pad_dims(d)));
  EJ_RC(run_join<false>(ctx, ctx->ws, true, X, n, ld, nullptr, 0, 0, d, eps, pair_results(pairs, dist2, capacity, counter), st, bounds, nb));
  // As each batch completes, its pairs go to the host on the copy stream while the next batch computes.
  unsigned long long lo = 0;
  for (int b = 0; b < nb; ++b) {
    EJ_TRY(hipEventSynchronize(ctx->batch_ev[b]));
    unsigned long long hi = ctx->batch_count[b];
    if (hi > capacity) hi = capacity;
    if (hi > lo) {
      EJ_TRY(hipMemcpyAsync(host_pairs + 2 * lo, pairs + 2 * lo, (hi - lo) * 2 * sizeof(uint32_t), hipMemcpyDeviceToHost, ctx->copy_stream));
      if (dist2) EJ_TRY(hipMemcpyAsync(host_dist2 + lo, dist2 + lo, (hi - lo) * sizeof(float), hipMemcpyDeviceToHost, ctx->copy_stream));
      lo = hi;
    }
  }
  EJ_TRY(hipStreamSynchronize(ctx->copy_stream));
  *host_n_pairs = ctx->batch_count[nb - 1];
  return EJOIN_OK;
}

int ejoin_selfjoin_pairs_noalloc(ejoin_ctx* ctx, const uint16_t* X, int64_t n, int32_t d, int64_t ld, float eps, uint32_t* pairs,
                                 float* dist2, uint64_t capacity, uint64_t* n_pairs, void* stream) {
  EJ_RC(check_common(ctx, X, n, d, ld));
  EJ_RC(check_pairs_out(pairs, capacity, n_pairs, eps));
  Workspace w;
  if (!carve_static(ctx->static_scratch, pad_rows(n), pad_dims(d), w)) return EJOIN_ESCRATCH;
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return EJOIN_EHIP;
  return run_join<false>(ctx, w, false, X, n, ld, nullptr, 0, 0, d, eps, pair_results(pairs, dist2, capacity, n_pairs),
                         static_cast<hipStream_t>(stream));
}

int ejoin_selfjoin_count_f32(ejoin_ctx* ctx, const float* X32, int64_t n, int32_t d, int64_t ld32, float eps, uint32_t* counts,
                             uint64_t* total_pairs, void* stream) {
  EJ_RC(check_f32(ctx, X32, n, d, ld32));
  EJ_RC(check_count_out(counts, total_pairs, eps));
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return EJOIN_EHIP;
  return run_join_split<true>(ctx, X32, n, d, ld32, eps, count_results(counts, nullptr, total_pairs), static_cast<hipStream_t>(stream));
}

int ejoin_selfjoin_pairs_f32(ejoin_ctx* ctx, const float* X32, int64_t n, int32_t d, int64_t ld32, float eps, uint32_t* pairs,
                             float* dist2, uint64_t capacity, uint64_t* n_pairs, void* stream) {
  EJ_RC(check_f32(ctx, X32, n, d, ld32));
  EJ_RC(check_pairs_out(pairs, capacity, n_pairs, eps));
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return EJOIN_EHIP;
  return run_join_split<false>(ctx, X32, n, d, ld32, eps, pair_results(pairs, dist2, capacity, n_pairs), static_cast<hipStream_t>(stream));
}

int ejoin_join_pairs(ejoin_ctx* ctx, const uint16_t* P, int64_t np, int64_t ldp, const uint16_t* Q, int64_t nq, int64_t ldq, int32_t d,
                     float eps, uint32_t* pairs, float* dist2, uint64_t capacity, uint64_t* n_pairs, void* stream) {
  EJ_RC(check_common(ctx, P, np, d, ldp));
  EJ_RC(check_common(ctx, Q, nq, d, ldq));
  EJ_RC(check_pairs_out(pairs, capacity, n_pairs, eps));
  return join_on_ctx<false>(ctx, P, np, ldp, Q, nq, ldq, d, eps, pair_results(pairs, dist2, capacity, n_pairs), stream);
}

int ejoin_join_count(ejoin_ctx* ctx, const uint16_t* P, int64_t np, int64_t ldp, const uint16_t* Q, int64_t nq, int64_t ldq, int32_t d,
                     float eps, uint32_t* counts_p, uint32_t* counts_q, uint64_t* total, void* stream) {
  EJ_RC(check_common(ctx, P, np, d, ldp));
  EJ_RC(check_common(ctx, Q, nq, d, ldq));
  EJ_RC(check_count_out(counts_p, total, eps));
  return join_on_ctx<true>(ctx, P, np, ldp, Q, nq, ldq, d, eps, count_results(counts_p, counts_q, total), stream);
}

int ejoin_set_create(ejoin_ctx* ctx, const uint16_t* X, int64_t n, int32_t d, int64_t ld, void* stream, ejoin_set** out) {
  if (!out) return EJOIN_EINVAL;
  *out = nullptr;
  EJ_RC(check_common(ctx, X, n, d, ld));
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return EJOIN_EHIP;
  hipStream_t st = static_cast<hipStream_t>(stream);
  ejoin_set* set = new (std::nothrow) ejoin_set();
  if (!set) return EJOIN_ENOMEM;
  set->ctx = ctx;
  set->n = n;
  set->pad = pad_rows(n);
  set->d = d;
  hipError_t e = hipMalloc(reinterpret_cast<void**>(&set->Xp), (size_t)packed_bytes(set->pad, pad_dims(d)));
  if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void**>(&set->s), (size_t)set->pad * sizeof(float));
  if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void**>(&set->max_bits), 256);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    (void)ejoin_set_destroy(set);
    return e == hipErrorOutOfMemory ? EJOIN_ENOMEM : fail_hip(ctx, e, "hipMalloc(prepared set)");
  }
  hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, st, set->max_bits, (int64_t)1, 0u);
  int rc = (hipGetLastError() == hipSuccess) ? EJOIN_OK : EJOIN_EHIP;
  if (rc == EJOIN_OK) rc = launch_norms(ctx, X, n, d, ld, set->s, set->max_bits, set->Xp, st);
  if (rc != EJOIN_OK) {
    (void)hipDeviceSynchronize();
    (void)ejoin_set_destroy(set);
    return rc;
  }
  *out = set;
  return EJOIN_OK;
}

int ejoin_set_destroy(ejoin_set* set) {
  if (!set) return EJOIN_EINVAL;
  DeviceGuard guard(set->ctx->device);
  if (set->Xp) (void)hipFree(set->Xp);
  if (set->s) (void)hipFree(set->s);
  if (set->max_bits) (void)hipFree(set->max_bits);
  delete set;
  return EJOIN_OK;
}

int ejoin_set_join_pairs(ejoin_ctx* ctx, ejoin_set* P, const uint16_t* Q, int64_t nq, int64_t ldq, float eps, uint32_t* pairs,
                         float* dist2, uint64_t capacity, uint64_t* n_pairs, void* stream) {
  if (!ctx || !P || P->ctx != ctx) return EJOIN_EINVAL;
  EJ_RC(check_common(ctx, Q, nq, P->d, ldq));
  EJ_RC(check_pairs_out(pairs, capacity, n_pairs, eps));
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return EJOIN_EHIP;
  return run_join_prepared<false>(ctx, P, Q, nq, ldq, eps, pair_results(pairs, dist2, capacity, n_pairs), static_cast<hipStream_t>(stream));
}

int ejoin_set_join_count(ejoin_ctx* ctx, ejoin_set* P, const uint16_t* Q, int64_t nq, int64_t ldq, float eps, uint32_t* counts_p,
                         uint32_t* counts_q, uint64_t* total, void* stream) {
  if (!ctx || !P || P->ctx != ctx) return EJOIN_EINVAL;
  EJ_RC(check_common(ctx, Q, nq, P->d, ldq));
  EJ_RC(check_count_out(counts_p, total, eps));
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return EJOIN_EHIP;
  return run_join_prepared<true>(ctx, P, Q, nq, ldq, eps, count_results(counts_p, counts_q, total), static_cast<hipStream_t>(stream));
}

int ejoin_convert_f32(ejoin_ctx* ctx, const float* X32, int64_t n, int32_t d, int64_t ld32, const float* center, float scale,
                      uint16_t* X16, int64_t ld16, void* stream) {
  if (!ctx || !X32 || !X16) return EJOIN_EINVAL;
  if (n < 1 || n >= (int64_t)0xFFFFFFFFll - TILE || d < 1 || d > 65536) return EJOIN_EINVAL;
  if (ld32 < d || ld16 < pad_dims(d) || (ld16 % KPAD) != 0 || !isfinite(scale)) return EJOIN_EINVAL;
  if ((reinterpret_cast<uintptr_t>(X16) & 127) != 0) return EJOIN_EINVAL;
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return EJOIN_EHIP;
  const int64_t per_row = ld16 / 8;
  if ((n * per_row + 255) / 256 > 0x7FFFFFFFll) return EJOIN_EUNSUPPORTED;
  const uintptr_t at = reinterpret_cast<uintptr_t>(X32);
  const bool past = ingest_past_the_caches(n, d, ld32, at, ld16);
  const bool four = past || (ingest_large(n, d, ld16) && (ld32 % 4 != 0 || at % 16 != 0));
  const int64_t chunks = four ? ld16 / 4 : per_row;  // of a row
  const uint32_t wide_log2 = (uint32_t)__builtin_ctz(ingest_wide(chunks));
  const int64_t rows = (256 >> wide_log2) * CONVERT_ROWS;
  hipLaunchKernelGGL((past ? k_convert_f32<4, true> : four ? k_convert_f32<4, false> : k_convert_f32<8, false>),
                     dim3((unsigned)((n + rows - 1) / rows * (chunks >> wide_log2))), dim3(256), 0, static_cast<hipStream_t>(stream), X32,
                     n, d, ld32, center, scale, X16, ld16, wide_log2, (uint32_t)(chunks >> wide_log2));
  EJ_TRY(hipGetLastError());
  return EJOIN_OK;
}

int ejoin_dist2_tile(ejoin_ctx* ctx, const uint16_t* X, int64_t n, int32_t d, int64_t ld, int64_t i0, int64_t j0, int32_t rows,
                     int32_t cols, float* out, void* stream) {
  EJ_RC(check_common(ctx, X, n, d, ld));
  if (!out || rows < 1 || cols < 1 || i0 < 0 || j0 < 0 || i0 + rows > n || j0 + cols > n) return EJOIN_EINVAL;
  if (rows > 32 * 65535 || cols > 32 * 65535) return EJOIN_EINVAL;
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return EJOIN_EHIP;
  EJ_RC(ensure_workspace(ctx, pad_rows(n), 0));
  const Workspace& w = ctx->ws;
  hipStream_t st = static_cast<hipStream_t>(stream);
  ctx->last_status = w.status;
  ctx->last_stream = st;
  // (no atomics on the status block: its state between calls is left as it is)
  uint32_t* maxima = w.maxima;
  DenseArgs a{X, w.s, maxima, 0, w.status, n, ld, (k_blocks(d) + 1) / 2 /* (rows are padded to a multiple of 64 coordinates) */, i0, j0, rows, cols, out};
  static_assert(dense_waves<128>() == 8 && dense_waves<64>() == 4, "as dense_norm_groups has them");
  const bool wide = dense_wide(ctx->num_cu, rows, cols);
  const int64_t groups = dense_groups(wide ? 128 : 64, rows, cols);
  if (const int64_t norm_groups = dense_norm_groups(ctx->num_cu, n, rows, cols)) {
    const DenseOneArgs one{w.s, (uint32_t)norm_groups, k_blocks(d), reinterpret_cast<unsigned long long*>(ctx->once), reinterpret_cast<uint32_t*>(ctx->once + ONCE_STATE_BYTES)};
    hipLaunchKernelGGL((wide ? k_dist2_tile<128, true> : k_dist2_tile<64, true>), dim3((unsigned)(groups + norm_groups)),
                       dim3(64 * (wide ? dense_waves<128>() : dense_waves<64>())), (wide ? dense_lds_bytes<128>() : dense_lds_bytes<64>()), st, a, one);
    EJ_TRY(hipGetLastError());
    return EJOIN_OK;
  }
  EJ_RC(launch_norms(ctx, X, n, d, ld, w.s, nullptr, nullptr, st, maxima, &a.nmaxima));
  // every workgroup of the dense kernel reads all maxima: from some 5 10^5 points on a launch that folds them first costs less
  // (d = 16, block of 100 x 100: 200,000 points 14.3 us without, 17.7 with; 500,000 17.9 and 18.6; 10^6 28.2 and 27.8; 5 10^6 145 and
  // 136; block of 4,000 x 4,000: 500,000 points 32.2 and 31.5; 10^6 44.7 and 41.4)
  constexpr uint32_t FOLD_MAXIMA = 2048;
  if (a.nmaxima > FOLD_MAXIMA) {
    hipLaunchKernelGGL(k_fold_max, dim3(1), dim3(512), 0, st, maxima, a.nmaxima);
    EJ_TRY(hipGetLastError());
    a.nmaxima = 1;
  }
  hipLaunchKernelGGL((wide ? k_dist2_tile<128, false> : k_dist2_tile<64, false>), dim3((unsigned)groups),
                     dim3(64 * (wide ? dense_waves<128>() : dense_waves<64>())), (wide ? dense_lds_bytes<128>() : dense_lds_bytes<64>()), st, a, NoArgs{});
  EJ_TRY(hipGetLastError());
  return EJOIN_OK;
}

int ejoin_status(ejoin_ctx* ctx, int* status) {
  if (!ctx || !status) return EJOIN_EINVAL;
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return EJOIN_EHIP;
  // the stream of the last call first: a blocking copy on the null stream does not order against non-blocking streams
  EJ_TRY(hipStreamSynchronize(ctx->last_stream));
  uint32_t st = 0;
  EJ_TRY(hipMemcpy(&st, ctx->last_status, sizeof(st), hipMemcpyDeviceToHost));
  *status = (int)st;
  return EJOIN_OK;
}

int ejoin_set_profiling(ejoin_ctx* ctx, int on) {
  if (!ctx) return EJOIN_EINVAL;
  ctx->profiling = on ? 1 : 0;
  ctx->ev_valid = 0;
  return EJOIN_OK;
}

int ejoin_last_kernel_ms(ejoin_ctx* ctx, float* prep_ms, float* join_ms) {
  if (!ctx || !ctx->ev_valid) return EJOIN_EINVAL;
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return EJOIN_EHIP;
  EJ_TRY(hipEventSynchronize(ctx->ev[3]));
  float a = 0.f, b = 0.f;
  EJ_TRY(hipEventElapsedTime(&a, ctx->ev[0], ctx->ev[1]));
  EJ_TRY(hipEventElapsedTime(&b, ctx->ev[2], ctx->ev[3]));
  if (prep_ms) *prep_ms = a;
  if (join_ms) *join_ms = b;
  return EJOIN_OK;
}

int ejoin_join_work(const ejoin_ctx* ctx, int64_t np, int64_t nq, int32_t d, int32_t split, int32_t* edge, int32_t* steps, int64_t* tiles) {
  if (!ctx || !edge || !steps || !tiles || np < 1 || nq < 0 || d < 1 || d > 65536 || (split && nq)) return EJOIN_EINVAL;
  *steps = split ? 3 * ((d + KSLICE - 1) / KSLICE) : k_blocks(d);
  const int once = split ? 0 : once_edge(ctx, np, nq ? nq : np, nq == 0, *steps, false);
  const int small = once ? once : small_tile(ctx, np, nq ? nq : np, nq == 0, *steps);
  *edge = small ? small : TILE;
  const int64_t a = (np + *edge - 1) / *edge, b = (nq + *edge - 1) / *edge;
  *tiles = nq ? a * b : a * (a + 1) / 2;
  return EJOIN_OK;
}

int ejoin_join_kernel(const ejoin_ctx* ctx, int64_t np, int64_t nq, int32_t d, int32_t split, int32_t count, int32_t* kernel) {
  if (!ctx || !kernel || np < 1 || nq < 0 || d < 1 || d > 65536 || (split == 2 ? nq == 0 : split && nq)) return EJOIN_EINVAL;
  const bool self = nq == 0, prepared = split == 2, fp32 = split && !prepared;
  const int nkb = fp32 ? 3 * ((d + KSLICE - 1) / KSLICE) : k_blocks(d);
  const int64_t nB = self ? np : nq;
  if (!split && once_edge(ctx, np, nB, self, nkb, count != 0)) *kernel = EJOIN_KERNEL_ONCE;
  else if (prepared && few_groups(np, nq, nkb, count != 0)) *kernel = EJOIN_KERNEL_FEW;
  else if (small_tile(ctx, np, nB, self, nkb)) *kernel = EJOIN_KERNEL_SMALL;
  else *kernel = !fp32 && plan_strip(ctx, np, nB, self, nkb, count != 0).use ? EJOIN_KERNEL_STRIP : EJOIN_KERNEL_TILES;
  return EJOIN_OK;
}

int64_t ejoin_tiles_evaluated(int64_t n) {
  if (n < 1) return 0;
  const int64_t t = (n + TILE - 1) / TILE;
  return t * (t + 1) / 2;
}

int64_t ejoin_tiles_evaluated2(int64_t np, int64_t nq) {
  if (np < 1 || nq < 1) return 0;
  return ((np + TILE - 1) / TILE) * ((nq + TILE - 1) / TILE);
}

}  // extern "C"
