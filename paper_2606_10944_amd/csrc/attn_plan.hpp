// Launch shapes of the attention kernels: host arithmetic without HIP.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace thin {

// A launch's threads per grid dimension are counted in 32 bits (2^24 workgroups
// of 256 are refused), so a longer row of workgroups takes several rows of a
// further dimension: x * rows >= blocks, x a multiple of `multiple`.
struct GridRows {
  int64_t x, rows;
};
inline GridRows grid_rows(int64_t blocks, int64_t threads, int64_t multiple = 1) {
  const int64_t most = (((int64_t)1 << 32) - 1) / threads / multiple * multiple;
  const int64_t rows = (blocks + most - 1) / most;
  const int64_t x = (blocks + rows - 1) / rows;
  return {(x + multiple - 1) / multiple * multiple, rows};
}

// S slices of `steps` equal steps of queries each: `parts` workgroups per slice
// take equal runs of whole steps, each workgroup after staging its slice's
// coreset (worth `stage`), `slots` workgroups on the device at once.  The split
// whose rounds of workgroups end first, among those that fill 1 to 8 rounds more
// or less; of equal ones the fewest workgroups.
struct StepSplit {
  int64_t parts;  // workgroups per slice
  int64_t run;    // steps of each
  double cost;
};
inline StepSplit split_steps(int64_t S, int64_t steps, int64_t slots, double stage, double step) {
  StepSplit best{0, 0, 0.0};
  const int64_t least = (S + slots - 1) / slots;  // rounds with one workgroup per slice
  for (int64_t r = least; r < least + 8; ++r) {
    const int64_t run = (steps + slots * r / S - 1) / (slots * r / S);
    const int64_t parts = (steps + run - 1) / run;
    const double cost = (double)((S * parts + slots - 1) / slots) * (stage + (double)run * step);
    if (best.parts == 0 || cost < best.cost * (1.0 - 1e-9)) best = {parts, run, cost};
    if (run == 1) break;
  }
  return best;
}

// Workgroups per slice of float attention over one chunk of at most 64 keys,
// which a workgroup stages once (worth about half a block) and keeps for its
// share of the slice's `blocks` blocks of 64 queries, dealt out in turn; several
// workgroups share a CU, `slots` fit the device.  A share of less than two
// blocks counts as whole blocks (one of the workgroups has two).  d = 64, 1024
// slots, us: one workgroup per block | 1024 / S of them | this: 64 x 4097 queries
// over 16 keys 50 | 48 | 48, 520 x 1000 94 | 124 | 95, 1000 x 256 51 | 46 | 46;
// over 64 keys 59 | 50 | 50, 123 | 128 | 103, 67 | 49 | 49.
inline int64_t split_blocks(int64_t S, int64_t blocks, int64_t slots) {
  int64_t best = 0;
  double least = 0.0;
  const int64_t r0 = (S + slots - 1) / slots;
  for (int64_t r = r0; r < r0 + 8; ++r) {
    const int64_t parts = std::min(blocks, slots * r / S);
    const double share = 2 * parts <= blocks ? (double)blocks / (double)parts
                                             : (double)((blocks + parts - 1) / parts);
    const double cost = (double)((S * parts + slots - 1) / slots) * (0.55 + share);
    if (best == 0 || cost < least * (1.0 - 1e-9)) best = parts, least = cost;
    if (parts == blocks) break;
  }
  return best;
}

// Workgroup `id` of S * parts, where `extra` of a slice's parts have a block more
// than the others: those come first.  Workgroups go to the CUs in turn, so every
// CU gets as many of them (slice after slice, part after part, they all fell on
// the same CUs where 256 is about a multiple of the parts; float rows, 16 keys: 20
// x 4097 queries, d = 64, 24.8 -> 19.7 us, d = 32 13.5 -> 11.9), and the longest
// start first.
struct Share {
  uint32_t slice, part;
};
constexpr Share share_of(uint32_t id, uint32_t S, uint32_t parts, uint32_t extra) {
  const uint32_t longer = S * extra;
  if (id < longer) return {id / extra, id % extra};
  return {(id - longer) / (parts - extra), extra + (id - longer) % (parts - extra)};
}

// Attention over 129 to 256 keys of d = 128 (one workgroup per CU): a step is
// 128 queries with one query tile per wave, or 256 with two, which read each
// fragment of the coreset once for both and so take 1.75 times as long as one
// (fitted over 1 to 513 slices of 33 to 65536 queries: 7.0 us and 11.4 with 256
// keys, 5.1 and 9.4 with 192; a further workgroup on a CU 11 to 14 us).  256
// keys, bf16 out, 512 workgroups of one tile | 256 of two, each rounded up per
// slice | this plan, us: 8 x 4096 queries 18.8 | 23.7 | 18.0, 64 x 1024 41.0 |
// 26.5 | 26.8, 24 x 16384 161 | 138 | 95, 12 x 65536 289 | 297 | 185, 96 x 16384
// 547 | 519 | 365, 32 x 65536 564 | 463 | 455.
struct TilePlan {
  int tiles;
  StepSplit split;
};
inline TilePlan attn_tile_plan(int64_t S, int64_t n_q, int64_t slots) {
  constexpr double kStage = 2.0;  // a further workgroup on a CU: its staging, in steps of one tile
  const TilePlan one{1, split_steps(S, (n_q + 127) / 128, slots, kStage, 1.0)};
  const TilePlan two{2, split_steps(S, (n_q + 255) / 256, slots, kStage, 1.75)};
  return two.split.cost < one.split.cost ? two : one;
}

}  // namespace thin
