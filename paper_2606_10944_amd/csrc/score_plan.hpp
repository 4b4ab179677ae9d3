// Launch rules of the Halve rounds: host arithmetic without HIP.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace thin {

// Float score launches of at most this many units of 32 x 32 take a wave per
// unit (score_units_kernel); beyond, the workgroups of pair_scores_kernel, which
// read each row once for 128 or 256 others.  (bf16 rows stay with those at every
// size: the matrix cores take their products sixteen times as fast and the launch
// is all latency; 32 buckets of 512 rows: 15 us against 19.)  The line was fitted
// to 1788 rounds measured in both forms (160 to 4096 rows in 1 to 160 buckets;
// whole calls of one or two rounds, us, units | workgroups):
// - the device holds so many units' waves (d = 32, 64: 3 and 2 per SIMD; d = 128:
//   eight fragments of three or four operands are 436 registers, one per SIMD), and
//   a first round's other form is two launches: first rounds, d = 64, 24 buckets of
//   1024 rows 112 | 134, 64 of 640 108 | 96; d = 128, 8 of 1024 103 | 126, 12 of
//   1024 133 | 127;
// - a smaller bucket's workgroups have less to do before they are done: d = 128, 40
//   of 400 rows 80 | 87, 56 of 320 77 | 72, 72 of 200 63 | 58;
// - the other form deals buckets to the eight XCDs, whole ones: fewer than eight
//   buckets leave XCDs idle (d = 128, 2 of 4096 rows 417 | 478, 3 of 2048 158 |
//   200), and more that eight does not divide some of them (later rounds, d = 128,
//   17 of 800 rows 340 | 355, 16 of 800 293 | 276).
// Over all those rounds the line costs 0.2 % against the faster form of each.
inline int64_t unit_launch_max(int64_t d, int64_t N, int64_t nbk, bool first_round) {
  int64_t most, per_row;
  if (d > 64) {
    most = first_round ? 4750 : 5250;
    per_row = first_round ? 11 : 7;
  } else {
    most = !first_round ? 16250 : d > 32 ? 13500 : 15500;
    per_row = first_round ? 30 : 12;
  }
  const int64_t units = std::min(most, per_row * N), dealt = (nbk + 7) / 8 * 8;
  return nbk < 8 ? units * dealt / nbk : units * (dealt + nbk) / (2 * nbk);
}

// A local launch of nbk buckets stages every row tile of a bucket at once, where
// that takes `lds` bytes per workgroup and the registers let by_registers
// workgroups share a CU, if that costs no resident workgroup: the launch fits the
// device all the same, or LDS holds as many as the registers.  1 to 32 buckets of
// 128 rows (float, d = 64) 20.3 us in a ring, 18.1 staged; of 256 rows (bf16, d =
// 64) 19.1, 17.5; 600 buckets of 160 rows (bf16, d = 64), two staged workgroups
// per CU against three, 23.5, 27.6.
inline bool local_staged(int64_t nbk, int64_t lds, int64_t by_registers) {
  const int64_t fit = ((int64_t)160 << 10) / lds;
  return fit >= 1 && (nbk <= 256 * fit || fit >= by_registers);
}

}  // namespace thin
