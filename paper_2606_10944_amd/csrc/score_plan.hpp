// Launch rules of the Halve rounds: host arithmetic without HIP.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace thin {

// Float score launches of at most this many units of 32 x 32 take a wave per
// unit (score_units_kernel); beyond, the workgroups of pair_scores_kernel, which
// read each row once for 128 or 256 others.  (bf16 rows stay with those at every
// size: the matrix cores take their products sixteen times as fast and the launch
// is all latency; 32 buckets of 512 rows: 15 us against 19.)  What sets the line
// is how many waves the device holds:
// - d = 32, 64 (3 and 2 waves per SIMD): a first round, whose other form is two
//   launches, is faster as units up to about 13000 of them (d = 64, whole call,
//   units against workgroups: 24 buckets of 1024 rows 0.84, 64 of 512 0.88, 100
//   of 512 1.13, 48 of 800 1.17), a later one up to about 6000 (64 of 320 1.01,
//   64 of 512 1.07, 32 of 800 1.06).
// - d = 128: eight fragments of three or four operands are 436 registers, one
//   wave per SIMD (first rounds: 64 buckets of 256 rows 1.00, 100 of 256 1.22, 32
//   of 512 0.98, 64 of 512 1.50; later ones: 32 of 512 1.04).
// - The workgroups of fewer than eight buckets run on as many XCDs (d = 128: 8
//   buckets of 1024 rows 0.84, 2 of 2048 0.84, 6 of 2048 1.24, one of 4096 0.63;
//   d = 64: 6 of 2048 0.84, one of 5600 0.64).
inline int64_t unit_launch_max(int64_t d, int64_t N, int64_t nbk, bool first_round) {
  constexpr int64_t kMost = 16384;
  if (d <= 64) return nbk < 8 ? kMost : first_round ? 13312 : 6144;
  const int64_t wide = !first_round ? 2048 : N < 512 ? 2560 : 4800;
  return std::min(kMost, std::max(wide, 36864 / nbk));
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
