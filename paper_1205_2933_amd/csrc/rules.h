// Launch rules that follow from sizes alone.  Plain C++, so that a host program can
// look at them over whole ranges.
#pragma once
#include <algorithm>

namespace mgdwf {

// Workgroups per coarse site of the MFMA restriction: at most 16, as many as make
// 2048 in all (eight per CU; reached from 128 to 512 sites), at least four.
inline int restrict_splits(int Vc) { return std::max(4, std::min(16, 2048 / std::max(1, Vc))); }

// The same of the one-field restriction (one right-hand side, or FP32 with an odd fifth
// dimension), whose workgroups take 256 rows at a time and reduce every column
// across their threads: a split without rows of its own only adds reductions, and so
// does one more than about two workgroups per CU (eight in FP64).  us, four splits /
// the count above / this rule: 256 sites of 256 rows, 24 columns, FP64 158 / 307 /
// 158; 16 sites of 80 rows, 12 columns, 12 FP32 fields 74 / 265 / 74; 32 sites of 4096
// rows, 24 columns, FP32 107 / 79 / 79.
inline int restrict_splits_general(int Vc, int rows, int nrhs, bool f64) {
  const long long wgs = (long long)std::max(1, Vc) * std::max(1, nrhs);
  const int want = (int)((f64 ? 2048 : 512) / wgs);
  return std::max(4, std::min(want, std::min(16, rows / 256)));
}

}  // namespace mgdwf
