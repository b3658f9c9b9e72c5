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

// Right-hand sides per workgroup (1 to 4) of the ordered squared apply, 0 where the
// general kernel, which has the same bits and reads the matrix once per 16, is the
// faster one.  A workgroup per site and group; as many groups as fit into the rounds of
// 256 workgroups that groups of four take anyway, of two and more right-hand sides
// where a site's groups land on different XCDs (Vc no multiple of 8) and each reads the
// matrix for itself.  Rounds cost 14 to 25 us at 48 dof (one to four right-hand sides),
// passes of the general kernel 45 to 75, and beyond 160 sites the matrix (0.1 GB) comes
// from HBM once per group: 512 sites, 12 right-hand sides 144 us in the general kernel,
// 180 in groups of four, 234 of eight; 128 sites, 12: 37 us in groups of three, 61 in
// the general kernel.  16 dof on 1024 sites and more keep the groups (12: 78 against 95),
// 64 dof there do not (one right-hand side: 194 against 184).
inline int sq_ordered_group(long long Vc, int n2, int nrhs) {
  const long long fewest = (nrhs + 3) / 4, rounds = (Vc * fewest + 255) / 256;
  if (nrhs > 4 && !(n2 == 16 && Vc >= 1024) && (Vc > (Vc % 8 != 0 ? 128 : 160) || rounds >= 3 * ((nrhs + 15) / 16))) return 0;
  if (nrhs == 1 && n2 == 64 && Vc >= 1024) return 0;
  const long long groups = std::max(fewest, 256 * rounds / Vc), least = Vc > 32 && Vc % 8 != 0 ? 2 : 1;
  return (int)std::min<long long>(nrhs, std::max(least, (nrhs + groups - 1) / groups));
}

}  // namespace mgdwf
