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
  const bool many = Vc > (Vc % 8 != 0 ? 128 : 160) || rounds >= 3 * ((nrhs + 15) / 16);
  if (nrhs > 4 && many && !(n2 == 16 && Vc >= 1024)) return 0;
  if (nrhs == 1 && n2 == 64 && Vc >= 1024) return 0;
  const long long groups = std::max(fewest, 256 * rounds / Vc), least = Vc > 32 && Vc % 8 != 0 ? 2 : 1;
  return (int)std::min<long long>(nrhs, std::max(least, (nrhs + groups - 1) / groups));
}

// Whether the squared MFMA kernels give the 16-row tiles of a site to different
// workgroups (16 rows each) or all to one; sites: coarse sites times groups of eight
// right-hand sides.  The split form's rounds of 256 workgroups are shorter but more:
// it takes one round of them, and two where a round of whole sites costs more than
// two of its own (64 dof except in an FP32 CG step, 48 dof in the FP32 product); beyond,
// a nearly empty last round decides.  us, split / whole sites, FP64 and FP32, one
// right-hand side: 48 dof, 80 sites 18.5 / 26.6 and 11.4 / 19.9, 128 sites 30.0 / 28.3
// and 18.1 / 20.7, 192 sites 45.1 / 36.2 and 25.8 / 23.5; 64 dof, 128 sites 47.1 / 50.2
// and 25.2 / 33.0, 162 sites 73.4 / 60.7 and 33.2 / 34.1; 32 dof, 128 sites 14.0 / 16.7 and
// 7.8 / 10.9, 144 sites 21.0 / 17.7 and 12.7 / 11.2; 12 right-hand sides, 48 dof on 120
// sites 50.4 / 29.3 and 29.1 / 21.8.
inline bool sq_split_rows(long long sites, int row_tiles, bool f64, bool cg_step) {
  const bool two = row_tiles >= 4 ? f64 || !cg_step : row_tiles == 3 && !f64 && !cg_step;
  return sites * row_tiles <= (two ? 512 : 256);
}

// Columns of a coarse build restricted together: the restriction reads the basis once
// per 32 right-hand sides, and three columns' nine pieces fill 27 (8^3x16x16, 24 columns:
// 8.8 ms against 17.7).  One at a time, as many fields as the build's steps need at
// least, where the 27 FP64 fields would pass 16 GB or take more than half of the
// memory that is free.
inline int coarse_build_columns(double field_bytes, double free_bytes) {
  return 27 * field_bytes <= std::min(16e9, 0.5 * free_bytes) ? 3 : 1;
}

}  // namespace mgdwf
