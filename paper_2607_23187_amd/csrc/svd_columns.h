// The columns that the workgroups of the one-sided SVD exchange: where a column's copies lie and
// which of them is current.
//
// In one rotation every workgroup loads the old columns p and q while their owners store the new
// ones, and the only wait of a rotation, the exchange of candidates, comes before both.  So old
// and new never share an address: two copies of every column are kept, a rotation loads the
// current copies of p and q, stores the other ones, and makes those current.  Every workgroup
// performs every rotation, so each keeps its own version bits and none are exchanged.
//   Loads of a new copy: its stores were acknowledged before the owner arrived at the next
//   exchange, which every later load follows.
//   Stores over an old copy: it was loaded last in the rotation that replaced it.  The rotation
//   that stores it again lies behind a further exchange, at which every workgroup arrives only
//   after those loads have returned.
#pragma once

#include <cstddef>

namespace je {

// Column k's version is bit k / 64 of lane k mod 64's word.
constexpr int kSvdVersionCols = 64 * 32;
constexpr int svd_version_lane(int k) { return k & 63; }
constexpr unsigned svd_version_bit(int k) { return 1u << (k >> 6); }

// Copy `version` (0: as loaded) of column k: n columns of stride ldc, then their other copies.
constexpr size_t svd_column_at(unsigned version, int k, int n, int ldc) {
  return ((size_t)(version ? n : 0) + (size_t)k) * (size_t)ldc;
}
constexpr size_t svd_column_doubles(int n, int ldc) { return 2 * (size_t)n * (size_t)ldc; }

}  // namespace je
