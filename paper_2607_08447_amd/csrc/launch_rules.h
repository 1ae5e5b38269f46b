// Index and launch arithmetic that kernels and their launchers share.  Plain
// constexpr functions (usable on the host and in kernels), without HIP types, so that
// they can be checked on the host over the whole range of sizes: 6 N <= 2^31, which
// allows a column of up to 3.5e8 planes.
#pragma once

#include <cstddef>

namespace hkp {

// complex entries per plane of the folded link-phase table
constexpr int kFoldRow = 12;
// first real of plane z in that table (beyond 32 bits from 9e7 planes)
constexpr std::size_t fold_offset(int z) { return (std::size_t)z * (2 * kFoldRow); }

// first of nz planes in range zc of zs: floor(zc nz / zs), without the product (zc nz
// exceeds 32 bits for long columns; a 64-bit division costs far more than these)
constexpr int range_begin(int zc, int nz, int zs) {
  const int q = nz / zs, r = nz - q * zs;
  return zc * q + zc * r / zs;
}

}  // namespace hkp
