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

constexpr int kCUs = 256;   // compute units of the GPU

// z-ranges for nlw workgroups of nz planes, at most zmax: the fewest planes marched on
// the CU that gets the most workgroups.  A workgroup marches nz / zs + 2 planes, a CU
// gets ceil(nlw zs / 256) of them, and c0 workgroups together take no longer per
// plane than one alone (a plane's latency against its share of the CU).  Measured for
// 480 FP32 recurrence workgroups (12 vectors of 128 x 40 x 40): 63 us in one range, 68
// in two; 384 (4 vectors of 256 x 48 x 48): 81 in one, 64 in four; 144 FP64 product
// ones (6 vectors of 96 x 32 x 32): 53 in one, 35 in two, 28 in three, 30 in four.
constexpr int kMaxSplit = 12;
constexpr int z_ranges(int nlw, int nz, int zmax, float c0) {
  constexpr float inv[kMaxSplit] = {1.0f,     1.0f / 2, 1.0f / 3, 1.0f / 4,  1.0f / 5,  1.0f / 6,
                                    1.0f / 7, 1.0f / 8, 1.0f / 9, 1.0f / 10, 1.0f / 11, 1.0f / 12};
  int best = 1;
  float cost = 1e30f;
#pragma unroll
  for (int zs = 1; zs <= kMaxSplit; ++zs) {
    const float per_cu = (float)(((unsigned)nlw * zs + kCUs - 1) / kCUs);
    const float c = (per_cu > c0 ? per_cu : c0) * ((float)nz * inv[zs - 1] + 2.0f);
    if (c < cost && zs <= zmax && zs <= nz) {
      best = zs;
      cost = c;
    }
  }
  return best;
}

// Split of a launch of nwg workgroups over all of its vectors: the ranges that its grid
// leaves room for, and the ranges of every vector where the host decides them (0: the
// device does, from its live vectors).  16 workgroups per CU need no split.  Where the
// live count is only known on the device there is room for twice the split that suits
// all vectors, and for two ranges at least: the few members of a large batch that are
// left at its end would fill a fraction of the CUs.
struct ZSplit {
  int room, fixed;
};
constexpr ZSplit z_split(long long nwg, int nz, bool on_device, float c0) {
  const int zs = nwg < 16 * kCUs ? z_ranges((int)nwg, nz, 8, c0) : 1;
  if (!on_device) return ZSplit{zs, zs};
  const int room = 2 * zs < kMaxSplit ? 2 * zs : kMaxSplit;
  return nwg * room > 0x7fffffffLL ? ZSplit{1, 1} : ZSplit{room, 0};
}

}  // namespace hkp
