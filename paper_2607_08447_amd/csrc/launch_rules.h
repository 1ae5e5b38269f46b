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
constexpr std::size_t fold_offset(int z) {
  return (std::size_t)((unsigned long long)(unsigned)z * (unsigned)(2 * kFoldRow));
}

// nz planes in zs <= kMaxSplit ranges, range zc from floor(zc nz / zs): without the product
// zc nz, which exceeds 32 bits for long columns, and without a division once nz is cut
// (the host does it for the launches that it splits)
constexpr int kMaxSplit = 12;
struct ZRanges {
  int zs;
  float inv;     // 1 / zs
};
struct ZCut {
  int q, r;      // nz = q zs + r
  unsigned m;    // floor(65536 / zs) + 1: (n m) >> 16 = floor(n / zs) for n < zs kMaxSplit
};
constexpr ZCut z_cut(int nz, const ZRanges& z) {
  const int q = nz / z.zs;
  return ZCut{q, nz - q * z.zs, (unsigned)(65536.0f * z.inv) + 1u};
}
constexpr int range_begin(int zc, const ZCut& c) {
  return zc * c.q + (int)(((unsigned)(zc * c.r) * c.m) >> 16);
}

constexpr int kCUs = 256;   // compute units of the whole GPU (a partition of it has fewer)

// z-ranges for nlw workgroups of nz planes, at most zmax: the fewest planes marched on
// the CU that gets the most workgroups.  A workgroup marches nz / zs + 2 planes, a CU
// gets ceil(nlw zs / cus) of them, and c0 workgroups together take no longer per
// plane than one alone (a plane's latency against its share of the CU).  Measured for
// 480 FP32 recurrence workgroups (12 vectors of 128 x 40 x 40): 63 us in one range, 68
// in two; 384 (4 vectors of 256 x 48 x 48): 81 in one, 64 in four; 144 FP64 product
// ones (6 vectors of 96 x 32 x 32): 53 in one, 35 in two, 28 in three, 30 in four.
// (icus: 1 / cus.  No division: a launch whose live count is only known on the device
// evaluates this in every workgroup, before its first plane)
constexpr ZRanges z_ranges(int nlw, int nz, int zmax, float c0, float cus, float icus) {
  constexpr float inv[kMaxSplit] = {1.0f,     1.0f / 2, 1.0f / 3, 1.0f / 4,  1.0f / 5,  1.0f / 6,
                                    1.0f / 7, 1.0f / 8, 1.0f / 9, 1.0f / 10, 1.0f / 11, 1.0f / 12};
  ZRanges best{1, 1.0f};
  float cost = 1e30f;
#pragma unroll
  for (int zs = 1; zs <= kMaxSplit; ++zs) {
    // the ceiling, by the reciprocal (half a workgroup's margin against its rounding)
    const float per_cu = (float)(int)(((float)nlw * (float)zs + cus - 0.5f) * icus);
    const float c = (per_cu > c0 ? per_cu : c0) * ((float)nz * inv[zs - 1] + 2.0f);
    if (c < cost && zs <= zmax && zs <= nz) {
      best = ZRanges{zs, inv[zs - 1]};
      cost = c;
    }
  }
  return best;
}

// Vectors that a launch with a work table is made for, of all members' `all`: the live
// ones where the host knows them (live >= 0; it reads the flags after every iteration), in
// a recorded launch at most those of the members still active when it was recorded
// (most; 0: all).
constexpr long long table_vectors(long long all, long long live, long long most) {
  return live >= 0 ? live : (most > 0 && most < all ? most : all);
}

// Split of a launch of nwg workgroups: the ranges that its grid leaves room for, and the
// ranges of every vector where the host decides them (0: the device does, from its live
// vectors; then with room for twice the split that suits all).  16 workgroups per CU need
// none; room for it in every launch would double the grid of large ones, half of it empty.
// The end of a large batch is split because its launches are made for what is left: 64
// members of 192 x 40 x 40 of which four are slow, mixed 0.690 -> 0.665 s launch by
// launch and 0.676 -> 0.664 s recorded.
struct ZSplit {
  int room;
  ZRanges fixed;
};
constexpr ZSplit z_split(long long nwg, int nz, bool on_device, float c0, int cus) {
  const ZRanges z = nwg < 16 * cus
                        ? z_ranges((int)nwg, nz, 8, c0, (float)cus, 1.0f / (float)cus)
                        : ZRanges{1, 1.0f};
  if (!on_device || nwg >= 16 * cus) return ZSplit{z.zs, z};
  return ZSplit{2 * z.zs < kMaxSplit ? 2 * z.zs : kMaxSplit, ZRanges{0, 0.0f}};
}

// Whether an iteration recorded for `recorded` active members is recorded anew for the
// `active` that are left: its launches were too large to be split (member_wgs: workgroups
// of one member's vectors), and a quarter of them would fill the chip less well.  (A
// recording takes a millisecond or two, such an iteration a hundred.)
constexpr bool record_anew(int recorded, int active, long long member_wgs, int cus) {
  return active > 0 && 4LL * active <= recorded && recorded * member_wgs >= 16 * cus;
}

// Launch shapes that the tuner times for a filter step: waves per spin, vectors side by
// side, whether rows may be copied, and the z split that the solver's launches use.  Row
// copies are timed where they exist, in FP64 on whole 64-wide tiles; in FP32 there is
// nothing to time, and the FP64 launches of a mixed solve take them wherever they can (58
// us a step against 61 staged, 2 vectors of 256 x 48 x 48).
struct TuneShape {
  int tile_y, vgroup, dma, zsplit;
};
constexpr int kMaxTuneShapes = 24;
constexpr int tune_shapes(int nx, int ny, int nb, bool fp64, TuneShape (&out)[kMaxTuneShapes]) {
  const int whole = nx % 64 == 0 ? 1 : 0;
  int n = 0;
  for (int dma = fp64 ? 0 : whole; dma <= whole; ++dma)
    for (int g = 0; g < 4; ++g) {
      const int vg = g == 3 ? nb : 1 << g;   // 1 (vector-major), 2, 4, nb (tile-major)
      if (vg > nb || (g == 3 && nb <= 4 && nb != 3)) continue;   // (once each)
      for (int ty = 1; ty <= 4; ty *= 2)
        if (ty <= 2 || ty <= 2 * ny) out[n++] = TuneShape{ty, vg, dma, 1};
    }
  return n;
}

}  // namespace hkp
