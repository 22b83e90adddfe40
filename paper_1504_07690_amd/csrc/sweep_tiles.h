// How the FP32 and FP64 sweeps deal their points to tiles (host and device; no HIP in here).
#pragma once
#include <cstdint>

namespace ssm {

// nb blocks of points in mt tiles, each of mb or mb - 1 consecutive blocks, mb = ceil(nb / mt): the
// kernel of mb blocks has a strip for either count and for no other.  Every block has exactly one
// tile, so that no two workgroups add into one row of Z.
struct SweepTiling {
  int nb, mt;
  constexpr int mb() const { return (nb + mt - 1) / mt; }
  constexpr int first(int tile) const { return (int)((int64_t)tile * nb / mt); }
  constexpr int count(int tile) const { return first(tile + 1) - first(tile); }
};

// The count mt (mb at most max_mb) that makes the busiest SIMD's share smallest.  A launch has strips
// x mt waves of ceil(nb / mt) blocks' matrix work on 1024 SIMDs.  While a SIMD gets only a few
// waves, whole waves count; with many, the mean does.  + 0.5 stands for the loads of a wave that
// do not grow with its blocks.  Long rows (64-bit addresses) make strips enough: the widest tiles.
constexpr SweepTiling sweep_tiling(int64_t strips, int nb, int max_mb, bool long_rows) {
  const int least = (nb + max_mb - 1) / max_mb;
  if (long_rows) return SweepTiling{nb, least};
  int best = nb;
  double cost = 0.0;
  for (int mt = least; mt <= nb; ++mt) {
    const int mb = (nb + mt - 1) / mt;
    const int64_t per_simd = (strips * mt + 1023) / 1024;
    const double c = per_simd <= 6 ? (double)per_simd * (mb + 0.5) : (double)strips * (nb + 0.5 * mt) / 1024.0;
    if (cost == 0.0 || c < cost) {
      cost = c;
      best = mt;
    }
  }
  return SweepTiling{nb, best};
}

}  // namespace ssm
