// Tiles of the fused iteration kernel: variants, their workgroups, and the choice of variant and
// height by the estimated time of a launch (host code without HIP).
#pragma once

namespace ofmi {

// Tile variants of the iteration kernel:
//   wide       64-column strips, about 12 threads per output column;
//   wide 32 /  the wide variant on strips of 32 or 16 output columns (plain launches of the
//   wide 16    box window): small levels spread over more CUs, hence a shorter path per band
//              where a level has fewer tiles than CUs.
//   wide 32x2 / the same strips with two bands per pass (plain launches, r <= kMaxPairRadius;
//   wide 16x2   with the Gaussian window tiles of one output band only, chosen by the host): a
//              tile of one output band runs its priming band and its output band together, one
//              dependent path.
//   narrow, wide lean, lean 32x2: the kernels of wide, wide and wide 32x2 (kept as configuration values;
//              at 5 threads per column, as narrow once stood for, 8 pairs of 640 x 480, r = 8, one band:
//              256.8 us, 146.3 us as wide).
enum TileVariant : int { kTileNarrow = 0, kTileWide = 1, kTileWideLean = 2, kTileWide32 = 3,
                         kTileWide16 = 4, kTileWide32x2 = 5, kTileWide16x2 = 6, kTileLean32x2 = 7 };
constexpr int kTileVariants = 8;
// Largest window radius of the two-bands-per-pass variants (two workgroups share a CU's
// LDS).
constexpr int kMaxPairRadius = 8;
// Added to a plain launch's variant: Gaussian-weighted window sums (taps in IterArgs::taps).
constexpr int kTileGauss = 16;

// Workgroup of a tile variant at radius R: output columns, bands per pass, threads, workgroups
// that share a CU.
struct TileShape {
  int tw, bb, threads, per_cu;
};
TileShape tile_shape(int variant, int R);
// Strip width (output columns per tile) of the iteration kernel for radius R (variants 0-2).
int strip_width_for(int R);
// Strip width of a plain launch's tile variant.
inline int tile_width(int variant, int R) {
  if (variant == kTileWide32 || variant == kTileWide32x2 || variant == kTileLean32x2) return 32;
  if (variant == kTileWide16 || variant == kTileWide16x2) return 16;
  return strip_width_for(R);
}
// Whether a plain launch of radius R (Gaussian-weighted window or not) has tile variant
// `variant`: narrow strips only with the box window, two bands per pass only up to
// kMaxPairRadius.
inline bool tile_variant_valid(int variant, int R, bool gaussian) {
  if (variant < kTileNarrow || variant >= kTileVariants) return false;
  if (gaussian && variant > kTileWideLean) return false;
  if ((variant == kTileWide32x2 || variant == kTileWide16x2 || variant == kTileLean32x2) &&
      R > kMaxPairRadius)
    return false;
  return true;
}

// `count` planes of one size at a level.
struct PlaneSize {
  int H, W, count;
};
// Estimated time of an iteration launch with one tile variant, by tile height (see the definition).
class LaunchCost {
 public:
  LaunchCost(int R, int variant, bool gauss);
  double at(const PlaneSize* s, int n, int nb) const;
  // Lowers `cost` to the least cost of tiles of 1, 1 + step, .. kMostBands bands of an H x W plane
  // where that is less, and then returns the lowest such height, else 0.
  int least(int H, int W, int step, double& cost) const;
  static constexpr int kMostBands = 32;

 private:
  double estimate(int tiles, double work, double tall, int nb) const;
  TileShape sh_;
  int N_, one_per_cu_;
  double base_, band_, one_band_;
};
// The tile height of least estimated cost among `cand` (wide tiles, as batches and pushes use).
int best_bands(const PlaneSize* s, int n, int R, const int* cand, int ncand);
// A plan's tiles at one level: variant and height; `one_band` runs the wide tiles of one output band
// of the Gaussian window.
struct TileChoice {
  int variant, nb, one_band;
};
TileChoice choose_tiles(int H, int W, int R, bool gauss);

}  // namespace ofmi
