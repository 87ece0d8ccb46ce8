// Choice of the iteration kernel's tiles from an estimate of a launch's time (host code).
#include "tiles.h"

#include <algorithm>
#include <array>
#include <utility>

#include "lk_iter_cfg.h"

namespace ofmi {

namespace {

template <int R, int TW, int BB>
constexpr TileShape shape() {
  using C = Cfg<R, TW, BB>;
  // workgroups per CU: 24 waves of 80 registers where the kernel is compiled for two, 160 KB LDS
  const int by_waves = waves_per_simd<R, TW, BB>() > 1 ? 24 / ((C::NT + 63) / 64) : 1;
  const int by_lds = (int)(160 * 1024 / C::LDS_BYTES);
  const int n = by_waves < by_lds ? by_waves : by_lds;
  return {TW, BB, C::NT, n < 1 ? 1 : n};
}

// Shapes of the variants of radius R (two bands per pass above kMaxPairRadius: none, wide).
template <int R>
constexpr std::array<TileShape, kTileVariants> shapes() {
  constexpr TileShape wide = shape<R, kStripWidth, 1>();
  constexpr int P = R <= kMaxPairRadius ? R : 0;
  constexpr TileShape w32 = R <= kMaxPairRadius ? shape<P, 32, 2>() : wide;
  constexpr TileShape w16 = R <= kMaxPairRadius ? shape<P, 16, 2>() : wide;
  return {wide, wide, wide, shape<R, 32, 1>(), shape<R, 16, 1>(),
          w32, w16, w32};
}
template <int... R>
constexpr std::array<std::array<TileShape, kTileVariants>, sizeof...(R)> all_shapes(
    std::integer_sequence<int, R...>) {
  return {shapes<R>()...};
}
constexpr auto kShapes = all_shapes(std::make_integer_sequence<int, 13>());

constexpr int kCus = 256;

}  // namespace

TileShape tile_shape(int variant, int R) { return kShapes[R][variant]; }

int strip_width_for(int R) {
  (void)R;   // every supported radius
  return kStripWidth;
}

// A launch's time by its tiles, fitted to event timings of every variant and tile height at r = 2, 4,
// 8, 10 on levels of 200^2 .. 2048^2 and on 16 pairs of 1024^2 (it ranks the heights as measured, or
// picks one within a few per cent).  A tile of nb output bands walks nb + 1 (the first primes the
// vertical sums) and costs a quarter band to start.  A band takes one unit on a CU of its own; k
// workgroups of t threads sharing the CU slow each other to 1 + 0.6 (k-1) t/768 (r = 8: 2.03 us
// alone, 3.3 us in twos).  Tiles beyond what the 256 CUs hold at once run in further rounds; many
// rounds even out, and only the total and a part of a last tile count.  Examples (r = 8, measured /
// model): 2048^2 at 8 bands 32.9 us / 16.8, 4 bands 36.3 / 18.8, 16 bands 42.1 / 19.3; 1024^2 at 2
// bands 14.4 / 7.2, 3 bands 16.6 / 8.8, 4 bands 15.0 / 7.3; 16 x 1024^2 at 31 bands 123, 16 bands 123,
// 8 bands 128, 4 bands 149, 2 bands 168 us.
// The Gaussian-weighted window's bands take longer (2 (2r+1) multiply-adds per product and sum),
// those of a two-band pass less so, as its vertical sums spread over all threads.  Fitted at r = 4
// and 8 on levels of 64^2 .. 1024^2, e.g. r = 8 (measured / model): 128^2 at one band in 64-column
// strips 9.5 us / 2.9, two-band passes on 32 columns 6.3 / 2.0, on 16 columns 5.7 / 1.8; 512^2 9.8 /
// 2.9, 9.1 / 2.8, 11.4 / 4.4; 1024^2 23.7 / 7.8, 24.9 / 8.6, 34.8 / 14, at two bands in 64-column
// strips 19.2 / 5.8.
LaunchCost::LaunchCost(int R, int variant, bool gauss) : sh_(tile_shape(variant, R)), N_(2 * R + 1) {
  // cost of the launch and a tile's ends, and of a band, by strip width and bands per pass
  const int tw = sh_.tw;
  const bool pair = sh_.bb == 2;
  base_ = pair || tw == 32 ? 1.5 : (tw == 16 ? 1.0 : 2.0);
  band_ = pair ? (tw == 16 ? 0.58 : 0.75) : (tw == 16 ? 0.85 : (tw == 32 ? 0.9 : 1.0));
  if (gauss) {
    base_ = R > 2 ? 5.0 / R : 2.0;
    band_ = pair ? std::min(0.8, tw == 16 ? 0.98 - 0.0575 * R : 1.1 - 0.06 * R) : 1.0;
  }
  // One-pass tiles form the output rows only and need few registers (17 to 36 up to r = 4), so that up
  // to r = 4 32 waves share a CU (r = 4, 512^2: 7.6 us at two bands in 64-column strips, 6.8 us so;
  // r = 2, 320^2: 5.9 us in 32-column strips, 5.2 us so).
  one_band_ = pair && !gauss ? band_ * 0.9 : band_;
  one_per_cu_ = pair && !gauss && R <= 4 ? 2048 / sh_.threads : sh_.per_cu;
}

double LaunchCost::estimate(int tiles, double work, double tall, int nb) const {
  auto shared = [&](int t) {   // slow-down of t tiles spread over the CUs
    return 1.0 + 0.6 * ((t + kCus - 1) / kCus - 1) * sh_.threads / 768.0;
  };
  const int slots = kCus * (nb == 1 ? one_per_cu_ : sh_.per_cu), full = tiles / slots, rest = tiles % slots;
  double t;
  if (full < 3)
    t = full * shared(slots) * tall + (rest ? shared(rest) * tall : 0.0);
  else
    t = shared(slots) * (work / slots + (rest ? 0.25 * tall : 0.0));
  return base_ + (nb == 1 ? one_band_ : band_) * t;
}

double LaunchCost::at(const PlaneSize* s, int n, int nb) const {
  long long tiles = 0;
  double work = 0, tall = 0;
  for (int i = 0; i < n; ++i) {
    const int bands = (s[i].H + N_ - 1) / N_, h = std::min(nb, bands);
    const int tx = (s[i].W + sh_.tw - 1) / sh_.tw, ty = (bands + nb - 1) / nb;
    tiles += (long long)s[i].count * tx * ty;
    work += (double)s[i].count * tx * (bands + 1.25 * ty);
    tall = std::max(tall, (h + 1 + sh_.bb - 1) / sh_.bb * sh_.bb + 0.25);
  }
  return estimate((int)std::min<long long>(tiles, 0x7fffffff), work, tall, nb);
}

// Heights that cannot be the best are passed over: below three rounds the cost is a factor of
// ceil(tiles / CUs) times the height of a tile, so of all heights with the same factor the lowest
// counts, and the next one worth a look is the lowest that takes a CU's tile off.  A level of at most
// one tile per CU at one band ends there (an exhaustive search took 4 to 9 us per plan of four levels).
int LaunchCost::least(int H, int W, int step, double& cost) const {
  const int bands = (H + N_ - 1) / N_, tx = (W + sh_.tw - 1) / sh_.tw;
  int best = 0;
  for (int nb = 1; nb <= kMostBands;) {
    const int ty = (bands + nb - 1) / nb, tiles = tx * ty;
    const double tall = (std::min(nb, bands) + 1 + sh_.bb - 1) / sh_.bb * sh_.bb + 0.25;
    const double c = estimate(tiles, tx * (bands + 1.25 * ty), tall, nb);
    if (c < cost) {
      cost = c;
      best = nb;
    }
    const int most = (tiles + kCus - 1) / kCus - 1, rows = kCus * most / tx;
    if (rows == 0) break;
    const int slots = kCus * (nb == 1 ? one_per_cu_ : sh_.per_cu);
    int next = nb + step;
    if (tiles / slots < 3 && (nb > 1 || one_per_cu_ == sh_.per_cu)) {
      next = std::max(next, (bands + rows - 1) / rows);
      next += (next - 1) % step;
    }
    nb = next;
  }
  return best;
}

int best_bands(const PlaneSize* s, int n, int R, const int* cand, int ncand) {
  // (the window's kind changes the cost of a launch and of a band of wide tiles, not the order)
  const LaunchCost model(R, kTileWide, false);
  int best = cand[0];
  double cost = 1e300;
  for (int i = 0; i < ncand; ++i) {
    const double c = model.at(s, n, cand[i]);
    if (c < cost) {
      cost = c;
      best = cand[i];
    }
  }
  return best;
}

// Variant and tile height of least estimated cost: 64-column strips, with the box window also strips
// of 32 columns (r <= 3, whose bands are short, and r > 8, which has no two-band passes) or 16
// (r > 8) and two bands per pass (r <= 8; whole passes: an odd height).
TileChoice choose_tiles(int H, int W, int R, bool gauss) {
  TileChoice t{kTileWide, 1, kTileWide};
  double cost = 1e300;
  auto consider = [&](int variant, int step) {
    const int nb = LaunchCost(R, variant, gauss).least(H, W, step, cost);
    if (nb) t.variant = variant, t.nb = nb;
  };
  consider(kTileWide, 1);
  if (!gauss) {
    if (R <= 3 || R > kMaxPairRadius) consider(kTileWide32, 1);
    if (R > kMaxPairRadius) consider(kTileWide16, 1);
    if (R <= kMaxPairRadius) {
      consider(kTileWide32x2, 2);
      consider(kTileWide16x2, 2);
    }
  } else if (R <= kMaxPairRadius) {
    // Gaussian window: tiles of one output band in 64-column strips run as two-band passes on 32
    // or 16 columns where that costs less (the sums are the same, as always).
    const PlaneSize s = {H, W, 1};
    double least = LaunchCost(R, kTileWide, true).at(&s, 1, 1);
    for (int v : {kTileWide32x2, kTileWide16x2}) {
      const double c = LaunchCost(R, v, true).at(&s, 1, 1);
      if (c < least) least = c, t.one_band = v;
    }
    if (least < cost) t.nb = 1;
  }
  return t;
}

}  // namespace ofmi
