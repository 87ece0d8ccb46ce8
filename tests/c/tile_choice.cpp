// The library's choice of tiles (host code) against an exhaustive search of the same estimate: the same
// variant and height for every radius and window over odd and even sizes, and its time per plan.
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cmath>

#include "../../paper_1306_2461_amd/csrc/tiles.hip"

using namespace ofmi;

namespace {

TileChoice exhaustive(int H, int W, int R, bool gauss) {
  const PlaneSize s = {H, W, 1};
  TileChoice t{kTileWide, 1, kTileWide};
  double cost = 1e300;
  auto consider = [&](int variant, int step) {
    const LaunchCost m(R, variant, gauss);
    for (int nb = 1; nb <= LaunchCost::kMostBands; nb += step) {
      const double c = m.at(&s, 1, nb);
      if (c < cost) cost = c, t.variant = variant, t.nb = nb;
    }
  };
  consider(kTileWide, 1);
  if (!gauss && (R <= 3 || R > kMaxPairRadius)) consider(kTileWide32, 1);
  if (!gauss && R > kMaxPairRadius) consider(kTileWide16, 1);
  if (!gauss && R <= kMaxPairRadius) consider(kTileWide32x2, 2), consider(kTileWide16x2, 2);
  if (gauss && R <= kMaxPairRadius) {
    double least = LaunchCost(R, kTileWide, true).at(&s, 1, 1);
    for (int v : {kTileWide32x2, kTileWide16x2}) {
      const double c = LaunchCost(R, v, true).at(&s, 1, 1);
      if (c < least) least = c, t.one_band = v;
    }
    if (least < cost) t.nb = 1;
  }
  return t;
}

int side(int lo, int hi) { return (int)std::lround(lo * std::pow((double)hi / lo, std::rand() / (double)RAND_MAX)); }

template <class F>
double us_per_call(F f, int n) {
  double best = 1e30;
  volatile int sink = 0;
  for (int rep = 0; rep < 7; ++rep) {
    const auto t0 = std::chrono::steady_clock::now();
    for (int i = 0; i < n; ++i) sink = sink + f(i).nb;
    const std::chrono::duration<double, std::micro> d = std::chrono::steady_clock::now() - t0;
    if (d.count() / n < best) best = d.count() / n;
  }
  return best;
}

}  // namespace

int main() {
  std::srand(1);
  int bad = 0, n = 0;
  for (int R = 0; R <= 12; ++R)
    for (int gauss = 0; gauss < 2; ++gauss)
      for (int i = 0; i < 4000; ++i) {
        const int H = i < 64 ? i + 1 : side(1, 16384), W = i < 64 ? side(1, 4096) : side(1, 16384);
        const TileChoice a = choose_tiles(H, W, R, gauss), b = exhaustive(H, W, R, gauss);
        ++n;
        if (a.variant != b.variant || a.nb != b.nb || a.one_band != b.one_band) {
          if (++bad <= 10)
            std::printf("%d x %d r=%d gauss=%d: variant %d bands %d / %d, exhaustive %d %d / %d\n", H, W, R, gauss,
                        a.variant, a.nb, a.one_band, b.variant, b.nb, b.one_band);
        }
      }
  std::printf("%d of %d choices differ\n", bad, n);
  // levels of a plan of 1024^2, the radii with the fewest and the most variants to look at
  const int sizes[] = {1024, 512, 256, 128};
  for (int R : {2, 4, 8, 10}) {
    const double c = us_per_call([&](int i) { return choose_tiles(sizes[i & 3], sizes[i & 3], R, false); }, 4000);
    const double e = us_per_call([&](int i) { return exhaustive(sizes[i & 3], sizes[i & 3], R, false); }, 4000);
    std::printf("r=%d: %.3f us per level, exhaustive %.3f us\n", R, c, e);
    if (c > e / 2) {
      std::printf("slow choice\n");
      ++bad;
    }
  }
  return bad ? 1 : 0;
}
