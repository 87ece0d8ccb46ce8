// One fused Gauss-Newton iteration of the dense window-based Lucas-Kanade method at one
// pyramid level (Sec. 2.4): warp of frame 2 by the current field, central-difference
// gradients of the warped frame, the five window sums, the 2x2 solve and the update.
//
// Work decomposition (gfx950, wave64):
//   * a workgroup owns a strip of TW output columns and TH output rows;
//   * it walks down the strip in bands of N = 2r+1 product rows; per band:
//       P1  warped frame of the band's new rows into LDS: a thread owns K1 successive rows of
//           one column, and the field it needs is in flight since P2 of the band before;
//       P2  the five products Ix^2, IxIy, Iy^2, Ix It, Iy It of the band's rows into LDS;
//       P3  horizontal window sums: one thread per (channel, row, 8-column segment); every
//           window of a segment holds one common column, so each window is a suffix sum plus
//           a prefix sum of its own values (no subtraction of values leaving the window);
//           r <= 3 takes direct sums (segments sit on multiples of 8 of the level's columns);
//           the Gaussian-weighted window takes a direct weighted sum per output instead;
//       P4  vertical window sums: one thread per (channel, column) holds the previous
//           band's horizontal sums in registers; the window of the band's row i is the
//           suffix sum of the previous band from row i+1 plus the prefix sum of the current
//           band up to row i (fixed order; bands sit on a global grid of period N), or the
//           direct weighted sum over the same rows for the Gaussian-weighted window;
//       P5  per-pixel 2x2 solve and update for the band's output rows.
//           The Gaussian sums are 2r+1 multiply-adds each and bound their P4: the rows of a column
//           are split over two threads (over all threads in two-band passes), results go where the
//           products were, and a tile's first band forms only the row that it outputs.  r = 8,
//           per iteration: 1024^2 21.7 -> 20.5 us, 128^2 10.4 -> 9.5 us in 64-column strips and
//           5.7 us in two-band passes on 16 columns (512^2, 32 columns: 11.9 -> 9.9 us);
//   The window sums therefore do not depend on how the image is cut into tiles.
//   * two-bands-per-pass variants run the five phases once over two bands' rows, so a one-band
//     tile (output band plus priming band) is one trip (Gaussian window: one-band tiles only).
//
// What bounds it: vector instructions (two thirds of the CUs' clocks on a full device) and the waits
// between the five phases; HBM is at about half of what a copy reaches.  Two workgroups per CU hide
// each other's barriers and load rounds, which asks for at most 80 registers per thread (three waves
// per SIMD each).  A third of the vector instructions of an earlier form went into per-item index
// arithmetic, and variants that kept more in flight (samples gathered a band ahead) spilled or fell to
// one workgroup per CU and were slower.  Measured on level 0 of 16 pairs of 1024^2 (r = 8, uint8, tiles
// of 16 bands, iterations of a level averaged): 139.8 us per launch before the per-column mapping,
// 8-bit samples and paired coarse rows below, 119.5 us with them, 113 us with the field handed on and
// the first band's unused rows left out (16.8 Mpx: 2.7 TB/s of algorithmic bytes); a plan's 2048^2
// level 0 (8 bands) 42.9 -> 32 us.
// Scratch: 32 bytes per thread in tiles of several two-band passes on 32 columns from a coarser level at
// r = 8 (11 MiB written per launch of 1024^2; one launch of a level, at the sizes whose least estimate
// they are), 8 and 12 in FP16 levels of 32-column strips at r = 9 and 10, 8 in Gaussian batches at r = 8
// (8-bit frames; FP16 from a coarser level); the other forms have none.  At one workgroup per CU, which
// would need none, Gaussian launches took 5 to 20 % longer.
// Vector memory instructions cost by form, not by bytes: 64 lanes at unit stride 4.7 clocks per CU
// (bytes or dwords), 64-bit, stride-2 or unaligned 16-bit lanes 16 clocks, so every load and store here
// is one element per lane at unit stride and a bilinear tap pair is two byte loads.
#pragma once

#include <type_traits>

#include "kernels.h"
#include "lk_iter_cfg.h"

namespace ofmi {

namespace {

// Adds every lane's count to *dst: a wave sum, then one atomic per wave.
__device__ __forceinline__ void add_count(unsigned long long* dst, unsigned c) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
  if ((threadIdx.x & 63) == 0 && c) atomicAdd(dst, (unsigned long long)c);
}

// Whether a launch hands its field rows on to P5 through LDS instead of reading the field planes
// again: from a coarser level a pixel's field takes eight loads and two interpolations.  Batched
// launches only (16 pairs of 1024^2, first iteration of level 0: 138.9 -> 124.1 us; a plan's tiles are
// shorter: 2048^2 level 0 32.3 us either way), and not of 16-bit frames, whose samples leave no
// registers for it (24 mixed pairs, level 1: 75.9 us, handed on 86.0 us with 36 bytes of scratch).
// r = 0 outputs a row above a tile's first sampled rows.
template <typename T, int R, int MODE, bool GAUSS, bool BUB>
constexpr bool field_handed() {
  return R > 0 && MODE == kFlowCoarse && !GAUSS && !BUB && sizeof(T) != 2;
}

// One tile: TW output columns from x0 = bx*TW and TH output rows from row y0, walked in
// nbands bands (TH is a multiple of N; nbands = TH/N + 1).  `sm4` is the workgroup's LDS.
// INTERIOR: the tile's whole warped-frame region (the tile grown by r + 1 px, all bands)
// lies inside the image, so no position needs clamping or an in-image test.
// pixel_mask: the tile holds masked pixels, whose flow is written as zero.
// GAUSS: window sums weighted by the separable taps a.taps[0..2r] (Gaussian-weighted window)
// instead of the unweighted box: every horizontal and vertical sum is a direct 2r+1-term
// weighted sum in a fixed order, so results remain independent of the tiling.
// BUB: the launch may carry the eq. 3 count (plain launches; checked at run time there).
// BB: bands per pass.  With BB = 2 the phases run over two bands' rows at once with twice the
// threads, so a tile of two bands (one output band and the band that primes the vertical
// sums) is one pass of the dependent path instead of two; P4 walks the two bands in order,
// with the same additions as two single-band passes.  nbands is then even.
// ONE (BB = 2): the tile is one pass (one output band).  Nothing is carried to a next pass (17
// registers at r = 8, which the launches from a coarser level otherwise spill), P4 forms only the rows
// that are output and P5 is a single round: r = 8, iterations of a 512^2 level on 32 columns 8.4 -> 7.8 us,
// of a 256^2 level on 16 columns 5.3 -> 5.1 us.
template <typename T, int R, int TW, int MODE, bool INTERIOR, bool GAUSS, int BB, bool BUB, bool ONE>
__device__ __forceinline__ void strip_tile(const IterArgs& a, int TH, int bands, int bx, int y0,
                                           bool pixel_mask, float4* sm4) {
  static_assert(!ONE || BB == 2, "one pass: both of its bands");
  const int nbands = ONE ? BB : bands;
  using C = Cfg<R, TW, BB>;
  constexpr int N = C::N, NR = C::NR, NT = C::NT, PC = C::PC, WC = C::WC, PP = C::PP, WP = C::WP,
                HP = C::HP, K1 = C::K1, G = C::G, F0 = C::P1_FIRST;
  constexpr bool FLOW = MODE != kFlowZero;
  static_assert(BB == 1 || BB == 2, "one or two bands per pass");
  float* pr = reinterpret_cast<float*>(sm4);    // [5][NR][PP] products (16-byte aligned rows)
  float* w2 = pr + C::PR_FLOATS;                // [W2ROWS][WP] warped frame from row tb-1
  float* hs = w2 + C::W2_FLOATS;                // [5][NR][HP] horizontal, then window sums
  float* fcu = hs + C::HS_FLOATS;               // [G][WP] field rows passed on to P2
  float* fcv = fcu + G * WP;
  float* ru = fcv + G * WP;                     // [RING][TW] field rows passed on to P5
  float* rv = ru + C::RING * TW;

  // Opaque per tile, so that a work-list kernel forms what depends on it per tile instead of
  // keeping it in registers across the tiles of both paths.
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int H = a.H, W = a.W;
  const int x0 = bx * TW;
  const Plane<T> I1((const T*)a.I1, H, W), I2((const T*)a.I2, H, W);
  const Plane<float> U(a.uin, MODE == kFlowCoarse ? a.Hc : H, MODE == kFlowCoarse ? a.Wc : W);
  const Plane<float> V(a.vin, MODE == kFlowCoarse ? a.Hc : H, MODE == kFlowCoarse ? a.Wc : W);
  const Plane<float> UO(a.uout, H, W), VO(a.vout, H, W);

  // This thread's column of the warped frame and its first row of a pass (threads past the last
  // group repeat that group: the same values to the same slots; where they are the most, at r = 0,
  // they sample nothing: a pair of 1024^2 192 -> 140 us, 8 pairs of 640 x 480 at one band
  // 514 -> 482 us).
  using DW = ConstDiv<WC, NT>;
  const int gq = (int)DW::q((unsigned)tid), lx = (int)DW::r((unsigned)tid, (unsigned)gq);
  const int gc = min(gq, G - 1), g = gc * K1;
  const int gx = INTERIOR ? x0 - R - 1 + lx : min(max(x0 - R - 1 + lx, 0), W - 1);
  const bool pcol_in = INTERIOR || (x0 - R - 1 + lx >= 0 && x0 - R - 1 + lx < W);
  const bool p2 = lx >= 1 && lx <= PC && gq < G;
  const bool own = NT / WC < 2 * G || gq < G;
  // EVEN: launches from a coarser level whose threads own pairs of rows start a pass one row early
  // where its first row is odd (its last one the pass before: the same value to the same slot), so that
  // every pair lies between the same two rows of the coarser level.  24 mixed pairs, first iteration of
  // level 0: 316 us with a third row for every pair (and 8 to 40 bytes of scratch in 20 forms), 288 us so.
  constexpr bool EVEN = MODE == kFlowCoarse && BB == 1 && K1 % 2 == 0;
  static_assert(!EVEN || G * K1 > C::P1_ROWS, "no row to spare for a pass that starts early");
  constexpr int kLast = (G - 1) * K1;            // the last group's first row
  // its last row (EVEN: of a pass that starts early, the only ones whose next pass asks for it)
  constexpr int kEnd = C::P1_ROWS - 1 - kLast + (EVEN ? 1 : 0);
  // Image row i from image row ys (clamped).
  auto row_at = [&](int ys, int i) { return INTERIOR ? ys + i : min(max(ys + i, 0), H - 1); };
  // Element (gx, row i from image row ys) of a plane: interior tiles add a scalar row base to a
  // per-thread offset.
  auto elem = [&](const auto& p, int ys, int i) {
    if constexpr (INTERIOR)
      return p.ld(__umul24((unsigned)i, (unsigned)W) + (unsigned)lx, ys * W + x0 - R - 1);
    else
      return p.ld(rowofs(row_at(ys, i), W, gx), 0);
  };
  // Field at column gx of K rows from row i of the rows from image row ys: loads, and row k's value.
  auto field = [&](auto& f, int ys, int i, auto rows) {
    constexpr int K = decltype(rows)::value;
    if constexpr (MODE == kFlowSame) {
#pragma unroll
      for (int k = 0; k < K; ++k) {
        f.u[k] = elem(U, ys + k, i);
        f.v[k] = elem(V, ys + k, i);
      }
    } else if constexpr (MODE == kFlowCoarse) {
#pragma unroll
      for (int k = 0; k < K; k += 2)
        f.template issue<INTERIOR>(k / 2, U, V, a.Hc, a.Wc, gx, INTERIOR ? ys + k + i : row_at(ys + k, i));
    }
  };
  auto field_at = [&](const auto& f, int ys, int i, int k) {
    return f.template at<INTERIOR>(k, row_at(ys + k, i), row_at(ys + k / 2 * 2, i));
  };
  // Frame 1 one row above this thread's k-th row of the pass whose LDS row 0 is image row yw.
  auto frame1 = [&](int yw, int k) {
    if (F0 == 0 && k == 0) return elem(I1, yw, max(g - 1, 0));
    return elem(I1, yw + F0 + k - 1, g);
  };
  using S = Sample<T>;

  // P4 ownership: channel and column of this thread (the first 5*TW threads).
  // The Gaussian-weighted window's takes the threads past those too: the first 5*TW threads one
  // part of the rows, the next 5*TW the following part, and so on.
  constexpr int P4S = !GAUSS ? 1 : (BB == 2 ? NT / (5 * TW) : (NT >= 10 * TW ? 2 : 1));
  const int vq = GAUSS ? tid / (5 * TW) : 0;
  const int vk = tid / TW - 5 * vq, vc = tid % TW;
  const bool p4 = GAUSS ? vq < P4S : vk < 5;
  // P5 ownership: output column and row of a round (the row is uniform over a wave on
  // 64-column strips).
  const int oc = tid % TW, orow = TW == 64 ? __builtin_amdgcn_readfirstlane(tid / TW) : tid / TW;
  const int ogx = INTERIOR ? x0 + oc : min(x0 + oc, W - 1);
  float prev[N];
#pragma unroll
  for (int i = 0; i < N; ++i) prev[i] = 0.f;

  // eq. 3 count of the final iteration: u values at or below the threshold written by this
  // thread (one atomic per wave at the end)
  const bool bub = BUB && a.bcount != nullptr;
  const float bthr = bub ? at(a.bthr, 0u) : 0.f;
  unsigned bcnt = 0;

  // Field rows passed on: thread group q reads slot q, the field at the row above its first:
  // the last row of group q-1 of the pass, for group 0 the last row of the pass before, which
  // the last group keeps in registers until then.
  float lu = 0.f, lv = 0.f;
  auto keep_field = [&](const float* fu, const float* fv, bool first) {
    if constexpr (FLOW) {
      const bool end = gc == G - 1;
      if (!(first && end)) {
        const int s = (end ? 0 : gc + 1) * WP + lx;
        fcu[s] = end ? lu : fu[K1 - 1];
        fcv[s] = end ? lv : fv[K1 - 1];
      }
      lu = fu[kEnd];
      lv = fv[kEnd];
    }
  };

  // HANDED: the field rows go on to P5 in LDS.  ring_row is the slot of the pass's first sampled row;
  // P2 writes them: every wave has then left P5 of the pass before.
  constexpr bool HANDED = field_handed<T, R, MODE, GAUSS, BUB>();
  constexpr int RING = C::RING;
  int ring_row = 0;
  auto wrap = [](int s) { return s >= RING ? s - RING : s; };
  // Rows of a pass that P5 visits, and its rounds.
  constexpr int R5 = ONE ? 2 * R : 0, N5 = ONE ? N : NR, K5 = (N5 + C::RG - 1) / C::RG;
  // Field at this thread's output pixel of round k (clamped row: one outside the tile or the
  // image is loaded and not used).
  auto centre = [&](FieldRows<MODE, 1>& c, int tb, int k) {
    const int gy = min(max(y0 + tb - 2 * R + R5 + C::RG * k + orow, 0), H - 1);
    if constexpr (MODE == kFlowCoarse) {
      c.template issue<false>(0, U, V, a.Hc, a.Wc, ogx, gy);
    } else if constexpr (MODE == kFlowSame) {
      c.u[0] = U.ld(rowofs(gy, W, ogx), 0);
      c.v[0] = V.ld(rowofs(gy, W, ogx), 0);
    }
  };
  // P5 of the pass whose first product row is tb: 2x2 solve and update of its output rows, with
  // the field c at this thread's output pixels.  Lanes without an output pixel store past the
  // plane (dropped), so that the number of stores in flight is known where the samples issued
  // before them are waited for.
  // (The Gaussian-weighted window's sums replace the products, whose last readers P3 were.)
  const float* win = GAUSS ? pr : hs;
  constexpr int VP = GAUSS ? PP : HP;
  auto solve = [&](int tb, FieldRows<MODE, 1>* c) {
    // slot of the pass's first output row, tile row tb - 2R: R + 1 above its first sampled one
    const int s0 = wrap(ring_row + N);
#pragma unroll
    for (int k = 0; k < K5; ++k) {
      const int r = R5 + orow + C::RG * k, j = tb + r - 2 * R;   // row of the pass, of the tile
      if (C::RG * (k + 1) > N5 && r >= R5 + N5) continue;
      __builtin_amdgcn_sched_barrier(0);   // one round's registers at a time
      if constexpr (MODE == kFlowCoarse && !HANDED) centre(c[k], tb, k);
      const int gy = y0 + j;
      const bool out = j >= 0 && j < TH && (INTERIOR || (x0 + oc < W && gy < H));
      float un = 0.f, vn = 0.f;
      // (a row above the tile: of its first band, uniform over a wave on 64-column strips)
      if (TW != 64 || j >= 0) {
        const float* s = win + r * VP + oc;
        float2 f5;
        if constexpr (HANDED) {
          const int q = wrap(s0 + r) * TW + oc;
          f5 = make_float2(ru[q], rv[q]);
        } else {
          f5 = c[k].template at<false>(0, gy, gy);
        }
        solve_update(s[0], s[NR * VP], s[2 * NR * VP], s[3 * NR * VP], s[4 * NR * VP], f5.x, f5.y,
                     un, vn);
      }
      const unsigned o = rowofs(gy, W, x0 + oc);
      if (pixel_mask) {   // masked-out pixels: zero flow
        if (out && at(a.mask, o) == 0) un = vn = 0.f;
      }
      UO.st(out ? o : 0x3fffffffu, un);
      VO.st(out ? o : 0x3fffffffu, vn);
      if constexpr (BUB) {
        if (bub) bcnt += out && un <= bthr ? 1u : 0u;
      }
    }
  };
  // The field at a pass's warped-frame rows: a same-level launch loads it during P2 of the pass
  // before (ahead of that pass's stores, which a later load would be waited for with), a
  // coarse-field launch, whose values take eight loads and more, in P1.
  constexpr bool AHEAD = MODE == kFlowSame;
  constexpr std::integral_constant<int, K1> kRows{};
  FieldRows<MODE, K1, EVEN> f;
  if constexpr (AHEAD) {
    if (own) field(f, y0 - R - 1 + F0, g, kRows);
  }
  for (int b = 0; b < nbands; b += BB) {
    const int tb = N * b;                        // first product row of the pass
    const int yw = y0 - R - 1 + tb;              // image row of LDS row 0
    const bool more = b + BB < nbands;
    const int early = EVEN ? (yw + F0) & 1 : 0;  // rows that the threads' rows start above LDS row F0
    const int ys = yw + F0 - early;              // image row of the first thread group's first row
    // ------------------------------------------------------------------ P1
    // Branch-free loads (clamped addresses).  In a tile's first band the two rows above it (LDS
    // rows 0 and 1) are sampled here too.
    float wu[K1], wv[K1], i1v[K1], wval[K1];
    {
      const bool ext = BB == 1 && b == 0 && tid < 2 * WC;
      FieldRows<MODE, 1> ef;
      if (ext) field(ef, yw, gq, std::integral_constant<int, 1>{});
      if constexpr (!AHEAD) {
        if (own) field(f, ys, g, kRows);
      }
#pragma unroll
      for (int k = 0; k < K1; ++k) {
        if (own) i1v[k] = frame1(yw - early, k);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < K1; ++k) {
        if (!own) continue;
        const float2 w = field_at(f, ys, g, k);
        wu[k] = w.x;
        wv[k] = w.y;
      }
      float eu = 0.f, ev = 0.f;
      S smp[K1], es;
      if (ext) {
        const float2 w = field_at(ef, yw, gq, 0);
        eu = w.x;
        ev = w.y;
        es.issue(I2, H, W, gx, row_at(yw, gq), eu, ev);
      }
#pragma unroll
      for (int k = 0; k < K1; ++k) {
        if (own) smp[k].issue(I2, H, W, gx, row_at(ys + k, g), wu[k], wv[k]);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (own) keep_field(wu, wv, b == 0);
      if (ext) {
        if (FLOW && gq == 1) {
          fcu[lx] = eu;
          fcv[lx] = ev;
        }
        w2[gq * WP + lx] = es.value();
      }
#pragma unroll
      for (int k = 0; k < K1; ++k) {
        if (!own) continue;
        wval[k] = smp[k].value();
        w2[(g + F0 + k - early) * WP + lx] = wval[k];
      }
    }
    __syncthreads();
    // ------------------------------------------------------------------ P2
    if constexpr (AHEAD) {
      if (more && own) field(f, yw + NR + F0, g, kRows);
    }
    if constexpr (HANDED) {
      const int c = lx - R - 1;
      if (c >= 0 && c < TW && gq < G) {
#pragma unroll
        for (int k = 0; k < K1; ++k) {
          const int i = g + k - early;
          if ((kLast + k < N || i < N) && (!EVEN || k > 0 || i >= 0)) {
            const int q = wrap(ring_row + i) * TW + c;
            ru[q] = wu[k];
            rv[q] = wv[k];
          }
        }
      }
    }
    // The products one row above each of this thread's warped rows: the row below is the
    // thread's own, the centre and the row above too from its second and third row on.
    if (p2) {
      constexpr int kSkip = 2 - F0;   // with two bands per pass rows -1 and 0 have no product above
      const float* wr = w2 + (g + F0 - early) * WP + lx;   // this thread's first warped row
      const int up = kSkip == 0 || g > 0 ? 1 : 0;
      // one, two rows above (two above LDS row 1: any row, for the product that is left out below)
      float c1 = wr[-up * WP], c2 = wr[-(EVEN && g < early ? 1 : 2) * up * WP];
      float fu = 0.f, fv = 0.f;       // field at the product position
      if constexpr (FLOW) {
        fu = fcu[gc * WP + lx];
        fv = fcv[gc * WP + lx];
      }
#pragma unroll
      for (int k = 0; k < K1; ++k) {
        const int i = g + k - early;   // sampled row of the pass
        if ((EVEN ? k > 0 || i >= 0 : kSkip == 0 || i >= kSkip) && (kLast + k < C::P1_ROWS || i < C::P1_ROWS)) {
          const int r = i - kSkip;
          const float* row = wr + (k - 1) * WP;
          float ix = 0.5f * (row[1] - row[-1]);
          float iy = 0.5f * (wval[k] - c2);
          float it = c1 - i1v[k];
          it = fmaf(-ix, fu, it);
          it = fmaf(-iy, fv, it);
          if constexpr (!INTERIOR) {   // no product outside the image
            const int gy = yw + 1 + r;
            const bool in = pcol_in && gy >= 0 && gy < H;
            ix = in ? ix : 0.f;
            iy = in ? iy : 0.f;
            it = in ? it : 0.f;
          }
          float* q = pr + r * PP + lx - 1;
          q[0] = ix * ix;
          q[NR * PP] = ix * iy;
          q[2 * NR * PP] = iy * iy;
          q[3 * NR * PP] = ix * it;
          q[4 * NR * PP] = iy * it;
        }
        c2 = c1;
        c1 = wval[k];
        if constexpr (FLOW) {
          fu = wu[k];
          fv = wv[k];
        }
      }
    }
    __syncthreads();
    // ------------------------------------------------------------------ P3
    // The last two warped rows are the next band's first two.
    if constexpr (BB == 1 && R == 0) {   // the row moved first is the next one's place
      if (more && tid < WP) {
        w2[tid] = w2[WP + tid];
        w2[WP + tid] = w2[2 * WP + tid];
      }
    } else if constexpr (BB == 1) {
      if (more && tid < 2 * WP) w2[tid] = w2[N * WP + tid];
    }
    // Items are (segment, channel and row), the row fastest over the lanes.
    using DS = ConstDiv<5 * NR, C::K3 * NT>;
#pragma unroll
    for (int k = 0; k < C::K3; ++k) {
      const int i = tid + k * NT;
      if (i < 5 * NR * C::NSEG) {
        const int seg = (int)DS::q((unsigned)i), rr = (int)DS::r((unsigned)i, (unsigned)seg);   // rr = ch * NR + row
        typedef float f4v __attribute__((ext_vector_type(4)));
        const f4v* src = reinterpret_cast<const f4v*>(pr + rr * PP + 8 * seg);
        // The empty asm takes the four values of a read as one 128-bit register operand, so each
        // read stays one 128-bit LDS load (the sums below use the values out of order, and the
        // loads were otherwise split into 32-bit pairs).
        f4v f[C::HL4];
        float vbuf[4 * C::HL4], hv[8];
#pragma unroll
        for (int q = 0; q < C::HL4; ++q) f[q] = src[q];
#pragma unroll
        for (int q = 0; q < C::HL4; ++q) {
          asm("" : "+v"(f[q]));
          vbuf[4 * q] = f[q].x;
          vbuf[4 * q + 1] = f[q].y;
          vbuf[4 * q + 2] = f[q].z;
          vbuf[4 * q + 3] = f[q].w;
        }
        if constexpr (GAUSS) {
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            float s = a.taps[0] * vbuf[j];
#pragma unroll
            for (int q = 1; q <= 2 * R; ++q) s = fmaf(a.taps[q], vbuf[j + q], s);
            hv[j] = s;
          }
        } else if constexpr (2 * R >= 7) {
          // Every window of the segment holds column 2R (the last column of window 0), so
          // window j is the suffix vbuf[j..2R] plus the prefix vbuf[2R+1..2R+j]: sums of
          // values inside the window only.  (A running sum that subtracts the value leaving
          // the window carries a rounding error relative to the largest product of the
          // segment rather than of the window, which ill-conditioned windows amplify.)
          float suf = vbuf[7];   // vbuf[7..2R], in load order
#pragma unroll
          for (int q = 8; q <= 2 * R; ++q) suf += vbuf[q];
          float sj[8];
          sj[7] = suf;
#pragma unroll
          for (int j = 6; j >= 0; --j) sj[j] = vbuf[j] + sj[j + 1];
          hv[0] = sj[0];
          float pre = 0.f;
#pragma unroll
          for (int j = 1; j < 8; ++j) {
            pre = j == 1 ? vbuf[2 * R + 1] : pre + vbuf[2 * R + j];
            hv[j] = sj[j] + pre;
          }
        } else {
          // r <= 3: direct sums, at most 6 additions per output
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            float s = vbuf[j];
#pragma unroll
            for (int q = 1; q <= 2 * R; ++q) s += vbuf[j + q];
            hv[j] = s;
          }
        }
        float4* dst = reinterpret_cast<float4*>(hs + rr * HP + 8 * seg);
        dst[0] = make_float4(hv[0], hv[1], hv[2], hv[3]);
        dst[1] = make_float4(hv[4], hv[5], hv[6], hv[7]);
      }
    }
    __syncthreads();
    // ------------------------------------------------------------------ P4
    FieldRows<MODE, 1> c5[K5];
    if constexpr (AHEAD) {
#pragma unroll
      for (int k = 0; k < K5; ++k) centre(c5[k], tb, k);
    }
    if (GAUSS && BB == 2 && p4) {
      // A tile of one pass: its output rows 2R .. 4R have their whole windows in the pass, M rows
      // per thread, each the taps in order from the window's top row.
      constexpr int M = (N + P4S - 1) / P4S;
      const int top = min(vq * M, N - 1);
      const float* col = hs + vk * NR * HP + vc;
      float x[M + 2 * R];
#pragma unroll
      for (int i = 0; i < M + 2 * R; ++i) x[i] = col[min(top + i, NR - 1) * HP];
      float* dst = pr + (vk * NR + 2 * R + top) * PP + vc;
#pragma unroll
      for (int m = 0; m < M; ++m) {
        float s = 0.f;
#pragma unroll
        for (int q = 0; q <= 2 * R; ++q) s = fmaf(a.taps[q], x[m + q], s);
        if (top + m < N) dst[m * PP] = s;
      }
    } else if (GAUSS && p4) {
      // Output row r of the band: previous-band rows r+1..N-1 then current rows 0..r, i.e.
      // window offsets 0..N-1 from its top row, weighted by the taps in that order.  A tile's
      // first band has one output row, its last.
      const float* col = hs + vk * N * HP + vc;
      float* dst = pr + vk * N * PP + vc;
      float cur[N];
#pragma unroll
      for (int r = 0; r < N; ++r) cur[r] = col[r * HP];
      auto rows = [&](auto first, auto last) {
#pragma unroll
        for (int r = decltype(first)::value; r <= decltype(last)::value; ++r) {
          float s = 0.f;
#pragma unroll
          for (int m = r + 1; m < N; ++m) s = fmaf(a.taps[m - r - 1], prev[m], s);
#pragma unroll
          for (int m = 0; m <= r; ++m) s = fmaf(a.taps[N - 1 - r + m], cur[m], s);
          dst[r * PP] = s;
        }
      };
      using std::integral_constant;
      constexpr int kCut = P4S == 2 ? R : -1;   // last row of the first part
      if (b == 0) {
        if (vq == P4S - 1) rows(integral_constant<int, N - 1>{}, integral_constant<int, N - 1>{});
      } else if (P4S == 2 && vq == 0) {
        rows(integral_constant<int, 0>{}, integral_constant<int, kCut>{});
      } else {
        rows(integral_constant<int, kCut + 1>{}, integral_constant<int, N - 1>{});
      }
#pragma unroll
      for (int r = 0; r < N; ++r) prev[r] = cur[r];
    } else if (p4) {
#pragma unroll
      for (int bb = 0; bb < BB; ++bb) {
        float* col = hs + vk * NR * HP + bb * N * HP + vc;
        // All reads before the first write: one LDS round trip instead of one per few rows.
        float cur[N];
#pragma unroll
        for (int r = 0; r < N; ++r) cur[r] = col[r * HP];
        __builtin_amdgcn_sched_barrier(0);
        // A tile's first band outputs its last row (with P5's skipped rows: 2048^2 level 0 at 8
        // bands 32.2 -> 31.7 us, 1024^2 at 2 bands 13.9 -> 13.6 us).
        if (BB == 1 && b == 0) {
          float s = cur[0];
#pragma unroll
          for (int r = 1; r < N; ++r) s += cur[r];
          col[(N - 1) * HP] = s;
#pragma unroll
          for (int r = 0; r < N; ++r) prev[r] = cur[r];
          continue;
        }
        // prev[r] <- prev[r] + ... + prev[N-1] (suffix sums of the previous band, in place)
#pragma unroll
        for (int r = N - 2; r >= 0; --r) prev[r] += prev[r + 1];
        float pre = 0.f;
#pragma unroll
        for (int r = 0; r < N; ++r) {
          pre = r == 0 ? cur[r] : pre + cur[r];
          if (!ONE || bb == 1 || r + 1 == N) col[r * HP] = r + 1 < N ? prev[r + 1] + pre : pre;
          prev[r] = cur[r];
        }
      }
    }
    __syncthreads();
    // ------------------------------------------------------------------ P5
    solve(tb, c5);
    ring_row = wrap(ring_row + N);
    // The next pass's P1 writes warped rows and field rows that this pass's P2 finished reading
    // before the barriers above; its P3 rewrites the window sums after two more barriers.
  }
  if constexpr (BUB) {
    if (bub) add_count(a.bcount, bcnt);
  }
}

// True when every position that the tile samples (columns x0-R-1 .. x0+TW+R, rows y0-R-1 .. the
// last row of the last pass's threads) lies inside the image, from a coarser level also the rows and
// columns after those positions' coarse ones.
template <class C, int MODE>
__device__ __forceinline__ bool tile_interior(const IterArgs& a, int nbands, int bx, int y0) {
  constexpr int E = MODE == kFlowCoarse ? 3 : 1;
  constexpr int R = (C::N - 1) / 2;
  const int x0 = bx * C::TW;
  const int last = y0 - R - 1 + C::N * nbands - C::NR + C::P1_FIRST + C::G * C::K1 - 1;
  return x0 - R - 1 >= 0 && x0 + C::TW + R <= a.W - E && y0 - R - 1 >= 0 && last <= a.H - E;
}

// Masked plans: a tile without an unmasked output pixel (TW columns from x0, TH rows from
// y0) is not computed; its workgroup writes zero flow over it (and counts those zeros for the
// eq. 3 count when the threshold is not negative).
template <int TW>
__device__ __forceinline__ void zero_tile(const IterArgs& a, int TH, int bx, int y0) {
  const int x0 = bx * TW;
  const int w = min(TW, a.W - x0), h = min(TH, a.H - y0);
  for (int i = threadIdx.x; i < w * h; i += blockDim.x) {
    const int r = i / w, c = i - r * w;
    const unsigned o = (unsigned)(y0 + r) * (unsigned)a.W + (unsigned)(x0 + c);
    at(a.uout, o) = 0.f;
    at(a.vout, o) = 0.f;
  }
  if (a.bcount != nullptr && threadIdx.x == 0 && 0.f <= at(a.bthr, 0u))
    atomicAdd(a.bcount, (unsigned long long)w * (unsigned long long)h);
}

// Workgroup index -> work index so that the workgroups one XCD runs (hardware dispatch is
// round-robin over the 8 XCDs) take a contiguous range of tiles, which share halos in L2.
__device__ __forceinline__ int xcd_order(int b, int nblocks) {
  constexpr int kXcd = 8;
  const int per = (nblocks + kXcd - 1) / kXcd;
  return (b % kXcd) * per + b / kXcd;
}

template <typename T, int R, int TW, int MODE, bool GAUSS, int BB, bool ONE>
__global__ __launch_bounds__((group_threads<R, TW, BB>()), (waves_per_simd<R, TW, BB>())) void lk_iter_strip(IterArgs a, int TH,
                                                                           int nbands, int tiles_x,
                                                                           int ntiles) {
  extern __shared__ float4 sm4[];
  const int t = xcd_order(blockIdx.x, gridDim.x);
  if (t >= ntiles) return;
  const int bx = t % tiles_x, y0 = t / tiles_x * TH;
  bool pixel_mask = false;
  if (a.mask) {
    const int f = a.tiles[t];
    if (f == 0) {
      zero_tile<TW>(a, TH, bx, y0);
      return;
    }
    pixel_mask = f == 1;
  }
  if (tile_interior<Cfg<R, TW, BB>, MODE>(a, nbands, bx, y0))
    strip_tile<T, R, TW, MODE, true, GAUSS, BB, true, ONE>(a, TH, nbands, bx, y0, pixel_mask, sm4);
  else
    strip_tile<T, R, TW, MODE, false, GAUSS, BB, true, ONE>(a, TH, nbands, bx, y0, pixel_mask, sm4);
}

// Batched form: workgroups stride over a work list of tiles of many pairs at the same
// (level, iteration) phase.  Work item = (pair | tile flag << 16, tile x, first output row,
// output rows, a multiple of 2r+1).  For a pair with a mask (in its arguments) the flag tells
// a tile without an unmasked pixel (0, zero-filled), one with masked pixels (1) and one
// without (2).
// MASK: launches of batches with masks (the mask code costs the unmasked launches about 5 %
// more instructions and is compiled out of them).
template <typename T, int R, int TW, int MODE, bool GAUSS, bool MASK>
__global__ __launch_bounds__((group_threads<R, TW, 1>()), (waves_per_simd<R, TW, 1>())) void lk_iter_batch(const IterArgs* __restrict__ args,
                                                                      const int4* __restrict__ tiles,
                                                                      int ntiles) {
  extern __shared__ float4 sm4[];
  using C = Cfg<R, TW>;
  const int stride = (int)gridDim.x;
  for (int t = xcd_order(blockIdx.x, gridDim.x); t < ntiles; t += stride) {
    const int4 w = tiles[t];
    const IterArgs a = args[w.x & 0xffff];
    const int nb = w.w / C::N + 1;
    bool pixel_mask = false;
    if constexpr (MASK) {
      if (a.mask) {
        const int f = (int)((unsigned)w.x >> 16);
        if (f == 0) {
          zero_tile<TW>(a, w.w, w.y, w.z);
          continue;
        }
        pixel_mask = f == 1;
      }
    }
    if (tile_interior<C, MODE>(a, nb, w.y, w.z))
      strip_tile<T, R, TW, MODE, true, GAUSS, 1, false, false>(a, w.w, nb, w.y, w.z, pixel_mask, sm4);
    else
      strip_tile<T, R, TW, MODE, false, GAUSS, 1, false, false>(a, w.w, nb, w.y, w.z, pixel_mask, sm4);
    __syncthreads();
  }
}

// nb output bands per tile take nb + 1 bands (the first primes the vertical sums), rounded up
// to whole passes of BB bands (a band past the tile's rows writes nothing).
template <typename T, int R, int MODE, bool GAUSS, int TWV = 0, int BB = 1, bool ONE = false>
hipError_t go_plain_v(const IterArgs& a, int nb, hipStream_t s) {
  constexpr int TW = TWV ? TWV : kStripWidth;
  using C = Cfg<R, TW, BB>;
  constexpr size_t kLds = C::LDS_BYTES;
  static_assert(kLds <= 160 * 1024, "LDS footprint above 160 KB");
  const int TH = C::N * nb;
  const int tx = (a.W + TW - 1) / TW, ty = (a.H + TH - 1) / TH;
  const int ntiles = tx * ty;
  const int grid = (ntiles + 7) / 8 * 8;
  const int nbands = (nb + 1 + BB - 1) / BB * BB;
  if constexpr (kLds > 65536) {
    static std::atomic<uint64_t> done{0};
    const hipError_t e =
        allow_lds(reinterpret_cast<const void*>(&lk_iter_strip<T, R, TW, MODE, GAUSS, BB, ONE>), kLds, done);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((lk_iter_strip<T, R, TW, MODE, GAUSS, BB, ONE>), dim3(grid),
                     dim3(C::NT), kLds, s, a, TH, nbands, tx, ntiles);
  return hipGetLastError();
}

template <typename T, int R, int MODE, bool GAUSS>
hipError_t go_plain_g(const IterArgs& a, int nb, int variant, hipStream_t s) {
  switch (variant) {
    case kTileNarrow:
    case kTileWide:
    case kTileWideLean: return go_plain_v<T, R, MODE, GAUSS>(a, nb, s);
  }
  if constexpr (!GAUSS) {
    switch (variant) {   // narrow strips, one band per pass: box window only
      case kTileWide32: return go_plain_v<T, R, MODE, false, 32>(a, nb, s);
      case kTileWide16: return go_plain_v<T, R, MODE, false, 16>(a, nb, s);
    }
  }
  if constexpr (R <= kMaxPairRadius) {   // two bands per pass (Gaussian: tiles of one pass)
    const bool w32 = variant == kTileWide32x2 || variant == kTileLean32x2;
    if (w32 || variant == kTileWide16x2) {
      if (nb == 1)
        return w32 ? go_plain_v<T, R, MODE, GAUSS, 32, 2, true>(a, nb, s)
                   : go_plain_v<T, R, MODE, GAUSS, 16, 2, true>(a, nb, s);
      if constexpr (!GAUSS)
        return w32 ? go_plain_v<T, R, MODE, false, 32, 2>(a, nb, s)
                   : go_plain_v<T, R, MODE, false, 16, 2>(a, nb, s);
    }
  }
  return hipErrorInvalidValue;
}

// variant bit kTileGauss selects the Gaussian-weighted window.
template <typename T, int R, int MODE>
hipError_t go_plain(const IterArgs& a, int nb, int variant, hipStream_t s) {
  if (variant & kTileGauss) return go_plain_g<T, R, MODE, true>(a, nb, variant & ~kTileGauss, s);
  return go_plain_g<T, R, MODE, false>(a, nb, variant, s);
}

template <typename T, int R, int MODE, bool GAUSS, bool MASK>
hipError_t go_batch_m(const BatchLaunch& b, hipStream_t s) {
  constexpr int TW = kStripWidth;
  using C = Cfg<R, TW>;
  constexpr size_t kLds = field_handed<T, R, MODE, GAUSS, false>() ? C::HANDED_LDS_BYTES : C::LDS_BYTES;
  if constexpr (kLds > 65536) {
    static std::atomic<uint64_t> done{0};
    const hipError_t e =
        allow_lds(reinterpret_cast<const void*>(&lk_iter_batch<T, R, TW, MODE, GAUSS, MASK>), kLds, done);
    if (e != hipSuccess) return e;
  }
  if (b.prime) {
    hipFuncAttributes attr;
    return hipFuncGetAttributes(
        &attr, reinterpret_cast<const void*>(&lk_iter_batch<T, R, TW, MODE, GAUSS, MASK>));
  }
  hipLaunchKernelGGL((lk_iter_batch<T, R, TW, MODE, GAUSS, MASK>), dim3(b.grid),
                     dim3(C::NT), kLds, s, b.args, b.tiles, b.ntiles);
  return hipGetLastError();
}

template <typename T, int R, int MODE, bool GAUSS>
hipError_t go_batch_v(const BatchLaunch& b, hipStream_t s) {
  return b.masked ? go_batch_m<T, R, MODE, GAUSS, true>(b, s)
                  : go_batch_m<T, R, MODE, GAUSS, false>(b, s);
}

// b.variant: OF_TILE_NARROW, _WIDE or _WIDE_LEAN, plus kTileGauss for the Gaussian window.
template <typename T, int R, int MODE>
hipError_t go_batch(const BatchLaunch& b, hipStream_t s) {
  switch (b.variant) {
    case kTileNarrow:
    case kTileWide:
    case kTileWideLean: return go_batch_v<T, R, MODE, false>(b, s);
    case kTileNarrow | kTileGauss:
    case kTileWide | kTileGauss:
    case kTileWideLean | kTileGauss: return go_batch_v<T, R, MODE, true>(b, s);
  }
  return hipErrorInvalidValue;
}

template <typename T, int R>
hipError_t go_r(const IterArgs* a, const BatchLaunch* b, int mode, int nb, int variant,
                hipStream_t s) {
  switch (mode) {
    case kFlowSame:
      return a ? go_plain<T, R, kFlowSame>(*a, nb, variant, s) : go_batch<T, R, kFlowSame>(*b, s);
    case kFlowCoarse:
      return a ? go_plain<T, R, kFlowCoarse>(*a, nb, variant, s) : go_batch<T, R, kFlowCoarse>(*b, s);
    case kFlowZero:
      return a ? go_plain<T, R, kFlowZero>(*a, nb, variant, s) : go_batch<T, R, kFlowZero>(*b, s);
  }
  return hipErrorInvalidValue;
}

// Plain launch (a != nullptr; tile height N*nb, tile variant `variant`) or batched launch
// (b != nullptr; its own variant) of a radius in [LO, HI].
template <typename T, int LO, int HI>
hipError_t launch_iter_t(const IterArgs* a, const BatchLaunch* b, int R, int mode, int nb,
                         int variant, hipStream_t s) {
  if (R == LO) return go_r<T, LO>(a, b, mode, nb, variant, s);
  if constexpr (LO < HI) return launch_iter_t<T, LO + 1, HI>(a, b, R, mode, nb, variant, s);
  return hipErrorInvalidValue;
}

}  // namespace

}  // namespace ofmi
