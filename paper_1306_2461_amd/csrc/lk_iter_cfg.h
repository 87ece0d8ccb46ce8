// Workgroup shapes of the fused iteration kernel by window radius, strip width and bands per pass
// (shared by the kernel and by the host's choice of tiles).
#pragma once

#include <stddef.h>

namespace ofmi {

// Output columns of the strips of variants 0-2.
constexpr int kStripWidth = 64;

// Threads of a workgroup own K1 successive rows of one column of a band's warped frame (WC =
// TW + 2R + 2 columns), so a thread's column, clamps and LDS offsets are formed once per tile, its
// global offset is a per-thread constant added to a scalar row base, and P2 finds part of the
// warped values and fields it needs in the thread's own registers.
// A workgroup takes the fewest rows per thread that 768 threads allow (three waves per SIMD: two
// workgroups share a CU), rounded up to whole groups of four waves, one per SIMD: e.g. r = 8 on
// 64-column strips samples 17 rows of 82 positions per band, two rows per thread at 768 threads.
// From r = 9 on 64-column strips would take three rows per thread, which spills at the 80 registers
// of two workgroups per CU: one workgroup of up to 1024 there.
template <int R, int TW>
constexpr bool two_groups() {
  return !(R > 8 && TW > 32);
}
template <int R, int TW, int BB>
constexpr int group_threads() {
  const int N = 2 * R + 1, WC = TW + 2 * R + 2;
  const int rows = BB == 1 ? N : BB * N + 2;
  int k = 1;
  while ((rows + k - 1) / k * WC > (two_groups<R, TW>() ? 768 : 1024)) ++k;
  const int nt = ((rows + k - 1) / k * WC + 255) / 256 * 256;
  return nt < 5 * TW ? 5 * TW : nt;
}

template <int R, int TW_, int BB = 1>
struct Cfg {
  static constexpr int N = 2 * R + 1;                 // band height = window height
  static constexpr int NR = BB * N;                   // product rows per pass (BB bands)
  static constexpr int TW = TW_;                      // output columns per strip
  static constexpr int NT = group_threads<R, TW_, BB>();   // threads per workgroup
  static constexpr int PC = TW + 2 * R;               // product columns
  static constexpr int WC = PC + 2;                   // warped-frame columns
  static constexpr int HL = 8 + 2 * R;                // products read per horizontal segment
  static constexpr int HL4 = (HL + 3) / 4;            // ... in float4 units
  // Row pitches of the products and of the window sums: an odd number of 16-byte words, so the
  // 128-bit reads and writes of P3, whose lanes take successive rows, spread over all banks.
  static constexpr int PP = (TW + 4 * HL4 - 8 + 3) / 8 * 8 + 4;
  static constexpr int HP = TW + 4;
  static constexpr int WP = WC + 1;                   // warped-frame row pitch
  // Warped-frame rows held in LDS: the rows -1 .. NR of the pass.  With one band per pass the
  // last two are moved to the front for the next pass instead of being sampled again.
  static constexpr int P1_ROWS = BB == 1 ? N : NR + 2;          // rows sampled per pass
  static constexpr int P1_FIRST = BB == 1 ? 2 : 0;              // ... from this LDS row
  static constexpr int NSEG = TW / 8;
  static constexpr int K1 = (P1_ROWS + NT / WC - 1) / (NT / WC);  // rows per thread in P1, P2
  static constexpr int G = (P1_ROWS + K1 - 1) / K1;             // threads per column
  // (a thread's rows past the last one are sampled too, into LDS rows that nothing reads)
  static constexpr int W2ROWS = P1_FIRST + G * K1;
  static constexpr int K3 = (5 * NR * NSEG + NT - 1) / NT;      // P3 items per thread
  static constexpr int RG = NT / TW;                            // P5 rows per round
  static_assert(NT >= WC && G * WC <= NT && NT % TW == 0 && 2 * WP <= NT,
                "workgroup too small for the strip");
  // LDS: products [5][NR][PP], warped rows, window sums [5][NR][HP], and the field rows that P2
  // reads from another thread: u and v of each thread's last row, [G][WP] each.
  static constexpr size_t PR_FLOATS = 5 * (size_t)NR * PP;
  static constexpr size_t W2_FLOATS = ((size_t)W2ROWS * WP + 3) / 4 * 4;
  static constexpr size_t HS_FLOATS = 5 * (size_t)NR * HP;
  static constexpr size_t FC_FLOATS = 2 * (size_t)G * WP;
  static constexpr size_t LDS_BYTES = (PR_FLOATS + W2_FLOATS + HS_FLOATS + FC_FLOATS) * sizeof(float);
  // Launches that hand their field rows on to P5: u and v at the strip's columns and the RING sampled
  // rows that P5 still needs, row t of the tile at t % RING (r <= 8: 77.6 KB in all at most, still two
  // workgroups per CU).
  static constexpr int RING = NR + R + 1;
  static constexpr size_t HANDED_LDS_BYTES = LDS_BYTES + 2 * (size_t)RING * TW * sizeof(float);
};

// Wavefronts per SIMD the register allocation aims at: two workgroups share a CU (one's barriers and
// load rounds hide behind the other's arithmetic), which leaves 80 registers per thread at three
// waves per SIMD each (from r = 11 the window rows of P4 need more).
template <int R, int TW, int BB>
constexpr int waves_per_simd() {
  return two_groups<R, TW>() && R <= 10 ? 2 * ((Cfg<R, TW, BB>::NT + 255) / 256) : 1;
}

}  // namespace ofmi
