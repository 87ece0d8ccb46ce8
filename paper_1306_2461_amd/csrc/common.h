// Device helpers shared by the HIP kernels: element loads/stores per storage type, the
// clamped bilinear sample with split coordinates, the prolongation read and the 2x2 solve.
#pragma once

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ofmi {

constexpr float kTau = 1e-5f;   // relative singularity threshold of the 2x2 solve
constexpr int kMaxTaps = 25;    // window taps for the largest supported radius (2*12 + 1)

// Field source of an iteration: the previous iteration at the same level, the coarser
// level's result (prolongation u <- 2 bilinear(u_c, x/2, y/2)), or zero (coarsest level).
enum FlowMode : int { kFlowSame = 0, kFlowCoarse = 1, kFlowZero = 2 };

struct IterArgs {
  const void* I1;      // frame 1 at this level
  const void* I2;      // frame 2 at this level
  const float* uin;    // source field (same level or coarse level), unused for kFlowZero
  const float* vin;
  float* uout;         // destination field, this level
  float* vout;
  int H, W;            // level size
  int Hc, Wc;          // coarse level size (kFlowCoarse)
  int mode;            // FlowMode
  const uint8_t* mask; // this level's mask (nonzero = computed) or nullptr (no mask)
  const uint8_t* tiles; // plain launches with a mask: one flag per iteration tile: 0 = no
                        // unmasked output pixel, 1 = some masked pixels, 2 = no masked pixel
                        // (batched launches carry the flag in the work item)
  float taps[kMaxTaps]; // Gaussian-weighted window: separable taps g[0..2r] (unused for the box)
  // Recirculation-bubble count (eq. 3), final iteration of a plan only: when bcount is set,
  // the launch adds to *bcount the number of written u values <= *bthr.
  const float* bthr;
  unsigned long long* bcount;
};

// Element access by an unsigned 32-bit element index whose byte offset is formed in 32 bits
// (planes are below 4 GiB), through the global address space: with the base pointer in
// scalar registers this selects the scalar-base + 32-bit vector-offset global addressing
// form, also where the pointer itself was read from memory (work lists) and the compiler
// could not infer the address space (it would otherwise emit flat accesses).
template <typename T>
using global_t = __attribute__((address_space(1))) T;

template <typename T>
__device__ __forceinline__ const global_t<T>& at(const T* p, unsigned i) {
  return *((const global_t<T>*)((const global_t<char>*)p + i * (unsigned)sizeof(T)));
}
template <typename T>
__device__ __forceinline__ global_t<T>& at(T* p, unsigned i) {
  return *((global_t<T>*)((global_t<char>*)p + i * (unsigned)sizeof(T)));
}

__device__ __forceinline__ float ld(const uint8_t* p, unsigned i) { return (float)at(p, i); }
__device__ __forceinline__ float ld(const float* p, unsigned i) { return at(p, i); }
__device__ __forceinline__ float ld(const __half* p, unsigned i) {
  return __half2float(__ushort_as_half(at(reinterpret_cast<const unsigned short*>(p), i)));
}

__device__ __forceinline__ void st(float* p, unsigned i, float x) { at(p, i) = x; }
__device__ __forceinline__ void st(__half* p, unsigned i, float x) {
  at(reinterpret_cast<unsigned short*>(p), i) = __half_as_ushort(__float2half_rn(x));
}

// A plane read through a buffer descriptor: element offset = a per-thread offset + a scalar one
// (both below 2^30, as planes are), so a load whose row base is uniform costs no vector address
// arithmetic.  The descriptor holds the plane's size; accesses past it read zero.
template <typename T>
struct Plane {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ Plane(const T* p, int H, int W)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(p), 0, (int)((unsigned)(H * W) * (unsigned)sizeof(T)),
                                            0x00027000)) {}
  __device__ __forceinline__ float ld(unsigned off, int soff) const {
    if constexpr (sizeof(T) == 1)
      return (float)(unsigned)__builtin_amdgcn_raw_buffer_load_b8(r, (int)off, soff, 0);
    else if constexpr (sizeof(T) == 2)
      return __half2float(__ushort_as_half(__builtin_amdgcn_raw_buffer_load_b16(r, (int)(off * 2u), soff * 2, 0)));
    else
      return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)(off * 4u), soff * 4, 0));
  }
  // Store to a float plane (an offset past it: dropped).
  __device__ __forceinline__ void st(unsigned off, float x) const {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), r, (int)(off * 4u), 0, 0);
  }
};

// Row-major offset y * W + x with a 24-bit multiply: the full-rate v_mul_u32_u24 (the 32-bit
// integer multiply issues at a quarter of the rate).  Plans keep H and W below 2^24 and H * W
// below 2^30, so every product of an in-image row and a width fits.
__device__ __forceinline__ unsigned rowofs(int y, int W, int x) {
  return __umul24((unsigned)y, (unsigned)W) + (unsigned)x;
}

// i / D and i % D for a compile-time divisor D and 0 <= i < LIMIT: a 24-bit multiply by
// floor(2^20 / D) + 1 and a shift (instead of the quarter-rate 32-bit high multiply), checked
// exact for every i in range at compile time.
template <int D, int LIMIT>
struct ConstDiv {
  static constexpr unsigned S = 20, M = (1u << S) / D + 1;
  static constexpr bool exact() {
    for (unsigned i = 0; i < (unsigned)LIMIT; ++i)
      if (((i * M) >> S) != i / (unsigned)D) return false;
    return true;
  }
  static_assert(D > 0 && (unsigned long long)LIMIT * M < (1ull << 32) && exact(),
                "24-bit reciprocal multiply not exact over the index range");
  __device__ static __forceinline__ unsigned q(unsigned i) {
    if constexpr ((D & (D - 1)) == 0) return i / (unsigned)D;
    else return __umul24(i, M) >> S;
  }
  // (a signed 24-bit multiply by -D, so that the subtraction folds into one full-rate
  // multiply-add rather than a 32-bit one)
  __device__ static __forceinline__ unsigned r(unsigned i, unsigned q) {
    return i + (unsigned)__mul24((int)q, -D);
  }
};

// Integer base and fraction of the sample coordinate x + d along one axis of length n,
// clamped into [0, n-1].  Splitting d = floor(d) + frac keeps the coordinate exact in FP32
// (x + d itself would round to the spacing of |x|).  The sample is interior when its base
// lies in [0, n-2]; otherwise the base is clamped and the fraction is 0.  Returns the base;
// `step` is 1 for an interior sample (the second tap is the next element) and 0 otherwise.
__device__ __forceinline__ int split_coord(int x, float d, int n, float& frac, unsigned& step) {
  const float fd = floorf(d);
  const int bu = x + (int)fminf(fmaxf(fd, -1048576.f), 1048576.f);
  const bool inside = (unsigned)bu < (unsigned)(n - 1);
  frac = inside ? d - fd : 0.f;
  step = inside ? 1u : 0u;
  return min(max(bu, 0), n - 1);
}

// floor(d) as an integer, saturated, in one instruction (a NaN: 0).
__device__ __forceinline__ int floor_i(float d) {
  int i;
  asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(i) : "v"(d));
  return i;
}
// The same, a NaN as the lowest.
__device__ __forceinline__ int floor_sat(float d) {
  int i;
  asm("v_max_f32 %0, 0xcf000000, %1\n\tv_cvt_flr_i32_f32 %0, %0" : "=v"(i) : "v"(d));
  return i;
}
// x clamped to [0, hi] (hi uniform) in one instruction.
__device__ __forceinline__ int clamp_i(int x, int hi) {
  int r;
  asm("v_med3_i32 %0, %1, 0, %2" : "=v"(r) : "v"(x), "s"(hi));
  return r;
}

// I(x + u, y + v) by bilinear interpolation with clamped coordinates, in two steps, so that a thread
// issues the loads of all its samples before it waits for the first: issue() forms the coordinates and
// starts the four loads, value() interpolates.
template <typename T>
struct Sample {
  float z00, z01, z10, z11, a, b;
  __device__ __forceinline__ void issue(const Plane<T>& I, int H, int W, int x, int y, float u, float v) {
    unsigned sx, sy;
    const int xi = split_coord(x, u, W, a, sx);
    const int yi = split_coord(y, v, H, b, sy);
    const unsigned o00 = rowofs(yi, W, xi);
    const unsigned o10 = o00 + (sy ? (unsigned)W : 0u);
    z00 = I.ld(o00, 0);
    z01 = I.ld(o00 + sx, 0);
    z10 = I.ld(o10, 0);
    z11 = I.ld(o10 + sx, 0);
  }
  __device__ __forceinline__ float value() const {
    const float t = fmaf(a, z01 - z00, z00);
    const float s = fmaf(a, z11 - z10, z10);
    return fmaf(b, s - t, t);
  }
};

// 8-bit frames: the same value in fewer instructions.  Along x the base is clamped to [0, n-2], so
// the second tap always is the next pixel; the fraction measured from the clamped base, clamped to
// [0, 1], is 0 before the image and 1 past it, and differences of 8-bit values are exact, so that a
// fraction of 1 gives the second tap exactly (a frame one pixel wide keeps base and fraction 0: its
// second tap, 8 bits of any pixel or 0 past the plane, counts nothing).  Along y, where the row results
// are rounded, the displacement is clamped instead, to [-y, n-1-y], which leaves the fraction 0 at the
// last row, whose second row then counts nothing.  A NaN becomes the lowest displacement, as in
// split_coord.  (Each axis in the other's form: 24-pair mixed batch 1.5 % slower.)
template <>
struct Sample<uint8_t> {
  float z00, z01, z10, z11, a, b;
  __device__ __forceinline__ void issue(const Plane<uint8_t>& I, int H, int W, int x, int y, float u, float v) {
    const int xi = clamp_i(__builtin_elementwise_add_sat(x, floor_sat(u)), max(W - 2, 0));
    a = __builtin_amdgcn_fmed3f(u - (float)(xi - x), 0.f, W >= 2 ? 1.f : 0.f);
    const float ny = (float)-y;
    const float vc = __builtin_amdgcn_fmed3f(v, ny, (float)(H - 1) + ny);
    const int iv = floor_i(vc);
    b = vc - (float)iv;
    const unsigned o = rowofs(y + iv, W, xi);
    z00 = I.ld(o, 0);
    z01 = I.ld(o + 1u, 0);
    z10 = I.ld(o, W);
    z11 = I.ld(o + 1u, W);
  }
  __device__ __forceinline__ float value() const {
    const float t = fmaf(a, z01 - z00, z00);
    const float s = fmaf(a, z11 - z10, z10);
    return fmaf(b, s - t, t);
  }
};

// Field of a launch's source at K successive rows of one column, in two steps (loads, then the
// values).  The source is a compile-time parameter, so every kernel reads its field straight-line.
// EVEN: the first row, before any clamp, is an even image row.
template <int MODE, int K, bool EVEN = false>
struct FieldRows {   // the previous iteration at the same level
  float u[K], v[K];
  template <bool INTERIOR>
  __device__ __forceinline__ float2 at(int k, int, int) const { return make_float2(u[k], v[k]); }
};
template <int K>
struct FieldRows<kFlowZero, K, false> {
  template <bool INTERIOR>
  __device__ __forceinline__ float2 at(int, int, int) const { return make_float2(0.f, 0.f); }
};
// The coarser level's Hc x Wc field: 2 * bilinear(coarse, x/2, y/2) at in-image pixel (x, y), base
// floor(x/2), floor(y/2), fractions 0 or 1/2: every row reads its base row and the row after it, also
// where the fraction is 0 (a field that is not finite there must not depend on how rows are dealt to
// threads).  A pair of rows from an even one on shares two rows of the coarser level.  Of a pair from
// an odd row on, the second lies one further down and also takes the row after the pair's, which the
// next pair has loaded, or TAIL does for the last pair of an even K.
template <int K, bool EVEN>
struct FieldRows<kFlowCoarse, K, EVEN> {
  static constexpr int NP = (K + 1) / 2;
  static constexpr bool TAIL = K % 2 == 0 && !EVEN;
  float u00[NP], u01[NP], u10[NP], u11[NP], v00[NP], v01[NP], v10[NP], v11[NP], fa;
  float u20, u21, v20, v21;   // TAIL
  // Pair p, whose first row is y.  INTERIOR: the coarse row and column after every row's base exist.
  template <bool INTERIOR>
  __device__ __forceinline__ void issue(int p, const Plane<float>& U, const Plane<float>& V, int Hc, int Wc, int x,
                                        int y) {
    const int x0 = x >> 1, y0 = y >> 1;
    fa = (x & 1) ? 0.5f : 0.f;
    const bool tail = TAIL && p == NP - 1;
    if constexpr (INTERIOR) {
      const unsigned o = rowofs(y0, Wc, x0);
      u00[p] = U.ld(o, 0), u01[p] = U.ld(o + 1u, 0), u10[p] = U.ld(o, Wc), u11[p] = U.ld(o + 1u, Wc);
      v00[p] = V.ld(o, 0), v01[p] = V.ld(o + 1u, 0), v10[p] = V.ld(o, Wc), v11[p] = V.ld(o + 1u, Wc);
      if (tail) {
        u20 = U.ld(o, 2 * Wc), u21 = U.ld(o + 1u, 2 * Wc);
        v20 = V.ld(o, 2 * Wc), v21 = V.ld(o + 1u, 2 * Wc);
      }
      return;
    }
    const unsigned dx = x0 < Wc - 1 ? 1u : 0u;
    const unsigned dy = y0 < Hc - 1 ? (unsigned)Wc : 0u;
    const unsigned i00 = rowofs(y0, Wc, x0);
    const unsigned i01 = i00 + dx, i10 = i00 + dy, i11 = i00 + dy + dx;
    u00[p] = U.ld(i00, 0), u01[p] = U.ld(i01, 0), u10[p] = U.ld(i10, 0), u11[p] = U.ld(i11, 0);
    v00[p] = V.ld(i00, 0), v01[p] = V.ld(i01, 0), v10[p] = V.ld(i10, 0), v11[p] = V.ld(i11, 0);
    if (tail) {
      const unsigned i20 = rowofs(min(y0 + 2, Hc - 1), Wc, x0), i21 = i20 + dx;
      u20 = U.ld(i20, 0), u21 = U.ld(i21, 0), v20 = V.ld(i20, 0), v21 = V.ld(i21, 0);
    }
  }
  __device__ __forceinline__ float across(float z0, float z1) const { return fmaf(fa, z1 - z0, z0); }
  // Row k, at image row y; ya: the first row of its pair.
  template <bool INTERIOR>
  __device__ __forceinline__ float2 at(int k, int y, int ya) const {
    const int p = k / 2;
    const float fb = (EVEN && INTERIOR ? k % 2 == 1 : (y & 1) != 0) ? 0.5f : 0.f;
    float tu = across(u00[p], u01[p]), tv = across(v00[p], v01[p]);
    float su = across(u10[p], u11[p]), sv = across(v10[p], v11[p]);
    if (!EVEN && k % 2 == 1) {
      const bool lower = (y >> 1) != (ya >> 1);
      const int n = p + 1 < NP ? p + 1 : p;
      const float nu = p + 1 < NP ? across(u10[n], u11[n]) : across(u20, u21);
      const float nv = p + 1 < NP ? across(v10[n], v11[n]) : across(v20, v21);
      tu = lower ? su : tu, tv = lower ? sv : tv;
      su = lower ? nu : su, sv = lower ? nv : sv;
    }
    return make_float2(2.f * fmaf(fb, su - tu, tu), 2.f * fmaf(fb, sv - tv, tv));
  }
};

// 1/x from the hardware reciprocal (1 ulp) refined by one Newton-Raphson step.
__device__ __forceinline__ float recip(float x) {
  const float r = __builtin_amdgcn_rcpf(x);
  return fmaf(r, fmaf(-x, r, 1.0f), r);
}

// New estimate at a pixel from its window sums and its current estimate (u, v).
// D = AC - B^2 uses Kahan's FMA-compensated difference of products.
__device__ __forceinline__ void solve_update(float A, float B, float C, float sx, float sy,
                                             float u, float v, float& un, float& vn) {
  const float bx = fmaf(B, v, fmaf(A, u, sx));
  const float by = fmaf(C, v, fmaf(B, u, sy));
  const float T = A + C;
  const float w = B * B;
  const float e = fmaf(-B, B, w);
  const float D = fmaf(A, C, -w) + e;
  float du = 0.f, dv = 0.f;
  // D > tau T^2 > 0 keeps the reciprocals finite.
  if (D > kTau * (T * T)) {
    const float inv = recip(D);
    du = -(fmaf(C, bx, -B * by)) * inv;
    dv = -(fmaf(A, by, -B * bx)) * inv;
  } else if (T > 0.f) {
    const float inv = recip(T * T);
    du = -(fmaf(A, bx, B * by)) * inv;
    dv = -(fmaf(B, bx, C * by)) * inv;
  }
  un = u + du;
  vn = v + dv;
}

}  // namespace ofmi
