// Host-side launchers of the HIP kernels (internal to the library).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

#include "common.h"
#include "device_once.h"
#include "tiles.h"

namespace ofmi {

enum class Elem : int { U8 = 0, F32 = 1, F16 = 2 };

inline size_t elem_bytes(Elem e) { return e == Elem::U8 ? 1 : (e == Elem::F16 ? 2 : 4); }

// One plane reduction job of a batched pyramid step.
struct ReduceJob {
  const void* in;
  void* out;
  int H, W, Ho, Wo;
};

// Output tile of the pyramid reduction kernels (columns x rows of the coarser level).
// 8-bit frames: a wave takes 128 columns, four waves the rows.
constexpr int kReduceTileW = 64, kReduceTileH = 16;
constexpr int kU8TileW = 128, kU8TileH = 32;
inline int reduce_blocks(Elem tin, int Ho, int Wo) {
  const int tw = tin == Elem::U8 ? kU8TileW : kReduceTileW, th = tin == Elem::U8 ? kU8TileH : kReduceTileH;
  return ((Wo + tw - 1) / tw) * ((Ho + th - 1) / th);
}

// Batched pyramid step over (job, output tile) work items.
hipError_t launch_reduce_batch(Elem tin, Elem tout, const ReduceJob* jobs, const int2* items,
                               int nitems, int grid, hipStream_t s);

// Mask pyramid step: out(i, j) = 1 if any of in(2i..2i+1, 2j..2j+1) (clamped) is nonzero.
hipError_t launch_mask_reduce(const uint8_t* in, int H, int W, uint8_t* out, int Ho, int Wo,
                              hipStream_t s);

// D = 2 or 3 successive pyramid reductions of up to two frames in one launch (levels f+1 ..
// f+D from level f; in[1] null for one frame): sizes H[0..D], W[0..D] of levels f .. f+D,
// out[frame][d-1] = level f+d.  Same bits as D launch_reduce calls.
struct ReduceChain {
  const void* in[2];
  void* out[2][3];
  int H[4], W[4];
  int D;
};
hipError_t launch_reduce_chain(Elem tin, Elem tout, const ReduceChain& c, hipStream_t s);

// One pyramid reduction of up to two frames of the same geometry (out = reduce(in)).
hipError_t launch_reduce(Elem tin, Elem tout, const void* in1, const void* in2, int H, int W,
                         void* out1, void* out2, int Ho, int Wo, hipStream_t s);

// Batched iteration launch: `grid` workgroups stride over `ntiles` work items (pair | tile
// flag << 16, tile x, first output row, output rows) with per-pair arguments args[pair]
// (device arrays); the flag (0 no unmasked pixel, 1 some masked pixels, 2 none) is read for
// pairs with a mask.
struct BatchLaunch {
  const IterArgs* args;
  const int4* tiles;
  int ntiles;
  int grid;
  int variant;   // TileVariant (narrow, wide, wide lean), plus kTileGauss for the Gaussian window
  bool masked;   // some pair of the launch has a mask (IterArgs::mask)
  // Load the kernel this launch would run on the current device, without launching it (a
  // kernel's first launch loads its code: milliseconds that a latency-bound caller primes
  // ahead instead of paying on a request).
  bool prime = false;
};

// Lets `kernel` take `bytes` of dynamic LDS (more than 64 KB: gfx950 has 160 KB per workgroup) on the
// current device; `done` belongs to the kernel.
inline hipError_t allow_lds(const void* kernel, size_t bytes, std::atomic<uint64_t>& done) {
  int dev = 0;
  const hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  return once_per_device(done, dev, hipSuccess, [&] {
    return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  });
}

// The iteration kernel's translation units: one per frame type and range of radii
// [kRadiusGroups[g], kRadiusGroups[g+1]).
constexpr int kRadiusGroups[] = {0, 4, 7, 9, 11, 13};
template <typename T, int GROUP>
hipError_t launch_iter_group(const IterArgs* a, const BatchLaunch* b, int R, int mode, int nb, int variant,
                             hipStream_t s);

// One fused Gauss-Newton iteration at one level (frames of element type `t`), tiles of height
// (2R+1)*nb, tile variant `variant` (TileVariant).
hipError_t launch_iter(Elem t, const IterArgs& a, int R, int nb, int variant, hipStream_t s);

// The same over a work list of many pairs' tiles at one (level, iteration) phase.
hipError_t launch_iter_batch(Elem t, const BatchLaunch& b, int R, int mode, hipStream_t s);

// Local equalisation of one frame or two of the same size (in2 null: one; uint8 or float32 in,
// float32 out).
hipError_t launch_normalize(Elem t, const void* in1, const void* in2, float* out1, float* out2, int H, int W,
                            int r, float eps, hipStream_t s);

// u = v = 0 over n elements (a fill kernel, safe under stream capture).
hipError_t launch_zero(float* u, float* v, size_t n, hipStream_t s);
// Zero flow over a work list of tiles (batch work items: pair in the low 16 bits of x, tile x,
// first row, rows; tw columns wide) into the output planes of args[pair] (tw divides 256).
hipError_t launch_zero_tiles(const IterArgs* args, const int4* tiles, int ntiles, int tw,
                             hipStream_t s);
// Loads the zero-tiles kernel's code on the current device (no launch).
hipError_t prime_zero_tiles();
// Copies of device memory, or of pinned host memory through its device mapping, by one kernel on
// stream s.
struct CopyJobs {
  static constexpr int kMost = 16;
  void* dst[kMost];
  const void* src[kMost];
  size_t bytes[kMost];
  int n = 0;
  bool full() const { return n == kMost; }
  void add(void* d, const void* s, size_t b) {
    dst[n] = d;
    src[n] = s;
    bytes[n++] = b;
  }
};
hipError_t launch_copies(const CopyJobs& jobs, hipStream_t s);
hipError_t launch_copy(void* dst, const void* src, size_t bytes, hipStream_t s);

// *c = 0 (a one-thread kernel, safe under stream capture).
hipError_t launch_zero_count(unsigned long long* c, hipStream_t s);

// *c = number of x[i] <= *thr over n elements (the threshold read on the device).
hipError_t launch_count_at_most(const float* x, long long n, const float* thr,
                                unsigned long long* c, hipStream_t s);

}  // namespace ofmi
