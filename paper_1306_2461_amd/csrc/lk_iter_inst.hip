// Instantiations of the fused iteration kernel for one frame type and one range of radii, given on
// the compiler's command line (OFMI_ITER_ELEM: u8, f32 or f16; OFMI_ITER_GROUP: index into
// kRadiusGroups): the kernel's translation units, which compile in parallel.
#include "lk_iter_impl.h"

namespace ofmi {

namespace {
using elem_u8 = uint8_t;
using elem_f32 = float;
using elem_f16 = __half;
#define OFMI_CAT(a, b) a##b
#define OFMI_ELEM(e) OFMI_CAT(elem_, e)
}  // namespace

template <>
hipError_t launch_iter_group<OFMI_ELEM(OFMI_ITER_ELEM), OFMI_ITER_GROUP>(const IterArgs* a, const BatchLaunch* b,
                                                                         int R, int mode, int nb, int variant,
                                                                         hipStream_t s) {
  return launch_iter_t<OFMI_ELEM(OFMI_ITER_ELEM), kRadiusGroups[OFMI_ITER_GROUP],
                       kRadiusGroups[OFMI_ITER_GROUP + 1] - 1>(a, b, R, mode, nb, variant, s);
}

}  // namespace ofmi
