// Instances of the generated tensor-product kernels: L_max = l_Y = 3, sender features up to order 3.
#include "tp_spec_kernels.h"

namespace tp {
namespace {

#include "generated/tp_gen_y3h3o3.inc"

}  // namespace

SpecEntry spec_l3h3() { return GeneratedShape<GenTP_y3h3o3>::entry(); }

}  // namespace tp
