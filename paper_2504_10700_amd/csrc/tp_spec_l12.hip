// Instances of the generated tensor-product kernels: L_max = l_Y = 1 and 2.
#include "tp_spec_kernels.h"

namespace tp {
namespace {

#include "generated/tp_gen_y2h0o2.inc"
#include "generated/tp_gen_y2h1o2.inc"
#include "generated/tp_gen_y2h2o2.inc"
#include "generated/tp_gen_y1h0o1.inc"
#include "generated/tp_gen_y1h1o1.inc"

}  // namespace

SpecEntry spec_l12(int i) {
  switch (i) {
    case 0: return GeneratedShape<GenTP_y2h0o2>::entry();
    case 1: return GeneratedShape<GenTP_y2h1o2>::entry();
    case 2: return GeneratedShape<GenTP_y2h2o2>::entry();
    case 3: return GeneratedShape<GenTP_y1h0o1>::entry();
    default: return GeneratedShape<GenTP_y1h1o1>::entry();
  }
}

}  // namespace tp
