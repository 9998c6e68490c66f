// Table of the generated shapes of the channelwise tensor product (see tp_spec.hip).
#pragma once
#include "tp_internal.h"

namespace tp {

struct SpecEntry {
  int l_Y, l_h, L_max, num_paths;
  const int (*ops)[3], (*flops)[3];   // per (edge, channel): forward, backward, second-order pass; of fp64 rows, of fp32 rows
  hipError_t (*forward)(const tp_plan* plan, const FwdArgs& a, hipStream_t stream);
  hipError_t (*backward)(const tp_plan* plan, const BwdArgs& a, hipStream_t stream);
  hipError_t (*double_backward)(const tp_plan* plan, const DblArgs& a, hipStream_t stream);
  int (*dY_parts)(const tp_plan* plan, int64_t n_in);   // of the backward
};

// The shapes with L_max = l_Y = 3 and sender features up to order 0 and 1, 2, 3, and those with
// L_max = l_Y = 1 and 2, each set compiled by a file of its own: entry i of the set.
SpecEntry spec_l3(int i);
SpecEntry spec_l3h2();
SpecEntry spec_l3h3();
SpecEntry spec_l12(int i);

}  // namespace tp
