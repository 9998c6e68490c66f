// Specialised kernels of the channelwise tensor product: hand-written memory / scheduling
// skeleton around generated straight-line arithmetic (csrc/generated/tp_gen_*.inc, written by
// codegen/generate_tp.py).
//
// Mapping (Algorithm 1 of arXiv 2504.10700 is independent per edge and channel; the pooling
// sums the edges of a receiver):
//   lane      = channel (64 consecutive channels per wave): a path's weights R[e][p][:] are one
//               contiguous 256 B row per wave, the sender's features h[j][k][:] 16 B per lane
//   workgroup = forward: one (receiving atom, 64-channel block); each of its four waves (two,
//               waves_per_unit) walks every fourth edge the atom receives and keeps its sum in registers.  Backward: one (sending
//               atom, one or two 64-channel blocks: BackwardBlocks); a wave walks every fourth (eighth) edge the atom sends, keeps the
//               atom's h rows and its dh sums in registers and gathers the receivers' dA rows; per edge
//               it writes dR and its blocks' share of dY, which is dY where the workgroup has all blocks.  Either way the waves' sums meet in
//               LDS: no atomics, a fixed summation order, one store per atom.  The second-order pass
//               walks by receiver (ddA in registers) and writes every edge's share of d2h, which a
//               small kernel sums per sender.
//   Y[e][:]   is the same for all lanes: it is read with scalar loads and enters the
//               arithmetic as scalar operands
// The next edge's rows are requested before the current edge is evaluated (two register sets
// in turn); the sender index of the edge after next is read one step further ahead so that
// no row load waits for an index.
//
// Generated shapes: L_max = l_Y in 1..3 with every l_h <= L_max, any number of channels; the kernels are in
// tp_spec_kernels.h, the instances of the other shapes in tp_spec_*.hip.
#include "tp_spec_kernels.h"

namespace tp {
namespace {

#include "generated/tp_gen_y3h0o3.inc"
#include "generated/tp_gen_y3h1o3.inc"

}  // namespace

SpecEntry spec_l3(int i) { return i == 0 ? GeneratedShape<GenTP_y3h0o3>::entry() : GeneratedShape<GenTP_y3h1o3>::entry(); }

namespace {

// Generated shapes by id: 1, 2, ..., kShapes.
constexpr int kShapes = 9;
const SpecEntry& entry(int id) {
  static const SpecEntry table[kShapes] = {spec_l3(0),  spec_l3(1),  spec_l3h2(), spec_l3h3(), spec_l12(0),
                                           spec_l12(1), spec_l12(2), spec_l12(3), spec_l12(4)};
  return table[id - 1];
}

}  // namespace

int spec_lookup(const tp_plan* plan) {
  const tp_config& c = plan->cfg;
  for (int id = 1; id <= kShapes; ++id) {
    const SpecEntry& e = entry(id);
    if (e.l_Y == c.l_Y && e.l_h == c.l_h && e.L_max == c.L_max && e.num_paths == static_cast<int>(plan->paths.size())) return id;
  }
  return 0;
}

int spec_dY_parts(const tp_plan* plan, int64_t n_in) { return entry(plan->specialised).dY_parts(plan, n_in); }

void spec_op_counts(const tp_plan* plan, int32_t ops[3], int32_t flops[3]) {
  const int id = plan->specialised, f32 = plan->cfg.dtype == SC_F32;
  for (int i = 0; i < 3; ++i) {
    ops[i] = id ? entry(id).ops[f32][i] : 0;
    flops[i] = id ? entry(id).flops[f32][i] : 0;
  }
}

hipError_t launch_spec_forward(const tp_plan* plan, const FwdArgs& a, hipStream_t stream) {
  return entry(plan->specialised).forward(plan, a, stream);
}
hipError_t launch_spec_backward(const tp_plan* plan, const BwdArgs& a, hipStream_t stream) {
  return entry(plan->specialised).backward(plan, a, stream);
}
hipError_t launch_spec_double_backward(const tp_plan* plan, const DblArgs& a, hipStream_t stream) {
  return entry(plan->specialised).double_backward(plan, a, stream);
}

}  // namespace tp
