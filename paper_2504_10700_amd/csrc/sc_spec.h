// Generated straight-line kernels for selected configurations (see sc_spec.hip).
#pragma once
#include "sc_internal.h"

namespace sc {

// One generated program and its launches.  wide: fp32 plans compute in fp64 (rows and weights stay
// fp32); bfloat16 rows and the component-major layout are not served.
struct SpecEntry {
  int l_max, nu_max, num_out, out_l[SC_MAX_OUT], out_parity[SC_MAX_OUT];
  int n_lm, P, S;
  bool wide;
  int32_t ops[3], flops[3];
  hipError_t (*prepare)(const sc_plan*, int64_t n, const int32_t* z, const void* W, const Workspace&, const LaunchShape&,
                        bool count, bool fold, bool window_order, hipStream_t);
  hipError_t (*forward)(const sc_plan*, int64_t n, const void* A, const int32_t* z, const void* W, void* B, const Workspace&,
                        const LaunchShape&, int group, bool window_order, bool component_major, bool direct, bool fold_table, hipStream_t);
  hipError_t (*backward)(const sc_plan*, int64_t n, const void* A, const void* dB, void* dA, const Workspace&,
                         const LaunchShape&, bool component_major, hipStream_t);
  hipError_t (*double_backward)(const sc_plan*, const void* A, const void* W, const void* dB, const void* H, void* ddB,
                                void* dA2, const Workspace&, const LaunchShape&, bool component_major, hipStream_t);
  hipError_t (*finalize)(const sc_plan*, void* dW, const Workspace&, const LaunchShape&, hipStream_t);
};
const SpecEntry* spec_entries_l2();
int spec_entries_l2_count();
const SpecEntry* spec_entries_l3n2();
int spec_entries_l3n2_count();

// Returns the id (> 0) of the generated kernel that serves this plan, 0 if none.
int spec_lookup(const sc_plan* plan);
// Size of the internal (reduced) path basis of a generated kernel.
int spec_basis_size(int id);
// VALU instructions (ops) and flops per (node, channel) of forward, backward, second-order pass.
void spec_op_counts(int id, int32_t ops[3], int32_t flops[3]);
// Waves per workgroup (= per tile) of the generated kernels.
int spec_waves_per_tile();

// Does the plan's generated kernel serve SC_COMPONENT_MAJOR?
bool spec_has_component_major(const sc_plan* plan);
// Plans that the table-driven kernels served before: a forward whose scratch has no room for the folded
// table runs with weights folded by the waves (launch_spec_forward, direct).
bool spec_scratch_optional(const sc_plan* plan);
// Bytes of a folded weight and of a per-tile dW value (the plan must have a generated kernel).
size_t spec_value_bytes(const sc_plan* plan);

// Bytes of the count matrix that the grouping roles of a direct forward keep in LDS.
inline size_t split_counts_bytes(const sc_plan* plan, const LaunchShape& shape) {
  return sizeof(int32_t) * static_cast<size_t>(shape.split_waves) * plan->cfg.num_elements;
}

// Does a forward without a prepare launch (direct) cost less than one with it?  groups: its launch also groups.
bool spec_direct_pays(const sc_plan* plan, int64_t n, const LaunchShape& shape, bool groups);

// Bytes of the folded-weight table wf[element][channel][stride] of a generated kernel.
size_t spec_folded_bytes(const sc_plan* plan);

// Launch 1: folds W into ws.wfold (fold) and / or counts the elements of z (count: first half
// of the grouping).  Nothing is launched if both are false.
// window_order: workgroups of the launch also write ws.wnode / ws.wkey, the order in which the forward launch of
// the same call visits the nodes.
hipError_t launch_spec_prepare(const sc_plan* plan, int64_t n, const int32_t* z, const void* W, const Workspace& ws,
                               const LaunchShape& shape, bool count, bool fold, bool window_order, hipStream_t stream);
// Second half of the grouping as a launch of its own (after launch_spec_prepare with count);
// table_only: offsets and tile table without the permutation (the batch is already grouped).
hipError_t launch_spec_scatter(const sc_plan* plan, int64_t n, const int32_t* z, const Workspace& ws,
                               const LaunchShape& shape, bool table_only, hipStream_t stream);
// Grouping and, if wanted, the folded table by one launch: the roles of a direct forward without the forward.
bool spec_group_direct_pays(const sc_plan* plan, int64_t n, const LaunchShape& shape);
hipError_t launch_spec_group(const sc_plan* plan, int64_t n, const int32_t* z, const void* W, const Workspace& ws,
                             const LaunchShape& shape, bool table_only, bool fold, hipStream_t stream);
// Forward over the nodes in natural order from ws.wfold, or (direct) with weights that every wave
// folds from W by itself; group: the second half of the grouping
// rides in the same launch (0 no, 1 permutation + tile table, 2 tile table only; with direct also 3: no, and an element index
// outside the range takes the nearest element's weights instead of leaving its row of B); with direct its
// roles need no prepare launch, and fold_table: the launch also writes ws.wfold.
// component_major: the per-node tensors are laid out [node][component][channel]
// (SC_COMPONENT_MAJOR; plans whose rows are stored in the arithmetic type only).
// window_order: the kernel follows ws.wnode / ws.wkey, written by the prepare launch of the same call.
hipError_t launch_spec_forward(const sc_plan* plan, int64_t n, const void* A, const int32_t* z, const void* W, void* B,
                               const Workspace& ws, const LaunchShape& shape, int group, bool window_order,
                               bool component_major, bool direct, bool fold_table, hipStream_t stream);
// The grouped passes read ws.perm (null: the batch is already grouped, identity) and ws.tiles; the backward reads ws.wfold, the second-order pass folds W itself.
hipError_t launch_spec_backward(const sc_plan* plan, int64_t n, const void* A, const void* dB, void* dA,
                                const Workspace& ws, const LaunchShape& shape, bool component_major,
                                hipStream_t stream);
hipError_t launch_spec_double_backward(const sc_plan* plan, int64_t n, const void* A, const void* W, const void* dB,
                                       const void* H, void* ddB, void* dA2, const Workspace& ws,
                                       const LaunchShape& shape, bool component_major, hipStream_t stream);

// dW reduction over the tiles of every element and unfold to the external paths.
hipError_t launch_spec_finalize(const sc_plan* plan, void* dW, const Workspace& ws, const LaunchShape& shape,
                                hipStream_t stream);

}  // namespace sc
