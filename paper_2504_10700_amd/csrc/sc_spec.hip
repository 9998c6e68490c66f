// The generated straight-line kernels as a table (kernels and skeleton: sc_spec_kernels.h), plan
// look-up and dispatch, and the programs of the largest configurations.  The other files
// (sc_spec_l2.hip, sc_spec_l3n2.hip) hold further programs; they are separate for build time.
#include "sc_spec_kernels.h"

namespace sc {
namespace {
#include "generated/sc_gen_l3n3_0e1o.inc"
#include "generated/sc_gen_l3n3_0e1o2e.inc"
#include "generated/sc_gen_l3n3_0e1o2e3o.inc"
#include "generated/sc_gen_l1n2_0e.inc"
#include "generated/sc_gen_l3n3_0e.inc"

// In the order of the ids (id = position + 1); id 1 is the program of the fused linear + contraction kernel.
const SpecEntry kOwn[] = {
    Entry<Gen_l3n3_0e1o, false>::make(), Entry<Gen_l3n3_0e1o2e, false>::make(),
    Entry<Gen_l3n3_0e1o2e3o, false>::make(), Entry<Gen_l1n2_0e, false>::make(), Entry<Gen_l3n3_0e, false>::make(),
};
constexpr int kNumOwn = sizeof(kOwn) / sizeof(kOwn[0]);

const SpecEntry* entry_of(int id) {
  if (id < 1) return nullptr;
  int i = id - 1;
  if (i < kNumOwn) return &kOwn[i];
  i -= kNumOwn;
  if (i < spec_entries_l2_count()) return &spec_entries_l2()[i];
  i -= spec_entries_l2_count();
  return i < spec_entries_l3n2_count() ? &spec_entries_l3n2()[i] : nullptr;
}

// bytes of a value of the arithmetic type
size_t arith_bytes(const SpecEntry& e, int dtype) { return dtype == SC_F64 || (e.wide && dtype == SC_F32) ? 8 : 4; }

bool matches(const sc_plan* plan, const SpecEntry& e) {
  const sc_config& c = plan->cfg;
  if (c.l_max != e.l_max || c.nu_max != e.nu_max || c.num_out != e.num_out) return false;
  for (int o = 0; o < e.num_out; ++o)
    if (c.out_l[o] != e.out_l[o] || c.out_parity[o] != e.out_parity[o]) return false;
  if (e.wide && c.dtype == SC_BF16) return false;
  // the grouped kernels keep kS + kNlm columns per wave in LDS: 160 KB per compute unit at most
  // (the four-irrep kernel in fp64 would need 171 KB: the table-driven kernels serve that plan)
  const size_t lds = arith_bytes(e, c.dtype) * static_cast<size_t>(kSpecWaves) * (e.S + e.n_lm) * kLanes;
  if (lds > 160 * 1024) return false;
  // channel counts that are not a multiple of 64 leave lanes of the last channel block idle; a multiple
  // of four (eight for bfloat16 rows) keeps every row block 16-byte aligned
  return c.num_channels % (c.dtype == SC_BF16 ? 8 : 4) == 0 && static_cast<int>(plan->table.paths.size()) == e.P;
}

}  // namespace

int spec_lookup(const sc_plan* plan) {
  for (int id = 1; const SpecEntry* e = entry_of(id); ++id)
    if (matches(plan, *e)) return id;
  return 0;
}

int spec_basis_size(int id) {
  const SpecEntry* e = entry_of(id);
  return e ? e->S : 0;
}

bool spec_has_component_major(const sc_plan* plan) {
  const SpecEntry* e = entry_of(plan->specialised);
  return e && !e->wide && plan->cfg.dtype != SC_BF16;
}

bool spec_scratch_optional(const sc_plan* plan) {
  const SpecEntry* e = entry_of(plan->specialised);
  return e && e->wide;
}

void spec_op_counts(int id, int32_t ops[3], int32_t flops[3]) {
  const SpecEntry* e = entry_of(id);
  for (int i = 0; i < 3; ++i) {
    ops[i] = e ? e->ops[i] : 0;
    flops[i] = e ? e->flops[i] : 0;
  }
}

int spec_waves_per_tile() { return kSpecWaves; }

size_t spec_value_bytes(const sc_plan* plan) { return arith_bytes(*entry_of(plan->specialised), plan->cfg.dtype); }

size_t spec_folded_bytes(const sc_plan* plan) {
  const size_t chblocks = (plan->cfg.num_channels + kLanes - 1) / kLanes;   // whole 64-channel rows
  return static_cast<size_t>(plan->cfg.num_elements) * chblocks * kLanes * spec_basis_size(plan->specialised) *
         spec_value_bytes(plan);
}

// What it costs: every wave reads the external weights of its nodes' elements (P rows per node and channel block, from
// L2) instead of folded rows; what it saves: a launch and its fold of all elements.  With 89 elements, us per call:
//  - evaluation alone (prepare + forward / direct): fp32, 128 channels, 0e+1o (P = 86) 61 nodes 7.6 / 4.8, 2000 9.6 / 7.5, 4000
//    13.6 / 13.6; 0e+1o+2e (159) 2000 13.8 / 12.9, 3000 16.4 / 17.0; 0e (28) 10 000 21.0 / 16.6; fp64 0e+1o 2000 20.4 / 17.9, 3000
//    23.3 / 24.2; bfloat16 rows, 256 channels, 2000 12.7 / 11.6, 3000 14.8 / 15.1.  Limit: 2.8e6 bytes of W per lane.
//  - with the grouping, whose workgroups then count the whole batch each (forward + backward): 0e+1o 40 nodes 20.0 / 17.8, 1400
//    26.8 / 23.6, 2731 30.9 / 30.9; 0e+1o+2e 700 34.7 / 31.1, 1400 37.3 / 37.2, 2000 40.6 / 42.3; fp64 0e+1o 700 32.6 / 29.9, 2000
//    52.9 / 55.5; l_max = 2 fp64 (41) 1400 26.2 / 22.7, 2731 31.7 / 31.6; four outputs, 64 channels (231) 700 34.2 / 29.5,
//    2000 43.5 / 47.8.  Limits: 1.4e6 bytes, 2048 nodes, and a count matrix that fits beside the roles' LDS.
bool spec_direct_pays(const sc_plan* plan, int64_t n, const LaunchShape& shape, bool groups) {
  const double bytes = static_cast<double>(n) * shape.chblocks * entry_of(plan->specialised)->P * (plan->cfg.dtype == SC_F64 ? 8 : 4);
  if (groups) return n <= 2048 && bytes <= 1.4e6 && split_counts_bytes(plan, shape) <= 16 * 1024;
  return n <= 10000 && bytes <= 2.8e6;
}

// For a backward or second-order pass that finds no grouping: one launch instead of prepare and scatter, whose workgroups then count
// the whole batch each.  us, two launches (and the gap between them) / one, 89 elements: fp32, 128 channels, 0e+1o 60 nodes 8.0 / 6.5, 500 8.9 / 6.5,
// 2000 10.2 / 7.6; 0e+1o+2e 1000 9.8 / 7.1; fp64 60 10.3 / 7.4, 2000 10.8 / 8.7.
bool spec_group_direct_pays(const sc_plan* plan, int64_t n, const LaunchShape& shape) {
  return n <= 2048 && split_counts_bytes(plan, shape) <= 16 * 1024;
}

hipError_t launch_spec_group(const sc_plan* plan, int64_t n, const int32_t* z, const void* W, const Workspace& ws,
                             const LaunchShape& shape, bool table_only, bool fold, hipStream_t stream) {
  return launch_spec_forward(plan, n, nullptr, z, W, nullptr, ws, shape, table_only ? 2 : 1, false, false, true, fold, stream);
}

hipError_t launch_spec_prepare(const sc_plan* plan, int64_t n, const int32_t* z, const void* W, const Workspace& ws,
                               const LaunchShape& shape, bool count, bool fold, bool window_order, hipStream_t stream) {
  return entry_of(plan->specialised)->prepare(plan, n, z, W, ws, shape, count, fold, window_order, stream);
}

hipError_t launch_spec_scatter(const sc_plan* plan, int64_t n, const int32_t* z, const Workspace& ws,
                               const LaunchShape& shape, bool table_only, hipStream_t stream) {
  if (!ws.tiles) return hipErrorInvalidValue;   // a workspace without room for tiles is never grouped
  const int scatter_wgs = table_only ? 0 : shape.split_waves / kGroupWavesPerWG;
  hipLaunchKernelGGL(spec_scatter_kernel, dim3(scatter_wgs + 1), dim3(kSpecThreads),
                     split_group_lds_bytes(plan->cfg.num_elements), stream, group_args(plan, n, z, ws, shape), scatter_wgs);
  return hipGetLastError();
}

hipError_t launch_spec_forward(const sc_plan* plan, int64_t n, const void* A, const int32_t* z, const void* W, void* B,
                               const Workspace& ws, const LaunchShape& shape, int group, bool window_order,
                               bool component_major, bool direct, bool fold_table, hipStream_t stream) {
  if (((group == 1 || group == 2) && !ws.tiles) || (group == 3 && !direct)) return hipErrorInvalidValue;
  return entry_of(plan->specialised)->forward(plan, n, A, z, W, B, ws, shape, group, window_order && ws.wnode && ws.wkey,
                                              component_major, direct, fold_table, stream);
}

hipError_t launch_spec_backward(const sc_plan* plan, int64_t n, const void* A, const void* dB, void* dA,
                                const Workspace& ws, const LaunchShape& shape, bool component_major,
                                hipStream_t stream) {
  return entry_of(plan->specialised)->backward(plan, n, A, dB, dA, ws, shape, component_major, stream);
}

hipError_t launch_spec_double_backward(const sc_plan* plan, int64_t, const void* A, const void* W, const void* dB,
                                       const void* H, void* ddB, void* dA2, const Workspace& ws,
                                       const LaunchShape& shape, bool component_major, hipStream_t stream) {
  return entry_of(plan->specialised)->double_backward(plan, A, W, dB, H, ddB, dA2, ws, shape, component_major, stream);
}

hipError_t launch_spec_finalize(const sc_plan* plan, void* dW, const Workspace& ws, const LaunchShape& shape,
                                hipStream_t stream) {
  return entry_of(plan->specialised)->finalize(plan, dW, ws, shape, stream);
}

}  // namespace sc
