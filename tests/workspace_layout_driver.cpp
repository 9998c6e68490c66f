// Driver for the layout of the contraction's workspaces (linked with the library and run by tests/test_lib_host.py; CPU
// only): every array that a launch may fill to the bound in LaunchShape lies inside its room, in the caller's workspace and in the
// forward-only scratch.
#include <cstdio>

#include "../paper_2504_10700_amd/csrc/sc_internal.h"

namespace sc {
size_t spec_value_bytes(const sc_plan* plan);
}

int main() {
  struct Case { int channels, l_max, nu, elements, outs, dtype, flags; };
  const Case cases[] = {{128, 3, 3, 89, 2, SC_F32, 0}, {64, 3, 3, 5, 1, SC_F32, 0}, {256, 3, 3, 89, 3, SC_F32, 0}, {128, 2, 3, 89, 2, SC_F64, 0},
                        {192, 3, 3, 1024, 2, SC_BF16, 0}, {100, 3, 2, 11, 2, SC_F64, 0}, {128, 3, 3, 89, 2, SC_F32, SC_PLAN_FORCE_GENERIC}};
  int checked = 0;
  for (const Case& c : cases)
    for (const int tile : {0, 16}) {
      sc_config cfg{};
      cfg.struct_size = sizeof(cfg);
      cfg.num_channels = c.channels, cfg.l_max = c.l_max, cfg.nu_max = c.nu, cfg.num_elements = c.elements, cfg.num_out = c.outs;
      for (int o = 0; o < c.outs; ++o) cfg.out_l[o] = o, cfg.out_parity[o] = o % 2 ? -1 : 1;
      cfg.dtype = c.dtype, cfg.flags = SC_PLAN_HOST_ONLY | c.flags, cfg.tile_nodes = tile;
      sc_plan* plan = nullptr;
      if (sc_plan_create(&cfg, &plan) != SC_OK) return std::printf("plan: %s\n", sc_last_error()), 2;
      for (const int64_t n : {1, 7, 1024, 1025, 1300, 3072, 10000, 24576, 24577, 65536, 200000})
        for (const bool forward_only : {false, true}) {
          const sc::LaunchShape shape = sc::launch_shape(plan, n);
          char* const base = reinterpret_cast<char*>(uintptr_t(1) << 40);
          const sc::Workspace w = sc::carve_workspace(plan, n, shape, base, forward_only);
          const char* const end = base + w.bytes;
          const char* const tiles = reinterpret_cast<const char*>(w.tiles);
          const char* const after = plan->specialised ? static_cast<const char*>(w.wfold) : forward_only ? end : static_cast<const char*>(w.partial);
          const size_t value = plan->specialised ? sc::spec_value_bytes(plan) : c.dtype == SC_F64 ? 8 : 4;
          const size_t rows = value * shape.max_tiles * shape.chblocks * plan->S * sc::kLanes;
          const bool fits = !tiles || tiles + sizeof(sc::TileDesc) * shape.max_tiles <= after;
          const bool rows_fit = forward_only ? !w.partial : static_cast<char*>(w.partial) + rows <= end;
          if (!fits || !rows_fit || (!tiles && !(forward_only && plan->specialised))) {
            std::printf("channels %d l_max %d tile %d n %lld forward_only %d: tiles %s, rows %s\n", c.channels, c.l_max, tile,
                        static_cast<long long>(n), forward_only, fits ? "fit" : "do not fit", rows_fit ? "fit" : "do not fit");
            return 3;
          }
          ++checked;
        }
      sc_plan_destroy(plan);
    }
  std::printf("workspace layouts checked: %d\n", checked);
  return 0;
}
