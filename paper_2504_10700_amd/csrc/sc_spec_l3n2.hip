// Generated kernels of models whose products have two factors, features up to l = 3 (see sc_spec_kernels.h).
#include "sc_spec_kernels.h"

namespace sc {
namespace {
#include "generated/sc_gen_l3n2_0e1o.inc"
#include "generated/sc_gen_l3n2_0e1o2e.inc"
#include "generated/sc_gen_l3n2_0e.inc"
#include "generated/sc_gen_l3n2_0e1o2e3o.inc"

const SpecEntry kEntries[] = {
    Entry<Gen_l3n2_0e1o, true>::make(),
    Entry<Gen_l3n2_0e1o2e, true>::make(),
    Entry<Gen_l3n2_0e, true>::make(),
    Entry<Gen_l3n2_0e1o2e3o, true>::make(),
};

}  // namespace

const SpecEntry* spec_entries_l3n2() { return kEntries; }
int spec_entries_l3n2_count() { return sizeof(kEntries) / sizeof(kEntries[0]); }

}  // namespace sc
