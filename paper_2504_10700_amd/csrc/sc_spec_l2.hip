// Generated kernels of models with features up to l = 2 (see sc_spec_kernels.h).
#include "sc_spec_kernels.h"

namespace sc {
namespace {
#include "generated/sc_gen_l2n3_0e1o.inc"
#include "generated/sc_gen_l2n3_0e1o2e.inc"
#include "generated/sc_gen_l2n3_0e.inc"
#include "generated/sc_gen_l2n2_0e1o.inc"
#include "generated/sc_gen_l2n2_0e1o2e.inc"
#include "generated/sc_gen_l2n2_0e.inc"

const SpecEntry kEntries[] = {
    Entry<Gen_l2n3_0e1o, true>::make(),
    Entry<Gen_l2n3_0e1o2e, true>::make(),
    Entry<Gen_l2n3_0e, true>::make(),
    Entry<Gen_l2n2_0e1o, true>::make(),
    Entry<Gen_l2n2_0e1o2e, true>::make(),
    Entry<Gen_l2n2_0e, true>::make(),
};

}  // namespace

const SpecEntry* spec_entries_l2() { return kEntries; }
int spec_entries_l2_count() { return sizeof(kEntries) / sizeof(kEntries[0]); }

}  // namespace sc
