// Field-evaluation kernels (compiled as a unit of its own).
#include "llg_kernels.hpp"

namespace llg {
template <int PHASE, int PMAX>
const void* instance(bool wide) {
    constexpr int mode = MODE_FIELD_ROWS + PHASE;
    return wide ? reinterpret_cast<const void*>(llg_field<field_wide_ug(PHASE, PMAX), FIELD_WIDE_POL, mode, PMAX>)
                : reinterpret_cast<const void*>(llg_field<1, 0, mode, PMAX>);
}
// phase 0 = rows, 1 = columns, 2 = outputs; wide: the shapes for many tiles per CU
const void* field_kernel(int phase, bool wide, int PMAX) {
    if (phase == 0) return PMAX >= 512 ? instance<0, 512>(wide) : instance<0, 256>(wide);
    if (phase == 1) return PMAX >= 512 ? instance<1, 512>(wide) : instance<1, 256>(wide);
    return PMAX >= 512 ? instance<2, 512>(wide) : instance<2, 256>(wide);
}
}  // namespace llg
