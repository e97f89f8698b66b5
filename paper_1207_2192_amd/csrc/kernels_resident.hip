// Resident small-disk kernels (compiled as a unit of its own).
#include "llg_resident.hpp"

namespace llg {
// mode: MODE_DEMAG (field, right-hand side, energy), MODE_RK4 or MODE_HEUN
const void* resident_kernel(int mode, bool series) {
    if (mode == MODE_RK4)
        return series ? reinterpret_cast<const void*>(llg_resident<MODE_RK4, true>)
                      : reinterpret_cast<const void*>(llg_resident<MODE_RK4, false>);
    if (mode == MODE_HEUN)
        return series ? reinterpret_cast<const void*>(llg_resident<MODE_HEUN, true>)
                      : reinterpret_cast<const void*>(llg_resident<MODE_HEUN, false>);
    return reinterpret_cast<const void*>(llg_resident<MODE_DEMAG, false>);
}
}  // namespace llg
