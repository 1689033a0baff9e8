// Resident CG kernels for d = 2 (cgres.h).
#include "cgres.h"

namespace hub {
ResKernel res_kernel_d2(int level, bool whole, bool pcg) {
    return res_kernel_d<2>(level, whole, pcg);
}
}  // namespace hub
