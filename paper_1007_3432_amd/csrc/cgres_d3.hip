// Resident CG kernels for d = 3 (cgres.h).
#include "cgres.h"

namespace hub {
ResKernel res_kernel_d3(int level, bool whole, bool pcg) {
    return res_kernel_d<3>(level, whole, pcg);
}
}  // namespace hub
