// Resident CG kernels for d = 1 (cgres.h).
#include "cgres.h"

namespace hub {
ResKernel res_kernel_d1(int level, bool whole, bool pcg) {
    return res_kernel_d<1>(level, whole, pcg);
}
}  // namespace hub
