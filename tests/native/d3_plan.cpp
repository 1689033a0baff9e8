// Prints the tile of the bare d = 3 product for nx, nt and precision given as
// arguments, three at a time (csrc/sweep.h, on the host).
#include <cstdio>
#include <cstdlib>

#include "sweep.h"

namespace hub {
hub_status set_error(hub_status s, const char*, ...) { return s; }
}  // namespace hub

int main(int argc, char** argv) {
    for (int k = 1; k + 2 < argc; k += 3) {
        hub::Geom g{};
        g.d = 3;
        g.nx = std::atoi(argv[k]);
        g.nt = std::atoi(argv[k + 1]);
        g.vs = g.nx * g.nx * g.nx;
        g.V = g.vs * g.nt;
        const hub::SweepPlan p = hub::plan_sweep(g, std::atoi(argv[k + 2]) == 64);
        const hub::D3Shape& s = hub::kD3Shapes[p.variant];
        std::printf("%dx%dx%d@%d\n", s.nx, s.ty, s.tz, s.block);
    }
    return 0;
}
