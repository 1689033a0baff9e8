// Prints the plan of the bare product for lattices that the row tiles take, or
// nearly take (csrc/sweep.h, on the host).
#include <cstdio>

#include "sweep.h"

namespace hub {
hub_status set_error(hub_status s, const char*, ...) { return s; }
}  // namespace hub

int main() {
    const int cases[][3] = {{2, 2, 2},   {2, 5, 7},   {2, 33, 60}, {2, 64, 145}, {2, 512, 4},
                            {2, 1024, 3}, {2, 1025, 3}, {3, 2, 2},  {3, 5, 20},   {3, 12, 50},
                            {3, 20, 96}, {3, 48, 48}, {3, 90, 6},  {3, 129, 2}};
    for (const auto& c : cases) {
        hub::Geom g{};
        g.d = c[0];
        g.nx = c[1];
        g.nt = c[2];
        g.vs = c[0] == 2 ? c[1] * c[1] : c[1] * c[1] * c[1];
        g.V = g.vs * c[2];
        const hub::SweepPlan p = hub::plan_sweep(g, true);
        std::printf("d%d_%dx%d kind %d level %d tiles %d x %d slices %d lds %d blocks %d\n", g.d,
                    g.nx, g.nt, p.kind, p.variant, p.tiles_y, p.tiles_z, p.tc, p.lds, p.grid);
    }
    return 0;
}
