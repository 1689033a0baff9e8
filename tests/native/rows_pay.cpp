// Prints "rows" or "two" (passes) for lattices given as d nx nt use, where use is
// b64, b32 (bare product), f (Chebyshev factor), s64 or s32 (solver)
// (csrc/sweep.h, on the host).
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "sweep.h"

namespace hub {
hub_status set_error(hub_status s, const char*, ...) { return s; }
}  // namespace hub

int main(int argc, char** argv) {
    for (int k = 1; k + 3 < argc; k += 4) {
        hub::Geom g{};
        g.d = std::atoi(argv[k]);
        g.nx = std::atoi(argv[k + 1]);
        g.nt = std::atoi(argv[k + 2]);
        g.vs = 1;
        for (int j = 0; j < g.d; ++j) g.vs *= g.nx;
        g.V = g.vs * g.nt;
        const char* use = argv[k + 3];
        const hub::SweepPlan p = hub::plan_sweep(g, !std::strstr(use, "32"), use[0] == 's',
                                                 use[0] == 'f');
        std::puts(p.kind == hub::kSweepRows ? "rows" : p.fused ? "other" : "two");
    }
    return 0;
}
