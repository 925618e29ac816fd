// Tile passes: two vectors (adjoint sweeps that carry psi and lambda).
#include "sv_pass.h"

namespace svk {

int launch_pass_c128_pair(const PassArgs& a, void* stream) { return run_pass<double, 13, 4, 2, 4, 1>(a, stream); }

int launch_pass_c64_pair(int T, int R, const PassArgs& a, void* stream) {
    if (T == 14) return run_pass<float, 14, 4, 2, 4, 4>(a, stream);  // 1024 threads
    if (R == 5) return run_pass<float, 13, 5, 2, 4, 2>(a, stream);
    return a.occ4 ? run_pass<float, 13, 4, 2, 4, 4>(a, stream) : run_pass<float, 13, 4, 2, 4, 1>(a, stream);
}

}  // namespace svk
