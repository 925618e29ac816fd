// Tile passes: complex64, one vector.
#include "sv_pass.h"

namespace svk {

int launch_pass_c64(int T, const PassArgs& a, void* stream) {
    if (T == 14) return a.occ4 ? run_pass<float, 14, 5, 1, 8, 4>(a, stream) : run_pass<float, 14, 5, 1, 8, 2>(a, stream);
    return run_pass<float, 13, 5, 1, 8, 4>(a, stream);
}

}  // namespace svk
