// Tile passes: complex128, one vector.
#include "sv_pass.h"

namespace svk {

int launch_pass_c128(int T, const PassArgs& a, void* stream) {
    // 14-bit tiles: 512 threads, one workgroup per CU (128 KiB half-tile exchanges)
    if (T == 14) return run_pass<double, 14, 5, 1, 8, 2>(a, stream);
    return run_pass<double, 13, 5, 1, 8, 2>(a, stream);
}

}  // namespace svk
