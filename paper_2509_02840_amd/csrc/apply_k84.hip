// apply_k84.hip -- the staged applier for blocks of 84 chains (K0 = 12, NW = 7).
#include "apply_kernel.h"

// For the compiler's three wavefronts per SIMD (168 VGPRs) the G = 4 instances
// spill 42 and 45 registers; the reloads are outside of the rotations, once a
// chunk or a block.  The G = 1 instances take 126 and 119 VGPRs of 128.

namespace bdu {

hipError_t launch_apply_k84(HandleDev *const *hs, int count, int panels, int G, int P, Gate gate, hipStream_t st)
{
    if (G == 4 && P == 1) return launch_t<12, 7, 1, 4, 1, 6, 3>(hs, count, panels, gate, st);
    if (G == 4 && P == 2) return launch_t<12, 7, 1, 4, 2, 6, 3>(hs, count, panels, gate, st);
    if (G == 1 && P == 2) return launch_t<12, 7, 1, 1, 2, 6, 4>(hs, count, panels, gate, st);
    return launch_t<12, 7, 1, 1, 1, 6, 4>(hs, count, panels, gate, st);
}

}  // namespace bdu
