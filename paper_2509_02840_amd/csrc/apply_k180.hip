// apply_k180.hip -- the staged applier for blocks of 180 chains (K0 = 12, NW = 15).
#include "apply_kernel.h"

// Spilled registers: 43 (G = 4), 24 (G = 3), both of 168 VGPRs, and 5 (G = 1,
// of 128); the reloads are outside of the rotations, once a chunk or a block.

namespace bdu {

hipError_t launch_apply_k180(HandleDev *const *hs, int count, int panels, int G, Gate gate, hipStream_t st)
{
    if (G == 4) return launch_t<12, 15, 1, 4, 1, 6, 3>(hs, count, panels, gate, st);
    if (G == 3) return launch_t<12, 15, 1, 3, 2, 4, 3>(hs, count, panels, gate, st);
    return launch_t<12, 15, 1, 1, 1, 6, 4>(hs, count, panels, gate, st);
}

}  // namespace bdu
