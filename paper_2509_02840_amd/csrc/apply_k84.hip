// apply_k84.hip -- the staged applier for blocks of 84 chains (K0 = 12, NW = 7).
#include "apply_kernel.h"

namespace bdu {

hipError_t launch_apply_k84(HandleDev *const *hs, int count, int panels, int G, int P, Gate gate, hipStream_t st)
{
    if (G == 4 && P == 1) return launch_t<12, 7, 1, 4, 1, 6, 3>(hs, count, panels, gate, st);
    if (G == 4 && P == 2) return launch_t<12, 7, 1, 4, 2, 6, 3>(hs, count, panels, gate, st);
    if (G == 1 && P == 2) return launch_t<12, 7, 1, 1, 2, 6, 4>(hs, count, panels, gate, st);
    return launch_t<12, 7, 1, 1, 1, 6, 4>(hs, count, panels, gate, st);
}

}  // namespace bdu
