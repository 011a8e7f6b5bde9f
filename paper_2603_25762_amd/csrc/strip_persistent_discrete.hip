// Persistent strip solve of 16/8-bit dense graphs, discrete variant.
#include "strip_persistent_kernel.h"

namespace qh {

void launch_strip_discrete(const BandLaunch &bl, const BandPersistArgs &a, hipStream_t st) {
    launch_strip_disc<true>(bl, a, st);
}

}  // namespace qh
