// Persistent strip solve of 16/8-bit dense graphs, ballistic variant.
#include "strip_persistent_kernel.h"

namespace qh {

void launch_strip_plain(const BandLaunch &bl, const BandPersistArgs &a, hipStream_t st) {
    launch_strip_disc<false>(bl, a, st);
}

}  // namespace qh
