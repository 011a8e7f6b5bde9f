// Persistent band solve, discrete variant (the coupling takes sgn(x_j)).
#include "band_persistent_kernel.h"

namespace qh {

void launch_band_discrete(const BandLaunch &bl, const BandPersistArgs &a, hipStream_t st) {
    launch_band_disc<true>(bl, a, st);
}

}  // namespace qh
