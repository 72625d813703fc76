// K-a: the factors of wide windowed bins, a file of its own because its loops
// must not hold their FP64 coefficients (52 registers) across iterations: the
// kernel would spill at its four waves per SIMD.  The others lose up to 4% by
// that (bins of 1200 x 8 samples: 870 -> 902 us).
#define PSF_DECORR_WINDOW
#include "k_decorr_bin.hpp"

namespace psf {

template __global__ void k_decorr<false, kWideWindow>(ObsView, double, double, double, double, const double*, int64_t,
                                                     int64_t, const float2*, float2*, BinRec*, float2*, float2*);

}  // namespace psf
