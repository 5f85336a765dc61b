// Instantiation of the plane march for spin storage codec 1 (one translation unit per
// codec so that the library builds in parallel).
#include "plane_march.h"

namespace hsg {
template hipError_t launch_plane_s<1>(const MultiPlaneArgs &, int, int, bool, bool, bool, bool, unsigned, size_t,
                                       hipStream_t);
}  // namespace hsg
