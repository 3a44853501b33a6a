// Variable-density vector tiles of radius 1, 2, 3.
#include "stencil_vdvec.h"

namespace sw {

SW_VDVEC_RADIUS(1)
SW_VDVEC_RADIUS(2)
SW_VDVEC_RADIUS(3)

}  // namespace sw
