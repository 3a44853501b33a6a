// Variable-density vector tiles of radius 5, 6.
#include "stencil_vdvec.h"

namespace sw {

SW_VDVEC_RADIUS(5)
SW_VDVEC_RADIUS(6)

}  // namespace sw
