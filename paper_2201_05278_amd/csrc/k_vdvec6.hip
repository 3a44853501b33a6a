// Variable-density vector tiles of radius 9.
#include "stencil_vdvec.h"

namespace sw {

SW_VDVEC_RADIUS(9)

}  // namespace sw
