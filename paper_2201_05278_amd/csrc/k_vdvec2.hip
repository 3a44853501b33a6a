// Variable-density vector tiles of radius 4.
#include "stencil_vdvec.h"

namespace sw {

SW_VDVEC_RADIUS(4)

}  // namespace sw
