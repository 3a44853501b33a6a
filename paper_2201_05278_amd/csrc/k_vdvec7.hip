// Variable-density vector tiles of radius 10.
#include "stencil_vdvec.h"

namespace sw {

SW_VDVEC_RADIUS(10)

}  // namespace sw
