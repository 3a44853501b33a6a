// Variable-density vector tiles of radius 8.
#include "stencil_vdvec.h"

namespace sw {

SW_VDVEC_RADIUS(8)

}  // namespace sw
