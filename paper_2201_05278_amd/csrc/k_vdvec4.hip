// Variable-density vector tiles of radius 7.
#include "stencil_vdvec.h"

namespace sw {

SW_VDVEC_RADIUS(7)

}  // namespace sw
