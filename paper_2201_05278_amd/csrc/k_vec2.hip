// Vector-tile stencils: single precision, radii 5 .. 7.
#include "stencil_vec.h"

namespace sw {

SW_VEC_RADIUS(float, 5)
SW_VEC_BATCH(5)
SW_VEC_RADIUS(float, 6)
SW_VEC_BATCH(6)
SW_VEC_RADIUS(float, 7)
SW_VEC_BATCH(7)

}  // namespace sw
