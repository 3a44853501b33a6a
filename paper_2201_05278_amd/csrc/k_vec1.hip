// Vector-tile stencils: single precision, radii 1 .. 4.
#include "stencil_vec.h"

namespace sw {

SW_VEC_RADIUS(float, 1)
SW_VEC_BATCH(1)
SW_VEC_RADIUS(float, 2)
SW_VEC_BATCH(2)
SW_VEC_RADIUS(float, 3)
SW_VEC_BATCH(3)
SW_VEC_RADIUS(float, 4)
SW_VEC_BATCH(4)

}  // namespace sw
