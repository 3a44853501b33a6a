// Vector-tile stencils: single precision, radii 8 .. 10.
#include "stencil_vec.h"

namespace sw {

SW_VEC_RADIUS(float, 8)
SW_VEC_BATCH(8)
SW_VEC_RADIUS(float, 9)
SW_VEC_BATCH(9)
SW_VEC_RADIUS(float, 10)
SW_VEC_BATCH(10)

}  // namespace sw
