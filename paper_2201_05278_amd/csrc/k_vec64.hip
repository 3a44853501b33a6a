// Vector-tile stencils: double precision (forward only).
#include "stencil_vec.h"

namespace sw {

SW_VEC_RADIUS(double, 1)
SW_VEC_RADIUS(double, 2)
SW_VEC_RADIUS(double, 3)
SW_VEC_RADIUS(double, 4)
SW_VEC_RADIUS(double, 5)
SW_VEC_RADIUS(double, 6)
SW_VEC_RADIUS(double, 7)
SW_VEC_RADIUS(double, 8)
SW_VEC_RADIUS(double, 9)
SW_VEC_RADIUS(double, 10)

}  // namespace sw
