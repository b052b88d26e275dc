// The plane kernel on FP32 grids (templates in dda_plane.h).
#include "dda_plane.h"

namespace dda {
DDA_INSTANTIATE_PLANE(float)
}
