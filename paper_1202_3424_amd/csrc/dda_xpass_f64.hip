// Passes 1 and 5 on FP64 grids (templates in dda_xpass.h).
#include "dda_xpass.h"

namespace dda {
DDA_INSTANTIATE_XPASSES(double)
}
