// FP64 resident-step kernels: every operation rounds as written, as in the FP64 step kernels.
#include "hexsv_resident.h"

namespace hexsv {
HEXSV_INSTANTIATE_RESIDENT(double)
}
