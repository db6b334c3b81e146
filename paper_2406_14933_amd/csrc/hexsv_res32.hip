// FP32 resident-step kernels (fused multiply-add allowed, as in the FP32 step kernels).
#include "hexsv_resident.h"

namespace hexsv {
HEXSV_INSTANTIATE_RESIDENT(float)
}
