// The prompt product with its SiLU epilogue (ff1_kernel.h).
#include "ff1_kernel.h"

namespace griffin {
FF1_TILES_OF(GRIFFIN_ACT_SILU)
}  // namespace griffin
