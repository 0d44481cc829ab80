// The prompt product on two shapes of tiles with its SiLU epilogue (ff1_kernel.h).
#include "ff1_kernel.h"

namespace griffin {
FF1_TWO_OF(GRIFFIN_ACT_SILU)
}  // namespace griffin
