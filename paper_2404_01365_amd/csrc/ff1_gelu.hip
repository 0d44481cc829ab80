// The prompt product with its GELU (tanh form) epilogue (ff1_kernel.h).
#include "ff1_kernel.h"

namespace griffin {
FF1_TILES_OF(GRIFFIN_ACT_GELU_TANH)
}  // namespace griffin
