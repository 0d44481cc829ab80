// The prompt product with its ReLU epilogue (ff1_kernel.h).
#include "ff1_kernel.h"

namespace griffin {
FF1_TILES_OF(GRIFFIN_ACT_RELU)
}  // namespace griffin
