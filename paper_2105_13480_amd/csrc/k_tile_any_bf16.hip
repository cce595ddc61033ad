// conv_tile instantiations: 1x1 and any stencil, fp32 Out.
#include "tile_kernel.h"

namespace cnnlib {
CNN_TILE_LAUNCHER(launch_tile_any_bf16, CNN_TILE_ANY(CNN_CASET, 3120, CNN_BF16))
}  // namespace cnnlib
