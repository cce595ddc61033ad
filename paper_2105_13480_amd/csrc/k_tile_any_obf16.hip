// conv_tile instantiations: 1x1 and any stencil, bf16 Out.
#include "tile_kernel.h"

namespace cnnlib {
CNN_TILE_LAUNCHER(launch_tile_any_obf16, CNN_TILE_ANY(CNN_CASET, 3220, CNN_BF16_OBF16))
}  // namespace cnnlib
