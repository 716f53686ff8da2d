// Grouped per-head MLP variants: 8 layers of 128, skip at layer 5, colour hidden layer of 64.
// float32 heads on the fp16 matrix units.
#include "mlp_kernel.h"

namespace derf {

const MlpVariant *mlp_split_8x128()
{
    return variant<Cfg<P_SPLIT, 128, 8, 5, 64, 10>>(mlp_f32_8x128());
}

}  // namespace derf
