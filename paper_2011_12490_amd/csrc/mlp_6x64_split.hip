// Grouped per-head MLP variants: 6 layers of 64, no skip, colour hidden layer of 32.
// float32 heads on the fp16 matrix units.
#include "mlp_kernel.h"

namespace derf {

const MlpVariant *mlp_split_6x64()
{
    return variant<Cfg<P_SPLIT, 64, 6, -1, 32, 10>>(mlp_f32_6x64());
}

}  // namespace derf
