// Grouped per-head MLP variants: 6 layers of 64, no skip, colour hidden layer of 32.
// float32 heads on the fp32 matrix units.
#include "mlp_kernel.h"

namespace derf {

const MlpVariant *mlp_f32_6x64()
{
    return variant<Cfg<P_F32, 64, 6, -1, 32, 10>>();
}

}  // namespace derf
