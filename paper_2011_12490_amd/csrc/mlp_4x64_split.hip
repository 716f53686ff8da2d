// Grouped per-head MLP variants: 4 layers of 64, no skip, colour straight from [h; gamma(d)] (pos_freqs 6).
// float32 heads on the fp16 matrix units.
#include "mlp_kernel.h"

namespace derf {

const MlpVariant *mlp_split_4x64()
{
    return variant<Cfg<P_SPLIT, 64, 4, -1, 0, 6>>(mlp_f32_4x64());
}

}  // namespace derf
