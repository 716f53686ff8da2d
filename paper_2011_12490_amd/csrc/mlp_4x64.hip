// Grouped per-head MLP variants: 4 layers of 64, no skip, colour straight from [h; gamma(d)] (pos_freqs 6).
#include "mlp_kernel.h"

namespace derf {

const MlpVariant *mlp_variant_4x64(bool bf16)
{
    return bf16 ? variant<Cfg<P_BF16, 64, 4, -1, 0, 6>>() : mlp_split_4x64();
}

}  // namespace derf
