// Registry part: F32 row-flattened configurations.
#include "variants.hpp"

namespace kl {

void add_variants_f32_rf(int kernel, std::vector<Variant> &out)
{
    KL_RF_SET(float, KL_F32, 4)
}

}  // namespace kl
