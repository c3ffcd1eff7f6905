// Registry part: F64 row-flattened configurations.
#include "variants.hpp"

namespace kl {

void add_variants_f64_rf(int kernel, std::vector<Variant> &out)
{
    KL_RF_SET(double, KL_F64, 2)
}

}  // namespace kl
