// Generated by gen_instances.py: BF16 inputs, 256x256 tiles (8 waves), A m-contiguous,
// B k-contiguous; single and grouped launches, Stream-K and data-parallel entries.
#include "sk_dispatch.hpp"

namespace sk {
KernelEntry pick_bf16_256_nk(const KernelKey &k) {
    return k.grouped ? entry<Dt::BF16, 256, 256, false, true, true, 8>(k)
                     : entry<Dt::BF16, 256, 256, false, true, false, 8>(k);
}
}  // namespace sk
