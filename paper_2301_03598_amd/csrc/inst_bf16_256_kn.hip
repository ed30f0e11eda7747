// Generated by gen_instances.py: BF16 inputs, 256x256 tiles (8 waves), A k-contiguous,
// B n-contiguous; single and grouped launches, Stream-K and data-parallel entries.
#include "sk_dispatch.hpp"

namespace sk {
KernelEntry pick_bf16_256_kn(const KernelKey &k) {
    return k.grouped ? entry<Dt::BF16, 256, 256, true, false, true, 8>(k)
                     : entry<Dt::BF16, 256, 256, true, false, false, 8>(k);
}
}  // namespace sk
