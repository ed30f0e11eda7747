// Generated by gen_instances.py: BF16 inputs, 128x128 tiles, A k-contiguous,
// B n-contiguous; single and grouped launches, Stream-K and data-parallel entries.
#include "sk_dispatch.hpp"

namespace sk {
KernelEntry pick_bf16_128_kn(const KernelKey &k) {
    return k.grouped ? entry<Dt::BF16, 128, 128, true, false, true>(k)
                     : entry<Dt::BF16, 128, 128, true, false, false>(k);
}
}  // namespace sk
