// Generated by gen_instances.py: BF16 inputs, 64x64 tiles, A k-contiguous,
// B n-contiguous; single and grouped launches, Stream-K and data-parallel entries.
#include "sk_dispatch.hpp"

namespace sk {
KernelEntry pick_bf16_64_kn(const KernelKey &k) {
    return k.grouped ? entry<Dt::BF16, 64, 64, true, false, true>(k)
                     : entry<Dt::BF16, 64, 64, true, false, false>(k);
}
}  // namespace sk
