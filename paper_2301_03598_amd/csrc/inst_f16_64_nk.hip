// Generated by gen_instances.py: F16 inputs, 64x64 tiles, A m-contiguous,
// B k-contiguous; single and grouped launches, Stream-K and data-parallel entries.
#include "sk_dispatch.hpp"

namespace sk {
KernelEntry pick_f16_64_nk(const KernelKey &k) {
    return k.grouped ? entry<Dt::F16, 64, 64, false, true, true>(k)
                     : entry<Dt::F16, 64, 64, false, true, false>(k);
}
}  // namespace sk
