// Generated by gen_instances.py: F8 inputs, 256x256 tiles (8 waves), A k-contiguous,
// B k-contiguous; single and grouped launches, Stream-K and data-parallel entries.
#include "sk_dispatch.hpp"

namespace sk {
KernelEntry pick_f8_256_kk(const KernelKey &k) {
    return k.grouped ? entry<Dt::F8, 256, 256, true, true, true, 8>(k)
                     : entry<Dt::F8, 256, 256, true, true, false, 8>(k);
}
}  // namespace sk
