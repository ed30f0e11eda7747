// Generated by gen_instances.py: F8 inputs, 64x64 tiles, A k-contiguous,
// B k-contiguous; single and grouped launches, Stream-K and data-parallel entries.
#include "sk_dispatch.hpp"

namespace sk {
KernelEntry pick_f8_64_kk(const KernelKey &k) {
    return k.grouped ? entry<Dt::F8, 64, 64, true, true, true>(k)
                     : entry<Dt::F8, 64, 64, true, true, false>(k);
}
}  // namespace sk
