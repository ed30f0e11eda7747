// Generated by gen_instances.py: F8 inputs, 128x128 tiles, A m-contiguous,
// B k-contiguous; single and grouped launches, Stream-K and data-parallel entries.
#include "sk_dispatch.hpp"

namespace sk {
KernelEntry pick_f8_128_nk(const KernelKey &k) {
    return k.grouped ? entry<Dt::F8, 128, 128, false, true, true>(k)
                     : entry<Dt::F8, 128, 128, false, true, false>(k);
}
}  // namespace sk
