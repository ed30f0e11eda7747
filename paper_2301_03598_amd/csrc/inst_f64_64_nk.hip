// Generated by gen_instances.py: F64 inputs, 64x64 tiles, A m-contiguous,
// B k-contiguous; single and grouped launches, Stream-K and data-parallel entries.
#include "sk_dispatch.hpp"

namespace sk {
KernelEntry pick_f64_64_nk(const KernelKey &k) {
    return k.grouped ? entry<Dt::F64, 64, 64, false, true, true>(k)
                     : entry<Dt::F64, 64, 64, false, true, false>(k);
}
}  // namespace sk
