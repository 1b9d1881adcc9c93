// Instantiations of the binary32 3x3 kernel on the small matrix instruction.
#include "k6_f32_3x3.hpp"

namespace ppc {

k6_fn k6_lookup(int wk, bool bound, bool ragged) {
#define PPC_K6(WK)                                                                                       \
    if (wk == WK)                                                                                        \
        return bound ? (ragged ? k6_f32_3x3<true, true, WK> : k6_f32_3x3<true, false, WK>)              \
                     : (ragged ? k6_f32_3x3<false, true, WK> : k6_f32_3x3<false, false, WK>);
    PPC_K6(4) PPC_K6(8) PPC_K6(16)
#undef PPC_K6
    return nullptr;
}

}  // namespace ppc
