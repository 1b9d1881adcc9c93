// Instantiations of the dense binary32 matrix-core kernels.
#include "k5_f32.hpp"

namespace ppc {

k5_conv_fn k5_conv_lookup(const K5Shape& s) {
#define PPC_K5(MT, NT, WK, WP) \
    if (s.mt == MT && s.nt == NT && s.wk == WK && s.wp == WP) return k5_conv_f32<MT, NT, WK, WP>;
    PPC_K5(2, 2, 1, 4) PPC_K5(2, 2, 2, 2) PPC_K5(2, 2, 4, 1) PPC_K5(2, 2, 8, 1)
    PPC_K5(1, 2, 1, 4) PPC_K5(1, 2, 4, 1) PPC_K5(1, 2, 8, 1)
    PPC_K5(1, 1, 4, 1) PPC_K5(1, 1, 8, 1) PPC_K5(1, 1, 16, 1)
#undef PPC_K5
    return nullptr;
}

k5_list_fn k5_list_lookup(const K5Shape& s) {
#define PPC_K5(NT, WK) \
    if (s.nt == NT && s.wk == WK) return k5_list_f32<NT, WK>;
    PPC_K5(2, 4) PPC_K5(2, 8) PPC_K5(1, 4) PPC_K5(1, 8) PPC_K5(1, 16)
#undef PPC_K5
    return nullptr;
}

}  // namespace ppc
