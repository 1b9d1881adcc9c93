// Instantiations of the dense binary32 matrix-core kernels.
#include "k5_f32.hpp"

#include <algorithm>

namespace ppc {

namespace {

template <int MT, int WP, int WK>
void launch_conv(const K5ConvArgs& a, int blocks, hipStream_t stream) {
    constexpr int lds = std::max(3 * WK * MT * 3072, WK > 1 ? WP * WK * 4096 : 0);       // the ring; the shares' sums
    static_assert(lds <= 160 * 1024, "a compute unit's LDS");
    // the kernel may use more than the default 64 KB of dynamic LDS; set once per instantiation
    static const hipError_t lds_attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&k5_conv_f32<MT, WP, WK>), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    (void)lds_attr;
    hipLaunchKernelGGL((k5_conv_f32<MT, WP, WK>), dim3((unsigned)blocks), dim3(64 * WP * WK), lds, stream, a);
}

template <int MT, int NT, int WK, int WP>
void launch_whole(const K5ConvArgs& a, int blocks, hipStream_t stream) {
    hipLaunchKernelGGL((k5_whole_f32<MT, NT, WK, WP>), dim3((unsigned)blocks), dim3(64 * WK * WP), 0, stream, a);
}

}  // namespace

k5_conv_fn k5_conv_lookup(const K5ConvShape& s) {
#define PPC_K5(MT, WP, WK) \
    if (s.mt == MT && s.wp == WP && s.wk == WK) return launch_conv<MT, WP, WK>;
    PPC_K5(4, 4, 1) PPC_K5(4, 4, 2) PPC_K5(4, 2, 4) PPC_K5(2, 4, 1) PPC_K5(2, 2, 2) PPC_K5(2, 2, 4) PPC_K5(2, 1, 4) PPC_K5(1, 4, 1)
#undef PPC_K5
    return nullptr;
}

k5_conv_fn k5_whole_lookup(const K5Shape& s) {
#define PPC_K5(MT, NT, WK, WP) \
    if (s.mt == MT && s.nt == NT && s.wk == WK && s.wp == WP) return launch_whole<MT, NT, WK, WP>;
    PPC_K5(2, 2, 1, 4) PPC_K5(2, 2, 2, 2) PPC_K5(2, 2, 4, 1) PPC_K5(1, 2, 1, 4) PPC_K5(1, 2, 4, 1) PPC_K5(1, 1, 4, 1)
#undef PPC_K5
    return nullptr;
}

k5_list_fn k5_list_lookup(const K5Shape& s) {
#define PPC_K5(NT, WK) \
    if (s.nt == NT && s.wk == WK) return k5_list_f32<NT, WK>;
    PPC_K5(2, 4) PPC_K5(1, 4)
#undef PPC_K5
    return nullptr;
}

}  // namespace ppc
