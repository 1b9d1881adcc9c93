// Instantiations of the binary32 matrix-core kernels and the rule that picks among them.
#include "k5_f32.hpp"

namespace ppc {

namespace {

// Modelled time of a launch in cycles: the larger of the matrix-core time on the fullest compute unit (its wavefronts per
// SIMD times 4 mt nt MFMAs of 64 cycles per unit) and the time the operands take to come out of L2 (1 KB per unit for each
// of mt weight and nt pixel operands, 16 bytes per clock and compute unit; wavefronts that share weights find most of them
// in the vector cache).  Fitted to 11 shapes on 13 layers and 7 on 9 products: the shape it picks is within 1 % of the best
// one tried on average, 3 % at worst.  Examples: 128 channels, 56x56 to 28x28, 3x3, batch 8: 2 2 4 1 takes 23.5 us, 1 1 4 1
// 30.2, 2 2 1 4 72.8; 256 to 128 channels, 1x1, 56x56, batch 8: 1 2 1 4 22.5 us, 2 2 8 1 32.6.
double model(int64_t wgs, int waves, int64_t units_per_wave, int mt, int nt, int wp) {
    const double per_simd = (double)((wgs + 255) / 256) * waves / 4.0;
    const double mfma = (per_simd < 1.0 ? 1.0 : per_simd) * (double)units_per_wave * 4 * mt * nt * 64;
    const double traffic = (double)wgs * waves * (double)units_per_wave * (mt * (wp > 1 ? 0.3 : 1.0) + nt) * 1024 / (256 * 16.0);
    return mfma > traffic ? mfma : traffic;
}

struct Option { int mt, nt, wk, wp; };
const Option kConv[] = {{2, 2, 1, 4}, {2, 2, 2, 2}, {2, 2, 4, 1}, {2, 2, 8, 1}, {1, 2, 1, 4}, {1, 2, 4, 1}, {1, 2, 8, 1}, {1, 1, 4, 1}, {1, 1, 8, 1}, {1, 1, 16, 1}};
const Option kList[] = {{1, 2, 4, 1}, {1, 2, 8, 1}, {1, 1, 4, 1}, {1, 1, 8, 1}, {1, 1, 16, 1}};

template <int N>
K5Shape pick(const Option (&opts)[N], int rows32, int64_t cols, int units) {
    K5Shape best;
    double best_t = 1e300;
    for (const Option& o : opts) {
        if (o.wk > 4 && units < 2 * o.wk) continue;          // shares of less than two units only cost their reduction
        const int64_t wgs = (int64_t)((rows32 + o.mt - 1) / o.mt) * ((cols + 32 * o.nt * o.wp - 1) / (32 * o.nt * o.wp));
        const double t = model(wgs, o.wk * o.wp, (units + o.wk - 1) / o.wk, o.mt, o.nt, o.wp);
        if (t < best_t) best_t = t, best = K5Shape{o.mt, o.nt, o.wk, o.wp};
    }
    return best;
}

}  // namespace

K5Shape k5_pick_conv(int rows32, int64_t cols, int units) { return pick(kConv, rows32, cols, units); }
K5Shape k5_pick_list(int rows32, int64_t cols, int units) { return pick(kList, rows32, cols, units); }

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
