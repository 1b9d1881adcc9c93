// How launches of the binary32 matrix-core kernels are dealt out, and what they are modelled to cost: used by the launcher and
// by the plan, which picks between the kernels.
#pragma once

#include <cstdint>
#include <initializer_list>

namespace ppc {

// The dense kernel: wavefront tiles of 32 mt filters x 32 nt pixels (columns), wk wavefronts of a workgroup on one tile's
// reduction, wp on different pixels.
struct K5Shape {
    int mt = 1, nt = 1, wk = 1, wp = 1;
};

// Modelled time of a launch in cycles: the larger of the matrix-core time on the fullest compute unit (its wavefronts per
// SIMD times 4 mt nt MFMAs of 64 cycles per unit) and the time the operands take to come out of L2 (1 KB per unit for each
// of mt weight and nt pixel operands, 16 bytes per clock and compute unit; wavefronts that share weights find most of them
// in the vector cache).  Fitted to 11 shapes on 13 layers and 7 on 9 products: the shape it picks is within 1 % of the best
// one tried on average, 3 % at worst.  Examples: 128 channels, 56x56 to 28x28, 3x3, batch 8: 2 2 4 1 takes 23.5 us, 1 1 4 1
// 30.2, 2 2 1 4 72.8; 256 to 128 channels, 1x1, 56x56, batch 8: 1 2 1 4 22.5 us, 2 2 8 1 32.6.
inline double k5_cycles(int64_t wgs, int waves, int64_t units_per_wave, int mt, int nt, int wp) {
    const double per_simd = (double)((wgs + 255) / 256) * waves / 4.0;
    const double mfma = (per_simd < 1.0 ? 1.0 : per_simd) * (double)units_per_wave * 4 * mt * nt * 64;
    const double traffic = (double)wgs * waves * (double)units_per_wave * (mt * (wp > 1 ? 0.3 : 1.0) + nt) * 1024 / (256 * 16.0);
    return mfma > traffic ? mfma : traffic;
}

inline constexpr K5Shape kK5Conv[] = {{2, 2, 1, 4}, {2, 2, 2, 2}, {2, 2, 4, 1}, {2, 2, 8, 1}, {1, 2, 1, 4}, {1, 2, 4, 1}, {1, 2, 8, 1}, {1, 1, 4, 1}, {1, 1, 8, 1}, {1, 1, 16, 1}};
inline constexpr K5Shape kK5List[] = {{1, 2, 4, 1}, {1, 2, 8, 1}, {1, 1, 4, 1}, {1, 1, 8, 1}, {1, 1, 16, 1}};

template <int N>
inline K5Shape k5_pick(const K5Shape (&opts)[N], int rows32, int64_t cols, int units, double* cycles = nullptr) {
    K5Shape best;
    double best_t = 1e300;
    for (const K5Shape& o : opts) {
        if (o.wk > 4 && units < 2 * o.wk) continue;          // shares of less than two units only cost their reduction
        const int64_t wgs = (int64_t)((rows32 + o.mt - 1) / o.mt) * ((cols + 32 * o.nt * o.wp - 1) / (32 * o.nt * o.wp));
        const double t = k5_cycles(wgs, o.wk * o.wp, (units + o.wk - 1) / o.wk, o.mt, o.nt, o.wp);
        if (t < best_t) best_t = t, best = o;
    }
    if (cycles) *cycles = best_t;
    return best;
}

// Its modelled microseconds.
inline double k5_model_conv(int rows32, int64_t cols, int units) {
    double cycles = 0.0;
    (void)k5_pick(kK5Conv, rows32, cols, units, &cycles);
    return 5.0 + 1.1 * cycles / 2350.0;
}
// The generic kernel, one lane per output walking its filter's kernel list: modelled microseconds for n images of c_in channels of
// in_px pixels and c_out filters with out_px stored outputs each, `kept` kernels of `taps` taps, at most `longest` in a filter.
// The walk costs up to 1.4 times as much where an image is larger than an L2 (4 MB); reading and writing is 0.27 us per MB.  Fitted
// to 209 layers (1x1 to 7x7, stride 1 and 2, pooled or not, 0.005 to 0.7 kept): 19 % rms, closest where it is near the dense product.
inline double lists_model(int n, int c_in, int64_t in_px, int c_out, int64_t out_px, int64_t kept, int taps, int64_t longest, bool pool) {
    const double windows = pool ? 4.0 : 1.0, waves = (double)(((int64_t)n * out_px + 255) / 256 * 4);
    const double image = (double)c_in * (double)in_px * 4e-6, over = image / 4.0 - 1.0, read = kept < c_in ? (double)kept / c_in : 1.0;
    const double far = 1.0 + 0.385 * (over < 0.0 ? 0.0 : over > 1.0 ? 1.0 : over);
    const double together = waves * (double)kept * windows * 1e-6 * (36.0 + 65.0 * taps) * far, alone = (double)longest * windows * (0.075 + 0.224 * taps);
    return 3.05 + (together > alone ? together : alone) + 0.27 * n * (image * read + (double)c_out * (double)out_px * 4e-6);
}
// The shape for a layer (or block-pruned product) of `rows32` 32-row tiles, `cols` pixels or columns and `units` reduction units per tile.
inline K5Shape k5_pick_conv(int rows32, int64_t cols, int units) { return k5_pick(kK5Conv, rows32, cols, units); }
inline K5Shape k5_pick_list(int rows32, int64_t cols, int units) { return k5_pick(kK5List, rows32, cols, units); }

// The 3x3 kernel on the small instruction: modelled microseconds of a layer of `fgroups` 16-filter groups, `ptiles` 256-pixel
// tiles and c_in channels of which a quad of filters uses `taps_used` taps on average, with the best number of wavefronts
// (4, 8 or 16) on a tile's channels; that number in *wk.
// A channel costs a SIMD 250 cycles and 33 per used (quad, tap); a wavefront with nobody to share the SIMD with takes about
// 1500.  Fitted to eleven layers (batch 1 to 32, 16 to 512 channels, 7x7 to 224x224): within 12 % on all but the smallest.
// They kept 0.3 to 0.5 of the kernels; with few used the taken branches weigh more, and the time is modelled with 550 and 21
// (191 layers with 0.005 to 0.7 kept: 17 % rms), which is the same around six used taps.
inline double k6_model(int fgroups, int64_t ptiles, int c_in, double taps_used, int* wk) {
    double best = 1e300, modelled = 0.0;
    for (int w : {4, 8, 16}) {
        const double share = (c_in + w - 1) / w;
        const double per_simd = (double)((fgroups * ptiles + 255) / 256) * w / 4.0;
        const double together = per_simd * share, alone = share * 1500.0;
        auto us = [&](double cycles) { return 7.0 + (cycles > alone ? cycles : alone) / 2350.0; };
        const double split = us(together * (250.0 + 33.0 * 4.0 * taps_used));
        if (split < best - 0.01) best = split, *wk = w, modelled = us(together * (550.0 + 85.0 * taps_used));
    }
    return modelled;
}

// The tiled vector kernel in binary32: modelled microseconds of `tiles` tiles of 64 lanes (`lw` across, `r` rows each), for each of
// which `blocks` workgroups stage c_in channels and `groups` groups of four filters, with `kernels` kept kernels each, walk them in
// `ks` shares and `chunks` chunks.  Staging costs by the row and by the slot of 16 bytes (rows on 16-byte boundaries) or 4; a channel
// and a kernel cost a SIMD 22 and 106 cycles a row; one wavefront alone waits for latencies.  Fitted to 491 layers, closest where
// the kernel is near the fastest: 29 % rms.
inline double k1_model(int64_t tiles, int lw, int r, bool slots16, int blocks, int groups, int ks, int c_in, double kernels, int chunks) {
    const double rows = 64.0 * r / lw + 2.0, share = (double)c_in / ks, per_share = kernels / ks;
    const double staging = (double)tiles * blocks * c_in * rows * (0.9 * lw * (slots16 ? 1 : 4) + 5.6) / 256.0;
    const double walk = (double)tiles * groups * ks / 1024.0 * r * (share * 22.0 + per_share * 106.0);
    const double alone = share * 240.0 + per_share * 610.0 + chunks * 2650.0;
    return 13.0 + (staging + walk > alone ? staging + walk : alone) / 2350.0;
}

}  // namespace ppc
