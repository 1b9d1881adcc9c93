// How launches of the binary32 matrix-core kernels are dealt out, and what they are modelled to cost: used by the launcher and
// by the plan, which picks between the kernels.
#pragma once

#include <cstdint>
#include <initializer_list>

namespace ppc {

// The sixteen channels that reduction group g of the dense convolution in parts loads: from channel k5_group_first on, the upper half of
// a wavefront k5_half_channels further, the j-th of a lane's eight at k5_step j.  All of them are channels of the layer: x ends behind the
// last one of the last image, and of the sum that is a load's address the hardware need not check the part that names the channel.  The
// last group therefore begins early, and what it holds again of the one before it meets zero weights.
constexpr int k5_group_first(int c_in, int g) { return 16 * g <= c_in - 16 ? 16 * g : c_in > 16 ? c_in - 16 : 0; }
constexpr int k5_half_channels(int c_in) { return c_in >= 16 ? 8 : c_in > 8 ? c_in - 8 : 0; }
constexpr int k5_step(int c_in, int j) { return j < c_in ? j : c_in - 1; }
// Where a channel's weight stands: its group, half and place.
struct K5Slot {
    int g, half, j;
};
constexpr K5Slot k5_slot(int c_in, int ci) {
    const int g = ci / 16, o = ci - k5_group_first(c_in, g), half = o >= 8 ? 1 : 0;
    return K5Slot{g, half, o - half * k5_half_channels(c_in)};
}

// The dense convolution: workgroups of wp x wk wavefronts of 32 mt filters x 32 pixels each, wk of them on one tile's reduction, wp on
// different pixels with the same weights.  Modelled microseconds of a launch: start, and per workgroup on a compute unit (the mean of
// their number and that number rounded up) `wg`, and per reduction unit of a wavefront `alone` or, where more, `wg_unit` per workgroup.
// Fitted to 64 layers (1x1 to 7x7, stride 1 and 2, 3 to 478 channels, 7x7 to 199 wide, batch 1 to 32): 7 to 19 % rms; the shape it
// picks is 3 % from the best of seventeen tried on average, 1.4 times at worst.  The shapes left out were never better by more than
// a percent or two.  Examples: 256 channels, 14x14, 3x3, batch 32: 4 2 4 takes 41 us, 2 2 2 53, 4 4 1 58; 256 to 128 channels, 1x1, 56x56,
// batch 8: 4 4 2 takes 17.0 us, 4 4 1 18.2, 2 2 2 20.
struct K5ConvShape {
    int mt = 1, wp = 1, wk = 1;
    double wg = 0.0, alone = 0.0, wg_unit = 0.0;
};
inline constexpr K5ConvShape kK5Conv[] = {{4, 4, 1, 1.97, 0.351, 0.521}, {4, 4, 2, 4.11, 0.046, 0.763}, {4, 2, 4, 3.70, 0.750, 0.844}, {2, 4, 1, 0.88, 0.393, 0.326},
                                          {2, 2, 2, 0.84, 0.386, 0.336}, {2, 2, 4, 2.46, 0.485, 0.583}, {2, 1, 4, 1.13, 0.300, 0.372}, {1, 4, 1, 0.45, 0.305, 0.231}};

// How many 32-filter tiles of operands there are for the rows32 of a layer: a wavefront takes up to four, of layers that have no more up to two.
constexpr int k5_padded_tiles(int rows32) { return rows32 <= 2 ? 2 : (rows32 + 3) / 4 * 4; }

// The shape for a layer of `rows32` 32-filter tiles, `cols` pixels and `units` reduction units; its modelled microseconds in *us.
inline const K5ConvShape& k5_pick_conv(int rows32, int64_t cols, int units, double* us = nullptr) {
    const K5ConvShape* best = nullptr;
    double best_t = 1e300;
    for (const K5ConvShape& o : kK5Conv) {
        if (o.mt > k5_padded_tiles(rows32)) continue;        // (never modelled fastest there)
        const int64_t wgs = (int64_t)((rows32 + o.mt - 1) / o.mt) * ((cols + 32 * o.wp - 1) / (32 * o.wp));
        const double even = wgs < 256 ? 1.0 : (double)wgs / 256.0, load = 0.5 * (even + (double)((wgs + 255) / 256));
        const double unit = load * o.wg_unit > o.alone ? load * o.wg_unit : o.alone;
        const double t = 5.8 + load * o.wg + (double)((units + o.wk - 1) / o.wk) * unit;
        if (t < best_t) best_t = t, best = &o;
    }
    if (us) *us = best_t;
    return *best;
}
// Tiles on the binary32 instruction: wavefronts of 32 mt filters x 32 nt pixels (columns), wk wavefronts of a workgroup on one tile's
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

// (More than four shares are never modelled faster than four: the same matrix-core time and more to sum.)
inline constexpr K5Shape kK5Whole[] = {{2, 2, 1, 4}, {2, 2, 2, 2}, {2, 2, 4, 1}, {1, 2, 1, 4}, {1, 2, 4, 1}, {1, 1, 4, 1}};
inline constexpr K5Shape kK5List[] = {{1, 2, 4, 1}, {1, 1, 4, 1}};

template <int N>
inline K5Shape k5_pick(const K5Shape (&opts)[N], int rows32, int64_t cols, int units, double* cycles = nullptr) {
    K5Shape best;
    double best_t = 1e300;
    for (const K5Shape& o : opts) {
        const int64_t wgs = (int64_t)((rows32 + o.mt - 1) / o.mt) * ((cols + 32 * o.nt * o.wp - 1) / (32 * o.nt * o.wp));
        const double t = k5_cycles(wgs, o.wk * o.wp, (units + o.wk - 1) / o.wk, o.mt, o.nt, o.wp);
        if (t < best_t) best_t = t, best = o;
    }
    if (cycles) *cycles = best_t;
    return best;
}
// The shape of k5_whole_f32 for a layer (units of eight channels), its modelled microseconds in *us; the shape for a block-pruned product
// of `rows32` 32-row tiles, `cols` columns and `units` reduction units per tile.
inline K5Shape k5_pick_whole(int rows32, int64_t cols, int units, double* us = nullptr) {
    double cycles = 0.0;
    const K5Shape s = k5_pick(kK5Whole, rows32, cols, units, &cycles);
    if (us) *us = 5.0 + 1.1 * cycles / 2350.0;
    return s;
}
inline K5Shape k5_pick_list(int rows32, int64_t cols, int units) { return k5_pick(kK5List, rows32, cols, units); }

// The faster one's microseconds, or those of k5_whole_f32 where the other is not allowed; `units` are the
// reduction units of sixteen channels, `whole_units` those of eight; out_mb is what the convolution stores, in MB, which costs k5_whole_f32 more.  On 420 layers (1x1 to 7x7, stride 1 and 2, 1 to 512 channels, 100 to
// 8 million pixels) the choice is 1.8 % from the faster one on average, 1.39 times at worst; parts everywhere would be 11 %.  Parts lose
// where there is little to share or few channels to a group of sixteen: 3 to 64 channels, 7x7, stride 2, 1080x1920: 267 us against
// 232; 3 to 32, 5x5, 2160x3840: 1253 against 984; 256 channels, 14x14, batch 32: 42 against 75.
inline double k5_model_conv(int rows32, int64_t cols, int units, int whole_units, bool parts_allowed, double out_mb, bool* whole = nullptr) {
    double us = 0.0, whole_us = 0.0;
    (void)k5_pick_conv(rows32, cols, units, &us);
    (void)k5_pick_whole(rows32, cols, whole_units, &whole_us);
    const bool take = !parts_allowed || 1.1 * whole_us - 1.0 + 0.1 * out_mb < us;       // (what its model leaves out)
    if (whole) *whole = take;
    return take ? whole_us : us;
}
// Whether a layer's sums are as near in parts as on the binary32 instruction: they are from eight products on (k5_f32.hpp has the
// errors); a window that overlaps the border has down to half its taps.  `fewest` is the kept taps of the filter that three quarters of the
// filters with any have at least as many as.
constexpr bool k5_parts_near(int64_t fewest, int ks) { return fewest >= (ks > 1 ? 16 : 8); }

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
