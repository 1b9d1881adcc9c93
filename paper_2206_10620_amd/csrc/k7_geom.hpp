// Geometry of the row-stacked matrix-core kernel (k7), shared by the host-side plan, the launcher and the device code.
#pragma once

#include <cstdint>

namespace ppc {

constexpr int kK7WeightBytes = 18 * 1024;   // operand fragments of one 16-channel chunk: 9 taps x 2 filter halves x 1 KB

// Four wavefronts compute 64 filters for tr rows x tc columns of the batch laid out as one tall image; a wavefront t rows of 32 columns,
// or 2 t rows of 16 (tc = 16: images up to 16 columns wide).
struct K7Geom {
    int t = 4, tc = 32;
    int tr = 16, trp = 18;      // rows, staged rows
    int pitch = 36;             // words per staged row and channel pair: four of which the last is the column on the left, the tile's columns;
                                // the column on the right is the first word of the next row
    int gpr = 6;                // groups of eight pixels, from a column that is a multiple of eight, that hold a staged row
    int tasks = 108;            // staged groups of a channel
    int rounds = 2;             // ... for each lane of a wavefront
    int plane = 2608, xbuf = 20864;         // LDS bytes of a channel pair, of a chunk
    int wbufs = 2;              // weight buffers
    int group = 0;              // LDS bytes of the buffers of four wavefronts: two of x, wbufs of weights
};
constexpr K7Geom k7_geom(int t, int tc) {
    K7Geom g;
    g.t = t, g.tc = tc, g.tr = 128 * t / tc, g.trp = g.tr + 2, g.pitch = tc + 4, g.gpr = tc == 16 ? 2 : tc / 8 + 2;
    g.tasks = g.trp * g.gpr, g.rounds = (g.tasks + 63) / 64;
    const int unit = t == 4 ? 16 : 256;     // (reads of two planes as one instruction: multiples of 256)
    g.plane = ((g.trp * g.pitch + 1) * 4 + unit - 1) / unit * unit;
    g.xbuf = 8 * g.plane;
    g.wbufs = t == 4 || tc == 64 ? 2 : 3;
    g.group = 2 * g.xbuf + g.wbufs * kK7WeightBytes;
    return g;
}
constexpr int kK7Tail = 4 * 256;            // behind the buffers: four tiles' bias values
constexpr int k7_lds(int t, int tc, int kg) { return kg * k7_geom(t, tc).group + kK7Tail; }
constexpr int kK7MaxLds = 160 * 1024;

// Workgroups of kg groups of four wavefronts, each on its share of a tile's chunks.  Modelled microseconds of a launch: 5.5 and, per
// workgroup that a compute unit has to run beside another one, wg and per chunk of a group `chunk` (`ragged` more where rows of the
// input end inside a group of eight pixels); at least `alone` of that.  Fitted to 70 layers (3 to 512 channels, 7x7 to 1920 wide, batch 1 to
// 32): 1 to 12 % rms, and the shape it picks is 2 % from the best of twelve tried on average, 10 % at worst.  One group takes several
// tiles in turn, two share one: those where there are few.  Examples, t tc kg: 8 x 64 to 64 channels, 224x224, pooled: 2 32 1 takes 32.9 us,
// 4 64 1 36; 64 to 64, 1080x1920: 4 64 1 185, 2 64 1 205; 8 x 512 to 512, 28x28: 2 32 2 36, 2 64 1 45.
struct K7Shape {
    int t, tc, kg;
    double alone, wg, chunk, ragged;
};
constexpr K7Shape kK7Shapes[] = {{2, 32, 1, 0.45, 0.985, 2.013, 0.116}, {2, 64, 1, 0.50, 0.996, 1.901, 0.006}, {4, 64, 1, 0.55, 1.682, 3.608, 0.259},
                                 {2, 16, 2, 1.00, 1.499, 1.168, 0.480}, {2, 32, 2, 1.00, 1.427, 1.817, 0.0},   {2, 64, 2, 1.00, 1.654, 1.694, 0.051}};
inline double k7_model(const K7Shape& s, int64_t items, int chunks, bool ragged) {
    const double even = (double)items / 256.0, full = (double)((items + 255) / 256);
    double load = s.kg == 1 ? 0.25 * (even + full) : 0.5 * ((even > 1.0 ? even : 1.0) + full);
    if (load < s.alone) load = s.alone;
    return 5.5 + load * (s.wg + (double)chunks / s.kg * (s.chunk + (ragged ? s.ragged : 0.0)));
}
constexpr bool k7_fits() {              // a workgroup of eight wavefronts and two of four into a compute unit's LDS
    for (const K7Shape& s : kK7Shapes)
        if ((s.kg == 1 ? 2 : 1) * k7_lds(s.t, s.tc, s.kg) > kK7MaxLds) return false;
    return true;
}
static_assert(k7_fits(), "a compute unit's LDS");

}  // namespace ppc
