// The launch rules that keep the kernels' loads inside their buffers, walked exhaustively on the CPU; with arguments, the shapes they pick.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <iterator>
#include <vector>

#include "block_rules.hpp"
#include "buffer_rules.hpp"
#include "f32_rules.hpp"
#include "reuse_rules.hpp"

using namespace ppc;

static int fail(const char* what, long a, long b, long c) {
    std::printf("FAIL %s %ld %ld %ld\n", what, a, b, c);
    return 1;
}

// Every 16-byte piece of a [k][n] binary16 matrix, as the wide and the split kernel classify it: a direct load ends inside x.
static int block_pieces() {
    for (int k = 1; k <= 40; ++k)
        for (int n = 1; n <= 40; ++n) {
            const uint32_t row_bytes = 2u * (uint32_t)n, x_bytes = row_bytes * (uint32_t)k;
            for (int r = 0; r < k; ++r)
                for (int c = 0; c < n; c += 8) {
                    const uint32_t off = (uint32_t)r * row_bytes + 2u * (uint32_t)c;
                    const bool wide_guarded = (uint32_t)r * row_bytes >= k4_edge_from(x_bytes, row_bytes) && k4_piece_ends_behind(off, x_bytes);
                    const bool split_guarded = k4_piece_ends_behind(off, x_bytes);
                    if (!wide_guarded && off + 16u > x_bytes) return fail("wide tile: direct load behind x", k, n, off);
                    if (!split_guarded && off + 16u > x_bytes) return fail("split tile: direct load behind x", k, n, off);
                    if (wide_guarded && off + 16u <= x_bytes) return fail("wide tile: guarded without need", k, n, off);
                }
        }
    return 0;
}

// Every row whose number the gather's lanes read has one, and the tables hold it, whatever n_max the plan was made for.
static int gather_rows() {
    for (int m = 4; m <= 132; m += 4)
        for (int n = 1; n < 140000; n = n < 9000 ? n + 1 : n * 17 / 16 + 1) {
            const ReuseGather g = reuse_gather_shape(n, m);
            if (g.rows < 1 || g.rows > kGatherMaxRows || g.wgs_x * g.rows < n) return fail("gather does not cover the rows", m, n, g.rows);
            if (reuse_numbered_rows(g) < g.wgs_x * g.rows) return fail("gather reads a row without a number", m, n, g.rows);
            if (reuse_numbered_rows(g) % 8 || reuse_numbered_rows(g) > reuse_row_pitch(n)) return fail("numbered rows outside the tables", m, n, g.rows);
            if (reuse_row_pitch(n) % 8) return fail("segments off the 16-byte words", m, n, 0);
        }
    return 0;
}

// Every channel that a reduction group of the binary32 convolution in parts loads, also those asked for past a share's end, is one of
// the layer's, and every channel has a place of its own that is loaded from it.
static int group_channels() {
    for (int c = 1; c <= 600; ++c) {
        const int groups = (c + 15) / 16;
        for (int g = 0; g <= 2 * groups + 2; ++g)
            for (int half = 0; half < 2; ++half)
                for (int j = 0; j < 8; ++j) {
                    const int ch = k5_group_first(c, g) + half * k5_half_channels(c) + k5_step(c, j);
                    if (ch < 0 || ch >= c) return fail("group loads a channel behind x", c, g, ch);
                }
        std::vector<char> taken((size_t)groups * 16, 0);
        for (int ci = 0; ci < c; ++ci) {
            const K5Slot s = k5_slot(c, ci);
            if (s.g < 0 || s.g >= groups || s.half < 0 || s.half > 1 || s.j < 0 || s.j > 7) return fail("no place for a channel", c, ci, s.g);
            if (k5_group_first(c, s.g) + s.half * k5_half_channels(c) + k5_step(c, s.j) != ci) return fail("a channel's place loads another one", c, ci, s.g);
            if (taken[(size_t)(s.g * 2 + s.half) * 8 + s.j]++) return fail("two channels in one place", c, ci, s.g);
        }
    }
    return 0;
}

// The 16-byte loads of a row's last pixels, with elements of eb bytes: what of them lies inside the buffer of their channel lies inside x, and
// every pixel of the row inside the buffer.
static int row_ends() {
    for (int eb : {2, 4})
        for (int n = 1; n <= 3; ++n)
            for (int c = 1; c <= 4; ++c)
                for (int h = 1; h <= 3; ++h)
                    for (int w = eb == 2 ? 2 : 1; w <= 40; w += eb == 2 ? 2 : 1) {
                        const int64_t plane = (int64_t)h * w * eb, img = plane * c, x_bytes = img * n;
                        for (int ib = 0; ib < n; ++ib)
                            for (int i = ib; i < n; ++i)
                                for (int ch = 0; ch < c; ++ch)
                                    for (int px = 0; px < w; px += 16 / eb) {
                                        const uint32_t records = buffer_records_from(buffer_records(x_bytes - ib * img), (uint32_t)(ch * plane));
                                        const int64_t off = (i - ib) * img + (int64_t)((h - 1) * w + px) * eb, base = ib * img + ch * plane;
                                        for (int e = 0; e < 4; ++e) {
                                            const bool in = off + 4 * e + 4 <= (int64_t)records;
                                            if (in && base + off + 4 * e + 4 > x_bytes) return fail("a row's load ends behind x", c, w, off + 4 * e);
                                            if (!in && px + 4 * e / eb < w) return fail("a pixel outside the buffer", c, w, off + 4 * e);
                                        }
                                    }
                    }
    return 0;
}

// Every 32-filter tile of weights that a wavefront of the binary32 dense product reads is there, whatever the batch.
static int weight_tiles() {
    for (int rows32 = 1; rows32 <= 40; ++rows32)
        for (int units = 1; units < 700; units += 1 + units / 20)
            for (int64_t cols = 1; cols < 40000000; cols = cols * 5 / 4 + 1) {
                const int mt = k5_pick_conv(rows32, cols, units).mt, whole_mt = k5_pick_whole(rows32, cols, units).mt;
                if ((rows32 + mt - 1) / mt * mt > k5_padded_tiles(rows32)) return fail("parts read a tile that is not there", rows32, units, mt);
                if ((rows32 + whole_mt - 1) / whole_mt * whole_mt > (rows32 + 1) / 2 * 2) return fail("a tile that is not there", rows32, units, whole_mt);
            }
    return 0;
}

// The shapes of the two kernels of the binary32 dense product for (32-filter tiles, pixels, units of sixteen channels, of eight), and how many
// shapes each has.
static int shapes(int argc, char** argv) {
    for (int i = 1; i + 3 < argc; i += 4) {
        const int rows32 = std::atoi(argv[i]), units = std::atoi(argv[i + 2]), whole_units = std::atoi(argv[i + 3]);
        const int64_t cols = std::atoll(argv[i + 1]);
        const K5ConvShape p = k5_pick_conv(rows32, cols, units);
        const K5Shape w = k5_pick_whole(rows32, cols, whole_units);
        std::printf("%d %d %d %d %d %d %d %d\n", p.mt, p.wp, p.wk, (units + p.wk - 1) / p.wk, w.mt, w.nt, w.wk, w.wp);
    }
    std::printf("%zu %zu\n", std::size(kK5Conv), std::size(kK5Whole));
    return 0;
}

int main(int argc, char** argv) {
    if (argc > 1) return shapes(argc, argv);
    if (block_pieces() || gather_rows() || group_channels() || row_ends() || weight_tiles()) return 1;
    std::printf("ok\n");
    return 0;
}
