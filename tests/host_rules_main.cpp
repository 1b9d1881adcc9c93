// The launch rules that keep the kernels' loads inside their buffers, walked exhaustively on the CPU.
#include <algorithm>
#include <cstdio>

#include "block_rules.hpp"

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

int main() {
    if (block_pieces()) return 1;
    std::printf("ok\n");
    return 0;
}
