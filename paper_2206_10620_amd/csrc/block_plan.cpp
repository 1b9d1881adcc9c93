// Plan step of the block-pruned matrix product (paper, section 2.1.2 for the sparsity; the split into a
// compile-time packing and a run-time kernel follows section 2.3.1).
#include "block_plan.hpp"

#include <algorithm>
#include <cstring>

#include "plan.hpp"

namespace ppc {

pp_status_t build_block_plan(const pp_block_gemm_desc_t& d, BlockHostPlan& p) {
    if (!d.weights) return PP_ERR_NULL;
    if (d.m < 1 || d.k < 1 || d.block_m < 1 || d.block_k < 1) return PP_ERR_SHAPE;
    if ((int64_t)d.m * d.k >= ((int64_t)1 << 31)) return PP_ERR_SHAPE;
    if (d.dtype != PP_F32 && d.dtype != PP_F16) return PP_ERR_UNSUPPORTED;
    if (d.flags & ~(uint32_t)(PP_FLAG_RELU | PP_FLAG_HOST_ONLY)) return PP_ERR_UNSUPPORTED;
    if (d.variant < 0 || d.variant > 2 || (d.variant == 2 && d.dtype != PP_F16)) return PP_ERR_UNSUPPORTED;
    p.m = d.m, p.k = d.k, p.bm = d.block_m, p.bk = d.block_k;
    p.flags = d.flags, p.dtype = d.dtype;
    p.forced = d.variant != 0;
    p.variant = d.variant ? d.variant : (d.dtype == PP_F16 ? 2 : 1);
    const int RT = kBlockRowTile;
    const int blocks_k = (d.k + d.block_k - 1) / d.block_k;
    p.row_tiles = (d.m + RT - 1) / RT;
    auto row_kept = [&](int r, int bj) { return !d.row_keep || d.row_keep[((int64_t)(r / d.block_m) * blocks_k + bj) * d.block_m + r % d.block_m] != 0; };
    auto col_kept = [&](int bi, int c) { return !d.col_keep || d.col_keep[((int64_t)bi * blocks_k + c / d.block_k) * d.block_k + c % d.block_k] != 0; };

    p.tile_off.assign(1, 0);
    p.tile_cols.clear();
    p.tile_len.clear();
    p.kept_weights = 0;
    std::vector<uint8_t> used((size_t)d.k);
    for (int t = 0; t < p.row_tiles; ++t) {
        const int r0 = t * RT, r1 = std::min(d.m, r0 + RT);
        std::fill(used.begin(), used.end(), 0);
        // the block rows this tile overlaps; a block contributes its kept columns if it keeps one of the tile's rows
        for (int bi = r0 / d.block_m; bi <= (r1 - 1) / d.block_m; ++bi)
            for (int bj = 0; bj < blocks_k; ++bj) {
                int rows_here = 0;
                for (int r = std::max(r0, bi * d.block_m); r < std::min(r1, (bi + 1) * d.block_m); ++r) rows_here += row_kept(r, bj) ? 1 : 0;
                if (!rows_here) continue;
                for (int c = bj * d.block_k; c < std::min(d.k, (bj + 1) * d.block_k); ++c)
                    if (col_kept(bi, c)) {
                        used[c] = 1;
                        p.kept_weights += rows_here;
                    }
            }
        int len = 0;
        for (int c = 0; c < d.k; ++c)
            if (used[c]) {
                p.tile_cols.push_back(c);
                ++len;
            }
        p.tile_len.push_back(len);
        while (len % kBlockChunk) {          // pad with a column that exists; its weights are zeros
            p.tile_cols.push_back(p.tile_cols.back());
            ++len;
        }
        p.tile_off.push_back((int32_t)p.tile_cols.size());
    }
    p.executed_weights = (int64_t)p.tile_cols.size() * RT;

    const bool half = d.dtype == PP_F16;
    // Calls put(row, column, value) for every kept weight of rows r0 .. r1 - 1, block by block.
    auto each_kept = [&](int r0, int r1, auto&& put) {
        for (int r = r0; r < r1; ++r) {
            const int bi = r / d.block_m;
            const float* w = d.weights + (int64_t)r * d.k;
            for (int bj = 0; bj < blocks_k; ++bj) {
                if (!row_kept(r, bj)) continue;
                const int c0 = bj * d.block_k, c1 = std::min(d.k, c0 + d.block_k);
                const uint8_t* keep = d.col_keep ? d.col_keep + ((int64_t)bi * blocks_k + bj) * d.block_k : nullptr;
                for (int c = c0; c < c1; ++c)
                    if (!keep || keep[c - c0]) put(r, c, w[c]);
            }
        }
    };
    std::vector<int32_t> place((size_t)d.k, 0);        // where a column sits in the current tile's list
    p.apk.assign(half ? p.tile_cols.size() * (size_t)RT : 0, 0);
    for (int t = 0; half && t < p.row_tiles; ++t) {
        for (int i = 0; i < p.tile_len[t]; ++i) place[p.tile_cols[(size_t)p.tile_off[t] + i]] = p.tile_off[t] + i;
        each_kept(t * RT, std::min(d.m, (t + 1) * RT), [&](int row, int c, float v) {
            const size_t at = (size_t)place[c], chunk = at / kBlockChunk, kk = at % kBlockChunk;
            const int r = row - t * RT;
            p.apk[((chunk * 2 + r / 32) * 64 + (r % 32) + 32 * (kk / 8)) * 8 + kk % 8] = f32_to_f16_rne(v);
        });
    }
    if (p.variant == 1) {
        // (a row group that a block prunes entirely takes none of the block's columns)
        const int R = kBlockRow32, tiles = (d.m + R - 1) / R;
        p.group_off32.assign(1, 0);
        p.list32.clear();
        std::vector<int32_t> cols;
        for (int t = 0; t < tiles; ++t) {
            const int r0 = t * R, r1 = std::min(d.m, r0 + R);
            std::fill(used.begin(), used.end(), 0);
            for (int bi = r0 / d.block_m; bi <= (r1 - 1) / d.block_m; ++bi)
                for (int bj = 0; bj < blocks_k; ++bj) {
                    bool any = false;
                    for (int r = std::max(r0, bi * d.block_m); r < std::min(r1, (bi + 1) * d.block_m) && !any; ++r) any = row_kept(r, bj);
                    if (!any) continue;
                    for (int c = bj * d.block_k; c < std::min(d.k, (bj + 1) * d.block_k); ++c) used[c] |= col_kept(bi, c) ? 1 : 0;
                }
            cols.clear();
            for (int c = 0; c < d.k; ++c)
                if (used[c]) cols.push_back(c);
            const size_t len = cols.size();
            while (cols.size() % 8) cols.push_back(-1);        // no column: the kernels read 0 there
            const size_t g0 = p.list32.size() / 8, ng = cols.size() / 8;
            p.list32.resize((g0 + ng) * 8);
            p.wpk32.resize((g0 + ng) * 256, 0.0f);
            for (size_t e = 0; e < cols.size(); ++e) p.list32[(g0 + e / 8) * 8 + (e & 1) * 4 + (e % 8) / 2] = cols[e];
            for (size_t e = 0; e < len; ++e) place[cols[e]] = (int32_t)e;
            each_kept(r0, r1, [&](int r, int c, float v) {
                const int e = place[c];
                p.wpk32[((g0 + e / 8) * 64 + (r - r0) + 32 * (e & 1)) * 4 + (e % 8) / 2] = half ? f16_to_f32(f32_to_f16_rne(v)) : v;
            });
            p.group_off32.push_back((int32_t)(g0 + ng));
        }
        p.list32.resize(p.list32.size() + 2 * kF32Pad * 8, 0);
        p.wpk32.resize(p.wpk32.size() + kF32Pad * 256, 0.0f);
    }
    p.bias.assign((size_t)p.row_tiles * RT, 0.0f);
    if (d.bias) std::memcpy(p.bias.data(), d.bias, (size_t)d.m * sizeof(float));
    return PP_OK;
}

pp_status_t unpack_block_tile(const BlockHostPlan& p, int tile, float* w_out) {
    if (tile < 0 || tile >= p.row_tiles) return PP_ERR_SHAPE;
    const int RT = kBlockRowTile;
    std::fill(w_out, w_out + (size_t)RT * p.k, 0.0f);
    if (p.variant == 1) {
        for (int t = 2 * tile; t < 2 * tile + 2 && t + 1 < (int)p.group_off32.size(); ++t)
            for (int64_t e = (int64_t)p.group_off32[t] * 8; e < (int64_t)p.group_off32[t + 1] * 8; ++e) {
                const int64_t g = e / 8;
                const int k8 = (int)(e % 8), c = p.list32[g * 8 + (k8 & 1) * 4 + k8 / 2];
                for (int r = 0; r < kBlockRow32; ++r) {
                    const float v = p.wpk32[(g * 64 + r + 32 * (k8 & 1)) * 4 + k8 / 2];
                    if (c >= 0) w_out[(size_t)((t & 1) * kBlockRow32 + r) * p.k + c] = v;
                    else if (v != 0.0f) return PP_ERR_PATTERN;      // padding must carry zeros
                }
            }
        return PP_OK;
    }
    for (int32_t at = p.tile_off[tile]; at < p.tile_off[tile + 1]; ++at) {
        const int c = p.tile_cols[at];
        const bool pad = at - p.tile_off[tile] >= p.tile_len[tile];
        const size_t chunk = (size_t)at / kBlockChunk, kk = (size_t)at % kBlockChunk;
        for (int r = 0; r < RT; ++r) {
            const float v = f16_to_f32(p.apk[((chunk * 2 + r / 32) * 64 + (r % 32) + 32 * (kk / 8)) * 8 + kk % 8]);
            if (pad) {
                if (v != 0.0f) return PP_ERR_PATTERN;      // padding must carry zeros
            } else {
                w_out[(size_t)r * p.k + c] = v;
            }
        }
    }
    return PP_OK;
}

}  // namespace ppc
