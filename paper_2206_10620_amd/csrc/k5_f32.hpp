// Matrix-core kernels for binary32 storage (gfx950): any convolution (kernel size, stride, fused 2x2 max-pool) and the
// block-pruned product, on v_mfma_f32_32x32x2_f32.  Inputs, products and sums are binary32 throughout.
//
// The binary32 matrix instruction is slow enough (32 x 32 x 2 in 64 cycles, 157 TFLOP/s for the chip) that its operands
// need no staging: a "B" operand is one value per lane -- output pixel lane % 32 at reduction index lane / 32 -- and 32
// neighbouring pixels of one channel row are 128 consecutive bytes of x, so a plain load is the operand.  Per wavefront
// and step a 64 x 64 tile issues one 256-byte load per 64-cycle MFMA, a quarter of what the vector cache delivers.
//
// Convolution (k5_conv_f32): the pruned weights are zero-filled to a dense matrix (a 32-filter tile uses every (channel,
// tap) pair at the densities that pattern pruning leaves), reduction index = (tap, channel), taps outermost.  A lane's
// byte offset into x then changes with the tap only; the channel is the scalar offset of a buffer load, and a tap that
// falls outside the image gives the lane an offset beyond the buffer, which loads as zero.  No address arithmetic, no
// masks in the loop.  Reduction and pixels are dealt over the wavefronts of a workgroup: WK of them split the reduction
// units (one unit = one tap x eight channels = four MFMAs per tile) and are summed through LDS in order, WP of them
// take different pixels with the same weights.
//
// A pruned tap is a zero weight here, and 0 x Inf is NaN where the definition skips the tap.  Outputs whose dense sum is not
// finite are therefore summed again from the kernel lists (k0_again); finite inputs pay one multiply-add per output for the test.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "f32_rules.hpp"
#include "k0_generic.hpp"

namespace ppc {

struct K5ConvArgs {
    const float* x;
    const float* wpk;       // [32-filter tile][unit][64 lanes][4]: lane l, value p: filter l % 32, channel min(8 g + 2 p, c_in - 2) + l / 32 of unit (tap, g)
    const float* bias;      // [tiles * 32]
    float* y;
    int32_t n, c_in, c_out, h, w, ho, wo, out_h, out_w;
    int32_t ks, stride, pool, relu;
    int32_t groups, units;  // groups of eight channels, ks * ks * groups
    int32_t pix;            // n * ho * wo convolution outputs
    int32_t ftiles, ptiles, items, per_xcd;
    int64_t x_bytes;
    const K0Args* lists;    // in device memory; its x, y and n are not set
};

typedef float k5_f16 __attribute__((ext_vector_type(16)));
typedef float k5_f4 __attribute__((ext_vector_type(4)));

constexpr int kK5Ahead = 3;                        // reduction units whose loads are in flight behind the one being multiplied
constexpr uint32_t kK5Outside = 0x80000000u;      // a byte offset no buffer of these kernels reaches: the load returns 0

__device__ __forceinline__ __amdgpu_buffer_rsrc_t k5_buffer(const void* base, int64_t bytes) {
    const uint32_t num = bytes > 0x7FFFFFFF ? 0x7FFFFFFFu : (uint32_t)bytes;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)num, 0x00027000);
}
__device__ __forceinline__ float k5_load(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, (int)soff, 0));
}

// Register i of a 32 x 32 tile holds row 8 (i / 4) + 4 (lane / 32) + i % 4, column lane % 32: the bias in that order.
__device__ __forceinline__ k5_f16 k5_bias(const float* b, bool on) {
    k5_f16 v(0.0f);
    if (on) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const k5_f4 b4 = *reinterpret_cast<const k5_f4*>(b + q * 8);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[q * 4 + i] = b4[i];
        }
    }
    return v;
}

// Adds the WK wavefronts' accumulators of one 32 x 32 tile in wavefront order; wavefront wk returns registers
// [16 / WK * wk, ...) of the sum in out[].
template <int WK>
__device__ __forceinline__ void k5_reduce(const k5_f16& acc, float* red, int wk, int lane, float (&out)[16 / WK]) {
    constexpr int R = 16 / WK;
    if constexpr (WK == 1) {
#pragma unroll
        for (int i = 0; i < 16; ++i) out[i] = acc[i];
    } else {
        __syncthreads();                                        // the area's last use is over
#pragma unroll
        for (int i = 0; i < 16; ++i) red[(wk * 16 + i) * 64 + lane] = acc[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < R; ++i) {
            float s = red[(wk * R + i) * 64 + lane];
#pragma unroll
            for (int k = 1; k < WK; ++k) s += red[(k * 16 + wk * R + i) * 64 + lane];
            out[i] = s;
        }
    }
}

// Whether any of the sums is infinite or NaN.
template <int R>
__device__ __forceinline__ bool k5_not_finite(const float (&v)[R]) {
    float z = 0.0f;
#pragma unroll
    for (int i = 0; i < R; ++i) z = __builtin_fmaf(v[i], 0.0f, z);
    return z != z;
}

template <int MT, int NT, int WK, int WP>
__global__ __launch_bounds__(64 * WK * WP) __attribute__((amdgpu_waves_per_eu(WK * WP == 16 ? 4 : 2))) void k5_conv_f32(const K5ConvArgs a) {
    __shared__ float red_all[WK > 1 ? WP * WK * 16 * 64 : 1];
    const int lane = (int)(threadIdx.x & 63u), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wk = wave % WK, wp = wave / WK;
    const int col = lane & 31, half = lane >> 5;
    // Workgroup ids go round-robin to the 8 XCDs: each takes a contiguous range of items, filter tiles fastest, so that
    // the workgroups sharing an L2 read the same pixels.
    const int item = (int)(blockIdx.x & 7u) * a.per_xcd + (int)(blockIdx.x >> 3);
    if (item >= a.items) return;
    const int ft = item % a.ftiles, pt = item / a.ftiles;
    const int j0 = (pt * WP + wp) * 32 * NT;                    // first pixel of this wavefront
    const int hw = a.h * a.w, ohw = a.ho * a.wo;
    const int img0 = (j0 < a.pix ? j0 : 0) / ohw;               // wave-uniform
    const int64_t img_elems = (int64_t)a.c_in * hw;
    const __amdgpu_buffer_rsrc_t xr = k5_buffer(a.x + img0 * img_elems, a.x_bytes - img0 * img_elems * 4);

    // a lane's pixels: image row / column of the first tap, offset of that tap from the first image of the tile
    int iy0[NT], ix0[NT], obase[NT];
    uint32_t base[NT];                                          // in elements
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int j = j0 + nt * 32 + col;
        int img = j / ohw, rem = j - img * ohw, oy, ox, opix;
        if (a.pool) {                                           // four consecutive pixels are one pooling window
            const int q = rem >> 2, py = q / a.out_w, px = q - py * a.out_w;
            oy = 2 * py + ((rem >> 1) & 1), ox = 2 * px + (rem & 1);
            opix = q;
        } else {
            oy = rem / a.wo, ox = rem - oy * a.wo;
            opix = rem;
        }
        const bool ok = j < a.pix;
        const int iy = oy * a.stride - a.ks / 2;
        iy0[nt] = ok ? iy : -1000000;                           // no tap of a pixel past the end is inside an image
        ix0[nt] = ox * a.stride - a.ks / 2;
        base[nt] = (uint32_t)(img - img0) * (uint32_t)img_elems + (uint32_t)(iy * a.w) + (uint32_t)ix0[nt] + (uint32_t)(a.c_in > 1 ? half * hw : 0);
        obase[nt] = ok ? img * a.c_out * a.out_h * a.out_w + opix : -1;
    }
    k5_f16 acc[MT][NT];                                         // the first reduction share starts from the bias
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const k5_f16 b = k5_bias(a.bias + (ft * MT + mt) * 32 + half * 4, wk == 0);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = b;
    }

    const int u0 = (int)((int64_t)a.units * wk / WK), u1 = (int)((int64_t)a.units * (wk + 1) / WK);
    const float* wbase = a.wpk + ((int64_t)ft * MT * a.units) * 256 + lane * 4;
    const uint32_t plane = (uint32_t)(hw * 4);
    const int last_pair = a.c_in >= 2 ? a.c_in - 2 : 0;
    int tap = u0 / a.groups, g = u0 - tap * a.groups;           // of the unit to load next
    uint32_t voff[NT];
    auto set_tap = [&]() {
        const int r = tap / a.ks, c = tap - r * a.ks;
        const uint32_t d = (uint32_t)(r * a.w + c);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const bool in = (unsigned)(iy0[nt] + r) < (unsigned)a.h && (unsigned)(ix0[nt] + c) < (unsigned)a.w;
            voff[nt] = in ? (base[nt] + d) * 4u : kK5Outside;
        }
    };
    constexpr int D = kK5Ahead + 1;
    k5_f4 wv[D][MT];
    float xv[D][NT][4];
    // the loads of one unit, one by one: weights first, then pair by pair the pixels
    constexpr int NL = MT + 4 * NT, NM = 4 * MT * NT;
    auto load_slot = [&](int set, int u, int i) {
        if (i < MT) {
            wv[set][i] = *reinterpret_cast<const k5_f4*>(wbase + ((int64_t)i * a.units + u) * 256);
        } else {
            const int p = (i - MT) / NT, nt = (i - MT) % NT;
            // pairs past the last channel read the last pair again: their weights are zeros
            const int ch = 8 * g + 2 * p < last_pair ? 8 * g + 2 * p : last_pair;
            xv[set][nt][p] = k5_load(xr, voff[nt], (uint32_t)ch * plane);
        }
    };
    auto next_unit = [&]() {
        if (++g == a.groups) {
            g = 0;
            ++tap;
            set_tap();
        }
    };
    auto load = [&](int set, int u) {
#pragma unroll
        for (int i = 0; i < NL; ++i) load_slot(set, u, i);
        next_unit();
    };
    auto multiply = [&](int set, auto&& between) {
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    acc[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[set][mt][p], xv[set][nt][p], acc[mt][nt], 0, 0, 0);
                    between((p * MT + mt) * NT + nt);
                }
    };
    // Loads run kK5Ahead units ahead, past the end too (padded weights, pixels inside x or outside the buffer): the loop
    // has no branch, so the compiler's wait counts let the younger loads stay in flight.  They are dealt out between the
    // MFMAs: issued in a block ahead of them, two and more wavefronts on a SIMD got in each other's way (a loop of 16 MFMAs
    // and 8 loads: 85 to 102 TFLOP/s in blocks, 130 dealt out, 155 without loads).
    set_tap();
#pragma unroll
    for (int d = 0; d < D - 1; ++d) load(d, u0 + d);
    __builtin_amdgcn_sched_barrier(0);
    int u = u0;
#pragma unroll 1
    for (; u + D <= u1; u += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            multiply(d, [&](int q) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = q * NL / NM; i < (q + 1) * NL / NM; ++i) load_slot((d + D - 1) % D, u + d + D - 1, i);
                __builtin_amdgcn_sched_barrier(0);
            });
            next_unit();
        }
    }
#pragma unroll
    for (int d = 0; d < D - 1; ++d)
        if (u + d < u1) multiply(d, [](int) {});

    // ---- epilogue: sum the reduction shares, bias, ReLU, pool, store (32 consecutive pixels of one filter per half wavefront) ----
    constexpr int R = 16 / WK;
    float* red = red_all + wp * (WK * 16 * 64);
    const int oplane = a.out_h * a.out_w;
    uint32_t again = 0;                                         // bit mt NT + nt: the lane's outputs of that tile
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            float v[R];
            k5_reduce<WK>(acc[mt][nt], red, wk, lane, v);
            const int co0 = (ft * MT + mt) * 32 + half * 4;
            if (k5_not_finite(v)) again |= 1u << (mt * NT + nt);
            if (a.relu) {
#pragma unroll
                for (int i = 0; i < R; ++i) v[i] = v[i] > 0.0f ? v[i] : 0.0f;
            }
            if (a.pool) {                                       // lanes 4 q .. 4 q + 3 hold one window
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    v[i] = __builtin_fmaxf(v[i], __shfl_xor(v[i], 1));
                    v[i] = __builtin_fmaxf(v[i], __shfl_xor(v[i], 2));
                }
            }
            if (obase[nt] >= 0 && (!a.pool || (lane & 3) == 0)) {
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    const int reg = wk * R + i, co = co0 + (reg >> 2) * 8 + (reg & 3);
                    if (co < a.c_out) a.y[obase[nt] + co * oplane] = v[i];
                }
            }
        }
    if (__builtin_amdgcn_ballot_w64(again != 0) == 0) return;
    if (a.pool) {                                               // any of a window's four
        again |= (uint32_t)__shfl_xor((int)again, 1);
        again |= (uint32_t)__shfl_xor((int)again, 2);
        if (lane & 3) again = 0;
    }
#pragma unroll 1
    for (int e = 0; e < MT * NT * R; ++e) {
        const int tile = e / R, reg = wk * R + e % R;
        const int j = j0 + tile % NT * 32 + col, co = (ft * MT + tile / NT) * 32 + half * 4 + (reg >> 2) * 8 + (reg & 3);
        if (((again >> tile) & 1u) && j < a.pix && co < a.c_out) {
            const int img = j / ohw, opix = a.pool ? (j - img * ohw) >> 2 : j - img * ohw, sy = opix / a.out_w;
            k0_again(a.lists, a.x, a.y, img, co, sy, opix - sy * a.out_w);
        }
    }
}

// Block-pruned product, binary32: a 32-row tile of the weight matrix with its own compact column list.  The B operand
// gathers rows of x: lane (column lane % 32, half lane / 32) of MFMA p of a group of eight list entries reads entry
// 2 p + half.  The list is stored so that a lane fetches its four entries of a group with one 16-byte load.  Entry -1 is no
// column: its row offset is 2^32 less a row, with the lane's column in [2^32 - row, 2^32), beyond any buffer, so it reads 0
// and an infinite or NaN x does not meet the padding's zero weights.
struct K5ListArgs {
    const float* x;             // [k][n]
    const float* wpk;           // [group][64 lanes][4]
    const float* bias;          // [tiles * 32]
    const int32_t* list;        // [group][half][4] columns
    const int32_t* group_off;   // [tiles + 1]
    float* y;                   // [m][n]
    int32_t m, n, row_tiles, col_tiles, items, per_xcd, relu;
    int64_t x_bytes;
};

template <int NT, int WK>
__global__ __launch_bounds__(64 * WK) __attribute__((amdgpu_waves_per_eu(WK == 16 ? 4 : 2))) void k5_list_f32(const K5ListArgs a) {
    __shared__ float red[WK > 1 ? WK * 16 * 64 : 1];
    const int lane = (int)(threadIdx.x & 63u), wk = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int col = lane & 31, half = lane >> 5;
    const int item = (int)(blockIdx.x & 7u) * a.per_xcd + (int)(blockIdx.x >> 3);
    if (item >= a.items) return;
    const int ct = item / a.row_tiles, rt = item - ct * a.row_tiles;
    const int g0 = a.group_off[rt], ng = a.group_off[rt + 1] - g0;
    const int u0 = g0 + (int)((int64_t)ng * wk / WK), u1 = g0 + (int)((int64_t)ng * (wk + 1) / WK);
    const __amdgpu_buffer_rsrc_t xr = k5_buffer(a.x, a.x_bytes);
    uint32_t jb[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int j = (ct * NT + nt) * 32 + col;
        jb[nt] = j < a.n ? (uint32_t)j * 4u : kK5Outside;       // a row offset is below 2^31: the sum stays outside
    }
    const uint32_t row_bytes = (uint32_t)a.n * 4u;
    k5_f16 acc[NT];
    {
        const k5_f16 b = k5_bias(a.bias + rt * 32 + half * 4, wk == 0);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[nt] = b;
    }
    constexpr int D = kK5Ahead + 1;
    k5_f4 wv[D];
    float xv[D][NT][4];
    int4 cols[D];
    auto load_list = [&](int set, int u) { cols[set] = *reinterpret_cast<const int4*>(a.list + (int64_t)u * 8 + half * 4); };
    constexpr int NL = 2 + 4 * NT, NM = 4 * NT;
    uint32_t ro[4];
    auto load_slot = [&](int set, int u, int i) {
        if (i == 0) {
            ro[0] = (uint32_t)cols[set].x * row_bytes, ro[1] = (uint32_t)cols[set].y * row_bytes;
            ro[2] = (uint32_t)cols[set].z * row_bytes, ro[3] = (uint32_t)cols[set].w * row_bytes;
            load_list(set, u + D);                              // as far ahead as the loads it is for: waiting for it leaves them in flight
        } else if (i == 1) {
            wv[set] = *reinterpret_cast<const k5_f4*>(a.wpk + (int64_t)u * 256 + lane * 4);
        } else {
            const int p = (i - 2) / NT, nt = (i - 2) % NT;
            xv[set][nt][p] = k5_load(xr, ro[p] + jb[nt], 0u);
        }
    };
    auto load = [&](int set, int u) {
#pragma unroll
        for (int i = 0; i < NL; ++i) load_slot(set, u, i);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto multiply = [&](int set, auto&& between) {
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                acc[nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[set][p], xv[set][nt][p], acc[nt], 0, 0, 0);
                between(p * NT + nt);
            }
    };
#pragma unroll
    for (int d = 0; d < D; ++d) load_list(d, u0 + d);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int d = 0; d < D - 1; ++d) load(d, u0 + d);
    __builtin_amdgcn_sched_barrier(0);
    int u = u0;
#pragma unroll 1
    for (; u + D <= u1; u += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            multiply(d, [&](int q) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = q * NL / NM; i < (q + 1) * NL / NM; ++i) load_slot((d + D - 1) % D, u + d + D - 1, i);
                __builtin_amdgcn_sched_barrier(0);
            });
        }
    }
#pragma unroll
    for (int d = 0; d < D - 1; ++d)
        if (u + d < u1) multiply(d, [](int) {});
    constexpr int R = 16 / WK;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        float v[R];
        k5_reduce<WK>(acc[nt], red, wk, lane, v);
        const int j = (ct * NT + nt) * 32 + col;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int reg = wk * R + i, row = rt * 32 + (reg >> 2) * 8 + half * 4 + (reg & 3);
            float o = v[i];
            if (a.relu) o = o > 0.0f ? o : 0.0f;
            if (row < a.m && j < a.n) a.y[(int64_t)row * a.n + j] = o;
        }
    }
}

typedef void (*k5_conv_fn)(K5ConvArgs);
typedef void (*k5_list_fn)(K5ListArgs);
k5_conv_fn k5_conv_lookup(const K5Shape& s);
k5_list_fn k5_list_lookup(const K5Shape& s);

}  // namespace ppc
