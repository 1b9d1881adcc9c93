// Matrix-core kernels for binary32 storage (gfx950): any convolution (kernel size, stride, fused 2x2 max-pool) and the
// block-pruned product.
//
// Convolution (k5_conv_f32): the pruned weights are zero-filled to a dense matrix (a 32-filter tile uses every (channel, tap) pair at
// the densities that pattern pruning leaves) and multiplied on the bfloat16 matrix instruction, which is sixteen times as fast as the
// binary32 one (32 x 32 x 16 in 32 cycles; the method is that of Henry, Tang and Heinecke, arXiv:1904.06376).  Every value is the sum of three bfloat16 parts, x1 + x2 + x3, exactly, if its last bit is not
// below bfloat16's smallest value, 2^-133: x is therefore scaled by 2^16 (sums from 2^112 on overflow and are summed again from the kernel lists), and layers
// with a weight that is not the sum of its parts (one below 2^-109 may not be) run on the binary32 instruction.  Of the nine products
// of parts the six down to 2^-16 are taken: what the other three leave out is at most a relative 2^-24.  x1 w1 has an accumulator of its own,
// rounded once per sixteen products, the small ones another at a 256th of its size: against 64 bits sums of eight or more products are
// as near as those of the binary32 instruction or nearer (relative error 1.06e-7 against 2.85e-7 over 2304 terms, 2.9e-8 against 5.4e-8
// over 64, 4.2e-8 against 4.3e-8 over 8 with a bias; all six in one accumulator would be 5.1e-7 over 2304).  Below that they are not (4.0e-8
// against 2.5e-8 for one product and a bias): such layers stay on the binary32 instruction (k5_parts_near).
// 256 channels, 14x14, 3x3, batch 32: 75 us on the binary32 instruction, 42.6 in parts, 41.6 without the scaling.
//
// Per lane and unit (one tap x sixteen channels) the operand of x is eight values of one output pixel: plain loads, a lane's offset
// changing with the tap only; the channel is the scalar offset of a buffer load, and a tap that falls outside the image gives the lane
// an offset beyond the buffer, which loads as zero.  The wavefront scales and splits them (13 vector instructions for two values) and uses each
// part for 32 mt filters.  Weights come as ready operands, 3 KB per tile and unit, through a ring of three buffers in LDS by direct
// loads, shared by the WP wavefronts of a reduction share; WK shares are summed through LDS in order.  What bounds it is that vector
// and matrix instructions of a wavefront overlap only when dealt out among each other: with loads, splitting and weight reads in
// blocks between groups of four matrix instructions the 14x14 layer took 49 us, one by one behind each instruction 41.  Order of
// units: taps fastest, so that the nine loads of a pixel's neighbourhood meet the vector cache.
//
// A pruned tap is a zero weight here, and 0 x Inf is NaN where the definition skips the tap.  Outputs whose dense sum is not
// finite are therefore summed again from the kernel lists (k0_again); finite inputs pay one multiply-add per output for the test.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "buffer_rules.hpp"
#include "f32_rules.hpp"
#include "k0_generic.hpp"
#include "lds_loads.hpp"

namespace ppc {

struct K5ConvArgs {
    const float* x;
    const void* wpk;        // [32-filter tile][unit][3 parts][64 lanes][8] bfloat16: lane l, value i: filter l % 32, the channel at (g, l / 32, i) (k5_slot) of unit (g, tap)
    const float* bias;      // [tiles * 32]
    float* y;
    int32_t n, c_in, c_out, h, w, ho, wo, out_h, out_w;
    int32_t ks, stride, pool, relu;
    int32_t groups, units;  // groups of sixteen channels (eight for k5_whole_f32), ks * ks * groups
    int32_t pix;            // n * ho * wo convolution outputs
    int32_t ftiles, ptiles, items, per_xcd;
    int32_t pixels_inner;   // order of the items: pixel tiles fastest, or filter tiles
    int64_t x_bytes;
    const K0Args* lists;    // in device memory; its x, y and n are not set
};

typedef float k5_f16 __attribute__((ext_vector_type(16)));
typedef float k5_f4 __attribute__((ext_vector_type(4)));
typedef float k5_f2 __attribute__((ext_vector_type(2)));
typedef __bf16 k5_b2 __attribute__((ext_vector_type(2)));
typedef __bf16 k5_b8 __attribute__((ext_vector_type(8)));
typedef uint32_t k5_u4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) unsigned char* k5_lds_ptr;

constexpr float kK5Scale = 65536.0f;               // of x ahead of its splitting
constexpr int kK5Ahead = 3;                        // reduction units whose loads are in flight behind the one being multiplied
constexpr uint32_t kK5Outside = 0x80000000u;      // a byte offset no buffer of these kernels reaches: the load returns 0

__device__ __forceinline__ __amdgpu_buffer_rsrc_t k5_buffer(const void* base, int64_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)buffer_records(bytes), 0x00027000);
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

template <int N, typename F, int I = 0>
__device__ __forceinline__ void k5_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        k5_for<N, F, I + 1>(static_cast<F&&>(f));
    }
}

// Two binary32 values as three pairs of bfloat16 parts, each part the rounding of what the parts before it leave: together they are
// the values themselves.  In five slices, behind that of the scaling, to be issued between matrix instructions.
template <int SLICE>
__device__ __forceinline__ void k5_split_slice(float& a, float& b, uint32_t (&part)[3]) {
    if constexpr (SLICE % 2 == 0) {
        part[SLICE / 2] = __builtin_bit_cast(uint32_t, __builtin_convertvector(k5_f2{a, b}, k5_b2));
    } else {
        a -= __builtin_bit_cast(float, part[SLICE / 2] << 16);
        b -= __builtin_bit_cast(float, part[SLICE / 2] & 0xFFFF0000u);
    }
}

// A lane's output pixel: image row / column of the first tap, offset of that tap (in elements) from the first image of the tile, plane
// offset of the output from the tensor's start (-1: none).
struct K5Pixel {
    int iy0, ix0, obase;
    uint32_t base;
};
__device__ __forceinline__ K5Pixel k5_pixel(const K5ConvArgs& a, int j, int img0, int first) {
    const int ohw = a.ho * a.wo, img = j / ohw, rem = j - img * ohw;
    int oy, ox, opix;
    if (a.pool) {                                               // four consecutive pixels are one pooling window
        const int q = rem >> 2, py = q / a.out_w, px = q - py * a.out_w;
        oy = 2 * py + ((rem >> 1) & 1), ox = 2 * px + (rem & 1);
        opix = q;
    } else {
        oy = rem / a.wo, ox = rem - oy * a.wo;
        opix = rem;
    }
    const bool ok = j < a.pix;
    const int iy = oy * a.stride - a.ks / 2;
    K5Pixel p;
    p.iy0 = ok ? iy : -1000000;                                 // no tap of a pixel past the end is inside an image
    p.ix0 = ox * a.stride - a.ks / 2;
    p.base = (uint32_t)(img - img0) * (uint32_t)(a.c_in * a.h * a.w) + (uint32_t)(iy * a.w) + (uint32_t)p.ix0 + (uint32_t)first;
    p.obase = ok ? img * a.c_out * a.out_h * a.out_w + opix : -1;
    return p;
}

// ReLU, pool and stores of registers [reg0, reg0 + R) of a tile whose register 0 is filter co0 of this lane: 32 consecutive pixels of one
// filter per half wavefront.
template <int R>
__device__ __forceinline__ void k5_store(const K5ConvArgs& a, float (&v)[R], int co0, int reg0, int obase, int lane) {
    if (a.relu) {
#pragma unroll
        for (int i = 0; i < R; ++i) v[i] = v[i] > 0.0f ? v[i] : 0.0f;
    }
    if (a.pool) {                                               // lanes 4 q .. 4 q + 3 hold one window
#pragma unroll
        for (int i = 0; i < R; ++i) {
            v[i] = __builtin_fmaxf(v[i], __shfl_xor(v[i], 1));
            v[i] = __builtin_fmaxf(v[i], __shfl_xor(v[i], 2));
        }
    }
    if (obase >= 0 && (!a.pool || (lane & 3) == 0)) {
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int reg = reg0 + i, co = co0 + (reg >> 2) * 8 + (reg & 3);
            if (co < a.c_out) a.y[obase + co * a.out_h * a.out_w] = v[i];
        }
    }
}

// Sums the outputs of the lane's pixel j again that were not finite: bit t of `again` stands for registers [reg0, reg0 + R) of tile
// ft0 + t.
template <int R>
__device__ __forceinline__ void k5_redo(const K5ConvArgs& a, uint32_t again, int tiles, int ft0, int j, int reg0, int half, int lane) {
    if (__builtin_amdgcn_ballot_w64(again != 0) == 0) return;
    if (a.pool) {                                               // any of a window's four
        again |= (uint32_t)__shfl_xor((int)again, 1);
        again |= (uint32_t)__shfl_xor((int)again, 2);
        if (lane & 3) again = 0;
    }
    const int ohw = a.ho * a.wo;
#pragma unroll 1
    for (int e = 0; e < tiles * R; ++e) {
        const int t = e / R, reg = reg0 + e % R, co = (ft0 + t) * 32 + half * 4 + (reg >> 2) * 8 + (reg & 3);
        if (((again >> t) & 1u) && j < a.pix && co < a.c_out) {
            const int img = j / ohw, opix = a.pool ? (j - img * ohw) >> 2 : j - img * ohw, sy = opix / a.out_w;
            k0_again(a.lists, a.x, a.y, img, co, sy, opix - sy * a.out_w);
        }
    }
}

template <int MT, int WP, int WK>
__global__ __launch_bounds__(64 * WK * WP) __attribute__((amdgpu_waves_per_eu(WK * WP == 16 ? 4 : 2))) void k5_conv_f32(const K5ConvArgs a) {
    constexpr int FR = 3 * MT;                                  // weight fragments of 1 KB in a unit
    constexpr int RING = 3;
    extern __shared__ __align__(16) unsigned char k5_smem[];    // [RING][WK][FR] fragments; at the end the shares' sums
    const int lane = (int)(threadIdx.x & 63u), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wp = wave % WP, wk = wave / WP;
    const int col = lane & 31, half = lane >> 5;
    // Workgroup ids go round-robin to the 8 XCDs: each takes a contiguous range of items, filter tiles fastest, so that the
    // workgroups sharing an L2 read the same pixels, or pixel tiles fastest, so that they read the same weights.
    const int item = (int)(blockIdx.x & 7u) * a.per_xcd + (int)(blockIdx.x >> 3);
    if (item >= a.items) return;
    const int inner = a.pixels_inner ? a.ptiles : a.ftiles, outer_i = item / inner, inner_i = item - outer_i * inner;
    const int ft = a.pixels_inner ? outer_i : inner_i, pt = a.pixels_inner ? inner_i : outer_i;
    const int j0 = (pt * WP + wp) * 32;                         // first pixel of this wavefront
    const int hw = a.h * a.w, ohw = a.ho * a.wo;
    const int img0 = (j0 < a.pix ? j0 : 0) / ohw;               // wave-uniform
    const int64_t img_elems = (int64_t)a.c_in * hw;
    const __amdgpu_buffer_rsrc_t xr = k5_buffer(a.x + img0 * img_elems, a.x_bytes - img0 * img_elems * 4);

    const K5Pixel px = k5_pixel(a, j0 + col, img0, half * k5_half_channels(a.c_in) * hw);
    // The products of the leading parts have an accumulator of their own, those of the others another: the first is rounded
    // once per unit, at the size of the sum, the second at a 256th of it.
    k5_f16 acc[MT], low[MT];                                    // the first reduction share starts from the bias
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        acc[mt] = k5_bias(a.bias + (ft * MT + mt) * 32 + half * 4, wk == 0) * kK5Scale;
        low[mt] = k5_f16(0.0f);
    }

    const int n_units = (a.units + WK - 1) / WK;                // of a share; units past the end multiply zeros
    const int u0 = wk * n_units, own = a.units - u0 < n_units ? a.units - u0 : n_units;
    const uint32_t plane = (uint32_t)(hw * 4);
    int lu = 0, tr = 0, tc = 0, g = 0;                          // the unit to load next: its tap and group
    {
        const int kk = a.ks * a.ks, t = u0 % kk;
        g = u0 / kk, tr = t / a.ks, tc = t - tr * a.ks;
    }
    constexpr int XD = 4;                                       // units of x in registers or on their way
    float xv[XD][8];
    uint32_t voff = 0u, xsoff = 0u;
    // The place of the unit to load next.  Without branches: what is computed ahead between the matrix instructions would be moved
    // behind them, to the block that uses it.
    auto next_x = [&]() __attribute__((always_inline)) {
        const uint32_t at = (px.base + (uint32_t)(tr * a.w + tc)) * 4u;
        const bool in = (lu < own) & ((unsigned)(px.iy0 + tr) < (unsigned)a.h) & ((unsigned)(px.ix0 + tc) < (unsigned)a.w);
        voff = in ? at : kK5Outside;
        xsoff = (uint32_t)k5_group_first(a.c_in, g) * plane;
        ++lu;
        const int row = tc + 1 == a.ks ? 1 : 0, group = row & (tr + 1 == a.ks ? 1 : 0);
        tc = row ? 0 : tc + 1;
        tr = group ? 0 : tr + row;
        g += group;
    };
    uint32_t step_bytes[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) step_bytes[j] = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)k5_step(a.c_in, j) * plane));
    auto load_x = [&](auto set_tag, int j) __attribute__((always_inline)) { xv[decltype(set_tag)::value][j] = k5_load(xr, voff, xsoff + step_bytes[j]); };
    const uint32_t lds0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)(k5_lds_ptr)k5_smem) + (uint32_t)(wk * FR * 1024);
    int wu = 0;
    uint32_t wbuf = 0;
    const unsigned char* wsrc = nullptr;
    uint32_t wdst = 0u;
    auto next_w = [&]() __attribute__((always_inline)) {
        const int u = u0 + wu < a.units ? u0 + wu : a.units - 1;
        wsrc = static_cast<const unsigned char*>(a.wpk) + ((int64_t)ft * MT * a.units + u) * 3072;
        wdst = lds0 + wbuf * (WK * FR * 1024);
        ++wu;
        if (++wbuf == RING) wbuf = 0;
    };
    constexpr int ND = (FR + WP - 1) / WP;                      // fragments that a wavefront brings
    auto load_w = [&](int i) __attribute__((always_inline)) {
        const int f = wp + WP * i;
        if (FR % WP == 0 || f < FR) load_lds16((uint32_t)lane * 16u, uniform_address(wsrc + (int64_t)(f / 3) * a.units * 3072 + f % 3 * 1024), wdst + (uint32_t)f * 1024u);
    };
    k5_u4 xf[2][3];                                             // the parts of this unit's pixels and of the next one's
    float sa[4], sb[4];
    uint32_t part[4][3];
    auto slice = [&](auto from_tag, auto to_tag, auto k_tag) __attribute__((always_inline)) {     // slice k % 6 of pair k / 6
        constexpr int from = decltype(from_tag)::value, to = decltype(to_tag)::value, k = decltype(k_tag)::value, j = k / 6;
        if constexpr (k % 6 == 0) sa[j] = xv[from][2 * j] * kK5Scale, sb[j] = xv[from][2 * j + 1] * kK5Scale;
        else k5_split_slice<k % 6 - 1>(sa[j], sb[j], part[j]);
        if constexpr (k % 6 == 5) {
#pragma unroll
            for (int i = 0; i < 3; ++i) xf[to][i][j] = part[j][i];
        }
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;
    auto fill_x = [&](auto set_tag) __attribute__((always_inline)) {
        next_x();
#pragma unroll
        for (int j = 0; j < 8; ++j) load_x(set_tag, j);
    };
    auto fill_w = [&]() __attribute__((always_inline)) {
        next_w();
#pragma unroll
        for (int i = 0; i < ND; ++i) load_w(i);
    };
    fill_x(I0{});
    fill_w();
    fill_x(I1{});
    fill_w();
    fill_x(I2{});
    fill_w();
    fill_x(I3{});
    k5_for<24>([&](auto k) __attribute__((always_inline)) { slice(I0{}, I0{}, k); });
    // At most YOUNGER of this wavefront's loads are on their way; past the barrier every wavefront's are there that it had waited for, and
    // the buffer of the unit before is free.
    auto arrive = [&](auto younger) __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);                      // (a load moved behind the wait would be counted as one ahead of it)
        __builtin_amdgcn_s_waitcnt(wait_vmcnt(decltype(younger)::value));
        if constexpr (WP > 1) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        } else {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    k5_u4 wf[3][MT];                                            // [part][filter tile]
    const unsigned char* wl = k5_smem + wk * FR * 1024 + lane * 16;
    int rbuf = 0;
    auto read_w = [&](int part) __attribute__((always_inline)) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) wf[part][mt] = *reinterpret_cast<const k5_u4*>(wl + rbuf * (WK * FR * 1024) + (mt * 3 + part) * 1024);
    };
    arrive(std::integral_constant<int, 2 * (FR / WP)>{});
#pragma unroll
    for (int i = 0; i < 3; ++i) read_w(i);
    // A unit: six products of parts, each for all filter tiles.  Everything else is issued between the matrix instructions, a few at
    // a time: the loads of x four units ahead, the splitting of the next unit's, and past the barrier the reads of the next unit's
    // weights and the loads of those three units ahead.  The last one to three units (at most LEFT of them with this one) load
    // nothing: a wait counts loads, so it has to be known which there are.
    auto step = [&](auto u_tag, auto left_tag) __attribute__((always_inline)) {
        constexpr int U = decltype(u_tag)::value, S = U & 1, NM = 6 * MT, LEFT = decltype(left_tag)::value;
        constexpr bool loads = LEFT == 0, more = LEFT != 1;
        // younger than this wavefront's part of the next unit's weights: x of two units and the weights of the unit after it
        constexpr int younger = loads ? 16 + FR / WP : LEFT == 3 ? FR / WP : 0;
        using From = std::integral_constant<int, (U + 1) % XD>;
        using To = std::integral_constant<int, S ^ 1>;
        constexpr int wp_of[6] = {0, 0, 0, 1, 1, 2}, xp_of[6] = {1, 0, 2, 0, 1, 0};
        if constexpr (loads) next_x();
        k5_for<NM>([&](auto m_tag) __attribute__((always_inline)) {
            constexpr int m = decltype(m_tag)::value, r = m / MT, mt = m % MT;
            const k5_b8 w = __builtin_bit_cast(k5_b8, wf[wp_of[r]][mt]), x = __builtin_bit_cast(k5_b8, xf[S][xp_of[r]]);
            k5_f16& c = r == 1 ? acc[mt] : low[mt];
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, x, c, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            k5_for<8>([&](auto j) __attribute__((always_inline)) {
                if constexpr (loads && decltype(j)::value * (NM / 2) / 8 == m) load_x(u_tag, decltype(j)::value);
            });
            k5_for<24>([&](auto k) __attribute__((always_inline)) {
                if constexpr (more && decltype(k)::value * NM / 24 == m) slice(From{}, To{}, k);
            });
            if constexpr (more && m == NM / 2 - 1) {
                arrive(std::integral_constant<int, younger>{});
                if (++rbuf == RING) rbuf = 0;
                read_w(0);
                if constexpr (loads) next_w();
            }
            if constexpr (loads && m >= NM / 2) {
#pragma unroll
                for (int i = 0; i < ND; ++i)
                    if (NM / 2 + i * (NM / 2) / ND == m) load_w(i);
            }
            if constexpr (more && m == 5 * MT - 1) read_w(1);
            if constexpr (more && m == NM - 1) read_w(2);
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    int s = 0;
#pragma unroll 1
    for (; s + XD <= n_units; s += XD) {
        step(I0{}, I0{});
        step(I1{}, I0{});
        step(I2{}, I0{});
        step(I3{}, I0{});
    }
    if (s < n_units) {
        step(I0{}, I3{});
        if (s + 1 < n_units) {
            step(I1{}, I2{});
            if (s + 2 < n_units) step(I2{}, I1{});
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");            // nothing is on its way to LDS any more

    // ---- epilogue: sum the reduction shares, bias, ReLU, pool, store (32 consecutive pixels of one filter per half wavefront) ----
    constexpr int R = 16 / WK;
    float* red = reinterpret_cast<float*>(k5_smem) + wp * (WK * 16 * 64);
    uint32_t again = 0;                                         // bit mt: the lane's outputs of that tile
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        float v[R];
        k5_reduce<WK>(acc[mt] + low[mt], red, wk, lane, v);
        if (k5_not_finite(v)) again |= 1u << mt;
#pragma unroll
        for (int i = 0; i < R; ++i) v[i] *= 1.0f / kK5Scale;
        k5_store<R>(a, v, (ft * MT + mt) * 32 + half * 4, wk * R, px.obase, lane);
    }
    k5_redo<R>(a, again, MT, ft * MT, j0 + col, wk * R, half, lane);
}

// The same convolution on the binary32 matrix instruction (v_mfma_f32_32x32x2_f32): layers with few tiles, with few products to a sum, or
// with weights that are not the sums of their parts.  Operands come straight from the vector cache: 32 neighbouring pixels of a channel's row are
// 128 consecutive bytes of x.  Wavefronts of 32 MT filters x 32 NT pixels, WK of a workgroup on one tile's reduction, WP on different pixels with
// the same weights.  With few tiles what a compute unit can read is the bound, and per 16 channels and tap a wavefront reads 2 KB of weights
// here, 3 KB in parts: 120 to 131 channels, 14x23, 3x3, batch 5 takes 8.1 us, 9.4 in parts; 444 to 358, 9x14, batch 3 21.2, 23.0; with many
// the instruction's rate is: 256 channels, 14x14, batch 32: 75 us here, 42 in parts.
// Here taps are outermost: a lane's byte offset into x changes with the tap only.
template <int MT, int NT, int WK, int WP>
__global__ __launch_bounds__(64 * WK * WP) __attribute__((amdgpu_waves_per_eu(2))) void k5_whole_f32(const K5ConvArgs a) {
    __shared__ float red_all[WK > 1 ? WP * WK * 16 * 64 : 1];
    const int lane = (int)(threadIdx.x & 63u), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wk = wave % WK, wp = wave / WK;
    const int col = lane & 31, half = lane >> 5;
    const int item = (int)(blockIdx.x & 7u) * a.per_xcd + (int)(blockIdx.x >> 3);
    if (item >= a.items) return;
    const int inner = a.pixels_inner ? a.ptiles : a.ftiles, outer_i = item / inner, inner_i = item - outer_i * inner;
    const int ft = a.pixels_inner ? outer_i : inner_i, pt = a.pixels_inner ? inner_i : outer_i;
    const int j0 = (pt * WP + wp) * 32 * NT;                    // first pixel of this wavefront
    const int hw = a.h * a.w, ohw = a.ho * a.wo;
    const int img0 = (j0 < a.pix ? j0 : 0) / ohw;               // wave-uniform
    const int64_t img_elems = (int64_t)a.c_in * hw;
    const __amdgpu_buffer_rsrc_t xr = k5_buffer(a.x + img0 * img_elems, a.x_bytes - img0 * img_elems * 4);
    K5Pixel px[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) px[nt] = k5_pixel(a, j0 + nt * 32 + col, img0, a.c_in > 1 ? half * hw : 0);
    k5_f16 acc[MT][NT];                                         // the first reduction share starts from the bias
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const k5_f16 b = k5_bias(a.bias + (ft * MT + mt) * 32 + half * 4, wk == 0);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = b;
    }

    const int u0 = (int)((int64_t)a.units * wk / WK), u1 = (int)((int64_t)a.units * (wk + 1) / WK);
    const float* wbase = static_cast<const float*>(a.wpk) + (int64_t)ft * MT * a.units * 256 + lane * 4;
    const uint32_t plane = (uint32_t)(hw * 4);
    const int last_pair = a.c_in >= 2 ? a.c_in - 2 : 0;
    int tap = u0 / a.groups, g = u0 - tap * a.groups;           // of the unit to load next
    uint32_t voff[NT];
    auto set_tap = [&]() __attribute__((always_inline)) {
        const int r = tap / a.ks, c = tap - r * a.ks;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const bool in = (unsigned)(px[nt].iy0 + r) < (unsigned)a.h && (unsigned)(px[nt].ix0 + c) < (unsigned)a.w;
            voff[nt] = in ? (px[nt].base + (uint32_t)(r * a.w + c)) * 4u : kK5Outside;
        }
    };
    constexpr int D = kK5Ahead + 1;
    k5_f4 wv[D][MT];
    float xv[D][NT][4];
    // the loads of one unit, one by one: weights first, then pair by pair the pixels
    constexpr int NL = MT + 4 * NT, NM = 4 * MT * NT;
    auto load_slot = [&](int set, int u, int i) __attribute__((always_inline)) {
        if (i < MT) {
            wv[set][i] = *reinterpret_cast<const k5_f4*>(wbase + ((int64_t)i * a.units + u) * 256);
        } else {
            const int p = (i - MT) / NT, nt = (i - MT) % NT;
            // pairs past the last channel read the last pair again: their weights are zeros
            const int ch = 8 * g + 2 * p < last_pair ? 8 * g + 2 * p : last_pair;
            xv[set][nt][p] = k5_load(xr, voff[nt], (uint32_t)ch * plane);
        }
    };
    auto next_unit = [&]() __attribute__((always_inline)) {
        if (++g == a.groups) {
            g = 0;
            ++tap;
            set_tap();
        }
    };
    auto multiply = [&](int set, auto&& between) __attribute__((always_inline)) {
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
    // has no branch, so the compiler's wait counts let the younger loads stay in flight.  They are dealt out between the MFMAs: in a
    // block ahead of them, two and more wavefronts on a SIMD got in each other's way (a loop of 16 MFMAs and 8 loads: 85 to
    // 102 TFLOP/s in blocks, 130 dealt out, 155 without loads).
    set_tap();
#pragma unroll
    for (int d = 0; d < D - 1; ++d) {
#pragma unroll
        for (int i = 0; i < NL; ++i) load_slot(d, u0 + d, i);
        next_unit();
    }
    __builtin_amdgcn_sched_barrier(0);
    int u = u0;
#pragma unroll 1
    for (; u + D <= u1; u += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            multiply(d, [&](int q) __attribute__((always_inline)) {
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

    constexpr int R = 16 / WK;
    float* red = red_all + wp * (WK * 16 * 64);
    uint32_t again[NT] = {};                                    // bit mt: the lane's outputs of that tile
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            float v[R];
            k5_reduce<WK>(acc[mt][nt], red, wk, lane, v);
            if (k5_not_finite(v)) again[nt] |= 1u << mt;
            k5_store<R>(a, v, (ft * MT + mt) * 32 + half * 4, wk * R, px[nt].obase, lane);
        }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) k5_redo<R>(a, again[nt], MT, ft * MT, j0 + nt * 32 + col, wk * R, half, lane);
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
__global__ __launch_bounds__(64 * WK) __attribute__((amdgpu_waves_per_eu(2))) void k5_list_f32(const K5ListArgs a) {
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

typedef void (*k5_conv_fn)(const K5ConvArgs& a, int blocks, hipStream_t stream);
typedef void (*k5_list_fn)(K5ListArgs);
k5_conv_fn k5_conv_lookup(const K5ConvShape& s);
k5_conv_fn k5_whole_lookup(const K5Shape& s);
k5_list_fn k5_list_lookup(const K5Shape& s);

}  // namespace ppc
