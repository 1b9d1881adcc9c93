// Binary32 pattern-pruned 3x3 convolution, stride 1, on the small matrix instruction v_mfma_f32_4x4x1_16b_f32 (gfx950).
//
// That instruction multiplies four filters' weights of one (channel, tap) by the inputs of 64 pixels in 8 cycles -- twice
// the rate of four vector multiply-adds and a binary32 fused multiply-add for every element.  Four filters are few enough
// for the sparsity to pay: at half the kernels kept with four of nine taps, 63 % of the (channel, tap) pairs are used by
// any of four filters (44 % at three kernels in ten), against all of them for the 32 filters of the wide instruction.
//
//   * A wavefront owns 16 filters (four quads) x 256 pixels: a lane holds four neighbouring pixels of a row, so that a
//     channel's window is three rows of six values in registers and every tap is a static choice among them; 64
//     accumulators.  Per channel and quad a 9-bit mask says which taps any of its filters uses: a scalar branch around
//     four instructions each.
//   * The weights of a channel are three registers: the instruction takes the four values of a (quad, tap) from one
//     16-byte block of a register and broadcasts them (cbsz = 4, abid = block), 16 of the 36 to a register.
//   * A lane loads its pixels of a row with one 16-byte load; the neighbours left and right come from the next lanes (DPP),
//     except across the wavefront's ends (one-lane loads) and the image's edge (zero).  Rows and lanes outside the image
//     have offsets beyond the buffer, which load as zero.
//   * The WK wavefronts of a workgroup split the channels and are summed through LDS in order.
//
// What binds: the matrix cores are busy 45 % of SIMD time (256 channels, 14x14, batch 32: 68.7 us) and 40 % (56x56, batch 1,
// one workgroup to most compute units: 27.3 us); the rest is the branches (some 30 cycles when one is taken, hidden only as
// far as there are other wavefronts) and the window's preparation.  Two rows per lane (128 accumulators) halved both per
// pixel but left two wavefronts on a SIMD: no gain.  Wavefronts sharing their pixels instead of splitting channels, and
// loads two channels ahead: slower.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "k5_f32.hpp"

namespace ppc {

struct K6Args {
    const float* x;
    float* y;
    const float* wpk;       // [16-filter group][c_in][64 lanes][4]: value v < 3 of lane 4 b + i: filter 4 q + i at tap t, 9 q + t = 16 v + b
    const uint32_t* used;   // [group][c_in][2]: bit t of quad 0 | bit 9 + t of quad 1; quads 2 and 3
    const float* bias;      // [groups * 16]
    int32_t n, c_in, c_out, h, w;
    int32_t mc;             // four-pixel pieces of a row
    int32_t pieces;         // n * h * mc
    int32_t fgroups, items, per_xcd, relu;
    int64_t x_bytes;
    const K0Args* lists;    // (in device memory) for outputs whose sum is not finite: a tap that only some of a quad's filters use is a zero weight of the others
};

typedef const __attribute__((address_space(4))) uint32_t* k6_const_u32;

// the buffer from a channel on, which a row's last load, past the row's end, needs
__device__ __forceinline__ __amdgpu_buffer_rsrc_t k6_channel(const void* base, uint32_t records) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)records, 0x00027000);
}
__device__ __forceinline__ k5_f4 k6_load4(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    return __builtin_bit_cast(k5_f4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, 0));
}

// Two rows at once: lane i <- v of lane i - 1 (left) or i + 1 (right), or e where the lane's bit of `edge` is set.
__device__ __forceinline__ void k6_from_left(float& d0, float& d1, float v0, float v1, float e0, float e1, uint64_t edge) {
    asm("s_nop 1\n\ts_mov_b64 vcc, %6\n\t"
        "v_cndmask_b32_dpp %0, %2, %4, vcc wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"
        "v_cndmask_b32_dpp %1, %3, %5, vcc wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:0"
        : "=&v"(d0), "=&v"(d1) : "v"(v0), "v"(v1), "v"(e0), "v"(e1), "s"(edge) : "vcc");
}
__device__ __forceinline__ void k6_from_right(float& d0, float& d1, float v0, float v1, float e0, float e1, uint64_t edge) {
    asm("s_nop 1\n\ts_mov_b64 vcc, %6\n\t"
        "v_cndmask_b32_dpp %0, %2, %4, vcc wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"
        "v_cndmask_b32_dpp %1, %3, %5, vcc wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:0"
        : "=&v"(d0), "=&v"(d1) : "v"(v0), "v"(v1), "v"(e0), "v"(e1), "s"(edge) : "vcc");
}

// BOUND: a wavefront's 64 pieces do not begin and end with rows (64 is no multiple of mc).  RAGGED: w is no multiple of 4.
template <bool BOUND, bool RAGGED, int WK>
__global__ __launch_bounds__(64 * WK) __attribute__((amdgpu_waves_per_eu(4))) void k6_f32_3x3(const K6Args a) {
    __shared__ float red[WK * 16 * 64];
    constexpr int RW = 3;                                           // rows of a window
    const int lane = (int)(threadIdx.x & 63u), wk = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // each XCD takes a contiguous range of items, filter groups fastest: the workgroups sharing an L2 read the same pixels
    const int item = (int)(blockIdx.x & 7u) * a.per_xcd + (int)(blockIdx.x >> 3);
    if (item >= a.items) return;
    const int fg = item % a.fgroups, pt = item / a.fgroups;
    const int hw = a.h * a.w, per_img = a.h * a.mc;
    const int j = pt * 64 + lane, img0 = pt * 64 / per_img;
    const int img = j / per_img, rem = j - img * per_img, oy = rem / a.mc, col = rem - oy * a.mc;
    const bool ok = j < a.pieces;
    const int64_t img_elems = (int64_t)a.c_in * hw;
    const __amdgpu_buffer_rsrc_t xr = k5_buffer(a.x + img0 * img_elems, a.x_bytes - img0 * img_elems * 4);
    const uint32_t records = buffer_records(a.x_bytes - img0 * img_elems * 4);
    uint32_t voff[RW], voff_l[BOUND ? RW : 1], voff_r[BOUND ? RW : 1];
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const bool in = ok && (unsigned)(oy + r - 1) < (unsigned)a.h;
        const uint32_t at = ((uint32_t)(img - img0) * (uint32_t)img_elems + (uint32_t)((oy + r - 1) * a.w) + (uint32_t)(4 * col)) * 4u;
        voff[r] = in ? at : kK5Outside;
        if constexpr (BOUND) {
            voff_l[r] = in && lane == 0 && col > 0 ? at - 4u : kK5Outside;
            voff_r[r] = in && lane == 63 && col + 1 < a.mc ? at + 16u : kK5Outside;
        }
    }
    const uint64_t first = __builtin_amdgcn_ballot_w64(col == 0) | 1ull, last = __builtin_amdgcn_ballot_w64(col + 1 == a.mc) | (1ull << 63);
    const bool tail = RAGGED && col + 1 == a.mc;                    // its values from w % 4 on belong to the next row
    const int keep = a.w & 3;

    k5_f4 acc[4][4];                                                // [quad][pixel]: four filters
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const k5_f4 b = wk == 0 ? *reinterpret_cast<const k5_f4*>(a.bias + fg * 16 + q * 4) : k5_f4(0.0f);
#pragma unroll
        for (int p = 0; p < 4; ++p) acc[q][p] = b;
    }
    const int c0 = a.c_in * wk / WK, c1 = a.c_in * (wk + 1) / WK;
    const float* wbase = a.wpk + (int64_t)fg * a.c_in * 256 + lane * 4;
    const k6_const_u32 ubase = (k6_const_u32)(uintptr_t)(a.used + (int64_t)fg * a.c_in * 2);
    const uint32_t plane = (uint32_t)(hw * 4);

    struct Chan {
        k5_f4 w, mid[RW];
        float el[RW], er[RW];
        uint32_t used[2];
    } ch[2];
    constexpr int NL = 1 + RW * (BOUND ? 3 : 1);
    auto load_slot = [&](Chan& k, int c, int i) {                   // c beyond the share: the last channel again (its masks are cleared)
        const int cc = c < a.c_in ? c : a.c_in - 1;
        if (i == 0) k.w = *reinterpret_cast<const k5_f4*>(wbase + (int64_t)cc * 256);
        else if (RAGGED && i <= RW) k.mid[i - 1] = k6_load4(k6_channel(a.x + img0 * img_elems + (int64_t)cc * hw, buffer_records_from(records, (uint32_t)cc * plane)), voff[i - 1], 0u);
        else if (i <= RW) k.mid[i - 1] = k6_load4(xr, voff[i - 1], (uint32_t)cc * plane);
        else if (BOUND && i <= 2 * RW) k.el[i - 1 - RW] = k5_load(xr, voff_l[BOUND ? i - 1 - RW : 0], (uint32_t)cc * plane);
        else if (BOUND && i <= 3 * RW) k.er[i - 1 - 2 * RW] = k5_load(xr, voff_r[BOUND ? i - 1 - 2 * RW : 0], (uint32_t)cc * plane);
    };
    auto load_used = [&](Chan& k, int c) {
        const int cc = c < a.c_in ? c : a.c_in - 1;
        const bool on = c < c1;
        const uint32_t u0 = ubase[2 * cc], u1 = ubase[2 * cc + 1];
        k.used[0] = on ? u0 : 0u, k.used[1] = on ? u1 : 0u;
    };
    // one channel: multiply k's window while the loads of channel cn arrive in nx
    auto step = [&](Chan& k, Chan& nx, int cn) {
        float left[RW + 1], right[RW + 1];
        if constexpr (RAGGED) {
#pragma unroll
            for (int r = 0; r < RW; ++r)
#pragma unroll
                for (int e = 1; e < 4; ++e) k.mid[r][e] = tail && e >= keep ? 0.0f : k.mid[r][e];
        }
#pragma unroll
        for (int r = 0; r < RW; r += 2) {
            const int s = r + 1 < RW ? r + 1 : r;
            k6_from_left(left[r], left[r + 1], k.mid[r].w, k.mid[s].w, BOUND ? k.el[r] : 0.0f, BOUND ? k.el[s] : 0.0f, first);
            k6_from_right(right[r], right[r + 1], k.mid[r].x, k.mid[s].x, BOUND ? k.er[r] : 0.0f, BOUND ? k.er[s] : 0.0f, last);
        }
        __builtin_amdgcn_sched_barrier(0);                          // the window is complete: only now the next channel's loads
        load_used(nx, cn);
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                const int kr = 9 * q + t;
                if (kr < NL) load_slot(nx, cn, kr);
                __builtin_amdgcn_sched_barrier(0);
                if ((k.used[q >> 1] >> (9 * (q & 1) + t)) & 1u) {
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        const int r = t / 3, cc = p + t % 3 - 1;
                        const float b = cc < 0 ? left[r] : cc > 3 ? right[r] : k.mid[r][cc < 0 ? 0 : cc > 3 ? 3 : cc];
                        // the block number is an immediate
#define PPC_K6(N) case N: acc[q][p] = __builtin_amdgcn_mfma_f32_4x4x1f32(k.w[kr / 16], b, acc[q][p], 4, N, 0); break;
                        switch (kr % 16) {
                            PPC_K6(0) PPC_K6(1) PPC_K6(2) PPC_K6(3) PPC_K6(4) PPC_K6(5) PPC_K6(6) PPC_K6(7)
                            PPC_K6(8) PPC_K6(9) PPC_K6(10) PPC_K6(11) PPC_K6(12) PPC_K6(13) PPC_K6(14) PPC_K6(15)
                        }
#undef PPC_K6
                    }
                }
            }
    };
#pragma unroll
    for (int i = 0; i < NL; ++i) load_slot(ch[0], c0, i);
    load_used(ch[0], c0);
#pragma unroll 1
    for (int c = c0; c < c1; c += 2) {
        step(ch[0], ch[1], c + 1);
        step(ch[1], ch[0], c + 2);
    }

    // ---- epilogue, quad by quad: sum the channel shares, ReLU, 16-byte stores (1 KB of one filter per wavefront) ----
    constexpr int R = 16 / WK;                                      // sums a wavefront finishes per lane: values 4 i + p (filter i, pixel p) from wk R on
    const int64_t obase = (int64_t)img * a.c_out * hw + oy * a.w + 4 * col;
    const int left_px = a.w - 4 * col;                              // pixels of the piece inside the row: at least 1
    uint32_t again = 0;                                             // bit q: the lane's outputs of that quad
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 16; ++e) red[(wk * 16 + e) * 64 + lane] = acc[q][e & 3][e >> 2];
        __syncthreads();
        float v[R];
#pragma unroll
        for (int e = 0; e < R; ++e) {
            float s = red[(wk * R + e) * 64 + lane];
#pragma unroll
            for (int k = 1; k < WK; ++k) s += red[(k * 16 + wk * R + e) * 64 + lane];
            v[e] = s;
        }
        if (k5_not_finite(v)) again |= 1u << q;
#pragma unroll
        for (int e = 0; e < R; ++e) v[e] = a.relu && !(v[e] > 0.0f) ? 0.0f : v[e];
        const int val = wk * R, co = fg * 16 + q * 4 + (val >> 2);
        if (!ok || co >= a.c_out) continue;
        float* dst = a.y + obase + (int64_t)co * hw + (val & 3);
        if constexpr (R == 4 && !RAGGED) {
            k5_f4 o;
            o.x = v[0], o.y = v[1], o.z = v[2], o.w = v[3];
            *reinterpret_cast<k5_f4*>(dst) = o;
        } else {
#pragma unroll
            for (int p = 0; p < R; ++p)
                if ((val & 3) + p < left_px) dst[p] = v[p];
        }
    }
    if (__builtin_amdgcn_ballot_w64(again != 0) == 0) return;
#pragma unroll 1
    for (int e = 0; e < 4 * R; ++e) {
        const int q = e / R, val = wk * R + e % R, co = fg * 16 + q * 4 + (val >> 2), px = val & 3;
        if (((again >> q) & 1u) && ok && co < a.c_out && px < left_px) k0_again(a.lists, a.x, a.y, img, co, oy, 4 * col + px);
    }
}

typedef void (*k6_fn)(K6Args);
// The kernel with wk wavefronts (4, 8 or 16) on a tile's channels.
k6_fn k6_lookup(int wk, bool bound, bool ragged);

}  // namespace ppc
