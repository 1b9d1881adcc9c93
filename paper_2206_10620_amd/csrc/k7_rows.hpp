// 3x3, stride-1 layers in binary16 on the matrix cores (gfx950): row-stacked tiles with the pixels as the product's rows.
//
// The pruned weights are zero-filled to a dense product, as in the other two kernels.  What bounds those is what goes through LDS and the
// vector cache for each matrix instruction, so here a wavefront works on T rows of 32 columns and 64 filters: an x fragment (32 pixels
// x 16 channels) of one staged row and column shift serves up to three rows of outputs, 3 (T + 2) fragments for 18 T instructions.
// Pixels are the rows of the instruction's first operand: LDS holds a plane of words for each pair of channels, a pixel a word, so that a
// shift by a column is an address and a fragment four reads, without conflicts where planes are
// multiples of 256 bytes (two rows: none counted on 512 channels, 28x28; four rows: 12 % of LDS cycles on the 1080p layer).  x comes by 16-byte loads of eight pixels of a
// channel, D chunks ahead in registers, and is interleaved by pairs of channels on its way to LDS; weights lie in memory as in LDS and come by
// direct loads, at half the vector cache's time for them.  One barrier a chunk, in its last but one step.
// Measured (direct-load kernel before): 64 channels, 1080x1920: 203 -> 187 us; 3 to 64, 224x224, batch 8: 28 -> 17.7; 64 to 64 pooled:
// 39 -> 31; 512 channels, 28x28, batch 8: 50 -> 36 (822 TFLOP/s); 67 to 140, 84x90, batch 2 (general kernel before): 26 -> 12.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "buffer_rules.hpp"
#include "k7_geom.hpp"
#include "lds_loads.hpp"
#include "mfma_geom.hpp"

namespace ppc {

struct K7Args {
    const void* x;
    void* y;
    const void* wpk;            // weight fragments [fb][q][9][2][64][8] binary16
    const float* bias;          // [fb*64]
    int64_t x_bytes;
    int32_t n, c_in, c_out, h, w;
    int32_t out_h, out_w;
    int32_t po;                 // rows per image of the tall image
    int32_t tiles_x, tiles_v;
    int32_t fb, q;              // filter blocks, channel chunks
    int32_t work_items, blocks_per_xcd;
    uint32_t magic_po;
    int32_t relu;
};

typedef _Float16 k7_h8 __attribute__((ext_vector_type(8)));
typedef _Float16 k7_h2 __attribute__((ext_vector_type(2)));
typedef float k7_f16 __attribute__((ext_vector_type(16)));
typedef float k7_f4 __attribute__((ext_vector_type(4)));
typedef uint32_t k7_u4 __attribute__((ext_vector_type(4)));
typedef uint32_t k7_u2 __attribute__((ext_vector_type(2)));
typedef k7_u4 k7_u4_any __attribute__((aligned(2)));        // rows of y start on any element
typedef k7_u2 k7_u2_any __attribute__((aligned(2)));
typedef uint32_t k7_u1_any __attribute__((aligned(2)));
typedef __attribute__((address_space(3))) unsigned char* k7_lds_ptr;

constexpr uint32_t kK7Outside = 0x80000000u;      // a byte offset that no tile's buffer reaches: the load returns 0

// n / d for n < 65536 and 1 <= d < 65536 with magic = floor(2^32 / d) + 1 (0 stands for d = 1)
__device__ __forceinline__ int k7_div(int n, uint32_t magic) { return magic ? (int)__umulhi((uint32_t)n, magic) : n; }

// A barrier for LDS traffic only: loads from memory stay in flight over it.
__device__ __forceinline__ void k7_lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// x fragments read from LDS before step j of a chunk (0 to 9; fragments past the chunk's own are the next one's): what the step and
// the one behind it need, and none of the next chunk before step 7.
constexpr int k7_ahead(int t, int j) {
    constexpr int two[10] = {4, 5, 6, 8, 9, 10, 12, 12, 14, 16};
    return t == 4 ? 2 * j + 4 : two[j];
}

// Transposes 16-byte pieces between four neighbouring lanes: lane 4 a + i gets, as piece k, piece i of lane 4 a + k.
__device__ __forceinline__ void k7_transpose4(k7_u4 (&x)[4], int lane) {
#pragma unroll
    for (int step = 1; step < 4; step *= 2) {
        const bool odd = (lane & step) != 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (k & step) continue;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int a = (int)x[k][e], b = (int)x[k + step][e];
                const int da = step == 1 ? __builtin_amdgcn_mov_dpp(a, 0xB1, 0xF, 0xF, true) : __builtin_amdgcn_mov_dpp(a, 0x4E, 0xF, 0xF, true);
                const int db = step == 1 ? __builtin_amdgcn_mov_dpp(b, 0xB1, 0xF, 0xF, true) : __builtin_amdgcn_mov_dpp(b, 0x4E, 0xF, 0xF, true);
                x[k][e] = (uint32_t)(odd ? db : a);
                x[k + step][e] = (uint32_t)(odd ? b : da);
            }
        }
    }
}

// Up to eight binary16 values, `count` of them (any number) inside the row.
__device__ __forceinline__ void k7_store8(unsigned char* p, k7_u4 v, int count) {
    if (count >= 8) {
        *reinterpret_cast<k7_u4_any*>(p) = v;
    } else if (count > 0) {
        if (count & 4) {
            *reinterpret_cast<k7_u2_any*>(p) = k7_u2{v[0], v[1]};
            p += 8;
            v[0] = v[2], v[1] = v[3];
        }
        if (count & 2) {
            *reinterpret_cast<k7_u1_any*>(p) = v[0];
            p += 4;
            v[0] = v[1];
        }
        if (count & 1) *reinterpret_cast<uint16_t*>(p) = (uint16_t)v[0];
    }
}

// T: rows of a wavefront that share the x fragments of T + 2.  TC: columns of a tile.  KG: groups of four wavefronts that share a tile, each on its own half of the chunks.
template <int T, int TC, int KG, bool RAGGED, bool POOL>
__global__ __launch_bounds__(256 * KG) __attribute__((amdgpu_waves_per_eu(2, 2))) void k7_rows(const K7Args a) {
    constexpr K7Geom G = k7_geom(T, TC);
    constexpr int NX = 3 * (T + 2), RX = NX / 2;    // x fragments of a chunk, in the ring
    constexpr int D = T == 4 ? 1 : 4;               // chunks of x in registers on their way to LDS
    constexpr int SR = G.rounds, WB = G.wbufs;
    constexpr int WR = T == 4 ? 2 : 3;              // steps whose weights are in registers
    extern __shared__ __align__(16) unsigned char smem[];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane((tid >> 6) & 3), kg = KG > 1 ? __builtin_amdgcn_readfirstlane(tid >> 8) : 0;
    const int p = lane & 31, kb = lane >> 5;

    const int xcd = (int)(blockIdx.x % 8u), slot = (int)(blockIdx.x / 8u), gslots = (int)(gridDim.x / 8u);
    const int first_item = xcd * a.blocks_per_xcd;
    const int left = a.work_items - first_item, avail = left < a.blocks_per_xcd ? left : a.blocks_per_xcd;
    const int my_n = avail > slot ? (avail - slot + gslots - 1) / gslots : 0;
    if (my_n == 0) return;
    const int QN = a.q / KG;                        // chunks of a tile that this group multiplies
    const int steps = my_n * QN;                    // ... and of all its tiles

    const int hw = a.h * a.w;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(k7_lds_ptr)smem;
    const int group0 = kg * G.group;                // this group's buffers
    constexpr int tail = KG * G.group;

    struct Tile { int fbi, ox0, v0; };
    auto decode = [&](int k) __attribute__((always_inline)) {
        int item = first_item + slot + k * gslots;
        Tile t;
        t.fbi = item % a.fb;
        item /= a.fb;
        t.ox0 = (item % a.tiles_x) * TC;
        t.v0 = (item / a.tiles_x) * G.tr;
        return t;
    };

    // ---- staging of x: a lane fetches eight pixels of the four channels of its wavefront ----
    uint32_t voff[SR], mask[RAGGED ? SR : 1][4];
    k7_u4 xreg[D < 2 ? 2 : D][SR][4];
    __amdgpu_buffer_rsrc_t xr;
    const unsigned char* xbase = nullptr;           // (RAGGED) what xr begins with, and its size
    uint32_t records = 0u;
    const int q0 = kg * QN;                         // first chunk of this group
    int xq = 0, xk = 0;                             // the chunk to load next: of tile xk, chunk xq of the group's
    const int64_t img_bytes = (int64_t)a.c_in * hw * 2;
    auto setup_tile = [&](int k) __attribute__((always_inline)) {
        const Tile t = decode(k);
        const int u0 = t.v0 - 1;                    // tall row of staged row 0
        const int img0 = (u0 + a.po) / a.po - 1, iy0 = u0 - img0 * a.po;
        const int ib = img0 > 0 ? img0 : 0;
        xbase = static_cast<const unsigned char*>(a.x) + ib * img_bytes;
        records = buffer_records(a.x_bytes - ib * img_bytes);
        xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(xbase), 0, (int)records, 0x00027000);
#pragma unroll
        for (int r = 0; r < SR; ++r) {
            const int task = r * 64 + lane, srow = task / G.gpr, sg = task - srow * G.gpr + (TC == 16 ? 1 : 0);       // group 0 and TC / 8 + 1 lie beside the tile
            const int tt = iy0 + srow, di = k7_div(tt, a.magic_po);
            const int img = img0 + di, iy = tt - di * a.po, ix = t.ox0 + 8 * (sg - 1);
            const bool ok = task < G.tasks && img >= 0 && img < a.n && iy < a.h && ix >= 0 && ix < a.w;
            voff[r] = ok ? (uint32_t)(img - ib) * (uint32_t)img_bytes + (uint32_t)(iy * a.w + ix) * 2u : kK7Outside;
        }
    };
    auto xload = [&](auto set_tag) __attribute__((always_inline)) {
        constexpr int set = decltype(set_tag)::value;
        if (xq == 0) {
            if (xk < my_n) setup_tile(xk);
            else {                                  // past the last chunk: nothing is fetched, the count of loads stays
#pragma unroll
                for (int r = 0; r < SR; ++r) voff[r] = kK7Outside;
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int ch = (q0 + xq) * kMfmaChunk + wave * 4 + j, chc = ch < a.c_in ? ch : a.c_in - 1;    // past the last channel: its values again, for zero weights
            const uint32_t at = (uint32_t)(chc * hw * 2);
            if constexpr (RAGGED) {                 // a row's last load may run past the row: the buffer begins at the channel, so that it ends with x
                const __amdgpu_buffer_rsrc_t cr = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(xbase + at), 0, (int)buffer_records_from(records, at), 0x00027000);
#pragma unroll
                for (int r = 0; r < SR; ++r) xreg[set][r][j] = __builtin_bit_cast(k7_u4, __builtin_amdgcn_raw_buffer_load_b128(cr, (int)voff[r], 0, 0));
            } else {
#pragma unroll
                for (int r = 0; r < SR; ++r) xreg[set][r][j] = __builtin_bit_cast(k7_u4, __builtin_amdgcn_raw_buffer_load_b128(xr, (int)voff[r], (int)at, 0));
            }
        }
        if (++xq == QN) xq = 0, ++xk;
    };
    // LDS holds a plane of words for every pair of channels, a pixel a word.  Groups inside the tile are two 16-byte writes; of the
    // groups beside it one pixel is needed.
    int dst[SR], mq = 0, mk = 0;                    // the chunk to write next, as above: loads are up to D chunks ahead, in another tile
    uint32_t where = 0u;                            // bit r: task r lies inside the tile; 2 + r: on its left; 4 + r: on its right
#pragma unroll
    for (int r = 0; r < SR; ++r) {
        const int task = r * 64 + lane, srow = task / G.gpr, sg = task - srow * G.gpr + (TC == 16 ? 1 : 0);
        dst[r] = group0 + wave * 2 * G.plane + (srow * G.pitch + (sg == 0 ? 3 : 8 * sg - 4)) * 4;
        if (task < G.tasks) where |= (sg == 0 ? 4u : sg <= TC / 8 ? 1u : 16u) << r;
    }
    auto xwrite = [&](auto set_tag, int buf_off) __attribute__((always_inline)) {
        constexpr int set = decltype(set_tag)::value;
        if constexpr (RAGGED) {                     // a row's last group runs into the next row, whose pixels are taken out again
            if (mq == 0) {
                const int ox0 = decode(mk).ox0;
#pragma unroll
                for (int r = 0; r < SR; ++r) {
                    const int task = r * 64 + lane, sg = task % G.gpr + (TC == 16 ? 1 : 0), in = a.w - ox0 - 8 * (sg - 1);
#pragma unroll
                    for (int e = 0; e < 4; ++e) mask[r][e] = in > 2 * e ? 0xFFFFFFFFu : 0u;      // (widths are even)
                }
            }
            if (++mq == QN) mq = 0, ++mk;
        }
#pragma unroll
        for (int r = 0; r < SR; ++r) {
            k7_u4 lo[2], hi[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                uint32_t d[8];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    uint32_t u = xreg[set][r][2 * c][e], v = xreg[set][r][2 * c + 1][e];
                    if constexpr (RAGGED) u &= mask[r][e], v &= mask[r][e];
                    d[2 * e] = __builtin_amdgcn_perm(v, u, 0x05040100u);
                    d[2 * e + 1] = __builtin_amdgcn_perm(v, u, 0x07060302u);
                }
                lo[c] = k7_u4{d[0], d[1], d[2], d[3]}, hi[c] = k7_u4{d[4], d[5], d[6], d[7]};
            }
            unsigned char* o = smem + buf_off + dst[r];
            if ((where >> r) & 1u) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    *reinterpret_cast<k7_u4*>(o + c * G.plane) = lo[c];
                    *reinterpret_cast<k7_u4*>(o + c * G.plane + 16) = hi[c];
                }
            }
            if (TC != 16 && ((where >> r) & 20u)) {
#pragma unroll
                for (int c = 0; c < 2; ++c) *reinterpret_cast<uint32_t*>(o + c * G.plane) = (where >> r) & 4u ? hi[c][3] : lo[c][0];
            }
        }
    };
    if constexpr (TC == 16) {                       // the columns beside such a tile are outside the images
        for (int i = tid & 255; i < 16 * G.trp; i += 256) {
            const int pl = i / G.trp, r = i - pl * G.trp;       // both buffers' planes lie in one row
            uint32_t* o = reinterpret_cast<uint32_t*>(smem + group0 + pl * G.plane) + r * G.pitch;
            o[3] = 0u, o[G.pitch] = 0u;
        }
    }

    // ---- weights: a chunk's 18 fragments of 1 KB lie in memory as they lie in LDS ----
    int wq = 0, wk = 0;
    const unsigned char* wptr = nullptr;
    const uint32_t w_off = (uint32_t)lane * 16u;
    auto wload = [&](uint32_t buf) __attribute__((always_inline)) {                // into weight buffer 0, 1 or 2, and on to the next chunk
        if (wq == 0) {
            const Tile t = decode(wk);
            wptr = static_cast<const unsigned char*>(a.wpk) + ((int64_t)t.fbi * a.q + q0) * kK7WeightBytes;
            if (kg == 0 && wave == 3) load_lds4((uint32_t)lane * 4u, uniform_address(a.bias + t.fbi * kMfmaFilters), lds0 + tail + (uint32_t)(wk & 3) * 256u);
        }
        const unsigned char* base = static_cast<const unsigned char*>(uniform_address(wptr));
        const uint32_t lds = (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds0 + (uint32_t)group0 + 2 * G.xbuf + buf * kK7WeightBytes));
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            const int f = wave + 4 * i;
            if (f < 18) load_lds16(w_off, base + f * 1024, lds + (uint32_t)f * 1024u);
        }
        wptr += kK7WeightBytes;
        if (++wq == QN) wq = 0, ++wk;
    };

    // ---- operand addresses ----
    constexpr int WC = TC >= 32 ? TC / 32 : 1;      // wavefronts side by side
    const int row0 = TC >= 32 ? (wave / WC) * T : wave * 2 * T + (p >> 4) * T;
    const int col0 = TC >= 32 ? (wave % WC) * 32 + p : p & 15;
    const int xa = group0 + kb * 4 * G.plane + (row0 * G.pitch + col0 + 3) * 4;
    int w0 = group0 + 2 * G.xbuf + lane * 16, w1 = w0 + kK7WeightBytes, w2 = w1 + kK7WeightBytes;      // of the chunks s, s + 1 and, with three buffers, s + 2

    k7_h8 xf[RX], wf[WR][2];
    auto read_x = [&](int idx, int buf) __attribute__((always_inline)) {           // fragment idx of the chunk in buffer buf, or idx - NX of the next
        const int i = idx < NX ? idx : idx - NX, b = idx < NX ? buf : buf ^ 1;
        const int c = i / (T + 2), r = i % (T + 2);
        const unsigned char* o = smem + xa + b * G.xbuf + (r * G.pitch + c) * 4;
        k7_u4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = *reinterpret_cast<const uint32_t*>(o + e * G.plane);
        xf[idx % RX] = __builtin_bit_cast(k7_h8, v);
    };
    auto read_w = [&](auto u_tag, int idx) __attribute__((always_inline)) {     // step idx = 3 c + kr uses tap 3 kr + c
        const int base = idx < 9 ? w0 : w1, i = idx < 9 ? idx : idx - 9;
        const int tap = (i % 3) * 3 + i / 3;
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) wf[(9 * decltype(u_tag)::value + idx) % WR][mt] = *reinterpret_cast<const k7_h8*>(smem + base + (tap * 2 + mt) * 1024);
    };
    k7_f16 acc[T][2];
    auto init_acc = [&](int k) __attribute__((always_inline)) {                    // from the bias, whose values came with the tile's first weights
        float b[2] = {0.0f, 0.0f};
        if (kg == 0) {
#pragma unroll
            for (int mt = 0; mt < 2; ++mt) b[mt] = *reinterpret_cast<const float*>(smem + tail + (k & 3) * 256 + (mt * 32 + p) * 4);
        }
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
            for (int mt = 0; mt < 2; ++mt) acc[i][mt] = k7_f16(b[mt]);
    };

    // ---- fill ----
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;
    using Next = std::integral_constant<int, D == 1 ? 0 : 1>;
    wload(0);
    xload(I0{});
    if (steps > 1) wload(1);
    xload(I1{});
    if constexpr (D > 2) xload(I2{});
    if (WB == 3 && steps > 2) wload(2);
    if constexpr (D > 3) xload(I3{});
    xwrite(I0{}, 0);
    if constexpr (D > 1) xload(I0{});
    xwrite(I1{}, G.xbuf);                           // (has waited for what was loaded before it, the first two chunks' weights among them)
    xload(Next{});
    k7_lds_barrier();
    init_acc(0);
#pragma unroll
    for (int i = 0; i < k7_ahead(T, 0); ++i) read_x(i, 0);
    read_w(I0{}, 0);
    if constexpr (WR == 3) read_w(I0{}, 1);

    int s = 0, q = 0, k = 0;                        // chunk being multiplied, its place in the tile, the tile
    uint32_t wbuf = 0;                              // s % WB
    // When chunk s begins, x of the chunks s + 2 to s + 1 + D is in registers or on its way.  Behind the barrier of chunk s the buffers
    // of chunk s are free: x of chunk s + 2 goes to LDS, the weights of chunk s + WB and x of chunk s + 2 + D are asked for.
    auto chunk = [&](auto u_tag) __attribute__((always_inline)) {
        constexpr int U = decltype(u_tag)::value, B = U & 1;
        auto one = [&](auto j_tag) __attribute__((always_inline)) {
            constexpr int J = decltype(j_tag)::value, C = J / 3, KR = J % 3;
            if constexpr (J == 7) {
                if constexpr (WR == 2) read_w(u_tag, 8);
                // All of this wavefront's reads of chunk s have left LDS.  Younger than its part of the weights of chunk s + 1 are the
                // loads of one chunk of x, or with three buffers of two and, if there are any, the weights of chunk s + 2.
                if constexpr (WB == 2) __builtin_amdgcn_s_waitcnt(wait_vmcnt(4 * SR));
                else if (s + 2 < steps) __builtin_amdgcn_s_waitcnt(wait_vmcnt(8 * SR + 4));
                else __builtin_amdgcn_s_waitcnt(wait_vmcnt(8 * SR));
                k7_lds_barrier();
            }
#pragma unroll
            for (int i = k7_ahead(T, J); i < k7_ahead(T, J + 1); ++i) read_x(i, B);
            if constexpr (WR == 3) read_w(u_tag, J + 2);
            else if constexpr (J != 7) read_w(u_tag, J + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < T; ++i) {
#pragma unroll
                for (int mt = 0; mt < 2; ++mt)
                    acc[i][mt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(xf[((T + 2) * C + KR + i) % RX], wf[(9 * U + J) % WR][mt], acc[i][mt], 0, 0, 0);
                if (i == 0) {
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (J == 7) {
                        if (s + 2 < steps) xwrite(std::integral_constant<int, (U + 2) % D>{}, B * G.xbuf);
                    }
                    if constexpr (J == 8) {
                        if (s + WB < steps) wload(wbuf);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        };
        one(I0{});
        one(I1{});
        one(I2{});
        one(I3{});
        one(std::integral_constant<int, 4>{});
        one(std::integral_constant<int, 5>{});
        one(std::integral_constant<int, 6>{});
        one(std::integral_constant<int, 7>{});
        one(std::integral_constant<int, 8>{});
        const int t = w0;
        w0 = w1;
        if constexpr (WB == 3) w1 = w2, w2 = t;
        else w1 = t;
        if (++wbuf == WB) wbuf = 0;
    };
    auto epilogue = [&](int k) __attribute__((always_inline)) {
        const Tile t = decode(k);
        const int oimg0 = t.v0 / a.po, oy0 = t.v0 - oimg0 * a.po;
        const int plane_out = a.out_h * a.out_w;
        // ReLU, or nothing: the larger of a value and a NaN is the value, and a NaN stays one
        const _Float16 floor16 = a.relu ? (_Float16)0.0f : (_Float16)__builtin_nanf("");
        // An accumulator holds one filter per lane, two rows of 32 columns: lower and upper lanes four columns each in turn.  They
        // exchange halves, so that the lower lanes hold the first row, the upper ones the second; then four neighbouring lanes
        // exchange pieces of 16 bytes, so that they store 64 bytes of one filter at a time: a store of 64 lanes to 32 filters
        // and rows takes the vector cache 78 ns, one to sixteen 19.
        const int piece = lane & 3;
#pragma unroll
        for (int ip = 0; ip < T; ip += 2) {
        if constexpr (POOL) {
            // pooled, a filter has 16 columns: the lower lanes take the first accumulator's filters, the upper ones the second's
            const int pr = (TC >= 32 ? row0 : wave * 2 * T + (lane & 1) * T) + ip;
            const int pcol = TC >= 32 ? (t.ox0 + (wave % WC) * 32 + (lane & 1) * 16) >> 1 : t.ox0 >> 1;
            const int tt = oy0 + pr, di = k7_div(tt, a.magic_po);
            const int img = oimg0 + di, y = tt - di * a.po;
            const int count = img < a.n && y < a.h ? a.out_w - pcol : 0;
            uint32_t d[2][4];
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float m[2];
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const int g = 4 * q + 2 * e;
                        m[e] = __builtin_fmaxf(__builtin_fmaxf(acc[ip][mt][g], acc[ip][mt][g + 1]), __builtin_fmaxf(acc[ip + 1][mt][g], acc[ip + 1][mt][g + 1]));
                    }
                    const k7_h2 h = __builtin_elementwise_max(k7_h2{(_Float16)m[0], (_Float16)m[1]}, k7_h2{floor16, floor16});
                    d[mt][q] = __builtin_bit_cast(uint32_t, h);
                }
            // d[mt]: columns 4 q + (0, 1) in the lower lanes, + (2, 3) in the upper ones
            k7_u4 pc[2];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const k7_u2 r = __builtin_amdgcn_permlane32_swap(d[0][q], d[1][q], false, false);
                pc[q >> 1][(q & 1) * 2] = r[0], pc[q >> 1][(q & 1) * 2 + 1] = r[1];
            }
            const bool odd = (lane & 1) != 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int u = (int)pc[0][e], v = (int)pc[1][e];
                const int du = __builtin_amdgcn_mov_dpp(u, 0xB1, 0xF, 0xF, true), dv = __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true);
                pc[0][e] = (uint32_t)(odd ? dv : u), pc[1][e] = (uint32_t)(odd ? v : du);
            }
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                const int co = t.fbi * kMfmaFilters + kb * 32 + (p & ~1) + f;
                if (count > 0 && co < a.c_out)
                    k7_store8(static_cast<unsigned char*>(a.y) + (((int64_t)img * a.c_out + co) * plane_out + (y >> 1) * a.out_w + pcol) * 2, pc[f], count);
            }
        } else {
            const int lrow = (TC >= 32 ? row0 : wave * 2 * T + (piece >> 1) * T) + ip + kb;
            const int lcol = t.ox0 + (TC >= 32 ? (wave % WC) * 32 + piece * 8 : (piece & 1) * 8);
            const int tt = oy0 + lrow, di = k7_div(tt, a.magic_po);
            const int img = oimg0 + di, y = tt - di * a.po;
            const bool in = img < a.n && y < a.h;
#pragma unroll
            for (int mt = 0; mt < 2; ++mt) {
                const int co = t.fbi * kMfmaFilters + mt * 32 + (p & ~3);
                const int64_t row_at = ((int64_t)img * a.c_out + co) * plane_out + y * a.out_w;
                k7_u4 pc[4];
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        uint32_t d[2];
#pragma unroll
                        for (int i = 0; i < 2; ++i) {
                            const k7_h2 h = __builtin_elementwise_max(k7_h2{(_Float16)acc[ip + i][mt][4 * q + 2 * e], (_Float16)acc[ip + i][mt][4 * q + 2 * e + 1]}, k7_h2{floor16, floor16});
                            d[i] = __builtin_bit_cast(uint32_t, h);
                        }
                        const k7_u2 r = __builtin_amdgcn_permlane32_swap(d[0], d[1], false, false);
                        pc[q][e] = r[0], pc[q][2 + e] = r[1];
                    }
                k7_transpose4(pc, lane);
                const int count = in ? a.out_w - lcol : 0;
#pragma unroll
                for (int f = 0; f < 4; ++f)
                    if (count > 0 && co + f < a.c_out) k7_store8(static_cast<unsigned char*>(a.y) + (row_at + (int64_t)f * plane_out + lcol) * 2, pc[f], count);
            }
        }
        }
    };

    // The loads of x stay outside every condition, past the last chunk too, where they fetch nothing: the compiler then counts
    // exactly which loads are younger than the ones it waits for.  (With a way out of the loop between the chunks it would not.)
    auto part = [&](auto u_tag) __attribute__((always_inline)) {
        constexpr int U = decltype(u_tag)::value;
        if (s < steps) chunk(u_tag);
        xload(std::integral_constant<int, (U + 2) % D>{});
        if constexpr (KG == 1) {
            if (s < steps && ++q == QN) {
                q = 0;
                epilogue(k);
                if (++k < my_n) init_acc(k);
            }
        }
        ++s;
    };
    do {
        part(I0{});
        part(I1{});
        if constexpr (D > 2) part(I2{}), part(I3{});
    } while (s < steps);
    if constexpr (KG > 1) {                         // one tile per workgroup: the buffers are free for the second group's sums
        __syncthreads();
        float* red = reinterpret_cast<float*>(smem) + wave * (T * 2 * 16 * 64) + lane * 4;
        if (kg == 1) {
#pragma unroll
            for (int i = 0; i < T * 2; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    *reinterpret_cast<k7_f4*>(red + (i * 4 + e) * 256) = k7_f4{acc[i / 2][i % 2][4 * e], acc[i / 2][i % 2][4 * e + 1], acc[i / 2][i % 2][4 * e + 2], acc[i / 2][i % 2][4 * e + 3]};
        }
        __syncthreads();
        if (kg == 1) return;
#pragma unroll
        for (int i = 0; i < T * 2; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const k7_f4 v = *reinterpret_cast<const k7_f4*>(red + (i * 4 + e) * 256);
#pragma unroll
                for (int b = 0; b < 4; ++b) acc[i / 2][i % 2][4 * e + b] += v[b];
            }
        epilogue(0);
    }
}

typedef void (*k7_launch_fn)(const K7Args& a, int blocks, int lds_bytes, hipStream_t stream);
// The instantiation for (rows per wavefront, tile columns, groups, width not a multiple of eight, pool); nullptr if not built.
k7_launch_fn k7_lookup(int rows, int cols, int groups, bool ragged, bool pool);

}  // namespace ppc
