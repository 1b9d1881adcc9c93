// Deep reuse (paper, section 2.3.2): kernels and C ABI (include/pp_deep_reuse.h).
//
// Both paths are four launches per pass and begin with an empty election table, whatever the pass before left:
//   reuse_clear           representatives <- "none"
// Neuron vectors whose length is a multiple of 4 and outputs whose number is a multiple of 4:
//   reuse_hash_tiled      signatures, segment by segment for tiles of rows staged in LDS; elects each cluster's lowest row
//   reuse_products_packed numbers a segment's clusters in ascending signature order and computes their products
//   reuse_gather_packed   y[i][:] = act(bias + sum_s P[s][cluster(i, s)][:]) with a segment's products in LDS
// Anything else:
//   reuse_hash            one lane per neuron vector, segments fastest (a wavefront reads one contiguous stretch of x),
//                         hyperplanes in LDS; the lowest row of every cluster is elected with integer minimum atomics
//   reuse_products        P[s][g][:] = x[rep(s,g)][segment s] . W[segment s][:]
//   reuse_gather          y[i][:] = act(bias + sum_s P[s][sig(i,s)][:])
// Signature bits are signs of binary32 fused multiply-add chains.  Integer work (signatures, representatives) is
// deterministic; the float sums run in a fixed order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstdint>
#include <new>
#include <vector>

#include "pp_deep_reuse.h"
#include "reuse_rules.hpp"

using namespace ppc;

namespace {

constexpr int kMaxSeg = 32;

typedef const __attribute__((address_space(4))) float* const_f32;

// count is rounded up to whole 16-byte words (the table has room for them)
__global__ __launch_bounds__(256) void reuse_clear(int32_t* rep, int count) {
    const int e = (int)(blockIdx.x * 256 + threadIdx.x) * 4;
    if (e < count) *reinterpret_cast<int4*>(rep + e) = int4{INT_MAX, INT_MAX, INT_MAX, INT_MAX};
}

// One lane per neuron vector, segments fastest: consecutive lanes read consecutive runs of L floats of x, so a
// wavefront reads one contiguous stretch of memory (a lane per row, with the hyperplanes as wave-uniform scalar
// operands, was measured ten times slower: its loads are a cache line apart).  The hyperplanes of all segments
// sit in LDS, loaded once per workgroup, which then walks the neuron vectors with the stride of the grid; the
// segment pitch is H * L + 1 floats, so lanes on different segments use different banks.  A lane's signature
// bits are the signs of H chains of fused multiply-adds in ascending l.  The representative of a cluster is
// the lowest row: one integer minimum atomic per lane, skipped when the table already holds a row at least as
// low (the table only ever decreases, so a stale read can cost an atomic, never a wrong result).
template <int L>
__global__ __launch_bounds__(256) void reuse_hash(const float* __restrict__ x, const float* __restrict__ hyper, uint16_t* __restrict__ sig,
                                                  int32_t* __restrict__ rep, int n, int k, int hash_bits) {
    extern __shared__ __attribute__((aligned(16))) unsigned char reuse_smem[];
    float* hp = reinterpret_cast<float*>(reuse_smem);
    const int S = k / L, G = 1 << hash_bits, pitch = hash_bits * L + 1;
    for (int e = (int)threadIdx.x; e < S * hash_bits * L; e += 256) {
        const int s = e / (hash_bits * L);
        hp[s * pitch + (e - s * hash_bits * L)] = hyper[e];
    }
    __syncthreads();
    // a lane takes the same segment of RPL consecutive rows, so that every hyperplane value it reads from LDS serves RPL
    // neuron vectors; consecutive lanes take consecutive segments, so each of its loads is part of one contiguous row
    constexpr int RPL = 4;
    const uint32_t groups = (uint32_t)((n + RPL - 1) / RPL), total = groups * (uint32_t)S;      // below 2^31: n * k is
    for (uint32_t e = blockIdx.x * 256u + threadIdx.x; e < total; e += gridDim.x * 256u) {      // e = (i / RPL) * S + s
        const int i0 = (int)(e / (uint32_t)S) * RPL, s = (int)(e % (uint32_t)S);
        float xv[RPL][L];
#pragma unroll
        for (int j = 0; j < RPL; ++j) {
            const int i = i0 + j < n ? i0 + j : n - 1;                  // rows past the end repeat the last one (not stored)
            const float* src = x + (int64_t)i * k + s * L;
            if constexpr (L % 4 == 0) {
#pragma unroll
                for (int l = 0; l < L; l += 4) {
                    const float4 v = *reinterpret_cast<const float4*>(src + l);
                    xv[j][l] = v.x, xv[j][l + 1] = v.y, xv[j][l + 2] = v.z, xv[j][l + 3] = v.w;
                }
            } else {
#pragma unroll
                for (int l = 0; l < L; ++l) xv[j][l] = src[l];
            }
        }
        const float* h0 = hp + s * pitch;
        unsigned g[RPL];
#pragma unroll
        for (int j = 0; j < RPL; ++j) g[j] = 0;
        for (int h = 0; h < hash_bits; ++h) {
            float p[RPL];
#pragma unroll
            for (int j = 0; j < RPL; ++j) p[j] = 0.0f;
#pragma unroll
            for (int l = 0; l < L; ++l) {
                const float hv = h0[h * L + l];
#pragma unroll
                for (int j = 0; j < RPL; ++j) p[j] = __builtin_fmaf(xv[j][l], hv, p[j]);
            }
#pragma unroll
            for (int j = 0; j < RPL; ++j) g[j] |= (p[j] > 0.0f ? 1u : 0u) << h;
        }
#pragma unroll
        for (int j = 0; j < RPL; ++j) {
            const int i = i0 + j;
            if (i < n) {
                sig[(int64_t)i * S + s] = (uint16_t)g[j];
                int32_t* slot = rep + (int64_t)s * G + g[j];
                if (__builtin_nontemporal_load(slot) > i) atomicMin(slot, i);
            }
        }
    }
}

// grid (ceil(G * m / 256), S)
__global__ __launch_bounds__(256) void reuse_products(const float* __restrict__ x, const float* __restrict__ w, const int32_t* __restrict__ rep,
                                                      float* __restrict__ P, int k, int m, int L, int G) {
    const int s = (int)blockIdx.y, e = (int)(blockIdx.x * 256 + threadIdx.x);
    if (e >= G * m) return;
    const int g = e / m, c = e - g * m;
    const int r = rep[(int64_t)s * G + g];
    if (r == INT_MAX) return;                                       // an empty cluster: nobody reads its products
    float acc = 0.0f;
    for (int l = 0; l < L; ++l) acc = __builtin_fmaf(x[(int64_t)r * k + s * L + l], w[(int64_t)(s * L + l) * m + c], acc);
    P[((int64_t)s * G + g) * m + c] = acc;
}

// V output columns per lane (4 when m is a multiple of 4, else 1), columns fastest
template <int V>
__global__ __launch_bounds__(256) void reuse_gather(const uint16_t* __restrict__ sig, const float* __restrict__ P, const float* __restrict__ bias,
                                                    float* __restrict__ y, int n, int m, int S, int G, int relu) {
    const int mv = m / V;
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (int64_t)n * mv) return;
    const int i = (int)(e / mv), c = (int)(e - (int64_t)i * mv) * V;
    float acc[V];
#pragma unroll
    for (int v = 0; v < V; ++v) acc[v] = bias[c + v];
    const uint16_t* srow = sig + (int64_t)i * S;
    for (int s = 0; s < S; ++s) {
        const float* p = P + ((int64_t)s * G + srow[s]) * m + c;
        if constexpr (V == 4) {
            const float4 v4 = *reinterpret_cast<const float4*>(p);
            acc[0] += v4.x, acc[1] += v4.y, acc[2] += v4.z, acc[3] += v4.w;
        } else {
            acc[0] += p[0];
        }
    }
#pragma unroll
    for (int v = 0; v < V; ++v)
        if (relu) acc[v] = acc[v] > 0.0f ? acc[v] : 0.0f;
    if constexpr (V == 4) {
        float4 o;
        o.x = acc[0], o.y = acc[1], o.z = acc[2], o.w = acc[3];
        *reinterpret_cast<float4*>(y + (int64_t)i * m + c) = o;
    } else {
        y[(int64_t)i * m + c] = acc[0];
    }
}

// ---- the tiled path ----

constexpr int kTileWaves = 4;
constexpr int reuse_rows_per_lane(int L) { return L <= 16 ? 2 : 1; }      // a wavefront's tile: 64 or 128 rows of one segment, at most 8 KB

typedef uint32_t reuse_u4 __attribute__((ext_vector_type(4)));
typedef float reuse_f4 __attribute__((ext_vector_type(4)));

template <typename P> __device__ __forceinline__ P* reuse_uniform(P* p) {
    const uint64_t v = (uint64_t)(uintptr_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (P*)(uintptr_t)(((uint64_t)hi << 32) | lo);
}
// every lane fetches 16 bytes at base + off into LDS at lds_dst + 16 * lane
__device__ __forceinline__ void reuse_dma16(uint32_t off, const void* base, uint32_t lds_dst) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds_dst) : "memory", "m0");
}

// A workgroup hashes one segment of a chunk of rows, a wavefront RPL * 64 consecutive rows at a time, lane = row, so that the
// hyperplanes are wave-uniform: they arrive by scalar loads and every multiply-add takes one of them from a scalar
// register.  The rows' pieces of x come in by direct loads into the wavefront's own part of LDS (a lane reading its row from
// memory would use 16 bytes of a cache line at a time: 1252 us), are read back as 16-byte words in an order that keeps the
// lanes on different banks, and the next rows' loads run while these are hashed.  The lowest row of each cluster is elected
// in an LDS table of the segment and handed to the global one at the end (electing in the global table row by row took
// 634 us: every workgroup's first rows meet an empty table, millions of atomics on some hundred addresses).  sig is
// segment-major: [S][row_pitch].
template <int L>
__global__ __launch_bounds__(64 * kTileWaves) void reuse_hash_tiled(const float* __restrict__ x, const float* __restrict__ hyper, uint16_t* __restrict__ sig,
                                                                   int32_t* __restrict__ rep, int n, int row_pitch, int k, int hash_bits, int chunk, int items, int per_xcd) {
    constexpr int RPL = reuse_rows_per_lane(L), TR = 64 * RPL, PP = L / 4, NI = TR * PP / 64;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[kTileWaves * TR * L * 4];
    extern __shared__ int32_t lowest[];                                           // [1 << hash_bits]
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int S = k / L, G = 1 << hash_bits;
    // segments fastest inside an XCD's range: neighbouring segments share cache lines of x
    const int item = (int)(blockIdx.x & 7u) * per_xcd + (int)(blockIdx.x >> 3);
    if (item >= items) return;
    const int s = item % S, first = item / S * chunk, last = first + chunk < n ? first + chunk : n;
    for (int g = tid; g < G; g += 64 * kTileWaves) lowest[g] = INT_MAX;
    __syncthreads();
    unsigned char* mine = smem + wave * TR * L * 4;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)mine;
    // slot of piece p of row r: pieces of 4 or 8 per row are exchanged so that eight consecutive rows use different banks
    auto slot_of = [](int r, int p) { return PP == 4 ? p ^ ((r >> 2) & 3) : PP == 8 ? p ^ ((r >> 1) & 7) : p; };
    auto fetch = [&](int row0) {                                                  // rows past the end repeat the last one
        const unsigned char* xt = reuse_uniform(reinterpret_cast<const unsigned char*>(x + (int64_t)row0 * k + s * L));
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int g = i * 64 + lane, r = g / PP, p = slot_of(r, g - r * PP);  // (an exchange is its own inverse)
            const int row = row0 + r < n ? r : n - 1 - row0;
            reuse_dma16((uint32_t)(row * k * 4 + p * 16), xt, lds0 + (uint32_t)(i * 1024));
        }
    };
    float xv[RPL][L];
    auto read = [&]() {
#pragma unroll
        for (int j = 0; j < RPL; ++j)
#pragma unroll
            for (int p = 0; p < PP; ++p) {
                const int r = j * 64 + lane;
                const reuse_f4 v = *reinterpret_cast<const reuse_f4*>(mine + (r * PP + slot_of(r, p)) * 16);
                xv[j][4 * p] = v.x, xv[j][4 * p + 1] = v.y, xv[j][4 * p + 2] = v.z, xv[j][4 * p + 3] = v.w;
            }
    };
    const const_f32 hp = (const_f32)(uintptr_t)reuse_uniform(hyper + (int64_t)s * hash_bits * L);
    int row0 = first + wave * TR;
    if (row0 < last) fetch(row0);
    for (; row0 < last; row0 += kTileWaves * TR) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        read();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (row0 + kTileWaves * TR < last) fetch(row0 + kTileWaves * TR);
        __builtin_amdgcn_sched_barrier(0);
        unsigned g[RPL];
#pragma unroll
        for (int j = 0; j < RPL; ++j) g[j] = 0;
        for (int h = 0; h < hash_bits; ++h) {
            float p[RPL];
#pragma unroll
            for (int j = 0; j < RPL; ++j) p[j] = 0.0f;
#pragma unroll
            for (int l = 0; l < L; ++l) {
                const float hv = hp[h * L + l];
#pragma unroll
                for (int j = 0; j < RPL; ++j) p[j] = __builtin_fmaf(xv[j][l], hv, p[j]);
            }
#pragma unroll
            for (int j = 0; j < RPL; ++j) g[j] |= (p[j] > 0.0f ? 1u : 0u) << h;
        }
#pragma unroll
        for (int j = 0; j < RPL; ++j) {
            const int i = row0 + j * 64 + lane;
            if (i < last) {
                sig[(int64_t)s * row_pitch + i] = (uint16_t)g[j];
                // the table only ever decreases: a stale read can cost an atomic, never a wrong result
                if (lowest[g[j]] > i) atomicMin(&lowest[g[j]], i);
            }
        }
    }
    __syncthreads();
    for (int g = tid; g < G; g += 64 * kTileWaves) {
        const int v = lowest[g];
        if (v != INT_MAX) atomicMin(rep + (int64_t)s * G + g, v);
    }
}

// Numbers the non-empty clusters of segment blockIdx.x in ascending signature order (used[s] is their count), writes every
// row's number (ids, [S][row_pitch]) and computes the products of the clusters, packed: [s][block of up to 64 columns]
// [cluster][columns of the block], each block of columns a contiguous run that the gather copies to LDS.  The gridDim.y
// workgroups of a segment number all its clusters each and share the rows and the products.
template <int L>
__global__ __launch_bounds__(256) void reuse_products_packed(const float* __restrict__ x, const float* __restrict__ w, const int32_t* __restrict__ rep,
                                                             const uint16_t* __restrict__ sig, float* __restrict__ P, uint16_t* __restrict__ ids,
                                                             int32_t* __restrict__ used, int n, int numbered, int row_pitch, int k, int m, int G) {
    __shared__ int wave_sum[4];
    __shared__ int list_n;
    __shared__ int list_rep[512];
    __shared__ int list_id[512];
    __shared__ uint16_t number[4096];
    const int s = (int)blockIdx.x, parts = (int)gridDim.y;
    // a part computes the clusters whose number is blockIdx.y modulo the parts: at most 512 of 4096
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int per = (G + 255) / 256;                                // consecutive signatures of a thread: at most 16
    int rv[16], mine = 0;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int g = tid * per + q;
        rv[q] = q < per && g < G ? rep[(int64_t)s * G + g] : INT_MAX;
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) mine += rv[q] != INT_MAX ? 1 : 0;
    int upto = mine;                                                // inclusive sum over the wavefront
#pragma unroll
    for (int d = 1; d < 64; d *= 2) {
        const int o = __shfl_up(upto, d);
        if (lane >= d) upto += o;
    }
    if (lane == 63) wave_sum[wave] = upto;
    if (tid == 0) list_n = 0;
    __syncthreads();
    int id = upto - mine;
    for (int v = 0; v < wave; ++v) id += wave_sum[v];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int g = tid * per + q;
        if (rv[q] == INT_MAX) {
            if (q < per && g < G) number[g] = 0;
            continue;
        }
        number[g] = (uint16_t)id;
        if (id % parts == (int)blockIdx.y) {
            list_rep[id / parts] = rv[q], list_id[id / parts] = id;
            atomicAdd(&list_n, 1);
        }
        ++id;
    }
    if (blockIdx.y == 0 && tid == 255) used[s] = id;
    __syncthreads();
    // Eight rows per thread and turn: 16-byte words of both tables.  Rows from n to the end of the gather's last workgroup
    // are numbered 0, so that their (unused) sums read inside the tables.
    for (int i = ((int)blockIdx.y * 256 + tid) * 8; i < numbered; i += parts * 256 * 8) {
        const reuse_u4 v = *reinterpret_cast<const reuse_u4*>(sig + (int64_t)s * row_pitch + i);
        reuse_u4 o;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t lo = i + 2 * q < n ? number[v[q] & 0xFFFFu] : 0u, hi = i + 2 * q + 1 < n ? number[v[q] >> 16] : 0u;
            o[q] = lo | (hi << 16);
        }
        *reinterpret_cast<reuse_u4*>(ids + (int64_t)s * row_pitch + i) = o;
    }
    const int todo = list_n * m;
    for (int e = tid; e < todo; e += 256) {
        const int q = e / m, c = e - q * m;
        const float* xr = x + (int64_t)list_rep[q] * k + s * L;
        const float* wc = w + (int64_t)s * L * m + c;
        float xl[L], wl[L];
#pragma unroll
        for (int l = 0; l < L; l += 4) {
            const reuse_f4 v = *reinterpret_cast<const reuse_f4*>(xr + l);
            xl[l] = v.x, xl[l + 1] = v.y, xl[l + 2] = v.z, xl[l + 3] = v.w;
        }
#pragma unroll
        for (int l = 0; l < L; ++l) wl[l] = wc[(int64_t)l * m];
        float acc = 0.0f;
#pragma unroll
        for (int l = 0; l < L; ++l) acc = __builtin_fmaf(xl[l], wl[l], acc);
        const int cb = c >> 6, width = m - cb * 64 < 64 ? m - cb * 64 : 64;
        P[((int64_t)s * m + cb * 64) * G + (int64_t)list_id[q] * width + (c & 63)] = acc;
    }
}

// A workgroup sums RPT rows per lane of one block of columns, four columns per lane.  Segment by segment the block's
// products and the rows' cluster numbers come in by direct loads to a ring of four places in LDS, three segments ahead of
// the one being summed (always 12 KB of products, so that the wait counts are constants; a segment of more, 48 clusters of
// 64 columns, is read from memory instead): the rows' reads are then LDS reads, 128 bytes per clock and compute unit
// instead of what L2 delivers (925 MB of reads for 100 352 rows of 36 segments: 55 us out of L2).
constexpr int kGatherSlots = 4, kGatherProducts = 12 * 1024;
template <int RPT>
__global__ __launch_bounds__(kGatherThreads) void reuse_gather_packed(const uint16_t* __restrict__ ids, const float* __restrict__ P,
                                                                      const int32_t* __restrict__ used, const float* __restrict__ bias, float* __restrict__ y,
                                                                      int n, int row_pitch, int m, int S, int G, int relu) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char reuse_smem[];      // kGatherSlots x (products, rows x 2 bytes rounded up to 1 KB)
    constexpr int WAVES = kGatherThreads / 64, AHEAD = kGatherSlots - 1, PI = kGatherProducts / 1024;
    static_assert(RPT % 4 == 0 && PI + kGatherMaxRows * 2 / 1024 <= 2 * WAVES, "a row group's numbers are whole 8-byte words; at most two loads per wavefront and segment");
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cb = (int)blockIdx.y, width = m - cb * 64 < 64 ? m - cb * 64 : 64, row_bytes = width * 4;
    const int lpr = (m < 64 ? m : 64) / 4, rpp = kGatherThreads / lpr;      // lanes per row, row groups
    const int rl = tid / lpr, cl = (tid - rl * lpr) * 4;
    const bool on = rl < rpp && cl < width;
    const int rows = rpp * RPT, row0 = (int)blockIdx.x * rows;
    const int id_loads = (rows * 2 + 1023) / 1024, slot_bytes = kGatherProducts + id_loads * 1024;
    reuse_f4 acc[RPT];
    const reuse_f4 b4 = on ? *reinterpret_cast<const reuse_f4*>(bias + cb * 64 + cl) : reuse_f4(0.0f);
#pragma unroll
    for (int j = 0; j < RPT; ++j) acc[j] = b4;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)reuse_smem;
    // load instruction q of a segment: products for q < PI, numbers after; wavefront w issues w, w + WAVES, ...
    const int mine = (PI + id_loads - wave + WAVES - 1) / WAVES;            // 0 to 2
    const uint32_t lane16 = (uint32_t)lane * 16u;
    int slot_in = 0, ahead = 0;
    auto fetch = [&]() {                                           // (both tables are padded at their ends)
        const float* ps = reuse_uniform(P + ((int64_t)ahead * m + cb * 64) * G);
        const uint16_t* is = reuse_uniform(ids + (int64_t)ahead * row_pitch + row0);
        const uint32_t dst = lds0 + (uint32_t)(slot_in * slot_bytes);
#pragma unroll
        for (int q = wave, t = 0; t < 2; q += WAVES, ++t) {
            if (q < PI) reuse_dma16(lane16, ps + q * 256, dst + (uint32_t)(q * 1024));
            else if (q < PI + id_loads) reuse_dma16(lane16, is + (q - PI) * 512, dst + (uint32_t)(q * 1024));
        }
        slot_in = slot_in + 1 == kGatherSlots ? 0 : slot_in + 1;
        ++ahead;
    };
    while (ahead < AHEAD && ahead < S) fetch();
    int slot = 0;
    int clusters = used[0];
    for (int s = 0; s < S; ++s) {
        const bool fits = clusters * row_bytes <= kGatherProducts;
        clusters = used[s + 1 < S ? s + 1 : S - 1];
        // segment s has landed for this wavefront ... (the two after it may be in flight)
        if (s + AHEAD > S) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        else if (mine == 2) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
        else if (mine == 1) asm volatile("s_waitcnt vmcnt(2)" ::: "memory");
        __syncthreads();                                           // ... and for all, and everyone is done with s - 1
        if (ahead < S) fetch();
        const unsigned char* place = reuse_smem + slot * slot_bytes;
        slot = slot + 1 == kGatherSlots ? 0 : slot + 1;
        if (!on) continue;
        uint32_t off[RPT];
#pragma unroll
        for (int j = 0; j < RPT; j += 4) {
            const uint2 w = *reinterpret_cast<const uint2*>(place + kGatherProducts + (rl * RPT + j) * 2);
            off[j] = (w.x & 0xFFFFu) * (uint32_t)row_bytes, off[j + 1] = (w.x >> 16) * (uint32_t)row_bytes;
            off[j + 2] = (w.y & 0xFFFFu) * (uint32_t)row_bytes, off[j + 3] = (w.y >> 16) * (uint32_t)row_bytes;
        }
        reuse_f4 v[RPT];
        // (the empty asm keeps each branch's additions inside it: sunk behind the two, their wait would also drain the loads in flight)
        if (fits) {
            const unsigned char* p = place + cl * 4;
#pragma unroll
            for (int j = 0; j < RPT; ++j) v[j] = *reinterpret_cast<const reuse_f4*>(p + off[j]);
#pragma unroll
            for (int j = 0; j < RPT; ++j) {
                acc[j] += v[j];
                asm volatile("" : "+v"(acc[j]));
            }
        } else {
            const unsigned char* p = reinterpret_cast<const unsigned char*>(P + ((int64_t)s * m + cb * 64) * G + cl);
#pragma unroll
            for (int j = 0; j < RPT; ++j) v[j] = *reinterpret_cast<const reuse_f4*>(p + off[j]);
#pragma unroll
            for (int j = 0; j < RPT; ++j) {
                acc[j] += v[j];
                asm volatile("" : "+v"(acc[j]));
            }
        }
    }
    if (!on) return;
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const int i = row0 + rl * RPT + j;
        if (relu)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[j][v] = acc[j][v] > 0.0f ? acc[j][v] : 0.0f;
        if (i < n) *reinterpret_cast<reuse_f4*>(y + (int64_t)i * m + cb * 64 + cl) = acc[j];
    }
}

typedef void (*hash_tiled_fn)(const float*, const float*, uint16_t*, int32_t*, int, int, int, int, int, int, int);
template <int L> hash_tiled_fn pick_hash_tiled(int seg_len) {
    if constexpr (L == 0) return nullptr;
    else return seg_len == L ? reuse_hash_tiled<L> : pick_hash_tiled<L - 4>(seg_len);
}
typedef void (*products_fn)(const float*, const float*, const int32_t*, const uint16_t*, float*, uint16_t*, int32_t*, int, int, int, int, int, int);
template <int L> products_fn pick_products(int seg_len) {
    if constexpr (L == 0) return nullptr;
    else return seg_len == L ? reuse_products_packed<L> : pick_products<L - 4>(seg_len);
}

typedef void (*hash_fn)(const float*, const float*, uint16_t*, int32_t*, int, int, int);
template <int L> hash_fn pick_hash(int seg_len) {
    if constexpr (L == 0) return nullptr;
    else return seg_len == L ? reuse_hash<L> : pick_hash<L - 1>(seg_len);
}

}  // namespace

struct pp_reuse_plan {
    int k = 0, m = 0, L = 0, H = 0, n_max = 0;
    uint32_t flags = 0;
    bool on_device = false;
    float* d_w = nullptr;
    float* d_bias = nullptr;
    float* d_hyper = nullptr;
    uint16_t* d_sig = nullptr;
    int32_t* d_rep = nullptr;
    float* d_P = nullptr;
    bool tiled = false;                 // L and m multiples of 4: the tiled path
    uint16_t* d_ids = nullptr;          // ... [S][row_pitch] number of a row's cluster in the segment (d_sig has the same layout then)
    int row_pitch = 0;                  // ... room for the rows of the gather's last workgroup
    int32_t* d_used = nullptr;          // ... [S] clusters of a segment
};

namespace {

void release(pp_reuse_plan_t* p) {
    void* bufs[] = {p->d_w, p->d_bias, p->d_hyper, p->d_sig, p->d_rep, p->d_P, p->d_ids, p->d_used};
    for (void* b : bufs)
        if (b) (void)hipFree(b);
}

template <typename T>
bool put(T** dst, const void* src, size_t bytes, size_t pad = 16) {
    void* p = nullptr;
    if (hipMalloc(&p, bytes + pad) != hipSuccess) return false;
    *dst = static_cast<T*>(p);
    if (hipMemset(p, 0, bytes + pad) != hipSuccess) return false;
    return !src || hipMemcpy(p, src, bytes, hipMemcpyHostToDevice) == hipSuccess;
}

}  // namespace

extern "C" {

pp_status_t pp_reuse_plan(const pp_reuse_desc_t* d, pp_reuse_plan_t** out_plan) {
    if (out_plan) *out_plan = nullptr;
    if (!d || !out_plan || !d->weights || !d->hyperplanes) return PP_ERR_NULL;
    if (d->k < 1 || d->m < 1 || d->n_max < 1 || d->seg_len < 1 || d->seg_len > kMaxSeg || d->k % d->seg_len != 0 || d->hash_bits < 1 ||
        d->hash_bits > 12)
        return PP_ERR_SHAPE;
    if ((int64_t)d->n_max * std::max(d->k, d->m) >= ((int64_t)1 << 31) || (int64_t)d->k * d->m >= ((int64_t)1 << 31)) return PP_ERR_SHAPE;
    if (d->flags & ~(uint32_t)(PP_FLAG_RELU | PP_FLAG_HOST_ONLY)) return PP_ERR_UNSUPPORTED;
    // the hash kernel keeps every segment's hyperplanes in LDS (H * L + 1 floats per segment)
    if ((int64_t)(d->k / d->seg_len) * (d->hash_bits * d->seg_len + 1) * 4 > 64 * 1024) return PP_ERR_UNSUPPORTED;
    pp_reuse_plan_t* p = new (std::nothrow) pp_reuse_plan_t();
    if (!p) return PP_ERR_ALLOC;
    p->k = d->k, p->m = d->m, p->L = d->seg_len, p->H = d->hash_bits, p->n_max = d->n_max, p->flags = d->flags;
    if (!(d->flags & PP_FLAG_HOST_ONLY)) {
        const int S = d->k / d->seg_len, G = 1 << d->hash_bits;
        std::vector<float> zero_bias;
        const float* bias = d->bias;
        if (!bias) {
            zero_bias.assign((size_t)d->m, 0.0f);
            bias = zero_bias.data();
        }
        p->tiled = d->seg_len % 4 == 0 && d->m % 4 == 0;
        p->row_pitch = p->tiled ? reuse_row_pitch(d->n_max) : d->n_max;
        bool ok = put(&p->d_w, d->weights, (size_t)d->k * d->m * 4) && put(&p->d_bias, bias, (size_t)d->m * 4) &&
                  put(&p->d_hyper, d->hyperplanes, (size_t)S * d->hash_bits * d->seg_len * 4, 256) &&
                  put(&p->d_sig, nullptr, (size_t)S * p->row_pitch * 2) && put(&p->d_rep, nullptr, (size_t)S * G * 4) &&
                  put(&p->d_P, nullptr, (size_t)S * G * d->m * 4, kGatherProducts);
        if (ok && p->tiled) {
            ok = put(&p->d_ids, nullptr, (size_t)S * p->row_pitch * 2, kGatherMaxRows * 2) && put(&p->d_used, nullptr, (size_t)S * 4);
        }
        if (!ok) {
            (void)hipGetLastError();
            release(p);
            delete p;
            return PP_ERR_DEVICE;
        }
        p->on_device = true;
    }
    *out_plan = p;
    return PP_OK;
}

pp_status_t pp_reuse_run(const pp_reuse_plan_t* p, const void* x_dev, void* y_dev, int32_t n, void* hip_stream) {
    if (!p || !x_dev || !y_dev) return PP_ERR_NULL;
    if (n < 1 || n > p->n_max) return PP_ERR_SHAPE;
    const uintptr_t xa = reinterpret_cast<uintptr_t>(x_dev), ya = reinterpret_cast<uintptr_t>(y_dev);
    if ((xa | ya) & 15u) return PP_ERR_ALIGN;
    const uintptr_t xe = xa + (uintptr_t)((int64_t)n * p->k * 4), ye = ya + (uintptr_t)((int64_t)n * p->m * 4);
    if (xa < ye && ya < xe) return PP_ERR_ALIGN;
    if (!p->on_device) return PP_ERR_UNSUPPORTED;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const int S = p->k / p->L, G = 1 << p->H;
    const float* x = static_cast<const float*>(x_dev);
    float* y = static_cast<float*>(y_dev);
    const int relu = (p->flags & PP_FLAG_RELU) ? 1 : 0;
    const hash_tiled_fn hash_tiled = p->tiled ? pick_hash_tiled<kMaxSeg>(p->L) : nullptr;
    const hash_fn hash = p->tiled ? nullptr : pick_hash<kMaxSeg>(p->L);
    if (!hash_tiled && !hash) return PP_ERR_UNSUPPORTED;
    (void)hipGetLastError();
    hipLaunchKernelGGL(reuse_clear, dim3((unsigned)((S * G + 1023) / 1024)), dim3(256), 0, stream, p->d_rep, S * G);
    if (p->tiled) {
        // rows per workgroup: whole rounds of its wavefronts' tiles, as many as leave three workgroups per compute unit
        const int round = kTileWaves * 64 * reuse_rows_per_lane(p->L);
        const int64_t rounds = (n + round - 1) / round;
        const int per_wg = (int)std::max<int64_t>(1, (rounds * S + 767) / 768);
        const int chunk = per_wg * round, chunks = (int)((rounds + per_wg - 1) / per_wg);
        const int items = chunks * S, per_xcd = (items + 7) / 8;
        hipLaunchKernelGGL(hash_tiled, dim3((unsigned)(per_xcd * 8)), dim3(64 * kTileWaves), (size_t)G * 4, stream, x, p->d_hyper, p->d_sig, p->d_rep, n, p->row_pitch, p->k, p->H, chunk,
                           items, per_xcd);
        // enough workgroups per segment for four in all on every other compute unit, and for lists of 512 clusters
        const int parts = std::max(std::max(1, G / 512), std::min(16, 512 / S));
        const ReuseGather gs = reuse_gather_shape(n, p->m);
        hipLaunchKernelGGL(pick_products<kMaxSeg>(p->L), dim3((unsigned)S, (unsigned)parts), dim3(256), 0, stream, x, p->d_w, p->d_rep, p->d_sig, p->d_P, p->d_ids, p->d_used, n,
                           reuse_numbered_rows(gs), p->row_pitch, p->k, p->m, G);
        const dim3 grid((unsigned)gs.wgs_x, (unsigned)gs.blocks_y);
        const size_t gather_lds = (size_t)kGatherSlots * (kGatherProducts + (gs.rows * 2 + 1023) / 1024 * 1024);
        hipLaunchKernelGGL(gs.rpt == 16 ? reuse_gather_packed<16> : gs.rpt == 8 ? reuse_gather_packed<8> : reuse_gather_packed<4>, grid, dim3(kGatherThreads), gather_lds, stream, p->d_ids,
                           p->d_P, p->d_used, p->d_bias, y, n, p->row_pitch, p->m, S, G, relu);
        return hipGetLastError() == hipSuccess ? PP_OK : PP_ERR_DEVICE;
    }
    const size_t lds = (size_t)S * (p->H * p->L + 1) * 4;
    const int64_t hash_blocks = std::min<int64_t>(((int64_t)((n + 3) / 4) * S + 255) / 256, 256 * 8);      // at most eight workgroups per compute unit
    hipLaunchKernelGGL(hash, dim3((unsigned)hash_blocks), dim3(256), lds, stream, x, p->d_hyper, p->d_sig, p->d_rep, n, p->k, p->H);
    hipLaunchKernelGGL(reuse_products, dim3((unsigned)((G * p->m + 255) / 256), (unsigned)S), dim3(256), 0, stream, x, p->d_w, p->d_rep, p->d_P, p->k,
                       p->m, p->L, G);
    if (p->m % 4 == 0) {
        const int64_t lanes = (int64_t)n * (p->m / 4);
        hipLaunchKernelGGL(reuse_gather<4>, dim3((unsigned)((lanes + 255) / 256)), dim3(256), 0, stream, p->d_sig, p->d_P, p->d_bias, y, n, p->m, S, G, relu);
    } else {
        const int64_t lanes = (int64_t)n * p->m;
        hipLaunchKernelGGL(reuse_gather<1>, dim3((unsigned)((lanes + 255) / 256)), dim3(256), 0, stream, p->d_sig, p->d_P, p->d_bias, y, n, p->m, S, G, relu);
    }
    return hipGetLastError() == hipSuccess ? PP_OK : PP_ERR_DEVICE;
}

pp_status_t pp_reuse_read_clusters(const pp_reuse_plan_t* p, int32_t n, uint16_t* sig_out, int32_t* rep_out) {
    if (!p) return PP_ERR_NULL;
    if (n < 1 || n > p->n_max) return PP_ERR_SHAPE;
    if (!p->on_device) return PP_ERR_UNSUPPORTED;
    if (hipDeviceSynchronize() != hipSuccess) return PP_ERR_DEVICE;
    const int S = p->k / p->L, G = 1 << p->H;
    try {
        if (sig_out) {
            std::vector<uint16_t> by_segment(p->tiled ? (size_t)p->row_pitch * S : 0);
            if (hipMemcpy(p->tiled ? by_segment.data() : sig_out, p->d_sig, (size_t)(p->tiled ? p->row_pitch : n) * S * 2, hipMemcpyDeviceToHost) != hipSuccess) return PP_ERR_DEVICE;
            if (p->tiled)
                for (int s = 0; s < S; ++s)
                    for (int i = 0; i < n; ++i) sig_out[(size_t)i * S + s] = by_segment[(size_t)s * p->row_pitch + i];
        }
        if (rep_out) {
            if (hipMemcpy(rep_out, p->d_rep, (size_t)S * G * 4, hipMemcpyDeviceToHost) != hipSuccess) return PP_ERR_DEVICE;
            for (size_t e = 0; e < (size_t)S * G; ++e)
                if (rep_out[e] == INT_MAX) rep_out[e] = -1;
        }
    } catch (const std::bad_alloc&) {
        return PP_ERR_ALLOC;
    }
    return PP_OK;
}

pp_status_t pp_reuse_destroy(pp_reuse_plan_t* p) {
    if (!p) return PP_OK;
    release(p);
    delete p;
    return PP_OK;
}

}  // extern "C"
