// One output of a layer straight from its reordered kernel lists: the generic kernel, and what the binary32 matrix-core kernels
// fall back on where a non-finite input met a weight that is not there.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace ppc {

struct K0Args {
    const void* x;
    void* y;
    const int32_t* filt_off;   // [c_out+1]
    const int32_t* kidx;       // [k_kept]
    const uint8_t* kpat;       // [k_kept]
    const float* w;            // [k_kept*taps] (binary16-rounded values for an fp16 plan)
    const int8_t* tap_dyx;     // [P*taps*2]
    const int32_t* perm;       // [c_out]
    const int32_t* place;      // [c_out] position of a filter: perm[place[co]] = co
    const float* bias;         // [c_out] by original index
    int32_t n, c_in, c_out, h, w_, taps, relu;
    int32_t stride, ho, wo, out_h, out_w, pool;
};

// The stored output (sy, sx) of image img and the filter at position pos: walks the filter's kernel list (same-pattern kernels
// consecutive) and reads the input from memory with bounds checks.
template <typename T>
__device__ __forceinline__ T k0_output(const K0Args& a, int img, int pos, int sy, int sx) {
    const int64_t hw = (int64_t)a.h * a.w_;
    const T* __restrict__ x = static_cast<const T*>(a.x);
    const int co = a.perm[pos];
    const int beg = a.filt_off[pos], end = a.filt_off[pos + 1];
    const int np = a.pool ? 2 : 1;
    float best = 0.0f;
    for (int py = 0; py < np; ++py)
        for (int px = 0; px < np; ++px) {
            const int oy = sy * np + py, ox = sx * np + px;     // the convolution's own output
            float acc = 0.0f;
            for (int e = beg; e < end; ++e) {
                const int ci = a.kidx[e];
                const int8_t* tp = a.tap_dyx + (int)a.kpat[e] * a.taps * 2;
                const float* wv = a.w + (int64_t)e * a.taps;
                const T* xc = x + ((int64_t)img * a.c_in + ci) * hw;
                for (int j = 0; j < a.taps; ++j) {
                    const int iy = oy * a.stride + tp[2 * j], ix = ox * a.stride + tp[2 * j + 1];
                    if (iy >= 0 && iy < a.h && ix >= 0 && ix < a.w_) acc = __builtin_fmaf(wv[j], (float)xc[iy * a.w_ + ix], acc);
                }
            }
            acc += a.bias[co];
            if (a.relu) acc = acc > 0.0f ? acc : 0.0f;
            const float v = (float)(T)acc;                      // pooling acts on stored values
            best = (py == 0 && px == 0) ? v : (v > best ? v : best);
        }
    return (T)best;
}

// The same for filter co of a binary32 layer, stored.  The arguments come from the plan's copy in memory: as part of a
// kernel's own they would be loaded by every wavefront at its start (256 channels, 14x14, batch 32: 68.9 us against 68.2).
__device__ __forceinline__ void k0_again(const K0Args* lists, const float* x, float* y, int img, int co, int sy, int sx) {
    K0Args a = *lists;
    a.x = x, a.y = y;
    static_cast<float*>(a.y)[(((int64_t)img * a.c_out + co) * a.out_h + sy) * a.out_w + sx] = k0_output<float>(a, img, a.place[co], sy, sx);
}

// Generic kernel: any pattern table, kernel size, stride, with or without the fused 2x2 max-pool.  One lane per stored output,
// one filter per blockIdx.y, so that the lists are walked with wave-uniform indices.  It serves binary16 plans that ask for it,
// very sparse binary32 layers, and binary32 images beyond the matrix-core kernel's 31-bit offsets.
template <typename T>
__global__ __launch_bounds__(256) void k0_generic(const K0Args a) {
    const int pos = blockIdx.y;
    const int64_t pix = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t ohw = (int64_t)a.out_h * a.out_w;
    if (pix >= (int64_t)a.n * ohw) return;
    const int img = (int)(pix / ohw);
    const int rem = (int)(pix - (int64_t)img * ohw);
    const int sy = rem / a.out_w, sx = rem - sy * a.out_w;      // stored output
    static_cast<T*>(a.y)[((int64_t)img * a.c_out + a.perm[pos]) * ohw + rem] = k0_output<T>(a, img, pos, sy, sx);
}

}  // namespace ppc
