// Host-side plan: the layer-wise representation after filter kernel reorder, and the packed
// device streams built from it (paper section 2.3.1, "Filter Kernel Reorder and Compact
// Filter-Kernel-Weight (FKW) Storage").  No HIP types here.
#pragma once

#include <cstdint>
#include <vector>

#include "pp_conv.h"
#include "tile_geom.hpp"
#include "mfma_geom.hpp"
#include "mfma3_geom.hpp"

namespace ppc {

struct Canonical {          // tuning-independent result of the reorder
    std::vector<int32_t> perm, kcount, pat_off, kidx;
    std::vector<uint8_t> kpat;
    std::vector<float> wpacked;
    int64_t k_kept = 0;
};

// One built-in four-tap pattern standing in for (part of) a layer pattern: its slot, and for each of its four
// taps (ascending) the index of the layer kernel's weight that goes there, or -1 for a zero.
struct CoverPart {
    int slot = 0;
    int src[4] = {-1, -1, -1, -1};
};

struct TiledLayout {        // geometry of the tiled kernel for one plan
    int np = 0;             // pattern slots compiled in (8 or 16)
    int f = 0, r = 0, lw = 0, wf = 0, ks = 0, cc = 0;
    int mode = 0;           // input staging: 0 through registers, 1 direct loads in 16-byte slots, 2 in 4-byte slots
    int nbuf = 1;           // tile buffers in LDS: 1, or the ring size of direct staging (2..8)
    int sw = 1;             // workgroups that share one output tile, each on its own range of channel chunks
    int groups = 0;         // G = ceil(c_out / f)
    int chunks = 0;         // Q = ceil(c_in / cc)
    int entry_words = 8;    // 32-bit words per entry: 8 (code, channel, 2 spare, 4 fp32 weights) or 4 (code, 2 words of binary16 pairs, channel)
    bool covered = false;   // some pattern runs as several built-in patterns with zero weights (no round trip of the stream)
    std::vector<std::vector<CoverPart>> cover;   // [pattern] the built-in patterns that stand for it
    int32_t idle_off = 0;   // first entry of the run of end-of-chunk entries walked by wavefronts without a filter group
    std::vector<uint32_t> stream;      // entries
    std::vector<int32_t> wave_off;     // [G*ks*sw] first entry of each (group, split) wavefront stream in each workgroup share
    std::vector<int32_t> slot_pos;     // [G*f] position in the reordered filter list of the filter in each slot, -1 for padding
    std::vector<int32_t> chan_map;     // [filter blocks][chunks*cc] input channel staged at each place of each chunk, -1 for padding
    std::vector<int32_t> perm_pad;     // [G*f] original filter index by slot, -1 for padding
    std::vector<float> bias_pad;       // [G*f]
};

// Matrix-core kernel: the pruned weights zero-filled to a dense [c_out][K*K*c_in] binary16 matrix,
// cut into MFMA operand fragments in the order the kernel reads them.
struct MfmaLayout {
    int tr = 0, tc = 0, ntw = 0;      // workgroup tile (rows of the tall virtual image x columns) and MFMA column tiles per wavefront
    int waves = 4;                    // wavefronts per workgroup (4 or 8)
    bool direct = false;              // the direct-load kernel (3x3, stride 1, whole chunks of 16 channels) runs this plan
    K3Geom g3;                        // ... with this geometry
    int cpad = 0;                     // ... on this many input channels: c_in rounded up to whole chunks (a larger value than c_in means x is copied into a zero-padded buffer first)
    bool rows = false;                // of the 3x3, stride 1 kernels the row-stacked one runs this plan, not the direct-load one
    int ksplit = 1;                   // ... and this many workgroups sharing a tile's reduction (partial sums to a workspace)
    bool pairs = true;                // images more than one pixel wide: input loaded as 32-bit pixel pairs
    int units = 0;                    // staging units (16 pixel pairs x 8 channels) of a wavefront
    int po = 0;                       // rows per image in the tall virtual output image (ho + separator rows)
    int trp = 0, twpa = 0;            // staged input rows per tile: (tr-1)*stride + K; staged columns: (tc-1)*stride + K + 2, rounded down to even
    int fb = 0, q = 0;                // filter blocks of 64, channel chunks of 16
    int upq = 1;                      // weight units per chunk: 1 (all taps at once) or K (one tap row at a time)
    int gw = 1;                       // output elements per store (8, 4, 2 or 1)
    int xbuf_bytes = 0, wbuf_bytes = 0, out_pitch = 0;
    int64_t lds_bytes = 0;
    std::vector<uint16_t> wpk;        // [fb][q][K*K][2][64][8] binary16 bits
    std::vector<float> bias_pad;      // [fb*64]
};

constexpr int kF32Pad = 4;                  // units the kernels of the binary32 instruction may load past the end
// Binary32 matrix-core kernels: the zero-filled dense weights in operand order, as they are or each in three bfloat16 parts.
struct F32Layout {
    bool whole = false;                     // as they are, for k5_whole_f32
    int asked = 0;                          // by the tuning: 1 for k5_whole_f32, 3 for k5_conv_f32
    int groups = 0, units = 0, tiles = 0;   // groups of sixteen channels (eight), ks * ks * groups, 32-filter tiles (rounded up to what a wavefront takes: k5_padded_tiles, or a multiple of two)
    std::vector<uint16_t> wpk;              // [tiles][units][3][64][8]
    std::vector<float> wpk_whole;          // [tiles][units][64][4], and kF32Pad units of zeros behind them
    std::vector<float> bias_pad;            // [tiles * 32]
};

// Binary32 3x3 kernel on the small matrix instruction: weights by 16-filter group and channel.
struct QuadLayout {
    int groups = 0;                         // of 16 filters
    std::vector<float> wpk;                 // [groups][c_in][64][4]
    std::vector<uint32_t> used;             // [groups][c_in][2] taps that any filter of a quad uses
    std::vector<float> bias_pad;            // [groups * 16]
    double taps_used = 0.0;                 // mean over quads and channels
};

struct HostPlan {
    int32_t c_in = 0, c_out = 0, h = 0, w = 0, n_hint = 1, num_patterns = 0, taps = 4;
    int32_t ks = 3, stride = 1;         // kernel size, stride
    bool pool = false;                  // fused 2x2 max-pool
    int32_t ho = 0, wo = 0;             // the convolution's output size
    int32_t out_h = 0, out_w = 0;       // size of y (pooled if pool)
    uint32_t flags = 0;
    int32_t dtype = 0;
    std::vector<uint64_t> masks;
    std::vector<float> bias;            // [c_out], zeros if absent
    Canonical canon;
    pp_conv_tuning_t chosen{};
    bool tiled = false;                 // the tiled vector kernel runs the plan
    TiledLayout tl;
    bool mfma = false;
    MfmaLayout ml;
    bool dense32 = false;               // binary32 layer that runs as a dense product on the matrix cores
    F32Layout fl;
    bool quads = false;                 // binary32 3x3, stride 1 layer that runs on the small matrix instruction
    QuadLayout ql;
    // generic kernel tables
    std::vector<int32_t> filt_off;      // [c_out+1] prefix of kcount
    std::vector<int8_t> tap_dyx;        // [P*taps*2] (dy, dx) per tap
};

// Validate desc; PP_OK or the error the header documents.
pp_status_t validate(const pp_conv_desc_t& d);
// Reorder (fills hp.canon and the scalar fields).  desc must be valid.
void build_canonical(const pp_conv_desc_t& d, HostPlan& hp);
// Choose variant and parameters, build the device-format arrays.  PP_ERR_UNSUPPORTED if the
// tuning request cannot be honoured.
pp_status_t build_layouts(const pp_conv_desc_t& d, HostPlan& hp);
// Choose the matrix-core kernel's tile and pack its weights (hp.ml).  PP_ERR_UNSUPPORTED if the layer
// or the tuning request does not fit.
pp_status_t build_mfma_layout(const pp_conv_tuning_t& t, HostPlan& hp);
// Pack the weights of a binary32 layer for the matrix-core kernel (hp.fl).
void build_f32_layout(HostPlan& hp);
// Pack the weights of a binary32 3x3, stride 1 layer for the small matrix instruction (hp.ql).
void mark_quad_taps(HostPlan& hp);
void pack_quads(HostPlan& hp);
// Decode tl.stream, or the operands of a binary32 3x3 plan, back to canonical order.
pp_status_t unpack_stream(const HostPlan& hp, int32_t* kidx, uint8_t* kpat, float* w);

// binary16 conversion used when packing weights (round to nearest even).
uint16_t f32_to_f16_rne(float v);
// A binary32 value as the sum of three bfloat16 ones (round to nearest even, each what the ones before it leave); bits below 2^-133 are
// left out.
void split_bf16(float v, uint16_t (&part)[3]);
float bf16_to_f32(uint16_t b);
float f16_to_f32(uint16_t b);

}  // namespace ppc
