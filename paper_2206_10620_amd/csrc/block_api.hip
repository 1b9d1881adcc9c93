// C ABI of the block-pruned matrix product (include/pp_block_gemm.h): plan upload, launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <new>

#include "block_plan.hpp"
#include "k4_block_gemm.hpp"
#include "k5_f32.hpp"

struct pp_block_gemm_plan {
    ppc::BlockHostPlan hp;
    bool on_device = false;
    void* d_apk = nullptr;
    float* d_bias = nullptr;
    int32_t* d_tile_off = nullptr;
    int32_t* d_tile_cols = nullptr;
    float* d_wpk32 = nullptr;
    int32_t* d_list32 = nullptr;
    int32_t* d_group_off32 = nullptr;
};

namespace {

using namespace ppc;

template <typename T>
bool put(T** dst, const void* src, size_t bytes, size_t pad_bytes = 0) {
    void* p = nullptr;
    if (hipMalloc(&p, bytes + pad_bytes + 16) != hipSuccess) return false;
    *dst = static_cast<T*>(p);
    if (hipMemset(p, 0, bytes + pad_bytes + 16) != hipSuccess) return false;
    if (bytes && hipMemcpy(p, src, bytes, hipMemcpyHostToDevice) != hipSuccess) return false;
    return true;
}

void release(pp_block_gemm_plan_t* p) {
    void* bufs[] = {p->d_apk, p->d_bias, p->d_tile_off, p->d_tile_cols, p->d_wpk32, p->d_list32, p->d_group_off32};
    for (void* b : bufs)
        if (b) (void)hipFree(b);
}

struct K4Shape {
    int cols;                                                  // columns of a workgroup
    void (*launch)(const K4Args& a, int blocks, hipStream_t stream);
};

template <bool RAGGED> void launch_wide_as(const K4Args& a, int blocks, hipStream_t stream) {
    static const hipError_t lds_attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&k4_block_gemm<RAGGED>), hipFuncAttributeMaxDynamicSharedMemorySize, kK4LdsBytes);
    (void)lds_attr;
    hipLaunchKernelGGL(k4_block_gemm<RAGGED>, dim3((unsigned)blocks), dim3(256), kK4LdsBytes, stream, a);
}
void launch_wide(const K4Args& a, int blocks, hipStream_t stream) {
    if (a.ragged) launch_wide_as<true>(a, blocks, stream);
    else launch_wide_as<false>(a, blocks, stream);
}
template <int NT, int WK> void launch_split(const K4Args& a, int blocks, hipStream_t stream) {
    constexpr int lds = k4_split_lds_bytes(NT, WK);
    static const hipError_t lds_attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&k4_split<NT, WK>), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    (void)lds_attr;
    hipLaunchKernelGGL((k4_split<NT, WK>), dim3((unsigned)blocks), dim3(64 * WK), lds, stream, a);
}

// Which tile a launch runs with: the smallest modelled time.  A workgroup of the split kernel walks chunks / wk chunks per
// wavefront, each worth 0.14 us of latency and, for every wavefront on the compute unit, nt + 2 KB through the vector cache
// (0.012 us per KB), and a round of them 2.1 us and its stores; the 512-column tile takes 3.65 us and, two to a compute unit,
// 0.74 us per chunk, 0.28 where few run, and 2.6 us more where pieces straddle rows.  Fitted to 370 products timed with every
// tile (1 to 8192 columns, 8 to 4096 rows, 4 to 4096 columns of weights, 1- to 64-wide blocks): the pick is 1.2 % from the best
// on average, 1.28 times at worst.  4096 x 4096 at 0.41 on 4096 columns: 512-column tile 63 us, 4 x 4 104 modelled; 1775 x 23 on
// 181 columns: 1 x 8 4.6 us, 512-column tile 9.8.
K4Shape k4_pick(const BlockHostPlan& hp, int n, int batch) {
    struct Split { int nt, wk, resident; K4Shape shape; };
    static const Split kSplits[] = {{1, 4, 4, {32, launch_split<1, 4>}}, {1, 8, 2, {32, launch_split<1, 8>}}, {2, 4, 3, {64, launch_split<2, 4>}},
                                    {2, 8, 1, {64, launch_split<2, 8>}}, {4, 4, 2, {128, launch_split<4, 4>}}, {4, 8, 1, {128, launch_split<4, 8>}}};
    const K4Shape wide{kBlockColTile, launch_wide};
    if (hp.k >= (1 << 24) || n >= (1 << 23)) return wide;       // the split kernel multiplies in 24 bits
    const double chunks = (double)hp.tile_cols.size() / kBlockChunk / hp.row_tiles;
    auto wgs = [&](int cols) { return (int64_t)hp.row_tiles * ((n + cols - 1) / cols) * batch; };
    const int64_t full = wgs(kBlockColTile) / 512, rest = wgs(kBlockColTile) % 512;
    K4Shape best = wide;
    double best_t = (double)full * (3.65 + chunks * 0.737) + (rest ? 3.65 + chunks * (0.276 + 0.0009 * (double)rest) : 0.0) + (n % 8 ? 2.6 : 0.0);
    for (const Split& s : kSplits) {
        const double share = chunks / s.wk > 1.0 ? chunks / s.wk : 1.0;
        auto round = [&](int64_t k) { return k == 0 ? 0.0 : share * 0.137 + (double)k * s.wk * share * (s.nt + 2) * 0.012 + 0.72 * s.nt * (0.25 + 0.75 * (double)k) + 2.1; };
        const int64_t p = (wgs(s.shape.cols) + 255) / 256;
        const double t = (double)(p / s.resident) * round(s.resident) + round(p % s.resident);
        if (t < best_t) best_t = t, best = s.shape;
    }
    return best;
}

}  // namespace

pp_status_t pp_block_gemm_launch_batched(const pp_block_gemm_plan_t* plan, const void* x_dev, void* y_dev, int32_t n, int32_t batch, int64_t x_stride,
                                         int64_t y_stride, void* hip_stream) {
    if (!plan || !x_dev || !y_dev) return PP_ERR_NULL;
    const BlockHostPlan& hp = plan->hp;
    if (n < 1 || batch < 1 || hp.dtype != PP_F16 || !plan->on_device) return PP_ERR_UNSUPPORTED;
    if ((int64_t)hp.k * n >= ((int64_t)1 << 31) || (int64_t)hp.m * n >= ((int64_t)1 << 31)) return PP_ERR_SHAPE;
    K4Args a;
    a.x = x_dev, a.y = y_dev, a.apk = plan->d_apk, a.bias = plan->d_bias;
    a.tile_off = plan->d_tile_off, a.tile_cols = plan->d_tile_cols;
    a.m = hp.m, a.n = n, a.row_tiles = hp.row_tiles;
    a.relu = (hp.flags & PP_FLAG_RELU) ? 1 : 0;
    a.ragged = (n % 8) != 0 ? 1 : 0;
    a.x_bytes = (uint32_t)((int64_t)hp.k * n * 2);
    a.x_stride = x_stride, a.y_stride = y_stride;
    const K4Shape sh = k4_pick(hp, n, batch);
    a.col_tiles = (n + sh.cols - 1) / sh.cols;
    const int64_t items = (int64_t)a.row_tiles * a.col_tiles * batch;
    if (items >= ((int64_t)1 << 28)) return PP_ERR_SHAPE;
    a.items = (int)items;
    a.per_xcd = (a.items + 7) / 8;
    (void)hipGetLastError();
    sh.launch(a, a.per_xcd * 8, static_cast<hipStream_t>(hip_stream));
    return hipGetLastError() == hipSuccess ? PP_OK : PP_ERR_DEVICE;
}

// Binary32 on the matrix cores.  PP_ERR_UNSUPPORTED if x does not fit 31-bit byte offsets.
static pp_status_t launch_list_f32(const pp_block_gemm_plan_t* plan, const void* x_dev, void* y_dev, int32_t n, hipStream_t stream) {
    const BlockHostPlan& hp = plan->hp;
    K5ListArgs a{};
    a.x_bytes = (int64_t)hp.k * n * 4;
    if (a.x_bytes >= ((int64_t)1 << 31)) return PP_ERR_UNSUPPORTED;
    a.x = static_cast<const float*>(x_dev), a.y = static_cast<float*>(y_dev);
    a.wpk = plan->d_wpk32, a.bias = plan->d_bias, a.list = plan->d_list32, a.group_off = plan->d_group_off32;
    a.m = hp.m, a.n = n, a.relu = (hp.flags & PP_FLAG_RELU) ? 1 : 0;
    a.row_tiles = (hp.m + kBlockRow32 - 1) / kBlockRow32;
    const K5Shape sh = k5_pick_list(a.row_tiles, n, hp.group_off32.back() / a.row_tiles);
    a.col_tiles = (n + 32 * sh.nt - 1) / (32 * sh.nt);
    const int64_t items = (int64_t)a.row_tiles * a.col_tiles;
    if (items >= ((int64_t)1 << 28)) return PP_ERR_UNSUPPORTED;
    a.items = (int32_t)items, a.per_xcd = (a.items + 7) / 8;
    const k5_list_fn fn = k5_list_lookup(sh);
    if (!fn) return PP_ERR_UNSUPPORTED;
    (void)hipGetLastError();
    hipLaunchKernelGGL(fn, dim3((unsigned)(a.per_xcd * 8)), dim3((unsigned)(64 * sh.wk)), 0, stream, a);
    return hipGetLastError() == hipSuccess ? PP_OK : PP_ERR_DEVICE;
}

extern "C" {

pp_status_t pp_block_gemm_plan(const pp_block_gemm_desc_t* desc, pp_block_gemm_plan_t** out_plan) {
    if (out_plan) *out_plan = nullptr;
    if (!desc || !out_plan) return PP_ERR_NULL;
    pp_block_gemm_plan_t* p = nullptr;
    try {
        p = new pp_block_gemm_plan_t();
        const pp_status_t st = build_block_plan(*desc, p->hp);
        if (st != PP_OK) {
            delete p;
            return st;
        }
    } catch (const std::bad_alloc&) {
        delete p;
        return PP_ERR_ALLOC;
    }
    if (!(desc->flags & PP_FLAG_HOST_ONLY)) {
        const BlockHostPlan& hp = p->hp;
        bool ok = put(&p->d_apk, hp.apk.data(), hp.apk.size() * sizeof(uint16_t));
        ok = ok && put(&p->d_bias, hp.bias.data(), hp.bias.size() * sizeof(float));
        ok = ok && put(&p->d_tile_off, hp.tile_off.data(), hp.tile_off.size() * sizeof(int32_t));
        ok = ok && put(&p->d_tile_cols, hp.tile_cols.data(), hp.tile_cols.size() * sizeof(int32_t), 256 * sizeof(int32_t));   // the kernels read ahead: a chunk, or two segments of 128
        if (hp.variant == 1) {
            ok = ok && put(&p->d_wpk32, hp.wpk32.data(), hp.wpk32.size() * sizeof(float));
            ok = ok && put(&p->d_list32, hp.list32.data(), hp.list32.size() * sizeof(int32_t));
            ok = ok && put(&p->d_group_off32, hp.group_off32.data(), hp.group_off32.size() * sizeof(int32_t));
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

pp_status_t pp_block_gemm_run(const pp_block_gemm_plan_t* plan, const void* x_dev, void* y_dev, int32_t n, void* hip_stream) {
    if (!plan || !x_dev || !y_dev) return PP_ERR_NULL;
    const BlockHostPlan& hp = plan->hp;
    if (n < 1 || (int64_t)hp.k * n >= ((int64_t)1 << 31) || (int64_t)hp.m * n >= ((int64_t)1 << 31)) return PP_ERR_SHAPE;
    const int64_t eb = hp.dtype == PP_F16 ? 2 : 4;
    const uintptr_t xa = reinterpret_cast<uintptr_t>(x_dev), ya = reinterpret_cast<uintptr_t>(y_dev);
    if ((xa | ya) & 15u) return PP_ERR_ALIGN;
    const uintptr_t xe = xa + (uintptr_t)((int64_t)hp.k * n * eb), ye = ya + (uintptr_t)((int64_t)hp.m * n * eb);
    if (xa < ye && ya < xe) return PP_ERR_ALIGN;
    if (hp.variant == 2 && hp.forced && (n % 8) != 0) return PP_ERR_UNSUPPORTED;        // what the header promises of a forced variant
    if (!plan->on_device) return PP_ERR_UNSUPPORTED;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const int relu = (hp.flags & PP_FLAG_RELU) ? 1 : 0;
    (void)hipGetLastError();
    if (hp.variant == 2) return pp_block_gemm_launch_batched(plan, x_dev, y_dev, n, 1, 0, 0, hip_stream);
    if (hp.dtype == PP_F32) {
        const pp_status_t st = launch_list_f32(plan, x_dev, y_dev, n, stream);
        if (st != PP_ERR_UNSUPPORTED) return st;
    }
    {
        const dim3 grid((unsigned)((n + 63) / 64), (unsigned)hp.row_tiles), block(64, 4);
        if (hp.row_tiles > 65535) return PP_ERR_SHAPE;
        if (hp.dtype == PP_F16)
            hipLaunchKernelGGL(k4_generic<_Float16>, grid, block, 0, stream, static_cast<const _Float16*>(x_dev), static_cast<_Float16*>(y_dev),
                               plan->d_wpk32, plan->d_bias, plan->d_group_off32, plan->d_list32, hp.m, n, relu);
        else
            hipLaunchKernelGGL(k4_generic<float>, grid, block, 0, stream, static_cast<const float*>(x_dev), static_cast<float*>(y_dev), plan->d_wpk32,
                               plan->d_bias, plan->d_group_off32, plan->d_list32, hp.m, n, relu);
    }
    return hipGetLastError() == hipSuccess ? PP_OK : PP_ERR_DEVICE;
}

pp_status_t pp_block_gemm_destroy(pp_block_gemm_plan_t* plan) {
    if (!plan) return PP_OK;
    release(plan);
    delete plan;
    return PP_OK;
}

pp_status_t pp_block_gemm_query(const pp_block_gemm_plan_t* plan, pp_block_gemm_info_t* out) {
    if (!plan || !out) return PP_ERR_NULL;
    const BlockHostPlan& hp = plan->hp;
    out->m = hp.m, out->k = hp.k, out->block_m = hp.bm, out->block_k = hp.bk;
    out->variant = hp.variant;
    out->row_tile = kBlockRowTile;
    out->row_tiles = hp.row_tiles;
    out->kept_weights = hp.kept_weights;
    out->executed_weights = hp.executed_weights;
    out->tile_off = hp.tile_off.data();
    out->tile_cols = hp.tile_cols.data();
    out->tile_len = hp.tile_len.data();
    return PP_OK;
}

pp_status_t pp_block_gemm_unpack(const pp_block_gemm_plan_t* plan, int32_t tile, float* w_out) {
    if (!plan || !w_out) return PP_ERR_NULL;
    return unpack_block_tile(plan->hp, tile, w_out);
}

}  // extern "C"
