// Internal to the C API: the handle structs behind include/hyb.h's opaque
// handles and the argument helpers shared by the entry-point sources.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "hyb.h"
#include "hyb_device.hpp"
#include "kernels.hpp"

struct hyb_bvh_s {
    int device = 0;
    void* memory = nullptr;    // one allocation, which the arrays below share
    float4* nodes4 = nullptr;  // four children per node (128 bytes)
    unsigned long long* boundary = nullptr;  // launch_mesh_boundary's sum
    int32_t* entry = nullptr;  // traversal entry pyramid (BvhHost::entry)
    hyb::EntryGrid grid;       // the pyramid's placement
    float4* tris = nullptr;
    int64_t n_nodes = 0, n_tris = 0;  // n_nodes counts the four-wide nodes
    int32_t depth = 0;
    float lo[3] = {0, 0, 0}, hi[3] = {0, 0, 0};
};

struct hyb_sdf_s {
    int device = 0;
    float* values = nullptr;  // n^3 FP32 samples as the kernels see them (dequantized), x fastest
    void* store = nullptr;    // the samples the kernels read: storage format, bricked layout
    float* scales = nullptr;  // I8 block scales
    int32_t n = 0, nb = 0;
    float grid4[4] = {0, 0, 0, 0};
    float lipschitz = 0.0f;
    float slope[3] = {0, 0, 0};  // per-axis bounds of |df/dx_i|
    bool certified = false;  // samples are FP32 roundings of a 1-Lipschitz function
    hyb_sdf_format fmt = HYB_SDF_F32;
    int32_t layout = 0;  // the kernels' storage format and brick layout (hyb::SdfFormat)
    float* blocks = nullptr;  // per-block maxima of launch_store (kept for updates)
    uint64_t version = 0;     // bumped whenever the samples and bounds change (batches re-read them)
    float* dev_bounds = nullptr;  // hyb::kDeviceBounds floats: the bounds of the last update
    bool deferred = false;        // the last update was deferred: the kernels read dev_bounds
    void* bwd_ws = nullptr;       // hyb_df_backward's sort buffers, grown on demand
    size_t bwd_ws_bytes = 0;
    int64_t bwd_n = 0;            // the ray count whose buffer size bwd_need holds
    size_t bwd_need = 0;
};

namespace hyb_api {

inline hyb_status from_hip(hipError_t e) {
    if (e == hipSuccess) return HYB_OK;
    if (e == hipErrorOutOfMemory) return HYB_ERR_OOM;
    return HYB_ERR_HIP;
}

#define HYB_TRY(expr)                               \
    do {                                            \
        hyb_status s_ = from_hip(expr);             \
        if (s_ != HYB_OK) return s_;                \
    } while (0)

inline bool same_device(int dev) {
    int cur = -1;
    return hipGetDevice(&cur) == hipSuccess && cur == dev;
}

inline bool valid_rays(const hyb_rays* r) {
    return r && r->ox && r->oy && r->oz && r->dx && r->dy && r->dz;
}

inline bool valid_hits(const hyb_hits* h) { return h && h->t && h->prim && h->u && h->v; }

// The certified-grid step slack of the kernels, or +inf.
inline float two_e_of(const hyb_sdf_s* s) {
    return (s->certified && s->fmt == HYB_SDF_F32) ? hyb::certified_slack(s->grid4[3], s->n) : __builtin_inff();
}

// Allocates the kernels' copy of the samples; *bytes receives its size.
inline hyb_status allocate_store(hyb_sdf_s* s, size_t* bytes) {
    const int fmt = s->fmt == HYB_SDF_F32 ? hyb::kF32 : (s->fmt == HYB_SDF_F16 ? hyb::f16_layout(s->n) : hyb::kI8);
    s->layout = fmt;
    const size_t count = static_cast<size_t>(hyb::brick_storage(fmt, s->n));
    const size_t elem = s->fmt == HYB_SDF_F32 ? 4 : (s->fmt == HYB_SDF_F16 ? 2 : 1);
    s->nb = hyb::i8_blocks(s->n);
    *bytes = count * elem;
    HYB_TRY(hipMalloc(&s->store, count * elem));
    if (s->fmt == HYB_SDF_I8_BRICK)
        HYB_TRY(hipMalloc(&s->scales, sizeof(float) * static_cast<size_t>(s->nb) * s->nb * s->nb));
    return HYB_OK;
}

// Where the kernels read the caller's n^3 samples.  Device memory of this device is
// read in place, if the allocation holds that many.  Other memory (of the host or
// another device, which kernels may not be able to read) is copied into s->values first.
inline hyb_status sample_source(hyb_sdf_s* s, const float*& in, hipStream_t stream) {
    const size_t bytes = sizeof(float) * static_cast<size_t>(s->n) * s->n * s->n;
    hipPointerAttribute_t at;
    if (hipPointerGetAttributes(&at, in) == hipSuccess && at.type == hipMemoryTypeDevice && at.device == s->device) {
        hipDeviceptr_t base = nullptr;
        size_t size = 0;
        HYB_TRY(hipMemGetAddressRange(&base, &size, const_cast<float*>(in)));
        const size_t offset = static_cast<size_t>(reinterpret_cast<const char*>(in) - static_cast<const char*>(base));
        return offset <= size && bytes <= size - offset ? HYB_OK : HYB_ERR_HIP;
    }
    (void)hipGetLastError();  // memory that HIP does not know is not an error here
    HYB_TRY(hipMemcpyAsync(s->values, in, bytes, hipMemcpyDefault, stream));
    in = s->values;
    return HYB_OK;
}

// Stores the samples `in` (launch_store) with their step bounds.  Deferred, the
// bounds stay on the device; else this waits for them, and a sample that is not
// finite (or an F16 overflow) is an error.
inline hyb_status store_samples(hyb_sdf_s* s, const float* in, bool deferred, hipStream_t stream) {
    if (in != s->values) {
        const hyb_status rc = sample_source(s, in, stream);
        if (rc != HYB_OK) return rc;
    }
    if (!s->blocks) HYB_TRY(hipMalloc(&s->blocks, sizeof(float) * hyb::kBoundValues * hyb::store_blocks(s->n)));
    if (!s->dev_bounds) HYB_TRY(hipMalloc(&s->dev_bounds, sizeof(float) * hyb::kDeviceBounds));
    HYB_TRY(hyb::launch_store(s->layout, in, s->n, s->grid4[3], s->values, s->store, s->scales, s->blocks, two_e_of(s),
                              s->dev_bounds, stream));
    if (!deferred) {
        float b[hyb::kDeviceBounds];
        HYB_TRY(hipMemcpyAsync(b, s->dev_bounds, sizeof(b), hipMemcpyDeviceToHost, stream));
        HYB_TRY(hipStreamSynchronize(stream));
        if (b[hyb::kBBad] != 0.0f) return HYB_ERR_INVALID_ARG;
        s->lipschitz = b[hyb::kBLipschitz];
        s->slope[0] = b[hyb::kBSlopeX];
        s->slope[1] = b[hyb::kBSlopeY];
        s->slope[2] = b[hyb::kBSlopeZ];
    }
    s->deferred = deferred;
    ++s->version;
    return HYB_OK;
}

inline bool valid_fmt(hyb_sdf_format f) { return f == HYB_SDF_F32 || f == HYB_SDF_F16 || f == HYB_SDF_I8_BRICK; }

inline bool valid_grid4(const float* g) {
    return g && std::isfinite(g[0]) && std::isfinite(g[1]) && std::isfinite(g[2]) && std::isfinite(g[3]) &&
           g[3] > 0.0f;
}

inline void fill_trace_args(hyb::TraceArgs& a, const hyb_rays* rays, hyb_hits* hits, int64_t n, float tmax, float tau,
                     float tau_end = 0.0f) {
    std::memset(&a, 0, sizeof(a));
    a.ox = rays->ox; a.oy = rays->oy; a.oz = rays->oz;
    a.dx = rays->dx; a.dy = rays->dy; a.dz = rays->dz;
    a.tmin = rays->tmin;
    a.tmax_ray = rays->tmax;
    a.tau_end = tau_end;
    a.t = hits->t; a.prim = hits->prim; a.u = hits->u; a.v = hits->v;
    a.tmax = tmax;
    a.tau = tau;
    a.n = n;
}

// Bytes of the kernels' bricked copy of a grid.
inline int64_t copy_bytes(const hyb_sdf_s* s) {
    const int64_t elem = s->layout == hyb::kF32 ? 4 : (s->layout == hyb::kI8 ? 1 : 2);
    return hyb::brick_storage(s->layout, s->n) * elem;
}

inline void fill_scene(hyb::TraceArgs& a, const hyb_bvh_s* b, const hyb_sdf_s* s) {
    a.xcd_run = hyb::xcd_run_for(s ? copy_bytes(s) : 0);
    if (b) {
        a.nodes = b->nodes4;
        a.entry = b->grid.res ? b->entry : nullptr;
        a.entry_lo_x = b->grid.lo[0];
        a.entry_lo_y = b->grid.lo[1];
        a.entry_lo_z = b->grid.lo[2];
        a.entry_inv = b->grid.res ? 1.0f / b->grid.size : 0.0f;
        a.entry_res = b->grid.res;
        a.entry_levels = b->grid.levels;
        a.tris = b->tris;
    }
    if (s) {
        a.sdf = s->store;
        a.fmt = s->layout;
        a.n_grid = s->n;
        a.lo_x = s->grid4[0];
        a.lo_y = s->grid4[1];
        a.lo_z = s->grid4[2];
        a.h = s->grid4[3];
        a.inv_h = 1.0f / s->grid4[3];
        a.inv_hd = 1.0 / (double)s->grid4[3];
        a.inv_l = hyb::inv_step(s->lipschitz);
        a.two_e = two_e_of(s);
        a.bounds = s->deferred ? s->dev_bounds : nullptr;
        a.slope_x = s->slope[0];
        a.slope_y = s->slope[1];
        a.slope_z = s->slope[2];
    }
}

inline hyb_status check_query(const hyb_rays* rays, int64_t n, float tmax, hyb_hits* hits) {
    if (n < 0 || n > HYB_MAX_RAYS || std::isnan(tmax) || tmax < 0.0f) return HYB_ERR_INVALID_ARG;
    if (n > 0 && (!valid_rays(rays) || !valid_hits(hits))) return HYB_ERR_INVALID_ARG;
    return HYB_OK;
}

}  // namespace hyb_api
