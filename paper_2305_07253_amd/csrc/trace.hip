// Trace kernels: the combined query and the two pure baselines.
//
// One ray per lane (in small launches, several lanes per ray).  Rays and hits are SoA
// arrays, so each of the seven input and four output streams is read or written with
// fully coalesced 256-byte wavefront accesses.  The BVH stack lives in LDS ([depth][thread] so the 64
// lanes of a wavefront hit 64 distinct banks), with a small private spill area
// for the rare paths deeper than the LDS part.
#include "hyb_device.hpp"
#include "kernels.hpp"

namespace hyb {

// Rays of a wavefront, as a power of two: 64, and fewer for a launch that would
// leave most of the chip idle.  Such a launch lasts as long as its slowest
// wavefront, which runs every path that any of its rays takes; with fewer rays
// each it runs fewer, on SIMDs that had nothing to do.  A wavefront of 2^k rays
// traces each in 64 >> k lanes alike (same instructions, same loads, same
// values stored), because wavefronts with few active lanes on an otherwise idle
// SIMD issue vector instructions at a quarter of the rate.
// Up to 2,048 wavefronts that way (two per SIMD): 1,000 rays of the small room
// at threshold 1 44 -> 25 us, triangles only 45 -> 24 us, of the GI scene 61 ->
// 30 and 103 -> 46 us; at 16,384 rays 78 -> 72 and 102 -> 78 us, at 65,536 92 ->
// 85 and 118 -> 105 us, at 262,144 (64 rays each already) 32 rays would take 146
// for 113 us.  The distance field alone diverges less: to 1,024 wavefronts and
// 8,192 rays (1,000 rays 29 -> 25 us, 4,096 34 -> 27 us), 16,384 rays took 3 to
// 5% longer.  Launches that share the chip with others pay for their spread: four
// streams of 1,000 rays each through the GI scene 27 -> 14 us a launch, of 16,384 28 to
// 31 -> 31, of 65,536 random rays in the small room 14 -> 17 (half as many wavefronts
// would take 14 there, and alone 50% longer at 4,000 rays).
uint32_t rays_shift(int mode, int64_t n) {
    if (mode == kDfOnly && n > 8192) return 6;
    const int64_t waves = mode == kDfOnly ? 1024 : 2048;
    uint32_t shift = 0;
    while (shift < 6 && n > (waves << shift)) ++shift;
    return shift;
}

// Wavefronts per SIMD the compiler is held to where that measured faster:
// one-cell F16 bricks, 74 VGPRs left alone, fit seven at 72; the combined I8
// query, which forms its solves again (df_resolve) to fit, seven at 70.
template <int MODE, int FMT, bool COUNT>
constexpr int trace_waves() {
    if (COUNT) return 1;
    if (FMT == kF16 && (MODE == kCombined || MODE == kDfOnly)) return 7;
    if (FMT == kI8 && MODE == kCombined) return 7;
    return 1;
}

template <int MODE, int FMT, bool COUNT, int SEG>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(trace_waves<MODE, FMT, COUNT>())))
void k_trace(TraceArgs a, uint32_t shift) {
    extern __shared__ int s_stack[];
    const int64_t i = ((int64_t)xcd_block(blockIdx.x, gridDim.x, a.xcd_run) << shift) +
                      (threadIdx.x & ((1u << shift) - 1));
    if (i >= a.n) return;
    trace_ray<MODE, FMT, COUNT, kLdsDepth, SEG>(a, i, s_stack + threadIdx.x, kBlock);
}

template <int MODE, int FMT, bool COUNT, int SEG>
static hipError_t launch_segments(const TraceArgs& a, hipStream_t stream) {
    const size_t lds = MODE == kDfOnly ? 0 : sizeof(int) * kLdsDepth * kBlock;
    const uint32_t shift = rays_shift(MODE, a.n);
    const int64_t blocks = (a.n + (int64_t(1) << shift) - 1) >> shift;
    hipLaunchKernelGGL((k_trace<MODE, FMT, COUNT, SEG>), dim3((unsigned)blocks), dim3(kBlock), lds, stream, a, shift);
    return hipGetLastError();
}

// Trees whose long segments bvh_closest searches at least as fast as bvh_closest_long:
// voted steps save lane use where many wavefronts' rays part ways, and cost a lane that
// goes its own way its turns, which is what a launch lasts in a small tree.
//   closest hit, 2^19 rays or fewer: 1,052 triangles, an image's rays scattered a little,
//   at 320x176 37 against 50 us and at 640x360 44 against 64, diffuse rays at 640x360 66
//   against 78, at 960x544 106 against 102, at 1920x1080 300 against 285; 2,772 triangles,
//   diffuse rays at 640x360 92 against 82
//   any hit: 1,052 triangles at 480x272 25 against 29 and 36 against 45, at 1920x1080 160
//   against 186; 4,884 triangles at 480x272 51 against 69, diffuse rays 146 against 137;
//   25,740 triangles at 480x272 62 against 67, diffuse rays 162 against 142
template <int MODE>
static bool small_tree(int64_t n_tris, int64_t n) {
    if constexpr (MODE == kShadow) return n_tris <= 8192;
    return n_tris == 0 || (n_tris <= 2048 && n <= (int64_t(1) << 19));
}

// Triangle segments of at most kShortSegment voxels take the traversal for short
// ones, all others (triangles only among them) the one for long ones or small trees.
template <int MODE, int FMT, bool COUNT>
static hipError_t launch(const TraceArgs& a, int64_t n_tris, hipStream_t stream) {
    if constexpr (MODE == kCombined || MODE == kShadow)
        if (short_segments(a)) return launch_segments<MODE, FMT, COUNT, kShortSegments>(a, stream);
    if constexpr (MODE != kDfOnly && !COUNT)
        if (small_tree<MODE>(n_tris, a.n)) return launch_segments<MODE, FMT, COUNT, kSmallTree>(a, stream);
    return launch_segments<MODE, FMT, COUNT, kLongSegments>(a, stream);
}

template <int MODE, bool COUNT>
static hipError_t launch_fmt(const TraceArgs& a, int64_t n_tris, hipStream_t stream) {
    if constexpr (MODE == kBvhOnly) return launch<MODE, kF32, COUNT>(a, n_tris, stream);
    switch (a.fmt) {
        case kF32: return launch<MODE, kF32, COUNT>(a, n_tris, stream);
        case kF16: return launch<MODE, kF16, COUNT>(a, n_tris, stream);
        case kF16B2: return launch<MODE, kF16B2, COUNT>(a, n_tris, stream);
        case kI8: return launch<MODE, kI8, COUNT>(a, n_tris, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_trace(int mode, bool counters, const TraceArgs& args, int64_t n_tris, hipStream_t stream) {
    if (args.n <= 0) return hipSuccess;
    TraceArgs a = args;
    if (a.xcd_run == 0) a.xcd_run = kXcdRun;  // xcd_block needs a run of at least 1
    switch (mode * 2 + (counters ? 1 : 0)) {
        case 0: return launch_fmt<kCombined, false>(a, n_tris, stream);
        case 1: return launch_fmt<kCombined, true>(a, n_tris, stream);
        case 2: return launch_fmt<kBvhOnly, false>(a, n_tris, stream);
        case 3: return launch_fmt<kBvhOnly, true>(a, n_tris, stream);
        case 4: return launch_fmt<kDfOnly, false>(a, n_tris, stream);
        case 5: return launch_fmt<kDfOnly, true>(a, n_tris, stream);
        case 6: return launch_fmt<kShadow, false>(a, n_tris, stream);
        case 7: return launch_fmt<kShadow, true>(a, n_tris, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace hyb
