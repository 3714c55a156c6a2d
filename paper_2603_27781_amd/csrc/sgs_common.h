// Internal definitions shared by the HIP translation units of libsgs.
// Every kernel here targets gfx950 (CDNA4, wave64) only.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include "../../include/sgs.h"

namespace sgs {

constexpr int kWave = 64;

// Constants of the rasterizer derived on the host from gs_config.
struct RasterConst {
    float z_near, blur, guard, alpha_min, alpha_max, T_min;
    float logit_min;  // (float)ln(alpha_min / (1 - alpha_min)): opacity cull
    int32_t tile;
};

// Plain-pointer view of the Gaussian planes, passed by value to kernels.
struct GaussPtrs {
    const float* mu;
    const float* log_scale;
    const float* quat;
    const float* logit;
    const float* color;
    const float* feat;
    int32_t n, n_feat;
};

struct GradPtrs {
    float* mu;
    float* log_scale;
    float* quat;
    float* logit;
    float* color;
    float* feat;
};

__host__ __device__ inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Tile order of the one-workgroup-per-tile launches.  Workgroup b runs on
// XCD b mod 8, and each XCD has its own L2; neighbouring tiles share most of
// their Gaussians, so the tiles go to the XCDs in runs of consecutive tiles
// (the runs dealt round-robin), and the tiles an XCD has in flight are
// neighbours whose shared Gaussian records come from its own L2 instead of
// each being fetched again by another XCD.
constexpr int kXcds = 8;
// log2 of the run length in tiles: about 32 k pixels, less for an image of
// under 64 such runs, so that every XCD gets eight runs and much the same
// share of it.  (With runs of 128 tiles whatever the image, a 333x251 one
// (336 tiles) used three XCDs and at 640x480 two XCDs had twice the tiles of
// the others: backward at F = 16, 30 k Gaussians 107 -> 57 us, 200 k
// Gaussians at 640x480 243 -> 201 us, forward 40 -> 26 and 87 -> 81 us.  One
// round of longer runs: 69 and 229 us.)  A power of two, so that a workgroup
// finds its tile with shifts.
inline int tile_run_log2(int ts, int total_tiles) {
    int run = 2;
    while ((1 << run) * ts * ts < 32768 && (16 * kXcds << run) <= total_tiles) ++run;
    return run;
}
inline unsigned tile_grid(int total_tiles, int run_log2) {
    const int runs = (total_tiles + (1 << run_log2) - 1) >> run_log2;
    return (unsigned)((runs + kXcds - 1) / kXcds * kXcds) << run_log2;
}
// The tile of workgroup b of a tile_grid launch, or -1 (no tile: exit).
__device__ __forceinline__ int tile_of_block(int b, int total_tiles, int run_log2) {
    const int x = b & (kXcds - 1), r = b / kXcds;
    const int t = (((r >> run_log2) * kXcds + x) << run_log2) + (r & ((1 << run_log2) - 1));
    return t < total_tiles ? t : -1;
}

// Index of the view owning global tile t (views sorted by tile_offset).
__device__ inline int view_of_tile(const gs_view* views, int n_views, int t) {
    int v = 0;
    while (v + 1 < n_views && views[v + 1].tile_offset <= t) ++v;
    return v;
}

// Pack two non-negative radii as binary16, rounded up (a conservative box).
__device__ inline float pack_radii(float rx, float ry) {
    __half hx = __float2half_ru(rx);
    __half hy = __float2half_ru(ry);
    uint32_t bits = (uint32_t)__half_as_ushort(hx) | ((uint32_t)__half_as_ushort(hy) << 16);
    return __uint_as_float(bits);
}

__device__ inline float2 unpack_radii(float packed) {
    uint32_t bits = __float_as_uint(packed);
    return make_float2(__half2float(__ushort_as_half((unsigned short)(bits & 0xffffu))),
                       __half2float(__ushort_as_half((unsigned short)(bits >> 16))));
}

// Inclusive scans over the wavefront with DPP (no LDS): row shifts by 1, 2,
// 4, 8 within rows of 16 lanes, then the row broadcasts of lanes 15 and 31
// carry the row totals across rows.  Lanes without a predecessor at a step
// take the identity (-1 for the max over non-negative values, 0 for the sum).
__device__ __forceinline__ int wave_max_scan(int x) {
    x = max(x, __builtin_amdgcn_update_dpp(-1, x, 0x111, 0xf, 0xf, false));  // row_shr:1
    x = max(x, __builtin_amdgcn_update_dpp(-1, x, 0x112, 0xf, 0xf, false));  // row_shr:2
    x = max(x, __builtin_amdgcn_update_dpp(-1, x, 0x114, 0xf, 0xf, false));  // row_shr:4
    x = max(x, __builtin_amdgcn_update_dpp(-1, x, 0x118, 0xf, 0xf, false));  // row_shr:8
    x = max(x, __builtin_amdgcn_update_dpp(-1, x, 0x142, 0xa, 0xf, false));  // row_bcast:15 into rows 1, 3
    x = max(x, __builtin_amdgcn_update_dpp(-1, x, 0x143, 0xc, 0xf, false));  // row_bcast:31 into rows 2, 3
    return x;
}
__device__ __forceinline__ int wave_add_scan(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
    return x;
}

// Exclusive scan of the block's NT thread totals (wave scans, then the wave
// totals in LDS); *total receives the block total.
template <int NT>
__device__ uint32_t block_exclusive(uint32_t v, uint32_t* s_tmp, uint32_t* total) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    // wave inclusive scan (DPP; two's-complement adds are the unsigned ones)
    const uint32_t x = (uint32_t)wave_add_scan((int)v);
    if (lane == kWave - 1) s_tmp[wave] = x;
    __syncthreads();
    uint32_t wbase = 0, tot = 0;
    for (int w = 0; w < NT / kWave; ++w) {
        const uint32_t s = s_tmp[w];
        if (w < wave) wbase += s;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return wbase + x - v;
}

// Fill kernel (used instead of hipMemsetAsync so that calls stay correct
// when captured in a HIP graph and replayed).
__global__ void k_fill_u32(uint32_t* p, uint32_t value, int64_t count);

hipError_t fill_u32(uint32_t* p, uint32_t value, int64_t count, hipStream_t s);

// ---------------------------------------------------------------------------
// launchers (each defined in the translation unit of its kernels)
// ---------------------------------------------------------------------------
hipError_t launch_project(const GaussPtrs& g, const gs_view* views_dev, int n_views, const RasterConst& c,
                          float* rec, uint32_t* rect, int32_t* touched, float* app, int app_stride,
                          hipStream_t s);

size_t binsort_workspace_bytes(int n, int n_views, int64_t capacity);
hipError_t launch_binsort(const uint32_t* rect, const int32_t* touched, int n,
                          const gs_view* views_dev, int n_views, int total_tiles, int max_tiles, int tile, void* ws,
                          int64_t capacity, uint32_t* tile_keys, int32_t* inst, int32_t* inst_gid,
                          int32_t* pair_first, int32_t* ranges, int64_t* counts, hipStream_t s);

// Gaussians staged per LDS batch: the caller's lds_batch at most (and its
// lds_batch_bwd as it is), fewer where the staged batch would leave too few
// workgroups per CU, but not where the tiles are so few that all are resident
// anyway (a larger batch has fewer barriers).  Times in us with 64, 128 and 256,
// scenes of 100 k to 300 k Gaussians unless said.
//
// Forward: one wavefront per workgroup at tile 8 (1200x680, F = 16 127, 173, 270;
// F = 32 205, 265, 503, but 64x64, 64 tiles, 102, 101, 94), 144-byte records at
// F = 32 and tile 16, of which 256 leave three workgroups per CU (16 tiles 111,
// 109, 102, 300 tiles 139, 128, 120, 1200 tiles 100, 96, 105, 25,800 tiles 1264,
// 1147, 1269).
inline int fwd_batch(int tile, int n_feat, int total_tiles, int lds_batch) {
    constexpr int CUS = 256;
    int most = 256;
    if (tile == 8) most = n_feat > 16 && total_tiles <= CUS ? 256 : 64;
    else if (tile == 16 && n_feat > 16 && total_tiles > 3 * CUS) most = 128;
    return lds_batch < most ? lds_batch : most;
}
// Backward, which also holds an accumulator of 10 + F (6 for the pose alone)
// floats per staged Gaussian.  At tile 16 with parameter gradients 128 at
// F = 16 (80 tiles 193, 185, 178, 300 tiles 235, 228, 254, 3225 tiles 387, 359,
// 474, 25,800 tiles 2432, 2312, 3374).  At F = 32 64 or 128, within 8 % of each
// other at every size: 128 is ahead up to 3225 tiles (300 tiles 329, 311, 490,
// 2400 tiles 479, 470, 776, 3225 tiles 574, 552, 1069; not at 1200 tiles, 261,
// 280, 418), 64 from 4800 on (760, 772, 1496; 8160 tiles 1052, 1078, 2139,
// 25,800 tiles 3750, 3832, 7808; 16 mixed views of 2M Gaussians 5149, 5529,
// 10939): the line lies between the two.  For the pose alone 128 at F = 16
// (25,800 tiles 1449, 1386, 1515).  At tile 8 64 (1200x680, F = 16 578, 761,
// 1522); at tile 32 the four times larger workgroups fit as they are (F = 16
// 511, 490, 485).
inline int bwd_batch(int tile, int n_feat, bool params, int total_tiles, int lds_batch, int lds_batch_bwd) {
    constexpr int CUS = 256;
    if (lds_batch_bwd != 0) return lds_batch_bwd;
    int most = 256;
    if (tile == 8) most = 64;
    else if (tile == 16 && n_feat == 16) most = params && total_tiles <= CUS ? 256 : 128;
    else if (tile == 16 && n_feat > 16 && params) most = total_tiles > 4096 ? 64 : 128;
    return lds_batch < most ? lds_batch : most;
}

hipError_t launch_render_fwd(const float* rec, const float* app, int n, int n_feat, const int32_t* inst,
                             const int32_t* inst_gid,
                             const int32_t* ranges, const gs_view* views_dev, int n_views, int total_tiles,
                             int64_t total_pixels, const RasterConst& c, int lds_batch, int persistent,
                             float* out, float* T_final, int32_t* last, int32_t* queue, hipStream_t s);

size_t slam_loss_workspace_bytes(int64_t P, const gs_view* views_host, int n_views, int n_feat,
                                 const gs_decoder* dec, const gs_slam_loss_opts& o);
hipError_t launch_slam_loss(const float* out, int n_feat, const float* rgb_t, const float* depth_t,
                            const int32_t* labels, const gs_decoder* dec, const gs_slam_loss_opts& o,
                            const gs_view* views_host, const gs_view* views_dev, int n_views, int64_t P,
                            float* grad_out, double* loss, float* median, uint8_t* masks, void* ws, hipStream_t s);
size_t loss_workspace_bytes(int64_t P);
hipError_t launch_loss(const float* out, int n_feat, const float* rgb_t, const float* depth_t,
                       const int32_t* labels, const float* decoder, int n_classes, const float* weights,
                       const gs_view* views_dev, int n_views, int64_t total_pixels, float* grad_out,
                       double* loss, void* ws, hipStream_t s);

int bwd_record_floats(int n_feat, bool params);
hipError_t launch_render_bwd(const float* rec, const float* app, int n, int n_feat, const int32_t* inst,
                             const int32_t* inst_gid, const int32_t* ranges, const gs_view* views_dev, int n_views,
                             int total_tiles, int64_t total_pixels, const RasterConst& c, int lds_batch,
                             int persistent, const float* T_final, const int32_t* last, const float* grad_out,
                             bool params, float* records, int32_t* queue, hipStream_t s);
hipError_t launch_reduce_records(const float* records, const int32_t* pair_first, const int32_t* touched, int n,
                                 int n_feat, int n_views, int64_t capacity, bool params, float* grad_geo,
                                 float* grad_app, hipStream_t s);

// accumulate: add to the planes of out; otherwise write every plane of every
// Gaussian (zeros where no view contributes).
hipError_t launch_project_bwd(const GaussPtrs& g, const gs_view* views_dev, int n_views, const RasterConst& c,
                              const int32_t* touched, const float* grad_geo, const float* grad_app,
                              const GradPtrs& out, bool accumulate, hipStream_t s);

size_t pose_workspace_bytes(int n, int n_views);
hipError_t launch_pose_grad(const GaussPtrs& g, const gs_view* views_dev, int n_views, const RasterConst& c,
                            const int32_t* touched, const float* grad_geo, void* ws, float* twist, hipStream_t s);

// Feature counts compiled into the render kernels.
inline bool feat_supported(int f) { return f == 0 || f == 8 || f == 16 || f == 32; }
inline int app_stride(int f) { return ((3 + f) + 3) / 4 * 4; }

}  // namespace sgs
