// Device side of the batch renderer: one fused geometry + rasterisation kernel and a resolve
// kernel, written for gfx950 (64-lane wavefronts, 160 KB LDS per CU).
//
// One work-group renders (a slice of) one environment's frame (paper Sec. 3.2: every
// environment of the batch is drawn in a single request).  The frame's visibility buffer --
// H*W packed keys (depth bits << 32 | triangle id) -- lives in LDS for the whole kernel, so the
// z-test is a 64-bit LDS atomic min and the frame is written to HBM exactly once.  Each wavefront
// streams clusters of <= 64 vertices / <= 128 triangles:
//   vertex phase   one lane per vertex: clip = M v, six-plane outcodes, projection, 1/256-px snap
//   cluster cull   all 64 vertices outside one plane (wave ballot)  -> next cluster
//   triangle phase two triangles per lane: outcode reject, bounding box vs pixel centres
//   compaction     survivors are appended to LDS queues with ballot + prefix count so
//                  that the expensive steps run on full wavefronts:
//                    small queue  (per wavefront) triangles touching few pixel centres (small_max), one lane per triangle
//                    clip ring    (per work-group) triangles straddling a frustum plane, one lane per triangle
//                  large triangles are rasterised by the whole wavefront, 8x8 pixels at a time.
// All float arithmetic follows one fixed IEEE sequence (explicit fmaf, no contraction, exact
// division) so that coverage and ids are reproducible bit for bit.
#pragma once
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bps {

struct SceneDev {
    const float* cverts;       // [C][3][64] cluster vertex positions, x then y then z
    const uint32_t* ctris;     // [C][128]   packed local indices, count in bits 24..31 of word 0
    const uint32_t* ctri_id;   // [C][128]   original triangle row
    const float* cbounds;      // [6][c_stride] cluster bounds: min x, y, z then max x, y, z
    const float* bbounds;      // [6][b_stride] bounds of each block of 64 consecutive clusters
    const float* verts;        // [V][3]     original arrays, used when shading
    const uint32_t* indices;   // [T][3]
    const uint8_t* colors;     // [V][3] or null
    const float* uvs;          // [V][2] or null (textured scenes)
    const uint32_t* texels;    // RGBA8 mip pyramid, level after level, or null
    const float* tri_rec;      // [T][16]    per-triangle shading record (scenes with colours or a texture), or null:
                               //            x0 y0 z0 x1 y1 z1 x2 y2 z2, then three packed RGB words or u0 v0 u1 v1 u2 v2
    uint32_t tex_w, tex_h, tex_levels, pad2;
    uint32_t n_clusters, n_tris, n_verts, c_stride, b_stride, pad;
};

// One work-group's share: tile `tile` of environment `env`'s frame, and of its scene the
// 64-cluster blocks split, split + n_splits, split + 2 n_splits, ... (split_of = n_splits << 16 | split)
struct WorkItem {
    uint32_t env, scene, split_of, tile;
};

struct FrameParams {
    int32_t H, W;
    int32_t tile_w, tile_h; // a work-group owns one tile of the frame (the whole frame when it fits)
    int32_t tiles_x;        // tiles side by side
    uint32_t tiles_x_recip; // 65536 / tiles_x rounded up: tile / tiles_x = tile * recip >> 16 for the kMaxWindows tiles there can be
    float two_per_w, two_per_h;   // 2 / W, 2 / H
    float sx, sy;          // 128*W, 128*H
    float xmax, ymax;      // 2*sx + 64, 2*sy + 64
    float background;
    int32_t merge;         // 0: resolve straight to the output; 1: atomic-min into the global buffer
    int32_t cull;          // 0: stream every cluster; 1: frustum-cull clusters; 2: frustum + occlusion cull
    int32_t list_cap;      // capacity of the work-group's survivor list, in clusters
    int32_t round_target;  // survivors queued before a round's testing stops
    int32_t first_round;   // the same for an environment's first round (kept short when occlusion culling is on)
    int32_t phase_timers;  // diagnostics: 1 also time the kernel's phases (slows it down), 2 / 3 path tallies
    int32_t bilinear;      // colour pass: sample textures with bilinear filtering instead of the nearest texel
    int32_t small_max = 0; // (set by launch_raster, for the instances that count: see small_max below)
};

constexpr unsigned long long kEmptyKey = ~0ull;
constexpr int kOrigin = 16384;         // packed screen coordinates are stored relative to pixel 64
// Pixel centres a "small" triangle may touch (one lane rasterises it; larger ones share a wavefront, four or one at a time).
// A drain of the queue takes as many steps as its largest triangle has centres, so the line lies where such steps cost what a
// pass over larger triangles costs.  That depends on the mesh too; the number is one per instance, so that the loop over
// the steps is unrolled.  Frames of 64x64 drawn whole: 12 (us per request with 8 / 10 / 12 / 16: 1024 of 500 k triangles
// 202.9 / 200.0 / 198.5 / 201.2; with 12 / 16: of 100 k 162.8 / 161.2, of 20 k 179 / 172, of 500 179 / 169).  Every other
// window, also those of frames of 64x64 that are cut: 20 (with 12 / 20: 61 at 72x104 55.6 / 53.3, 4096 at 128x128 1923 / 1919,
// 512 at 128x128 of 100 k 284 / 274, 200 at 64x64 of 20 k 70.7 / 67.7, 512 at 128x128 of 500 263 / 273, 16 at 64x64 of 100 k
// 21.9 / 22.4; one environment in 64 windows with 20 / 24 17.1 / 18.6).
constexpr int small_max(int frame) { return frame == 1 || frame == 128 ? 20 : 12; }
constexpr uint32_t kInvalid = 0x40u;   // outcode bit: vertex unusable, drop its triangles
constexpr uint32_t kNoProject = 0x80u; // outcode bit: vertex has no finite screen position (w <= 0 or overflow)

// per-wave LDS block: 64 staged vertices (8 B + 4 B outcode each), small queue 8 x 64 words
constexpr uint32_t kListCap64 = 1216;   // survivor-list capacity of the fixed-layout instances (two groups per compute unit)
constexpr uint32_t kWaveLdsBytes = 64 * 12 + 8 * 64 * 4;

// The work-group's ring of triangles waiting for the clipper.  A wavefront adds at most 128 entries
// between two looks at the ring and then drains it below 64, and at most 64 entries per wavefront are
// claimed but not yet read: never more than 64 + 192 per wavefront in use, so 256 per wavefront
// (rounded up to a power of two) cannot wrap onto a live entry.
__host__ __device__ constexpr uint32_t clip_ring_entries(int threads) {
    uint32_t need = 256u * (uint32_t)(threads / 64), n = 256u;
    while (n < need) n *= 2u;
    return n;
}

constexpr int kOrderCap = 1024;        // blocks of one item that can be depth-sorted
constexpr int kHizTiles = 64;          // 8x8-pixel tiles of a window of at most 64x64 pixels
constexpr int kDepthBins = 128;        // bins of the per-round depth sort of surviving clusters

// visibility buffer, per-wave blocks, survivor list (8 B record + two 2 B sort words per cluster),
// block order, depth histogram, depth tiles, the window's planes, eight counters, clip ring
__host__ __device__ inline size_t lds_bytes(int tile_h, int tile_w, int threads, int list_cap) {
    return (size_t)((tile_h * tile_w + 1) & ~1) * 8 + (size_t)(threads / 64) * kWaveLdsBytes + (size_t)list_cap * 12 + kOrderCap * 2 +
           kDepthBins * 4 + kHizTiles * 4 + 8 * 48 + 32 + (size_t)clip_ring_entries(threads) * 4;
}

// DIAG = true is the instance launched while diagnostics are on; it alone keeps counters and timers.
// CULL = FrameParams::cull of the launch (0 none, 1 frustum, 2 frustum + occlusion).
// FRAME = 64 or 128: the frame is square of that size and drawn as 64x64 windows; 1 = any frame and window,
// with the LDS layout of those two (a 64x64 key buffer and kListCap64 survivors, whatever the window's size), also with
// 1024 threads for launches that put one group on a compute unit (choose_cut);
// 0 = any frame, window, layout.
template <int NT, bool DIAG, int CULL, int FRAME>
__global__ void k_raster(const SceneDev* __restrict__ scenes, const WorkItem* __restrict__ items,
                         const float* __restrict__ view_proj, FrameParams fp, unsigned long long* __restrict__ gvis,
                         float* __restrict__ out_depth, uint32_t* __restrict__ out_id,
                         unsigned long long* __restrict__ stats);

__global__ void k_resolve(unsigned long long* __restrict__ gvis, size_t n, float background,
                          float* __restrict__ out_depth, uint32_t* __restrict__ out_id);

__global__ void k_fill_keys(unsigned long long* __restrict__ gvis, size_t n);
__global__ void k_zero_words(unsigned long long* __restrict__ p, size_t n);

// Launches a kernel; `done`, if given, is an event that is reached when the kernel has finished.  The event is the end
// of the kernel's own packet: recorded behind it, it takes a packet of its own, which costs a request 3 us (one environment
// 22.1 -> 19.1 us, 16 in a small room 24.5 -> 21.7, 61 at 72x104 54.6 -> 51.7, 512 104.6 -> 101.6).
template <class T>
struct same { using type = T; };      // (no deduction from the arguments)
template <class... P>
hipError_t launch_kernel(hipEvent_t done, void (*kernel)(P...), dim3 grid, dim3 block, size_t lds, hipStream_t stream,
                         typename same<P>::type... args) {
    if (done) {
        void* list[] = {&args...};
        return hipExtLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, list, lds, stream, nullptr, done, 0);
    }
    hipLaunchKernelGGL(kernel, grid, block, lds, stream, args...);
    return hipGetLastError();
}

hipError_t launch_raster(hipEvent_t done, int threads, dim3 grid, size_t lds, hipStream_t stream, const SceneDev* scenes, const WorkItem* items,
                   const float* view_proj, const FrameParams& fp, bool fixed_layout, bool wide, unsigned long long* gvis,
                   float* out_depth, uint32_t* out_id, unsigned long long* stats);
// Fills ordered[n_items] with the items in launch order, costliest first; cost is scratch, one word
// per item.
constexpr uint32_t kMaxPlannedItems = 16384;
void launch_plan(hipStream_t stream, const SceneDev* scenes, const WorkItem* items, const float* view_proj,
                 const FrameParams& fp, uint32_t n_items, uint32_t* cost, WorkItem* ordered);
// wide_lds: what launches of the 1024-thread instances with a layout chosen at run time ask for; 0 = there are none.
hipError_t prepare_raster(int threads, size_t lds, bool fixed_layout, size_t wide_lds);
// Work items handed over as kernel arguments (no host-to-device copy, no staging memory): up to
// kPackedItemsPerLaunch items per launch, each packed as env (14 bits: at most kMaxPlannedItems items) |
// scene (12 bits) | tile (6 bits); one work-group per environment and tile, i.e. split_of = 1 << 16.
constexpr uint32_t kPackedEnvBits = 14, kPackedSceneBits = 12;
constexpr uint32_t kMaxWindows = 64;      // windows a frame is cut into at most
static_assert(kMaxWindows <= 1u << (32 - kPackedEnvBits - kPackedSceneBits), "a window's number fits its bits");
static_assert(kMaxPlannedItems <= 1u << kPackedEnvBits, "every environment of a request has an item");
static_assert(kMaxWindows * kMaxWindows <= 65536u, "exact division by a multiplication (FrameParams::tiles_x_recip)");
constexpr uint32_t kPackedItemsPerLaunch = 960;
struct PackedItems {
    uint32_t word[kPackedItemsPerLaunch];
};
void launch_unpack_items(hipStream_t stream, const PackedItems& packed, uint32_t first, uint32_t count, WorkItem* items);
hipError_t launch_downsample(hipEvent_t done, hipStream_t stream, const float* depth, const uint8_t* rgb, uint32_t B, int H, int W,
                       float* out_depth, uint8_t* out_rgb);
// Fills sc.tri_rec from the scene's original arrays (once per scene, on the stream that uploads it).
void launch_build_shade_records(hipStream_t stream, const SceneDev& sc, float* tri_rec);
hipError_t launch_shade(hipEvent_t done, hipStream_t stream, const SceneDev* scenes, const uint32_t* env_scene, const float* view_proj,
                  const FrameParams& fp, uint32_t B, const uint32_t* tri_id, uint8_t* out_rgb);

}  // namespace bps
