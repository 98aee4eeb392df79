// Host-side re-packing of an indexed triangle mesh into fixed-size clusters.
//
// A cluster holds at most 64 distinct vertices and 128 triangles, so one 64-lane wavefront
// transforms each vertex of a cluster once (one lane per vertex) and then handles two
// triangles per lane.  This is part of scene upload (paper Sec. 3.2 "Scene asset sharing"),
// off the per-frame path.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <vector>

namespace bps {

constexpr uint32_t kClusterVerts = 64;
constexpr uint32_t kClusterTris = 128;

// The clusters of a scene.  The mesh is cut into chunks, which are turned into clusters side by side on up to kMostThreads
// threads: a cluster's seed is the triangle that comes first along the diagonal of its chunk, and where nothing connected
// is left the triangle nearest to the seed stands in.  Chunks cost a few clusters along their borders.  Against the whole
// mesh by one thread, seeds and stand-ins along a Morton curve ("whole"; clusters, faces of their boxes over the mesh's
// area, time):
//   500 k triangles   whole 5370, 1.85, 29.5 ms   chunks of 65536 5350, 1.57, 9.8 ms   of 16384 5410, 1.66, 6.2 ms
//   100 k             whole 1136, 2.21, 5.5 ms    chunks of 8192  1149, 1.82
// Frames: 1024 of 64x64 242 -> 234 us, 256 of 64x64 (200 k triangles) 97 -> 93, 1024 RGB-D (1 M triangles) 404 -> 391.
// What chunks cost more than that are meshes whose neighbours lie anywhere (a fan of 200 k triangles with its rim's
// vertices at random: whole 3340 clusters in 920 ms, chunks 5054 in 149 ms or 5828 in 69).
constexpr uint32_t kMostThreads = 12;
// Triangles per chunk: when the caller waits for the scene anyway, and when it is only to be on its way soon (a share
// of the mesh for every thread, but no chunks that would cost more clusters than "whole").  Small meshes come in two
// halves either way: in one, which one thread works through, they took longer than "whole", and in three their boxes are
// larger (a load that is waited for, its copy included, on a 16-core host; faces of the boxes; request of 78 environments):
//   40 k triangles       whole 2.6 ms, one chunk 4.0, halves 2.2, thirds 1.6 (6453, 5168, 5164, 5198)
//   10 k                 whole 0.78, one chunk 1.02, halves 0.69 (6787, 5832, 5265)
//   20 k, a single room  (845, 668, 688, thirds 690)   one chunk 47.2 us, halves 47.7, thirds 48.8
// Below 6144 a second thread saves less than its start costs (4 k: whole 0.24 ms, one chunk 0.29, halves 0.32).
inline uint32_t chunk_triangles(uint32_t T, bool caller_waits) {
    if (T < 6144u) return 6144u;
    const uint32_t half = T / 2u + 1u;
    if (caller_waits) return T < 65536u ? half : 65536u;
    if (T < 4u * 8192u) return std::min(half, std::max(5000u, T / 4u + 1u));
    return std::min(std::max(8192u, T / kMostThreads + 1u), 16384u);
}

class SceneClusters {
public:
    // vertices [V][3], indices [T][3]; every index has to be that of a vertex.
    SceneClusters(const float* vertices, const uint32_t* indices, uint32_t T, uint32_t chunk_tris);
    ~SceneClusters();
    uint32_t count() const { return (uint32_t)order_.size(); }
    // Copies the clusters out, in the order the renderer wants:
    //   verts   [count][3][64]  x, y, z planes; unused lanes repeat the cluster's first vertex
    //   tris    [count][128]    local indices i0 | i1 << 8 | i2 << 16, 0 in unused slots; how many are used in bits 24..31
    //                           of a cluster's first word
    //   tri_id  [count][128]    row of the triangle in the caller's index array, 0xFFFFFFFF in unused slots
    //   bounds  [6][stride]     axis-aligned, min xyz then max xyz
    // Null arrays are left out.
    void write(float* verts, uint32_t* tris, uint32_t* tri_id, float* bounds, size_t stride);

private:
    SceneClusters(const SceneClusters&) = delete;
    struct Impl;
    Impl* impl_;
    std::vector<uint64_t> order_;              // chunk << 32 | cluster of the chunk
};

}  // namespace bps
