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

struct ClusterSet {
    uint32_t count = 0;
    // per cluster: x[64], y[64], z[64]; unused lanes repeat the cluster's first vertex
    std::vector<float> verts;
    // per cluster: 128 words, local indices i0 | i1 << 8 | i2 << 16; unused slots are 0 (a
    // degenerate triangle); bits 24..31 of word 0 hold the number of used slots
    std::vector<uint32_t> tris;
    // per cluster: 128 words, row of the triangle in the caller's index array (0xFFFFFFFF unused)
    std::vector<uint32_t> tri_id;
    // per cluster: axis-aligned bounds, min xyz then max xyz
    std::vector<float> bounds;
};

// vertices [V][3], indices [T][3]; every index must already be < V.
ClusterSet build_clusters(const float* vertices, uint32_t V, const uint32_t* indices, uint32_t T);

// The clusters of a scene that is being loaded.  The mesh is cut into chunks, which are turned into clusters side by
// side on up to kMostThreads threads, by the rule of build_clusters with two differences: a cluster's seed is the
// triangle that comes first along the diagonal of its chunk, and where nothing connected is left the triangle nearest to
// the seed stands in.  Both make the clusters' boxes smaller; chunks cost a few clusters along their borders.
//   500 k triangles   build_clusters   5370 clusters, faces of their boxes 1.85 times the mesh's area   29.5 ms
//                     chunks of 65536  5350, 1.57                                                        9.8 ms
//                     chunks of 16384  5410, 1.66                                                        6.2 ms
//   100 k             build_clusters   1136, 2.21                                                        5.5 ms
//                     chunks of 8192   1149, 1.82
// Frames: 1024 of 64x64 242 -> 234 us, 256 of 64x64 (200 k triangles) 97 -> 93, 1024 RGB-D (1 M triangles) 404 -> 391.
constexpr uint32_t kMostThreads = 12;
// Triangles per chunk: when the caller waits for the scene anyway, and when it is only to be on its way soon (a share
// of the mesh for every thread, but chunks no smaller than the clusters of build_clusters are matched by).  Small meshes
// come in two or three chunks either way: in one, which one thread works through, they took longer than with
// build_clusters, and more chunks than that cost clusters.
//   40 k triangles   build_clusters 5.3 ms, one chunk 8.3, three 4.3 (faces of the boxes 4920, 3967, 3993)
//   10 k             2.2, 3.0, two 1.8 (4879, 3702, 3677)
//   4 k              0.8, 1.0, two 0.7 (804, 631, 680); below 2048 a second thread would start too late
inline uint32_t chunk_triangles(uint32_t T, bool caller_waits) {
    if (T < 2048u) return 2048u;
    const uint32_t few = T / (T < 16384u ? 2u : 3u) + 1u;
    if (caller_waits) return T < 65536u ? few : 65536u;
    if (T < 4u * 8192u) return std::min(few, std::max(5000u, T / 4u + 1u));
    return std::min(std::max(8192u, T / kMostThreads + 1u), 16384u);
}

class SceneClusters {
public:
    // Every coordinate finite, every index that of a vertex.
    SceneClusters(const float* vertices, const uint32_t* indices, uint32_t T, uint32_t chunk_tris);
    ~SceneClusters();
    uint32_t count() const { return (uint32_t)order_.size(); }
    // Copies the clusters out, in the order the renderer wants; arrays as in ClusterSet, bounds in six planes of
    // `stride` values.
    void write(float* verts, uint32_t* tris, uint32_t* tri_id, float* bounds, size_t stride);

private:
    SceneClusters(const SceneClusters&) = delete;
    struct Impl;
    Impl* impl_;
    std::vector<uint64_t> order_;              // chunk << 32 | cluster of the chunk
};

}  // namespace bps
