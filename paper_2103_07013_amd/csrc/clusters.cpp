// Cluster builder: a mesh is cut into chunks, and each is turned into clusters, compact patches of at most 64 distinct
// vertices and 128 triangles that grow over the mesh's vertex adjacency.
#include "clusters.h"

#include <sched.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <condition_variable>
#include <cstring>
#include <exception>
#include <functional>
#include <memory>
#include <mutex>
#include <numeric>
#include <thread>
#include <type_traits>

namespace bps {
namespace {

// Clusters of one chunk.
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

inline uint32_t spread10(uint32_t v) {  // 10 bits -> every third bit
    v &= 0x3FFu;
    v = (v | (v << 16)) & 0x030000FFu;
    v = (v | (v << 8)) & 0x0300F00Fu;
    v = (v | (v << 4)) & 0x030C30C3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

// Candidate triangles kept per growing cluster.  Ordinary meshes stay far below it; the bound keeps
// the work per cluster fixed on meshes with vertices of enormous valence (triangles left out are
// simply picked up by a later cluster).
constexpr size_t kMaxCandidates = 512;

// The renderer tests 64 consecutive clusters as one block.  Median splits along the longest axis of
// the cluster centres, cut at multiples of 64, put clusters that are close in space into the same
// block (much tighter block boxes than runs of a space-filling curve give).
void split_blocks(std::vector<uint32_t>& order, size_t first, size_t last, const std::vector<float>& centre) {
    const size_t n = last - first;
    if (n <= 64) return;
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (size_t i = first; i < last; ++i)
        for (int a = 0; a < 3; ++a) {
            lo[a] = std::min(lo[a], centre[3 * (size_t)order[i] + a]);
            hi[a] = std::max(hi[a], centre[3 * (size_t)order[i] + a]);
        }
    int axis = 0;
    for (int a = 1; a < 3; ++a)
        if (hi[a] - lo[a] > hi[axis] - lo[axis]) axis = a;
    const size_t mid = first + ((n + 63) / 64 / 2) * 64;
    std::nth_element(order.begin() + first, order.begin() + mid, order.begin() + last, [&](uint32_t x, uint32_t y) {
        const float fx = centre[3 * (size_t)x + axis], fy = centre[3 * (size_t)y + axis];
        return fx < fy || (fx == fy && x < y);
    });
    split_blocks(order, first, mid, centre);
    split_blocks(order, mid, last, centre);
}

// Triangles in the order of their 30-bit codes, equal codes by triangle: three counting passes of 10 bits.
std::vector<uint32_t> sorted_by_code(const std::vector<uint32_t>& code) {
    const size_t n = code.size();
    std::vector<uint32_t> count(3 * 1024, 0), a(n), b(n);
    for (size_t i = 0; i < n; ++i)
        for (int pass = 0; pass < 3; ++pass) ++count[1024 * pass + ((code[i] >> (10 * pass)) & 1023u)];
    for (int pass = 0; pass < 3; ++pass) {
        uint32_t at = 0;
        for (uint32_t d = 0; d < 1024; ++d) {
            const uint32_t c = count[1024 * pass + d];
            count[1024 * pass + d] = at;
            at += c;
        }
    }
    for (size_t i = 0; i < n; ++i) a[count[code[i] & 1023u]++] = (uint32_t)i;
    for (size_t i = 0; i < n; ++i) b[count[1024 + ((code[a[i]] >> 10) & 1023u)]++] = a[i];
    for (size_t i = 0; i < n; ++i) a[count[2048 + (code[b[i]] >> 20)]++] = b[i];
    return a;
}

// The candidates of a growing cluster, in one list per number of vertices they would bring in (0 to 3), kept up to date
// as vertices join.  A list holds keys: distance from the seed above, order of listing below, so that the smallest key
// is the nearest candidate and the first listed of equals.  Choosing the cheapest reads the first list that is not
// empty, a dozen keys, instead of nine coordinates and three marks for each of some eighty candidates.
struct Candidates {
    static constexpr uint32_t kNone = 0xFFFFFFFFu;
    std::vector<uint64_t> keys[4];
    std::vector<uint32_t> tri, at;      // by order of listing: the triangle, its place in its list
    std::vector<uint8_t> fresh;         //                      and which list that is
    size_t live = 0;

    void clear() {
        for (auto& k : keys) k.clear();
        tri.clear();
        at.clear();
        fresh.clear();
        live = 0;
    }
    void insert(uint32_t seq, uint32_t f, uint64_t key) {
        fresh[seq] = (uint8_t)f;
        at[seq] = (uint32_t)keys[f].size();
        keys[f].push_back(key);
    }
    uint64_t remove(uint32_t seq) {
        std::vector<uint64_t>& k = keys[fresh[seq]];
        const uint64_t key = k[at[seq]];
        k[at[seq]] = k.back();
        at[(uint32_t)k.back()] = at[seq];
        k.pop_back();
        return key;
    }
    uint32_t list(uint32_t t, uint32_t f, float distance) {
        uint32_t bits;
        std::memcpy(&bits, &distance, 4);      // never negative or NaN: its bits order like its value
        const uint32_t seq = (uint32_t)tri.size();
        tri.push_back(t);
        at.push_back(0u);
        fresh.push_back(0);
        insert(seq, f, ((uint64_t)bits << 32) | seq);
        ++live;
        return seq;
    }
    void move(uint32_t seq, uint32_t f) {
        if (fresh[seq] != f) insert(seq, f, remove(seq));
    }
    void drop(uint32_t seq) {
        remove(seq);
        --live;
    }
    uint32_t cheapest() const {
        for (const auto& k : keys)
            if (!k.empty()) return (uint32_t)*std::min_element(k.begin(), k.end());
        return kNone;
    }
};

// The threads of one load.  run() hands out tasks 0 .. n - 1 to them and to the caller and returns when all are done.
class Team {
public:
    explicit Team(unsigned threads) {
        try {
            for (unsigned k = 1; k < threads; ++k) workers_.emplace_back([this] { work(); });
        } catch (const std::exception&) {      // no more threads to be had: the ones there are will do
        }
    }
    ~Team() {
        {
            std::lock_guard<std::mutex> g(mu_);
            quit_ = true;
        }
        wake_.notify_all();
        for (std::thread& t : workers_) t.join();
    }
    // (the task is only referred to: run() itself allocates nothing and throws what a task throws)
    template <class Task>
    void run(size_t n, Task&& task) {
        const Call call{[](void* t, size_t k) { (*static_cast<std::remove_reference_t<Task>*>(t))(k); }, &task};
        {
            std::lock_guard<std::mutex> g(mu_);
            task_ = &call;
            n_ = n;
            next_ = 0;
            failed_ = nullptr;
            ++round_;
        }
        if (n > 1) wake_.notify_all();
        take();
        std::unique_lock<std::mutex> g(mu_);
        idle_.wait(g, [this] { return busy_ == 0; });
        task_ = nullptr;                       // (a thread that wakes up late finds nothing)
        if (failed_) std::rethrow_exception(failed_);
    }

private:
    struct Call {
        void (*of)(void*, size_t);
        void* task;
    };
    void take() {
        for (;;) {
            const size_t k = next_.fetch_add(1);
            if (k >= n_) return;
            try {
                task_->of(task_->task, k);
            } catch (...) {
                std::lock_guard<std::mutex> g(mu_);
                if (!failed_) failed_ = std::current_exception();
            }
        }
    }
    void work() {
        uint64_t seen = 0;
        std::unique_lock<std::mutex> g(mu_);
        for (;;) {
            wake_.wait(g, [&] { return quit_ || (task_ && round_ != seen); });
            if (quit_) return;
            seen = round_;
            ++busy_;
            g.unlock();
            take();
            g.lock();
            if (--busy_ == 0) idle_.notify_one();
        }
    }
    std::vector<std::thread> workers_;
    std::mutex mu_;
    std::condition_variable wake_, idle_;
    const Call* task_ = nullptr;
    size_t n_ = 0;
    std::atomic<size_t> next_{0};
    unsigned busy_ = 0;
    uint64_t round_ = 0;
    bool quit_ = false;
    std::exception_ptr failed_;
};

unsigned usable_cpus() {
    cpu_set_t set;
    CPU_ZERO(&set);
    if (sched_getaffinity(0, sizeof(set), &set) != 0) return 1;
    return (unsigned)std::max(1, CPU_COUNT(&set));
}

// A triangle on its way into a chunk: centroid relative to a place among the triangles, times 3/64 (so that neither sums nor
// differences of finite numbers overflow).  The place is a median, so that a few triangles far away, which a box would have to
// hold, cost the others none of their precision.
struct Item {
    float c[3];
    uint32_t tri;
};
struct Range {
    size_t first, last;
};

// Slabs with about the same number of triangles each: count[s] of n triangles lie on step s along an axis; slab[s] is the
// slab that the step's middle triangle falls into.
constexpr uint32_t kSteps = 2048;
void cut(const uint32_t* count, size_t n, uint32_t parts, uint32_t* slab) {
    size_t before = 0;
    for (uint32_t s = 0; s < kSteps; ++s) {
        slab[s] = (uint32_t)std::min<size_t>(parts - 1, (before + count[s] / 2) * parts / n);
        before += count[s];
    }
}
// (bps_pack_clusters takes coordinates that are not finite; places that are compared must be numbers)
inline float finite_or_zero(float f) { return std::isfinite(f) ? f : 0.0f; }
struct Box {
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    void add(const float (&c)[3]) {
        for (int a = 0; a < 3; ++a) {
            lo[a] = std::min(lo[a], c[a]);
            hi[a] = std::max(hi[a], c[a]);
        }
    }
    int longest() const {
        int axis = 0;
        for (int a = 1; a < 3; ++a)
            if (hi[a] - lo[a] > hi[axis] - lo[axis]) axis = a;
        return axis;
    }
};
// Steps of equal length along the longest side of a box.
struct Steps {
    explicit Steps(const Box& box) : axis(box.longest()), base(box.lo[axis]), scale(((float)kSteps - 0.5f) / std::max(box.hi[axis] - base, 1e-30f)) {}
    uint32_t of(const Item& it) const { return std::min((uint32_t)((it.c[axis] - base) * scale), kSteps - 1); }
    int axis;
    float base, scale;
};
// Cuts in[r] into `parts` slabs along the longest side of its centroids' box and puts them into out[r] one after the other.
std::vector<Range> slabs(const Item* in, Item* out, Range r, uint32_t parts) {
    Box box;
    for (size_t i = r.first; i < r.last; ++i) box.add(in[i].c);
    const Steps steps(box);
    std::vector<uint32_t> count(kSteps, 0), slab(kSteps);
    for (size_t i = r.first; i < r.last; ++i) ++count[steps.of(in[i])];
    cut(count.data(), r.last - r.first, parts, slab.data());
    std::vector<size_t> at(parts, 0);
    for (uint32_t k = 0; k < kSteps; ++k) at[slab[k]] += count[k];
    std::vector<Range> made;
    size_t first = r.first;
    for (uint32_t p = 0; p < parts; ++p) {
        const size_t size = at[p];
        at[p] = first;
        if (size) made.push_back({first, first + size});
        first += size;
    }
    for (size_t i = r.first; i < r.last; ++i) out[at[slab[steps.of(in[i])]]++] = in[i];
    return made;
}
// Halves a range at the median along its longest side until no part has more than `most` triangles.  For what steps of equal
// length do not separate: most triangles on one of them, because a few lie far away or because all have one place.
void halve(Item* items, Range r, size_t most, bool whole, std::vector<Range>& made) {
    if (r.last - r.first <= most) {
        // (a median may leave its two sides in any order; chunks are grown from triangles in the order of their numbers)
        if (!whole) std::sort(items + r.first, items + r.last, [](const Item& x, const Item& y) { return x.tri < y.tri; });
        made.push_back(r);
        return;
    }
    Box box;
    for (size_t i = r.first; i < r.last; ++i) box.add(items[i].c);
    const int axis = box.longest();
    const size_t mid = r.first + (r.last - r.first) / 2;
    std::nth_element(items + r.first, items + mid, items + r.last, [axis](const Item& x, const Item& y) {
        return x.c[axis] < y.c[axis] || (x.c[axis] == y.c[axis] && x.tri < y.tri);
    });
    halve(items, {r.first, mid}, most, false, made);
    halve(items, {mid, r.last}, most, false, made);
}

// A chunk's vertices by number of first use.
class VertexNumbers {
public:
    VertexNumbers() : slot_(4096, {0xFFFFFFFFu, 0u}) {}
    uint32_t of(uint32_t vertex) {
        size_t k = place(vertex);
        if (slot_[k].first == vertex) return slot_[k].second;
        if (2 * numbered.size() >= slot_.size()) {
            slot_.assign(4 * slot_.size(), {0xFFFFFFFFu, 0u});
            for (uint32_t n = 0; n < (uint32_t)numbered.size(); ++n) slot_[place(numbered[n])] = {numbered[n], n};
            k = place(vertex);
        }
        slot_[k] = {vertex, (uint32_t)numbered.size()};
        numbered.push_back(vertex);
        return slot_[k].second;
    }
    std::vector<uint32_t> numbered;

private:
    size_t place(uint32_t vertex) const {      // where it is, or would be (no vertex is 0xFFFFFFFF: it would not be < V)
        size_t k = (size_t)(((uint64_t)vertex * 0x9E3779B97F4A7C15ull) >> 32) & (slot_.size() - 1);
        while (slot_[k].first != vertex && slot_[k].first != 0xFFFFFFFFu) k = (k + 1) & (slot_.size() - 1);
        return k;
    }
    std::vector<std::pair<uint32_t, uint32_t>> slot_;
};

// The triangles left of a chunk, for the nearest of them: in groups of 64 neighbours along a Morton curve, and 32 such groups
// to a district.
class Neighbourhood {
public:
    Neighbourhood(const Item* item, uint32_t n, const float (&lo)[3], float scale) : left_(n), place_(n) {
        std::vector<uint32_t> code(n);
        for (uint32_t t = 0; t < n; ++t) {
            code[t] = 0;
            for (int a = 0; a < 3; ++a)
                code[t] |= spread10((uint32_t)std::min(1023.0f, std::max(0.0f, (item[t].c[a] - lo[a]) * scale))) << a;
        }
        const std::vector<uint32_t> in_order = sorted_by_code(code);
        groups_.resize((n + kGroup - 1) / kGroup);
        districts_.resize((groups_.size() + kDistrict - 1) / kDistrict);
        for (uint32_t g = 0; g < (uint32_t)groups_.size(); ++g) {
            Part part;
            part.left = std::min(kGroup, n - g * kGroup);
            for (uint32_t k = g * kGroup; k < g * kGroup + part.left; ++k) {
                left_[k] = item[in_order[k]];
                left_[k].tri = in_order[k];
                place_[in_order[k]] = k;
                part.box.add(left_[k].c);
            }
            Part& district = districts_[g / kDistrict];
            district.box.add(part.box.lo);
            district.box.add(part.box.hi);
            district.left += part.left;
            groups_[g] = part;
        }
    }
    void take(uint32_t t) {      // (the last of its group moves to its place)
        const uint32_t k = place_[t], g = k / kGroup, last = g * kGroup + --groups_[g].left;
        --districts_[g / kDistrict].left;
        left_[k] = left_[last];
        place_[left_[k].tri] = k;
    }
    // From now on next() looks around c.
    void look_from(const float (&c)[3]) {
        std::copy(c, c + 3, from_);
        asked_ = 0;
    }
    // The triangle nearest to that place in the maximum norm that is not taken; 0xFFFFFFFF if there is none.  Groups are
    // opened one after the other, the nearest first, until none that is left can hold a nearer triangle.  Loose triangles
    // would have most groups opened for every cluster: a cluster that asks again and again takes them from the groups
    // that are open, and so does one that has opened six.  (Without districts each cluster looked at every group of the
    // chunk seven times: 50 k loose triangles in one chunk 63.7 ms, now 36.)
    uint32_t next(const std::vector<uint8_t>& taken) {
        if (asked_++ == 0) {
            opened_ = 0;
            seen_.clear();
            around_.clear();
            for (uint32_t d = 0; d < (uint32_t)districts_.size(); ++d) list(districts_[d], kIsDistrict | d);
        } else if (asked_ == 2) {      // seldom more than that: looked through once more
            seen_.erase(std::remove_if(seen_.begin(), seen_.end(), [&](const Place& p) { return taken[p.second] != 0; }), seen_.end());
            if (!seen_.empty()) std::iter_swap(seen_.begin(), std::min_element(seen_.begin(), seen_.end()));
        } else {
            if (asked_ == 3) std::make_heap(seen_.begin(), seen_.end(), std::greater<Place>());
            while (!seen_.empty() && taken[seen_.front().second]) {
                std::pop_heap(seen_.begin(), seen_.end(), std::greater<Place>());
                seen_.pop_back();
            }
        }
        for (;;) {
            const bool found = !seen_.empty();
            if (found && (asked_ > 2 || opened_ >= 6)) break;
            if (around_.empty()) break;
            const auto nearest = std::min_element(around_.begin(), around_.end());
            if (found && seen_.front().first < nearest->first) break;
            const uint32_t what = nearest->second;
            *nearest = around_.back();
            around_.pop_back();
            if (what & kIsDistrict) {
                const uint32_t from = (what & ~kIsDistrict) * kDistrict;
                for (uint32_t g = from; g < std::min<size_t>(groups_.size(), (size_t)from + kDistrict); ++g) list(groups_[g], g);
                continue;
            }
            ++opened_;
            for (uint32_t k = what * kGroup; k < what * kGroup + groups_[what].left; ++k) {
                float d = 0.0f;
                for (int a = 0; a < 3; ++a) d = std::max(d, std::fabs(left_[k].c[a] - from_[a]));
                seen_.push_back({d, left_[k].tri});
                if (asked_ > 2)
                    std::push_heap(seen_.begin(), seen_.end(), std::greater<Place>());
                else if (seen_.back() < seen_.front())
                    std::swap(seen_.back(), seen_.front());
            }
        }
        return seen_.empty() ? 0xFFFFFFFFu : seen_.front().second;
    }

private:
    static constexpr uint32_t kGroup = 64, kDistrict = 32, kIsDistrict = 0x80000000u;
    typedef std::pair<float, uint32_t> Place;      // distance and what is there: a triangle, a group, a district | kIsDistrict
    struct Part {
        Box box;
        uint32_t left = 0;      // triangles not taken: a group's first ones
    };
    void list(const Part& p, uint32_t what) {
        if (!p.left) return;
        float d = 0.0f;
        for (int a = 0; a < 3; ++a) d = std::max(d, std::max(p.box.lo[a] - from_[a], from_[a] - p.box.hi[a]));
        around_.push_back({d, what});
    }
    std::vector<Item> left_;         // group by group
    std::vector<uint32_t> place_;    // by triangle: where in left_
    std::vector<Part> groups_, districts_;
    float from_[3];
    uint32_t asked_ = 0, opened_ = 0;
    std::vector<Place> seen_;        // triangles of the groups that are open, the nearest in front (a heap from the third question on)
    std::vector<Place> around_;      // districts and groups that are not
};

// Region growing.  A cluster starts at the first triangle along the chunk's diagonal that is not assigned and grows by the
// triangle that costs least: fewest vertices not yet in the cluster first, then the one whose centroid is nearest the
// seed's in the maximum norm, which makes square axis-aligned patches (compact clusters have small boxes and small
// screen footprints, which is what the renderer's culling tests look at).  Candidates are the unassigned triangles that
// touch a vertex of the cluster; where the mesh offers none (unconnected triangles) the one nearest to the seed stands in.
ClusterSet grow_chunk(const float* vertices, const uint32_t* indices, const Item* item, uint32_t n) {
    ClusterSet out;
    // ---- a mesh of its own: vertices numbered by first use, the triangles at each of them
    std::vector<uint32_t> ix(3 * (size_t)n), vertex;
    {
        VertexNumbers numbers;
        for (uint32_t t = 0; t < n; ++t)
            for (int k = 0; k < 3; ++k) ix[3 * (size_t)t + k] = numbers.of(indices[3 * (size_t)item[t].tri + k]);
        vertex = std::move(numbers.numbered);
    }
    const uint32_t V = (uint32_t)vertex.size();
    std::vector<uint32_t> vstart(V + 1, 0), vtris(3 * (size_t)n);
    for (uint32_t i : ix) ++vstart[i + 1];
    for (uint32_t v = 0; v < V; ++v) vstart[v + 1] += vstart[v];
    {
        std::vector<uint32_t> fill(vstart.begin(), vstart.end() - 1);
        for (uint32_t t = 0; t < n; ++t)
            for (int k = 0; k < 3; ++k) vtris[fill[ix[3 * (size_t)t + k]]++] = t;
    }
    // ---- along the diagonal of the chunk's box
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (uint32_t t = 0; t < n; ++t)
        for (int a = 0; a < 3; ++a) {
            lo[a] = std::min(lo[a], item[t].c[a]);
            hi[a] = std::max(hi[a], item[t].c[a]);
        }
    const float side = std::max({hi[0] - lo[0], hi[1] - lo[1], hi[2] - lo[2], 1e-30f});
    std::vector<uint32_t> in_order;
    {
        std::vector<uint32_t> code(n);
        const float scale = 1073741823.0f / (3.0f * side);
        for (uint32_t t = 0; t < n; ++t) {
            const float along = (item[t].c[0] - lo[0]) + (item[t].c[1] - lo[1]) + (item[t].c[2] - lo[2]);
            code[t] = (uint32_t)std::min(1073741760.0f, along * scale);      // (the largest float below 2^30)
        }
        in_order = sorted_by_code(code);
    }
    Neighbourhood near(item, n, lo, 1023.0f / side);

    std::vector<uint32_t> vfirst(vstart.begin(), vstart.end() - 1);   // first entry of a vertex's list that may be free
    std::vector<uint32_t> stamp(V, 0xFFFFFFFFu);     // cluster that last used the vertex
    std::vector<uint8_t> local(V, 0), taken(n, 0);
    std::vector<uint32_t> listed(n, 0xFFFFFFFFu), place(n);           // cluster whose candidates hold the triangle, its number there
    Candidates cand;
    const size_t expect = n / 85 + 2;
    out.verts.reserve(expect * 192);
    out.tris.reserve(expect * 128);
    out.tri_id.reserve(expect * 128);
    uint32_t head = 0;
    for (;;) {
        while (head < n && taken[in_order[head]]) ++head;
        if (head >= n) break;
        const uint32_t c = out.count++, seed = in_order[head];
        const size_t vbase = out.verts.size(), tbase = out.tris.size();
        out.verts.resize(vbase + 192, 0.0f);
        out.tris.resize(tbase + 128, 0u);
        out.tri_id.resize(tbase + 128, 0xFFFFFFFFu);
        uint32_t nv = 0, nt = 0;
        float bl[3] = {INFINITY, INFINITY, INFINITY}, bh[3] = {-INFINITY, -INFINITY, -INFINITY};
        const float at[3] = {item[seed].c[0], item[seed].c[1], item[seed].c[2]};
        cand.clear();
        near.look_from(at);
        auto fresh_of = [&](uint32_t t) {
            const uint32_t* i = &ix[3 * (size_t)t];
            uint32_t d = stamp[i[0]] != c ? 1u : 0u;
            if (i[1] != i[0] && stamp[i[1]] != c) ++d;
            if (i[2] != i[0] && i[2] != i[1] && stamp[i[2]] != c) ++d;
            return d;
        };
        auto distance = [&](uint32_t t) {
            float d = 0.0f;
            for (int a = 0; a < 3; ++a) d = std::max(d, std::fabs(item[t].c[a] - at[a]));
            return d;
        };
        auto add = [&](uint32_t t) {
            taken[t] = 1;
            near.take(t);
            uint32_t li[3];
            for (int k = 0; k < 3; ++k) {
                const uint32_t v = ix[3 * (size_t)t + k];
                if (stamp[v] != c) {
                    stamp[v] = c;
                    local[v] = (uint8_t)nv;
                    for (int a = 0; a < 3; ++a) {
                        const float f = vertices[3 * (size_t)vertex[v] + a];
                        out.verts[vbase + 64 * a + nv] = f;
                        bl[a] = std::min(bl[a], f);
                        bh[a] = std::max(bh[a], f);
                    }
                    ++nv;
                    // triangles once taken stay taken: skip the taken head of the vertex's list for good
                    uint32_t& from = vfirst[v];
                    const uint32_t end = vstart[v + 1];
                    while (from < end && taken[vtris[from]]) ++from;
                    // Candidates at this vertex now need one vertex fewer; the other triangles here become candidates
                    // as long as there is room.  A list much longer than that is not walked to its end: every
                    // candidate's cost is worked out anew instead.
                    const bool walk = end - from <= 4 * kMaxCandidates;
                    for (uint32_t q = from; q < end && (walk || cand.live < kMaxCandidates); ++q) {
                        const uint32_t o = vtris[q];
                        if (taken[o] || (q > from && vtris[q - 1] == o)) continue;      // (a vertex may occur twice in a triangle)
                        if (listed[o] == c) {
                            if (walk) cand.move(place[o], cand.fresh[place[o]] - 1u);
                        } else if (cand.live < kMaxCandidates) {
                            listed[o] = c;
                            place[o] = cand.list(o, fresh_of(o), distance(o));
                        }
                    }
                    if (!walk)
                        for (uint32_t q = 0; q < (uint32_t)cand.tri.size(); ++q)
                            if (!taken[cand.tri[q]]) cand.move(q, fresh_of(cand.tri[q]));
                }
                li[k] = local[v];
            }
            out.tris[tbase + nt] = li[0] | (li[1] << 8) | (li[2] << 16);
            out.tri_id[tbase + nt] = item[t].tri;
            ++nt;
        };
        add(seed);
        while (nt < kClusterTris) {
            const uint32_t cheapest = cand.cheapest();
            const bool connected = cheapest != Candidates::kNone;
            const uint32_t best = connected ? cand.tri[cheapest] : near.next(taken);
            if (best == 0xFFFFFFFFu || nv + (connected ? cand.fresh[cheapest] : fresh_of(best)) > kClusterVerts) break;
            add(best);
            if (connected) cand.drop(cheapest);
        }
        for (uint32_t l = nv; l < kClusterVerts; ++l)
            for (int a = 0; a < 3; ++a) out.verts[vbase + 64 * a + l] = out.verts[vbase + 64 * a];
        out.tris[tbase] |= nt << 24;
        out.bounds.insert(out.bounds.end(), bl, bl + 3);
        out.bounds.insert(out.bounds.end(), bh, bh + 3);
    }
    return out;
}

}  // namespace

struct SceneClusters::Impl {
    std::vector<ClusterSet> chunks;
    Team team;
    explicit Impl(unsigned threads) : team(threads) {}
};

SceneClusters::SceneClusters(const float* vertices, const uint32_t* indices, uint32_t T, uint32_t chunk_tris) : impl_(nullptr) {
    const uint32_t n_chunks = T / chunk_tris + (T % chunk_tris ? 1 : 0);
    // (a chunk of less than 1024 triangles is done before a second thread has started)
    std::unique_ptr<Impl> impl(new Impl(T < 2048 ? 1u : std::min({kMostThreads, usable_cpus(), std::max(n_chunks, T / 65536u)})));
    Team& team = impl->team;
    float origin[3];
    for (int x = 0; x < 3; ++x) {
        constexpr size_t kSamples = 63;
        float sample[kSamples];
        for (size_t k = 0; k < kSamples; ++k) sample[k] = finite_or_zero(vertices[3 * (size_t)indices[3 * (k * T / kSamples)] + x]);
        std::nth_element(sample, sample + kSamples / 2, sample + kSamples);
        origin[x] = sample[kSamples / 2] * (1.0f / 64.0f);
    }
    std::unique_ptr<Item[]> a(new Item[T]), b(n_chunks > 1 ? new Item[T] : nullptr);
    constexpr size_t kBatch = 8192;
    const size_t batches = ((size_t)T + kBatch - 1) / kBatch;
    std::vector<Box> boxes(batches);
    team.run(batches, [&](size_t k) {
        Box box;      // (in registers: neighbouring batches' boxes share cache lines)
        for (size_t t = k * kBatch; t < std::min<size_t>(T, (k + 1) * kBatch); ++t) {
            Item it;
            it.tri = (uint32_t)t;
            for (int x = 0; x < 3; ++x) {
                float c = 0.0f;
                for (int j = 0; j < 3; ++j) c += vertices[3 * (size_t)indices[3 * t + j] + x] * (1.0f / 64.0f) - origin[x];
                it.c[x] = finite_or_zero(c);
            }
            box.add(it.c);
            a[t] = it;
        }
        boxes[k] = box;
    });
    // ---- slabs along the longest side, each cut into slabs again: near-cubes of about the same number of triangles
    std::vector<Range> ranges{{0, T}};
    Item* items = a.get();
    if (n_chunks > 1) {
        for (size_t k = 1; k < batches; ++k) {
            boxes[0].add(boxes[k].lo);
            boxes[0].add(boxes[k].hi);
        }
        const Steps steps(boxes[0]);
        std::vector<uint32_t> counts(batches * kSteps, 0);      // by batch: triangles on each step
        team.run(batches, [&](size_t k) {
            for (size_t t = k * kBatch; t < std::min<size_t>(T, (k + 1) * kBatch); ++t) ++counts[k * kSteps + steps.of(a[t])];
        });
        const uint32_t first_cut = n_chunks <= 3 ? n_chunks : (uint32_t)std::ceil(std::sqrt((double)n_chunks));
        std::vector<uint32_t> all(kSteps, 0), slab(kSteps);
        for (size_t k = 0; k < batches; ++k)
            for (uint32_t s = 0; s < kSteps; ++s) all[s] += counts[k * kSteps + s];
        cut(all.data(), T, first_cut, slab.data());
        std::vector<size_t> at(batches * first_cut, 0);      // where a batch's triangles of a slab go
        for (size_t k = 0; k < batches; ++k)
            for (uint32_t s = 0; s < kSteps; ++s) at[k * first_cut + slab[s]] += counts[k * kSteps + s];
        ranges.clear();
        size_t first = 0;
        for (uint32_t p = 0; p < first_cut; ++p) {
            const size_t from = first;
            for (size_t k = 0; k < batches; ++k) {
                const size_t n = at[k * first_cut + p];
                at[k * first_cut + p] = first;
                first += n;
            }
            if (first > from) ranges.push_back({from, first});
        }
        team.run(batches, [&](size_t k) {
            for (size_t t = k * kBatch; t < std::min<size_t>(T, (k + 1) * kBatch); ++t) b[at[k * first_cut + slab[steps.of(a[t])]]++] = a[t];
        });
        items = n_chunks > 3 ? a.get() : b.get();
        std::vector<std::vector<Range>> parts(ranges.size());
        team.run(ranges.size(), [&](size_t k) {
            std::vector<Range> made{ranges[k]};
            const size_t n = ranges[k].last - ranges[k].first;
            if (n_chunks > 3) made = slabs(b.get(), a.get(), ranges[k], (uint32_t)std::max<size_t>(1, (n + chunk_tris / 2) / chunk_tris));
            for (Range r : made) halve(items, r, 2 * (size_t)chunk_tris, true, parts[k]);
        });
        ranges.clear();
        for (const auto& p : parts) ranges.insert(ranges.end(), p.begin(), p.end());
    }
    impl->chunks.resize(ranges.size());
    team.run(ranges.size(), [&](size_t k) {
        impl->chunks[k] = grow_chunk(vertices, indices, items + ranges[k].first, (uint32_t)(ranges[k].last - ranges[k].first));
    });
    // ---- blocks of 64 clusters that are close in space
    std::vector<float> centre;
    std::vector<uint64_t> number;
    for (size_t k = 0; k < impl->chunks.size(); ++k)
        for (uint32_t c = 0; c < impl->chunks[k].count; ++c) {
            const float* box = &impl->chunks[k].bounds[6 * (size_t)c];
            for (int x = 0; x < 3; ++x) centre.push_back(finite_or_zero(0.5f * box[x] + 0.5f * box[3 + x]));
            number.push_back((uint64_t)k << 32 | c);
        }
    std::vector<uint32_t> order(number.size());
    std::iota(order.begin(), order.end(), 0u);
    split_blocks(order, 0, order.size(), centre);
    order_.resize(order.size());
    for (size_t k = 0; k < order.size(); ++k) order_[k] = number[order[k]];
    impl_ = impl.release();
}

SceneClusters::~SceneClusters() { delete impl_; }

void SceneClusters::write(float* verts, uint32_t* tris, uint32_t* tri_id, float* bounds, size_t stride) {
    constexpr size_t kBatch = 256;
    impl_->team.run((order_.size() + kBatch - 1) / kBatch, [&](size_t k) {
        for (size_t c = k * kBatch; c < std::min(order_.size(), (k + 1) * kBatch); ++c) {
            const ClusterSet& from = impl_->chunks[order_[c] >> 32];
            const size_t s = (uint32_t)order_[c];
            if (verts) std::memcpy(verts + c * 192, &from.verts[s * 192], 192 * sizeof(float));
            if (tris) std::memcpy(tris + c * 128, &from.tris[s * 128], 128 * sizeof(uint32_t));
            if (tri_id) std::memcpy(tri_id + c * 128, &from.tri_id[s * 128], 128 * sizeof(uint32_t));
            for (int x = 0; bounds && x < 6; ++x) bounds[(size_t)x * stride + c] = from.bounds[s * 6 + x];
        }
    });
}

}  // namespace bps
