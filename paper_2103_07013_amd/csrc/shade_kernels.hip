// Colour resolve for RGB-D frames (stand-in for the paper's textured RGB sensor, Sec. 4.1):
// per-vertex uint8 colours, perspective-correct interpolation at the pixel centre of the
// triangle that won the z-test.  Runs after k_raster, one thread per pixel: the winner's
// three vertices are transformed, clipped and set up again with the raster kernel's results
// bit for bit, so the barycentric weights are the ones the z-test used.
//   cn = fma(e2/w2, c2, fma(e1/w1, c1, (e0/w0) c0)),  out = clamp(rint(cn / num), 0, 255)
#include "raster_device.h"
#include "raster_kernels.h"

namespace bps {
namespace {

using namespace dev;

typedef float float4v __attribute__((ext_vector_type(4)));

struct CVert {
    Clip4 c;
    float r, g, b;
};

struct SVert {
    uint32_t xy;
    float iw, r, g, b;
};

// Field-by-field choice (choosing between whole objects goes through their addresses and would
// put both into private memory).
__device__ __forceinline__ CVert pick(bool first, const CVert& x, const CVert& y) {
    CVert o;
    o.c.x = first ? x.c.x : y.c.x; o.c.y = first ? x.c.y : y.c.y; o.c.z = first ? x.c.z : y.c.z; o.c.w = first ? x.c.w : y.c.w;
    o.r = first ? x.r : y.r; o.g = first ? x.g : y.g; o.b = first ? x.b : y.b;
    return o;
}
__device__ __forceinline__ SVert pick(bool first, const SVert& x, const SVert& y) {
    SVert o;
    o.xy = first ? x.xy : y.xy;
    o.iw = first ? x.iw : y.iw;
    o.r = first ? x.r : y.r; o.g = first ? x.g : y.g; o.b = first ? x.b : y.b;
    return o;
}

// Colour of pixel (i, j) from one snapped fan triangle; returns false when it does not cover the pixel.
__device__ __forceinline__ bool piece_colour(const SVert& v0, const SVert& v1, const SVert& v2, int i, int j,
                                             float& depth, float (&rgb)[3], float& uv_area2, int& area2) {
    Setup s = make_setup(v0.xy, v1.xy, v2.xy, v0.iw, v1.iw, v2.iw);
    if (s.A2 == 0) return false;
    // (values are selected one by one: choosing between two objects by reference would force both
    // into private memory)
    struct Attr { float r, g, b; };
    const Attr a = {v0.r, v0.g, v0.b};
    const Attr b = {s.swapped ? v2.r : v1.r, s.swapped ? v2.g : v1.g, s.swapped ? v2.b : v1.b};
    const Attr c = {s.swapped ? v1.r : v2.r, s.swapped ? v1.g : v2.g, s.swapped ? v1.b : v2.b};
    int px = (i << 8) + 128 - kOrigin, py = (j << 8) + 128 - kOrigin;
    int E0 = __mul24(s.dx0, py - s.Y1) - __mul24(s.dy0, px - s.X1);
    int E1 = __mul24(s.dx1, py - s.Y2) - __mul24(s.dy1, px - s.X2);
    int E2 = __mul24(s.dx2, py - s.Y0) - __mul24(s.dy2, px - s.X0);
    if (((E0 + s.b0) | (E1 + s.b1) | (E2 + s.b2)) < 0) return false;
    float e0 = (float)E0, e1 = (float)E1, e2 = (float)E2;
    float num = fmaf(e2, s.iw2, fmaf(e1, s.iw1, e0 * s.iw0));
    depth = (float)s.A2 / num;
    float w0 = e0 * s.iw0, w1 = e1 * s.iw1, w2 = e2 * s.iw2;
    rgb[0] = fmaf(w2, c.r, fmaf(w1, b.r, w0 * a.r)) / num;
    rgb[1] = fmaf(w2, c.g, fmaf(w1, b.g, w0 * a.g)) / num;
    rgb[2] = fmaf(w2, c.b, fmaf(w1, b.b, w0 * a.b)) / num;
    // for textured scenes slots r, g hold (u, v): twice the triangle's uv area over its pixel area
    float du1 = b.r - a.r, dv1 = b.g - a.g, du2 = c.r - a.r, dv2 = c.g - a.g;
    uv_area2 = fabsf(fmaf(du1, dv2, -(du2 * dv1)));
    area2 = s.A2;
    return true;
}

__device__ __forceinline__ uint8_t to_u8(float v) {
    if (!(v == v)) return 0;
    int q = __float2int_rn(fminf(fmaxf(v, -1.0f), 256.0f));
    return (uint8_t)min(max(q, 0), 255);
}

__device__ __forceinline__ uint32_t pack_rgb(float r, float g, float b) {
    return (uint32_t)to_u8(r) | ((uint32_t)to_u8(g) << 8) | ((uint32_t)to_u8(b) << 16);
}

// Colour of a texture sample at (u, v), packed RGB.
__device__ __forceinline__ uint32_t sample_texture(const SceneDev& sc, bool bilinear, float u, float v, float uv_area2,
                                                   int area2) {
    // mip level: how often the texels-per-pixel ratio can be quartered while it is at least 4, which its exponent
    // tells (not for NaN, whose comparisons are all false)
    const float ratio = ((uv_area2 * (float)sc.tex_w) * (float)sc.tex_h) * 65536.0f / (float)area2;
    const int quarters = ratio >= 4.0f ? (int)((__float_as_uint(ratio) >> 23) - 127u) >> 1 : 0;
    const uint32_t L = min((uint32_t)quarters, sc.tex_levels - 1u);
    // Level L starts after the texels of the levels above it; the levels of a texture with sides of 2^a and 2^b
    // shrink by four up to level min(a, b), so their sum is a geometric one.  Below that only one side halves.
    const uint32_t lw = max(sc.tex_w >> L, 1u), lh = max(sc.tex_h >> L, 1u);
    const uint32_t square_levels = 31u - (uint32_t)__builtin_clz(min(sc.tex_w, sc.tex_h)), whole = sc.tex_w * sc.tex_h;
    const uint32_t K = min(L, square_levels);
    uint32_t off = ((whole - (whole >> (2u * K))) << 2) * 0xAAAAAAABu;      // exact: the sum is a third of this
    for (uint32_t l = square_levels; l < L; ++l) off += max(sc.tex_w >> l, 1u) * max(sc.tex_h >> l, 1u);
    float fu = u - floorf(u), fv = v - floorf(v);
    if (!(fu >= 0.0f && fu < 1.0f)) fu = 0.0f;
    if (!(fv >= 0.0f && fv < 1.0f)) fv = 0.0f;
    const BPS_GLOBAL uint32_t* texels = gptr(sc.texels);
    if (bilinear) {
        // the four texels around the sample position, wrapped around the texture's (power-of-two) sides
        const float x = fu * (float)lw - 0.5f, y = fv * (float)lh - 0.5f;
        const float fx0 = floorf(x), fy0 = floorf(y);
        const float tx = x - fx0, ty = y - fy0;
        const uint32_t x0 = (uint32_t)(int)fx0 & (lw - 1), x1 = (uint32_t)((int)fx0 + 1) & (lw - 1);
        const uint32_t r0 = off + ((uint32_t)(int)fy0 & (lh - 1)) * lw, r1 = off + ((uint32_t)((int)fy0 + 1) & (lh - 1)) * lw;
        const uint32_t t00 = texels[r0 + x0], t01 = texels[r0 + x1], t10 = texels[r1 + x0], t11 = texels[r1 + x1];
        float o[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const float c00 = (float)((t00 >> (8 * c)) & 0xFFu), c01 = (float)((t01 >> (8 * c)) & 0xFFu);
            const float c10 = (float)((t10 >> (8 * c)) & 0xFFu), c11 = (float)((t11 >> (8 * c)) & 0xFFu);
            const float top = fmaf(tx, c01 - c00, c00), bot = fmaf(tx, c11 - c10, c10);
            o[c] = fmaf(ty, bot - top, top);
        }
        return pack_rgb(o[0], o[1], o[2]);
    }
    const uint32_t x = min((uint32_t)(fu * (float)lw), lw - 1), y = min((uint32_t)(fv * (float)lh), lh - 1);
    return texels[off + y * lw + x] & 0x00FFFFFFu;
}

// Texel or interpolated colour of one covering fan piece (rgb holds (u, v, -) for textured scenes).
__device__ __forceinline__ uint32_t piece_output(const SceneDev& sc, bool textured, bool bilinear, const float (&rgb)[3],
                                                 float uv_area2, int area2) {
    return textured ? sample_texture(sc, bilinear, rgb[0], rgb[1], uv_area2, area2) : pack_rgb(rgb[0], rgb[1], rgb[2]);
}

// Vertex k of a triangle from its shading record: one 64-byte record per triangle holds the three
// positions and the three colours (or texture coordinates), so a pixel's gather is one cache line
// instead of one per index, position and colour.
__device__ __forceinline__ CVert record_vertex(const float4v (&rec)[4], bool textured, const float (&M)[16], int k) {
    const float f[16] = {rec[0].x, rec[0].y, rec[0].z, rec[0].w, rec[1].x, rec[1].y, rec[1].z, rec[1].w,
                         rec[2].x, rec[2].y, rec[2].z, rec[2].w, rec[3].x, rec[3].y, rec[3].z, rec[3].w};
    CVert o;
    o.c = to_clip(M, f[3 * k], f[3 * k + 1], f[3 * k + 2]);
    if (textured) {
        o.r = f[9 + 2 * k];
        o.g = f[10 + 2 * k];
        o.b = 0.0f;
    } else {
        const uint32_t rgb = __float_as_uint(f[9 + k]);
        o.r = (float)(rgb & 0xFFu);
        o.g = (float)((rgb >> 8) & 0xFFu);
        o.b = (float)((rgb >> 16) & 0xFFu);
    }
    return o;
}

// Fetches the records of a wavefront's 64 pixels.  A lane that read its own 64-byte record with four
// 16-byte loads would hit one cache line four times while it is still on its way, and the cache
// handles such hits on a pending line one after the other.  So four lanes share a record instead:
// each load instruction of the wavefront then fetches sixteen whole records (sixteen different
// lines), and the pieces change hands through `stage` (4 KB of this wavefront, LDS).  Piece k of record r sits
// at 4 r + (k ^ (r / 4 mod 4)), so that the sixteen lanes an LDS read serves together touch sixteen different
// places.
__device__ __forceinline__ void load_records(const SceneDev& sc, uint32_t id, bool valid, int lane, float4v* stage,
                                             float4v (&rec)[4]) {
    const BPS_GLOBAL float4v* base = (const BPS_GLOBAL float4v*)sc.tri_rec;
    const uint32_t mine = valid ? id : 0u;      // (any record will do: its piece is not looked at)
    const uint32_t part = (uint32_t)lane & 3u;
    float4v piece[4];      // all four loads are on their way before the first is waited for
#pragma unroll
    for (int s = 0; s < 4; ++s) piece[s] = base[(size_t)(uint32_t)__shfl((int)mine, 16 * s + (lane >> 2), 64) * 4 + part];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int from = 16 * s + (lane >> 2);
        stage[4 * from + (int)(part ^ (((uint32_t)from >> 2) & 3u))] = piece[s];
    }
    wave_lds_sync();
#pragma unroll
    for (int k = 0; k < 4; ++k) rec[k] = stage[4 * lane + (k ^ ((lane >> 2) & 3))];
    wave_lds_sync();     // the stage is used again below
}

// Clipped polygons of up to kClipSlots triangles: seven words per corner, the corners of one triangle in a ring
// of kMaxPoly (each plane's pass reads the corners behind and writes the ones ahead), the triangle fastest.
// A pass that reads n corners overtakes itself only if more than 16 - n of them are entered from outside, at most
// n / 2 can be, and n is at most 10 before the last plane: it never does.
constexpr int kClipSlots = 8;
static_assert(kMaxPoly * 7 * kClipSlots * 4 <= 64 * 64, "the polygons fit in the wavefront's stage");

struct PolyRing {
    float* at;      // this triangle's column
    __device__ __forceinline__ float* corner(int q) const { return at + (q & (kMaxPoly - 1)) * 7 * kClipSlots; }
    __device__ __forceinline__ void put(int q, const CVert& v) const {
        float* p = corner(q);
        p[0] = v.c.x; p[kClipSlots] = v.c.y; p[2 * kClipSlots] = v.c.z; p[3 * kClipSlots] = v.c.w;
        p[4 * kClipSlots] = v.r; p[5 * kClipSlots] = v.g; p[6 * kClipSlots] = v.b;
    }
    __device__ __forceinline__ CVert get(int q) const {
        const float* p = corner(q);
        CVert v;
        v.c.x = p[0]; v.c.y = p[kClipSlots]; v.c.z = p[2 * kClipSlots]; v.c.w = p[3 * kClipSlots];
        v.r = p[4 * kClipSlots]; v.g = p[5 * kClipSlots]; v.b = p[6 * kClipSlots];
        return v;
    }
    __device__ __forceinline__ void put_projected(int q, uint32_t xy, float iw, const CVert& v) const {
        float* p = corner(q);
        p[0] = __uint_as_float(xy); p[kClipSlots] = iw; p[2 * kClipSlots] = v.r; p[3 * kClipSlots] = v.g; p[4 * kClipSlots] = v.b;
    }
    __device__ __forceinline__ SVert get_projected(int q) const {
        const float* p = corner(q);
        SVert v;
        v.xy = __float_as_uint(p[0]); v.iw = p[kClipSlots]; v.r = p[2 * kClipSlots]; v.g = p[3 * kClipSlots]; v.b = p[4 * kClipSlots];
        return v;
    }
};

// The point at t of the way from the inside corner a to the outside corner b.
__device__ __forceinline__ CVert along(const CVert& a, const CVert& b, float t) {
    CVert o;
    o.c.x = fmaf(t, b.c.x - a.c.x, a.c.x);
    o.c.y = fmaf(t, b.c.y - a.c.y, a.c.y);
    o.c.z = fmaf(t, b.c.z - a.c.z, a.c.z);
    o.c.w = fmaf(t, b.c.w - a.c.w, a.c.w);
    o.r = fmaf(t, b.r - a.r, a.r);
    o.g = fmaf(t, b.g - a.g, a.g);
    o.b = fmaf(t, b.b - a.b, a.b);
    return o;
}

// Where the edge from the inside corner a to the outside corner b, at distances da and db, crosses the plane.
__device__ __forceinline__ CVert crossing(const CVert& a, const CVert& b, float da, float db) { return along(a, b, da / (da - db)); }

// Clips one triangle against the planes of oc_or in the rule's order and projects what is left.  Returns the number
// of corners, which start at `first` of the ring; 0 when nothing is left or a corner cannot be projected.
__device__ __forceinline__ int clip_polygon(const PolyRing& ring, const CVert& a, const CVert& b, const CVert& c,
                                            uint32_t oc_or, const FrameParams& fp, int& first) {
    ring.put(0, a);
    ring.put(1, b);
    ring.put(2, c);
    int cnt = 3, from = 0;
    uint32_t todo = ((oc_or >> 4) & 3u) | ((oc_or & 15u) << 2);      // near, far, left, right, top, bottom
    while (todo != 0u && cnt >= 3) {
        const int p = __builtin_ctz(todo), k = p < 2 ? p + 4 : p - 2;
        todo &= todo - 1u;
        int m = 0;
        const int to = from + cnt;
        CVert prev = ring.get(to - 1);
        float dprev = plane_dist(prev.c, k);
        for (int q = 0; q < cnt; ++q) {
            const CVert v = ring.get(from + q);
            const float dv = plane_dist(v.c, k);
            const bool cin = dv >= 0.0f, pin = dprev >= 0.0f;
            if (cin != pin && m < kMaxPoly) {
                ring.put(to + m, crossing(pick(cin, v, prev), pick(cin, prev, v), cin ? dv : dprev, cin ? dprev : dv));
                ++m;
            }
            if (cin && m < kMaxPoly) {
                ring.put(to + m, v);
                ++m;
            }
            prev = v;
            dprev = dv;
        }
        cnt = m;
        from = to;
    }
    first = from;
    if (cnt < 3) return 0;
    bool ok = true;
    for (int q = 0; q < cnt; ++q) {
        const CVert v = ring.get(from + q);
        bool unused;
        uint32_t xy;
        float iw;
        ok = project(v.c, fp, xy, iw, unused) && ok;
        ring.put_projected(from + q, xy, iw, v);
    }
    return ok ? cnt : 0;
}

// n / d for n < 2^31 by a multiplication (d > 0): exact for the usual round-up multiplier of 33 bits.
struct Divider {
    uint32_t mul, shift;
};
Divider make_divider(uint32_t d) {
    uint32_t shift = 0;
    while ((1ull << shift) < d) ++shift;
    return Divider{(uint32_t)(((1ull << 32) * ((1ull << shift) - d)) / d + 1ull), shift};
}
__device__ __forceinline__ uint32_t divide(uint32_t n, const Divider& d) { return (__umulhi(n, d.mul) + n) >> d.shift; }

}  // namespace

// The packed coordinates of a triangle differ by no more than 16 bits hold.
__device__ __forceinline__ bool fits_16_bits(uint32_t xy0, uint32_t xy1, uint32_t xy2) {
    const short2v mn = __builtin_elementwise_min(as_s2(xy0), __builtin_elementwise_min(as_s2(xy1), as_s2(xy2)));
    const short2v mx = __builtin_elementwise_max(as_s2(xy0), __builtin_elementwise_max(as_s2(xy1), as_s2(xy2)));
    return (as_u32(mx - mn) & 0x80008000u) == 0u;
}

// Colour of a pixel inside the triangle s with edge functions E0, E1, E2 there; the attributes are those of its
// oriented vertices.  One reciprocal serves the three quotients.  usable: the caller's own conditions for the short
// forms; returns whether these hold and `out` was set.
template <bool TEXTURED>
__device__ __forceinline__ bool attribute_output(const SceneDev& sc, const FrameParams& fp, const PackedSetup& s, int E0, int E1,
                                                 int E2, float ar, float ag, float ab, float br, float bg, float bb, float cr,
                                                 float cg, float cb, bool usable, uint32_t& out) {
    const float e0 = (float)E0, e1 = (float)E1, e2 = (float)E2;
    const float w0 = e0 * s.iw0, num = fmaf(e2, s.iw2, fmaf(e1, s.iw1, w0)), w1 = e1 * s.iw1, w2 = e2 * s.iw2;
    const float y = recip_normal(num);
    auto quotient = [&](float n) {      // div_in_range(n, num)
        const float q = n * y;
        return fmaf(fmaf(-num, q, n), y, q);
    };
    auto mean = [&](float a, float b, float c) { return fmaf(w2, c, fmaf(w1, b, w0 * a)); };
    if (TEXTURED) {
        const float nu = mean(ar, br, cr), nv = mean(ag, bg, cg);
        // texture coordinates may be of any size; zero divides like the numbers in between
        auto in_range = [](float n) { return ((fabsf(n) < 0x1p90f) & (fabsf(n) > 0x1p-60f)) | (n == 0.0f); };
        usable = usable & in_range(nu) & in_range(nv);
        const float du1 = br - ar, dv1 = bg - ag, du2 = cr - ar, dv2 = cg - ag;
        if (usable)
            out = sample_texture(sc, fp.bilinear != 0, quotient(nu), quotient(nv), fabsf(fmaf(du1, dv2, -(du2 * dv1))), s.A2);
    } else {
        // a mean of values in 0..255 rounds to one of 0..255: the rounding of an addition leaves it in the low byte
        const uint32_t r = __float_as_uint(quotient(mean(ar, br, cr)) + 12582912.0f);
        const uint32_t g = __float_as_uint(quotient(mean(ag, bg, cg)) + 12582912.0f);
        const uint32_t b = __float_as_uint(quotient(mean(ab, bb, cb)) + 12582912.0f);
        const uint32_t rgb = __builtin_amdgcn_perm(b, __builtin_amdgcn_perm(g, r, 0x0C0C0400u), 0x0C040100u);
        out = usable ? rgb : out;
    }
    return usable;
}

// Colour pass: one thread per pixel, one 8x8-pixel tile per wavefront, everything within the wavefront.  A winner
// whose three vertices lie inside every clip plane (nine in ten) is projected and shaded from registers with the
// short forms of the raster kernel (one test per vertex and axis, packed 16-bit set-up, one reciprocal for the three
// quotients, no coverage test: the winner covers its pixel).  A winner that crosses one plane keeps three or four
// corners and is clipped in registers too.  The others (1 % at 64x64 with 1 M triangles, more where triangles are
// large) share few triangles per tile: one lane per different triangle clips it into LDS, eight at a time, and the
// pixels look for their fan piece there.
// What bounds it: vector-ALU issue and the chain of loads (id, record, texels) in about equal parts, so short code
// and many wavefronts: 72 registers let seven per SIMD run (12 words spilled on the general path), 66 -> 61 us against
// five.  Before, as two kernels with a queue of the pixels that cross several planes between them, 772 -> 460 vector
// instructions per wavefront: 1024 frames of 64x64, 1 M triangles, 97 -> 61 us; 192 frames of 128x128 with textures,
// where large triangles kept the second kernel's few wavefronts waiting, 161 -> 60 us.
template <bool TEXTURED>
__device__ __forceinline__ uint32_t shade_tile(const SceneDev& sc, const float* __restrict__ view_proj, const FrameParams& fp,
                                               uint32_t id, bool valid, int i, int j, int lane, float4v* stage) {
    float M[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) M[k] = view_proj[k];
    float4v rec[4];
    load_records(sc, id, valid, lane, stage, rec);
    const CVert a = record_vertex(rec, TEXTURED, M, 0), b = record_vertex(rec, TEXTURED, M, 1),
                c = record_vertex(rec, TEXTURED, M, 2);
    const float iw0 = recip_normal(a.c.w), iw1 = recip_normal(b.c.w), iw2 = recip_normal(c.c.w);
    auto inside = [](const Clip4& q) { return (fabsf(q.x) <= q.w) & (fabsf(q.y) <= q.w) & (q.z >= 0.0f) & (q.z <= q.w); };
    const bool regular = valid & inside(a.c) & inside(b.c) & inside(c.c) & iw_in_range(iw0) & iw_in_range(iw1) & iw_in_range(iw2);
    uint32_t out = 0;
    bool done = false;
    const uint32_t centre = pack_xy((i << 8) + 128, (j << 8) + 128);
    if (regular) {
        const uint32_t xy0 = snap_xy(fmaf(a.c.x * iw0, fp.sx, fp.sx), fmaf(a.c.y * iw0, fp.sy, fp.sy));
        const uint32_t xy1 = snap_xy(fmaf(b.c.x * iw1, fp.sx, fp.sx), fmaf(b.c.y * iw1, fp.sy, fp.sy));
        const uint32_t xy2 = snap_xy(fmaf(c.c.x * iw2, fp.sx, fp.sx), fmaf(c.c.y * iw2, fp.sy, fp.sy));
        const PackedSetup s = make_packed_setup(xy0, xy1, xy2, iw0, iw1, iw2);
        int E0, E1, E2;
        packed_edges(s, centre, E0, E1, E2);
        const bool sw = s.swapped, fits = fits_16_bits(xy0, xy1, xy2);
        if (TEXTURED) {
            done = attribute_output<true>(sc, fp, s, E0, E1, E2, a.r, a.g, 0.0f, sw ? c.r : b.r, sw ? c.g : b.g, 0.0f,
                                          sw ? b.r : c.r, sw ? b.g : c.g, 0.0f, fits, out);
        } else {
            const uint32_t ca = __float_as_uint(rec[2].y), cb = __float_as_uint(sw ? rec[2].w : rec[2].z),
                           cc = __float_as_uint(sw ? rec[2].z : rec[2].w);
            auto f = [](uint32_t rgb, int shift) { return (float)((rgb >> shift) & 0xFFu); };
            done = attribute_output<false>(sc, fp, s, E0, E1, E2, f(ca, 0), f(ca, 8), f(ca, 16), f(cb, 0), f(cb, 8), f(cb, 16),
                                           f(cc, 0), f(cc, 8), f(cc, 16), fits, out);
        }
    }
    if (ballot64(valid && !done) == 0ull) return out;
    // ---- Crossing exactly one plane: the vertex S on its own side, the one before it P and the one after it N leave
    // the corners X1 (between P and S), X2 (between S and N) and either S or N and P.  The order is the general
    // clipper's: the edges c-a, a-b, b-c in turn, a crossing first and then the edge's end if that is inside.
    {
        auto out_of = [](bool oa, bool ob, bool oc) -> bool { return oa | ob | oc; };
        const bool pl[6] = {
            out_of(!(a.c.x >= -a.c.w), !(b.c.x >= -b.c.w), !(c.c.x >= -c.c.w)), out_of(!(a.c.x <= a.c.w), !(b.c.x <= b.c.w), !(c.c.x <= c.c.w)),
            out_of(!(a.c.y >= -a.c.w), !(b.c.y >= -b.c.w), !(c.c.y >= -c.c.w)), out_of(!(a.c.y <= a.c.w), !(b.c.y <= b.c.w), !(c.c.y <= c.c.w)),
            out_of(!(a.c.z >= 0.0f), !(b.c.z >= 0.0f), !(c.c.z >= 0.0f)), out_of(!(a.c.z <= a.c.w), !(b.c.z <= b.c.w), !(c.c.z <= c.c.w))};
        bool some = false, more = false;
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            more = more | (some & pl[k]);
            some = some | pl[k];
        }
        if (valid & !done & some & !more) {
            // distance w + x, w - x, w + y, w - y, z or w - z
            const bool along_x = pl[0] | pl[1], along_y = pl[2] | pl[3], negative = pl[1] | pl[3] | pl[5];
            const float with_w = pl[4] ? 0.0f : 1.0f;
            auto dist = [&](const Clip4& q) {
                const float v = along_x ? q.x : along_y ? q.y : q.z;
                return fmaf(with_w, q.w, negative ? -v : v);
            };
            const float da = dist(a.c), db = dist(b.c), dc = dist(c.c);
            const bool ia = da >= 0.0f, ib = db >= 0.0f, ic = dc >= 0.0f;
            const bool is_a = ib == ic, is_c = !is_a & (ia == ib), is_b = !is_a & !is_c;
            const CVert S = pick(is_a, a, pick(is_b, b, c)), P = pick(is_a, c, pick(is_b, a, b)), N = pick(is_a, b, pick(is_b, c, a));
            const float dS = is_a ? da : is_b ? db : dc, dP = is_a ? dc : is_b ? da : db, dN = is_a ? db : is_b ? dc : da;
            const bool s_in = is_a ? ia : is_b ? ib : ic;
            const float n1 = s_in ? dS : dP, d1 = n1 - (s_in ? dP : dS), n2 = s_in ? dS : dN, d2 = n2 - (s_in ? dN : dS);
            auto usable = [](float n, float d) { return iw_in_range(d) & ((n == 0.0f) | iw_in_range(n)); };
            bool fits = usable(n1, d1) & usable(n2, d2);
            auto snapped = [&](const CVert& v) {
                SVert o;
                o.iw = recip_normal(v.c.w);
                o.xy = snap_xy(fmaf(v.c.x * o.iw, fp.sx, fp.sx), fmaf(v.c.y * o.iw, fp.sy, fp.sy));
                o.r = v.r; o.g = v.g; o.b = v.b;
                fits = fits & iw_in_range(o.iw);
                return o;
            };
            const SVert X1 = snapped(along(pick(s_in, S, P), pick(s_in, P, S), div_in_range(n1, d1)));
            const SVert X2 = snapped(along(pick(s_in, S, N), pick(s_in, N, S), div_in_range(n2, d2)));
            const SVert A = snapped(pick(s_in, S, N));
            const bool fits3 = fits;                  // without P, which is a corner only if S is outside
            const SVert B = snapped(P);
            fits = s_in ? fits3 : fits;
            const SVert o0 = pick(is_c, X2, pick(is_b & !s_in, B, X1));
            const SVert o1 = pick((is_c & s_in) | (is_b & !s_in), X1, pick(is_a & !s_in, X2, A));
            const SVert o2 = pick((is_c & s_in) | (is_a & !s_in), A, pick(is_c & !s_in, B, X2));
            const SVert o3 = pick(is_a, B, pick(is_b, A, X1));
            PackedSetup s = make_packed_setup(o0.xy, o1.xy, o2.xy, o0.iw, o1.iw, o2.iw);
            const PackedSetup s2 = make_packed_setup(o0.xy, o2.xy, o3.xy, o0.iw, o2.iw, o3.iw);
            int E0, E1, E2, F0, F1, F2;
            packed_edges(s, centre, E0, E1, E2);
            packed_edges(s2, centre, F0, F1, F2);
            const bool fits1 = fits_16_bits(o0.xy, o1.xy, o2.xy), fits2 = s_in | fits_16_bits(o0.xy, o2.xy, o3.xy);
            const bool in1 = (s.A2 != 0) & (E0 >= s.t0) & (E1 >= s.t1) & (E2 >= s.t2);
            const bool in2 = !s_in & (s2.A2 != 0) & (F0 >= s2.t0) & (F1 >= s2.t1) & (F2 >= s2.t2);
            fits = fits & fits1 & fits2 & (in1 != in2);      // exactly one piece covers the centre, or the general path decides
            const SVert u = pick(in1, o1, o2), v = pick(in1, o2, o3);
            const bool sw = in1 ? s.swapped : s2.swapped;
            s.A2 = in1 ? s.A2 : s2.A2;
            s.iw1 = in1 ? s.iw1 : s2.iw1;
            s.iw2 = in1 ? s.iw2 : s2.iw2;
            E0 = in1 ? E0 : F0;
            E1 = in1 ? E1 : F1;
            E2 = in1 ? E2 : F2;
            done = attribute_output<TEXTURED>(sc, fp, s, E0, E1, E2, o0.r, o0.g, o0.b, sw ? v.r : u.r, sw ? v.g : u.g, sw ? v.b : u.b,
                                              sw ? u.r : v.r, sw ? u.g : v.g, sw ? u.b : v.b, fits, out);
        }
    }
    const bool multi = valid && !done;
    uint32_t oc_or = 0;
    if (multi) oc_or = outcode(a.c) | outcode(b.c) | outcode(c.c);
    // ---- everything else, several planes above all: one lane per different triangle clips
    const u64 multi_mask = ballot64(multi);
    u64 todo = multi_mask;
    while (todo != 0ull) {
        int slot = -1, clipper = 0, n_slots = 0;
        while (todo != 0ull && n_slots < kClipSlots) {
            const int l = __builtin_ctzll(todo);
            const bool mine = multi && id == (uint32_t)bcast_i((int)id, l);
            if (mine) {
                slot = n_slots;
                clipper = l;
            }
            todo &= ~ballot64(mine);
            ++n_slots;
        }
        PolyRing ring;
        ring.at = reinterpret_cast<float*>(stage) + max(slot, 0);
        int cnt = 0, first = 0;
        if (slot >= 0 && lane == clipper) cnt = clip_polygon(ring, a, b, c, oc_or, fp, first);
        wave_lds_sync();
        cnt = __shfl(cnt, clipper, 64);
        first = __shfl(first, clipper, 64);
        if (slot >= 0 && cnt >= 3) {
            // the fan pieces of one triangle tile it; should rounding ever make two of them
            // cover this pixel, the nearer one is the one the z-test kept (first one on a tie)
            float best = 0.0f;
            bool found = false;
            const SVert s0 = ring.get_projected(first);
            SVert s1 = ring.get_projected(first + 1);
            for (int q = 1; q + 1 < cnt; ++q) {
                const SVert s2 = ring.get_projected(first + q + 1);
                float d, rgb[3], uv_area2;
                int area2;
                if (piece_colour(s0, s1, s2, i, j, d, rgb, uv_area2, area2) && (!found || d < best)) {
                    found = true;
                    best = d;
                    out = piece_output(sc, TEXTURED, fp.bilinear != 0, rgb, uv_area2, area2);
                }
                s1 = s2;
            }
        }
        wave_lds_sync();
    }
    return out;
}

// Work-groups are dealt to the eight dies round-robin by index.  The groups of one frame (of four tiles each) are
// mapped to one die, so that pixels of neighbouring tiles that show the same triangle find its record in that
// die's L2: eight consecutive indices belong to eight different frames; what is left of the batch goes in order.
__global__ __launch_bounds__(256, 7) void k_shade(const SceneDev* __restrict__ scenes, const uint32_t* __restrict__ env_scene,
                                               const float* __restrict__ view_proj, FrameParams fp, uint32_t B,
                                               uint32_t groups_per_frame, Divider by_groups, Divider by_tiles_x,
                                               const uint32_t* __restrict__ tri_id, uint8_t* __restrict__ out_rgb,
                                               int dword_stores) {
    __shared__ float4v stage_all[4 * 256];
    const uint32_t in_sets = (B & ~7u) * groups_per_frame;
    uint32_t env, part;
    if (blockIdx.x < in_sets) {
        const uint32_t turn = blockIdx.x >> 3, set = divide(turn, by_groups);
        env = set * 8u + (blockIdx.x & 7u);
        part = turn - set * groups_per_frame;
    } else {
        const uint32_t at = blockIdx.x - in_sets, k = divide(at, by_groups);
        env = (B & ~7u) + k;
        part = at - k * groups_per_frame;
    }
    const uint32_t tiles_x = (uint32_t)fp.W >> 3, tiles = tiles_x * ((uint32_t)fp.H >> 3);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), tile = part * 4u + wave;
    if (tile >= tiles) return;
    const uint32_t ty = divide(tile, by_tiles_x), tx = tile - ty * tiles_x;
    const int lane = (int)(threadIdx.x & 63u);
    const int i = (int)(tx * 8u) + (lane & 7), j = (int)(ty * 8u) + (lane >> 3);
    const size_t frame = (size_t)env * (size_t)(fp.H * fp.W);
    const SceneDev sc = scenes[env_scene[env]];
    const uint32_t id = tri_id[frame + (uint32_t)(j * fp.W + i)];
    const bool valid = id != 0xFFFFFFFFu && sc.tri_rec != nullptr && id < sc.n_tris;
    float4v* stage = stage_all + 256 * wave;
    const float* vp = view_proj + (size_t)env * 16;
    uint32_t out = 0;
    if (ballot64(valid) != 0ull)
        out = sc.texels != nullptr ? shade_tile<true>(sc, vp, fp, id, valid, i, j, lane, stage)
                                   : shade_tile<false>(sc, vp, fp, id, valid, i, j, lane, stage);
    uint8_t* frame_rgb = out_rgb + 3 * frame;
    if (dword_stores) {
        // a row of the tile is 24 bytes: six words, each the end of one pixel and the start of the next
        const int row = (lane * 43) >> 8, word = lane - 6 * row;             // lane / 6 for lanes below 64
        const int half = word >= 3 ? 1 : 0, cut = word - 3 * half, px = (8 * row + 4 * half + cut) & 63;
        const uint32_t lo = (uint32_t)__shfl((int)out, px, 64), hi = (uint32_t)__shfl((int)out, (px + 1) & 63, 64);
        const uint32_t v = (lo >> (8 * cut)) | (hi << (24 - 8 * cut));
        if (lane < 48)
            *reinterpret_cast<uint32_t*>(frame_rgb + (uint32_t)(3 * (((int)(ty * 8u) + row) * fp.W + (int)(tx * 8u)) + 4 * word)) = v;
    } else {
        uint8_t* o = frame_rgb + (uint32_t)(3 * (j * fp.W + i));
        o[0] = (uint8_t)out;
        o[1] = (uint8_t)(out >> 8);
        o[2] = (uint8_t)(out >> 16);
    }
}

// 2x2 box filter from the rendered frame to the output frame (the paper renders its 128-pixel
// observations at twice the resolution and downsamples, Sec. 4.1).  Depth: ((a + b) + (c + d)) / 4
// in float32 in that order; colour: (a + b + c + d + 2) >> 2 per channel.
__global__ __launch_bounds__(256) void k_downsample(const float* __restrict__ depth, const uint8_t* __restrict__ rgb,
                                                    uint32_t B, int H, int W, float* __restrict__ out_depth,
                                                    uint8_t* __restrict__ out_rgb) {
    const int oh = H >> 1, ow = W >> 1;
    size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= (size_t)B * oh * ow) return;
    const int x = (int)(p % ow), y = (int)((p / ow) % oh);
    const size_t b = p / ((size_t)ow * oh);
    const size_t s = b * H * W + (size_t)(2 * y) * W + 2 * x;
    out_depth[p] = ((depth[s] + depth[s + 1]) + (depth[s + W] + depth[s + W + 1])) * 0.25f;
    if (rgb && out_rgb)
        for (int c = 0; c < 3; ++c)
            out_rgb[3 * p + c] = (uint8_t)(((int)rgb[3 * s + c] + (int)rgb[3 * (s + 1) + c] + (int)rgb[3 * (s + W) + c] +
                                            (int)rgb[3 * (s + W + 1) + c] + 2) >> 2);
}

hipError_t launch_downsample(hipEvent_t done, hipStream_t stream, const float* depth, const uint8_t* rgb, uint32_t B, int H, int W,
                       float* out_depth, uint8_t* out_rgb) {
    size_t n = (size_t)B * (H / 2) * (W / 2);
    return launch_kernel(done, &k_downsample, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, depth, rgb, B, H, W, out_depth, out_rgb);
}

// One thread per triangle: gather its three positions and colours (or texture coordinates) from the
// uploaded arrays into its 64-byte shading record.
__global__ __launch_bounds__(256) void k_build_shade_records(SceneDev sc, float* __restrict__ tri_rec) {
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= sc.n_tris) return;
    float f[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) f[k] = 0.0f;
    for (int k = 0; k < 3; ++k) {
        const uint32_t vi = sc.indices[3 * t + k];
        f[3 * k] = sc.verts[3 * (size_t)vi];
        f[3 * k + 1] = sc.verts[3 * (size_t)vi + 1];
        f[3 * k + 2] = sc.verts[3 * (size_t)vi + 2];
        if (sc.uvs) {
            f[9 + 2 * k] = sc.uvs[2 * (size_t)vi];
            f[10 + 2 * k] = sc.uvs[2 * (size_t)vi + 1];
        } else if (sc.colors) {
            const uint8_t* col = sc.colors + 3 * (size_t)vi;
            f[9 + k] = __uint_as_float((uint32_t)col[0] | ((uint32_t)col[1] << 8) | ((uint32_t)col[2] << 16));
        }
    }
    float4* dst = reinterpret_cast<float4*>(tri_rec) + 4 * t;
#pragma unroll
    for (int k = 0; k < 4; ++k) dst[k] = make_float4(f[4 * k], f[4 * k + 1], f[4 * k + 2], f[4 * k + 3]);
}

void launch_build_shade_records(hipStream_t stream, const SceneDev& sc, float* tri_rec) {
    hipLaunchKernelGGL(k_build_shade_records, dim3((sc.n_tris + 255u) / 256u), dim3(256), 0, stream, sc, tri_rec);
}

hipError_t launch_shade(hipEvent_t done, hipStream_t stream, const SceneDev* scenes, const uint32_t* env_scene, const float* view_proj,
                  const FrameParams& fp, uint32_t B, const uint32_t* tri_id, uint8_t* out_rgb) {
    const uint32_t tiles_x = (uint32_t)fp.W / 8u, tiles = tiles_x * ((uint32_t)fp.H / 8u), per_frame = (tiles + 3u) / 4u;
    const int dword_stores = (reinterpret_cast<uintptr_t>(out_rgb) & 3u) == 0u ? 1 : 0;      // frames are multiples of 4 bytes
    return launch_kernel(done, &k_shade, dim3(B * per_frame), dim3(256), 0, stream, scenes, env_scene, view_proj, fp, B, per_frame,
                         make_divider(per_frame), make_divider(tiles_x), tri_id, out_rgb, dword_stores);
}

}  // namespace bps
