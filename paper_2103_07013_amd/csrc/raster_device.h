// Device helpers shared by the raster and shading kernels: wave intrinsics, the vertex transform,
// outcodes, projection / snapping and the integer triangle set-up.  Both kernels must evaluate
// exactly the same IEEE operation sequence, so the code lives in one place.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "raster_kernels.h"

namespace bps {
namespace dev {

typedef unsigned long long u64;

// Loads through pointers that arrive inside structs would otherwise be generic ("flat") accesses.
#define BPS_GLOBAL __attribute__((address_space(1)))
template <class T>
__device__ __forceinline__ const BPS_GLOBAL T* gptr(const T* p) {
    return (const BPS_GLOBAL T*)p;
}

__device__ __forceinline__ u64 ballot64(bool p) { return __builtin_amdgcn_ballot_w64(p); }

__device__ __forceinline__ uint32_t rank_below(u64 mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Orders this wavefront's LDS writes before its later LDS reads by other lanes.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ int bcast_i(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }
__device__ __forceinline__ float bcast_f(float v, int lane) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// Snapped screen coordinates travel as two signed 16-bit halves, x low and y high, relative to
// kOrigin = 64 pixels, so that the whole range [-64, 256*128 + 64] of a 128-pixel axis fits and
// bounding boxes can be computed with packed 16-bit instructions.
__device__ __forceinline__ uint32_t pack_xy(int X, int Y) {
    return ((uint32_t)(X - kOrigin) & 0xFFFFu) | ((uint32_t)(Y - kOrigin) << 16);
}
__device__ __forceinline__ int unpack_x(uint32_t xy) { return (int)(short)(xy & 0xFFFFu); }
__device__ __forceinline__ int unpack_y(uint32_t xy) { return (int)xy >> 16; }

// ---------------------------------------------------------------------------------------------
// Triangle in snapped screen space, oriented so that A2 > 0, with its edge set-up.
struct Setup {
    int X0, Y0, X1, Y1, X2, Y2;   // 1/256-px coordinates relative to kOrigin
    float iw0, iw1, iw2;
    int A2;
    int dx0, dy0, dx1, dy1, dx2, dy2;   // edge k is opposite vertex k
    int b0, b1, b2;                     // 0 on a top-left edge, -1 otherwise
    bool swapped;                       // vertices 1 and 2 were exchanged to make A2 positive
};

__device__ __forceinline__ int tl_bias(int dx, int dy) { return (dy < 0 || (dy == 0 && dx > 0)) ? 0 : -1; }

__device__ __forceinline__ Setup make_setup(uint32_t xy0, uint32_t xy1, uint32_t xy2, float iw0, float iw1, float iw2) {
    Setup s;
    s.X0 = unpack_x(xy0); s.Y0 = unpack_y(xy0);
    s.X1 = unpack_x(xy1); s.Y1 = unpack_y(xy1);
    s.X2 = unpack_x(xy2); s.Y2 = unpack_y(xy2);
    s.iw0 = iw0; s.iw1 = iw1; s.iw2 = iw2;
    int a2 = __mul24(s.X1 - s.X0, s.Y2 - s.Y0) - __mul24(s.X2 - s.X0, s.Y1 - s.Y0);
    s.swapped = a2 < 0;
    if (a2 < 0) {   // two-sided: swap vertices 1 and 2
        int t;
        t = s.X1; s.X1 = s.X2; s.X2 = t;
        t = s.Y1; s.Y1 = s.Y2; s.Y2 = t;
        float f = s.iw1; s.iw1 = s.iw2; s.iw2 = f;
        a2 = -a2;
    }
    s.A2 = a2;
    s.dx0 = s.X2 - s.X1; s.dy0 = s.Y2 - s.Y1;
    s.dx1 = s.X0 - s.X2; s.dy1 = s.Y0 - s.Y2;
    s.dx2 = s.X1 - s.X0; s.dy2 = s.Y1 - s.Y0;
    s.b0 = tl_bias(s.dx0, s.dy0);
    s.b1 = tl_bias(s.dx1, s.dy1);
    s.b2 = tl_bias(s.dx2, s.dy2);
    return s;
}

// Correctly rounded 1 / w from the hardware approximation and one correction step: equal to the IEEE
// quotient whenever the result is a normal number (compared once for all 2^32 arguments on gfx950; a test draws
// a frame for every mantissa of w).  Zeros, denormals, infinities and arguments whose reciprocal is not normal
// come out as something that is not normal either.  3 instructions instead of the 11 of a division.
__device__ __forceinline__ float recip_normal(float w) {
    const float r = __builtin_amdgcn_rcpf(w);
    return fmaf(fmaf(-w, r, 1.0f), r, r);
}
constexpr int kClassNormal = 0x108;      // v_cmp_class: +normal | -normal
__device__ __forceinline__ float recip(float w) {
    float r = recip_normal(w);
    if (!__builtin_amdgcn_classf(r, kClassNormal)) r = 1.0f / w;
    return r;
}

// Correctly rounded a / b for operands and quotients far from the ends of the exponent range.  With
// y = RN(1/b) the product q0 = RN(a y) lies within half a unit of every midpoint that a / b can come
// within 2^-47 of, the remainder a - b q0 is exact, and RN(q0 + remainder y) is then the IEEE quotient
// (Markstein's correction).  6 instructions instead of 11 and no use of VCC.
__device__ __forceinline__ float div_in_range(float a, float b) {
    const float y = recip_normal(b);
    const float q = a * y;
    return fmaf(fmaf(-b, q, a), y, q);
}
// Vertices whose 1/w lies in [2^-60, 2^60] keep every depth of their triangles in that range: the
// interpolated 1/w times A2 < 2^31 then stays within [2^-60, 2^91], which div_in_range is made for.
__device__ __forceinline__ bool iw_in_range(float iw) {      // one subtraction, one compare; false for NaN and negatives
    return __float_as_uint(iw) - 0x21800000u <= 0x5D800000u - 0x21800000u;
}

typedef short short2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ short2v as_s2(uint32_t v) { return __builtin_bit_cast(short2v, v); }
__device__ __forceinline__ uint32_t as_u32(short2v v) { return __builtin_bit_cast(uint32_t, v); }

// Set-up of a triangle on packed 16-bit coordinates: half the instructions of make_setup.  Only for
// triangles whose coordinate differences fit 16 bits (a whole 64-pixel frame does; on larger frames the
// callers check the box).  E2 follows from E0 + E1 + E2 = A2.
struct PackedSetup {
    uint32_t v1, v2;          // reference vertices of edges 0 and 1
    uint32_t e0, e1;          // edge vectors v2 - v1 and v0 - v2
    float iw0, iw1, iw2;
    int A2;
    bool swapped;             // vertices 1 and 2 were exchanged to make A2 positive
    int t0, t1, t2;           // smallest value of E that is inside: 0 on a top-left edge, 1 otherwise
};
// Top-left: dy < 0, or dy = 0 and dx > 0, with dy in the high half; dx = dy = 0 only if A2 = 0.
__device__ __forceinline__ int packed_threshold(uint32_t e) { return (int)e < 0x8000 ? 0 : 1; }
__device__ __forceinline__ int cross16(uint32_t a, uint32_t b) {
    return __mul24(unpack_x(a), unpack_y(b)) - __mul24(unpack_x(b), unpack_y(a));
}
__device__ __forceinline__ PackedSetup make_packed_setup(uint32_t xy0, uint32_t xy1, uint32_t xy2, float iw0, float iw1,
                                                         float iw2) {
    PackedSetup s;
    const int a2 = cross16(as_u32(as_s2(xy1) - as_s2(xy0)), as_u32(as_s2(xy2) - as_s2(xy0)));
    const bool swap = a2 < 0;      // two-sided: exchange vertices 1 and 2
    s.swapped = swap;
    s.A2 = swap ? -a2 : a2;
    s.v1 = swap ? xy2 : xy1;
    s.v2 = swap ? xy1 : xy2;
    s.iw0 = iw0;
    s.iw1 = swap ? iw2 : iw1;
    s.iw2 = swap ? iw1 : iw2;
    s.e0 = as_u32(as_s2(s.v2) - as_s2(s.v1));
    s.e1 = as_u32(as_s2(xy0) - as_s2(s.v2));
    s.t0 = packed_threshold(s.e0);
    s.t1 = packed_threshold(s.e1);
    s.t2 = packed_threshold(as_u32(as_s2(s.v1) - as_s2(xy0)));
    return s;
}
// Edge functions at pixel centre p (packed like the vertices): dx (py - Y) - dy (px - X).
__device__ __forceinline__ void packed_edges(const PackedSetup& s, uint32_t p, int& E0, int& E1, int& E2) {
    E0 = cross16(s.e0, as_u32(as_s2(p) - as_s2(s.v1)));
    E1 = cross16(s.e1, as_u32(as_s2(p) - as_s2(s.v2)));
    E2 = s.A2 - E0 - E1;
}

// The part of the frame one work-group owns: pixels [x0, x0 + w) x [y0, y0 + h), and the same
// rectangle in normalised device coordinates (aL <= x/w <= aR, aT <= y/w <= aB).
struct Window {
    int x0, y0, w, h;
    int pitch;                // pixels from one row of the key buffer to the next
    int corner;               // y0 * pitch + x0: pixel (i, j) of the frame is j * pitch + i - corner there
    int small_max;            // pixel centres of the largest triangle that one lane rasterises
    float aL, aR, aT, aB;
};

// Coverage test and z-test of pixel (i, j) against one set-up triangle; vis holds the window's pixels.
__device__ __forceinline__ void shade_pixel(const Setup& s, int i, int j, bool active, uint32_t id, u64* vis,
                                            const Window& win) {
    int px = (i << 8) + 128 - kOrigin, py = (j << 8) + 128 - kOrigin;
    int E0 = __mul24(s.dx0, py - s.Y1) - __mul24(s.dy0, px - s.X1);
    int E1 = __mul24(s.dx1, py - s.Y2) - __mul24(s.dy1, px - s.X2);
    int E2 = __mul24(s.dx2, py - s.Y0) - __mul24(s.dy2, px - s.X0);
    bool in = active && s.A2 != 0 && (((E0 + s.b0) | (E1 + s.b1) | (E2 + s.b2)) >= 0);
    if (in) {
        float e0 = (float)E0, e1 = (float)E1, e2 = (float)E2;
        float num = fmaf(e2, s.iw2, fmaf(e1, s.iw1, e0 * s.iw0));
        float depth = (float)s.A2 / num;
        u64 key = ((u64)__float_as_uint(depth) << 32) | (u64)id;
        atomicMin(&vis[__mul24(j - win.y0, win.pitch) + (i - win.x0)], key);   // 24-bit multiply: full rate
    }
}

// ---------------------------------------------------------------------------------------------
// Vertex transform, shared by the vertex phase and the clip path so both see identical bits.
struct Clip4 { float x, y, z, w; };

__device__ __forceinline__ Clip4 to_clip(const float (&M)[16], float x, float y, float z) {
    Clip4 c;
    c.x = fmaf(M[2], z, fmaf(M[1], y, fmaf(M[0], x, M[3])));
    c.y = fmaf(M[6], z, fmaf(M[5], y, fmaf(M[4], x, M[7])));
    c.z = fmaf(M[10], z, fmaf(M[9], y, fmaf(M[8], x, M[11])));
    c.w = fmaf(M[14], z, fmaf(M[13], y, fmaf(M[12], x, M[15])));
    return c;
}

// The same transform on the matrix cores, which the rest of the kernel leaves idle: v_mfma_f32_4x4x1 works on sixteen
// blocks of four lanes, and with the matrix's rows down the four lanes of a block as A, one coordinate per lane as B and
// the last column as C, lane l's four results are the clip coordinates of lane l's point.  One product and one sum per
// step, rounded once like fmaf: the same bits as to_clip but in what NaNs carry (a test compares them on five kinds of
// numbers, denormals and infinities among them), in 3 instructions instead of 12.  With fmaf in its place in the vertex
// phase alone 4096 environments at 128x128 take 1917 to 1941 us instead of 1904, 1024 of 500 k triangles 199 to 201 instead
// of 197 to 199; with fmaf everywhere 1915 to 1924 and 198 to 201.
// It ignores which lanes are switched off, so it is only called where the whole wavefront is.
typedef float float4m __attribute__((ext_vector_type(4)));
struct ClipRows {
    float a0, a1, a2;      // row lane % 4 of the matrix: coefficients of x, y and z
    float4m last;          // the column that is added
};
__device__ __forceinline__ float4m mfma_4x4x1(float a, float b, float4m c) { return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ Clip4 to_clip(const ClipRows& R, float x, float y, float z) {
    const float4m c = mfma_4x4x1(R.a2, z, mfma_4x4x1(R.a1, y, mfma_4x4x1(R.a0, x, R.last)));
    return Clip4{c.x, c.y, c.z, c.w};
}

__device__ __forceinline__ float plane_dist(const Clip4& v, int k) {
    switch (k) {
    case 0: return v.w + v.x;
    case 1: return v.w - v.x;
    case 2: return v.w + v.y;
    case 3: return v.w - v.y;
    case 4: return v.z;
    default: return v.w - v.z;
    }
}

// x*0 is 0 for every finite x and NaN otherwise, so one fma chain tests all four coordinates.
__device__ __forceinline__ bool all_finite(const Clip4& c) {
    float t = fmaf(c.x, 0.0f, fmaf(c.y, 0.0f, fmaf(c.z, 0.0f, c.w * 0.0f)));
    return t == t;
}

__device__ __forceinline__ uint32_t outcode(const Clip4& c) {
    uint32_t oc = 0;
    oc |= !(c.w + c.x >= 0.0f) ? 1u : 0u;
    oc |= !(c.w - c.x >= 0.0f) ? 2u : 0u;
    oc |= !(c.w + c.y >= 0.0f) ? 4u : 0u;
    oc |= !(c.w - c.y >= 0.0f) ? 8u : 0u;
    oc |= !(c.z >= 0.0f) ? 16u : 0u;
    oc |= !(c.w - c.z >= 0.0f) ? 32u : 0u;
    if (!all_finite(c)) oc |= kInvalid;
    return oc;
}

// Round to the nearest 1/256 pixel (ties to even) and pack.  Adding 1.5 * 2^23 - kOrigin rounds to an
// integer in the addition itself and leaves X - kOrigin in the low 16 bits of the sum, for every
// coordinate that can be packed: 2 additions and a byte permute instead of the 8 instructions of two
// conversions, subtractions and a merge.
__device__ __forceinline__ uint32_t snap_xy(float fx, float fy) {
    constexpr float magic = 12582912.0f - (float)kOrigin;
    static_assert(kOrigin % 2 == 0, "ties go to even coordinates");
    return __builtin_amdgcn_perm(__float_as_uint(fy + magic), __float_as_uint(fx + magic), 0x05040100u);
}

// Perspective divide + snap.  Returns false when the vertex cannot be placed on the sub-pixel grid
// of the frame (the numeric rule then drops its triangle).  can_project tells whether the vertex is
// in front of the eye with finite screen coordinates; such a vertex outside the frame is packed
// with its coordinates clamped to the 16-bit range, which keeps it on its side of the frame.
__device__ __forceinline__ bool project(const Clip4& c, const FrameParams& fp, uint32_t& xy, float& iw,
                                        bool& can_project) {
    iw = recip(c.w);
    float xn = c.x * iw, yn = c.y * iw;
    float fx = fmaf(xn, fp.sx, fp.sx), fy = fmaf(yn, fp.sy, fp.sy);
    bool ok = (c.w > 0.0f) && fx >= -64.0f && fx <= fp.xmax && fy >= -64.0f && fy <= fp.ymax;
    can_project = (c.w > 0.0f) && fabsf(fx) < 3.0e38f && fabsf(fy) < 3.0e38f;
    const float lowest = (float)(kOrigin - 32768), highest = (float)(kOrigin + 32767);
    xy = snap_xy(__builtin_amdgcn_fmed3f(fx, lowest, highest), __builtin_amdgcn_fmed3f(fy, lowest, highest));
    return ok;
}

constexpr int kMaxPoly = 16;   // a triangle cut by six planes has at most 9 corners; rounding can add a few

}  // namespace dev
}  // namespace bps
