// Fused geometry + rasterisation kernel for gfx950.  See raster_kernels.h for the plan.
//
// Numeric rule implemented here (the paper, Sec. 3.2, leaves it to the graphics API):
//   clip = M v by nested fma; planes w+x, w-x, w+y, w-y, z, w-z >= 0; Sutherland-Hodgman in the
//   order near, far, left, right, top, bottom with crossings interpolated from the inside vertex;
//   X = rint(fma(x/w, 128 W, 128 W)) in 1/256 px; integer edge functions with the top-left rule;
//   depth = A2 / (e0/w0 + e1/w1 + e2/w2); per pixel the minimum of (depth bits << 32 | id).
#include "raster_device.h"
#include "raster_kernels.h"

namespace bps {
namespace {

using namespace dev;

// ---------------------------------------------------------------------------------------------
// Per-wave state kept in LDS.
struct WaveLds {
    float2* stage;      // [64] staged vertices of the current cluster: (packed xy bits, 1/w)
    uint32_t* stage_oc; // [64] their outcodes
    uint32_t* smallq;   // [8][64] struct-of-arrays: xy0 xy1 xy2 iw0 iw1 iw2 id box
    uint32_t* tally;    // diagnostics (wave-private registers, dead code in the production instances): see kT*
};
// diagnostics tallies
enum { kTSmall = 0, kTLarge = 1, kTDrains = 2, kTDrainIters = 3, kTDrainDepth = 4, kTEmits = 5, kTMedPasses = 6, kTLargeSteps = 7,
       kTPushes = 8, kTClipDrains = 9, kTClipPasses = 10, kTFanIters = 11, kTPopPasses = 12, kTSlots = 13, kTClusters = 14,
       kTPhaseAPasses = 15, kTCount = 16 };

// One lane per queued small triangle: at most win.small_max pixel centres each.
__device__ __forceinline__ void drain_small(const WaveLds& L, int n, int lane, u64* vis, const Window& win,
                                            const BPS_GLOBAL uint32_t* ctri_id) {
    bool have = lane < n;
    // the queue holds the triangle's slot in the cluster arrays; its id is fetched here, one
    // gather per 64 triangles, and arrives while the edge set-up is computed
    const uint32_t ref = have ? L.smallq[6 * 64 + lane] : 0u;
    const uint32_t id = ctri_id[ref];
    uint32_t xy0 = L.smallq[0 * 64 + lane], xy1 = L.smallq[1 * 64 + lane], xy2 = L.smallq[2 * 64 + lane];
    float iw0 = __uint_as_float(L.smallq[3 * 64 + lane]), iw1 = __uint_as_float(L.smallq[4 * 64 + lane]),
          iw2 = __uint_as_float(L.smallq[5 * 64 + lane]);
    const uint32_t box = L.smallq[7 * 64 + lane];
    const PackedSetup s = make_packed_setup(xy0, xy1, xy2, iw0, iw1, iw2);
    const int i_lo = (int)(box & 0xFFu), j_lo = (int)((box >> 8) & 0xFFu);
    const int nx = (int)((box >> 16) & 0xFFu), ny = (int)(box >> 24);
    int cnt = (have && s.A2 != 0) ? nx * ny : 0;
    asm volatile("" : "+v"(cnt));      // one compare per step below, not the conjunction it came from
    // Edge functions at the first pixel centre, then stepped: one pixel to the right changes edge k by
    // -256 dy_k, and going from the end of a row to the start of the next by 256 dx_k + 256 (nx - 1) dy_k.
    // Same integers as evaluating each pixel afresh (all of them are areas inside the triangle's box);
    // the third one is what the other two leave of A2.
    int E0, E1, E2;
    packed_edges(s, pack_xy((i_lo << 8) + 128, (j_lo << 8) + 128), E0, E1, E2);
    const int dy0 = unpack_y(s.e0), dy1 = unpack_y(s.e1);
    const int right0 = -(dy0 << 8), right1 = -(dy1 << 8);
    const int wrap0 = (unpack_x(s.e0) + __mul24(nx - 1, dy0)) << 8, wrap1 = (unpack_x(s.e1) + __mul24(nx - 1, dy1)) << 8;
    int at = __mul24(j_lo, win.pitch) + i_lo - win.corner, col = 0;
    const int at_wrap = win.pitch - nx + 1;
    const float a2f = (float)s.A2;
    ++L.tally[kTDrains];
    for (int k = 0; k < win.small_max; ++k) {
        const bool act = k < cnt;
        if (ballot64(act) == 0) break;
        ++L.tally[kTDrainIters];
        const bool in = act & (E0 >= s.t0) & (E1 >= s.t1) & (E2 >= s.t2);
        if (ballot64(in) != 0ull) ++L.tally[kTDrainDepth];
        if (in) {
            const float num = fmaf((float)E2, s.iw2, fmaf((float)E1, s.iw1, (float)E0 * s.iw0));
            const float depth = div_in_range(a2f, num);
            atomicMin(&vis[at], ((u64)__float_as_uint(depth) << 32) | (u64)id);
        }
        const bool row_end = ++col == nx;
        E0 += row_end ? wrap0 : right0;
        E1 += row_end ? wrap1 : right1;
        E2 = s.A2 - E0 - E1;
        at += row_end ? at_wrap : 1;
        col = row_end ? 0 : col;
    }
    // The ids have arrived by now in all but the rarest drains (no pixel covered at all).  Without a use on every
    // path the compiler waits for them where their register is next written, in the triangle phase, and with them
    // for the next cluster's words, which are behind them in the order of return.
    asm volatile("" :: "v"(id));
}

// The lane's bit of a mask as a condition (no instruction: conditions are masks).
__device__ __forceinline__ bool in_mask(u64 mask) { return __builtin_amdgcn_inverse_ballot_w64(mask); }

// Append small triangles to the wave's queue; whenever it reaches 64 entries, drain them.
__device__ __forceinline__ void push_small(const WaveLds& L, int& count, uint32_t xy0, uint32_t xy1,
                                           uint32_t xy2, float iw0, float iw1, float iw2, uint32_t ref, uint32_t box,
                                           int lane, u64* vis, const Window& win,
                                           const BPS_GLOBAL uint32_t* ctri_id, u64 mask) {
    // mask = the lanes that want (callers build it from ballots of single comparisons,
    // which cost one compare each, instead of a ballot of the combined condition)
    if (__builtin_expect(mask == 0, 0)) return;
    int n = __popcll(mask);
    L.tally[kTSmall] += (uint32_t)n;
    ++L.tally[kTPushes];
    const int rank = (int)rank_below(mask);
    int pos = count + rank;            // position if the queue were unbounded
    auto put = [&]() {
        L.smallq[0 * 64 + pos] = xy0; L.smallq[1 * 64 + pos] = xy1; L.smallq[2 * 64 + pos] = xy2;
        L.smallq[3 * 64 + pos] = __float_as_uint(iw0); L.smallq[4 * 64 + pos] = __float_as_uint(iw1);
        L.smallq[5 * 64 + pos] = __float_as_uint(iw2);
        L.smallq[6 * 64 + pos] = ref; L.smallq[7 * 64 + pos] = box;
    };
    if (__builtin_expect(count + n < 64, 1)) {
        if (in_mask(mask)) put();
        count += n;
        return;
    }
    const u64 first = mask & ballot64(pos < 64);
    if (in_mask(first)) put();
    wave_lds_sync();
    drain_small(L, 64, lane, vis, win, ctri_id);
    wave_lds_sync();
    pos -= 64;
    if (in_mask(mask & ~first)) put();
    count += n - 64;
}

// Whole wavefront on one large triangle: 8x8 pixel blocks over its bounding box.
__device__ __forceinline__ void raster_large(uint32_t xy0, uint32_t xy1, uint32_t xy2, float iw0, float iw1, float iw2,
                                             uint32_t id, int i_lo, int i_hi, int j_lo, int j_hi, int lane, u64* vis,
                                             const Window& win, uint32_t* tally) {
    Setup s = make_setup(xy0, xy1, xy2, iw0, iw1, iw2);
    int li = lane & 7, lj = lane >> 3;
    for (int by = j_lo >> 3; by <= (j_hi >> 3); ++by) {
        int j = (by << 3) + lj;
        bool jok = j >= j_lo && j <= j_hi;
        for (int bx = i_lo >> 3; bx <= (i_hi >> 3); ++bx) {
            int i = (bx << 3) + li;
            bool act = jok && i >= i_lo && i <= i_hi;
            ++tally[kTLargeSteps];
            shade_pixel(s, i, j, act, id, vis, win);
        }
    }
}

// The same on packed coordinates (for triangles that the small and medium paths could take but for their size): tiles
// of 8x8 pixels from the box's first one on, which are fewer than those of a fixed grid (4 instead of 5.6 on average for
// a box of 12x12), edge functions stepped from tile to tile, and the short division.  Coarse meshes and larger frames
// are bound by this: 512 environments of 30 k triangles 131 -> 113 us per request, 1000 at 128x128 of 100 k 628 -> 543,
// 192 textured at 128x128 243 -> 222, 61 at 72x104 65.5 -> 61.5; 1024 of 500 k triangles 236.8 -> 236.1.
// One triangle per lane of `big` is set up, at the cost of setting up one; the wavefront then draws one after the other,
// handing round what the loop over its tiles needs (11 words instead of 8, and no products of its own): 1000 at 128x128
// of 100 k triangles 550 -> 531 us, 512 of 30 k 115 -> 110, 192 textured at 128x128 223 -> 219, 4096 at 128x128 of 500 k
// 2227 -> 2200.  What bounds a tile is the chain of its instructions, scalar ones and waits between the units among
// them: here and for medium triangles one comparison of a sign bit decides instead of five combined by the scalar unit,
// and which 4x4 pixels of the medium ones are entered is known once per pass.  192 textured at 128x128 218 -> 209 us, 61
// at 72x104 56.9 -> 54.7, 4096 at 128x128 1994 -> 1963, 512 106.0 -> 104.5.
__device__ __forceinline__ void raster_large_packed(uint32_t xy0, uint32_t xy1, uint32_t xy2, float iw0, float iw1, float iw2,
                                                    uint32_t id, uint32_t box, u64 big, int lane, u64* vis, const Window& win, uint32_t* tally) {
    const PackedSetup s = make_packed_setup(xy0, xy1, xy2, iw0, iw1, iw2);
    int first0, first1, unused;      // edge functions at the box's first pixel
    packed_edges(s, pack_xy((int)((box & 0xFFu) << 8) + 128, (int)(((box >> 8) & 0xFFu) << 8) + 128), first0, first1, unused);
    const int inside = s.t0 | (s.t1 << 1) | (s.t2 << 2);
    const int li = lane & 7, lj = lane >> 3;
    big &= ballot64(s.A2 != 0);
    while (big) {
        const int src = __builtin_ctzll(big);
        big &= big - 1;
        const uint32_t b = (uint32_t)bcast_i((int)box, src);
        // (in vector registers from here on: the scalar unit would wait for each of them)
        uint32_t e0 = (uint32_t)bcast_i((int)s.e0, src), e1 = (uint32_t)bcast_i((int)s.e1, src), at0 = b;
        int A2 = bcast_i(s.A2, src), t = bcast_i(inside, src);
        const float w0 = bcast_f(s.iw0, src), w1 = bcast_f(s.iw1, src), w2 = bcast_f(s.iw2, src);
        const uint32_t tri = (uint32_t)bcast_i((int)id, src);
        asm volatile("" : "+v"(e0), "+v"(e1), "+v"(A2), "+v"(t), "+v"(at0));
        const float a2f = (float)A2;
        const int dx0 = unpack_x(e0), dy0 = unpack_y(e0), dx1 = unpack_x(e1), dy1 = unpack_y(e1);
        // sign bits tell what is inside: of an edge (E0 >= t0, E1 >= t1, and E2 >= t2 with E2 = A2 - E0 - E1), of the box
        int E0 = bcast_i(first0, src) + ((__mul24(dx0, lj) - __mul24(dy0, li)) << 8);
        int E1 = bcast_i(first1, src) + ((__mul24(dx1, lj) - __mul24(dy1, li)) << 8);
        const int t0 = t & 1, t1 = (t >> 1) & 1, most = A2 - (t >> 2);
        const int nx = (int)((b >> 16) & 0xFFu), ny = (int)(b >> 24);
        int row = __mul24((int)((at0 >> 8) & 0xFFu) + lj, win.pitch) + ((int)(at0 & 0xFFu) + li) - win.corner;
        const int right0 = dy0 << 11, right1 = dy1 << 11, down0 = dx0 << 11, down1 = dx1 << 11;
        int in_rows = lj - ny;
        for (int y = 0; y < ny; y += 8) {
            int F0 = E0, F1 = E1, at = row, in_columns = li - nx;
            for (int x = 0; x < nx; x += 8) {
                ++tally[kTLargeSteps];
                const int outside = (F0 - t0) | (F1 - t1) | (most - F0 - F1);
                if ((~outside & in_rows & in_columns) < 0) {
                    const float num = fmaf((float)(A2 - F0 - F1), w2, fmaf((float)F1, w1, (float)F0 * w0));
                    atomicMin(&vis[at], ((u64)__float_as_uint(div_in_range(a2f, num)) << 32) | (u64)tri);
                }
                F0 -= right0;
                F1 -= right1;
                at += 8;
                in_columns += 8;
            }
            E0 += down0;
            E1 += down1;
            row += 8 * win.pitch;
            in_rows += 8;
        }
    }
}

// Pixel centres inside a triangle's bounding box, both axes at once with packed 16-bit
// arithmetic.  Pixel i has its centre at 256 (i - 64) + 128 in packed coordinates, so the first
// centre at or right of x is (x + 127) >> 8 and the last centre at or left of x is (x - 128) >> 8
// (both minus 64).  Returns false when the box, clamped to the work-group's window of the frame,
// holds no centre; otherwise lo = first pixel - 64 and ext = last - first per axis.
// The sign bits of `wide` tell that the whole box is more than 16 bits wide or high.
__device__ __forceinline__ bool centre_box(uint32_t xy0, uint32_t xy1, uint32_t xy2, const Window& win, short2v& lo,
                                           short2v& ext, uint32_t& wide) {
    short2v a = as_s2(xy0), b = as_s2(xy1), c = as_s2(xy2);
    short2v mn = __builtin_elementwise_min(a, __builtin_elementwise_min(b, c));
    short2v mx = __builtin_elementwise_max(a, __builtin_elementwise_max(b, c));
    wide = as_u32(mx - mn);
    lo = (mn + (short)127) >> (short)8;
    short2v hi = (mx - (short)128) >> (short)8;
    short2v lo_clamp = {(short)(win.x0 - 64), (short)(win.y0 - 64)};
    short2v hi_clamp = {(short)(win.x0 + win.w - 65), (short)(win.y0 + win.h - 65)};
    lo = __builtin_elementwise_max(lo, lo_clamp);
    hi = __builtin_elementwise_min(hi, hi_clamp);
    ext = hi - lo;                              // both halves >= 0: some pixel centre is inside
    return (as_u32(ext) & 0x80008000u) == 0;
}

// Classification and hand-off of one candidate triangle per lane whose box holds a pixel centre.
// ref = cluster * 128 + slot addresses the triangle's original id in ctri_id; small triangles
// carry it through the queue, only large ones look the id up here.
template <int FRAME>
__device__ __forceinline__ void emit(const WaveLds& L, int& small_count, short2v lo, short2v ext, uint32_t wide,
                                     bool tame,
                                     uint32_t xy0, uint32_t xy1, uint32_t xy2, float iw0, float iw1, float iw2,
                                     uint32_t ref, const BPS_GLOBAL uint32_t* ctri_id, int lane, u64* vis,
                                     const Window& win, u64 vmask) {
    // vmask = the lanes that have one
    // first pixel and size per axis as four bytes: i | j << 8 | nx << 16 | ny << 24
    const uint32_t first = as_u32(lo + (short)64), size = as_u32(ext + (short)1);
    const uint32_t box = __builtin_amdgcn_perm(size, first, 0x06040200u);
    const bool few = __mul24((int)(size & 0xFFFFu), (int)(size >> 16)) <= win.small_max;
    const bool within8 = (as_u32(ext) & 0xFFF8FFF8u) == 0u;
    // The small and medium paths compute on packed 16-bit differences and divide in a narrowed exponent
    // range: triangles with a vertex outside that range, or wider than 16 bits hold, are drawn as large ones.
    // (all the comparisons stand before the first branch: what the scalar unit reads of them it then waits for once)
    const u64 few_mask = ballot64(few), narrow_mask = FRAME == 64 ? ~0ull : ballot64((wide & 0x80008000u) == 0u);
    if (vmask == 0) return;
    ++L.tally[kTEmits];
    const u64 packed_mask = !tame ? 0ull : vmask & narrow_mask;
    const u64 small_mask = packed_mask & few_mask;
    push_small(L, small_count, xy0, xy1, xy2, iw0, iw1, iw2, ref, box, lane, vis, win, ctri_id, small_mask);
    u64 med = packed_mask & ~small_mask & ballot64(within8);
    u64 big = vmask & ~small_mask & ~med;
    L.tally[kTLarge] += (uint32_t)__popcll(med | big);
    // (the three expectations here keep what only larger triangles need out of the registers of the usual way: 1024 of
    // 64x64 of 500 k triangles 237.0 -> 233.5 us, 4096 at 128x128 2221 -> 2197)
    if (__builtin_expect((med | big) == 0ull, 1)) return;
    uint32_t id = 0u;
    if (in_mask(med | big)) id = ctri_id[ref];
    // medium triangles (box within 8x8 pixels): four per pass, sixteen lanes each, 4x4 pixels per step
    while (med) {
        ++L.tally[kTMedPasses];
        uint32_t four = 0u;     // the lanes of the next four, a byte each, and 64 where there are no more
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            four |= (med ? (uint32_t)__builtin_ctzll(med) : 64u) << (8 * k);
            med &= med - 1;     // 0 & anything stays 0
        }
        int which = lane;
        asm volatile("" : "+v"(which));      // (what follows from it would be kept, and spilled, over the kernel)
        const int f = (int)((four >> ((which >> 1) & 24)) & 0xFFu);      // (permutes take it modulo 64)
        const bool on = f < 64;
        const uint32_t mxy0 = (uint32_t)__shfl((int)xy0, f, 64), mxy1 = (uint32_t)__shfl((int)xy1, f, 64),
                       mxy2 = (uint32_t)__shfl((int)xy2, f, 64);
        const float miw0 = __shfl(iw0, f, 64), miw1 = __shfl(iw1, f, 64), miw2 = __shfl(iw2, f, 64);
        const uint32_t mid = (uint32_t)__shfl((int)id, f, 64), mbox = (uint32_t)__shfl((int)box, f, 64);
        const PackedSetup st = make_packed_setup(mxy0, mxy1, mxy2, miw0, miw1, miw2);
        const float a2f = (float)st.A2;
        const int mi = (int)(mbox & 0xFFu), mj = (int)((mbox >> 8) & 0xFFu);
        const int mnx = on && st.A2 != 0 ? (int)((mbox >> 16) & 0xFFu) : 0, mny = (int)(mbox >> 24);
        const int li = lane & 3, lj = (lane >> 2) & 3;
        // 4x4 pixels at the corner of the box, to the right of them, below, and beside; sign bits as in raster_large_packed
        const u64 wider = ballot64(mnx > 4), taller = ballot64(mnx != 0 && mny > 4);
        int E0, E1, E2;
        packed_edges(st, pack_xy(((mi + li) << 8) + 128, ((mj + lj) << 8) + 128), E0, E1, E2);
        const int most = st.A2 - st.t2, right0 = unpack_y(st.e0) << 10, right1 = unpack_y(st.e1) << 10;
        const int at = __mul24(mj + lj, win.pitch) + (mi + li) - win.corner;
        auto tile = [&](int F0, int F1, int in_columns, int in_rows, int where) {
            const int outside = (F0 - st.t0) | (F1 - st.t1) | (most - F0 - F1);
            if ((~outside & in_rows & in_columns) < 0) {
                const float num = fmaf((float)(st.A2 - F0 - F1), st.iw2, fmaf((float)F1, st.iw1, (float)F0 * st.iw0));
                atomicMin(&vis[where], ((u64)__float_as_uint(div_in_range(a2f, num)) << 32) | (u64)mid);
            }
        };
        tile(E0, E1, li - mnx, lj - mny, at);
        if (wider != 0ull) tile(E0 - right0, E1 - right1, li + 4 - mnx, lj - mny, at + 4);
        if (taller != 0ull) {
            E0 += unpack_x(st.e0) << 10;
            E1 += unpack_x(st.e1) << 10;
            tile(E0, E1, li - mnx, lj + 4 - mny, at + 4 * win.pitch);
            if (wider != 0ull) tile(E0 - right0, E1 - right1, li + 4 - mnx, lj + 4 - mny, at + 4 * win.pitch + 4);
        }
    }
    u64 general = big & ~packed_mask;
    big &= packed_mask;
    while (__builtin_expect(general != 0ull, 0)) {
        int src = __builtin_ctzll(general);
        general &= general - 1;
        const uint32_t bbox = (uint32_t)bcast_i((int)box, src);
        const int bi = (int)(bbox & 0xFFu), bj = (int)((bbox >> 8) & 0xFFu);
        raster_large((uint32_t)bcast_i((int)xy0, src), (uint32_t)bcast_i((int)xy1, src), (uint32_t)bcast_i((int)xy2, src),
                     bcast_f(iw0, src), bcast_f(iw1, src), bcast_f(iw2, src), (uint32_t)bcast_i((int)id, src), bi,
                     bi + (int)((bbox >> 16) & 0xFFu) - 1, bj, bj + (int)(bbox >> 24) - 1, lane, vis, win, L.tally);
    }
    if (__builtin_expect(big != 0ull, 0)) raster_large_packed(xy0, xy1, xy2, iw0, iw1, iw2, id, box, big, lane, vis, win, L.tally);
    asm volatile("" :: "v"(id));      // (as at the end of drain_small)
}

// Conservative test of an axis-aligned box against the planes that bound the work-group's window
// of the frame, in world space: near z >= 0, far w - z >= 0 and the four side planes
// x - aL w >= 0, aR w - x >= 0, y - aT w >= 0, aB w - y >= 0 (aL = -1, aR = +1 for a whole frame,
// i.e. w + x >= 0 and w - x >= 0).  For each plane the largest value over the box is compared with a
// negative margin proportional to the magnitude of the terms, so that rounding in this test and
// in the per-vertex transform can never cull a box holding a vertex the exact rule keeps; window
// edges lie half a pixel outside the outermost pixel centres, far more than vertex snapping moves
// anything.  NaNs compare false and therefore never cull.
//
// With p a plane, q the magnitudes of the terms its coefficients are made of, c the box's centre and e its half
// extents, largest value plus margin is
//   (p_w + eps q_w) + sum p_a c_a + sum (|p_a| + eps q_a) e_a + sum (eps q_a) |c_a|,
// ten products with one row of coefficients per plane: a chain of ten 4x4x1 matrix instructions gives one box per lane
// against four planes (see ClipRows), two chains against all of them.  Rows sit in LDS, [8][12], rows 6 and 7 repeat 4 and 5.
constexpr int kPlaneRow = 12;

// Window `tile` of a frame.  Its edges are rounded by a few units in the last place, which is nothing beside the half
// pixel that they lie outside of the pixel centres.
__device__ __forceinline__ void place_window(Window& win, uint32_t tile, const FrameParams& fp) {
    const int ty = (int)((tile * fp.tiles_x_recip) >> 16), tx = (int)tile - ty * fp.tiles_x;
    win.x0 = tx * fp.tile_w;
    win.y0 = ty * fp.tile_h;
    win.w = min(fp.tile_w, fp.W - win.x0);
    win.h = min(fp.tile_h, fp.H - win.y0);
    win.aL = (float)win.x0 * fp.two_per_w - 1.0f;
    win.aR = (float)(win.x0 + win.w) * fp.two_per_w - 1.0f;
    win.aT = (float)win.y0 * fp.two_per_h - 1.0f;
    win.aB = (float)(win.y0 + win.h) * fp.two_per_h - 1.0f;
}
__device__ __forceinline__ void fill_planes(float* rows, const float (&M)[16], const Window& win, int row) {
    const float eps = 1.52587890625e-05f;   // 2^-16
    const int k = row < 6 ? row : row - 2;
    // (row_r - a row_3) for the low side, (a row_3 - row_r) for the high side; near = row_2, far = row_3 - row_2
    const float a = k == 0 ? win.aL : k == 1 ? win.aR : k == 2 ? win.aT : k == 3 ? win.aB : k == 4 ? 0.0f : 1.0f;
    const float sg = (k == 1 || k == 3 || k == 5) ? -1.0f : 1.0f, aa = fabsf(a);
    float* o = rows + kPlaneRow * row;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        float r0 = M[t], r1 = M[4 + t], r2 = M[8 + t];
        asm("" : "+s"(r0), "+s"(r1), "+s"(r2));      // (or the choice becomes one of addresses, and M an array in private memory)
        const float r = k >= 4 ? r2 : k >= 2 ? r1 : r0;
        const float p = sg * (r - a * M[12 + t]), q = eps * (fabsf(r) + aa * fabsf(M[12 + t]));
        if (t == 3) {
            o[9] = p + q;
        } else {
            o[t] = p;
            o[3 + t] = fabsf(p) + q;
            o[6 + t] = q;
        }
    }
}
// (the whole wavefront calls it, see ClipRows)
__device__ __forceinline__ bool box_outside_frustum(const float* rows, int lane, float lx, float ly, float lz, float hx, float hy,
                                                    float hz) {
    // (an offset the compiler does not know: known addresses would each be kept, and spilled, over the kernel)
    int at = kPlaneRow * (lane & 3);
    asm volatile("" : "+v"(at));
    const float4m* row = reinterpret_cast<const float4m*>(rows + at);
    const float tx = 0.5f * lx, ty = 0.5f * ly, tz = 0.5f * lz;
    const float cx = fmaf(0.5f, hx, tx), cy = fmaf(0.5f, hy, ty), cz = fmaf(0.5f, hz, tz);
    const float ex = fmaf(0.5f, hx, -tx), ey = fmaf(0.5f, hy, -ty), ez = fmaf(0.5f, hz, -tz);
    float4m d[2];
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        const float4m r0 = row[g * kPlaneRow], r1 = row[g * kPlaneRow + 1], r2 = row[g * kPlaneRow + 2];
        float4m v = mfma_4x4x1(r2.y, 1.0f, float4m{0.0f, 0.0f, 0.0f, 0.0f});
        v = mfma_4x4x1(r0.x, cx, v); v = mfma_4x4x1(r0.y, cy, v); v = mfma_4x4x1(r0.z, cz, v);
        v = mfma_4x4x1(r0.w, ex, v); v = mfma_4x4x1(r1.x, ey, v); v = mfma_4x4x1(r1.y, ez, v);
        v = mfma_4x4x1(r1.z, fabsf(cx), v); v = mfma_4x4x1(r1.w, fabsf(cy), v); v = mfma_4x4x1(r2.x, fabsf(cz), v);
        d[g] = v;
    }
    // negative and finite: an overflow on the way tells nothing
    const float least = fminf(fminf(fminf(d[0].x, d[0].y), fminf(d[0].z, d[0].w)), fminf(d[1].x, d[1].y));
    constexpr int kNegativeFinite = 0x18;
    return __builtin_amdgcn_classf(least, kNegativeFinite);
}

// Inclusive prefix sum over the wavefront, by lane permutes of the vector unit (no trips to LDS).
__device__ __forceinline__ uint32_t wave_prefix_sum(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);      // rows of 16: 1, 2, 4, 8 lanes to the right
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);      // last lane of a row to the next row
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);      // lane 31 to the upper half
    return v;
}

// Where the entries of each of kDepthBins bins start when the bins' counts are laid end to end: lane k holds bins 2 k
// (low half) and 2 k + 1.  Every wavefront works that out for itself, which saves the barrier that one of them handing
// it round would need.
__device__ __forceinline__ uint32_t bin_starts(const uint32_t* hist, int lane, uint32_t& total) {
    static_assert(kDepthBins == 128, "two bins to a lane");
    const uint32_t h0 = hist[2 * lane], h1 = hist[2 * lane + 1], incl = wave_prefix_sum(h0 + h1), before = incl - (h0 + h1);
    total = (uint32_t)bcast_i((int)incl, 63);
    return before | ((before + h0) << 16);
}
__device__ __forceinline__ uint32_t start_of_bin(uint32_t starts, uint32_t bin) {      // (the whole wavefront calls it)
    return ((uint32_t)__shfl((int)starts, (int)(bin >> 1), 64) >> (16u * (bin & 1u))) & 0xFFFFu;
}

constexpr uint32_t kNoCluster = 0xFFFFFFFFu;
constexpr uint32_t kNoPixel = 0xFFFFFFFFu;   // box_footprint: the box cannot cover any pixel centre

// Screen footprint and nearest possible depth of a box, for the occlusion test made when the
// cluster is popped.  Every triangle inside the box rasterises with a depth that is a convex
// combination of clip w values attained inside the box, onto pixels inside the projection of the
// box.  So if the smallest w over the box (minus a rounding margin) is larger than the depth
// already stored at every pixel whose centre the projected box can reach, nothing in the box can
// win the z-test.  Returns the packed test record, or 0 when no bound can be given (the box
// may reach the eye plane, clip w is far from 1, or the box is more than 32 pixels wide or high):
//   bit 0 testable | x0 6 bits | y0 6 bits (both relative to the window) | width-1 5 bits |
//   height-1 5 bits, and in wbits18 the exponent and top ten mantissa bits of the w bound
//   (truncated, i.e. rounded towards the eye)
// The eight corners are transformed like vertices (fourteen matrix instructions, the whole wavefront calls it).
__device__ __forceinline__ uint32_t box_footprint(const ClipRows& R, const float (&M)[16], const FrameParams& fp, const Window& win,
                                                 float lx, float ly, float lz, float hx, float hy, float hz,
                                                 uint32_t& wbits18) {
    const float eps = 1.52587890625e-05f;   // 2^-16
    wbits18 = 0u;
    float ax = fmaxf(fabsf(lx), fabsf(hx)), ay = fmaxf(fabsf(ly), fabsf(hy)), az = fmaxf(fabsf(lz), fabsf(hz));
    float4m corner[8];
    {
        const float4m x0 = mfma_4x4x1(R.a0, lx, R.last), x1 = mfma_4x4x1(R.a0, hx, R.last);
        const float4m y0 = mfma_4x4x1(R.a1, ly, x0), y1 = mfma_4x4x1(R.a1, ly, x1), y2 = mfma_4x4x1(R.a1, hy, x0), y3 = mfma_4x4x1(R.a1, hy, x1);
        corner[0] = mfma_4x4x1(R.a2, lz, y0); corner[1] = mfma_4x4x1(R.a2, lz, y1); corner[2] = mfma_4x4x1(R.a2, lz, y2);
        corner[3] = mfma_4x4x1(R.a2, lz, y3); corner[4] = mfma_4x4x1(R.a2, hz, y0); corner[5] = mfma_4x4x1(R.a2, hz, y1);
        corner[6] = mfma_4x4x1(R.a2, hz, y2); corner[7] = mfma_4x4x1(R.a2, hz, y3);
    }
    float wmin = corner[0].w;
#pragma unroll
    for (int k = 1; k < 8; ++k) wmin = fminf(wmin, corner[k].w);
    float wmag = fmaf(fabsf(M[12]), ax, fmaf(fabsf(M[13]), ay, fmaf(fabsf(M[14]), az, fabsf(M[15]))));
    float wcons = wmin - eps * wmag;
    // (outside this range A2 / (e0/w0 + e1/w1 + e2/w2) can overflow or lose its precision, and a depth need no longer
    // be a mean of clip w values)
    const bool bound = wcons > 0x1p-60f && wmag < 0x1p100f;
    float x0 = 3.0e38f, x1 = -3.0e38f, y0 = 3.0e38f, y1 = -3.0e38f;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const float rw = __builtin_amdgcn_rcpf(corner[k].w);   // approximate is fine: slack follows (and no corner is nearer than wcons)
        const float sx = corner[k].x * rw, sy = corner[k].y * rw;
        x0 = fminf(x0, sx); x1 = fmaxf(x1, sx);
        y0 = fminf(y0, sy); y1 = fmaxf(y1, sy);
    }
    // pixels whose centres (i + 0.5) lie inside the projected box, with 1/64 pixel of slack for
    // vertex snapping (1/512 px) and rounding; none at all means nothing in the box can cover a centre
    const float hw = 0.5f * (float)fp.W, hh = 0.5f * (float)fp.H, slack = 0.015625f;
    float fx0 = ceilf(fmaf(x0, hw, hw) - 0.5f - slack), fx1 = floorf(fmaf(x1, hw, hw) - 0.5f + slack);
    float fy0 = ceilf(fmaf(y0, hh, hh) - 0.5f - slack), fy1 = floorf(fmaf(y1, hh, hh) - 0.5f + slack);
    if (!(bound && fx0 == fx0 && fx1 == fx1 && fy0 == fy0 && fy1 == fy1)) return 0u;   // NaN somewhere: no bound
    fx0 = fmaxf(fx0, (float)win.x0); fy0 = fmaxf(fy0, (float)win.y0);
    fx1 = fminf(fx1, (float)(win.x0 + win.w - 1)); fy1 = fminf(fy1, (float)(win.y0 + win.h - 1));
    if (fx0 > fx1 || fy0 > fy1) return kNoPixel;
    int ix0 = (int)fx0, ix1 = (int)fx1, iy0 = (int)fy0, iy1 = (int)fy1;
    int bw = ix1 - ix0, bh = iy1 - iy0;
    if (bw > 31 || bh > 31) return 0u;
    wbits18 = __float_as_uint(wcons) >> 13;      // positive: the sign bit is clear, 18 bits remain
    return 1u | ((uint32_t)(ix0 - win.x0) << 1) | ((uint32_t)(iy0 - win.y0) << 7) | ((uint32_t)bw << 13) | ((uint32_t)bh << 18);
}

// Survivor record, laid out for the vector unit to take apart (every lane does, see pop_visible):
//   low word   cluster 23 bits | footprint's width-1 5 bits | its height-1, low 4 bits
//   high word  height-1, top bit | more than one pass of 64 pixels 1 bit | first pixel: x 6 bits, y 6 bits | w bound 18 bits
// A cluster without a footprint to test has the pixel 0 and a w bound of 0, which nothing stored is nearer than.
__device__ __forceinline__ u64 make_record(uint32_t cluster, uint32_t foot, uint32_t wbits18) {
    if (!(foot & 1u)) return (u64)cluster;
    const uint32_t first = (foot >> 1) & 0xFFFu, bw = (foot >> 13) & 31u, bh = (foot >> 18) & 31u;
    const uint32_t many = (bh << (32 - __clz((int)bw))) > 63u ? 1u : 0u;      // rows of a power of two of pixels, see there
    return ((u64)((bh >> 4) | (many << 1) | (first << 2) | (wbits18 << 14)) << 32) | (u64)(cluster | (bw << 23) | (bh << 28));
}

// Depth bin of a survivor record: exponent and top three mantissa bits of its w bound, i.e.
// eight bins per octave from 2^-7 upwards; records without a bound (near or large boxes) go first.
__device__ __forceinline__ int depth_bin(u64 e) {
    int k = (int)(e >> 53) - 120 * 8;     // exponent and three mantissa bits of the w bound
    return min(max(k, 0), kDepthBins - 1);
}

// The clip ring is shared by the work-group: with one ring a clipper pass of 64 triangles comes up
// eight times sooner than with a queue per wavefront, and what waits for the clipper are the triangles
// along the window's border, without which no footprint touching a border pixel can be found hidden.
//   tail  entries reserved by producers (one LDS atomic per wavefront and push)
//   head  entries claimed by consumers
// An entry is written right after its reservation and reads kClipEmpty until then; the consumer of a
// claimed entry waits for it to turn up and puts kClipEmpty back.
constexpr uint32_t kClipEmpty = 0xFFFFFFFFu;      // no entry: cluster << 7 | slot stays below 2^30
struct ClipRing {
    uint32_t* slot;      // [mask + 1]
    uint32_t* tail;
    uint32_t* head;
    uint32_t mask;
};

// tail_seen: the ring's tail right after this wavefront's reservation
__device__ __forceinline__ void push_clip(const ClipRing& R, uint32_t ref, u64 mask, int lane, uint32_t& tail_seen) {
    if (mask == 0) return;
    const uint32_t count = (uint32_t)__popcll(mask);
    uint32_t pos = 0;
    if (lane == 0) pos = atomicAdd(R.tail, count);
    pos = __builtin_amdgcn_readfirstlane(pos);
    if (in_mask(mask)) R.slot[(pos + rank_below(mask)) & R.mask] = ref;
    tail_seen = pos + count;
}

// Claims up to 64 entries if at least `at_least` are waiting; returns how many (0: none) and hands
// lane k < n its entry.  head_seen, tail_seen: the ring's head and tail as last seen by this wavefront
// (the true head is never behind head_seen).
__device__ __forceinline__ int pop_clip(const ClipRing& R, uint32_t at_least, int lane, uint32_t& ref, uint32_t& head_seen,
                                        uint32_t& tail_seen) {
    uint32_t start = 0, n = 0, h = 0, t = 0;
    if (lane == 0) {
        h = __hip_atomic_load(R.head, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        for (;;) {
            t = __hip_atomic_load(R.tail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            const uint32_t waiting = t - h;
            if (waiting < at_least || waiting == 0u) break;
            const uint32_t take = min(waiting, 64u);
            const uint32_t seen = atomicCAS(R.head, h, h + take);
            if (seen == h) { start = h; n = take; h += take; break; }
            h = seen;
        }
    }
    start = __builtin_amdgcn_readfirstlane(start);
    n = __builtin_amdgcn_readfirstlane(n);
    head_seen = __builtin_amdgcn_readfirstlane(h);
    tail_seen = __builtin_amdgcn_readfirstlane(t);
    ref = kClipEmpty;
    if ((uint32_t)lane < n) {
        // The producer writes the entry right after reserving it and waits for nothing in between, so the
        // wait is a few cycles at most; it is bounded all the same, so that every wavefront leaves the
        // kernel whatever happens (a lane whose entry never turned up draws nothing).
        uint32_t* s = &R.slot[(start + (uint32_t)lane) & R.mask];
        for (int spin = 0; spin < (1 << 22); ++spin) {
            ref = __hip_atomic_load(s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (ref != kClipEmpty) break;
        }
        __hip_atomic_store(s, kClipEmpty, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    return (int)n;
}

// A copy of a uniform pointer: a pointer that is loaded with its neighbours is spilled, and comes back, with all of them.
template <class T>
__device__ __forceinline__ T* apart(T* p) {
    T* q;
    asm volatile("s_mov_b64 %0, %1" : "=s"(q) : "s"(p));
    return q;
}

struct ClusterData {      // of the scene: see SceneDev
    const BPS_GLOBAL float* verts;
    const BPS_GLOBAL uint32_t* tris;
    const BPS_GLOBAL uint32_t* tri_id;
};

// A straddling triangle per lane, clipped and projected: corners 0 .. cnt - 1.
struct Clipped {
    uint32_t ref;                            // cluster * 128 + slot
    int cnt;                                 // 0: nothing to draw
    uint32_t p0, p1, p2, p3, p4;             // packed positions
    float w0, w1, w2, w3, w4;                // 1/w
};

// Distance of a corner from the lane's plane: z, w - z, w + x, w - x, w + y or w - y.
struct LanePlane {
    bool x, y, negative, no_w;
    __device__ __forceinline__ float dist(const Clip4& q) const {
        float qx = q.x, qy = q.y, qz = q.z;
        asm("" : "+v"(qx), "+v"(qy), "+v"(qz));      // (or the choice becomes one of addresses, and q an object in private memory)
        const float v = x ? qx : y ? qy : qz;
        return fmaf(no_w ? 0.0f : 1.0f, q.w, negative ? -v : v);
    }
};

__device__ __forceinline__ Clip4 pick(bool first, const Clip4& p, const Clip4& q) {
    return Clip4{first ? p.x : q.x, first ? p.y : q.y, first ? p.z : q.z, first ? p.w : q.w};
}
__device__ __forceinline__ Clip4 along(const Clip4& a, const Clip4& b, float t) {      // from the inside corner a to b
    return Clip4{fmaf(t, b.x - a.x, a.x), fmaf(t, b.y - a.y, a.y), fmaf(t, b.z - a.z, a.z), fmaf(t, b.w - a.w, a.w)};
}

// One lane per queued straddling triangle: clip and project.  Triangles that cross one plane (nine in ten) or two
// are clipped in registers; three and more, and numbers outside the range of the short divisions, by the general
// clipper (clip_general), which few wavefronts of a finely tessellated scene enter.  The general clipper alone kept its
// polygons in private memory (a trip to L2 per corner) and met every crossing and every corner in a branch of its own: 10 %
// of the kernel's vector instructions, and the longest wait at the end of a round.  61 frames of 72x104: 71.5 -> 67.5 us per
// request, 256 of 64x64: 108.5 -> 104.5, 4096 of 128x128: 2410 -> 2365; 1024 of 64x64 unchanged.
// general: 0, or 64 and the planes that the lane's triangle crosses (bit k: the k-th of the rule's order), if that takes the
// general clipper.
__device__ __forceinline__ void clip_triangles(uint32_t* tally, uint32_t ref, bool have, const ClusterData& sc, const ClipRows& R,
                                               const FrameParams& fp, Clipped& out, uint32_t& general) {
    if (!have) ref = 0u;
    out.ref = ref;
    const uint32_t c = ref >> 7;
    const uint32_t t = sc.tris[ref] & 0x00FFFFFFu;
    const BPS_GLOBAL float* cv = sc.verts + (size_t)c * 192;
    float p[3][3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const uint32_t vi = (t >> (8 * k)) & 0xFFu;
        p[k][0] = cv[vi]; p[k][1] = cv[64 + vi]; p[k][2] = cv[128 + vi];
    }
    // (all nine loads on their way before the first is waited for)
    asm volatile("" : "+v"(p[0][0]), "+v"(p[0][1]), "+v"(p[0][2]), "+v"(p[1][0]), "+v"(p[1][1]), "+v"(p[1][2]), "+v"(p[2][0]), "+v"(p[2][1]),
                 "+v"(p[2][2]));
    Clip4 tri[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) tri[k] = to_clip(R, p[k][0], p[k][1], p[k][2]);
    ++tally[kTClipDrains];
    // ---- which planes the triangle crosses, in the rule's order near, far, left, right, top, bottom
    auto outside = [&](auto test) -> bool { return test(tri[0]) | test(tri[1]) | test(tri[2]); };
    const bool cross[6] = {outside([](const Clip4& q) { return !(q.z >= 0.0f); }),  outside([](const Clip4& q) { return !(q.z <= q.w); }),
                           outside([](const Clip4& q) { return !(q.x >= -q.w); }), outside([](const Clip4& q) { return !(q.x <= q.w); }),
                           outside([](const Clip4& q) { return !(q.y >= -q.w); }), outside([](const Clip4& q) { return !(q.y <= q.w); })};
    bool one = false, two = false, more = false;      // lanes with at least that many planes
    bool f[6], g[6];                                  // the lane's first and second plane
    general = 64u;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        general |= cross[k] ? 1u << k : 0u;
        f[k] = cross[k] & !one;
        g[k] = cross[k] & one & !two;
        more = more | (cross[k] & two);
        two = two | (cross[k] & one);
        one = one | cross[k];
    }
    auto usable = [](float num, float den) -> bool { return iw_in_range(den) & ((num == 0.0f) | iw_in_range(num)); };
    bool fits = have & one & !more;
    // ---- first plane: the vertex S on its own side, P before it and N after it leave the corners X1 (between P and
    // S), X2 (between S and N) and either S or N and P.  The general clipper takes the edges c-a, a-b, b-c in turn,
    // a crossing first and then the edge's end if that is inside: that decides where the polygon starts.
    const LanePlane first{bool(f[2] | f[3]), bool(f[4] | f[5]), bool(f[1] | f[3] | f[5]), f[0]};
    const float da = first.dist(tri[0]), db = first.dist(tri[1]), dc = first.dist(tri[2]);
    const bool ia = da >= 0.0f, ib = db >= 0.0f, ic = dc >= 0.0f;
    const bool is_a = ib == ic, is_c = !is_a & (ia == ib), is_b = !is_a & !is_c;
    Clip4 Q0, Q1, Q2, Q3;
    int m;
    {
        const Clip4 S = pick(is_a, tri[0], pick(is_b, tri[1], tri[2])), P = pick(is_a, tri[2], pick(is_b, tri[0], tri[1])),
                    N = pick(is_a, tri[1], pick(is_b, tri[2], tri[0]));
        const float dS = is_a ? da : is_b ? db : dc, dP = is_a ? dc : is_b ? da : db, dN = is_a ? db : is_b ? dc : da;
        const bool s_in = is_a ? ia : is_b ? ib : ic;
        const float n1 = s_in ? dS : dP, d1 = n1 - (s_in ? dP : dS), n2 = s_in ? dS : dN, d2 = n2 - (s_in ? dN : dS);
        fits = fits & usable(n1, d1) & usable(n2, d2);
        const Clip4 X1 = along(pick(s_in, S, P), pick(s_in, P, S), div_in_range(n1, d1));
        const Clip4 X2 = along(pick(s_in, S, N), pick(s_in, N, S), div_in_range(n2, d2));
        const Clip4 A = pick(s_in, S, N);
        Q0 = pick(is_c, X2, pick(is_b & !s_in, P, X1));
        Q1 = pick((is_c & s_in) | (is_b & !s_in), X1, pick(is_a & !s_in, X2, A));
        Q2 = pick((is_c & s_in) | (is_a & !s_in), A, pick(is_c & !s_in, P, X2));
        Q3 = pick(s_in, Q2, pick(is_a, P, pick(is_b, A, X1)));      // three corners: the last one twice
        m = s_in ? 3 : 4;
    }
    auto snapped = [&](const Clip4& q, uint32_t& xy, float& iw) -> bool {
        iw = recip_normal(q.w);
        const float fx = fmaf(q.x * iw, fp.sx, fp.sx), fy = fmaf(q.y * iw, fp.sy, fp.sy);
        xy = snap_xy(fx, fy);
        // well inside what the numeric rule accepts
        return iw_in_range(iw) & (fabsf(fx - fp.sx) <= fp.sx + 32.0f) & (fabsf(fy - fp.sy) <= fp.sy + 32.0f);
    };
    ++tally[kTClipPasses];
    if (ballot64(have & two & fits) == 0ull) {
        fits = fits & snapped(Q0, out.p0, out.w0);
        fits = fits & snapped(Q1, out.p1, out.w1);
        fits = fits & snapped(Q2, out.p2, out.w2);
        fits = fits & snapped(Q3, out.p3, out.w3);
        out.p4 = out.p3;
        out.w4 = out.w3;
        out.cnt = m;
    } else {
        // ---- second plane: the same rule over the three or four corners; lanes without one keep every corner
        ++tally[kTClipPasses];
        const LanePlane second{bool(g[2] | g[3]), bool(g[4] | g[5]), bool(g[1] | g[3] | g[5]), g[0]};
        const Clip4 Q[4] = {Q0, Q1, Q2, Q3};
        float d[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) d[k] = two ? second.dist(Q[k]) : 1.0f;
        int at = 0, turns = 0;
        out.p0 = out.p1 = out.p2 = out.p3 = out.p4 = 0u;
        out.w0 = out.w1 = out.w2 = out.w3 = out.w4 = 0.0f;
        auto put = [&](bool want, uint32_t xy, float iw) {
            out.p0 = (want & (at == 0)) ? xy : out.p0; out.w0 = (want & (at == 0)) ? iw : out.w0;
            out.p1 = (want & (at == 1)) ? xy : out.p1; out.w1 = (want & (at == 1)) ? iw : out.w1;
            out.p2 = (want & (at == 2)) ? xy : out.p2; out.w2 = (want & (at == 2)) ? iw : out.w2;
            out.p3 = (want & (at == 3)) ? xy : out.p3; out.w3 = (want & (at == 3)) ? iw : out.w3;
            out.p4 = (want & (at == 4)) ? xy : out.p4; out.w4 = (want & (at == 4)) ? iw : out.w4;
            at += want ? 1 : 0;
        };
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int before = (k + 3) & 3;      // (three corners: the fourth repeats the third)
            const bool in = d[k] >= 0.0f, in_before = d[before] >= 0.0f, turn = in != in_before, keep = in & (k < m);
            const float num = in ? d[k] : d[before], den = num - (in ? d[before] : d[k]);
            uint32_t xy;
            float iw;
            bool ok = snapped(along(pick(in, Q[k], Q[before]), pick(in, Q[before], Q[k]), div_in_range(num, den)), xy, iw);
            fits = fits & (!turn | (ok & usable(num, den)));
            put(turn, xy, iw);
            ok = snapped(Q[k], xy, iw);
            fits = fits & (!keep | ok);
            put(keep, xy, iw);
            turns += turn ? 1 : 0;
        }
        fits = fits & (turns <= 2);
        out.cnt = at;
    }
    if (!fits) out.cnt = 0;
    general = have & !fits ? general : 0u;
}

// The general clipper: the first 64 / wide of the triangles in `waiting` (a bit per lane that holds one, with `ref` and
// `general` of clip_triangles), `wide` lanes each: 16, which is as many corners as the rule keeps of a polygon, or 8, and what
// turns out to have more is put into `again`.  A lane holds a corner and the one before it; at a plane it puts out the
// crossing between the two, then the corner, and its place among what the row puts out is a count of bits, so that a plane
// takes one trip through LDS (x and y, then z and w, where the staged vertices are between clusters) however many corners
// there are.  Lane j of a row then holds the piece (0, j, j + 1) of the polygon: returns whether there is one.
// What bounds it is the chain of steps of one wavefront where few triangles come here, and vector issue where many do, so
// polygons stay out of private memory (where all 64 triangles of a clipper's run fit) and out of one lane's loop over its
// corners (of which LDS holds three at a time: several planes crossed by most triangles cost up to 4 times the request).
// Us per request, private memory / three at a time / rows of 16 only / this: 16 environments in a room of 500 triangles
// 34.9 / 37.4 / 27.6 / 25.4, 200 of them at 24x24 40.1 / 45.7 / 31.1 / 29.1; among 2000 triangles as large as the room
// 1024 environments 2270 / 2580 / 2030 / 2000 and one 67 / 277 / 98 / 67; one among 20000 of them 230 / - / - / 248.
__device__ __forceinline__ bool clip_general(const WaveLds& L, int wide, u64& waiting, u64& again, uint32_t ref, uint32_t general,
                                             const ClusterData& sc, const ClipRows& R, const FrameParams& fp, int lane, uint32_t& of,
                                             uint32_t& p0, uint32_t& p1, uint32_t& p2, float& w0, float& w1, float& w2) {
    static_assert(kMaxPoly == 16, "a corner per lane of the widest row");
    asm volatile("" : "+v"(lane));      // (what follows from it is worked out here and not kept, and spilled, over the kernel)
    const int j = lane & (wide - 1), row = lane - j;
    const uint32_t row_mask = (1u << wide) - 1u;
    const uint32_t rank = rank_below(waiting) * (uint32_t)wide;      // the lane's own triangle: the row that takes it
    const u64 taken = waiting & ballot64(rank < 64u);
    wave_lds_sync();
    if (in_mask(taken)) L.stage[rank] = make_float2(__uint_as_float(ref), __uint_as_float(general));
    wave_lds_sync();
    const bool on = row < __popcll(waiting) * wide;
    waiting &= ~taken;
    const float2 mine = L.stage[row];
    of = on ? __float_as_uint(mine.x) : 0u;
    uint32_t todo = on ? __float_as_uint(mine.y) & 63u : 0u;
    int n = on ? 3 : 0;
    const uint32_t t = sc.tris[of] & 0x00FFFFFFu, vi = (t >> (8 * min(j, 2))) & 0xFFu;
    const BPS_GLOBAL float* cv = sc.verts + (size_t)(of >> 7) * 192;
    Clip4 v = to_clip(R, cv[vi], cv[64 + vi], cv[128 + vi]), u;
    {
        const int before = row + (j == 0 ? 2 : j - 1);
        u = Clip4{__shfl(v.x, before, 64), __shfl(v.y, before, 64), __shfl(v.z, before, 64), __shfl(v.w, before, 64)};
    }
    u64 large = 0ull;      // rows whose polygon has become too large for them
    for (;;) {
        const u64 open = ballot64(todo != 0u) & ballot64(n >= 3);
        if (open == 0ull) break;
        ++L.tally[kTClipPasses];
        const uint32_t p = (uint32_t)__builtin_ctz(todo | 64u);      // near, far, left, right, top, bottom
        auto dist = [&](float x, float y, float z, float w) -> float {      // z, w - z, w + x, w - x, w + y or w - y
            const float s = p < 2u ? z : p < 4u ? x : y;
            return (p == 0u ? 0.0f : w) + ((p & 1u) ? -s : s);
        };
        const float dv = dist(v.x, v.y, v.z, v.w), du = dist(u.x, u.y, u.z, u.w);
        const bool in = dv >= 0.0f;
        const u64 inside = ballot64(in), there = open & ballot64(j < n);
        const u64 keeps = there & inside, turns = there & (inside ^ ballot64(du >= 0.0f));
        // (a crossing is taken from the inside corner to the outside one; u - v is v - u but for its sign)
        const float da = in ? dv : du, part = da / (da - (in ? du : dv)), towards = in ? part : -part;
        const Clip4 x = {fmaf(towards, u.x - v.x, in ? v.x : u.x), fmaf(towards, u.y - v.y, in ? v.y : u.y), fmaf(towards, u.z - v.z, in ? v.z : u.z),
                         fmaf(towards, u.w - v.w, in ? v.w : u.w)};
        const uint32_t row_keeps = (uint32_t)(keeps >> row) & row_mask, row_turns = (uint32_t)(turns >> row) & row_mask;
        const uint32_t below = (1u << j) - 1u;
        const int at = __popc(row_keeps & below) + __popc(row_turns & below);
        int m = __popc(row_keeps) + __popc(row_turns);
        const int at_v = at + (in_mask(turns) ? 1 : 0);
        const bool put_x = in_mask(turns) & (at < wide), put_v = in_mask(keeps) & (at_v < wide);
        if (wide < kMaxPoly) {
            const u64 more = open & ballot64(m > wide);
            large |= more;
            m = in_mask(more) ? 0 : m;
        }
        m = min(m, kMaxPoly);
        const int before = row + (j == 0 ? max(m - 1, 0) : j - 1);
        float2* const out = L.stage + row;
        wave_lds_sync();
        if (put_x) out[at] = make_float2(x.x, x.y);
        if (put_v) out[at_v] = make_float2(v.x, v.y);
        wave_lds_sync();
        const float2 v_xy = L.stage[lane], u_xy = L.stage[before];
        wave_lds_sync();
        if (put_x) out[at] = make_float2(x.z, x.w);
        if (put_v) out[at_v] = make_float2(v.z, v.w);
        wave_lds_sync();
        const float2 v_zw = L.stage[lane], u_zw = L.stage[before];
        if (in_mask(open)) {
            v = Clip4{v_xy.x, v_xy.y, v_zw.x, v_zw.y};
            u = Clip4{u_xy.x, u_xy.y, u_zw.x, u_zw.y};
            n = m;
            todo &= todo - 1u;
        }
    }
    bool unused;
    const bool ok = project(v, fp, p1, w1, unused);
    const u64 dropped = ballot64(j < n) & ~ballot64(ok);      // one corner without a place drops the triangle
    wave_lds_sync();
    L.stage[lane] = make_float2(__uint_as_float(p1), w1);
    wave_lds_sync();
    const float2 first = L.stage[row], next = L.stage[row + min(j + 1, wide - 1)];
    p0 = __float_as_uint(first.x); w0 = first.y;
    p2 = __float_as_uint(next.x); w2 = next.y;
    again |= taken & ballot64(((large >> (rank & 63u)) & 1ull) != 0ull);
    return ((uint32_t)(dropped >> row) & row_mask) == 0u && j >= 1 && j + 1 < n;
}

// Clips up to 64 queued triangles and hands the pieces (0, k, k + 1) of their polygons to emit(): the k-th ones of all that
// were clipped in registers together, then all the pieces of eight of the others at a time.
template <int FRAME>
__device__ __forceinline__ void draw_clipped(const WaveLds& L, uint32_t ref, int n, int& small_count, const ClusterData& sc,
                                             const ClipRows& R, const FrameParams& fp, const Window& win, int lane, u64* vis) {
    Clipped cl;
    uint32_t general;
    clip_triangles(L.tally, ref, lane < n && ref != kClipEmpty, sc, R, fp, cl, general);
    u64 waiting = ballot64(general != 0u), again = 0ull;
    int wide = 8;
#pragma unroll 1
    for (int k = 0;; ++k) {
        bool live = k + 2 < cl.cnt, tame = true;
        uint32_t of = cl.ref, a = cl.p0, b = cl.p1, d = cl.p2;
        float wa = cl.w0, wb = cl.w1, wd = cl.w2;
        if (__builtin_expect(ballot64(live) != 0ull, 1)) {
            // the next piece's corners
            cl.p1 = cl.p2; cl.p2 = cl.p3; cl.p3 = cl.p4;
            cl.w1 = cl.w2; cl.w2 = cl.w3; cl.w3 = cl.w4;
        } else {
            if (__builtin_expect((waiting | again) == 0ull, 1)) break;
            if (waiting == 0ull) {
                waiting = again;
                again = 0ull;
                wide = kMaxPoly;
            }
            live = clip_general(L, wide, waiting, again, cl.ref, general, sc, R, fp, lane, of, a, b, d, wa, wb, wd);
            tame = ballot64(live && !(iw_in_range(wa) && iw_in_range(wb) && iw_in_range(wd))) == 0ull;
        }
        ++L.tally[kTFanIters];
        short2v lo, ext;
        uint32_t wide;
        const bool has = live && centre_box(a, b, d, win, lo, ext, wide);
        emit<FRAME>(L, small_count, lo, ext, wide, tame, a, b, d, wa, wb, wd, of, sc.tri_id, lane, vis, win, ballot64(has));
    }
}

}  // namespace

// =============================================================================================
// What bounds it: vector-ALU issue while the device is full, and the latency of one work-group at the
// end of a launch; HBM is at a seventh of its rate.  So the steps that every cluster, triangle or pixel
// goes through are kept short: exact reciprocals and quotients in 3 and 6 instructions (recip_normal,
// div_in_range), snapping by the rounding of one addition (snap_xy), set-up on packed 16-bit
// coordinates (PackedSetup), and no outcodes, range tests or clamps for clusters wholly inside the frustum.
// 1024 environments of 500 k triangles at 64x64: 104.0 M -> 82.5 M vector instructions per launch, request
// 274 -> 251 us; 4096 at 128x128 (1 M triangles): 2.70 -> 2.54 ms.  Of what remains a wavefront waits 40 % of its
// time, most of it on LDS round trips: clusters come off the list ahead of their use, no load is left in flight that
// only one path uses, and the planes of the box tests sit in LDS instead of registers (no vector register is spilled
// in the instances that draw by default, and 81 to 90 scalar ones): 78.8 M instructions, 238 us; 2.27 ms.  With clusters of
// smaller boxes and raster_large_packed: 238 -> 229 us; 2.29 -> 2.17 ms.  With transforms on the matrix cores (their share:
// see ClipRows), a shorter set-up, a draw loop without waits between the vector and the scalar unit, and one comparison per
// step: 75.7 M vector instructions, matrix ones included (the vector units issue in 80 % of the cycles in which a compute
// unit is busy, 82 % at 4096), 228 -> 199 us; 2.18 -> 1.90 ms.
template <int NT, bool DIAG, int CULL, int FRAME>
__global__ __launch_bounds__(NT, 4) void k_raster(const SceneDev* __restrict__ scenes, const WorkItem* __restrict__ items,
                                               const float* __restrict__ view_proj, FrameParams fp,
                                               unsigned long long* __restrict__ gvis, float* __restrict__ out_depth,
                                               uint32_t* __restrict__ out_id, unsigned long long* __restrict__ stats_block) {
    extern __shared__ __align__(16) unsigned char smem[];
    // The DIAG = false instance carries no counters or timers at all: everything below that feeds
    // only the diagnostics record is dead code there and costs neither registers nor instructions.
    unsigned long long* const stats = DIAG ? stats_block : nullptr;
    const bool phase_timers = DIAG && fp.phase_timers == 1;
    constexpr int NW = NT / 64;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // LDS is sized for a full tile; edge tiles may be smaller.  The 64x64 instance also fixes the
    // capacity of the survivor list, so that every LDS address below is a compile-time constant.
    // FRAME = 64 or 128: an instance for square frames of that size, drawn as 64x64 windows (the
    // paper's two resolutions).  The frame parameters the loops use are constants there.
    // FRAME = 1: any frame and any window of at most 64x64 pixels, with the same constant LDS layout.
    FrameParams fq = fp;
    if (FRAME > 1) {
        fq.H = FRAME; fq.W = FRAME; fq.tile_w = 64; fq.tile_h = 64;
        fq.sx = 128.0f * FRAME; fq.sy = 128.0f * FRAME; fq.xmax = 256.0f * FRAME + 64.0f; fq.ymax = 256.0f * FRAME + 64.0f;
    }
    const int HW = FRAME ? 64 * 64 : (fp.tile_w * fp.tile_h + 1) & ~1;      // (even: what follows is 16-byte aligned)
    const int list_cap = FRAME ? (int)kListCap64 : fp.list_cap;

    u64* vis = reinterpret_cast<u64*>(smem);
    unsigned char* wbase = smem + (size_t)HW * 8 + (size_t)wave * kWaveLdsBytes;
    uint32_t tally[kTCount] = {};
    WaveLds L;
    L.tally = tally;
    L.stage = reinterpret_cast<float2*>(wbase);
    L.stage_oc = reinterpret_cast<uint32_t*>(wbase + 64 * 8);
    L.smallq = reinterpret_cast<uint32_t*>(wbase + 64 * 12);

    unsigned char* shared = smem + (size_t)HW * 8 + (size_t)NW * kWaveLdsBytes;
    u64* list = reinterpret_cast<u64*>(shared);                                 // [list_cap] surviving clusters
    uint16_t* order = reinterpret_cast<uint16_t*>(shared + (size_t)list_cap * 8);   // [kOrderCap] blocks, near to far
    uint16_t* perm = reinterpret_cast<uint16_t*>(shared + (size_t)list_cap * 8 + kOrderCap * 2);   // [list_cap] pop order
    uint16_t* slot_in_bin = perm + list_cap;                                                       // [list_cap]
    uint32_t* hist = reinterpret_cast<uint32_t*>(slot_in_bin + list_cap);                          // [kDepthBins]
    uint32_t* hiz = hist + kDepthBins;                                                                // [kHizTiles]
    static_assert(kWaveLdsBytes % 16 == 0, "planes are read four words at a time (list capacities are multiples of 64)");
    float* planes = reinterpret_cast<float*>(hiz + kHizTiles);                                        // [8][kPlaneRow]
    uint32_t* counters = reinterpret_cast<uint32_t*>(planes + 8 * kPlaneRow);
    uint32_t* list_count = counters;       // survivors appended in this round
    uint32_t* pop_count = counters + 1;    // survivors handed out in this round
    uint32_t* next_block = counters + 2;   // blocks handed out so far (whole item)
    uint32_t* reserved = counters + 3;     // upper bound on list_count once every tester has appended
    ClipRing ring;
    ring.tail = counters + 5;
    ring.head = counters + 6;
    ring.slot = counters + 8;
    ring.mask = clip_ring_entries(NT) - 1u;

    const WorkItem item = items[blockIdx.x];     // the host or the planner has put the items in launch order
    // (field by field: the record is loaded sixteen registers at a time, and whatever of it were still needed later would be
    // spilled, and come back, with all the rest)
    SceneDev sc = scenes[item.scene];
    asm volatile("" : "+s"(sc.cverts), "+s"(sc.ctris), "+s"(sc.ctri_id), "+s"(sc.cbounds), "+s"(sc.bbounds), "+s"(sc.n_clusters), "+s"(sc.c_stride),
                 "+s"(sc.b_stride));
    float M[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) M[k] = view_proj[(size_t)item.env * 16 + k];
    ClipRows R;
    {
        const float* row = view_proj + (size_t)item.env * 16 + 4 * (lane & 3);
        R.a0 = row[0]; R.a1 = row[1]; R.a2 = row[2];
        R.last = float4m{M[3], M[7], M[11], M[15]};
    }

    // this work-group's window of the frame
    Window win;
    win.pitch = 64;
    win.small_max = DIAG ? fp.small_max : small_max(FRAME);
    if (FRAME == 64) {
        // the instance for 64x64 frames (the paper's main resolution): the window is the frame, and
        // with its origin and size known to the compiler the pixel arithmetic of every loop shrinks
        win.x0 = 0; win.y0 = 0; win.w = 64; win.h = 64;
        win.aL = -1.0f; win.aR = 1.0f; win.aT = -1.0f; win.aB = 1.0f;
    } else if (FRAME == 128) {
        // 128x128 frames: four windows of known size; only the origin depends on the item
        win.x0 = (int)(item.tile & 1u) * 64; win.y0 = (int)(item.tile >> 1) * 64; win.w = 64; win.h = 64;
        win.aL = (float)win.x0 * (1.0f / 64.0f) - 1.0f; win.aR = win.aL + 1.0f;
        win.aT = (float)win.y0 * (1.0f / 64.0f) - 1.0f; win.aB = win.aT + 1.0f;
    } else {
        place_window(win, item.tile, fp);
        if (FRAME == 0) win.pitch = win.w;
    }
    win.corner = __mul24(win.y0, win.pitch) + win.x0;
    const int nslots = win.h * win.pitch;      // (columns beyond the window's width are never looked at)
    int small_count = 0;
    uint32_t clip_tail_seen = 0u, clip_head_seen = 0u;    // this wavefront's last view of the clip ring
    // diagnostics (only when the host passes a counter block): per-wave tallies, one atomic each at the end
    uint32_t st_tested = 0, st_boxed = 0, st_drawn = 0, st_straddle = 0, st_hidden = 0, st_hiz = 0;
    const unsigned long long t_start = stats ? wall_clock64() : 0ull;
    // phase timers (diagnostics only): ticks[k] accumulates the time since the previous TICK
    unsigned long long t_prev = t_start;
    uint32_t ticks[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#define TICK(k) do { if (phase_timers) { unsigned long long t_ = wall_clock64(); ticks[k] += (uint32_t)(t_ - t_prev); t_prev = t_; } } while (0)
    const uint32_t full_tri_mask = 0x00FFFFFFu;
    const BPS_GLOBAL float* g_cverts = apart(gptr(sc.cverts));
    const BPS_GLOBAL uint32_t* g_ctris = apart(gptr(sc.ctris));
    const BPS_GLOBAL uint32_t* g_ctri_id = apart(gptr(sc.ctri_id));
    const BPS_GLOBAL float* g_bounds = gptr(sc.cbounds);
    const uint32_t S = item.split_of >> 16, item_split = item.split_of & 0xFFFFu;
    const uint32_t nblocks_total = (sc.n_clusters + 63u) / 64u;
    const uint32_t nb_item = nblocks_total > item_split ? (nblocks_total - item_split + S - 1u) / S : 0u;
    const BPS_GLOBAL float* g_bbounds = gptr(sc.bbounds);
    // CULL is the culling level the instance is compiled for: 0 none (every cluster of the scene is
    // streamed), 1 frustum tests only, 2 frustum and occlusion tests (the default)
    constexpr bool occlusion = CULL > 1;
    const uint32_t* vis_hi = reinterpret_cast<const uint32_t*>(vis) + 1;   // depth word of pixel p is vis_hi[2 p]

    // ---- prologue: LDS cleared, and the item's blocks ordered near to far
    // What bounds it is one wavefront's chain of steps.  Hence three barriers before the first round instead of five and
    // two in the depth sort instead of four, prefix sums by lane permutes, bounds fetched ahead, no divisions, a first block
    // per wavefront without a trip to the counters, and box tests on the matrix cores.  Together, us per request: 1
    // environment 25.9 -> 24.6, 16 in a small room 27.1 -> 25.7, 61 at 72x104 58.7 -> 56.8, 512 119.9 -> 117.1, 1024 of
    // 500 k triangles 230.2 -> 224.4, 4096 at 128x128 2220 -> 2180; this part of a group 2.0 -> 1.5 us of 10 (one
    // environment).  The box tests' own share does not show: as fmaf chains of the same ten terms they take the same
    // requests (1024: 197 and 199 us against 195 and 199, 4096: 1904 against 1895 and 1906).
    const bool sorted = CULL != 0 && nb_item <= kOrderCap && nb_item > 1;
    // A wavefront's part of the block order is a block per lane, and on with the next NT blocks; the bounds of the
    // first ones arrive while LDS is being cleared.
    constexpr int kOrderPasses = (kOrderCap + NT - 1) / NT;
    float blk_lo[3], blk_hi[3];
    auto fetch_block = [&](uint32_t b) {
        const uint32_t gb = min(b, nb_item - 1u) * S + item_split;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            blk_lo[a] = g_bbounds[(size_t)a * sc.b_stride + gb];
            blk_hi[a] = g_bbounds[(size_t)(a + 3) * sc.b_stride + gb];
        }
    };
    if (sorted && (uint32_t)wave * 64u < nb_item) fetch_block((uint32_t)tid);
    if (CULL != 0 && tid < 8) fill_planes(planes, M, win, tid);
    if (FRAME) {
#pragma unroll
        for (int p = 0; p < 64 * 64 / 2; p += NT) reinterpret_cast<ulong2*>(vis)[p + tid] = make_ulong2(kEmptyKey, kEmptyKey);
    } else {
        for (int p = tid; p < nslots; p += NT) vis[p] = kEmptyKey;
    }
    // (every wavefront begins with the block of its own number: see below)
    const bool own_first = (uint32_t)list_cap >= 64u * NW;
    if (tid < 8) counters[tid] = own_first ? (tid == 2 ? (uint32_t)NW : tid == 3 ? 64u * NW : 0u) : 0u;
    for (int t = tid; t < kHizTiles; t += NT) hiz[t] = 0xFFFFFFFFu;   // nothing drawn yet: no tile hides anything
#pragma unroll
    for (uint32_t t = 0; t < clip_ring_entries(NT); t += NT)
        if (clip_ring_entries(NT) % NT == 0u || t + (uint32_t)tid < clip_ring_entries(NT)) ring.slot[t + (uint32_t)tid] = kClipEmpty;
    // the bin counts of the two counting sorts below: zero whenever no sort is under way
    for (int t = tid; t < kDepthBins; t += NT) hist[t] = 0u;
    __syncthreads();
    uint32_t nb_visit = nb_item;
    if (sorted) {
        // Counting sort of the blocks in view on the smallest clip w over the block's bounding box
        // (exactly attained at a corner), in the logarithmic depth bins of the survivor sort: any order
        // is a correct one, near to far lets occluders come first.  Blocks wholly outside one frustum
        // plane get no place in the order and are never visited.
        uint32_t key[kOrderPasses];      // bin | place in the bin << 8, or all ones
#pragma unroll
        for (int q = 0; q < kOrderPasses; ++q) {
            key[q] = 0xFFFFFFFFu;
            const uint32_t base = (uint32_t)(wave * 64 + q * NT);
            if (base >= nb_item) continue;
            if (q > 0) fetch_block(base + (uint32_t)lane);
            float wmin = M[15];
#pragma unroll
            for (int a = 0; a < 3; ++a) wmin += fminf(M[12 + a] * blk_lo[a], M[12 + a] * blk_hi[a]);
            if (!box_outside_frustum(planes, lane, blk_lo[0], blk_lo[1], blk_lo[2], blk_hi[0], blk_hi[1], blk_hi[2]) &&
                base + (uint32_t)lane < nb_item) {
                // exponent and top three mantissa bits from 2^-7 upwards; boxes reaching the eye plane first
                const int k = wmin > 0.0f ? (int)(__float_as_uint(wmin) >> 20) - 120 * 8 : 0;
                const uint32_t bin = (uint32_t)min(max(k, 0), kDepthBins - 1);
                key[q] = bin | (atomicAdd(&hist[bin], 1u) << 8);
            }
        }
        __syncthreads();
        const uint32_t starts = bin_starts(hist, lane, nb_visit);
#pragma unroll
        for (int q = 0; q < kOrderPasses; ++q) {
            const uint32_t b = (uint32_t)(tid + q * NT);
            if (ballot64(key[q] != 0xFFFFFFFFu) == 0ull) continue;
            const uint32_t at = start_of_bin(starts, key[q] & 0x7Fu) + (key[q] >> 8);
            if (key[q] != 0xFFFFFFFFu) order[at] = (uint16_t)b;
        }
        __syncthreads();
        for (int t = tid; t < kDepthBins; t += NT) hist[t] = 0u;      // (used again after the next barrier)
    }

    // The item's clusters are the 64-cluster blocks split, split + S, ... of its scene, visited
    // near to far in rounds:
    //   phase A  wavefronts take blocks from the ordered list; every lane tests one cluster's
    //            bounds against the frustum and works out its screen footprint; survivors are
    //            appended (ballot + prefix count, one LDS atomic per wavefront) to the work-group's
    //            list until enough are queued or the list could overflow
    //   phase B  wavefronts pop clusters from the list one at a time; a cluster whose footprint
    //            pixels all hold nearer depths by then is skipped (one lane per footprint pixel)
    TICK(4);
    // the first round is kept short: what it draws (the nearest blocks) lets later rounds reject
    // hidden clusters before they are queued
    uint32_t round_target = occlusion ? min((uint32_t)fp.round_target, (uint32_t)fp.first_round) : (uint32_t)fp.round_target;
    const int htx = FRAME ? 8 : (win.w + 7) >> 3;     // Hi-Z tiles per row of the window
    bool later_round = false;             // something has been drawn: the depth buffer can reject
    // A wavefront's first block of a round is the one of its own number among those still waiting, which needs no trip to
    // the counters; what follows is handed out as wavefronts ask.
    uint32_t own = own_first ? (uint32_t)wave : kNoCluster;
    for (;;) {
        for (;;) {
            uint32_t blk = own;
            if (own == kNoCluster) {
                if (*list_count >= round_target) break;
                uint32_t r0 = 0;
                if (lane == 0) r0 = atomicAdd(reserved, 64u);
                r0 = __builtin_amdgcn_readfirstlane(r0);
                if (r0 + 64u > (uint32_t)list_cap) {
                    if (lane == 0) atomicSub(reserved, 64u);
                    break;
                }
                if (lane == 0) blk = atomicAdd(next_block, 1u);
                blk = __builtin_amdgcn_readfirstlane(blk);
            }
            own = kNoCluster;
            if (blk >= nb_visit) {
                if (lane == 0) atomicSub(reserved, 64u);
                break;
            }
            const uint32_t jb = sorted ? (uint32_t)order[blk] : blk;
            if (occlusion && sorted && jb == 0xFFFFu) {      // struck out: the whole block is hidden
                if (lane == 0) atomicSub(reserved, 64u);
                continue;
            }
            ++tally[kTPhaseAPasses];
            const uint32_t cl = (jb * S + item_split) * 64u + (uint32_t)lane;
            bool visible = cl < sc.n_clusters;
            uint32_t foot = 0u, wb18 = 0u;
            st_tested += (uint32_t)__popcll(ballot64(visible));
            if (CULL != 0) {
                const uint32_t cc = visible ? cl : 0u;
                float lx = g_bounds[cc], ly = g_bounds[sc.c_stride + cc], lz = g_bounds[2 * sc.c_stride + cc];
                float hx = g_bounds[3 * sc.c_stride + cc], hy = g_bounds[4 * sc.c_stride + cc],
                      hz = g_bounds[5 * sc.c_stride + cc];
                visible = visible & !box_outside_frustum(planes, lane, lx, ly, lz, hx, hy, hz);
                if (occlusion && ballot64(visible) != 0ull) {
                    foot = box_footprint(R, M, fq, win, lx, ly, lz, hx, hy, hz, wb18);
                    const bool in_view = visible;
                    visible = visible & (foot != kNoPixel);
                    if (visible && (foot & 1u)) {
                        // coarse test against the largest depth per 8x8 tile as of the end of the last round
                        const int fx = (int)((foot >> 1) & 63u), fy = (int)((foot >> 7) & 63u);     // window-relative
                        const int bw = (int)((foot >> 13) & 31u), bh = (int)((foot >> 18) & 31u);
                        if (bw <= 7 && bh <= 7) {     // at most 2 x 2 tiles: their corners are all of them
                            const int tx0 = fx >> 3, tx1 = (fx + bw) >> 3;
                            const int ty0 = fy >> 3, ty1 = (fy + bh) >> 3;
                            uint32_t zmax = max(max(hiz[ty0 * htx + tx0], hiz[ty0 * htx + tx1]),
                                                max(hiz[ty1 * htx + tx0], hiz[ty1 * htx + tx1]));
                            if ((wb18 << 13) > zmax) visible = false;
                        }
                        // Footprints of at most 4x4 pixels are then checked pixel by pixel, all 64 clusters
                        // at once (no wavefront is drawing during this phase): the same test a wavefront
                        // would make alone when it pops the cluster, at a fortieth of the cost.
                        const bool fine = visible && later_round && bw <= 3 && bh <= 3;
                        if (ballot64(fine) != 0ull) {
                            // one footprint row per step: its up to four depth words are read together
                            const uint32_t bound = wb18 << 13;
                            int at = __mul24(fy, win.pitch) + fx;
                            uint32_t farthest = 0u;
                            for (int row = 0; row < 4; ++row) {
                                const bool act = fine && row <= bh;
                                if (ballot64(act) == 0ull) break;
                                const uint32_t d0 = act ? vis_hi[2 * at] : 0u;
                                const uint32_t d1 = act && bw >= 1 ? vis_hi[2 * (at + 1)] : 0u;
                                const uint32_t d2 = act && bw >= 2 ? vis_hi[2 * (at + 2)] : 0u;
                                const uint32_t d3 = act && bw >= 3 ? vis_hi[2 * (at + 3)] : 0u;
                                farthest = max(farthest, max(max(d0, d1), max(d2, d3)));
                                at += win.pitch;
                            }
                            if (fine && farthest < bound) visible = false;
                        }
                    }
                    st_hiz += (uint32_t)__popcll(ballot64(in_view && !visible && foot != kNoPixel));
                }
            }
            const u64 keep = ballot64(visible);
            const uint32_t n_keep = (uint32_t)__popcll(keep);
            uint32_t base = 0;
            if (lane == 0) {
                base = atomicAdd(list_count, n_keep);
                atomicSub(reserved, 64u - n_keep);
            }
            base = __builtin_amdgcn_readfirstlane(base);
            if (visible) list[base + rank_below(keep)] = make_record(cl, foot, wb18);
        }
        TICK(1);
        __syncthreads();
        TICK(2);
        const uint32_t n_list = *list_count;
        // every block has been handed out: this is the last round (the same for all wavefronts:
        // next_block only moves during phase A)
        const bool last_round = *next_block >= nb_visit;
        st_boxed += wave == 0 ? n_list : 0u;

        // Order the round's survivors near to far (counting sort on a logarithmic depth key, eight
        // bins per octave) so that occluders are drawn before what they hide.
        const bool by_depth = occlusion && n_list > 64u;
        if (by_depth) {
            if (FRAME) {
                // the instances with a fixed list capacity put the records themselves in order (every thread
                // carries its few records over a barrier), so that taking a cluster off the list is one read
                constexpr int kPerThread = ((int)kListCap64 + NT - 1) / NT;
                u64 rec[kPerThread];
                uint32_t key[kPerThread];      // bin | place in the bin << 8
#pragma unroll
                for (int k = 0; k < kPerThread; ++k) {
                    const uint32_t i = (uint32_t)tid + (uint32_t)(k * NT);
                    key[k] = 0u;
                    if (i >= n_list) continue;
                    rec[k] = list[i];
                    const uint32_t bin = (uint32_t)depth_bin(rec[k]);
                    key[k] = bin | (atomicAdd(&hist[bin], 1u) << 8);
                }
                __syncthreads();
                uint32_t unused;
                const uint32_t starts = bin_starts(hist, lane, unused);
#pragma unroll
                for (int k = 0; k < kPerThread; ++k) {
                    const uint32_t i = (uint32_t)tid + (uint32_t)(k * NT), at = start_of_bin(starts, key[k] & 0x7Fu) + (key[k] >> 8);
                    if (i < n_list) list[at] = rec[k];
                }
            } else {
                for (uint32_t i = tid; i < n_list; i += NT)
                    slot_in_bin[i] = (uint16_t)atomicAdd(&hist[depth_bin(list[i])], 1u);
                __syncthreads();
                uint32_t unused;
                const uint32_t starts = bin_starts(hist, lane, unused);
                for (uint32_t base = (uint32_t)wave * 64u; base < n_list; base += NT) {
                    const uint32_t i = min(base + (uint32_t)lane, n_list - 1u), at = start_of_bin(starts, (uint32_t)depth_bin(list[i]));
                    perm[at + slot_in_bin[i]] = (uint16_t)i;      // (lanes past the end repeat the last entry)
                }
            }
            __syncthreads();
            for (int t = tid; t < kDepthBins; t += NT) hist[t] = 0u;      // (used again after further barriers)
            TICK(3);
        }

        // Clusters come off the list ahead of their use, so that fewer LDS round trips wait for one another: the next
        // place is drawn from the counter while a record is tested, and its record is read while the cluster that
        // passed is fetched and the one before it is drawn (three trips in a row took 400 cycles per record).  A
        // cluster whose footprint pixels all hold nearer depths by now cannot win anywhere and is dropped here (one
        // lane per footprint pixel); the words of the first that may win are fetched while the one before it is
        // processed.
        //
        // A record is taken apart by the vector unit, by all lanes alike: a scalar instruction that reads what a vector
        // one has written waits 16 to 20 cycles, one of the vector unit none.  The same holds for masks: comparisons stand
        // together, before the scalar instructions that combine them.  Done so here, in the vertex phase and in emit, 1024
        // environments of 500 k triangles take 209 us instead of 227, 4096 at 128x128 2046 instead of 2200, 512 109 instead
        // of 118, 256 84.4 instead of 91.0, one 23.6 instead of 25.1.
        uint32_t drawn = 0;      // lane 0: the place drawn last, in flight
        auto draw_place = [&]() {
            if (lane == 0) drawn = atomicAdd(pop_count, 1u);
        };
        draw_place();
        uint32_t pop = __builtin_amdgcn_readfirstlane(drawn);      // place of the record in flight
        auto read_record = [&]() -> u64 {
            // past the end: any record of the list, it is not looked at (the order has no entries there to follow)
            uint32_t at = pop;
            asm volatile("" : "+v"(at));
            if (by_depth && !FRAME) return list[perm[min(at, n_list - 1u)]];
            return list[min(at, (uint32_t)list_cap - 1u)];
        };
        u64 record = read_record();
        float nx_ = 0, ny_ = 0, nz_ = 0;
        uint32_t nt0 = 0, nt1 = 0, c_next = 0;
        bool found = false;
        auto pop_visible = [&]() {
            found = false;
            while (pop < n_list) {
                uint32_t lo32 = (uint32_t)record, hi32 = (uint32_t)(record >> 32);
                asm volatile("" : "+v"(lo32), "+v"(hi32));
                draw_place();
                const uint32_t bw = (lo32 >> 23) & 31u, bh = __builtin_amdgcn_alignbit(hi32, lo32, 28) & 31u;
                const uint32_t bound = (hi32 >> 14) << 13;
                // the wavefront covers the footprint in passes of 64 pixels: rows of 1, 2, 4, ... 32
                // pixels (the smallest power of two that holds the width), as many rows as fit; lanes
                // beyond its right or lower edge read the edge's pixel once more
                const uint32_t cols_log2 = 32u - (uint32_t)__clz((int)bw);
                const uint32_t qx = min(__builtin_amdgcn_ubfe((uint32_t)lane, 0u, cols_log2), bw), qy = (uint32_t)lane >> cols_log2;
                uint32_t corner;
                if (FRAME) corner = (hi32 >> 2) & 0xFFFu;
                else corner = __mul24((hi32 >> 8) & 63u, win.pitch) + ((hi32 >> 2) & 63u);
                corner += qx;
                ++tally[kTPopPasses];
                const uint32_t d = vis_hi[2u * (corner + __mul24(min(qy, bh), win.pitch))];
                u64 nearer = ballot64(d >= bound);
                pop = __builtin_amdgcn_readfirstlane(drawn);
                record = read_record();
                if (__builtin_expect(nearer == 0ull && ballot64((hi32 & 2u) != 0u) != 0ull, 0)) {
                    const uint32_t rows_per_pass = 64u >> cols_log2;
                    for (uint32_t row0 = rows_per_pass; nearer == 0ull && ballot64(row0 <= bh) != 0ull; row0 += rows_per_pass) {
                        ++tally[kTPopPasses];
                        nearer = ballot64(vis_hi[2u * (corner + __mul24(min(row0 + qy, bh), win.pitch))] >= bound);
                    }
                }
                if (nearer == 0ull) { ++st_hidden; continue; }
                c_next = lo32 & 0x007FFFFFu;
                const BPS_GLOBAL float* cv = g_cverts + (size_t)c_next * 192;
                nx_ = cv[lane]; ny_ = cv[64 + lane]; nz_ = cv[128 + lane];
                const BPS_GLOBAL uint32_t* ct = g_ctris + (size_t)c_next * 128;
                nt0 = ct[lane]; nt1 = ct[64 + lane];
                found = true;
                return;
            }
        };
        pop_visible();
        // Each turn takes either 64 triangles from the clip ring or the next cluster, so that the clipper and the
        // code that draws its pieces are inlined in one place (62 -> 40 KB of code; the instruction cache holds 64 KB
        // for two compute units).
        for (;;) {
            const bool streaming = found;
            // The ring is looked at while streaming only when this wavefront's own view says 64 may be waiting: its
            // view of the tail dates from its last push, its view of the head is never ahead of the head, so every
            // push that leaves 64 or more waiting is followed by a look.  When the list is used up, whatever waits is
            // taken: what the wavefront has queued goes into the depth buffer then, so that the depth tiles and the
            // next round's tests see everything this round drew (triangles waiting for the clipper are the ones
            // along the window's border: until they are drawn, no footprint that touches a border pixel can be
            // found hidden).  After the last round this overlaps the clusters that slower wavefronts still draw;
            // whatever they add to the ring, they take when they get here.
            if (streaming ? clip_tail_seen - clip_head_seen >= 64u : occlusion || last_round) {
                uint32_t clip_ref;
                const int n = pop_clip(ring, streaming ? 64u : 1u, lane, clip_ref, clip_head_seen, clip_tail_seen);
                if (n != 0) {
                    wave_lds_sync();
                    draw_clipped<FRAME>(L, clip_ref, n, small_count, ClusterData{g_cverts, g_ctris, g_ctri_id}, R, fq, win, lane, vis);
                    continue;
                }
            }
            if (!streaming) break;
            const uint32_t c = c_next;
            float x = nx_, y = ny_, z = nz_;
            uint32_t t0 = nt0, t1 = nt1;
            pop_visible();

            // ---- vertex phase
            const Clip4 cp = to_clip(R, x, y, z);
            ++tally[kTClusters];
            uint32_t xy, oc = 0;
            float iw = recip_normal(cp.w);
            // A vertex inside all planes with 1/w in the usual range is finite, projects, and lands within the
            // frame: no further test, no clamping.  Most clusters hold nothing else.  (The maximum is NaN if one of the three is.)
            const float most = __builtin_elementwise_maximum(__builtin_elementwise_maximum(fabsf(cp.x), fabsf(cp.y)), cp.z);
            const bool all_inside = (ballot64(most <= cp.w) & ballot64(cp.z >= 0.0f) & ballot64(iw_in_range(iw))) == ~0ull;
            if (!all_inside) {
                // outside of plane k; w + x >= 0 and x >= -w agree for all finite values (rounding keeps the sign of
                // a sum), and a vertex that is not finite drops its triangles whatever these say
                const u64 m0 = ballot64(!(cp.x >= -cp.w)), m1 = ballot64(!(cp.x <= cp.w)), m2 = ballot64(!(cp.y >= -cp.w));
                const u64 m3 = ballot64(!(cp.y <= cp.w)), m4 = ballot64(!(cp.z >= 0.0f)), m5 = ballot64(!(cp.z <= cp.w));
                if (m0 == ~0ull || m1 == ~0ull || m2 == ~0ull || m3 == ~0ull || m4 == ~0ull || m5 == ~0ull) continue;
            }
            ++st_drawn;
            bool tame = true;
            if (all_inside) {
                xy = snap_xy(fmaf(cp.x * iw, fq.sx, fq.sx), fmaf(cp.y * iw, fq.sy, fq.sy));
            } else {
                bool can_project;
                const bool ok = project(cp, fq, xy, iw, can_project);
                oc = outcode(cp);
                if (oc == 0 && !ok) oc = kInvalid;
                if (!can_project) oc |= kNoProject;
                tame = ballot64(can_project && !iw_in_range(iw)) == 0ull;
            }
            wave_lds_sync();   // earlier reads of the stage are done
            // the slot index is laundered so that its LDS address is recomputed here (one add) rather
            // than kept in a register across the whole loop, where it was spilled and its reload
            // made the wavefront wait for the cluster prefetch as well
            int stage_slot = lane;
            asm volatile("" : "+v"(stage_slot));
            L.stage[stage_slot] = make_float2(__uint_as_float(xy), iw);
            if (!all_inside) L.stage_oc[stage_slot] = oc;
            wave_lds_sync();

            // ---- triangle phase: two slots per lane
            // (slots past the cluster's last triangle hold its first vertex three times, which neither straddles nor has an area)
            const uint32_t word0 = __builtin_amdgcn_readfirstlane(t0);      // its top byte: slots in use
#pragma unroll 1
            for (int slot = 0; slot < 2; ++slot) {
                if (slot == 1 && word0 <= 0x40FFFFFFu) break;
                ++tally[kTSlots];
                uint32_t t = (slot == 0 ? t0 : t1) & full_tri_mask;
                const uint32_t i0 = t & 0xFFu, i1 = (t >> 8) & 0xFFu, i2 = t >> 16;
                float2 a = L.stage[i0], b = L.stage[i1], d = L.stage[i2];
                short2v lo, ext;
                uint32_t wide;
                const bool has = centre_box(__float_as_uint(a.x), __float_as_uint(b.x), __float_as_uint(d.x), win, lo, ext, wide);
                u64 drawable = ballot64(has);      // masks are combined on the scalar unit
                if (__builtin_expect(!all_inside, 0)) {
                    uint32_t oa = L.stage_oc[i0], ob = L.stage_oc[i1], od = L.stage_oc[i2];
                    uint32_t o_or = oa | ob | od, o_and = oa & ob & od;
                    const u64 live = ballot64((o_or & kInvalid) == 0) & ballot64((o_and & 0x3Fu) == 0);
                    const u64 crossing = ballot64((o_or & 0x3Fu) != 0), behind = ballot64((o_or & kNoProject) != 0);
                    // A straddler whose three vertices all project (w > 0) cannot reach a pixel centre
                    // outside the box of its projected vertices: only the others need the clipper.
                    const u64 straddling = live & crossing & (drawable | behind);
                    drawable &= live & ~crossing;
                    st_straddle += (uint32_t)__popcll(straddling);
                    push_clip(ring, (c << 7) | (uint32_t)(slot * 64 + lane), straddling, lane, clip_tail_seen);
                }
                emit<FRAME>(L, small_count, lo, ext, wide, tame, __float_as_uint(a.x), __float_as_uint(b.x),
                     __float_as_uint(d.x), a.y, b.y, d.y, c * 128u + (uint32_t)(slot * 64 + lane), g_ctri_id, lane, vis,
                     win, drawable);
            }
        }
        TICK(5);
        if ((occlusion || last_round) && small_count > 0) {
            wave_lds_sync();
            drain_small(L, small_count, lane, vis, win, g_ctri_id);
            wave_lds_sync();
            small_count = 0;
        }
        if (last_round) break;
        __syncthreads();
        const uint32_t waiting_from = *next_block;      // stable: it only moves during phase A
        if (tid == 0) { *list_count = 0u; *pop_count = 0u; *reserved = own_first ? 64u * NW : 0u; }
        if (own_first) own = waiting_from + (uint32_t)wave;
        if (occlusion) {   // (more blocks are waiting, or the loop would have ended above)
            // Whole blocks are tested against the new depth tiles as well: thread k takes the k-th block
            // still waiting.  Its bounds are fetched now and arrive while the tiles are being built.
            float blo[3] = {0.0f, 0.0f, 0.0f}, bhi[3] = {0.0f, 0.0f, 0.0f};
            uint32_t my_rank = waiting_from + (uint32_t)tid;
            bool my_block = sorted && my_rank < nb_visit && order[my_rank] != 0xFFFFu;
            if (my_block) {
                const uint32_t gb = (uint32_t)order[my_rank] * S + item_split;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    blo[a] = g_bbounds[(size_t)a * sc.b_stride + gb];
                    bhi[a] = g_bbounds[(size_t)(a + 3) * sc.b_stride + gb];
                }
            }
            // Hi-Z: largest stored depth word per 8x8-pixel tile of the window (empty pixels read as
            // 0xFFFFFFFF); one thread per tile row reads its eight words, eight neighbouring lanes hold the
            // rows of one tile (a 64x64 window is one pass of the 512 threads)
            const int hty = (win.h + 7) >> 3;
            for (int u = tid; u < htx * hty * 8; u += NT) {
                const int t = u >> 3, py = ((t / htx) << 3) + (u & 7), px0 = (t % htx) << 3;
                uint32_t dbits = 0u;
                if (py < win.h) {
                    const uint32_t* row = vis_hi + 2 * (__mul24(py, win.pitch) + px0);
#pragma unroll
                    for (int k = 0; k < 8; ++k) dbits = max(dbits, px0 + k < win.w ? row[2 * k] : 0u);
                }
#pragma unroll
                for (int sh = 4; sh >= 1; sh >>= 1) dbits = max(dbits, (uint32_t)__shfl_xor((int)dbits, sh, 64));
                if ((u & 7) == 0) hiz[t] = dbits;
            }
            __syncthreads();
            // A block whose box lies behind the largest depth of every tile its footprint touches hides
            // all of its clusters (their boxes are inside it; depths only ever decrease): its entry in
            // the visiting order is struck out and phase A passes over it.
            if (ballot64(my_block) != 0ull) {
                uint32_t wb18 = 0u;
                const uint32_t foot = box_footprint(R, M, fq, win, blo[0], blo[1], blo[2], bhi[0], bhi[1], bhi[2], wb18);
                bool dead = foot == kNoPixel;
                if (my_block && !dead && (foot & 1u)) {
                    const int fx = (int)((foot >> 1) & 63u), fy = (int)((foot >> 7) & 63u);
                    const int bw = (int)((foot >> 13) & 31u), bh = (int)((foot >> 18) & 31u);
                    uint32_t zmax = 0u;
                    for (int ty = fy >> 3; ty <= (fy + bh) >> 3; ++ty)
                        for (int tx = fx >> 3; tx <= (fx + bw) >> 3; ++tx) zmax = max(zmax, hiz[ty * htx + tx]);
                    dead = (wb18 << 13) > zmax;
                }
                if (my_block && dead) order[my_rank] = 0xFFFFu;
            }
        } else {
            __syncthreads();
        }
        if (own_first && tid == 0) *next_block = waiting_from + NW;
        round_target = (uint32_t)fp.round_target;
        later_round = true;
        __syncthreads();
        TICK(6);
    }
    TICK(7);
    if (stats) __syncthreads();   // the record below reuses the survivor list: every wavefront must be done with it
    // diagnostics: per-wave tallies go through LDS (the survivor list is free by now) and leave as
    // one record of 16 words per work-group, without atomics
    if (stats && lane == 0) {
        uint32_t* rec = reinterpret_cast<uint32_t*>(list) + wave * 16;
        const uint32_t dt = (uint32_t)(wall_clock64() - t_start);
        rec[0] = st_tested; rec[1] = st_boxed; rec[2] = st_drawn; rec[3] = st_straddle; rec[4] = st_hidden; rec[5] = dt;
        rec[6] = tally[kTSmall]; rec[7] = tally[kTLarge]; rec[8] = st_hiz;
        for (int k = 1; k < 8; ++k) rec[8 + k] = ticks[k];
        // path tallies instead of the phase timers: first or second half of them
        if (fp.phase_timers == 2) for (int k = 0; k < 7; ++k) rec[9 + k] = tally[2 + k];
        if (fp.phase_timers == 3) for (int k = 0; k < 7; ++k) rec[9 + k] = tally[9 + k];
        if (fp.phase_timers == 0) {
            // without phase timers the last words tell where and when the group ran: the sum of the
            // wavefronts' durations (against word 5: how unevenly they finish), the environment, start
            // and end on the device-wide 100 MHz clock, and the hardware id (compute unit, shader
            // engine in the low 24 bits, die above)
            rec[12] = dt;
            if (wave == 0) {
                rec[11] = item.env;
                rec[13] = (uint32_t)t_start;
                rec[14] = (uint32_t)wall_clock64();
                rec[15] = (__builtin_amdgcn_s_getreg((31 << 11) | 4) & 0xFFFFFFu) |
                          (__builtin_amdgcn_s_getreg((3 << 11) | 20) << 24);
            }
        }
    }
    __syncthreads();
    if (stats && tid < 16) {
        const uint32_t* rec = reinterpret_cast<const uint32_t*>(list);
        unsigned long long sum = 0, mx = 0;
        for (int w = 0; w < NW; ++w) { sum += rec[w * 16 + tid]; mx = max(mx, (unsigned long long)rec[w * 16 + tid]); }
        stats[(size_t)blockIdx.x * 16 + tid] = tid == 5 ? mx : sum;      // word 5: longest wavefront of the group
    }

    // ---- resolve this work-group's frame
    const size_t base = (size_t)item.env * fq.H * fq.W;
    for (int p = tid; p < nslots; p += NT) {
        const int y = FRAME ? p >> 6 : p / win.w, x = FRAME ? p & 63 : p - y * win.w;
        if (FRAME == 1 && x >= win.w) continue;
        const size_t o = base + (size_t)(win.y0 + y) * fq.W + (size_t)(win.x0 + x);
        const u64 key = vis[p];
        const bool hit = key != kEmptyKey;
        if (fp.merge) {
            if (hit) atomicMin(&gvis[o], key);
        } else {
            out_depth[o] = hit ? __uint_as_float((uint32_t)(key >> 32)) : fp.background;
            if (out_id) out_id[o] = hit ? (uint32_t)key : 0xFFFFFFFFu;
        }
    }
}

// Resolve of the global visibility buffer (used when an environment was split over several
// work-groups); leaves the buffer cleared for the next request.
__global__ void k_resolve(unsigned long long* __restrict__ gvis, size_t n, float background,
                          float* __restrict__ out_depth, uint32_t* __restrict__ out_id) {
    size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    u64 key = gvis[p];
    bool hit = key != kEmptyKey;
    out_depth[p] = hit ? __uint_as_float((uint32_t)(key >> 32)) : background;
    if (out_id) out_id[p] = hit ? (uint32_t)key : 0xFFFFFFFFu;
    if (hit) gvis[p] = kEmptyKey;
}

// Launch planning.  Work-groups are dispatched in index order, so handing out the most expensive
// items first (longest processing time first) shortens the tail of the launch.  An item's cost
// is estimated as the number of its scene's 64-cluster blocks that are not wholly outside the
// environment's frustum; k_dispatch_order then sorts all items by decreasing cost.
__global__ __launch_bounds__(64) void k_item_cost(const SceneDev* __restrict__ scenes, const WorkItem* __restrict__ items,
                                                  const float* __restrict__ view_proj, FrameParams fp, uint32_t n_items,
                                                  uint32_t* __restrict__ cost) {
    const uint32_t i = blockIdx.x;
    if (i >= n_items) return;
    const WorkItem item = items[i];
    const SceneDev sc = scenes[item.scene];
    const BPS_GLOBAL float* bb = gptr(sc.bbounds);
    const uint32_t nblocks = (sc.n_clusters + 63u) / 64u;
    const uint32_t S = item.split_of >> 16, item_split = item.split_of & 0xFFFFu;
    Window win;
    place_window(win, item.tile, fp);
    __shared__ __align__(16) float planes[8 * kPlaneRow];
    const int lane = (int)threadIdx.x;
    float M[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) M[k] = view_proj[(size_t)item.env * 16 + k];
    if (lane < 8) fill_planes(planes, M, win, lane);
    wave_lds_sync();
    uint32_t count = 0;
    for (uint32_t first = item_split; first < nblocks; first += S * 64u) {
        const uint32_t at = first + S * (uint32_t)lane, gb = min(at, nblocks - 1u);
        float lx = bb[gb], ly = bb[sc.b_stride + gb], lz = bb[2 * sc.b_stride + gb];
        float hx = bb[3 * sc.b_stride + gb], hy = bb[4 * sc.b_stride + gb], hz = bb[5 * sc.b_stride + gb];
        count += box_outside_frustum(planes, lane, lx, ly, lz, hx, hy, hz) | (at >= nblocks) ? 0u : 1u;
    }
#pragma unroll
    for (int sh = 32; sh >= 1; sh >>= 1) count += (uint32_t)__shfl_xor((int)count, sh, 64);
    if (threadIdx.x == 0) cost[i] = count;
}

// Dispatch order = all items by decreasing estimated cost (counting sort over 2048 linear cost
// buckets): consecutive work-group indices go to consecutive dies, so every die receives an even
// sample of the cost distribution, costliest first.
__global__ __launch_bounds__(1024) void k_dispatch_order(const uint32_t* __restrict__ cost, uint32_t n_items,
                                                         const WorkItem* __restrict__ items, WorkItem* __restrict__ ordered) {
    constexpr uint32_t kBuckets = 2048;
    constexpr int kPerThread = (int)(kMaxPlannedItems / 1024u);      // every thread keeps its items' costs in registers
    __shared__ uint32_t bucket[kBuckets];
    __shared__ uint32_t scan[1024];
    static_assert(kMaxPlannedItems <= 65536u, "item indices are kept as 16-bit words");
    __shared__ uint16_t order_lds[kMaxPlannedItems];                  // the order, before the die-affinity pass
    __shared__ uint32_t largest;
    const uint32_t tid = threadIdx.x;
    uint32_t my_cost[kPerThread];
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
        const uint32_t i = tid + (uint32_t)k * 1024u;
        my_cost[k] = i < n_items ? cost[i] : 0u;
    }
    for (uint32_t b = tid; b < kBuckets; b += 1024u) bucket[b] = 0u;
    if (tid == 0) largest = 0u;
    __syncthreads();
    {
        uint32_t mx = 0;
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) mx = max(mx, my_cost[k]);
#pragma unroll
        for (int sh = 32; sh >= 1; sh >>= 1) mx = max(mx, (uint32_t)__shfl_xor((int)mx, sh, 64));
        if ((tid & 63u) == 0u) atomicMax(&largest, mx);
    }
    __syncthreads();
    const float scale = largest ? (float)(kBuckets - 1) / (float)largest : 0.0f;
    auto bucket_of = [&](uint32_t c) -> uint32_t {      // bucket 0 holds the costliest items
        return kBuckets - 1u - min((uint32_t)((float)c * scale), kBuckets - 1u);
    };
    uint32_t my_slot[kPerThread];      // position inside the bucket
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
        const uint32_t i = tid + (uint32_t)k * 1024u;
        my_slot[k] = i < n_items ? atomicAdd(&bucket[bucket_of(my_cost[k])], 1u) : 0u;
    }
    __syncthreads();
    // exclusive prefix sum over the buckets: two per thread, then a scan over the 1024 pair sums
    const uint32_t a0 = bucket[2 * tid], a1 = bucket[2 * tid + 1];
    // inclusive scan of the 1024 pair sums: within each wavefront by shuffles, then over the 16
    // wavefront totals
    uint32_t incl = a0 + a1;
#pragma unroll
    for (int step = 1; step < 64; step <<= 1) {
        const uint32_t up = (uint32_t)__shfl_up((int)incl, step, 64);
        if ((tid & 63u) >= (uint32_t)step) incl += up;
    }
    if ((tid & 63u) == 63u) scan[tid >> 6] = incl;
    __syncthreads();
    uint32_t offset = 0;
    for (uint32_t wv = 0; wv < (tid >> 6); ++wv) offset += scan[wv];
    const uint32_t before = offset + incl - (a0 + a1);
    __syncthreads();       // scan[] is reused below, bucket[] is overwritten now
    bucket[2 * tid] = before;
    bucket[2 * tid + 1] = before + a0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
        const uint32_t i = tid + (uint32_t)k * 1024u;
        if (i < n_items) order_lds[bucket[bucket_of(my_cost[k])] + my_slot[k]] = (uint16_t)i;
    }
    __syncthreads();
    // Die affinity.  Position p of the order runs on die p % 8, and the host lays the items out so
    // that item i's scene is mostly used by items with the same i % 8.  Within every run of 64
    // consecutive positions (items of nearly equal cost, eight positions per die) the items are
    // rearranged so that as many as possible land on their own die; each die still gets eight
    // items of every cost class, but now finds its scenes in its own L2.
    uint32_t* slot_item = scan;                       // [16 waves][64]: the window being rebuilt
    const uint32_t lane = tid & 63u, wave = tid >> 6;
    for (uint32_t base = wave * 64u; base + 64u <= n_items; base += 1024u) {
        const uint32_t item = (uint32_t)order_lds[base + lane];
        const uint32_t home = item & 7u;
        uint32_t* mine = slot_item + wave * 64u;
        mine[lane] = 0xFFFFFFFFu;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        bool placed = false;
        for (uint32_t d = 0; d < 8u; ++d) {
            const unsigned long long want = __builtin_amdgcn_ballot_w64(home == d);
            const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(want >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)want, 0u));
            if (home == d && rank < 8u) {
                mine[rank * 8u + d] = item;
                placed = true;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // the rest take the free positions in order
        const unsigned long long free_mask = __builtin_amdgcn_ballot_w64(mine[lane] == 0xFFFFFFFFu);
        const unsigned long long left_mask = __builtin_amdgcn_ballot_w64(!placed);
        if (!placed) {
            uint32_t r = __builtin_amdgcn_mbcnt_hi((uint32_t)(left_mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)left_mask, 0u));
            unsigned long long m = free_mask;
            for (uint32_t k = 0; k < r; ++k) m &= m - 1ull;      // drop the r lowest free positions
            mine[__builtin_ctzll(m)] = item;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // the raster kernel reads its item at its own work-group index: one dependent load fewer
        // than going through the order
        ordered[base + lane] = items[mine[lane]];
    }
    for (uint32_t i = (n_items & ~63u) + tid; i < n_items; i += 1024u) ordered[i] = items[order_lds[i]];
}

void launch_plan(hipStream_t stream, const SceneDev* scenes, const WorkItem* items, const float* view_proj,
                 const FrameParams& fp, uint32_t n_items, uint32_t* cost, WorkItem* ordered) {
    hipLaunchKernelGGL(k_item_cost, dim3(n_items), dim3(64), 0, stream, scenes, items, view_proj, fp, n_items, cost);
    hipLaunchKernelGGL(k_dispatch_order, dim3(1), dim3(1024), 0, stream, cost, n_items, items, ordered);
}

__global__ __launch_bounds__(64) void k_unpack_items(PackedItems packed, uint32_t first, uint32_t count,
                                                     WorkItem* __restrict__ items) {
    const uint32_t k = blockIdx.x * 64u + threadIdx.x;
    if (k >= count) return;
    const uint32_t w = packed.word[k];
    WorkItem it;
    it.env = w & ((1u << kPackedEnvBits) - 1u);
    it.scene = (w >> kPackedEnvBits) & ((1u << kPackedSceneBits) - 1u);
    it.split_of = 1u << 16;
    it.tile = w >> (kPackedEnvBits + kPackedSceneBits);
    items[first + k] = it;
}

void launch_unpack_items(hipStream_t stream, const PackedItems& packed, uint32_t first, uint32_t count, WorkItem* items) {
    hipLaunchKernelGGL(k_unpack_items, dim3((count + 63u) / 64u), dim3(64), 0, stream, packed, first, count, items);
}

__global__ void k_zero_words(unsigned long long* __restrict__ p, size_t n) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

__global__ void k_fill_keys(unsigned long long* __restrict__ gvis, size_t n) {
    size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n) gvis[p] = kEmptyKey;
}

namespace {
template <bool DIAG, int CULL>
const void* raster_entry(int threads) {
    return threads == 256   ? reinterpret_cast<const void*>(&k_raster<256, DIAG, CULL, 0>)
           : threads == 384 ? reinterpret_cast<const void*>(&k_raster<384, DIAG, CULL, 0>)
           : threads == 512 ? reinterpret_cast<const void*>(&k_raster<512, DIAG, CULL, 0>)
                            : reinterpret_cast<const void*>(&k_raster<1024, DIAG, CULL, 0>);
}
}  // namespace

hipError_t prepare_raster(int threads, size_t lds, bool fixed_layout, size_t wide_lds) {
    const void* entries[6] = {raster_entry<false, 0>(threads), raster_entry<false, 1>(threads), raster_entry<false, 2>(threads),
                              raster_entry<true, 0>(threads),  raster_entry<true, 1>(threads),  raster_entry<true, 2>(threads)};
    for (const void* f : entries) {
        hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    if (!fixed_layout) return hipSuccess;
    const void* fixed[3] = {reinterpret_cast<const void*>(&k_raster<512, false, 2, 64>),
                            reinterpret_cast<const void*>(&k_raster<512, false, 2, 128>),
                            reinterpret_cast<const void*>(&k_raster<512, false, 2, 1>)};
    for (const void* f : fixed) {
        hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes(64, 64, 512, (int)kListCap64));
        if (e != hipSuccess) return e;
    }
    if (!wide_lds) return hipSuccess;
    hipError_t e = hipFuncSetAttribute(raster_entry<true, 2>(1024), hipFuncAttributeMaxDynamicSharedMemorySize, (int)wide_lds);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_raster<1024, false, 2, 1>), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)lds_bytes(64, 64, 1024, (int)kListCap64));
}

hipError_t launch_raster(hipEvent_t done, int threads, dim3 grid, size_t lds, hipStream_t stream, const SceneDev* scenes, const WorkItem* items,
                   const float* view_proj, const FrameParams& request, bool fixed_layout, bool wide, unsigned long long* gvis,
                   float* out_depth, uint32_t* out_id, unsigned long long* stats) {
    // The default configuration runs on instances whose LDS layout is a compile-time constant: one each for
    // 64x64 and 128x128 frames drawn as 64x64 windows, and one for every other frame and window size.
    int frame = 0;
    if (threads == 512 && request.cull == 2 && fixed_layout) {
        const bool full = request.tile_w == 64 && request.tile_h == 64;
        frame = full && !wide && request.W == 64 && request.H == 64 ? 64 : full && !wide && request.W == 128 && request.H == 128 ? 128 : 1;
    }
    // (the instances that count are no such, and count what the one does that draws the request otherwise)
    FrameParams fp = request;
    fp.small_max = small_max(frame);
    if (frame != 0 && !stats) {
        const size_t lds64 = lds_bytes(64, 64, 512, (int)kListCap64);
        if (wide) {
            return launch_kernel(done, &k_raster<1024, false, 2, 1>, grid, dim3(1024), lds_bytes(64, 64, 1024, (int)kListCap64), stream, scenes,
                                 items, view_proj, fp, gvis, out_depth, out_id, stats);
        }
#define BPS_LAUNCH_FIXED(FRAME)                                                                                        \
    return launch_kernel(done, &k_raster<512, false, 2, FRAME>, grid, dim3(512), lds64, stream, scenes, items, view_proj, fp, gvis, \
                         out_depth, out_id, stats)
        if (frame == 64) BPS_LAUNCH_FIXED(64);
        else if (frame == 128) BPS_LAUNCH_FIXED(128);
        else BPS_LAUNCH_FIXED(1);
#undef BPS_LAUNCH_FIXED
    }
#define BPS_LAUNCH3(NT, DIAG, CULL)                                                                                    \
    return launch_kernel(done, &k_raster<NT, DIAG, CULL, 0>, grid, dim3(NT), lds, stream, scenes, items, view_proj, fp, gvis,   \
                         out_depth, out_id, stats)
#define BPS_LAUNCH2(NT, DIAG)                                                                                          \
    do {                                                                                                               \
        if (fp.cull == 0) BPS_LAUNCH3(NT, DIAG, 0);                                                                    \
        else if (fp.cull == 1) BPS_LAUNCH3(NT, DIAG, 1);                                                               \
        else BPS_LAUNCH3(NT, DIAG, 2);                                                                                 \
    } while (0)
#define BPS_LAUNCH(NT)                                                                                                 \
    do {                                                                                                               \
        if (stats) BPS_LAUNCH2(NT, true);                                                                              \
        else BPS_LAUNCH2(NT, false);                                                                                   \
    } while (0)
    if (wide) BPS_LAUNCH(1024);      // (diagnostics of what the instance above draws otherwise)
    else if (threads == 256) BPS_LAUNCH(256);
    else if (threads == 384) BPS_LAUNCH(384);
    else if (threads == 512) BPS_LAUNCH(512);
    else BPS_LAUNCH(1024);
#undef BPS_LAUNCH
#undef BPS_LAUNCH2
#undef BPS_LAUNCH3
}

}  // namespace bps
