// Drawing-quality metrics (Section 5.2): edge crossings, the standard
// deviation of edge lengths, and the similarity of the drawing's Gabriel
// graph to the graph (mean Jaccard index of the neighbourhoods).
//
// Coordinates are taken at single precision, so a product of two coordinates
// is exact in double.  Orientation and in-disc signs are first evaluated in
// double with an a-priori error bound; where the value is within the bound
// of zero the sign is taken exactly, from the polynomial multiplied out into
// such products and summed with expansion arithmetic (two-sum chains).
//
//   edge_list_kernel      edges {u, v}, u < v, in row order (the part of a
//                         sorted row above v is a suffix found by bisection)
//   cross_*_kernel        edges sorted by the place of their two ends (on a
//                         four-dimensional Hilbert curve) and cut into groups
//                         of 64 with a box around the left ends and one
//                         around the right ends
//   crossings_kernel      wavefront per group, an edge per lane, against a
//                         range of groups: boxes apart, nothing; else every
//                         edge of the other group, one per lane, against this
//                         group's boxes (no edge of it can be crossed, all of
//                         them are, or neither is sure); and only the unsure
//                         ones against each of the 64 edges, by filtered
//                         signs
//   lengths kernels       per-edge length, fixed-order sums (mean, then the
//                         squared deviations)
//   grid kernels          points binned into a uniform grid (about two per
//                         cell)
//   gabriel_degree_kernel a few lanes per point u (in cell order): rings of cells
//                         around u until each of the eight 45-degree octants
//                         around u is settled: the nearest point w found in it
//                         blocks everything at squared distance >= 2 |w - u|^2
//                         (such a v sees w within 45 degrees of its own
//                         direction, so w lies in the disc with diameter uv),
//                         or, with no point found, the rings cover the part of
//                         the bounding box the octant reaches; then every
//                         point not excluded that way is tested for an empty
//                         disc with diameter uv (cells scanned outwards from
//                         the disc's centre)
//   gabriel_edge_kernel   the same disc test for each graph edge (for the
//                         Jaccard intersections)
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <vector>

#include "device_util.h"
#include "gila_internal.h"

namespace gila {

namespace {
struct MBuf {
    hipStream_t st;
    void* p = nullptr;
    explicit MBuf(hipStream_t s) : st(s) {}
    ~MBuf() { dfree_on(p, st); }
    template <class T>
    int alloc(size_t count) {
        return dalloc(&p, count * sizeof(T) + 64);
    }
    template <class T>
    T* as() const {
        return static_cast<T*>(p);
    }
};
int mgrid(int64_t items) {
    return (int)std::max<int64_t>(1, std::min<int64_t>(8192, (items + kBlock - 1) / kBlock));
}
}  // namespace

// Lanes that share one point's search, and the cells and points that one of them visits
// before the point gets a wavefront of its own, by the number of points.  A lane more
// shortens the walks, which is the time while the device has lanes to spare (it holds 2^18
// of these), but the lanes of a group repeat each other's work between rings and wait for
// the one with the fullest cell.  Similarity in ms with 1 / 2 / 8 lanes (budgets 2048, 1280,
// 4096): 10k points at random 3.0 / 1.7 / 0.9, smoothed 9.7 / 10 / 5.0; 65k 4.1 / 3.1 / 2.1
// and 7.8 / 5.8 / 5.5; 131k 5.2 / 3.9 / 3.3 and 9.8 / 7.0 / 11, in clusters of 50
// 38 / 41 / 43, on a lattice 1.3 / 1.3 / 1.8; 262k at random 6.3 / 6.6 / 5.8, in clusters
// 126 / 139 / 187, on a lattice 1.7 / 1.9 / 2.5.
struct GabrielPlan {
    int lanes;
    int64_t budget;
};
inline GabrielPlan gabriel_plan(int32_t n) {
    if (n <= 65536) return {8, 4096};
    if (n <= 131072) return {2, 1280};
    return {1, 2048};
}

// ------------------------------------------------------------------ points and edges
template <class V>
__global__ __launch_bounds__(kBlock) void to_float_kernel(int32_t n, const V* __restrict__ pos,
                                                          float2* __restrict__ out) {
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * kBlock)
        out[v] = make_float2((float)pos[v].x, (float)pos[v].y);
}

// first entry of row v above v, and how many there are
__global__ __launch_bounds__(kBlock) void upper_count_kernel(int32_t n, const int64_t* __restrict__ rp,
                                                             const int32_t* __restrict__ ci,
                                                             int64_t* __restrict__ first,
                                                             int64_t* __restrict__ cnt) {
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * kBlock) {
        int64_t lo = rp[v], hi = rp[v + 1];
        const int64_t end = hi;
        while (lo < hi) {
            const int64_t mid = lo + ((hi - lo) >> 1);
            if (ci[mid] <= v) lo = mid + 1;
            else hi = mid;
        }
        first[v] = lo;
        cnt[v] = end - lo;
    }
}

// Wavefront per vertex: its upper entries become edges eo[v] ...
__global__ __launch_bounds__(kBlock) void edge_list_kernel(int32_t n, const int64_t* __restrict__ rp,
                                                           const int32_t* __restrict__ ci,
                                                           const int64_t* __restrict__ first,
                                                           const int64_t* __restrict__ eo,
                                                           int2* __restrict__ ends) {
    const int64_t waves = (int64_t)gridDim.x * kWaves;
    for (int64_t v = (int64_t)blockIdx.x * kWaves + wave_id(); v < n; v += waves) {
        const int64_t f = first[v], len = rp[v + 1] - f, o = eo[v];
        for (int64_t j = lane64(); j < len; j += 64) ends[o + j] = make_int2((int32_t)v, ci[f + j]);
    }
}

// ------------------------------------------------------------------ exact signs
// Knuth's two-sum: s is the rounded a + b and s + e == a + b exactly.
__device__ __forceinline__ void two_sum(double a, double b, double& s, double& e) {
#pragma clang fp contract(off)
    s = a + b;
    const double bb = s - a;
    e = (a - (s - bb)) + (b - bb);
}

// Exact sign of t[0] + ... + t[K-1].  Each term is merged into a growing
// expansion by a chain of two-sums (Shewchuk's grow-expansion); the pieces
// stay nonoverlapping with the largest last, so the sign of the sum is that
// of the last nonzero piece.
template <int K>
__device__ __forceinline__ int exact_sum_sign(const double (&t)[K]) {
    double h[K];
#pragma unroll
    for (int i = 0; i < K; ++i) {
        double q = t[i];
#pragma unroll
        for (int j = 0; j < i; ++j) two_sum(q, h[j], q, h[j]);
        h[i] = q;
    }
    int sg = 0;
#pragma unroll
    for (int j = 0; j < K; ++j) sg = h[j] > 0.0 ? 1 : (h[j] < 0.0 ? -1 : sg);
    return sg;
}

// orient(a, b, c) = (b - a) x (c - a) multiplied out (the two a.x a.y
// products cancel); products of single-precision values are exact in double.
__device__ __noinline__ int orient_exact(float ax, float ay, float bx, float by, float cx, float cy) {
    const double t[6] = {(double)bx * cy, -((double)bx * ay), -((double)ax * cy),
                         -((double)by * cx), (double)by * ax, (double)ay * cx};
    return exact_sum_sign(t);
}

// ------------------------------------------------------------------ crossings
constexpr int kCrossGroup = 64;           // edges per group: one per lane
constexpr int64_t kCrossSortMin = 4096;   // edges sorted by place from here on
constexpr int64_t kCrossWaves = 262144;   // wavefronts to cut the group pairs into

// A segment's line: for a point (x, y), orient(p0, p1, (x, y)) =
// dx y - dy x - k, evaluated as fma(dx, y, fma(-dy, x, -k)).  Its rounding
// error is below 2u |dx| |y| + 3u |dy| |x| + 3u (|x1 y0| + |y1 x0|) plus
// second-order terms (u = 2^-53; coordinates are floats, so x1 y0 and y1 x0
// are exact), hence below bnd = 8u((|dx| + |dy|) M + |x1 y0| + |y1 x0|) for
// every point with coordinates of magnitude at most M.  The line is scaled by
// the power of two that brings bnd into [1/2, 1), which is exact, so a sign is
// certain where the scaled value is at least 1 in magnitude.  A line with
// bnd = 0 (all its values are 0) stays unscaled and is never certain.
struct Line {
    double dx, dy, k;
};

__device__ __forceinline__ Line make_line(float4 z, double M) {
#pragma clang fp contract(off)
    Line L;
    L.dx = (double)z.z - (double)z.x;
    L.dy = (double)z.w - (double)z.y;
    const double s = (double)z.z * z.y, u = (double)z.w * z.x;
    L.k = s - u;
    const double bnd = ((fabs(L.dx) + fabs(L.dy)) * M + (fabs(s) + fabs(u))) * 0x1p-50;
    if (bnd > 0.0) {
        int ex = 0;
        (void)frexp(bnd, &ex);
        L.dx = ldexp(L.dx, -ex);
        L.dy = ldexp(L.dy, -ex);
        L.k = ldexp(L.k, -ex);
    }
    return L;
}

__device__ __forceinline__ double side(const Line& L, double x, double y) {
    return fma(L.dx, y, fma(-L.dy, x, -L.k));
}

// The unsure edges of the other group as the pair test reads them from LDS
// (16-byte broadcasts: the ends, the direction, and two entries' k at once).
struct CrossEntries {
    double2 p0[kCrossGroup], p1[kCrossGroup], d[kCrossGroup];
    alignas(16) double k[kCrossGroup];
    int at[kCrossGroup];  // place in the group
};

// Filtered signs of one pair per lane: edge i of the lane, the entry's edge.
// sure: all four signs are certain; cross: the ends of each lie on opposite
// sides of the other's line (where sure).
__device__ __forceinline__ void pair_masks(const Line& li, double ax, double ay, double bx, double by,
                                           double2 p0, double2 p1, double2 d, double k,
                                           uint64_t& sure, uint64_t& cross) {
    const Line lc{d.x, d.y, k};
    const double d1 = side(li, p0.x, p0.y);
    const double d2 = side(li, p1.x, p1.y);
    const double d3 = side(lc, ax, ay);
    const double d4 = side(lc, bx, by);
    const int w1 = __double2hiint(d1), w2 = __double2hiint(d2);
    const int w3 = __double2hiint(d3), w4 = __double2hiint(d4);
    // smallest magnitude, by the high words taken as floats (a double's high
    // word orders as the double does)
    float low;
    asm("v_min3_f32 %0, |%1|, |%2|, |%3|" : "=v"(low) : "v"(w1), "v"(w2), "v"(w3));
    asm("v_min_f32 %0, %1, |%2|" : "=v"(low) : "v"(low), "v"(w4));
    constexpr float kOne = 1.875f;  // the high word of 1.0 as a float
    sure = __builtin_amdgcn_ballot_w64(low >= kOne);
    cross = __builtin_amdgcn_ballot_w64(((w1 ^ w2) & (w3 ^ w4)) < 0);
}

// A group's boxes: of its edges' left ends and of their right ends.
struct alignas(32) CrossBox {
    float px0, py0, px1, py1, qx0, qy0, qx1, qy1;
};

// bit b of an 8-bit value to bit 4 b
__device__ __forceinline__ uint32_t spread4(uint32_t q) {
    q = (q | (q << 12)) & 0x000F000Fu;
    q = (q | (q << 6)) & 0x03030303u;
    return (q | (q << 3)) & 0x11111111u;
}

// Place of a cell of the 256^4 grid on a four-dimensional Hilbert curve, by
// the transposed form of J. Skilling, "Programming the Hilbert curve" (2004).
// Consecutive places are neighbouring cells: boxes around 64 of them leave
// 22% of R-MAT 17's pairs unsure, against 27% in Morton order.
__device__ __forceinline__ uint32_t hilbert4(uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3) {
    uint32_t x[4] = {x0, x1, x2, x3};
#pragma unroll
    for (uint32_t q = 128u; q > 1u; q >>= 1) {
        const uint32_t p = q - 1u;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool on = x[i] & q;
            const uint32_t t = on ? 0u : (x[0] ^ x[i]) & p;
            x[0] ^= on ? p : t;
            x[i] ^= t;
        }
    }
#pragma unroll
    for (int i = 1; i < 4; ++i) x[i] ^= x[i - 1];
    uint32_t t = 0;
#pragma unroll
    for (uint32_t q = 128u; q > 1u; q >>= 1) t ^= (x[3] & q) ? q - 1u : 0u;
    return (spread4(x[0] ^ t) << 3) | (spread4(x[1] ^ t) << 2) | (spread4(x[2] ^ t) << 1) | spread4(x[3] ^ t);
}

__device__ __forceinline__ bool left_first(float2 a, float2 b) {
    return a.x < b.x || (a.x == b.x && a.y <= b.y);
}

// Place of (left end, right end) on the curve, eight bits per coordinate.
__global__ __launch_bounds__(kBlock) void cross_key_kernel(int64_t m, const int2* __restrict__ ends,
                                                           const float2* __restrict__ p, float2 lo,
                                                           float2 scale, uint32_t* __restrict__ key) {
    const auto cell = [](float x, float l, float s) {
        const float c = (x - l) * s;  // (a NaN from an overflowing range lands in cell 0)
        return c >= 255.f ? 255u : (c > 0.f ? (uint32_t)c : 0u);
    };
    for (int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x; e < m;
         e += (int64_t)gridDim.x * kBlock) {
        float2 a = p[ends[e].x], b = p[ends[e].y];
        if (!left_first(a, b)) {
            const float2 t = a;
            a = b;
            b = t;
        }
        key[e] = hilbert4(cell(a.x, lo.x, scale.x), cell(a.y, lo.y, scale.y), cell(b.x, lo.x, scale.x),
                          cell(b.y, lo.y, scale.y));
    }
}

// Wavefront per group: its edges' ends, left one (smaller x, then y) first,
// and the group's boxes.  order: null for row order.
__global__ __launch_bounds__(kBlock) void cross_prepare_kernel(int64_t m, int64_t groups,
                                                               const int2* __restrict__ ends,
                                                               const float2* __restrict__ p,
                                                               const int32_t* __restrict__ order,
                                                               float4* __restrict__ seg,
                                                               CrossBox* __restrict__ box) {
    const int64_t waves = (int64_t)gridDim.x * kWaves;
    for (int64_t g = (int64_t)blockIdx.x * kWaves + wave_id(); g < groups; g += waves) {
        const int64_t t = g * kCrossGroup + lane64();
        const int64_t at = t < m ? t : m - 1;  // lanes past the end repeat the last edge in the box
        const int2 e = ends[order ? (int64_t)order[at] : at];
        float2 a = p[e.x], b = p[e.y];
        if (!left_first(a, b)) {
            const float2 q = a;
            a = b;
            b = q;
        }
        if (t < m) seg[t] = make_float4(a.x, a.y, b.x, b.y);
        float lo[4] = {a.x, a.y, b.x, b.y}, hi[4] = {a.x, a.y, b.x, b.y};
        for (int off = 32; off >= 1; off >>= 1)
            for (int q = 0; q < 4; ++q) {
                lo[q] = fminf(lo[q], __shfl_xor(lo[q], off, 64));
                hi[q] = fmaxf(hi[q], __shfl_xor(hi[q], off, 64));
            }
        if (lane64() == 0) box[g] = CrossBox{lo[0], lo[1], hi[0], hi[1], lo[2], lo[3], hi[2], hi[3]};
    }
}

// Exact crossing decision for a pair the filter could not settle.
__device__ __forceinline__ int cross_exact(int2 ea, int2 ec, const float2* __restrict__ p) {
    if (ea.x == ec.x || ea.x == ec.y || ea.y == ec.x || ea.y == ec.y) return 0;
    const float2 a = p[ea.x], b = p[ea.y], c = p[ec.x], d = p[ec.y];
    const int o1 = orient_exact(a.x, a.y, b.x, b.y, c.x, c.y);
    const int o2 = orient_exact(a.x, a.y, b.x, b.y, d.x, d.y);
    if (o1 * o2 >= 0) return 0;
    const int o3 = orient_exact(c.x, c.y, d.x, d.y, a.x, a.y);
    const int o4 = orient_exact(c.x, c.y, d.x, d.y, b.x, b.y);
    return o3 * o4 < 0 ? 1 : 0;
}

// Range of orient(p, q, z) over p in the box's left part, q in its right one:
// (p - z) x (q - z), whose four factors vary independently, so the products'
// ranges give it exactly (up to rounding).
__device__ __forceinline__ void orient_range(const CrossBox& B, float zx, float zy, float& lo, float& hi) {
    const float ux0 = B.px0 - zx, ux1 = B.px1 - zx, uy0 = B.py0 - zy, uy1 = B.py1 - zy;
    const float wx0 = B.qx0 - zx, wx1 = B.qx1 - zx, wy0 = B.qy0 - zy, wy1 = B.qy1 - zy;
    const float a0 = ux0 * wy0, a1 = ux0 * wy1, a2 = ux1 * wy0, a3 = ux1 * wy1;
    const float b0 = uy0 * wx0, b1 = uy0 * wx1, b2 = uy1 * wx0, b3 = uy1 * wx1;
    lo = fminf(fminf(fminf(a0, a1), a2), a3) - fmaxf(fmaxf(fmaxf(b0, b1), b2), b3);
    hi = fmaxf(fmaxf(fmaxf(a0, a1), a2), a3) - fminf(fminf(fminf(b0, b1), b2), b3);
}

// What a group's boxes say of an edge (ends z0, z1): 0 it crosses none of the
// group, 1 all of it, 2 unsure.  eps covers the rounding of every value
// compared, so 0 and 1 are what the exact signs give for each edge of the
// group: the values are differences of two products of coordinate differences.
// With u = 2^-24 a coordinate difference, at most 2 M, errs by 2 M u, a product
// of two by 12 M^2 u (8 from its factors, 4 from itself) and the whole, at most
// 8 M^2, by 2 * 12 + 8 = 32 M^2 u = 2^-19 M^2 and terms in u^2; eps is twice that.
// (An edge that shares an end with one of the group, or is one of it, is never
// found to cross all: that orientation is 0.)
__device__ __forceinline__ int group_verdict(const CrossBox& B, float4 z, float eps) {
    if (fmaxf(z.x, z.z) < fminf(B.px0, B.qx0) || fminf(z.x, z.z) > fmaxf(B.px1, B.qx1) ||
        fmaxf(z.y, z.w) < fminf(B.py0, B.qy0) || fminf(z.y, z.w) > fmaxf(B.py1, B.qy1))
        return 0;
    // the edge's line over the two boxes
    const float dx = z.z - z.x, dy = z.w - z.y;
    const auto side_range = [&](float x0, float x1, float y0, float y1, float& lo, float& hi) {
        const float a0 = dx * (y0 - z.y), a1 = dx * (y1 - z.y);
        const float b0 = dy * (x0 - z.x), b1 = dy * (x1 - z.x);
        lo = fminf(a0, a1) - fmaxf(b0, b1);
        hi = fmaxf(a0, a1) - fminf(b0, b1);
    };
    float pl, ph, ql, qh;
    side_range(B.px0, B.px1, B.py0, B.py1, pl, ph);
    side_range(B.qx0, B.qx1, B.qy0, B.qy1, ql, qh);
    if ((pl > eps && ql > eps) || (ph < -eps && qh < -eps)) return 0;
    float l0, h0, l1, h1;
    orient_range(B, z.x, z.y, l0, h0);
    orient_range(B, z.z, z.w, l1, h1);
    if ((l0 > eps && l1 > eps) || (h0 < -eps && h1 < -eps)) return 0;
    const bool apart = (pl > eps && qh < -eps) || (ph < -eps && ql > eps);
    const bool across = (l0 > eps && h1 < -eps) || (h0 < -eps && l1 > eps);
    return apart && across ? 1 : 2;
}

// Wavefront (group blockIdx.x * kWaves + wave, range blockIdx.y of `span`
// groups): its 64 edges i, one per lane, against every edge j of the range.  A
// crossing is a pair with no shared end whose ends lie strictly on opposite
// sides of the other's line.  PAIRS_ONCE: only j > i in sorted order counts
// (each crossing once, for the total); otherwise every j != i counts and
// per_edge[] accumulates.
//
// Bound by the pair test (eight FMA, three operations on the high words for
// certainty -- a double's high word orders as the double, and as a float
// pattern -- and three for the signs, against 20 operations before, with four
// conversions) and, about equally, by its three 16-byte LDS broadcasts; what
// makes the difference is how few pairs reach it: a quarter on a smoothed
// drawing of R-MAT 17 (groups' boxes apart for 56% of the pairs, 13% decided
// by the boxes), 6% on a Watts-Strogatz graph's.  Reading the other edge
// through the scalar cache instead of LDS left the loop waiting for its misses
// (57 ms on R-MAT 17).
template <bool PAIRS_ONCE>
__global__ __launch_bounds__(kBlock, 6) void crossings_kernel(int64_t m, int64_t groups, int64_t span,
                                                              double M, float eps,
                                                              const float4* __restrict__ seg,
                                                              const CrossBox* __restrict__ box,
                                                              const int32_t* __restrict__ order,
                                                              const int2* __restrict__ ends,
                                                              const float2* __restrict__ p,
                                                              unsigned long long* __restrict__ per_edge,
                                                              unsigned long long* __restrict__ total) {
    __shared__ CrossEntries s_entry[kWaves];
    const int64_t g = (int64_t)blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane(wave_id());
    int64_t h0 = (int64_t)blockIdx.y * span;
    const int64_t h1 = min(h0 + span, groups);
    if (g >= groups || (PAIRS_ONCE && h1 <= g)) return;
    if (PAIRS_ONCE) h0 = max(h0, g);
    const int lane = lane64();
    CrossEntries& mine = s_entry[wave_id()];
    const int64_t i = g * kCrossGroup + lane;
    const uint64_t live = __ballot(i < m);
    const float4 ei = seg[min(i, m - 1)];
    const Line li = make_line(ei, M);
    const double ax = ei.x, ay = ei.y, bx = ei.z, by = ei.w;
    const auto id_of = [&](int64_t t) { return order ? (int64_t)order[t] : t; };
    // the group's boxes are uniform: read through the scalar cache (written by
    // an earlier launch)
    typedef const __attribute__((address_space(4))) CrossBox* BoxPtr;
    const BoxPtr bp = (BoxPtr)(box + g);
    CrossBox B;
    B.px0 = bp->px0;
    B.py0 = bp->py0;
    B.px1 = bp->px1;
    B.py1 = bp->py1;
    B.qx0 = bp->qx0;
    B.qy0 = bp->qy0;
    B.qx1 = bp->qx1;
    B.qy1 = bp->qy1;
    const float gx0 = fminf(B.px0, B.qx0), gx1 = fmaxf(B.px1, B.qx1);
    const float gy0 = fminf(B.py0, B.qy0), gy1 = fmaxf(B.py1, B.qy1);
    int64_t whole = 0;  // edges found to cross the whole group (uniform)
    int64_t sure_cnt = 0;
    int cnt = 0;
    for (int64_t hb = h0; hb < h1; hb += 64) {
        const int64_t h = hb + lane;
        bool near = false;
        if (h < h1) {
            const CrossBox C = box[h];
            near = fminf(C.px0, C.qx0) <= gx1 && fmaxf(C.px1, C.qx1) >= gx0 &&
                   fminf(C.py0, C.qy0) <= gy1 && fmaxf(C.py1, C.qy1) >= gy0;
        }
        uint64_t todo = __ballot(near);
        while (todo) {
            const int64_t hj = hb + __builtin_ctzll(todo);
            todo &= todo - 1ull;
            const int64_t j0 = hj * kCrossGroup;
            int verdict = 0;
            float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
            if (j0 + lane < m) {
                z = seg[j0 + lane];
                verdict = group_verdict(B, z, eps);
            }
            // (in its own group an edge is never found to cross all)
            whole += __popcll(__ballot(verdict == 1));
            const uint64_t open = __ballot(verdict == 2);
            __builtin_amdgcn_wave_barrier();  // the previous group's entries have been read
            if (verdict == 2) {
                const Line lj = make_line(z, M);
                const int at = __popcll(open & ((1ull << lane) - 1ull));
                mine.p0[at] = make_double2(z.x, z.y);
                mine.p1[at] = make_double2(z.z, z.w);
                mine.d[at] = make_double2(lj.dx, lj.dy);
                mine.k[at] = lj.k;
                mine.at[at] = lane;
            }
            __builtin_amdgcn_wave_barrier();
            const int count = __popcll(open);
            const auto take = [&](uint64_t sure, uint64_t cross, uint64_t keep) {
                const uint64_t yes = sure & cross & keep;
                if (PAIRS_ONCE) sure_cnt += __popcll(yes);
                else cnt += (int)((yes >> lane) & 1ull);
            };
            const auto settle = [&](uint64_t slow, int64_t at) {
                if ((slow >> lane) & 1ull) cnt += cross_exact(ends[id_of(i)], ends[id_of(j0 + at)], p);
            };
            if (hj != g) {
                // two entries a step: their reads and chains overlap
                int q = 0;
                for (; q + 1 < count; q += 2) {
                    const double2 k = *reinterpret_cast<const double2*>(&mine.k[q]);
                    uint64_t sure0, cross0, sure1, cross1;
                    pair_masks(li, ax, ay, bx, by, mine.p0[q], mine.p1[q], mine.d[q], k.x, sure0, cross0);
                    pair_masks(li, ax, ay, bx, by, mine.p0[q + 1], mine.p1[q + 1], mine.d[q + 1], k.y,
                               sure1, cross1);
                    take(sure0, cross0, live);
                    take(sure1, cross1, live);
                    if (~(sure0 & sure1) & live) [[unlikely]] {
                        settle(~sure0 & live, mine.at[q]);
                        settle(~sure1 & live, mine.at[q + 1]);
                    }
                }
                if (q < count) {
                    uint64_t sure, cross;
                    pair_masks(li, ax, ay, bx, by, mine.p0[q], mine.p1[q], mine.d[q], mine.k[q], sure, cross);
                    take(sure, cross, live);
                    if (~sure & live) [[unlikely]] settle(~sure & live, mine.at[q]);
                }
            } else {
                for (int q = 0; q < count; ++q) {  // i < j, or i != j
                    const int at = __builtin_amdgcn_readfirstlane(mine.at[q]);
                    const uint64_t keep = live & (PAIRS_ONCE ? (1ull << at) - 1ull : ~(1ull << at));
                    uint64_t sure, cross;
                    pair_masks(li, ax, ay, bx, by, mine.p0[q], mine.p1[q], mine.d[q], mine.k[q], sure, cross);
                    take(sure, cross, keep);
                    if (~sure & keep) [[unlikely]] settle(~sure & keep, at);
                }
            }
        }
    }
    if (!PAIRS_ONCE && i < m) {
        const int64_t own = (int64_t)cnt + whole;
        if (per_edge && own) atomicAdd(&per_edge[id_of(i)], (unsigned long long)own);
    }
    const int64_t w = wave_sum((int64_t)(i < m ? cnt : 0)) + sure_cnt + whole * __popcll(live);
    if (lane == 0 && w) atomicAdd(total, (unsigned long long)w);
}

// ------------------------------------------------------------------ edge lengths
__global__ __launch_bounds__(kBlock) void lengths_sum_kernel(int64_t m, const int2* __restrict__ ends,
                                                             const float2* __restrict__ p,
                                                             double mean, int pass,
                                                             double* __restrict__ partial) {
    __shared__ double s[kWaves];
    double acc = 0.0;
    for (int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x; e < m;
         e += (int64_t)gridDim.x * kBlock) {
        const float2 a = p[ends[e].x], b = p[ends[e].y];
        const double dx = (double)b.x - (double)a.x, dy = (double)b.y - (double)a.y;
        const double l = sqrt(dx * dx + dy * dy);
        acc += pass == 0 ? l : (l - mean) * (l - mean);
    }
    const double t = block_sum(acc, s);
    if (threadIdx.x == 0) partial[blockIdx.x] = t;
}

// ------------------------------------------------------------------ grid
struct Grid {
    float x0, y0, inv;  // cell of x: floor((x - x0) * inv)
    int32_t gx, gy;
};

__device__ __forceinline__ int32_t cell_x(const Grid& g, float x) {
    const float f = (x - g.x0) * g.inv;
    int32_t c = f >= 0.f ? (int32_t)f : 0;
    return c < g.gx ? c : g.gx - 1;
}
__device__ __forceinline__ int32_t cell_y(const Grid& g, float y) {
    const float f = (y - g.y0) * g.inv;
    int32_t c = f >= 0.f ? (int32_t)f : 0;
    return c < g.gy ? c : g.gy - 1;
}

__global__ __launch_bounds__(kBlock) void bounds_kernel(int32_t n, const float2* __restrict__ p,
                                                        unsigned int* __restrict__ box) {
    // box: ordered keys of xmin, ymin (min) and of -xmax, -ymax (min)
    __shared__ unsigned int s_k[4][kBlock];
    unsigned int k[4] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
    auto key = [](float f) {
        const unsigned int u = __float_as_uint(f);
        return (u >> 31) ? ~u : (u | 0x80000000u);
    };
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * kBlock) {
        const float2 q = p[v];
        k[0] = min(k[0], key(q.x));
        k[1] = min(k[1], key(q.y));
        k[2] = min(k[2], key(-q.x));
        k[3] = min(k[3], key(-q.y));
    }
    for (int c = 0; c < 4; ++c) s_k[c][threadIdx.x] = k[c];
    __syncthreads();
    for (int h = kBlock / 2; h > 0; h >>= 1) {
        if (threadIdx.x < h)
            for (int c = 0; c < 4; ++c) s_k[c][threadIdx.x] = min(s_k[c][threadIdx.x], s_k[c][threadIdx.x + h]);
        __syncthreads();
    }
    if (threadIdx.x < 4) atomicMin(&box[threadIdx.x], s_k[threadIdx.x][0]);
}

__global__ __launch_bounds__(kBlock) void cell_count_kernel(int32_t n, Grid g, const float2* __restrict__ p,
                                                            int32_t* __restrict__ cell,
                                                            int64_t* __restrict__ cnt) {
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * kBlock) {
        const int32_t c = cell_y(g, p[v].y) * g.gx + cell_x(g, p[v].x);
        cell[v] = c;
        atomicAdd((unsigned long long*)&cnt[c], 1ull);
    }
}

__global__ __launch_bounds__(kBlock) void cell_fill_kernel(int32_t n, const int32_t* __restrict__ cell,
                                                           const int64_t* __restrict__ start,
                                                           unsigned long long* __restrict__ cursor,
                                                           int32_t* __restrict__ pts) {
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * kBlock) {
        const int32_t c = cell[v];
        const unsigned long long at = atomicAdd(&cursor[c], 1ull);
        pts[start[c] + (int64_t)at] = (int32_t)v;
    }
}

// (w - u).(w - v) multiplied out into products of floats (exact in double)
__device__ __noinline__ int disc_sign_exact(float2 u, float2 v, float2 w) {
    const double t[8] = {(double)w.x * w.x, -((double)w.x * v.x), -((double)u.x * w.x),
                         (double)u.x * v.x, (double)w.y * w.y, -((double)w.y * v.y),
                         -((double)u.y * w.y), (double)u.y * v.y};
    return exact_sum_sign(t);
}

// w lies in the closed disc with diameter uv: (w - u).(w - v) <= 0.  The
// double evaluation errs by less than 3u(|l| + |r|) plus second-order terms
// (u = 2^-53, as for a 2x2 determinant of rounded differences); when the
// result is within 8u of zero the sign is taken exactly.
__device__ __forceinline__ bool in_disc(float2 u, float2 v, float2 w) {
#pragma clang fp contract(off)
    const double l = ((double)w.x - (double)u.x) * ((double)w.x - (double)v.x);
    const double r = ((double)w.y - (double)u.y) * ((double)w.y - (double)v.y);
    const double d = l + r;
    const double b = (fabs(l) + fabs(r)) * 0x1p-50;
    if (d > b) return false;
    if (d < -b) return true;
    return disc_sign_exact(u, v, w) <= 0;
}

// The cells at Chebyshev distance exactly k from (cx, cy) inside columns
// [x0, x1] and rows [y0, y1] ((cx, cy) itself inside), numbered
// 0 .. count - 1 so that a thread or the lanes of a wavefront can take them
// in turn: row cy - k in full (if inside), row cy + k in full (if inside and
// k > 0), then the rows between at columns cx - k and cx + k (each if
// inside).  A ring costs only its cells inside.
struct RingShape {
    int64_t gx, count;
    int32_t cx, cy, k, xa, wtop, wbot, mid0, sides;  // sides: 1 left column, 2 right, 3 both
};

__device__ __forceinline__ RingShape ring_shape(const Grid& g, int32_t cx, int32_t cy, int32_t k, int32_t x0,
                                                int32_t x1, int32_t y0, int32_t y1) {
    RingShape R;
    R.gx = g.gx;
    R.cx = cx;
    R.cy = cy;
    R.k = k;
    R.xa = max(cx - k, x0);
    const int32_t w = min(cx + k, x1) - R.xa + 1;
    R.wtop = cy - k >= y0 ? w : 0;
    R.wbot = k > 0 && cy + k <= y1 ? w : 0;
    R.mid0 = max(cy - k + 1, y0);
    const int32_t nmid = k > 0 ? max(min(cy + k - 1, y1) - R.mid0 + 1, 0) : 0;
    R.sides = k > 0 ? (cx - k >= x0 ? 1 : 0) | (cx + k <= x1 ? 2 : 0) : 0;
    R.count = (int64_t)R.wtop + R.wbot + (int64_t)nmid * __popc(R.sides);
    return R;
}

__device__ __forceinline__ int64_t ring_cell(const RingShape& R, int64_t i) {
    if (i < R.wtop) return (int64_t)(R.cy - R.k) * R.gx + R.xa + i;
    i -= R.wtop;
    if (i < R.wbot) return (int64_t)(R.cy + R.k) * R.gx + R.xa + i;
    i -= R.wbot;
    int64_t y;
    int32_t x;
    if (R.sides == 3) {
        y = R.mid0 + (i >> 1);
        x = (i & 1) ? R.cx + R.k : R.cx - R.k;
    } else {
        y = R.mid0 + i;
        x = R.sides == 1 ? R.cx - R.k : R.cx + R.k;
    }
    return y * R.gx + x;
}

// Visit the cells of a ring in order; f(cell) returns true to stop, and then
// so does this (returning true).
template <class F>
__device__ __forceinline__ bool ring_cells(const Grid& g, int32_t cx, int32_t cy, int32_t k, int32_t x0,
                                           int32_t x1, int32_t y0, int32_t y1, F&& f) {
    const RingShape R = ring_shape(g, cx, cy, k, x0, x1, y0, y1);
    for (int64_t i = 0; i < R.count; ++i)
        if (f(ring_cell(R, i))) return true;
    return false;
}

// Cells visited (and points looked at) by the Gabriel searches, counted
// against a thread's budget.
struct Work {
    int64_t n = 0;
};

// No point other than iu, iv in the closed disc with diameter uv.  Cells are
// scanned outwards from the disc's centre, where a blocking point is most
// likely to be.
__device__ bool gabriel_pair_dev(const Grid& g, const int64_t* __restrict__ start,
                                 const int32_t* __restrict__ pts, const float2* __restrict__ p,
                                 int32_t iu, int32_t iv, Work& work) {
    const float2 u = p[iu], v = p[iv];
    const float cx = 0.5f * (u.x + v.x), cy = 0.5f * (u.y + v.y);
    const double dx = (double)v.x - (double)u.x, dy = (double)v.y - (double)u.y;
    // half the diameter, rounded up, plus one cell either way against rounding
    const float r = (float)(0.5 * sqrt(dx * dx + dy * dy)) * 1.0001f + 1e-30f;
    const int32_t x0 = max(cell_x(g, cx - r) - 1, 0), x1 = min(cell_x(g, cx + r) + 1, g.gx - 1);
    const int32_t y0 = max(cell_y(g, cy - r) - 1, 0), y1 = min(cell_y(g, cy + r) + 1, g.gy - 1);
    const int32_t ccx = min(max(cell_x(g, cx), x0), x1), ccy = min(max(cell_y(g, cy), y0), y1);
    const int32_t K = max(max(ccx - x0, x1 - ccx), max(ccy - y0, y1 - ccy));
    for (int32_t k = 0; k <= K; ++k) {
        const bool blocked = ring_cells(g, ccx, ccy, k, x0, x1, y0, y1, [&](int64_t c) {
            ++work.n;
            for (int64_t q = start[c]; q < start[c + 1]; ++q) {
                ++work.n;
                const int32_t w = pts[q];
                if (w != iu && w != iv && in_disc(u, v, p[w])) return true;
            }
            return false;
        });
        if (blocked) return false;
    }
    return true;
}

// octant of the direction (dx, dy), from signs and |dx| vs |dy| only
__device__ __forceinline__ int octant(double dx, double dy) {
    return (dx < 0.0 ? 4 : 0) + (dy < 0.0 ? 2 : 0) + (fabs(dx) < fabs(dy) ? 1 : 0);
}

// The cells of ring k (k >= 4) around (cx, cy) that can hold points of
// octant o, numbered like a ring's.  With (p, q) a cell's index offsets
// along the octant's major and minor axes, signed towards it, a point of the
// octant with true offsets A >= B >= 0 (in cell widths) has |p - A| < 2 and
// |q - B| < 2 (one for its place in the cell, one for a cell index computed
// in float), so p >= -1, q >= -1 and p >= q - 3: on ring k these are p = k
// with q in [-1, k] and q = k with p in [k - 3, k - 1].  Only offsets inside
// the grid are numbered (a degenerate grid of one row would otherwise cost k
// steps per ring).
struct SectorShape {
    int64_t gx, count;
    int32_t c0, c1, s0, s1, k, qa, na, pa;
    bool major_y;
};

__device__ __forceinline__ SectorShape sector_shape(const Grid& g, int32_t cx, int32_t cy, int32_t k, int o) {
    SectorShape S;
    const int32_t sx = (o & 4) ? -1 : 1, sy = (o & 2) ? -1 : 1;
    S.major_y = o & 1;
    S.gx = g.gx;
    S.k = k;
    // centre, extent and sign of the major (0) and minor (1) axes
    S.c0 = S.major_y ? cy : cx;
    S.s0 = S.major_y ? sy : sx;
    S.c1 = S.major_y ? cx : cy;
    S.s1 = S.major_y ? sx : sy;
    const int32_t n0 = S.major_y ? g.gy : g.gx, n1 = S.major_y ? g.gx : g.gy;
    // signed offsets t with c + s t inside [0, n): t in [lo, hi], lo <= 0 <= hi
    auto lo = [](int32_t c, int32_t n, int32_t s) { return s > 0 ? -c : c - (n - 1); };
    auto hi = [](int32_t c, int32_t n, int32_t s) { return s > 0 ? n - 1 - c : c; };
    S.qa = max(-1, lo(S.c1, n1, S.s1));
    S.na = k <= hi(S.c0, n0, S.s0) ? max(min(k, hi(S.c1, n1, S.s1)) - S.qa + 1, 0) : 0;
    S.pa = max(k - 3, lo(S.c0, n0, S.s0));
    const int32_t nb = k <= hi(S.c1, n1, S.s1) ? max(min(k - 1, hi(S.c0, n0, S.s0)) - S.pa + 1, 0) : 0;
    S.count = (int64_t)S.na + nb;
    return S;
}

__device__ __forceinline__ int64_t sector_cell(const SectorShape& S, int64_t i) {
    const int32_t pp = i < S.na ? S.k : S.pa + (int32_t)(i - S.na);
    const int32_t qq = i < S.na ? S.qa + (int32_t)i : S.k;
    const int64_t a = S.c0 + S.s0 * pp, b = S.c1 + S.s1 * qq;
    return S.major_y ? a * S.gx + b : b * S.gx + a;
}

// Full ring, or only the sectors of the octants in `open` when that visits
// fewer cells (k + 5 per octant against 8k).
__device__ __forceinline__ bool use_full_ring(int32_t k, unsigned open) {
    return k <= 3 || (int32_t)__popc(open) * (k + 5) >= 8 * k;
}

// Minimum over aligned groups of G lanes, in every lane of the group.
template <int G>
__device__ __forceinline__ double group_min(double v) {
#pragma unroll
    for (int off = G / 2; off >= 1; off >>= 1) v = fmin(v, __shfl_xor(v, off, 64));
    return v;
}

// Gabriel degree of point iu.  Rings of cells around u find the nearest
// point of each 45-degree octant until the octant is settled; a second walk
// over the same rings (or sectors) tests every point of an octant that is
// not blocked.  The G lanes of an aligned group take the cells of each ring in
// turn (all of them call this for the same point and get the same result).
// With G < 64 the group gives up (returns -1) once a lane has visited more
// than `budget` cells and points.  box = (xmin, xmax, ymin, ymax).
template <int G>
__device__ int32_t gabriel_degree_of(int32_t iu, const Grid& g, const int64_t* __restrict__ start,
                                     const int32_t* __restrict__ pts, const float2* __restrict__ p,
                                     float cell, float4 box, int64_t budget) {
    const int lane = threadIdx.x % G;
    constexpr int stride = G;
    const uint64_t group = G == 64 ? ~0ull : ((1ull << (G & 63)) - 1ull) << (lane64() / G * G);
    const auto any = [&](bool b) { return (__ballot(b) & group) != 0ull; };
    Work work;
    const float2 u = p[iu];
    const int32_t cx = cell_x(g, u.x), cy = cell_y(g, u.y);
    // reach[o]: the largest squared distance from u to a point of the
    // bounding box in octant o (its wedge is bounded by the box edges A
    // along x and B along y; the far corner of the wedge's part inside is at
    // (A, min(A, B)) or (min(A, B), B))
    double reach[8], best[8];
    int32_t ko[8];
    for (int o = 0; o < 8; ++o) {
        const double A = (o & 4) ? (double)u.x - box.x : (double)box.y - u.x;
        const double B = (o & 2) ? (double)u.y - box.z : (double)box.w - u.y;
        const double mn = fmin(A, B);
        reach[o] = ((o & 1) ? B * B : A * A) + mn * mn;
        // an octant that needs dx < 0 (dy < 0) with u on the box's left
        // (lower) edge holds no point at all
        if (((o & 4) && A == 0.0) || ((o & 2) && B == 0.0)) reach[o] = 0.0;
        best[o] = INFINITY;
        ko[o] = 0;
    }
    // f(cell, octant) for this thread's (lane's) cells of ring k: the whole
    // ring (octant -1) or the sectors of the octants in `open`
    auto each_cell = [&](int32_t k, unsigned open, auto&& f) {
        if (use_full_ring(k, open)) {
            const RingShape R = ring_shape(g, cx, cy, k, 0, g.gx - 1, 0, g.gy - 1);
            for (int64_t i = lane; i < R.count; i += stride) f(ring_cell(R, i), -1);
        } else {
            for (int o = 0; o < 8; ++o) {
                if (!(open >> o & 1)) continue;
                const SectorShape S = sector_shape(g, cx, cy, k, o);
                for (int64_t i = lane; i < S.count; i += stride) f(sector_cell(S, i), o);
            }
        }
    };
    // rings beyond kmax lie entirely outside the grid
    const int32_t kmax = max(max(cx, g.gx - 1 - cx), max(cy, g.gy - 1 - cy));
    unsigned open = 0xFFu;  // octants not yet settled
    for (int32_t k = 0; open; ++k) {
        each_cell(k, open, [&](int64_t c, int) {
            ++work.n;
            for (int64_t q = start[c]; q < start[c + 1]; ++q) {
                ++work.n;
                const int32_t w = pts[q];
                if (w == iu) continue;
                const double dx = (double)p[w].x - (double)u.x, dy = (double)p[w].y - (double)u.y;
                const double r2 = dx * dx + dy * dy;
                if (r2 <= 0.0) continue;  // a coincident point has no direction
                const int o = octant(dx, dy);
                best[o] = r2 < best[o] ? r2 : best[o];
            }
        });
        for (int o = 0; o < 8; ++o) best[o] = group_min<G>(best[o]);
        if (G < 64 && any(work.n > budget)) return -1;
        // every point of an octant visited so far within (k - 2) cells' width
        // of u has been seen (a cell index computed in float can be one off);
        // an octant is settled at ring ko once that covers twice its nearest
        // squared distance (beyond, its points are blocked) or, with no point
        // found, its reach (it has none)
        const double cover = k >= 2 ? (double)(k - 2) * (double)cell : 0.0;
        for (int o = 0; o < 8; ++o) {
            if (!(open >> o & 1)) continue;
            const double need = (best[o] < INFINITY ? 2.0 * best[o] : reach[o]) * (1.0 + 1e-9);
            if ((k >= 2 && need <= cover * cover) || k >= kmax) {
                ko[o] = k;
                open &= ~(1u << o);
            }
        }
    }
    int32_t K = 0;
    for (int o = 0; o < 8; ++o) K = max(K, ko[o]);
    // candidates: points of octant o on rings up to ko[o] that are not blocked
    int32_t deg = 0;
    bool over = false;
    for (int32_t k = 0; k <= K && !over; ++k) {
        unsigned live = 0;
        for (int o = 0; o < 8; ++o) live |= (ko[o] >= k ? 1u : 0u) << o;
        each_cell(k, live, [&](int64_t c, int only) {
            if (G < 64 && (over = over || work.n > budget)) return;
            ++work.n;
            for (int64_t q = start[c]; q < start[c + 1]; ++q) {
                ++work.n;
                const int32_t iv = pts[q];
                if (iv == iu) continue;
                const double dx = (double)p[iv].x - (double)u.x, dy = (double)p[iv].y - (double)u.y;
                const double r2 = dx * dx + dy * dy;
                const int o = octant(dx, dy);
                if (r2 > 0.0) {
                    if (only >= 0 ? o != only : !(live >> o & 1)) continue;
                    if (r2 >= 2.0 * best[o] * (1.0 + 1e-9)) continue;  // blocked
                } else if (only > 0) {
                    continue;  // a coincident point is taken once, with octant 0
                }
                deg += gabriel_pair_dev(g, start, pts, p, iu, iv, work) ? 1 : 0;
            }
        });
        if (G < 64) over = any(over);
    }
    return over ? -1 : group_sum<G>(deg);
}

// L lanes per point (in cell order: a wavefront's points are neighbours); a point
// whose search exceeds the budget is listed in hard[] for gabriel_wave_kernel
// instead (gabriel_plan).
template <int L>
__global__ __launch_bounds__(kBlock, 4) void gabriel_degree_kernel(int32_t n, Grid g,
                                                                const int64_t* __restrict__ start,
                                                                const int32_t* __restrict__ pts,
                                                                const float2* __restrict__ p,
                                                                float cell, float4 box, int64_t budget,
                                                                int32_t* __restrict__ gdeg,
                                                                int32_t* __restrict__ hard,
                                                                int32_t* __restrict__ hard_count) {
    for (int64_t t = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / L; t < n;
         t += (int64_t)gridDim.x * (kBlock / L)) {
        const int32_t iu = pts[t];
        const int32_t deg = gabriel_degree_of<L>(iu, g, start, pts, p, cell, box, budget);
        if (threadIdx.x % L != 0) continue;
        if (deg >= 0)
            gdeg[iu] = deg;
        else
            hard[atomicAdd(hard_count, 1)] = iu;
    }
}

// Wavefront per listed point (at most 128 VGPRs, as above).
__global__ __launch_bounds__(kBlock, 4) void gabriel_wave_kernel(Grid g, const int64_t* __restrict__ start,
                                                              const int32_t* __restrict__ pts,
                                                              const float2* __restrict__ p, float cell,
                                                              float4 box, const int32_t* __restrict__ hard,
                                                              const int32_t* __restrict__ hard_count,
                                                              int32_t* __restrict__ gdeg) {
    const int32_t count = *hard_count;
    const int64_t waves = (int64_t)gridDim.x * kWaves;
    for (int64_t i = (int64_t)blockIdx.x * kWaves + wave_id(); i < count; i += waves) {
        const int32_t iu = hard[i];
        const int32_t deg = gabriel_degree_of<64>(iu, g, start, pts, p, cell, box, 0);
        if (lane64() == 0) gdeg[iu] = deg;
    }
}

// Gabriel test of every adjacency entry: inter[v] = graph neighbours of v
// that are Gabriel neighbours.
__global__ __launch_bounds__(kBlock) void gabriel_edge_kernel(int32_t n, Grid g,
                                                              const int64_t* __restrict__ start,
                                                              const int32_t* __restrict__ pts,
                                                              const float2* __restrict__ p,
                                                              const int64_t* __restrict__ rp,
                                                              const int32_t* __restrict__ ci,
                                                              int32_t* __restrict__ inter) {
    const int64_t waves = (int64_t)gridDim.x * kWaves;
    for (int64_t v = (int64_t)blockIdx.x * kWaves + wave_id(); v < n; v += waves) {
        int32_t c = 0;
        Work work;
        for (int64_t e = rp[v] + lane64(); e < rp[v + 1]; e += 64)
            c += gabriel_pair_dev(g, start, pts, p, (int32_t)v, ci[e], work) ? 1 : 0;
        c = wave_sum(c);
        if (lane64() == 0) inter[v] = c;
    }
}

__global__ __launch_bounds__(kBlock) void jaccard_kernel(int32_t n, const int64_t* __restrict__ rp,
                                                         const int32_t* __restrict__ gdeg,
                                                         const int32_t* __restrict__ inter,
                                                         double* __restrict__ jac,
                                                         double* __restrict__ partial,
                                                         unsigned long long* __restrict__ gsum) {
    __shared__ double s[kWaves];
    double acc = 0.0;
    unsigned long long ge = 0;
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * kBlock) {
        const int64_t both = inter[v];
        const int64_t uni = (rp[v + 1] - rp[v]) + gdeg[v] - both;
        const double J = uni == 0 ? 1.0 : (double)both / (double)uni;
        if (jac) jac[v] = J;
        acc += J;
        ge += (unsigned long long)gdeg[v];
    }
    const double t = block_sum(acc, s);
    if (threadIdx.x == 0) partial[blockIdx.x] = t;
    const unsigned long long w = wave_sum(ge);
    if (lane64() == 0 && w) atomicAdd(gsum, w);
}

// Sum of partial[0 .. count) in a fixed order (the same bits on every run):
// thread t adds partial[t], partial[t + 256], ... in turn, then a fixed tree.
__global__ __launch_bounds__(kBlock) void ordered_sum_kernel(int32_t count, const double* __restrict__ partial,
                                                             double* __restrict__ out) {
    __shared__ double s_v[kBlock];
    double a = 0.0;
    for (int32_t i = threadIdx.x; i < count; i += kBlock) a += partial[i];
    s_v[threadIdx.x] = a;
    __syncthreads();
    for (int h = kBlock / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) s_v[threadIdx.x] += s_v[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = s_v[0];
}

template <class V>
static int drawing_metrics(const gila_csr* g, const V* pos, int32_t what, hipStream_t s,
                           gila_metrics* out, int64_t* edge_crossings, double* jaccard) {
    const int32_t n = g->n;
    *out = gila_metrics{};
    out->similarity = 1.0;
    if (n == 0) return GILA_OK;
    MBuf pf(s), first(s), cnt(s), eo(s), ends(s), ws(s);
    GILA_TRY(pf.alloc<float2>((size_t)n));
    hipLaunchKernelGGL(to_float_kernel<V>, dim3(mgrid(n)), dim3(kBlock), 0, s, n, pos, pf.as<float2>());
    GILA_HIP(hipGetLastError());
    // bounding box (finite coordinates only)
    MBuf box(s);
    GILA_TRY(box.alloc<unsigned int>(4));
    GILA_HIP(hipMemsetAsync(box.p, 0xFF, 4 * sizeof(unsigned int), s));
    hipLaunchKernelGGL(bounds_kernel, dim3(mgrid(n)), dim3(kBlock), 0, s, n, pf.as<float2>(),
                       box.as<unsigned int>());
    GILA_HIP(hipGetLastError());
    unsigned int hb[4];
    GILA_HIP(hipMemcpyAsync(hb, box.p, sizeof(hb), hipMemcpyDeviceToHost, s));
    GILA_HIP(hipStreamSynchronize(s));
    auto val = [](unsigned int k) {
        const unsigned int u = (k >> 31) ? (k & 0x7FFFFFFFu) : ~k;
        float f;
        std::memcpy(&f, &u, 4);
        return f;
    };
    const float xmin = val(hb[0]), ymin = val(hb[1]), xmax = -val(hb[2]), ymax = -val(hb[3]);
    if (!std::isfinite(xmin) || !std::isfinite(xmax) || !std::isfinite(ymin) || !std::isfinite(ymax))
        return fail(GILA_EINVAL, "positions must be finite");
    const double M = std::max(std::max(std::fabs((double)xmin), std::fabs((double)xmax)),
                              std::max(std::fabs((double)ymin), std::fabs((double)ymax)));
    // edge list
    GILA_TRY(first.alloc<int64_t>((size_t)n));
    GILA_TRY(cnt.alloc<int64_t>((size_t)n));
    GILA_TRY(eo.alloc<int64_t>((size_t)n + 1));
    GILA_TRY(ws.alloc<int64_t>((size_t)scan_workspace_count(n)));
    hipLaunchKernelGGL(upper_count_kernel, dim3(mgrid(n)), dim3(kBlock), 0, s, n, g->row_ptr,
                       g->col_idx, first.as<int64_t>(), cnt.as<int64_t>());
    GILA_HIP(hipGetLastError());
    GILA_TRY(enqueue_exclusive_scan_i64(cnt.as<int64_t>(), eo.as<int64_t>(), n, ws.as<int64_t>(), s));
    int64_t m = 0;
    GILA_HIP(hipMemcpyAsync(&m, eo.as<int64_t>() + n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    GILA_HIP(hipStreamSynchronize(s));
    GILA_TRY(ends.alloc<int2>((size_t)std::max<int64_t>(m, 1)));
    const int rgrid = (int)std::max<int64_t>(1, std::min<int64_t>(16384, ((int64_t)n + kWaves - 1) / kWaves));
    hipLaunchKernelGGL(edge_list_kernel, dim3(rgrid), dim3(kBlock), 0, s, n, g->row_ptr, g->col_idx,
                       first.as<int64_t>(), eo.as<int64_t>(), ends.as<int2>());
    GILA_HIP(hipGetLastError());
    if ((what & GILA_METRIC_CROSSINGS) && m > 0) {
        MBuf tot(s);
        GILA_TRY(tot.alloc<unsigned long long>(1));
        GILA_HIP(hipMemsetAsync(tot.p, 0, sizeof(unsigned long long), s));
        // groups of 64 edges in the order of their places (row order for few
        // edges, whose pairs cost less than the sort, and for more than the
        // sort's 32-bit places hold)
        const int64_t groups = (m + kCrossGroup - 1) / kCrossGroup;
        MBuf key(s), order(s), seg(s), cbox(s);
        const bool sorted = m >= kCrossSortMin && m < INT32_MAX;
        if (sorted) {
            GILA_TRY(key.alloc<uint32_t>((size_t)m));
            GILA_TRY(order.alloc<int32_t>((size_t)m));
            const float sx = (float)(256.0 / std::max(1e-300, (double)xmax - (double)xmin));
            const float sy = (float)(256.0 / std::max(1e-300, (double)ymax - (double)ymin));
            hipLaunchKernelGGL(cross_key_kernel, dim3(mgrid(m)), dim3(kBlock), 0, s, m, ends.as<int2>(),
                               pf.as<float2>(), make_float2(xmin, ymin), make_float2(sx, sy),
                               key.as<uint32_t>());
            GILA_HIP(hipGetLastError());
            GILA_TRY(stable_order_by_key((int32_t)m, key.as<uint32_t>(), ~0u, order.as<int32_t>(), s));
        }
        const int32_t* by_place = sorted ? order.as<int32_t>() : nullptr;
        GILA_TRY(seg.alloc<float4>((size_t)m));
        GILA_TRY(cbox.alloc<CrossBox>((size_t)groups));
        hipLaunchKernelGGL(cross_prepare_kernel, dim3(mgrid(groups * 64)), dim3(kBlock), 0, s, m, groups,
                           ends.as<int2>(), pf.as<float2>(), by_place, seg.as<float4>(),
                           cbox.as<CrossBox>());
        // about kCrossWaves wavefronts, each one group against a range of `span`
        int64_t span = std::max<int64_t>(1, groups * groups / kCrossWaves);
        span = std::max<int64_t>(span, (groups + 65534) / 65535);
        const dim3 grid((unsigned)((groups + kWaves - 1) / kWaves), (unsigned)((groups + span - 1) / span));
        // rounding of the values that the group verdicts compare; drawings so
        // small or large that their squares leave float's range get none
        const float eps = M > 1e-12 && M < 1e18 ? (float)(0x1p-18 * M * M) : INFINITY;
        if (edge_crossings) {
            GILA_HIP(hipMemsetAsync(edge_crossings, 0, sizeof(int64_t) * (size_t)m, s));
            hipLaunchKernelGGL(crossings_kernel<false>, grid, dim3(kBlock), 0, s, m, groups, span, M, eps,
                               seg.as<float4>(), cbox.as<CrossBox>(), by_place, ends.as<int2>(),
                               pf.as<float2>(),
                               reinterpret_cast<unsigned long long*>(edge_crossings),
                               tot.as<unsigned long long>());
        } else {
            hipLaunchKernelGGL(crossings_kernel<true>, grid, dim3(kBlock), 0, s, m, groups, span, M, eps,
                               seg.as<float4>(), cbox.as<CrossBox>(), by_place, ends.as<int2>(),
                               pf.as<float2>(), nullptr, tot.as<unsigned long long>());
        }
        GILA_HIP(hipGetLastError());
        unsigned long long t = 0;
        GILA_HIP(hipMemcpyAsync(&t, tot.p, sizeof(t), hipMemcpyDeviceToHost, s));
        GILA_HIP(hipStreamSynchronize(s));
        out->crossings = (int64_t)(edge_crossings ? t / 2 : t);
    }
    if ((what & GILA_METRIC_LENGTHS) && m > 0) {
        const int lg = mgrid(m);
        MBuf part(s), sum(s);
        GILA_TRY(part.alloc<double>((size_t)lg));
        GILA_TRY(sum.alloc<double>(1));
        double tot = 0.0;
        hipLaunchKernelGGL(lengths_sum_kernel, dim3(lg), dim3(kBlock), 0, s, m, ends.as<int2>(),
                           pf.as<float2>(), 0.0, 0, part.as<double>());
        hipLaunchKernelGGL(ordered_sum_kernel, dim3(1), dim3(kBlock), 0, s, lg, part.as<double>(), sum.as<double>());
        GILA_HIP(hipMemcpyAsync(&tot, sum.p, sizeof(double), hipMemcpyDeviceToHost, s));
        GILA_HIP(hipStreamSynchronize(s));
        const double mean = tot / (double)m;
        hipLaunchKernelGGL(lengths_sum_kernel, dim3(lg), dim3(kBlock), 0, s, m, ends.as<int2>(),
                           pf.as<float2>(), mean, 1, part.as<double>());
        hipLaunchKernelGGL(ordered_sum_kernel, dim3(1), dim3(kBlock), 0, s, lg, part.as<double>(), sum.as<double>());
        GILA_HIP(hipMemcpyAsync(&tot, sum.p, sizeof(double), hipMemcpyDeviceToHost, s));
        GILA_HIP(hipStreamSynchronize(s));
        out->edge_length_mean = mean;
        out->edge_length_std = std::sqrt(tot / (double)m);
    }
    if (what & GILA_METRIC_SIMILARITY) {
        // grid of about two points per cell over the bounding box
        const double w = std::max(1e-30, (double)xmax - (double)xmin);
        const double h = std::max(1e-30, (double)ymax - (double)ymin);
        double cell = std::sqrt(2.0 * w * h / (double)n);
        cell = std::max(cell, std::max(w, h) / 65536.0);
        cell = std::max(cell, 1e-30);
        Grid gr;
        gr.x0 = xmin;
        gr.y0 = ymin;
        gr.gx = (int32_t)std::min(65536.0, std::floor(w / cell) + 1);
        gr.gy = (int32_t)std::min(65536.0, std::floor(h / cell) + 1);
        gr.inv = (float)(1.0 / cell);
        const int64_t G = (int64_t)gr.gx * gr.gy;
        MBuf cellof(s), ccnt(s), cstart(s), cur(s), pts(s), gdeg(s), inter(s), part(s), sum(s), gs(s),
            ws2(s);
        GILA_TRY(cellof.alloc<int32_t>((size_t)n));
        GILA_TRY(ccnt.alloc<int64_t>((size_t)G));
        GILA_TRY(cstart.alloc<int64_t>((size_t)G + 1));
        GILA_TRY(cur.alloc<unsigned long long>((size_t)G));
        GILA_TRY(pts.alloc<int32_t>((size_t)n));
        GILA_TRY(gdeg.alloc<int32_t>((size_t)n));
        GILA_TRY(inter.alloc<int32_t>((size_t)n));
        GILA_TRY(ws2.alloc<int64_t>((size_t)scan_workspace_count(G)));
        GILA_HIP(hipMemsetAsync(ccnt.p, 0, sizeof(int64_t) * G, s));
        GILA_HIP(hipMemsetAsync(cur.p, 0, sizeof(unsigned long long) * G, s));
        hipLaunchKernelGGL(cell_count_kernel, dim3(mgrid(n)), dim3(kBlock), 0, s, n, gr, pf.as<float2>(),
                           cellof.as<int32_t>(), ccnt.as<int64_t>());
        GILA_HIP(hipGetLastError());
        GILA_TRY(enqueue_exclusive_scan_i64(ccnt.as<int64_t>(), cstart.as<int64_t>(), G,
                                            ws2.as<int64_t>(), s));
        hipLaunchKernelGGL(cell_fill_kernel, dim3(mgrid(n)), dim3(kBlock), 0, s, n, cellof.as<int32_t>(),
                           cstart.as<int64_t>(), cur.as<unsigned long long>(), pts.as<int32_t>());
        // (GILA_GABRIEL_BUDGET overrides the budget; 0 sends every point to a
        // wavefront of its own)
        const GabrielPlan plan = gabriel_plan(n);
        int64_t budget = plan.budget;
        if (const char* e = getenv("GILA_GABRIEL_BUDGET")) budget = std::max<int64_t>(0, std::atoll(e));
        MBuf hard(s), hcount(s);
        GILA_TRY(hard.alloc<int32_t>((size_t)n));
        GILA_TRY(hcount.alloc<int32_t>(1));
        GILA_HIP(hipMemsetAsync(hcount.p, 0, sizeof(int32_t), s));
        const float4 fbox = make_float4(xmin, xmax, ymin, ymax);
        const auto degrees = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(mgrid((int64_t)n * plan.lanes)), dim3(kBlock), 0, s, n, gr,
                               cstart.as<int64_t>(), pts.as<int32_t>(), pf.as<float2>(), (float)cell, fbox,
                               budget, gdeg.as<int32_t>(), hard.as<int32_t>(), hcount.as<int32_t>());
        };
        if (plan.lanes == 8) degrees(gabriel_degree_kernel<8>);
        else if (plan.lanes == 2) degrees(gabriel_degree_kernel<2>);
        else degrees(gabriel_degree_kernel<1>);
        hipLaunchKernelGGL(gabriel_wave_kernel, dim3(mgrid((int64_t)n * 64)), dim3(kBlock), 0, s, gr,
                           cstart.as<int64_t>(), pts.as<int32_t>(), pf.as<float2>(), (float)cell, fbox,
                           hard.as<int32_t>(), hcount.as<int32_t>(), gdeg.as<int32_t>());
        hipLaunchKernelGGL(gabriel_edge_kernel, dim3(rgrid), dim3(kBlock), 0, s, n, gr,
                           cstart.as<int64_t>(), pts.as<int32_t>(), pf.as<float2>(), g->row_ptr,
                           g->col_idx, inter.as<int32_t>());
        GILA_HIP(hipGetLastError());
        const int jg = mgrid(n);
        GILA_TRY(part.alloc<double>((size_t)jg));
        GILA_TRY(sum.alloc<double>(1));
        GILA_TRY(gs.alloc<unsigned long long>(1));
        GILA_HIP(hipMemsetAsync(gs.p, 0, sizeof(unsigned long long), s));
        hipLaunchKernelGGL(jaccard_kernel, dim3(jg), dim3(kBlock), 0, s, n, g->row_ptr, gdeg.as<int32_t>(),
                           inter.as<int32_t>(), jaccard, part.as<double>(), gs.as<unsigned long long>());
        hipLaunchKernelGGL(ordered_sum_kernel, dim3(1), dim3(kBlock), 0, s, jg, part.as<double>(), sum.as<double>());
        GILA_HIP(hipGetLastError());
        double tot = 0.0;
        unsigned long long ge = 0;
        GILA_HIP(hipMemcpyAsync(&tot, sum.p, sizeof(double), hipMemcpyDeviceToHost, s));
        GILA_HIP(hipMemcpyAsync(&ge, gs.p, sizeof(ge), hipMemcpyDeviceToHost, s));
        GILA_HIP(hipStreamSynchronize(s));
        out->similarity = tot / (double)n;
        out->gabriel_edges = (int64_t)(ge / 2);
    }
    out->edges = m;
    GILA_HIP(hipStreamSynchronize(s));
    return GILA_OK;
}

}  // namespace gila

using namespace gila;

extern "C" {

int gila_drawing_metrics(const gila_csr* g_dev, int32_t precision, const void* pos_dev,
                         int32_t what, void* stream, gila_metrics* out,
                         int64_t* edge_crossings_dev, double* jaccard_dev) {
    TraceRange trace_range("gila_drawing_metrics");
    clear_error();
    SettleOnReturn settle(stream);
    if (!out) return fail(GILA_EINVAL, "out is NULL");
    if (precision != GILA_FP64 && precision != GILA_FP32 && precision != GILA_FP32_KAHAN)
        return fail(GILA_EINVAL, "unknown precision %d", precision);
    hipStream_t s = (hipStream_t)stream;
    GILA_TRY(validate_graph(g_dev, s));
    if (g_dev->n > 0 && !pos_dev) return fail(GILA_EINVAL, "pos_dev is NULL");
    if (precision == GILA_FP64)
        return drawing_metrics<double2>(g_dev, (const double2*)pos_dev, what, s, out,
                                        edge_crossings_dev, jaccard_dev);
    return drawing_metrics<float2>(g_dev, (const float2*)pos_dev, what, s, out, edge_crossings_dev,
                                   jaccard_dev);
}

}  // extern "C"
