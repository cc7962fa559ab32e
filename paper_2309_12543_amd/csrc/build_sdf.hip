// Link SDF construction (Sec. III-A: per-link signed distance fields
// precomputed on the link's local grid) and training labels: the exact signed
// distance from a point to a link mesh.
//   * unsigned distance: closest point on a triangle by the Voronoi regions of
//     Ericson, Real-Time Collision Detection (2005), Sec. 5.1.5;
//   * inside/outside: a part whose edges all cancel (a closed part) has an
//     integer winding number, counted as signed crossings of an upward ray;
//     any other part takes the generalised winding number (Jacobson et al.
//     2013), the sum of signed solid angles (Van Oosterom & Strackee 1983)
//     over 4 pi, above 1/2;
//   * a link made of several parts takes the minimum over parts.
// One lane per point.  Every point against every triangle is bound by FP32
// VALU issue (about 120 instructions for a distance and 170 for a solid angle
// with its three roots and arctangent), so the work is cut instead: triangles
// are staged in LDS with a box per group of 2 and per 16, a lane only takes the
// groups whose box lies nearer than its best distance so far (its nearest group
// first), and the wave's (point, group) pairs go through queues in LDS, 64 at
// a time, so that lanes with few groups do not wait for lanes with many.  Seven
// 64^3 grids of 268 to 524 triangles a link: 4.40 ms of kernels with every
// triangle for every node, 0.492 ms now (58 % VALU busy); the labels of 7 x 262,144
// samples 4.70 -> 0.326 ms (90 %).  The costliest waves are those near a
// part's axis, where every triangle is about as near as the next; the calls
// that take several links run them in one launch, so one link's last waves
// overlap the next link's.
#include <algorithm>

#include "grid_sample.hpp"

namespace {

using namespace lsdf;

// Threads of a workgroup.  A launch of few workgroups takes small ones: each SIMD
// then has one wave to issue for instead of two, on twice the CUs.  One that fills
// the chip takes large ones, as every workgroup stages the mesh for itself and two
// are all that fit a CU; so does one with a mesh that small ones stage in more than
// one go.  In us, with 512 and 256 threads: 31 triangles that are not closed on 16^3
// nodes 34.5 and 30.1 (8 and 16 workgroups), 63 on 32^3 53.9 and 46.2, their labels
// at 500 points 56.2 and 44.4; a box on 16^3 14.5 and 13.8, closed 256 triangles on
// 32^3 46.0 and 44.2; but on 64^3, 1,024 workgroups of 256, a box 18.5 and 28.4, and
// closed 512 triangles on 32^3 71.4 and 73.5.
constexpr int kBlock = 512, kSmallBlock = 256;
constexpr int64_t kMostSmall = 256;   // small workgroups of a launch: one a CU
constexpr int kWavesPerSimd = 4;   // two workgroups a CU: 128 registers a lane, 80 KB of LDS a workgroup

struct BuildArgs {
    int32_t comp_first[LSDF_MAX_COMPONENTS + 1];
    float lo[3];
    float h[3];
    int32_t n[3];
    int32_t ncomp;
    int32_t nv;
    int32_t dtype;       // storage type of the output grid
    int32_t bricks;      // waves take bricks of nodes rather than runs of x
    int32_t blocks;      // workgroups of this link's grid
    const float* verts;
    const int32_t* tris;
    void* out;
};

struct V3 {
    float x, y, z;
};
__device__ inline V3 sub(V3 a, V3 b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ inline float dot(V3 a, V3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ inline float fdot(V3 a, V3 b) { return fmaf(a.x, b.x, fmaf(a.y, b.y, a.z * b.z)); }
__device__ inline V3 cross(V3 a, V3 b) { return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x}; }

// u v - x y within 2 units in the last place whatever cancels (Kahan's difference
// of products).
__device__ inline float diff_of_products(float u, float v, float x, float y) {
    const float m = x * y;
    return fmaf(u, v, -m) + fmaf(-x, y, m);
}

// Squared distance from p to triangle (a, b, c), by the Voronoi regions of
// its vertices, edges and face: the closest point is a + v ab + w ac, or b + w bc
// on edge bc, or a vertex itself, with v and w quotients over one denominator,
// which the first region whose condition holds gives (selected from the last to
// the first; a negative denominator marks what starts from b, or is c).  A
// condition is one compare of a minimum: comparisons combined in scalar registers
// left a wave waiting on the scalar unit for most of the 1,500 cycles a triangle
// took.
// Over grids of an arm's links, against double precision: with plain cross terms
// the face's point strayed along the face by up to 2 um beside thin triangles, and
// bc's as a + v ab + w ac rounds twice and leaves the edge; root mean square error
// 3.30e-9 m (3.11e-9 where every region has a division, products and sums of its
// own) and 6e-7 at worst, 2 um from the surface.  3.02e-9 and 6e-8 so, for 4 % of a
// grid's time.
__device__ inline float dist2_point_triangle(V3 p, V3 a, V3 b, V3 c) {
    constexpr float kFromB = -1.0f, kAtC = -3e38f;   // denominators that mark a vertex
    const V3 ab = sub(b, a), ac = sub(c, a), ap = sub(p, a), bp = sub(p, b), cp = sub(p, c);
    const float d1 = fdot(ab, ap), d2 = fdot(ac, ap);
    const float d3 = fdot(ab, bp), d4 = fdot(ac, bp);
    const float d5 = fdot(ab, cp), d6 = fdot(ac, cp);
    const float vc = diff_of_products(d1, d4, d3, d2);
    const float vb = diff_of_products(d5, d2, d1, d6);
    const float va = diff_of_products(d3, d6, d5, d4);
    const float e43 = d4 - d3, e56 = d5 - d6, s = va + vb + vc;
    // the face; a degenerate triangle (s <= 0) takes a: its edges come first
    float v = vb, w = vc, den = s;
    auto take = [&](bool on, float v_, float w_, float den_) {
        v = on ? v_ : v;
        w = on ? w_ : w;
        den = on ? den_ : den;
    };
    take(s <= 0.0f, 0.0f, 0.0f, 1.0f);
    take(fminf(-va, fminf(e43, e56)) >= 0.0f, 0.0f, -e43, -(e43 + e56));   // edge bc
    take(fminf(-vb, fminf(d2, -d6)) >= 0.0f, 0.0f, d2, d2 - d6);           // edge ac
    take(fminf(d6, -e56) >= 0.0f, 0.0f, 0.0f, kAtC);                       // c
    take(fminf(-vc, fminf(d1, -d3)) >= 0.0f, d1, 0.0f, d1 - d3);           // edge ab
    take(fminf(d3, -e43) >= 0.0f, 0.0f, 0.0f, kFromB);                     // b
    take(fmaxf(d1, d2) <= 0.0f, 0.0f, 0.0f, 1.0f);                         // a
    // quotients rounded as divisions, from one reciprocal (Markstein)
    const float inv = 1.0f / den;
    auto over_den = [&](float x) {
        const float q = x * inv;
        return fmaf(fmaf(-q, den, x), inv, q);
    };
    v = over_den(v);
    w = over_den(w);
    const bool from_b = den < 0.0f;
    const V3 o = den == kAtC ? c : from_b ? b : a, e = from_b ? sub(c, b) : ac;
    // the point itself rounds with the mesh's size, p - o would with p's distance
    const V3 d = sub(p, {fmaf(w, e.x, fmaf(v, ab.x, o.x)), fmaf(w, e.y, fmaf(v, ab.y, o.y)),
                         fmaf(w, e.z, fmaf(v, ab.z, o.z))});
    return fdot(d, d);
}

// Signed solid angle of triangle (a, b, c) seen from p:
// tan(Omega/2) = det[A B C] / (|A||B||C| + (A.B)|C| + (A.C)|B| + (B.C)|A|).
__device__ float solid_angle(V3 p, V3 a, V3 b, V3 c) {
    const V3 A = sub(a, p), B = sub(b, p), C = sub(c, p);
    const float det = dot(A, cross(B, C));
    const float la = sqrtf(dot(A, A)), lb = sqrtf(dot(B, B)), lc = sqrtf(dot(C, C));
    const float den = la * lb * lc + dot(A, B) * lc + dot(A, C) * lb + dot(B, C) * la;
    return 2.0f * atan2f(det, den);
}

// u x v in the plane, within 2 units in the last place whatever cancels (Kahan's
// difference of products): its sign, and where it is 0, are exact.
__device__ inline double cross2(double ux, double uy, double vx, double vy) {
    const double w = uy * vx;
    return fma(ux, vy, -w) + fma(-uy, vx, w);
}

// Crossings of triangle (a, b, c) by the ray from p along +z, signed: +1
// leaving through it, -1 entering.  The planar winding of the triangle's
// shadow around p uses the half-open rule and an edge term whose sign is exact,
// so two triangles that share an edge agree on it and the crossings of a closed
// part add up to its winding number.  Where it is not 0 the three terms are of
// one sign, and the height at which the ray crosses the triangle's plane is the
// corners' mean weighted by them, a sum without cancellation among the weights:
// however thin the shadow, only within rounding of the surface itself can its
// sign be wrong.  (In FP32 the shadow of a vertical triangle is a sliver of
// rounding width, in which a point level with the triangle but beside it was
// called inside the part, by up to 15 cm on a wedge's end.)  The differences
// round in double at most, alike for every triangle at a vertex.
__device__ inline int crossing(V3 p, V3 a, V3 b, V3 c) {
    const double px = p.x, py = p.y, pz = p.z;
    const double ax = a.x - px, ay = a.y - py, bx = b.x - px, by = b.y - py, cx = c.x - px, cy = c.y - py;
    const double ab = cross2(ax, ay, bx, by), bc = cross2(bx, by, cx, cy), ca = cross2(cx, cy, ax, ay);
    const int la = ay <= 0.0, lb = by <= 0.0, lc = cy <= 0.0;
    // +1 for an edge that passes p on its right going up, -1 going down
    auto edge = [](double e, int turn) { return e * turn > 0.0 ? turn : 0; };
    const int w = edge(ab, la - lb) + edge(bc, lb - lc) + edge(ca, lc - la);
    const double height = fma(bc, a.z - pz, fma(ca, b.z - pz, ab * (c.z - pz)));
    return w * height > 0.0 ? w : 0;
}

constexpr int kStage = 1024;           // triangle slots in LDS (a larger mesh takes several rounds)
constexpr int kGroup = 2;              // triangles per box
constexpr int kSuper = 16;             // triangles per outer box
constexpr int kWaves = kBlock / 64;
constexpr int kScan = 8;               // outer boxes looked at together
constexpr int kNoPair = 0xffff;        // no (lane, group) pair has this number

struct MeshLds {
    float4 tri_a[kStage], tri_b[kStage];        // a, b and two of c: 9 floats in 3 aligned loads
    float tri_c[kStage];
    // boxes: lo.x, lo.y, lo.z, hi.x | hi.y, hi.z
    float4 group_a[kStage / kGroup], super_a[kStage / kSuper];
    float2 group_b[kStage / kGroup], super_b[kStage / kSuper];
    uint32_t best[kWaves][64];                  // squared distance of each lane's point (float bits, >= 0)
    int32_t count[kWaves][64];                  // crossings of each lane's point; its first group
    uint16_t outer[kWaves][64 + kScan * 64];    // (lane, outer box) pairs waiting: lane | box << 6
    uint16_t inner[kWaves][64 + kSuper / kGroup * 64];   // (lane, box) pairs waiting
    uint32_t part_lo[LSDF_MAX_COMPONENTS][3];   // the parts' boxes, order-preserving bits
    uint32_t part_hi[LSDF_MAX_COMPONENTS][3];
    uint32_t loose[LSDF_MAX_COMPONENTS][2];     // the parts' edge sums: 0 when every edge cancels
};

// Orders LDS accesses of one wave's lanes (the hardware keeps them in order;
// this keeps the compiler from moving them).
__device__ inline void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ inline uint32_t mix32(uint32_t h) {   // two multiply-xorshift rounds (odd multipliers, digits of pi: a bijection)
    h ^= h >> 16;
    h *= 0x243f6a89u;
    h ^= h >> 15;
    h *= 0x85a308d3u;
    return h ^ (h >> 16);
}

// Term of directed edge u -> v in a part's edge sum: the opposite edge's term
// negated, so the sum over a part is 0 exactly when every directed edge meets
// its opposite (up to a 2^-64 chance over the two sums).
__device__ inline uint32_t edge_term(uint32_t u, uint32_t v) {
    constexpr uint32_t k = 0x13198a2fu;
    return mix32(u + k * v) - mix32(v + k * u);
}

// One vertex index, clamped into range: a bad mesh gives a wrong grid, never
// an out-of-bounds read.
__device__ inline int vertex_index(const BuildArgs& p, int k) { return min(max(p.tris[k], 0), p.nv - 1); }

// Edge sums of part comp into s.loose: over vertex indices, or over vertex
// positions (a part whose triangles repeat their vertices).  The whole
// workgroup, between barriers of the caller's.
template <int BLOCK>
__device__ void edge_sums(const BuildArgs& p, MeshLds& s, int comp, bool positions) {
    uint32_t sum[2] = {0u, 0u};
    for (int t = p.comp_first[comp] + threadIdx.x; t < p.comp_first[comp + 1]; t += BLOCK) {
        uint32_t h[2][3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const int vi = vertex_index(p, 3 * t + c);
            uint32_t id = (uint32_t)vi, id2 = (uint32_t)vi;
            if (positions) {
                id = id2 = 0u;
                for (int a = 0; a < 3; ++a) {   // + 0: -0 and +0 are one position
                    const uint32_t bits = __float_as_uint(p.verts[3 * vi + a] + 0.0f);
                    id = mix32(id + bits);
                    id2 = mix32(id2 + bits * 0x03707345u);
                }
            }
            h[0][c] = id * 0xa4093823u;
            h[1][c] = id2 * 0x299f31d1u + 0x082efa99u;
        }
#pragma unroll
        for (int q = 0; q < 2; ++q)
            sum[q] += edge_term(h[q][0], h[q][1]) + edge_term(h[q][1], h[q][2]) + edge_term(h[q][2], h[q][0]);
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) sum[q] += __shfl_xor(sum[q], o, 64);
        if ((threadIdx.x & 63) == 0 && sum[q] != 0u) atomicAdd(&s.loose[comp][q], sum[q]);
    }
}

__device__ inline int padded_slots(int n) { return (n + kSuper - 1) / kSuper * kSuper; }

// The triangles of part comp from its triangle `first` on, at most cnt, into
// slots from slot0 (a multiple of kSuper) on, with their boxes.  The last
// outer box's empty slots repeat the last triangle.  The whole workgroup,
// between barriers of the caller's; returns the slots taken.
template <int BLOCK>
__device__ int stage_triangles(const BuildArgs& p, MeshLds& s, int comp, int first, int cnt, int slot0) {
    const int padded = padded_slots(cnt);
    for (int k = threadIdx.x; k < padded; k += BLOCK) {   // whole outer boxes: 16 adjacent lanes
        const int t = p.comp_first[comp] + first + min(k, cnt - 1);
        float v[9];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const int vi = vertex_index(p, 3 * t + c);
#pragma unroll
            for (int a = 0; a < 3; ++a) v[3 * c + a] = p.verts[3 * vi + a];
        }
        const int slot = slot0 + k;
        s.tri_a[slot] = make_float4(v[0], v[1], v[2], v[3]);
        s.tri_b[slot] = make_float4(v[4], v[5], v[6], v[7]);
        s.tri_c[slot] = v[8];
        float lo[3], hi[3], e = 0.0f;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            lo[a] = fminf(v[a], fminf(v[3 + a], v[6 + a]));
            hi[a] = fmaxf(v[a], fmaxf(v[3 + a], v[6 + a]));
            e = fmaxf(e, fmaxf(fabsf(lo[a]), fabsf(hi[a])));
        }
        // widened by 32 units in the last place of the largest coordinate,
        // beyond the rounding of a closest point
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            lo[a] -= 4e-6f * e;
            hi[a] += 4e-6f * e;
        }
#pragma unroll
        for (int o = 1; o < kSuper; o <<= 1) {
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                lo[a] = fminf(lo[a], __shfl_xor(lo[a], o, 64));
                hi[a] = fmaxf(hi[a], __shfl_xor(hi[a], o, 64));
            }
            if (2 * o == kGroup && slot % kGroup == 0) {
                s.group_a[slot / kGroup] = make_float4(lo[0], lo[1], lo[2], hi[0]);
                s.group_b[slot / kGroup] = make_float2(hi[1], hi[2]);
            }
        }
        if (slot % kSuper == 0) {
            s.super_a[slot / kSuper] = make_float4(lo[0], lo[1], lo[2], hi[0]);
            s.super_b[slot / kSuper] = make_float2(hi[1], hi[2]);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                atomicMin(&s.part_lo[comp][a], ordered_bits(lo[a]));
                atomicMax(&s.part_hi[comp][a], ordered_bits(hi[a]));
            }
        }
    }
    return padded;
}

__device__ inline V3 point_of(V3 p, int lane) { return {__shfl(p.x, lane, 64), __shfl(p.y, lane, 64), __shfl(p.z, lane, 64)}; }

struct Tri {
    V3 a, b, c;
};
__device__ inline Tri read_triangle(const MeshLds& s, int slot) {
    const float4 u = s.tri_a[slot], v = s.tri_b[slot];
    const float w = s.tri_c[slot];
    return {{u.x, u.y, u.z}, {u.w, v.x, v.y}, {v.z, v.w, w}};
}

// A lower bound of the squared distance from p to a box's triangles.
__device__ inline float box_dist2(const float4& a, const float2& b, V3 p) {
    const float x = fmaxf(fmaxf(a.x - p.x, p.x - a.w), 0.0f);
    const float y = fmaxf(fmaxf(a.y - p.y, p.y - b.x), 0.0f);
    const float z = fmaxf(fmaxf(a.z - p.z, p.z - b.y), 0.0f);
    return (x * x + y * y + z * z) * 0.99999f;
}

// May the upward ray from p meet a box's triangles?
__device__ inline bool ray_meets(const float4& a, const float2& b, V3 p) {
    return fmaxf(fmaxf(fmaxf(a.x - p.x, p.x - a.w), fmaxf(a.y - p.y, p.y - b.x)), p.z - b.y) <= 0.0f;
}

// Finds the (point, group) pairs a wave wants: want(outer box) is asked of
// every lane for outer boxes [first, last), then wanted(point, its lane, group)
// for the groups of those that answered.  Both kinds of pairs wait in queues
// of the wave's; batch(queue, count) gets the wanted ones, 64 at a time (the
// last ones fewer), whichever lanes they came from.  ni pairs wait already.
// One loop with one place for each action: inlined at several, the kernel
// outgrew the instruction cache and its registers.
template <typename Outer, typename Inner, typename Batch>
__device__ inline void queue_groups(MeshLds& s, int first, int last, int ni, V3 p, Outer want, Inner wanted,
                                    Batch batch) {
    const int lane = threadIdx.x & 63;
    const uint64_t below = (1ull << lane) - 1;
    uint16_t* outer = s.outer[threadIdx.x >> 6];
    uint16_t* inner = s.inner[threadIdx.x >> 6];
    int no = 0;   // pairs with an outer box waiting; all counts are wave-uniform
    for (int o = first;;) {
        const bool scanned = o >= last;
        if (ni >= 64 || (scanned && no == 0 && ni > 0)) {
            const int cnt = min(ni, 64);
            ni -= cnt;
            wave_fence();
            batch(inner + ni, cnt);
            wave_fence();
        } else if (no >= 64 || (scanned && no > 0)) {
            const int cnt = min(no, 64);
            no -= cnt;
            wave_fence();
            const bool on = lane < cnt;
            const int e = on ? outer[no + lane] : lane;
            const V3 pt = point_of(p, e & 63);
            bool w[kSuper / kGroup];
#pragma unroll
            for (int j = 0; j < kSuper / kGroup; ++j) w[j] = on && wanted(pt, e & 63, (e >> 6) * (kSuper / kGroup) + j);
#pragma unroll
            for (int j = 0; j < kSuper / kGroup; ++j) {
                const uint64_t m = __ballot(w[j]);
                if (w[j])
                    inner[ni + __builtin_popcountll(m & below)] =
                        (uint16_t)((e & 63) | ((e >> 6) * (kSuper / kGroup) + j) << 6);
                ni += __builtin_popcountll(m);
            }
        } else if (!scanned) {
            // kScan outer boxes at a time, their loads in flight together
            bool w[kScan];
#pragma unroll
            for (int j = 0; j < kScan; ++j) w[j] = want(min(o + j, last - 1));
#pragma unroll
            for (int j = 0; j < kScan; ++j) {
                const bool on = w[j] && o + j < last;
                const uint64_t m = __ballot(on);
                if (on) outer[no + __builtin_popcountll(m & below)] = (uint16_t)(lane | (o + j) << 6);
                no += __builtin_popcountll(m);
            }
            o += kScan;
        } else {
            break;
        }
    }
}

// The smallest squared distance from q to group g's triangles, which are
// taken side by side: one after another, a lone wave took 2,000 cycles for
// each, waiting on the one chain of dependent operations.
__device__ inline float group_dist2(const MeshLds& s, V3 q, int g) {
    float d = INFINITY;
#pragma unroll
    for (int k = 0; k < kGroup; ++k) {
        const Tri t = read_triangle(s, kGroup * g + k);
        d = fminf(d, dist2_point_triangle(q, t.a, t.b, t.c));
    }
    return d;
}

// Lowers b2, the squared distance from pt to triangles seen before, by those
// in slots [lo, hi) of [0, slots) (multiples of kSuper), for the lanes with go.
__device__ inline void nearest(MeshLds& s, int slots, V3 pt, bool go, int lo, int hi, float& b2) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    lo /= kSuper;
    hi /= kSuper;
    // the lane's nearest outer box, and the nearest group in it, first
    float near2 = INFINITY;
    int near = lo;
#pragma unroll 8
    for (int o = 0; o < slots / kSuper; ++o) {
        const float l = box_dist2(s.super_a[o], s.super_b[o], pt);
        const float in = (uint32_t)(o - lo) < (uint32_t)(hi - lo) ? l : INFINITY;
        near = in < near2 ? o : near;
        near2 = fminf(near2, in);
    }
    go = go && near2 <= b2;
    const uint64_t m = __ballot(go);
    if (m == 0) return;
    int seed = near * (kSuper / kGroup);
    float seed2 = INFINITY;
#pragma unroll
    for (int j = 0; j < kSuper / kGroup; ++j) {
        const int g = near * (kSuper / kGroup) + j;
        const float l = box_dist2(s.group_a[g], s.group_b[g], pt);
        if (l < seed2) {
            seed2 = l;
            seed = g;
        }
    }
    s.best[wave][lane] = __float_as_uint(b2);
    s.count[wave][lane] = seed;
    float reach = go ? b2 : -1.0f;   // no box lies nearer than -1
    const int seeds = __builtin_popcountll(m);
    if (go) s.inner[wave][__builtin_popcountll(m & ((1ull << lane) - 1))] = (uint16_t)(lane | seed << 6);
    // the seeds are a first, part-filled batch: 64 pairs with fillers
    if (lane >= seeds) s.inner[wave][lane] = kNoPair;
    queue_groups(
        s, 0, slots / kSuper, 64, pt,
        [&](int o) {
            const float l = (uint32_t)(o - lo) < (uint32_t)(hi - lo) ? box_dist2(s.super_a[o], s.super_b[o], pt) : NAN;
            return l <= reach;
        },
        [&](V3 q, int from, int g) {
            return g != s.count[wave][from] &&
                   box_dist2(s.group_a[g], s.group_b[g], q) <= __uint_as_float(s.best[wave][from]);
        },
        [&](const uint16_t* queue, int cnt) {
            const int pair = lane < cnt ? queue[lane] : kNoPair;
            const int e = pair == kNoPair ? lane : pair;
            const V3 q = point_of(pt, e & 63);
            if (pair != kNoPair) atomicMin(&s.best[wave][e & 63], __float_as_uint(group_dist2(s, q, e >> 6)));
            wave_fence();
            if (go) b2 = reach = __uint_as_float(s.best[wave][lane]);
        });
}

// Signed distance of pt to the mesh.  Every lane of the workgroup takes part
// in staging; lanes with want == false take no triangles.
template <int BLOCK>
__device__ inline float mesh_sdf(const BuildArgs& p, MeshLds& s, V3 pt, bool want) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int slots = 0;
    for (int c = 0; c < p.ncomp; ++c) slots += padded_slots(p.comp_first[c + 1] - p.comp_first[c]);
    const bool whole = slots <= kStage;   // the mesh is staged once, else a part's kStage triangles at a time
    for (int k = threadIdx.x; k < 3 * LSDF_MAX_COMPONENTS; k += BLOCK) {
        s.part_lo[k / 3][k % 3] = 0xffffffffu;
        s.part_hi[k / 3][k % 3] = 0u;
        if (k < 2 * LSDF_MAX_COMPONENTS) s.loose[k / 2][k % 2] = 0u;
    }
    __syncthreads();
    for (int c = 0, at = 0; c < p.ncomp; ++c) {
        edge_sums<BLOCK>(p, s, c, false);
        if (whole) at += stage_triangles<BLOCK>(p, s, c, 0, p.comp_first[c + 1] - p.comp_first[c], at);
    }
    __syncthreads();
    uint32_t open = 0;   // parts whose indices do not cancel: their positions may
    for (int c = 0; c < p.ncomp; ++c)
        if (s.loose[c][0] != 0u || s.loose[c][1] != 0u) open |= 1u << c;
    if (open) {
        __syncthreads();
        if (threadIdx.x < 2 * LSDF_MAX_COMPONENTS) s.loose[threadIdx.x / 2][threadIdx.x % 2] = 0u;
        __syncthreads();
        for (int c = 0; c < p.ncomp; ++c)
            if (open >> c & 1) edge_sums<BLOCK>(p, s, c, true);
        __syncthreads();
    }

    // the signs: the parts pt is inside of
    uint32_t inside = 0;
    for (int c = 0, at = 0; c < p.ncomp; ++c) {
        const int nt = p.comp_first[c + 1] - p.comp_first[c];
        const int step = whole ? nt : kStage;
        const bool closed = s.loose[c][0] == 0u && s.loose[c][1] == 0u;
        float omega = 0.0f;
        int crossed = 0;
        for (int first = 0; first < nt; first += step) {
            const int cnt = min(step, nt - first);
            if (!whole) {
                __syncthreads();   // the triangles staged before are done with
                stage_triangles<BLOCK>(p, s, c, first, cnt, 0);
                __syncthreads();
            }
            if (!closed) {
                if (want)
                    for (int k = at; k < at + cnt; ++k) {
                        const Tri t = read_triangle(s, k);
                        omega += solid_angle(pt, t.a, t.b, t.c);
                    }
                continue;
            }
            // outside a closed part's box (known once it is staged whole) its winding number is 0
            const bool in_box =
                want && (!whole || (pt.x >= from_ordered_bits(s.part_lo[c][0]) && pt.x <= from_ordered_bits(s.part_hi[c][0]) &&
                                    pt.y >= from_ordered_bits(s.part_lo[c][1]) && pt.y <= from_ordered_bits(s.part_hi[c][1]) &&
                                    pt.z >= from_ordered_bits(s.part_lo[c][2]) && pt.z <= from_ordered_bits(s.part_hi[c][2])));
            if (!__ballot(in_box)) continue;
            s.count[wave][lane] = 0;
            queue_groups(
                s, at / kSuper, (at + padded_slots(cnt)) / kSuper, 0, pt,
                [&](int o) { return in_box && ray_meets(s.super_a[o], s.super_b[o], pt); },
                [&](V3 q, int, int g) { return ray_meets(s.group_a[g], s.group_b[g], q); },
                [&](const uint16_t* queue, int n) {
                    const int e = lane < n ? queue[lane] : lane;
                    const V3 q = point_of(pt, e & 63);
                    int w = 0;
#pragma unroll
                    for (int k = 0; k < kGroup; ++k) {
                        const int slot = kGroup * (e >> 6) + k;
                        const Tri t = read_triangle(s, slot);
                        const int x = crossing(q, t.a, t.b, t.c);
                        w += slot < at + cnt ? x : 0;   // not the repeated last triangle
                    }
                    if (lane < n && w != 0) atomicAdd(&s.count[wave][e & 63], w);
                });
            crossed += s.count[wave][lane];
        }
        if (closed ? crossed > 0 : omega * (float)(0.25 / M_PI) > 0.5f) inside |= 1u << c;
        if (whole) at += padded_slots(nt);
    }

    // the distances: of a point outside every part to the nearest triangle of
    // all, of one inside some to the farthest of those parts.  A mesh staged
    // whole takes one pass, each lane over the slots it wants (and more while
    // a lane is inside further parts); a larger one a pass per round.
    float out2 = INFINITY, in2 = -1.0f, part2 = INFINITY;
    uint32_t left = inside;
    for (int c = 0, first = 0; c < p.ncomp;) {
        int lo = 0, hi = slots;
        bool go = want, last = true;
        if (whole) {
            const int part = left ? __builtin_ctz(left) : -1;
            left &= left - 1u;
            for (int k = 0, at = 0; k < p.ncomp; ++k) {
                const int n = padded_slots(p.comp_first[k + 1] - p.comp_first[k]);
                if (k == part) {
                    lo = at;
                    hi = at + n;
                }
                at += n;
            }
            go = want && (inside != 0 ? part >= 0 : c == 0);
        } else {
            const int nt = p.comp_first[c + 1] - p.comp_first[c];
            const int cnt = min(kStage, nt - first);
            __syncthreads();
            hi = stage_triangles<BLOCK>(p, s, c, first, cnt, 0);
            __syncthreads();
            go = want && (inside == 0 || (inside >> c & 1));
            last = first + cnt == nt;
            first = last ? 0 : first + kStage;
        }
        float b2 = inside ? part2 : out2;
        nearest(s, whole ? slots : hi, pt, go, lo, hi, b2);
        if (go) (inside ? part2 : out2) = b2;
        if (last) {
            if (go && inside) in2 = fmaxf(in2, part2);
            part2 = INFINITY;
            ++c;
        }
        if (whole && !__ballot(want && left != 0)) break;
    }
    return inside ? -sqrtf(in2) : sqrtf(out2);
}

struct BuildBatch {
    BuildArgs link[LSDF_MAX_LINKS];
};

// Grid nodes: node idx of the grid described by p.
// y: the link of the batch.
template <int BLOCK>
__global__ __launch_bounds__(BLOCK, kWavesPerSimd * BLOCK / kBlock) void build_sdf_kernel(BuildBatch batch) {
    __shared__ MeshLds lds;
    const BuildArgs& p = batch.link[blockIdx.y];
    if (blockIdx.x >= (unsigned)p.blocks) return;   // the batch's largest grid sets the launch
    uint32_t kx, ky, kz;   // (fewer than 2^32 threads: 32-bit quotients)
    if (p.bricks) {
        // a wave takes 4 x 4 x 4 nodes, which want the same few groups of triangles
        const uint32_t bx = ((uint32_t)p.n[0] + 3) / 4, by = ((uint32_t)p.n[1] + 3) / 4;
        const uint32_t brick = blockIdx.x * (BLOCK / 64) + (threadIdx.x >> 6);
        const uint32_t row = brick / bx, layer = row / by;
        const uint32_t t = threadIdx.x & 63;
        kx = 4 * (brick - row * bx) + (t & 3);
        ky = 4 * (row - layer * by) + (t >> 2 & 3);
        kz = 4 * layer + (t >> 4);
    } else {
        const uint32_t k = blockIdx.x * BLOCK + threadIdx.x, row = k / (uint32_t)p.n[0];
        kx = k - row * (uint32_t)p.n[0];
        kz = row / (uint32_t)p.n[1];
        ky = row - kz * (uint32_t)p.n[1];
    }
    const bool active = kx < (uint32_t)p.n[0] && ky < (uint32_t)p.n[1] && kz < (uint32_t)p.n[2];
    const int64_t idx = ((int64_t)kz * p.n[1] + ky) * p.n[0] + kx;
    const V3 pt = {fmaf((float)kx, p.h[0], p.lo[0]), fmaf((float)ky, p.h[1], p.lo[1]),
                   fmaf((float)kz, p.h[2], p.lo[2])};
    const float sdf = mesh_sdf<BLOCK>(p, lds, pt, active);
    if (active) {
        // one rounding, to nearest even, into the storage type
        if (p.dtype == LSDF_BF16)
            static_cast<uint16_t*>(p.out)[idx] = __builtin_bit_cast(uint16_t, (__bf16)sdf);
        else if (p.dtype == LSDF_F16)
            static_cast<_Float16*>(p.out)[idx] = (_Float16)sdf;
        else
            static_cast<float*>(p.out)[idx] = sdf;
    }
}

struct LabelBatch {
    BuildArgs mesh[LSDF_MAX_LINKS];
    LinkGrid lg[LSDF_MAX_LINKS];
    const float* points[LSDF_MAX_LINKS];
    float* out[LSDF_MAX_LINKS];
    const void* grid;
    int64_t N;
};
static_assert(sizeof(LabelBatch) <= 4096, "kernel arguments of a batch");

// Labels: the grid value inside the grid box, the exact distance outside.
// y: the link of the batch.
template <bool CUBIC, int DT, int BLOCK>
__global__ __launch_bounds__(BLOCK, kWavesPerSimd * BLOCK / kBlock) void label_kernel(LabelBatch p) {
    __shared__ MeshLds lds;
    const int link = blockIdx.y;
    const LinkGrid& lg = p.lg[link];
    const float* points = p.points[link];
    const int64_t j = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
    const bool active = j < p.N;
    const int64_t jj = active ? j : p.N - 1;
    const V3 pt = {points[3 * jj + 0], points[3 * jj + 1], points[3 * jj + 2]};
    const float ident[12] = {1.f, 0.f, 0.f, 0.f, 0.f, 1.f, 0.f, 0.f, 0.f, 0.f, 1.f, 0.f};
    const GridMap gm = grid_map(lg, ident);
    const float g =
        sample_or_inf<CUBIC, DT>(static_cast<const typename GridT<DT>::T*>(p.grid) + lg.offset, lg, gm, pt.x, pt.y, pt.z);
    const bool exact = active && !(g < INFINITY);
    float v = g;
    if (__syncthreads_or(exact)) {
        const float e = mesh_sdf<BLOCK>(p.mesh[link], lds, pt, exact);
        if (exact) v = e;
    }
    if (active) p.out[link][j] = v;
}

}  // namespace

namespace {

// Does a launch of `blocks` small workgroups over n meshes take them?
bool small_blocks(int64_t blocks, int32_t n, const int32_t* nt) {
    return blocks <= kMostSmall && *std::max_element(nt, nt + n) <= kSmallBlock;
}

int mesh_args(const float* verts, int32_t nv, const int32_t* tris, int32_t nt, const int32_t* comp_first,
              int32_t ncomp, BuildArgs* p) {
    using namespace lsdf;
    if (nv < 1 || nt < 1) return fail(LSDF_E_SHAPE, "mesh: empty (nv = %d, nt = %d)", (int)nv, (int)nt);
    if (!verts || !tris) return fail(LSDF_E_INVALID_ARG, "mesh: NULL device pointer");
    if (comp_first) {
        if (ncomp < 1 || ncomp > LSDF_MAX_COMPONENTS)
            return fail(LSDF_E_SHAPE, "mesh: ncomp = %d out of [1, %d]", (int)ncomp, LSDF_MAX_COMPONENTS);
        if (comp_first[0] != 0 || comp_first[ncomp] != nt)
            return fail(LSDF_E_SHAPE, "mesh: comp_first must run from 0 to nt");
        for (int k = 0; k <= ncomp; ++k) {
            if (k > 0 && comp_first[k] <= comp_first[k - 1])
                return fail(LSDF_E_SHAPE, "mesh: comp_first must increase strictly");
            p->comp_first[k] = comp_first[k];
        }
        p->ncomp = ncomp;
    } else {
        p->comp_first[0] = 0;
        p->comp_first[1] = nt;
        p->ncomp = 1;
    }
    p->nv = nv;
    p->verts = verts;
    p->tris = tris;
    return LSDF_OK;
}

}  // namespace

LSDF_API int lsdf_sdf_labels(const float* verts, int32_t nv, const int32_t* tris, int32_t nt,
                             const int32_t* comp_first, int32_t ncomp, const lsdf_grid* desc, const void* grid_buf,
                             const float* points, int64_t N, float* out, void* stream) {
    return lsdf_sdf_labels_links(1, &verts, &nv, &tris, &nt, &comp_first, &ncomp, desc, grid_buf, &points, N, &out, stream);
}

LSDF_API int lsdf_sdf_labels_links(int32_t n, const float* const* verts, const int32_t* nv, const int32_t* const* tris,
                                   const int32_t* nt, const int32_t* const* comp_first, const int32_t* ncomp,
                                   const lsdf_grid* grids, const void* grid_buf, const float* const* points, int64_t N,
                                   float* const* out, void* stream) {
    using namespace lsdf;
    clear_error();
    if (n < 1 || n > LSDF_MAX_LINKS) return fail(LSDF_E_SHAPE, "sdf_labels: %d links out of [1, %d]", (int)n, LSDF_MAX_LINKS);
    if (!grids) return fail(LSDF_E_INVALID_ARG, "sdf_labels: desc is NULL");
    if (!verts || !nv || !tris || !nt || !comp_first || !ncomp || !points || !out)
        return fail(LSDF_E_INVALID_ARG, "sdf_labels: NULL array");
    if (N < 0) return fail(LSDF_E_SHAPE, "sdf_labels: N < 0");
    LabelBatch a{};
    bool cubic = true;
    for (int i = 0; i < n; ++i) {
        int rc = mesh_args(verts[i], nv[i], tris[i], nt[i], comp_first[i], ncomp[i], &a.mesh[i]);
        if (rc != LSDF_OK) return rc;
        if ((rc = prepare_link_grid(grids[i], i, &a.lg[i])) != LSDF_OK) return rc;
        if (grids[i].dtype != grids[0].dtype) return fail(LSDF_E_UNSUPPORTED, "sdf_labels: grids must share a dtype");
        cubic = cubic && a.lg[i].cubic;
        a.points[i] = points[i];
        a.out[i] = out[i];
    }
    if (N == 0) return LSDF_OK;
    for (int i = 0; i < n; ++i)
        if (!grid_buf || !points[i] || !out[i]) return fail(LSDF_E_INVALID_ARG, "sdf_labels: NULL device pointer");
    a.grid = grid_buf;
    a.N = N;
    const bool small = small_blocks(n * ((N + kSmallBlock - 1) / kSmallBlock), n, nt);
    const int block = small ? kSmallBlock : kBlock;
    const dim3 grid((unsigned)((N + block - 1) / block), (unsigned)n);
    hipStream_t st = as_stream(stream);
    auto launch = [&](auto few, auto many) { hipLaunchKernelGGL(small ? few : many, grid, dim3(block), 0, st, a); };
    switch (grids[0].dtype * 2 + (cubic ? 1 : 0)) {
        case LSDF_F32 * 2 + 1: launch(label_kernel<true, LSDF_F32, kSmallBlock>, label_kernel<true, LSDF_F32, kBlock>); break;
        case LSDF_F32 * 2: launch(label_kernel<false, LSDF_F32, kSmallBlock>, label_kernel<false, LSDF_F32, kBlock>); break;
        case LSDF_BF16 * 2 + 1: launch(label_kernel<true, LSDF_BF16, kSmallBlock>, label_kernel<true, LSDF_BF16, kBlock>); break;
        case LSDF_BF16 * 2: launch(label_kernel<false, LSDF_BF16, kSmallBlock>, label_kernel<false, LSDF_BF16, kBlock>); break;
        case LSDF_F16 * 2 + 1: launch(label_kernel<true, LSDF_F16, kSmallBlock>, label_kernel<true, LSDF_F16, kBlock>); break;
        default: launch(label_kernel<false, LSDF_F16, kSmallBlock>, label_kernel<false, LSDF_F16, kBlock>); break;
    }
    return check_launch("sdf_labels");
}

LSDF_API int lsdf_build_link_sdf(const float* verts, int32_t nv, const int32_t* tris, int32_t nt,
                                 const int32_t* comp_first, int32_t ncomp, const lsdf_grid* desc,
                                 void* grid_buf, void* stream) {
    return lsdf_build_link_sdfs(1, &verts, &nv, &tris, &nt, &comp_first, &ncomp, desc, grid_buf, stream);
}

LSDF_API int lsdf_build_link_sdfs(int32_t n, const float* const* verts, const int32_t* nv, const int32_t* const* tris,
                                  const int32_t* nt, const int32_t* const* comp_first, const int32_t* ncomp,
                                  const lsdf_grid* grids, void* grid_buf, void* stream) {
    using namespace lsdf;
    clear_error();
    if (n < 1 || n > LSDF_MAX_LINKS)
        return fail(LSDF_E_SHAPE, "build_link_sdf: %d links out of [1, %d]", (int)n, LSDF_MAX_LINKS);
    if (!grids) return fail(LSDF_E_INVALID_ARG, "build_link_sdf: desc is NULL");
    if (!verts || !nv || !tris || !nt || !comp_first || !ncomp)
        return fail(LSDF_E_INVALID_ARG, "build_link_sdf: NULL array");
    BuildBatch batch{};
    int64_t lanes[LSDF_MAX_LINKS], all = 0;   // all: workgroups of kSmallBlock
    int32_t most = 0;
    for (int i = 0; i < n; ++i) {
        BuildArgs& p = batch.link[i];
        const lsdf_grid& desc = grids[i];
        int rc = mesh_args(verts[i], nv[i], tris[i], nt[i], comp_first[i], ncomp[i], &p);
        if (rc != LSDF_OK) return rc;
        if (!grid_buf) return fail(LSDF_E_INVALID_ARG, "build_link_sdf: grid_buf is NULL");
        LinkGrid g;
        if ((rc = prepare_link_grid(desc, i, &g)) != LSDF_OK) return rc;
        for (int a = 0; a < 3; ++a) {
            p.lo[a] = desc.lo[a];
            p.h[a] = (float)(((double)desc.hi[a] - (double)desc.lo[a]) / (double)(desc.n[a] - 1));
            p.n[a] = desc.n[a];
        }
        p.dtype = desc.dtype;
        p.out = static_cast<char*>(grid_buf) + desc.elem_offset * (desc.dtype == LSDF_F32 ? 4 : 2);
        const int64_t nodes = (int64_t)p.n[0] * p.n[1] * p.n[2];
        // bricks unless their padding would leave more than half the lanes idle (thin grids)
        // or take 2^32 threads, which no launch may have (2 x 1,024 x 2^20 nodes)
        const int64_t bricks = (int64_t)((p.n[0] + 3) / 4) * ((p.n[1] + 3) / 4) * ((p.n[2] + 3) / 4);
        p.bricks = bricks * 64 <= 2 * nodes && bricks * 64 <= ((int64_t)1 << 32) - kBlock;
        lanes[i] = p.bricks ? bricks * 64 : nodes;
        all += (lanes[i] + kSmallBlock - 1) / kSmallBlock;
    }
    const bool small = small_blocks(all, n, nt);
    const int block = small ? kSmallBlock : kBlock;
    for (int i = 0; i < n; ++i) {
        batch.link[i].blocks = (int32_t)((lanes[i] + block - 1) / block);   // lanes < 2^32
        most = std::max(most, batch.link[i].blocks);
    }
    const auto kernel = small ? build_sdf_kernel<kSmallBlock> : build_sdf_kernel<kBlock>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)most, (unsigned)n), dim3(block), 0, as_stream(stream), batch);
    return check_launch("build_link_sdf");
}
