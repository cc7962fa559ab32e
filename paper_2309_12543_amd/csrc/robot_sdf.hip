// The paper's own pipeline (Sec. III-A, Eq. 1-4): per configuration, a
// "Robot SDF" over the voxels of the environment, the minimum over links of
// each link's SDF transformed by its pose and aligned to the environment
// grid; at run time the distance of a configuration is a pure gather, the
// minimum of its Robot SDF over the voxels the obstacle points occupy.
// It is kept here as the comparator of the per-point query: heavy
// preparation and C x V voxels of memory against a trivial runtime.
//
// Build: every value is first set to +inf at full store width; then, per
// (configuration, link), only the voxels whose centre can lie in the link's
// grid box are sampled and take an atomic minimum (about 1 in 1,000 of a
// configuration's 2 million at 128^3).
//   * link i's block at configuration c covers voxels k .. k + 2m - 1 per
//     axis, with k from the alignment of Eq. 1-3 (computed in double from
//     the link origin: T_O = t - lo, k = round(T_O / r) - m) and m the
//     block half-width in voxels (the farthest corner of the link's grid box
//     from the link origin, rounded up, plus two voxels, so that the block
//     holds every voxel whose centre can fall in the box);
//   * a voxel's value is the minimum, over the links whose block covers it,
//     of the link grid's interpolant at the voxel centre moved into the link
//     frame (the transformation of Eq. 4), +inf where no such link's box
//     holds the centre.  The centre is lo + (v + 1/2) r (double, rounded
//     once to float) and the interpolant uses the plain query's arithmetic,
//     so each value is bit-identical to the plain query at that point.
// Bound by the HBM writes of the +inf fill.  200 configurations over 128^3
// voxels (1.68 GB): 472 us with one thread per voxel column that tested every
// link and stored 256 B a wave; 243 us of fill and 66 us of samples (gathers and
// HBM atomics in about equal parts) now.
// Runtime: zero an occupancy bitmap and a counter; voxelise the points
// (floor((x - lo) / r) in double), keeping the first point of each voxel
// in a list of distinct occupied voxels; one workgroup per configuration
// takes the minimum of its Robot SDF over the list.
#include <algorithm>

#include "grid_sample.hpp"

namespace {

using lsdf::GridT;
using lsdf::LinkGrid;

constexpr int kBlock = 256;
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct LinkBlock {   // per (configuration, link): the voxels to look at and the grid map
    uint32_t range[3];   // first voxel and one past the last per axis, 16 bits each
    int32_t pad;
    lsdf::GridMap gm;
};
static_assert(sizeof(LinkBlock) == 64, "LinkBlock layout");

struct LinkBlockNN {   // per (configuration, link) of the network build
    int32_t k[3];
    uint32_t held_lo;                // (both of the first entry's: held_voxels)
    float h[LSDF_FRNN_HIDDEN];       // hidden layer of f at this rotation, unit 4 s + g at 8 g + s
    float dtinv[3];
    uint32_t held_hi;
};
static_assert(sizeof(LinkBlockNN) == 160, "LinkBlockNN layout");

struct BuildArgs {
    LinkGrid link[LSDF_MAX_LINKS];
    int32_t halfw[LSDF_MAX_LINKS];   // m_i
    double lo[3];
    double r;
    int32_t n[3];
    int32_t C, L;
    const float* link_T;
    LinkBlock* blocks;               // [C][L]
    float* rs;                       // [C][n_z][n_y][n_x]
};

// The voxels of the environment link i's block covers at configuration c, cut
// to those whose centre can lie in the link's grid box: the box's corners are
// mapped back to the world with the inverse of the grid map, the box widened by
// 1e-3 + 1e-5 half + 1e-4 |w| grid steps, far beyond the FP32 rounding of a mapped centre.
// A map with no sound inverse (no pose of a rigid link) keeps the whole block.
__device__ inline void align(const BuildArgs& a, int64_t t) {
    if (t >= (int64_t)a.C * a.L) return;
    const int i = (int)(t % a.L);
    const LinkGrid& lg = a.link[i];
    const float* T = a.link_T + t * 12;
    LinkBlock b{};
    // the plain query's world-to-grid map of this pose (the transformation
    // of Eq. 4 with the grid scaling folded in)
    b.gm = lsdf::grid_map(lg, T);
    const double m[3][3] = {{b.gm.m00, b.gm.m01, b.gm.m02}, {b.gm.m10, b.gm.m11, b.gm.m12}, {b.gm.m20, b.gm.m21, b.gm.m22}};
    const double w[3] = {b.gm.w0, b.gm.w1, b.gm.w2};
    double adj[3][3], norm = 0.0;   // adj = det m^-1
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const int r1 = (c + 1) % 3, r2 = (c + 2) % 3, c1 = (r + 1) % 3, c2 = (r + 2) % 3;
            adj[r][c] = m[r1][c1] * m[r2][c2] - m[r1][c2] * m[r2][c1];
            norm = fmax(norm, fabs(m[r][c]));
        }
    const double det = m[0][0] * adj[0][0] + m[0][1] * adj[1][0] + m[0][2] * adj[2][0];
    // (the inverse's rounding, about 1e-16 norm^3 / det, stays below the widening)
    const bool sound = fabs(det) > 1e-6 * norm * norm * norm;
    const float tr[3] = {T[3], T[7], T[11]};
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        // Eq. 1-2: T_O = t - lo, k = round(T_O / r) - m
        const int32_t k = (int32_t)rint(((double)tr[ax] - a.lo[ax]) / a.r) - a.halfw[i];
        int64_t lo = k, hi = (int64_t)k + 2 * a.halfw[i];
        if (sound) {
            double c = 0.0, e = 0.0;
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                c -= adj[ax][q] / det * w[q];
                e += fabs(adj[ax][q] / det) * ((double)lg.half[q] * (1.0 + 1e-5) + 1e-3 + 1e-4 * fabs(w[q]));
            }
            // voxel v's centre lies at lo + (v + 1/2) r; one voxel more at either end
            const double v0 = floor((c - e - a.lo[ax]) / a.r) - 1.0, v1 = ceil((c + e - a.lo[ax]) / a.r) + 1.0;
            lo = max(lo, (int64_t)fmin(fmax(v0, -1e9), 1e9));
            hi = min(hi, (int64_t)fmin(fmax(v1, -1e9), 1e9));
        }
        lo = min(max(lo, (int64_t)0), (int64_t)a.n[ax]);
        hi = min(max(hi, lo), (int64_t)a.n[ax]);
        b.range[ax] = (uint32_t)lo | (uint32_t)hi << 16;   // n <= 4096
    }
    a.blocks[t] = b;
}

// What held_voxels needs of a network build.
struct HeldArgs {
    LinkBlockNN* blocks;
    int64_t count;       // C L
    int32_t n[3], w;     // the environment, 2 m
};

// Per axis, the block voxels that the environment holds in any configuration
// and link: lo to hi - 1, a byte per axis from the low one (hi = 0: none).
__device__ inline void held_voxels(const HeldArgs& a) {
    __shared__ int range[kBlock / 64][6];
    int r[6] = {a.w, a.w, a.w, 0, 0, 0};
#pragma unroll 4
    for (int64_t t = threadIdx.x; t < a.count; t += kBlock) {
        int l[3], h[3];
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            const int k = min(max(a.blocks[t].k[ax], -a.w), a.n[ax]);
            l[ax] = max(-k, 0);
            h[ax] = min(a.n[ax] - k, a.w);
        }
        const bool some = l[0] < h[0] && l[1] < h[1] && l[2] < h[2];
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            r[ax] = min(r[ax], some ? l[ax] : a.w);
            r[3 + ax] = max(r[3 + ax], some ? h[ax] : 0);
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            r[ax] = min(r[ax], __shfl_xor(r[ax], o, 64));
            r[3 + ax] = max(r[3 + ax], __shfl_xor(r[3 + ax], o, 64));
        }
#pragma unroll
    for (int k = 0; k < 6; ++k)
        if ((threadIdx.x & 63) == 0) range[threadIdx.x >> 6][k] = r[k];
    __syncthreads();
    if (threadIdx.x != 0) return;
#pragma unroll
    for (int k = 0; k < 6; ++k)
        for (int v = 1; v < kBlock / 64; ++v) r[k] = k < 3 ? min(r[k], range[v][k]) : max(r[k], range[v][k]);
    a.blocks->held_lo = (uint32_t)(r[0] | r[1] << 8 | r[2] << 16);
    a.blocks->held_hi = (uint32_t)(r[3] | r[4] << 8 | r[5] << 16);
}

// Every value of the Robot SDFs to +inf, before the minima: one 16 B store a
// thread, so that the resident workgroups sweep the memory in order (1.68 GB in
// 243 us, 6.9 TB/s; 4 stores a thread 276 us, a grid-stride loop 290 to 410 us,
// non-temporal stores no better).
// What goes beside a fill, in workgroups of its own before the fill's: it needs
// no launch then (40 x 7 blocks outside 64^3 voxels, nothing but the fill to do:
// 16.4 us with the alignment in a launch before it, 13.0 beside it; 8^3 voxels
// 8.0 and 6.6 us).  At the alignment's 78 registers the fill keeps its rate; held
// to 64 it spills, 14.1 us.
struct NoneBeside {
    unsigned groups() const { return 0; }
    __device__ void run() const {}
};
struct HeldBeside {
    HeldArgs held;
    unsigned groups() const { return 1; }
    __device__ void run() const { held_voxels(held); }
};
struct AlignBeside {
    BuildArgs a;
    unsigned groups() const { return (unsigned)(((int64_t)a.C * a.L + kBlock - 1) / kBlock); }
    __device__ void run() const { align(a, (int64_t)blockIdx.x * kBlock + threadIdx.x); }
};

template <class Beside>
__global__ __launch_bounds__(kBlock) void fill_inf_kernel(float* out, int64_t n, int64_t head, int64_t quads, unsigned first,
                                                          Beside beside) {
    if (blockIdx.x < first) {
        beside.run();
        return;
    }
    // out[head] is 16-byte aligned; the odd values at either end go one by one
    const int64_t t = (int64_t)(blockIdx.x - first) * kBlock + threadIdx.x;
    const f32x4 inf = {INFINITY, INFINITY, INFINITY, INFINITY};
    if (t < quads) reinterpret_cast<f32x4*>(out + head)[t] = inf;
    if (t < head) out[t] = INFINITY;
    if (t < 4 && head + 4 * quads + t < n) out[head + 4 * quads + t] = INFINITY;
}

template <class Beside>
int launch_fill_inf(const char* who, float* out, int64_t n, const Beside& beside, hipStream_t s) {
    // launches of at most 2^30 quads each (2^22 workgroups)
    constexpr int64_t kMost = (int64_t)1 << 32;
    for (int64_t at = 0; at < n; at += kMost) {
        float* p = out + at;
        const int64_t cnt = std::min(kMost, n - at);
        const int64_t head = std::min<int64_t>(cnt, (4 - (int64_t)((reinterpret_cast<uintptr_t>(p) >> 2) & 3)) & 3);
        const int64_t quads = (cnt - head) / 4;
        const unsigned first = at == 0 ? beside.groups() : 0, groups = (unsigned)(quads / kBlock + 1);
        if (first)
            hipLaunchKernelGGL(fill_inf_kernel<Beside>, dim3(first + groups), dim3(kBlock), 0, s, p, cnt, head, quads, first, beside);
        else
            hipLaunchKernelGGL(fill_inf_kernel<NoneBeside>, dim3(groups), dim3(kBlock), 0, s, p, cnt, head, quads, 0u, NoneBeside{});
        const int rc = lsdf::check_launch(who);
        if (rc != LSDF_OK) return rc;
    }
    return LSDF_OK;
}

// Minimum of v (not NaN, not -0) into *p, which holds +inf or other such
// minima: the bits of non-negative floats order like signed integers, those of
// negative ones against unsigned.
__device__ inline void atomic_min(float* p, float v) {
    if (v >= 0.0f)
        atomicMin(reinterpret_cast<int*>(p), __float_as_int(v));
    else
        atomicMax(reinterpret_cast<unsigned*>(p), __float_as_uint(v));
}

constexpr int kBuildShares = 16;   // workgroups that share a pair's voxels

// One (configuration, link) per workgroup (y: shares of its voxels): samples
// the voxels in its range, x fastest over the threads, and takes an atomic
// minimum for those in the box.
template <bool CUBIC, int DT>
__global__ __launch_bounds__(kBlock) void build_kernel(BuildArgs a, const typename GridT<DT>::T* __restrict__ grid) {
    const int64_t V = (int64_t)a.n[0] * a.n[1] * a.n[2];
    for (int64_t t = blockIdx.x; t < (int64_t)a.C * a.L; t += gridDim.x) {
        const LinkBlock b = a.blocks[t];
        const int i = (int)(t % a.L);
        const LinkGrid& lg = a.link[i];
        float* rs = a.rs + t / a.L * V;
        const int x0 = b.range[0] & 0xffff, y0 = b.range[1] & 0xffff, z0 = b.range[2] & 0xffff;
        const uint32_t nx = (b.range[0] >> 16) - x0, ny = (b.range[1] >> 16) - y0, nz = (b.range[2] >> 16) - z0;
        const int64_t count = (int64_t)nx * ny * nz;
        for (int64_t v = (int64_t)blockIdx.y * kBlock + threadIdx.x; v < count; v += (int64_t)gridDim.y * kBlock) {
            const uint32_t row = (uint32_t)v / nx, vx = x0 + ((uint32_t)v - row * nx);   // at most 2^32 voxels
            const uint32_t vz = z0 + row / ny, vy = y0 + row % ny;
            const float x = (float)(a.lo[0] + ((double)vx + 0.5) * a.r);
            const float y = (float)(a.lo[1] + ((double)vy + 0.5) * a.r);
            const float z = (float)(a.lo[2] + ((double)vz + 0.5) * a.r);
            const float val = lsdf::sample_or_inf<CUBIC, DT>(grid + lg.offset, lg, b.gm, x, y, z);
            if (val < INFINITY) atomic_min(&rs[((int64_t)vz * a.n[1] + vy) * a.n[0] + vx], val);
        }
    }
}

// The same build with the transformation of Eq. 5: each block voxel's
// link-frame position comes from the grid-transformation network,
// G = f(R) + dt_inv with dt_inv = -R^T dt / e_r, l = e_r G, e_r = m r, for a
// block half-width m shared by all links (the network's).
struct BuildNNArgs {
    LinkGrid link[LSDF_MAX_LINKS];
    double lo[3];
    double r;
    int32_t n[3];
    int32_t C, L, m;
    float er;                        // m r
    const float* link_T;
    const float* params;             // W1[32][9], b1[32], W2[3V][32], b2[3V]
    LinkBlockNN* blocks;             // [C][L]
    float* rs;
};

// One thread per hidden unit of each (configuration, link); unit 0's also
// aligns the block.
__global__ __launch_bounds__(kBlock) void align_nn_kernel(BuildNNArgs a) {
    const int64_t t = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / LSDF_FRNN_HIDDEN;
    const int u = threadIdx.x % LSDF_FRNN_HIDDEN;
    if (t >= (int64_t)a.C * a.L) return;
    const float* T = a.link_T + t * 12;
    LinkBlockNN& b = a.blocks[t];
    const float x[9] = {T[0], T[1], T[2], T[4], T[5], T[6], T[8], T[9], T[10]};
    const float* W1 = a.params;
    float acc = W1[LSDF_FRNN_HIDDEN * 9 + u];
#pragma unroll
    for (int k = 0; k < 9; ++k) acc = fmaf(W1[u * 9 + k], x[k], acc);
    b.h[8 * (u & 3) + (u >> 2)] = fmaxf(acc, 0.0f);
    if (u != 0) return;
    double dt[3];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        // Eq. 1-3: T_O = t - lo, k = round(T_O / r) - m, dt = T_O - (k + m) r
        const double t_o = (double)T[4 * ax + 3] - a.lo[ax];
        const int32_t k = (int32_t)rint(t_o / a.r) - a.m;
        dt[ax] = t_o - ((double)k + (double)a.m) * a.r;
        b.k[ax] = k;
    }
    // dt_inv = -R^T dt / e_r  (R[row][col] = T[4 row + col])
#pragma unroll
    for (int ax = 0; ax < 3; ++ax)
        b.dtinv[ax] = (float)(-((double)T[ax] * dt[0] + (double)T[4 + ax] * dt[1] + (double)T[8 + ax] * dt[2]) /
                              (double)a.er);
}

// One wave takes 16 block voxels and runs over its share of the (link, 16
// configurations) groups.  f's output layer is a product of K = 32 over 3
// outputs a voxel and is done on FP32 MFMA (v_mfma_f32_16x16x4: one chain of
// fused multiply-adds per output in the order of K, the bits of a scalar
// loop): A the voxels' weights of one component (lane l: voxel l mod 16, k =
// 4 s + l / 16), kept in registers over all groups, B the hidden layers (lane
// l: configuration l mod 16, the same k), so that lane l ends with the 3
// components of voxels 4 (l / 16) + r at configuration l mod 16.  A point in
// the link's box is sampled and its value goes to the environment voxel by an
// atomic minimum (one in some tens of points is; the values were set to +inf
// before).
// Bound by MFMA issue (2 x 96 FLOP a block voxel, link and configuration: 35
// of 85 us; the samples and their atomics take about 25 more) beside the +inf
// fill (HBM).  40 configurations x 7 links, 44^3 block voxels, 128^3 voxels:
// 2.01 ms a call with one thread per environment voxel, which read its 384 B
// of weights from L2 for every link and configuration; 0.138 ms now.  The four
// points' gathers issued together, and 5 or 6 waves a SIMD, measured the same.
// A wave whose voxels no configuration has in the environment (held_voxels)
// leaves before it loads any weights: 40 x 7 blocks all outside 64^3 voxels 73
// -> 17 us (26 with a thread per environment voxel), 0.138 ms with it and
// without where the environment holds nearly all; a ballot over each group's own
// voxels costs 7 us of that.
constexpr int kTile = 16;            // block voxels and configurations per MFMA tile
constexpr int64_t kNNWaves = 8192;   // waves of a build, about
constexpr int kSteps = LSDF_FRNN_HIDDEN / 4;

template <bool CUBIC, int DT>
__global__ __launch_bounds__(kBlock) void build_nn_kernel(BuildNNArgs a, const typename GridT<DT>::T* __restrict__ grid) {
    const int lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
    const int w = 2 * a.m, V = w * w * w;   // at most 128^3
    const int j0 = ((int)blockIdx.x * (kBlock / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6))) * kTile;
    if (j0 >= V) return;
    {
        // an environment that the blocks stick out of holds few of their voxels,
        // or none: a wave with none of them has nothing to do
        const int last = min(j0 + kTile, V) - 1;
        const uint32_t lo = a.blocks->held_lo, hi = a.blocks->held_hi;
        const int z0 = j0 / (w * w), z1 = last / (w * w), y0 = j0 / w - z0 * w, y1 = last / w - z1 * w;
        if (z1 < (int)(lo >> 16) || z0 >= (int)(hi >> 16)) return;
        if (z0 == z1 && (y1 < (int)(lo >> 8 & 0xff) || y0 >= (int)(hi >> 8 & 0xff))) return;
    }
    const float* W2 = a.params + LSDF_FRNN_HIDDEN * 10;
    const float* b2 = W2 + (int64_t)3 * V * LSDF_FRNN_HIDDEN;
    float wt[3][kSteps];
    const int ja = min(j0 + col, V - 1);
#pragma unroll
    for (int ax = 0; ax < 3; ++ax)
#pragma unroll
        for (int s = 0; s < kSteps; ++s) wt[ax][s] = W2[(int64_t)(3 * ja + ax) * LSDF_FRNN_HIDDEN + 4 * s + g];
    f32x4 bias[3];
    uint32_t jv[4];   // voxel coordinates in the block, a byte each (2 m <= 128)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int jc = min(j0 + 4 * g + r, V - 1);
        const int jz = jc / (w * w), jy = (jc - jz * w * w) / w;
        jv[r] = (uint32_t)(jc - (jz * w + jy) * w) | (uint32_t)jy << 8 | (uint32_t)jz << 16;
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) bias[ax][r] = b2[3 * jc + ax];
    }
    const int cgroups = (a.C + kTile - 1) / kTile;
    const int64_t env_v = (int64_t)a.n[0] * a.n[1] * a.n[2];
    for (int gr = blockIdx.y; gr < a.L * cgroups; gr += gridDim.y) {
        const int i = gr / cgroups;
        const int c = (gr - i * cgroups) * kTile + col;
        const LinkBlockNN& b = a.blocks[(int64_t)min(c, a.C - 1) * a.L + i];
        f32x4 y[3] = {bias[0], bias[1], bias[2]};
        const f32x4 h0 = *reinterpret_cast<const f32x4*>(&b.h[8 * g]), h1 = *reinterpret_cast<const f32x4*>(&b.h[8 * g + 4]);
#pragma unroll
        for (int s = 0; s < kSteps; ++s)
#pragma unroll
            for (int ax = 0; ax < 3; ++ax)
                y[ax] = __builtin_amdgcn_mfma_f32_16x16x4f32(wt[ax][s], s < 4 ? h0[s] : h1[s - 4], y[ax], 0, 0, 0);
        const int k0 = b.k[0], k1 = b.k[1], k2 = b.k[2];
        const float t[3] = {b.dtinv[0], b.dtinv[1], b.dtinv[2]};
        const LinkGrid& lg = a.link[i];
        const typename GridT<DT>::T* G = grid + lg.offset;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            // link-frame point e_r (f + dt_inv), then centred grid coordinates v_a = l_a invh_a + cen_a
            const float v0 = fmaf(lg.invh[0], a.er * (y[0][r] + t[0]), lg.cen[0]);
            const float v1 = fmaf(lg.invh[1], a.er * (y[1][r] + t[1]), lg.cen[1]);
            const float v2 = fmaf(lg.invh[2], a.er * (y[2][r] + t[2]), lg.cen[2]);
            const uint32_t vx = (uint32_t)k0 + (jv[r] & 0xff), vy = (uint32_t)k1 + (jv[r] >> 8 & 0xff),
                           vz = (uint32_t)k2 + (jv[r] >> 16);
            const bool covered = vx < (uint32_t)a.n[0] && vy < (uint32_t)a.n[1] && vz < (uint32_t)a.n[2] && c < a.C &&
                                 j0 + 4 * g + r < V;
            if (covered && lsdf::inside<CUBIC>(lg, v0, v1, v2)) {
                const float val = lsdf::cell_value<DT>(G, lg, v0, v1, v2);
                // (a NaN, from a NaN or infinite node, is no value, as in build_kernel)
                if (val < INFINITY) atomic_min(&a.rs[(int64_t)c * env_v + ((int64_t)vz * a.n[1] + vy) * a.n[0] + vx], val);
            }
        }
    }
}

struct RuntimeArgs {
    double lo[3];
    double r;
    int32_t n[3];
    int32_t C;
    const float* points;
    int64_t M;
    uint32_t* bitmap;    // [ceil(V / 32)]
    uint32_t* count;     // distinct occupied voxels
    uint32_t* list;      // [min(M, V)]
    int64_t bitmap_words;
    const float* rs;
    float* out_dist;
};

__global__ __launch_bounds__(kBlock) void runtime_zero_kernel(RuntimeArgs a) {
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (t < a.bitmap_words) a.bitmap[t] = 0u;
    if (t == 0) *a.count = 0u;
}

// Voxels a workgroup's points fall in are first made unique in an LDS hash
// set (open addressing, twice as many slots as points, so every insertion
// ends within the table), and only one point per distinct voxel sets the
// voxel's bit with a device atomic: points of one obstacle lie together in
// the cloud, and their atomics on the same few bitmap words would otherwise
// run one after another.
constexpr int kHashSlots = 2 * kBlock;
constexpr uint32_t kHashEmpty = 0xffffffffu;

__global__ __launch_bounds__(kBlock) void voxelise_kernel(RuntimeArgs a) {
    __shared__ uint32_t s_key[kHashSlots];
    for (int k = threadIdx.x; k < kHashSlots; k += kBlock) s_key[k] = kHashEmpty;
    __syncthreads();
    const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    bool inside = j < a.M;
    int64_t q[3] = {0, 0, 0};
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const double u = inside ? floor(((double)a.points[3 * j + ax] - a.lo[ax]) / a.r) : -1.0;
        inside = inside && u >= 0.0 && u < (double)a.n[ax];   // points outside the environment are dropped
        q[ax] = inside ? (int64_t)u : 0;
    }
    const int64_t v = (q[2] * a.n[1] + q[1]) * (int64_t)a.n[0] + q[0];
    // this point stands for its voxel in the workgroup when it inserts the
    // voxel into the set first (voxel 2^32 - 1, the empty key, always does)
    bool rep = inside && (uint32_t)v == kHashEmpty;
    if (inside && !rep) {
        uint32_t h = ((uint32_t)v * 2654435761u) % (uint32_t)kHashSlots;
        for (int probe = 0; probe < kHashSlots; ++probe) {
            const uint32_t prev = atomicCAS(&s_key[h], kHashEmpty, (uint32_t)v);
            if (prev == kHashEmpty) {
                rep = true;
                break;
            }
            if (prev == (uint32_t)v) break;
            h = (h + 1u) % (uint32_t)kHashSlots;
        }
    }
    const uint32_t bit = 1u << (v & 31);
    const bool first = rep && !(atomicOr(&a.bitmap[v >> 5], bit) & bit);   // first point of this voxel
    // the wave's new voxels take consecutive list slots: one counter atomic per wave
    const uint64_t mask = __ballot(first);
    if (mask == 0) return;
    const int lane = threadIdx.x & 63;
    const int leader = __builtin_ctzll(mask);
    uint32_t base = 0;
    if (lane == leader) base = atomicAdd(a.count, (uint32_t)__builtin_popcountll(mask));
    base = __shfl(base, leader, 64);
    if (first) a.list[base + (uint32_t)__builtin_popcountll(mask & ((1ull << lane) - 1))] = (uint32_t)v;
}

// One workgroup per configuration: the minimum of its Robot SDF over the
// occupied voxels.
__global__ __launch_bounds__(kBlock) void gather_kernel(RuntimeArgs a) {
    const int c = blockIdx.x;
    const int64_t V = (int64_t)a.n[0] * a.n[1] * a.n[2];
    const float* rs = a.rs + (int64_t)c * V;
    const uint32_t cnt = *a.count;
    // four independent loads in flight per step
    float b0 = INFINITY, b1 = INFINITY, b2 = INFINITY, b3 = INFINITY;
    uint32_t k = threadIdx.x;
    for (; k + 3 * kBlock < cnt; k += 4 * kBlock) {
        const uint32_t v0 = a.list[k], v1 = a.list[k + kBlock], v2 = a.list[k + 2 * kBlock], v3 = a.list[k + 3 * kBlock];
        b0 = fminf(b0, rs[v0]);
        b1 = fminf(b1, rs[v1]);
        b2 = fminf(b2, rs[v2]);
        b3 = fminf(b3, rs[v3]);
    }
    for (; k < cnt; k += kBlock) b0 = fminf(b0, rs[a.list[k]]);
    float best = fminf(fminf(b0, b1), fminf(b2, b3));
    // workgroup minimum
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) best = fminf(best, __shfl_xor(best, off));
    __shared__ float wmin[kBlock / 64];
    if ((threadIdx.x & 63) == 0) wmin[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x == 0) {
        float m = wmin[0];
        for (int w = 1; w < kBlock / 64; ++w) m = fminf(m, wmin[w]);
        a.out_dist[c] = m;
    }
}

// Block half-width of a link: the farthest grid-box corner from the link
// origin, in voxels, rounded up, plus two.
double block_halfwidth(const lsdf_grid& g, float voxel) {
    double far2 = 0.0;
    for (int k = 0; k < 8; ++k) {
        double s = 0.0;
        for (int ax = 0; ax < 3; ++ax) {
            const double cc = (k >> ax) & 1 ? g.hi[ax] : g.lo[ax];
            s += cc * cc;
        }
        far2 = std::max(far2, s);
    }
    return std::ceil(std::sqrt(far2) / (double)voxel) + 2.0;
}

int check_env(const char* who, const lsdf_env* env, int64_t* V) {
    using lsdf::fail;
    if (!env) return fail(LSDF_E_INVALID_ARG, "%s: env is NULL", who);
    if (!lsdf::finite3(env->lo) || !std::isfinite(env->voxel) || !(env->voxel > 0.0f))
        return fail(LSDF_E_INVALID_ARG, "%s: env needs a finite corner and a positive voxel edge", who);
    for (int a = 0; a < 3; ++a)
        if (env->n[a] < 1 || env->n[a] > 4096)
            return fail(LSDF_E_SHAPE, "%s: env n[%d] = %d out of [1, 4096]", who, a, (int)env->n[a]);
    *V = (int64_t)env->n[0] * env->n[1] * env->n[2];
    if (*V > ((int64_t)1 << 32)) return fail(LSDF_E_SHAPE, "%s: more than 2^32 voxels", who);
    return LSDF_OK;
}

// room for either form's per-(configuration, link) table
size_t blocks_bytes(int64_t C, int64_t L) {
    return ((size_t)(C * L) * std::max(sizeof(LinkBlock), sizeof(LinkBlockNN)) + 255) / 256 * 256;
}

}  // namespace

LSDF_API int lsdf_robot_sdf_size(int32_t C, const lsdf_env* env, size_t* bytes) {
    using namespace lsdf;
    clear_error();
    int64_t V = 0;
    int rc = check_env("robot_sdf_size", env, &V);
    if (rc != LSDF_OK) return rc;
    if (C < 0) return fail(LSDF_E_SHAPE, "robot_sdf_size: C < 0");
    if (!bytes) return fail(LSDF_E_INVALID_ARG, "robot_sdf_size: bytes is NULL");
    *bytes = (size_t)C * (size_t)V * 4;
    return LSDF_OK;
}

LSDF_API int lsdf_robot_sdf_build_workspace_size(int32_t C, int32_t L, size_t* bytes) {
    using namespace lsdf;
    clear_error();
    if (C < 0 || L < 1 || L > LSDF_MAX_LINKS) return fail(LSDF_E_SHAPE, "robot_sdf_build_workspace_size: bad C or L");
    if (!bytes) return fail(LSDF_E_INVALID_ARG, "robot_sdf_build_workspace_size: bytes is NULL");
    *bytes = blocks_bytes(C, L);
    return LSDF_OK;
}

LSDF_API int lsdf_robot_sdf_build(const float* link_T, int32_t C, int32_t L, const lsdf_grid* grids,
                                  const void* grid_buf, const lsdf_env* env, float* robot_sdf, void* workspace,
                                  size_t ws_bytes, void* stream) {
    using namespace lsdf;
    clear_error();
    int64_t V = 0;
    int rc = check_env("robot_sdf_build", env, &V);
    if (rc != LSDF_OK) return rc;
    if (C < 0) return fail(LSDF_E_SHAPE, "robot_sdf_build: C < 0");
    if (L < 1 || L > LSDF_MAX_LINKS) return fail(LSDF_E_SHAPE, "robot_sdf_build: L = %d out of [1, %d]", (int)L, LSDF_MAX_LINKS);
    if (!grids) return fail(LSDF_E_INVALID_ARG, "robot_sdf_build: grids is NULL");
    if (C == 0) return LSDF_OK;
    if (!link_T || !grid_buf || !robot_sdf || !workspace)
        return fail(LSDF_E_INVALID_ARG, "robot_sdf_build: NULL device pointer");
    if ((reinterpret_cast<uintptr_t>(workspace) & 255) != 0)
        return fail(LSDF_E_INVALID_ARG, "robot_sdf_build: workspace is not 256-byte aligned");
    if (ws_bytes < blocks_bytes(C, L))
        return fail(LSDF_E_SHAPE, "robot_sdf_build: workspace has %zu bytes, needs %zu", ws_bytes, blocks_bytes(C, L));
    BuildArgs a{};
    bool cubic = true;
    const int dtype = grids[0].dtype;
    for (int i = 0; i < L; ++i) {
        rc = prepare_link_grid(grids[i], i, &a.link[i]);
        if (rc != LSDF_OK) return rc;
        if (grids[i].dtype != dtype) return fail(LSDF_E_UNSUPPORTED, "robot_sdf_build: grids must share a dtype");
        cubic = cubic && a.link[i].cubic;
        const double hw = block_halfwidth(grids[i], env->voxel);
        if (hw > 65536.0) return fail(LSDF_E_SHAPE, "robot_sdf_build: link %d's block is too wide", i);
        a.halfw[i] = (int32_t)hw;
    }
    for (int ax = 0; ax < 3; ++ax) {
        a.lo[ax] = env->lo[ax];
        a.n[ax] = env->n[ax];
    }
    a.r = env->voxel;
    a.C = C;
    a.L = L;
    a.link_T = link_T;
    a.blocks = static_cast<LinkBlock*>(workspace);
    a.rs = robot_sdf;
    hipStream_t s = as_stream(stream);
    const int64_t CL = (int64_t)C * L;
    if ((rc = launch_fill_inf("robot_sdf_build (align and fill)", robot_sdf, (int64_t)C * V, AlignBeside{a}, s)) != LSDF_OK) return rc;
    // x: (configuration, link) pairs, y: shares of a pair's voxels
    const dim3 gd((unsigned)std::min<int64_t>(CL, 1 << 20), kBuildShares), bd(kBlock);
    switch (dtype * 2 + (cubic ? 1 : 0)) {
        case LSDF_F32 * 2 + 1: hipLaunchKernelGGL((build_kernel<true, LSDF_F32>), gd, bd, 0, s, a, static_cast<const float*>(grid_buf)); break;
        case LSDF_F32 * 2: hipLaunchKernelGGL((build_kernel<false, LSDF_F32>), gd, bd, 0, s, a, static_cast<const float*>(grid_buf)); break;
        case LSDF_BF16 * 2 + 1: hipLaunchKernelGGL((build_kernel<true, LSDF_BF16>), gd, bd, 0, s, a, static_cast<const uint16_t*>(grid_buf)); break;
        case LSDF_BF16 * 2: hipLaunchKernelGGL((build_kernel<false, LSDF_BF16>), gd, bd, 0, s, a, static_cast<const uint16_t*>(grid_buf)); break;
        case LSDF_F16 * 2 + 1: hipLaunchKernelGGL((build_kernel<true, LSDF_F16>), gd, bd, 0, s, a, static_cast<const _Float16*>(grid_buf)); break;
        default: hipLaunchKernelGGL((build_kernel<false, LSDF_F16>), gd, bd, 0, s, a, static_cast<const _Float16*>(grid_buf)); break;
    }
    return check_launch("robot_sdf_build");
}

LSDF_API int lsdf_robot_sdf_build_frnn(const float* link_T, int32_t C, int32_t L, const lsdf_grid* grids,
                                       const void* grid_buf, const lsdf_env* env, const float* frnn_params,
                                       int32_t m, float* robot_sdf, void* workspace, size_t ws_bytes,
                                       void* stream) {
    using namespace lsdf;
    clear_error();
    int64_t V = 0;
    int rc = check_env("robot_sdf_build_frnn", env, &V);
    if (rc != LSDF_OK) return rc;
    if (C < 0) return fail(LSDF_E_SHAPE, "robot_sdf_build_frnn: C < 0");
    if (L < 1 || L > LSDF_MAX_LINKS) return fail(LSDF_E_SHAPE, "robot_sdf_build_frnn: L = %d out of [1, %d]", (int)L, LSDF_MAX_LINKS);
    if (m < 1 || m > LSDF_FRNN_MAX_HALF) return fail(LSDF_E_SHAPE, "robot_sdf_build_frnn: m = %d out of [1, %d]", (int)m, LSDF_FRNN_MAX_HALF);
    if (!grids) return fail(LSDF_E_INVALID_ARG, "robot_sdf_build_frnn: grids is NULL");
    if (C == 0) return LSDF_OK;
    if (!link_T || !grid_buf || !robot_sdf || !workspace || !frnn_params)
        return fail(LSDF_E_INVALID_ARG, "robot_sdf_build_frnn: NULL device pointer");
    if ((reinterpret_cast<uintptr_t>(workspace) & 255) != 0)
        return fail(LSDF_E_INVALID_ARG, "robot_sdf_build_frnn: workspace is not 256-byte aligned");
    if (ws_bytes < blocks_bytes(C, L))
        return fail(LSDF_E_SHAPE, "robot_sdf_build_frnn: workspace has %zu bytes, needs %zu", ws_bytes, blocks_bytes(C, L));
    BuildNNArgs a{};
    bool cubic = true;
    const int dtype = grids[0].dtype;
    for (int i = 0; i < L; ++i) {
        rc = prepare_link_grid(grids[i], i, &a.link[i]);
        if (rc != LSDF_OK) return rc;
        if (grids[i].dtype != dtype) return fail(LSDF_E_UNSUPPORTED, "robot_sdf_build_frnn: grids must share a dtype");
        cubic = cubic && a.link[i].cubic;
        if (block_halfwidth(grids[i], env->voxel) > (double)m)
            return fail(LSDF_E_SHAPE, "robot_sdf_build_frnn: the network's block (m = %d) does not hold link %d's box",
                        (int)m, i);
    }
    for (int ax = 0; ax < 3; ++ax) {
        a.lo[ax] = env->lo[ax];
        a.n[ax] = env->n[ax];
    }
    a.r = env->voxel;
    a.C = C;
    a.L = L;
    a.m = m;
    a.er = (float)((double)m * (double)env->voxel);
    a.link_T = link_T;
    a.params = frnn_params;
    a.blocks = static_cast<LinkBlockNN*>(workspace);
    a.rs = robot_sdf;
    hipStream_t s = as_stream(stream);
    const int64_t CL = (int64_t)C * L;
    hipLaunchKernelGGL(align_nn_kernel, dim3((unsigned)((CL * LSDF_FRNN_HIDDEN + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, a);
    if ((rc = check_launch("robot_sdf_build_frnn (align)")) != LSDF_OK) return rc;
    const HeldBeside held{{a.blocks, CL, {a.n[0], a.n[1], a.n[2]}, 2 * m}};
    if ((rc = launch_fill_inf("robot_sdf_build_frnn (fill)", robot_sdf, (int64_t)C * V, held, s)) != LSDF_OK) return rc;
    // x: 64 block voxels, y: shares of the groups, about 8 waves a SIMD in all
    // (a wave's weights, loaded once, serve its whole share: 16 a SIMD 5 us
    // slower, 32 a SIMD 37 us)
    const int64_t bv = (int64_t)8 * m * m * m, xb = (bv + kTile * (kBlock / 64) - 1) / (kTile * (kBlock / 64));
    const int64_t groups = (int64_t)L * ((C + kTile - 1) / kTile);
    const dim3 gd((unsigned)xb, (unsigned)std::min<int64_t>({groups, 65535, (kNNWaves / (kBlock / 64) + xb - 1) / xb}));
    const dim3 bd(kBlock);
    switch (dtype * 2 + (cubic ? 1 : 0)) {
        case LSDF_F32 * 2 + 1: hipLaunchKernelGGL((build_nn_kernel<true, LSDF_F32>), gd, bd, 0, s, a, static_cast<const float*>(grid_buf)); break;
        case LSDF_F32 * 2: hipLaunchKernelGGL((build_nn_kernel<false, LSDF_F32>), gd, bd, 0, s, a, static_cast<const float*>(grid_buf)); break;
        case LSDF_BF16 * 2 + 1: hipLaunchKernelGGL((build_nn_kernel<true, LSDF_BF16>), gd, bd, 0, s, a, static_cast<const uint16_t*>(grid_buf)); break;
        case LSDF_BF16 * 2: hipLaunchKernelGGL((build_nn_kernel<false, LSDF_BF16>), gd, bd, 0, s, a, static_cast<const uint16_t*>(grid_buf)); break;
        case LSDF_F16 * 2 + 1: hipLaunchKernelGGL((build_nn_kernel<true, LSDF_F16>), gd, bd, 0, s, a, static_cast<const _Float16*>(grid_buf)); break;
        default: hipLaunchKernelGGL((build_nn_kernel<false, LSDF_F16>), gd, bd, 0, s, a, static_cast<const _Float16*>(grid_buf)); break;
    }
    return check_launch("robot_sdf_build_frnn");
}

namespace {

size_t words256(int64_t words) { return ((size_t)words * 4 + 255) / 256 * 256; }

void runtime_layout(int64_t V, int64_t M, int64_t* bitmap_words, size_t* list_off, size_t* total) {
    *bitmap_words = (V + 31) / 32;
    const size_t count_off = words256(*bitmap_words);
    *list_off = count_off + 256;
    *total = *list_off + words256(std::min<int64_t>(M, V));
}

}  // namespace

LSDF_API int lsdf_robot_sdf_query_workspace_size(const lsdf_env* env, int64_t M, size_t* bytes) {
    using namespace lsdf;
    clear_error();
    int64_t V = 0;
    int rc = check_env("robot_sdf_query_workspace_size", env, &V);
    if (rc != LSDF_OK) return rc;
    if (M < 0) return fail(LSDF_E_SHAPE, "robot_sdf_query_workspace_size: M < 0");
    if (!bytes) return fail(LSDF_E_INVALID_ARG, "robot_sdf_query_workspace_size: bytes is NULL");
    int64_t bw = 0;
    size_t lo = 0;
    runtime_layout(V, M, &bw, &lo, bytes);
    return LSDF_OK;
}

LSDF_API int lsdf_robot_sdf_query(const float* robot_sdf, int32_t C, const lsdf_env* env, const float* points,
                                  int64_t M, float* out_dist, void* workspace, size_t ws_bytes, void* stream) {
    using namespace lsdf;
    clear_error();
    int64_t V = 0;
    int rc = check_env("robot_sdf_query", env, &V);
    if (rc != LSDF_OK) return rc;
    if (C < 0 || M < 0 || M > LSDF_MAX_POINTS) return fail(LSDF_E_SHAPE, "robot_sdf_query: size out of range");
    if (C == 0) return LSDF_OK;
    if (!robot_sdf || !out_dist || !workspace || (M > 0 && !points))
        return fail(LSDF_E_INVALID_ARG, "robot_sdf_query: NULL device pointer");
    if ((reinterpret_cast<uintptr_t>(workspace) & 255) != 0)
        return fail(LSDF_E_INVALID_ARG, "robot_sdf_query: workspace is not 256-byte aligned");
    RuntimeArgs a{};
    size_t list_off = 0, need = 0;
    runtime_layout(V, M, &a.bitmap_words, &list_off, &need);
    if (ws_bytes < need) return fail(LSDF_E_SHAPE, "robot_sdf_query: workspace has %zu bytes, needs %zu", ws_bytes, need);
    for (int ax = 0; ax < 3; ++ax) {
        a.lo[ax] = env->lo[ax];
        a.n[ax] = env->n[ax];
    }
    a.r = env->voxel;
    a.C = C;
    a.points = points;
    a.M = M;
    char* ws = static_cast<char*>(workspace);
    a.bitmap = reinterpret_cast<uint32_t*>(ws);
    a.count = reinterpret_cast<uint32_t*>(ws + words256(a.bitmap_words));
    a.list = reinterpret_cast<uint32_t*>(ws + list_off);
    a.rs = robot_sdf;
    a.out_dist = out_dist;
    hipStream_t s = as_stream(stream);
    hipLaunchKernelGGL(runtime_zero_kernel, dim3((unsigned)((a.bitmap_words + kBlock - 1) / kBlock)), dim3(kBlock), 0, s,
                       a);
    if ((rc = check_launch("robot_sdf_query (zero)")) != LSDF_OK) return rc;
    if (M > 0) {
        hipLaunchKernelGGL(voxelise_kernel, dim3((unsigned)((M + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, a);
        if ((rc = check_launch("robot_sdf_query (voxelise)")) != LSDF_OK) return rc;
    }
    hipLaunchKernelGGL(gather_kernel, dim3((unsigned)C), dim3(kBlock), 0, s, a);
    return check_launch("robot_sdf_query (gather)");
}
