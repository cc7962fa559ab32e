// Learned per-link SDF surrogate: evaluation, clearance with exact-grid
// fallback, training (forward, backward, weight gradients, Adam) and labels.
#include <algorithm>
#include <cmath>

#include "grid_sample.hpp"
#include "mlp_common.hpp"

namespace {

using namespace lsdf;
using namespace lsdf::mlp;

constexpr int kBlock = 512;                 // 8 waves
constexpr int kWaves = kBlock / 64;
constexpr int kSplit = 512;                 // samples per weight-gradient split
constexpr int kBlocksPerCu = 2;             // 69 KB of LDS per block
// The clearance query: 12 waves share one copy of the staged weights, the 3
// waves per SIMD that its register budget (168 VGPRs) allows; one workgroup
// per CU
constexpr int kQueryBlock = 768;
constexpr int kQueryWaves = kQueryBlock / 64;
constexpr int kTileChunk = 8;               // 32-pair tiles a wave takes at a time: 256 points of one configuration
constexpr int kChunkPts = kTileChunk * TILE;
constexpr int kRounds = kChunkPts / 64;      // a chunk's points, one per lane
constexpr int kMaxTake = 16;                // chunks a wave takes at a time, at most
constexpr int kQueueCap = TILE + kChunkPts;        // pairs waiting: fewer than a tile, and a chunk's

struct Domain {
    float cen[3];
    float inv[3];    // 1 / half
    float core[3];   // half extents of the core box
    float bound;     // remainder bound B (+inf: unbounded)
    float inv_bound; // 1 / B, 0 when B = +inf
};

// A pair's link-frame point relative to the domain centre (u), its
// normalised network input (xh) and whether it lies in the domain, from the
// pose (R, t) and the world point: the same operations in every kernel that
// decides or evaluates pairs, so that they agree bit for bit.
__device__ inline bool pair_frame(const float (&R)[9], const float (&tr)[3], const Domain& dm, float x, float y,
                                  float z, float (&u)[3], float (&xh)[3]) {
    const float dx = x - tr[0], dy = y - tr[1], dz = z - tr[2];
    float mx = 0.0f;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float l = fmaf(R[a], dx, fmaf(R[3 + a], dy, R[6 + a] * dz));   // (R^T d)_a
        u[a] = l - dm.cen[a];
        xh[a] = u[a] * dm.inv[a];
        mx = fmaxf(mx, fabsf(xh[a]));
    }
    return mx <= 1.0f;
}

// Whether every point of sphere (x, y, z, radius) has E - B above thr at this
// pose: E at the centre (pair_frame's and core_distance's arithmetic) less
// the radius, less B, above thr.
__device__ inline bool sphere_beyond(const float4& sph, const float (&R)[9], const float (&tr)[3], const Domain& dm,
                                     float thr) {
    float u[3], xh[3];
    pair_frame(R, tr, dm, sph.x, sph.y, sph.z, u, xh);
    return (core_distance(u[0], u[1], u[2], dm.core) - sph.w) - dm.bound > thr;
}

// A pose's rotation (row-major) and translation.
struct Pose {
    float R[9], t[3];
};
__device__ inline void load_pose(const float* T, Pose& o) {
#pragma unroll
    for (int r = 0; r < 3; ++r) {
#pragma unroll
        for (int s = 0; s < 3; ++s) o.R[3 * r + s] = T[4 * r + s];
        o.t[r] = T[4 * r + 3];
    }
}

__device__ inline float wave_min(float v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = fminf(v, __shfl_xor(v, off, 64));
    return v;
}

__device__ inline float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// ---------------------------------------------------------------------------
// evaluation at given link-frame points
// ---------------------------------------------------------------------------

struct EvalArgs {
    Domain d;
    const float* params;
    const float* points;
    float* out;
    int64_t N;
    int64_t tiles;
};

__global__ __launch_bounds__(kBlock) void mlp_eval_kernel(EvalArgs p) {
    __shared__ __align__(16) __bf16 sW2[WTILE_ELEMS];
    __shared__ __align__(16) __bf16 sW3[WTILE_ELEMS];
    __shared__ SmallParams sp;
    stage_weights(sW2, p.params + OFF_W2, false);
    stage_weights(sW3, p.params + OFF_W3, false);
    stage_small(&sp, p.params);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int64_t t = (int64_t)blockIdx.x * kWaves + wave; t < p.tiles; t += (int64_t)gridDim.x * kWaves) {
        float xh[NT][3], e[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int64_t j = min(t * TILE + 16 * nt + (lane & 15), p.N - 1);
            float u[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                u[a] = p.points[3 * j + a] - p.d.cen[a];
                xh[nt][a] = u[a] * p.d.inv[a];
            }
            e[nt] = core_distance(u[0], u[1], u[2], p.d.core);
        }
        float m[NT];
        forward_tile<NT>(sW2, sW3, &sp, xh, m);
        if (lane < 16) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const int64_t j = t * TILE + 16 * nt + lane;
                float t;
                if (j < p.N) p.out[j] = bounded_share(m[nt], p.d.bound, p.d.inv_bound, t) + e[nt];
            }
        }
    }
}

// ---------------------------------------------------------------------------
// clearance: network per pair, exact grid below the margin
// ---------------------------------------------------------------------------

struct QueryMlpArgs {
    LinkGrid link[LSDF_MAX_LINKS];
    Domain dom[LSDF_MAX_LINKS];
    const float* link_T;
    const float* params;
    const void* grid;
    const float* points;
    uint32_t* keys;
    const float* ubound;     // [C][L] upper bounds U of the first kernel, or NULL (no bound: no skipping)
    const float4* chunk_sph; // [ceil(M / 256)] spheres bounding each chunk's points (when ubound != NULL)
    const int32_t* seed;     // [2][C][L] the chunks holding the pair that gave U and the sampled pair
                             // nearest the core box (-1: none), taken first
    int64_t M;
    int32_t take;            // chunks a wave takes at a time
    int32_t C;
    int32_t L;
    float margin;
};

// The value of E - B above which a pair of (c, i) cannot hold its minimum: the
// upper bound U, the smallest value found so far by any wave (the key; a stale
// read is larger, so still a bound from above), and the margin, below which a
// pair may take the grid's value.
__device__ inline float threshold(const QueryMlpArgs& p, int c, int i) {
    float lim = p.ubound[(int64_t)c * p.L + i];
    const uint32_t kv = __hip_atomic_load(&p.keys[(int64_t)c * p.L + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (kv) lim = fminf(lim, lsdf::from_ordered_bits(~kv));
    return fmaxf(lim, p.margin);
}

// Orders one wave's accesses to its queue (the hardware keeps them in order;
// this keeps the compiler from moving them).
__device__ inline void queue_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// A pair waiting for the network: its point relative to the domain centre, its
// configuration, and the point's number (for the grid's value).
struct PairQueue {
    float4 u_c[kQueryWaves][kQueueCap];   // u, configuration bits
    int64_t point[kQueryWaves][kQueueCap];
};

// The clearance query.  Every workgroup takes every link in turn (its weights
// staged once per link); a link's chunks (256 points of one configuration) are
// dealt round-robin to the workgroups, and a workgroup's waves take them a
// few at a time from a counter in LDS: the pairs a bounded query must
// evaluate cluster (points near a link, at configurations near the obstacle),
// so a fixed share per wave would leave the workgroup waiting on its busiest
// wave at every link.  A lane tests one of the chunks taken; the pairs of those
// that pass are tested one per lane, and the pairs that may hold a minimum wait
// in a queue of the wave's, from which the network takes 32 at a time,
// whichever chunks and configurations they came from.  (Evaluating every
// 16-pair half of a tile that held one such pair ran the network on 1.4 times
// the pairs, and each pair was tested by four lanes.)
// Bound by the VALU work of the network's SiLUs (72 % VALU busy): 500 x 100,000
// x 7 with the network on 5.7 % of the pairs 4.69 -> 3.26 ms, 60 x 8,000 x 7
// 0.80 -> 0.20 ms.
template <bool CUBIC, int DT>
// The register budget of 3 waves per SIMD (168 VGPRs) also schedules the tile
// loop better than the default 2 (248).
__global__ __launch_bounds__(kQueryBlock) __attribute__((amdgpu_waves_per_eu(3, 3))) void query_mlp_kernel(QueryMlpArgs p) {
    __shared__ __align__(16) __bf16 sW2[WTILE_ELEMS];
    __shared__ __align__(16) __bf16 sW3[WTILE_ELEMS];
    __shared__ SmallParams sp;
    __shared__ PairQueue sq;
    __shared__ int s_next;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float4* const q_u = sq.u_c[wave];
    int64_t* const q_j = sq.point[wave];
    const int64_t groups = (p.M + kChunkPts - 1) / kChunkPts;   // chunks per configuration
    const int64_t nchunks = (int64_t)p.C * groups;
    // a bounded query first takes, per configuration, the chunk that holds the
    // pair that gave U (slots below C), then the chunk holding the sampled
    // pair nearest the core box (slots C to 2 C: where a minimum that falls
    // back to the grid lies), so that the keys hold a small value early and
    // the other chunks skip against it; every other chunk then follows (the
    // seed slots of (c, i) process their chunks in any case)
    const int64_t nseed = p.seed ? 2 * (int64_t)p.C : 0;
    for (int i = 0; i < p.L; ++i) {
        const float* P = p.params + (int64_t)i * NPARAM;
        __syncthreads();   // every wave is done with the previous link's weights and chunks
        if (threadIdx.x == 0) s_next = 0;
        stage_weights(sW2, P + OFF_W2, false);
        stage_weights(sW3, P + OFF_W3, false);
        stage_small(&sp, P);
        __syncthreads();

        const LinkGrid& lg = p.link[i];
        const Domain& dm = p.dom[i];
        const typename GridT<DT>::T* G = static_cast<const typename GridT<DT>::T*>(p.grid) + lg.offset;
        int run_c = -1;          // configuration whose minimum so far is `run` (unbounded query)
        float run = INFINITY;
        int waiting = 0;         // pairs in the queue, wave-uniform, below kBatch between rounds
        auto put = [&](int c, float v) {
            if (v < INFINITY) atomicMax(&p.keys[(int64_t)c * p.L + i], ~lsdf::ordered_bits(v));
        };
        // the network on the last n <= TILE pairs of the queue
        auto evaluate = [&](int n) {
            waiting -= n;
            queue_fence();
            float xh[NT][3], e[NT], m[NT];
            int c[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const float4 q = q_u[waiting + min(16 * nt + (lane & 15), n - 1)];
                const float u[3] = {q.x, q.y, q.z};
#pragma unroll
                for (int a = 0; a < 3; ++a) xh[nt][a] = u[a] * dm.inv[a];
                e[nt] = core_distance(u[0], u[1], u[2], dm.core);
                c[nt] = __float_as_int(q.w);
            }
            static_assert(NT == 2, "a batch of two 16-pair halves");
            forward_tile<NT>(sW2, sW3, &sp, xh, m);
            float best = INFINITY;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                float v = INFINITY;
                if (lane < 16 && 16 * nt + lane < n) {
                    // below the margin the grid's value replaces the estimate;
                    // a point outside the grid box keeps the estimate, since
                    // the grid has no value there
                    float tb;
                    const float est = bounded_share(m[nt], dm.bound, dm.inv_bound, tb) + e[nt];
                    v = est;
                    if (est < p.margin) {
                        const float* x = p.points + 3 * q_j[waiting + 16 * nt + lane];
                        const GridMap gm = grid_map(lg, p.link_T + ((int64_t)c[nt] * p.L + i) * 12);
                        const float g = sample_or_inf<CUBIC, DT>(G, lg, gm, x[0], x[1], x[2]);
                        if (g < INFINITY) v = g;
                    }
                }
                m[nt] = v;
                best = fminf(best, v);
            }
            const int c0 = __builtin_amdgcn_readfirstlane(c[0]);
            if (__ballot(c[0] != c0 || c[1] != c0)) {   // pairs of several configurations
                if (lane < 16) {
                    put(c[0], m[0]);
                    put(c[1], m[1]);
                }
            } else if (p.ubound) {
                // the minimum goes to the key at once, so that later chunks of
                // (c, i), on any wave, skip against it
                best = wave_min(best);
                if (lane == 0) put(c0, best);
            } else {
                if (c0 != run_c) {
                    if (run_c >= 0 && lane == 0) put(run_c, run);
                    run_c = c0;
                    run = INFINITY;
                }
                run = fminf(run, wave_min(best));
            }
            queue_fence();
        };
        for (;;) {
            int slot = 0;
            if (lane == 0) slot = atomicAdd(&s_next, p.take);
            slot = __builtin_amdgcn_readfirstlane(slot);
            const int64_t v0 = (int64_t)blockIdx.x + (int64_t)slot * gridDim.x;
            if (v0 >= nseed + nchunks) break;
            // a lane per chunk taken: its configuration and whether it is to be
            // done at all (a chunk whose bounding sphere keeps every pair's E - B
            // above the threshold is not: E is 1-Lipschitz in the link-frame
            // point, so E >= E(centre) - radius over the sphere, the radius
            // widened far beyond the FP32 rounding of E)
            const int64_t vs = v0 + (int64_t)lane * gridDim.x;
            bool take = lane < p.take && vs < nseed + nchunks;
            int c = 0, grp = 0;
            if (take) {
                if (vs < nseed) {
                    c = (int)(vs < p.C ? vs : vs - p.C);
                    grp = p.seed[vs * p.L + i];
                    // the near chunk when it is not the first one already
                    take = grp >= 0 && !(vs >= p.C && grp == p.seed[(int64_t)c * p.L + i]);
                } else {
                    c = (int)((vs - nseed) / groups);
                    grp = (int)((vs - nseed) - (int64_t)c * groups);
                    if (p.seed)   // taken in the seed slots
                        take = grp != p.seed[(int64_t)c * p.L + i] && grp != p.seed[((int64_t)p.C + c) * p.L + i];
                }
            }
            if (take && p.ubound) {
                Pose o;
                load_pose(p.link_T + ((int64_t)c * p.L + i) * 12, o);
                take = !sphere_beyond(p.chunk_sph[grp], o.R, o.t, dm, threshold(p, c, i));
            }
            // a chunk's points, fetched while the chunk before it is evaluated
            float x[kRounds][3];
            auto fetch = [&](int g) {
                const int64_t j0 = (int64_t)g * kChunkPts + lane;
#pragma unroll
                for (int r = 0; r < kRounds; ++r)
#pragma unroll
                    for (int a = 0; a < 3; ++a) x[r][a] = p.points[3 * min(j0 + 64 * r, p.M - 1) + a];
            };
            uint64_t left = __ballot(take);
            if (left) fetch(__builtin_amdgcn_readlane(grp, __builtin_ctzll(left)));
            while (left) {   // wave-uniform
                const int from = __builtin_ctzll(left);
                left &= left - 1;
                const int cc = __builtin_amdgcn_readlane(c, from);
                const int64_t j0 = (int64_t)__builtin_amdgcn_readlane(grp, from) * kChunkPts + lane;
                Pose o;
                load_pose(p.link_T + ((int64_t)cc * p.L + i) * 12, o);
                // the threshold again: it may have fallen since
                const float thr = p.ubound ? threshold(p, cc, i) : INFINITY;
                // a pair with E - B above thr cannot hold the minimum (its value
                // exceeds the value of some pair: a found minimum, or the upper
                // bound U of a pair that cannot fall back); compared squared,
                // with room for the rounding on either side (a pair too many
                // changes nothing)
                const float reach = fmaxf(thr + dm.bound, 0.0f) * 1.00001f + 1e-6f, reach2 = reach * reach;
                float u[kRounds][3];
                uint64_t mask[kRounds];
#pragma unroll
                for (int r = 0; r < kRounds; ++r) {
                    float xh[3];
                    const bool in = pair_frame(o.R, o.t, dm, x[r][0], x[r][1], x[r][2], u[r], xh);
                    mask[r] = __ballot(j0 + 64 * r < p.M && in && core_distance2(u[r][0], u[r][1], u[r][2], dm.core) <= reach2);
                }
#pragma unroll
                for (int r = 0; r < kRounds; ++r) {
                    if (mask[r] >> lane & 1) {
                        const int at = waiting + __builtin_popcountll(mask[r] & ((1ull << lane) - 1));
                        q_u[at] = make_float4(u[r][0], u[r][1], u[r][2], __int_as_float(cc));
                        q_j[at] = j0 + 64 * r;
                    }
                    waiting += __builtin_popcountll(mask[r]);
                }
                if (left) fetch(__builtin_amdgcn_readlane(grp, __builtin_ctzll(left)));
                while (waiting >= TILE) evaluate(TILE);
            }
        }
        if (waiting > 0) evaluate(waiting);
        if (run_c >= 0 && lane == 0) put(run_c, run);
    }
}

// Bounding spheres of the learned query's chunks (256 points), eight lanes per
// chunk, 32 points each: the centre of the points' box and the largest
// distance to it, widened by a relative 1e-5 and by 1e-4 m, which covers the
// FP32 rounding of the pose and of E (about 1e-6 m on clouds a few metres
// across) many times over.
__global__ __launch_bounds__(256) void mlp_sphere_kernel(const float* __restrict__ points, int64_t M, float4* chunk_sph) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    const int64_t j0 = k / kTileChunk * kChunkPts + k % kTileChunk;   // every eighth point
#pragma unroll 8
    for (int t = 0; t < TILE; ++t) {
        const int64_t j = min(j0 + t * kTileChunk, M - 1);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            lo[a] = fminf(lo[a], points[3 * j + a]);
            hi[a] = fmaxf(hi[a], points[3 * j + a]);
        }
    }
    float cen[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
        for (int o = 1; o < kTileChunk; o <<= 1) {
            lo[a] = fminf(lo[a], __shfl_xor(lo[a], o, 64));
            hi[a] = fmaxf(hi[a], __shfl_xor(hi[a], o, 64));
        }
        cen[a] = 0.5f * (lo[a] + hi[a]);
    }
    float r2 = 0.0f;
#pragma unroll 8
    for (int t = 0; t < TILE; ++t) {
        const int64_t j = min(j0 + t * kTileChunk, M - 1);
        const float dx = points[3 * j] - cen[0], dy = points[3 * j + 1] - cen[1], dz = points[3 * j + 2] - cen[2];
        r2 = fmaxf(r2, fmaf(dx, dx, fmaf(dy, dy, dz * dz)));
    }
#pragma unroll
    for (int o = 1; o < kTileChunk; o <<= 1) r2 = fmaxf(r2, __shfl_xor(r2, o, 64));
    if (k % kTileChunk == 0 && k / kTileChunk * kChunkPts < M)
        chunk_sph[k / kTileChunk] = make_float4(cen[0], cen[1], cen[2], fmaf(sqrtf(r2), 1.00001f, 1e-4f));
}

// First kernel of a bounded learned query: per (configuration c, link i),
// U = the smallest E + B over a sample of the in-domain pairs with
// E - B >= margin (pairs whose estimate, at least E - B, cannot fall below
// the margin and so cannot take the grid's value): the first point of every
// 32-point tile; +inf if none.  Every such pair's value is at most its
// E + B, so U bounds the minimum from above (over any sample of pairs), and a
// pair with E - B > U cannot hold it.  Also the chunk holding the sampled
// pair that gave U (the query takes it first).  A workgroup takes one link
// and kBoundConfigs configurations (their poses in scalar registers) and
// strides over the tiles; the pair arithmetic is pair_frame's and
// core_distance's, as in the query.
constexpr int kBoundBlock = 256;
constexpr int kBoundConfigs = 4;

struct BoundArgs {
    Domain dom[LSDF_MAX_LINKS];
    const float* link_T;
    const float* points;
    float* ubound;           // [C][L]
    int32_t* seed;           // [2][C][L] chunk (256 points) of a pair that gave U, -1 if U = +inf; then
                             // that of the sampled in-domain pair with the smallest E, -1 if none
    int64_t M;
    int32_t C;
    int32_t L;
    float margin;
};

__global__ __launch_bounds__(kBoundBlock) void mlp_bound_kernel(BoundArgs p) {
    const int i = blockIdx.y;
    const int c0 = blockIdx.x * kBoundConfigs;
    const Domain& dm = p.dom[i];
    float R[kBoundConfigs][9], tr[kBoundConfigs][3], ub[kBoundConfigs], en[kBoundConfigs];
    int ag[kBoundConfigs], ng[kBoundConfigs];
#pragma unroll
    for (int k = 0; k < kBoundConfigs; ++k) {
        const int c = min(c0 + k, p.C - 1);
        const float* T = p.link_T + ((int64_t)c * p.L + i) * 12;
        for (int r = 0; r < 3; ++r) {
            for (int s = 0; s < 3; ++s) R[k][3 * r + s] = T[4 * r + s];
            tr[k][r] = T[4 * r + 3];
        }
        ub[k] = INFINITY;
        ag[k] = -1;
        en[k] = INFINITY;
        ng[k] = -1;
    }
    for (int64_t j = (int64_t)threadIdx.x * TILE; j < p.M; j += (int64_t)kBoundBlock * TILE) {
        const float x = p.points[3 * j + 0], y = p.points[3 * j + 1], z = p.points[3 * j + 2];
#pragma unroll
        for (int k = 0; k < kBoundConfigs; ++k) {
            float u[3], xh[3];
            if (!pair_frame(R[k], tr[k], dm, x, y, z, u, xh)) continue;
            const float e = core_distance(u[0], u[1], u[2], dm.core);
            if (e - dm.bound >= p.margin && e + dm.bound < ub[k]) {
                ub[k] = e + dm.bound;
                ag[k] = (int)(j / kChunkPts);
            }
            if (e < en[k]) {
                en[k] = e;
                ng[k] = (int)(j / kChunkPts);
            }
        }
    }
    __shared__ float s_ub[kBoundConfigs][kBoundBlock / 64], s_en[kBoundConfigs][kBoundBlock / 64];
    __shared__ int s_ag[kBoundConfigs], s_ng[kBoundConfigs];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x < kBoundConfigs) {
        s_ag[threadIdx.x] = INT32_MAX;
        s_ng[threadIdx.x] = INT32_MAX;
    }
#pragma unroll
    for (int k = 0; k < kBoundConfigs; ++k) {
        const float w = wave_min(ub[k]), we = wave_min(en[k]);
        if (lane == 0) {
            s_ub[k][wave] = w;
            s_en[k][wave] = we;
        }
    }
    __syncthreads();
    // the block minima, and the lowest chunk holding a pair that gives each
#pragma unroll
    for (int k = 0; k < kBoundConfigs; ++k) {
        float v = INFINITY, ve = INFINITY;
        for (int w = 0; w < kBoundBlock / 64; ++w) {
            v = fminf(v, s_ub[k][w]);
            ve = fminf(ve, s_en[k][w]);
        }
        if (v < INFINITY && ub[k] == v) atomicMin(&s_ag[k], ag[k]);
        if (ve < INFINITY && en[k] == ve) atomicMin(&s_ng[k], ng[k]);
    }
    __syncthreads();
    if (threadIdx.x < kBoundConfigs && c0 + (int)threadIdx.x < p.C) {
        float v = INFINITY, ve = INFINITY;
        for (int w = 0; w < kBoundBlock / 64; ++w) {
            v = fminf(v, s_ub[threadIdx.x][w]);
            ve = fminf(ve, s_en[threadIdx.x][w]);
        }
        const int64_t o = (int64_t)(c0 + threadIdx.x) * p.L + i;
        p.ubound[o] = v;
        p.seed[o] = v < INFINITY ? s_ag[threadIdx.x] : -1;
        p.seed[(int64_t)p.C * p.L + o] = ve < INFINITY ? s_ng[threadIdx.x] : -1;
    }
}

// ---------------------------------------------------------------------------
// training
// ---------------------------------------------------------------------------

// Per-link slices of the training workspace ([L][...] arrays).
struct TrainBufs {
    float* dz1;     // [L][B / 32][128][32] (act_at), as are the next five
    __bf16* h1;
    __bf16* h2;
    __bf16* h3;
    __bf16* dz2;
    __bf16* dz3;
    float* xh;      // [L][B][3]
    float* dm;      // [L][B]
    float* loss;    // [L][B / TILE_TRAIN]
    float* gpart;   // [L][nsplit][NPARAM]
};

// Place of unit u of sample c in a link's plane: 32 samples of all units
// together.  With a unit's B samples in a row (16 KB apart at B = 8,192) the
// 16 rows of an operand's load and of a tile's store all met the same memory
// channel.
__device__ inline int64_t act_at(int u, int64_t c) { return ((c >> 5) * H + u) * 32 + (c & 31); }

struct TrainArgs {
    Domain dom[LSDF_MAX_LINKS];
    TrainBufs w;
    const float* params;
    const float* samples;
    const float* labels;
    const int32_t* bidx;
    int64_t N;
    int32_t B;
    int32_t nsplit;
};

// Forward and backward pass of one wave tile of the batch (16 samples per
// wave), in one kernel: the pre-activations never leave the registers.
// SiLU(z) and SiLU'(z) share one sigmoid, s = 1 / (1 + exp(-z)):
// SiLU = z s, SiLU' = s (1 + z (1 - s)).  SiLU'(z2) and SiLU'(z3) of every
// unit a lane holds are kept for the backward pass; SiLU'(z1), needed last,
// is recomputed from the inputs then (the same bits), which keeps the kernel
// within its registers.  A lane's units in a result tile (16 mt + 4 g + r) are the units of its B
// operand slots (perm_unit), so the kept derivatives line up with the
// backward products with no exchange.
// 7 x 8,192 samples: 74 -> 53 us with the activations stored 32 samples of all
// units at a time (66) and the 128 KB of weights staged once for all rounds.
// Stored for the weight gradients: the rounded activations h1, h2, h3, the
// rounded deltas dz3, dz2 and the FP32 delta dz1, the normalised inputs and
// dm = d(loss)/dm; the loss per tile.
#ifndef LSDF_TRAIN_BLOCK
#define LSDF_TRAIN_BLOCK 512
#endif
constexpr int kTrainBlock = LSDF_TRAIN_BLOCK;
constexpr int kTrainWaves = kTrainBlock / 64;
static_assert(kSplit % (TILE_TRAIN * kTrainWaves) == 0, "a batch of whole workgroups");

__global__ __launch_bounds__(kTrainBlock) void train_fwdbwd_kernel(TrainArgs p) {
    __shared__ __align__(16) __bf16 sW2[WTILE_ELEMS];
    __shared__ __align__(16) __bf16 sW3[WTILE_ELEMS];
    __shared__ __align__(16) __bf16 sW3t[WTILE_ELEMS];
    __shared__ __align__(16) __bf16 sW2t[WTILE_ELEMS];
    __shared__ SmallParams sp;
    const int l = blockIdx.y;
    const float* P = p.params + (int64_t)l * NPARAM;
    stage_weights(sW2, P + OFF_W2, false);
    stage_weights(sW3, P + OFF_W3, false);
    stage_weights(sW3t, P + OFF_W3, true);
    stage_weights(sW2t, P + OFF_W2, true);
    stage_small(&sp, P);
    __syncthreads();
    static_assert(NT_TRAIN == 1, "one 16-sample column tile per wave");
    const int lane = threadIdx.x & 63;
    const int g = lane >> 4;
    const int col = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t B = p.B;
    const int64_t lB = (int64_t)l * B;
    const int64_t plane = (int64_t)l * H * B;
    for (int tt = blockIdx.x * kTrainWaves + wave; tt < p.B / TILE_TRAIN; tt += gridDim.x * kTrainWaves) {
        const int64_t s_idx = (int64_t)tt * TILE_TRAIN + col;   // this lane's sample in the batch
        int64_t k = p.bidx ? (int64_t)p.bidx[lB + s_idx] : s_idx;
        k = min(max(k, (int64_t)0), p.N - 1);              // a bad index reads a valid sample
        const int64_t idx = (int64_t)l * p.N + k;
        const Domain& d = p.dom[l];
        float xh[3], u3[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            u3[a] = p.samples[3 * idx + a] - d.cen[a];
            xh[a] = u3[a] * d.inv[a];
        }
        const float e_core = core_distance(u3[0], u3[1], u3[2], d.core);
        if (lane < 16) {
#pragma unroll
            for (int a = 0; a < 3; ++a) p.w.xh[(lB + s_idx) * 3 + a] = xh[a];
        }
        // where this lane's unit 4 g of its sample goes in each plane
        const int64_t at = plane + act_at(4 * g, s_idx);
        __bf16 *const h1 = p.w.h1 + at, *const h2 = p.w.h2 + at, *const h3 = p.w.h3 + at;
        __bf16 *const dz2 = p.w.dz2 + at, *const dz3 = p.w.dz3 + at;
        float* const dz1 = p.w.dz1 + at;
        asm volatile("" ::: "memory");

        // ---- forward ----
        float g2[8][4], g3[8][4];   // SiLU' of this lane's units
        bf16x8 b[4];
        const float xk = input_operand(xh, g);
#pragma unroll
        for (int mt = 0; mt < 8; ++mt) {
            const f32x4 z = input_layer(&sp, mt, lane, xk);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const __bf16 h = (__bf16)silu(z[r]);
                b[mt >> 1][(mt & 1) * 4 + r] = h;
                h1[(16 * mt + r) * 32] = h;
            }
        }
        float m = 0.0f;
#pragma unroll
        for (int layer = 0; layer < 2; ++layer) {
            const __bf16* sW = layer == 0 ? sW2 : sW3;
            const float* bias = layer == 0 ? sp.b2 : sp.b3;
            f32x4 acc[8];
#pragma unroll
            for (int mt = 0; mt < 8; ++mt)
                acc[mt] = f32x4{bias[16 * mt + 4 * g], bias[16 * mt + 4 * g + 1], bias[16 * mt + 4 * g + 2],
                                bias[16 * mt + 4 * g + 3]};
            asm volatile("" ::: "memory");   // the layer's weight reads stay inside the layer
#pragma unroll
            for (int mt = 0; mt < 8; ++mt)
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lds_a(sW, mt, s, lane), b[s], acc[mt], 0, 0, 0);
            if (layer == 0) {
#pragma unroll
                for (int mt = 0; mt < 8; ++mt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float z = acc[mt][r];
                        const float sg = sigmoid(z);
                        const __bf16 h = (__bf16)(z * sg);
                        g2[mt][r] = silu_grad_of(z, sg);
                        b[mt >> 1][(mt & 1) * 4 + r] = h;
                        h2[(16 * mt + r) * 32] = h;
                    }
            } else {
                float part = 0.0f;
#pragma unroll
                for (int mt = 0; mt < 8; ++mt)
#pragma unroll
                    for (int r = 0; r < 4; r += 2) {
                        const int u = 16 * mt + 4 * g + r;
                        __bf16 hh[2];
#pragma unroll
                        for (int q = 0; q < 2; ++q) {
                            const float z = acc[mt][r + q];
                            const float sg = sigmoid(z);
                            hh[q] = (__bf16)(z * sg);
                            g3[mt][r + q] = silu_grad_of(z, sg);
                            h3[(16 * mt + r + q) * 32] = hh[q];
                        }
                        const bf16x2 hp = {hh[0], hh[1]};
                        const bf16x2 wp = {sp.w4b[u], sp.w4b[u + 1]};
                        part = __builtin_amdgcn_fdot2_f32_bf16(hp, wp, part, false);
                    }
                part += __shfl_xor(part, 16, 64);
                part += __shfl_xor(part, 32, 64);
                m = part + sp.b4;
            }
        }
        // loss of the estimate (bounded network share + core distance) and its
        // derivative with respect to the network's output m
        float tb;
        const float share = bounded_share(m, d.bound, d.inv_bound, tb);
        const float r_ = (share + e_core) - p.labels[idx];
        float dm = (r_ > 0.0f ? 1.0f : (r_ < 0.0f ? -1.0f : 0.0f)) / (float)B;
        if (d.inv_bound != 0.0f) dm *= 1.0f - tb * tb;
        float absr = lane < 16 ? fabsf(r_) : 0.0f;
        if (lane < 16) p.w.dm[lB + s_idx] = dm;
        absr = wave_sum(absr);
        if (lane == 0) p.w.loss[(int64_t)l * (B / TILE_TRAIN) + tt] = absr;

        // ---- backward ----
        // dz3 = dm * w4 * SiLU'(z3), rounded: B operand of dh2 = W3^T dz3
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int u = perm_unit(s, 8 * g + e);
                const __bf16 db = (__bf16)(dm * sp.w4[u] * g3[2 * s + (e >> 2)][e & 3]);
                b[s][e] = db;
                dz3[(16 * (2 * s + (e >> 2)) + (e & 3)) * 32] = db;   // unit u
            }
#pragma unroll
        for (int layer = 0; layer < 2; ++layer) {
            const __bf16* sW = layer == 0 ? sW3t : sW2t;
            f32x4 acc[8];
#pragma unroll
            for (int mt = 0; mt < 8; ++mt) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
            asm volatile("" ::: "memory");
#pragma unroll
            for (int mt = 0; mt < 8; ++mt)
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lds_a(sW, mt, s, lane), b[s], acc[mt], 0, 0, 0);
#pragma unroll
            for (int mt = 0; mt < 8; ++mt) {
                const f32x4 z1 = layer == 0 ? f32x4{} : input_layer(&sp, mt, lane, xk);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if (layer == 0) {
                        // dz2 = (W3^T dz3) * SiLU'(z2), rounded: B operand of dh1 = W2^T dz2
                        const __bf16 db = (__bf16)(acc[mt][r] * g2[mt][r]);
                        b[mt >> 1][(mt & 1) * 4 + r] = db;
                        dz2[(16 * mt + r) * 32] = db;
                    } else {
                        // dz1 = (W2^T dz2) * SiLU'(z1), kept in FP32
                        dz1[(16 * mt + r) * 32] = acc[mt][r] * silu_grad_of(z1[r], sigmoid(z1[r]));
                    }
                }
            }
        }
    }
}

// Weight gradients over one split of the batch.  Workgroups with z = 0:
// dW3 = dz3^T h2 and dW2 = dz2^T h1 on MFMA (K = samples), a 64 x 64 output
// quarter per wave, the next K step's operands (1 KB each, contiguous) loaded
// while the current one multiplies.  z = 1: W1 and b1; z = 2: w4 and b4; z = 3:
// b3; z = 4: b2: 16 units per wave, a lane sums samples 8 g to 8 g + 7 of each
// 32 of a unit, in the order total() needs.
// Bound by memory (147 MB of activations and partial sums at 7 x 8,192): 83 ->
// 28.5 us with the activations 32 samples of all units at a time (rows of B
// samples are 16 KB apart, all on one channel) and a wave per 16 small gradients
// instead of one.  (A workgroup per product, 64 x 32 a wave: 33 us; biases from
// the products' operands: 36 us, spills.)
__global__ __launch_bounds__(kBlock) void train_wgrad_kernel(TrainArgs p) {
    const int l = blockIdx.y;
    const int split = blockIdx.x;
    const int lane = threadIdx.x & 63;
    const int g = lane >> 4;
    const int col = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t B = p.B;
    const int64_t plane = (int64_t)l * H * B;
    const int64_t k0 = (int64_t)split * kSplit;
    constexpr int kSteps = kSplit / 32, kStep = 32 * H;
    // the lane's operand slots: unit col of a tile of 16, samples 8 g .. 8 g + 7
    const int64_t at = plane + act_at(0, k0) + col * 32 + 8 * g;
    float* gp = p.w.gpart + ((int64_t)l * p.nsplit + split) * NPARAM;

    // a unit's sum from the lane's sums of every 64th sample: in the order of a
    // butterfly over 64 lanes that hold one each
    auto total = [&](const float (&s)[2][8]) {
        float t[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            t[k] = s[0][k] + s[1][k];
            t[k] += __shfl_xor(t[k], 32, 64);
            t[k] += __shfl_xor(t[k], 16, 64);
        }
        return ((t[0] + t[4]) + (t[2] + t[6])) + ((t[1] + t[5]) + (t[3] + t[7]));
    };

    if (blockIdx.z == 0) {
        const bool third = wave < 4;
        const int r0 = 64 * (wave >> 1 & 1), c0 = 64 * (wave & 1);
        const __bf16* A = (third ? p.w.dz3 : p.w.dz2) + at + r0 * 32;   // out
        const __bf16* Bm = (third ? p.w.h2 : p.w.h1) + at + c0 * 32;    // in
        f32x4 acc[4][4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        bf16x8 a[2][4], bb[2][4];
        auto load = [&](int k) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                a[k % 2][t] = *reinterpret_cast<const bf16x8*>(A + k * kStep + t * 512);
                bb[k % 2][t] = *reinterpret_cast<const bf16x8*>(Bm + k * kStep + t * 512);
            }
        };
        load(0);
#pragma unroll
        for (int k = 0; k < kSteps; ++k) {
            if (k + 1 < kSteps) load(k + 1);
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
#pragma unroll
                for (int nt = 0; nt < 4; ++nt)
                    acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[k % 2][mt], bb[k % 2][nt], acc[mt][nt], 0, 0, 0);
            }
        }
        const int off = third ? OFF_W3 : OFF_W2;
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int nt = 0; nt < 4; ++nt)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    gp[off + (r0 + 16 * mt + 4 * g + r) * H + (c0 + 16 * nt + col)] = acc[mt][nt][r];
        return;
    }

    static_assert(kWaves * 16 == H, "a tile of 16 units per wave");
    const int64_t lB = (int64_t)l * B;
    const int u = 16 * wave + col;
    if (blockIdx.z == 1) {
        const float* d1 = p.w.dz1 + at + wave * 512;
        const float* x = p.w.xh + (lB + k0 + 8 * g) * 3;
        float s[4][2][8] = {};
#pragma unroll 2
        for (int k = 0; k < kSteps; ++k) {
            float d[8], xs[24];
#pragma unroll
            for (int t = 0; t < 2; ++t) *reinterpret_cast<float4*>(d + 4 * t) = reinterpret_cast<const float4*>(d1 + k * kStep)[t];
#pragma unroll
            for (int t = 0; t < 6; ++t) *reinterpret_cast<float4*>(xs + 4 * t) = reinterpret_cast<const float4*>(x + k * 96)[t];
#pragma unroll
            for (int t = 0; t < 8; ++t) {
#pragma unroll
                for (int a = 0; a < 3; ++a) s[a][k % 2][t] = fmaf(d[t], xs[3 * t + a], s[a][k % 2][t]);
                s[3][k % 2][t] += d[t];
            }
        }
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const float t = total(s[a]);
            if (g == 0) gp[a < 3 ? OFF_W1 + 3 * u + a : OFF_B1 + u] = t;
        }
    } else if (blockIdx.z == 2) {
        const __bf16* h = p.w.h3 + at + wave * 512;
        const float* dm = p.w.dm + lB + k0 + 8 * g;
        float s[2][8] = {}, sb[2][8] = {};
#pragma unroll 4
        for (int k = 0; k < kSteps; ++k) {
            const bf16x8 hv = *reinterpret_cast<const bf16x8*>(h + k * kStep);
            float d[8];
#pragma unroll
            for (int t = 0; t < 2; ++t) *reinterpret_cast<float4*>(d + 4 * t) = reinterpret_cast<const float4*>(dm + k * 32)[t];
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                s[k % 2][t] = fmaf(d[t], (float)hv[t], s[k % 2][t]);
                sb[k % 2][t] += d[t];
            }
        }
        const float t = total(s), tb = total(sb);
        if (g == 0) gp[OFF_W4 + u] = t;
        if (wave == 0 && lane == 0) gp[OFF_B4] = tb;
    } else {
        const bool third = blockIdx.z == 3;
        const __bf16* d = (third ? p.w.dz3 : p.w.dz2) + at + wave * 512;
        float s[2][8] = {};
#pragma unroll 8
        for (int k = 0; k < kSteps; ++k) {
            const bf16x8 v = *reinterpret_cast<const bf16x8*>(d + k * kStep);
#pragma unroll
            for (int t = 0; t < 8; ++t) s[k % 2][t] += (float)v[t];
        }
        const float t = total(s);
        if (g == 0) gp[(third ? OFF_B3 : OFF_B2) + u] = t;
    }
}

struct ReduceArgs {
    TrainBufs w;
    float* params;
    float* m;
    float* v;
    float* grad_out;
    float* loss_out;
    int32_t L;
    int32_t B;
    int32_t nsplit;
    int32_t adam;
    float lr;      // step size
    float beta1;
    float beta2;
    float eps;
    float c1;      // 1 - beta1^t
    float c2;      // 1 - beta2^t
};

// Sums the split partials into the gradient; optionally applies Adam.
__global__ __launch_bounds__(256) void train_reduce_kernel(ReduceArgs p) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k < (int64_t)p.L * NPARAM) {
        const int l = (int)(k / NPARAM);
        const int pk = (int)(k - (int64_t)l * NPARAM);
        // the split partials in order, their loads issued 8 at a time
        float gsum = 0.f;
        for (int s0 = 0; s0 < p.nsplit; s0 += 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                v[u] = s0 + u < p.nsplit ? p.w.gpart[((int64_t)l * p.nsplit + s0 + u) * NPARAM + pk] : 0.f;
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (s0 + u < p.nsplit) gsum += v[u];
        }
        if (p.grad_out) p.grad_out[k] = gsum;
        if (p.adam) {
            const float mk = p.beta1 * p.m[k] + (1.0f - p.beta1) * gsum;
            const float vk = p.beta2 * p.v[k] + (1.0f - p.beta2) * gsum * gsum;
            p.m[k] = mk;
            p.v[k] = vk;
            p.params[k] -= p.lr * (mk / p.c1) / (sqrtf(vk / p.c2) + p.eps);
        }
    }
    // mean loss per link: wave l sums link l's tiles (lanes stride them, then a butterfly)
    if (p.loss_out && k < (int64_t)p.L * 64) {
        const int l = (int)(k >> 6), lane = (int)(k & 63);
        const int tiles = p.B / TILE_TRAIN;
        float s = 0.f;
        for (int t = lane; t < tiles; t += 64) s += p.w.loss[(int64_t)l * tiles + t];
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
        if (lane == 0) p.loss_out[l] = s / (float)p.B;
    }
}

// ---------------------------------------------------------------------------
// host helpers
// ---------------------------------------------------------------------------

int make_domain(const lsdf_mlp_domain& d, int index, Domain* out) {
    for (int a = 0; a < 3; ++a) {
        if (!std::isfinite(d.centre[a]) || !std::isfinite(d.half[a]) || !(d.half[a] > 0.0f))
            return fail(LSDF_E_INVALID_ARG, "mlp domain %d: centre must be finite and half > 0", index);
        if (!std::isfinite(d.core_half[a]) || !(d.core_half[a] >= 0.0f))
            return fail(LSDF_E_INVALID_ARG, "mlp domain %d: core_half must be finite and >= 0", index);
        out->cen[a] = d.centre[a];
        out->inv[a] = (float)(1.0 / (double)d.half[a]);
        out->core[a] = d.core_half[a];
    }
    if (!(d.bound > 0.0f))   // NaN, zero or negative; +inf is allowed
        return fail(LSDF_E_INVALID_ARG, "mlp domain %d: bound must be > 0 (or +inf)", index);
    out->bound = d.bound;
    out->inv_bound = std::isinf(d.bound) ? 0.0f : (float)(1.0 / (double)d.bound);
    return LSDF_OK;
}

int device_cus() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    return cus;
}

size_t align256(size_t x) { return (x + 255) / 256 * 256; }

// Carves the training workspace; returns the bytes it needs.
size_t train_layout(int32_t L, int32_t B, char* base, TrainBufs* w) {
    const size_t f_plane = align256((size_t)L * H * B * sizeof(float));
    const size_t h_plane = align256((size_t)L * H * B * sizeof(__bf16));
    const int nsplit = B / kSplit;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char* p = base ? base + off : nullptr;
        off += align256(bytes);
        return p;
    };
    TrainBufs t{};
    t.dz1 = (float*)take(f_plane);
    t.h1 = (__bf16*)take(h_plane);
    t.h2 = (__bf16*)take(h_plane);
    t.h3 = (__bf16*)take(h_plane);
    t.dz2 = (__bf16*)take(h_plane);
    t.dz3 = (__bf16*)take(h_plane);
    t.xh = (float*)take((size_t)L * B * 3 * sizeof(float));
    t.dm = (float*)take((size_t)L * B * sizeof(float));
    t.loss = (float*)take((size_t)L * (B / TILE_TRAIN) * sizeof(float));
    t.gpart = (float*)take((size_t)L * nsplit * NPARAM * sizeof(float));
    if (w) *w = t;
    return off;
}

int check_train_sizes(int32_t L, int32_t B, int64_t N) {
    if (L < 1 || L > LSDF_MAX_LINKS) return fail(LSDF_E_SHAPE, "mlp train: L = %d out of [1, %d]", (int)L, LSDF_MAX_LINKS);
    if (B < kSplit || B % kSplit != 0) return fail(LSDF_E_SHAPE, "mlp train: B = %d must be a positive multiple of %d", (int)B, kSplit);
    if (N < 1) return fail(LSDF_E_SHAPE, "mlp train: N = %lld < 1", (long long)N);
    return LSDF_OK;
}

int train_common(const float* params, float* adam_m, float* adam_v, int64_t t, float lr, float beta1, float beta2,
                 float eps, bool adam, const lsdf_mlp_domain* domains, int32_t L, const float* samples,
                 const float* labels, int64_t N, const int32_t* batch_index, int32_t B, float* loss_out,
                 float* grad_out, void* workspace, size_t ws_bytes, void* stream) {
    int rc = check_train_sizes(L, B, N);
    if (rc != LSDF_OK) return rc;
    if (!params || !domains || !samples || !labels || !workspace)
        return fail(LSDF_E_INVALID_ARG, "mlp train: NULL pointer");
    if (adam && (!adam_m || !adam_v)) return fail(LSDF_E_INVALID_ARG, "mlp train: NULL Adam moments");
    if (adam && t < 1) return fail(LSDF_E_INVALID_ARG, "mlp train: step t = %lld < 1", (long long)t);
    if (adam && !(std::isfinite(lr) && std::isfinite(beta1) && std::isfinite(beta2) && std::isfinite(eps) &&
                  beta1 >= 0.f && beta1 < 1.f && beta2 >= 0.f && beta2 < 1.f && eps >= 0.f))
        return fail(LSDF_E_INVALID_ARG, "mlp train: bad Adam hyper-parameters");
    if ((reinterpret_cast<uintptr_t>(workspace) & 255) != 0)
        return fail(LSDF_E_INVALID_ARG, "mlp train: workspace is not 256-byte aligned");
    const size_t need = train_layout(L, B, nullptr, nullptr);
    if (ws_bytes < need) return fail(LSDF_E_SHAPE, "mlp train: workspace has %zu bytes, needs %zu", ws_bytes, need);
    TrainArgs a{};
    for (int i = 0; i < L; ++i) {
        rc = make_domain(domains[i], i, &a.dom[i]);
        if (rc != LSDF_OK) return rc;
    }
    train_layout(L, B, static_cast<char*>(workspace), &a.w);
    a.params = params;
    a.samples = samples;
    a.labels = labels;
    a.bidx = batch_index;
    a.N = N;
    a.B = B;
    a.nsplit = B / kSplit;
    hipStream_t s = as_stream(stream);
    // one workgroup per CU at a time (LDS): as many rounds of tiles as they
    // need, so that the weights are staged once
    const int groups = B / (TILE_TRAIN * kTrainWaves), cus = std::max(1, device_cus());
    const int rounds = (int)(((int64_t)groups * L + cus - 1) / cus);
    const dim3 tiles_grid((groups + rounds - 1) / rounds, L);
    hipLaunchKernelGGL(train_fwdbwd_kernel, tiles_grid, dim3(kTrainBlock), 0, s, a);
    if ((rc = check_launch("mlp train forward and backward")) != LSDF_OK) return rc;
    hipLaunchKernelGGL(train_wgrad_kernel, dim3(a.nsplit, L, 5), dim3(kBlock), 0, s, a);
    if ((rc = check_launch("mlp train weight gradients")) != LSDF_OK) return rc;
    ReduceArgs r{};
    r.w = a.w;
    r.params = const_cast<float*>(params);
    r.m = adam_m;
    r.v = adam_v;
    r.grad_out = grad_out;
    r.loss_out = loss_out;
    r.L = L;
    r.B = B;
    r.nsplit = a.nsplit;
    r.adam = adam ? 1 : 0;
    if (adam) {
        r.lr = lr;
        r.beta1 = beta1;
        r.beta2 = beta2;
        r.eps = eps;
        r.c1 = (float)(1.0 - std::pow((double)beta1, (double)t));
        r.c2 = (float)(1.0 - std::pow((double)beta2, (double)t));
    }
    const int64_t total = (int64_t)L * NPARAM;
    hipLaunchKernelGGL(train_reduce_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, r);
    return check_launch("mlp train reduce");
}

}  // namespace

LSDF_API int lsdf_mlp_eval(const float* params, const lsdf_mlp_domain* domain, const float* points, int64_t N,
                           float* out, void* stream) {
    clear_error();
    if (!domain) return fail(LSDF_E_INVALID_ARG, "mlp_eval: domain is NULL");
    if (N < 0) return fail(LSDF_E_SHAPE, "mlp_eval: N < 0");
    if (N == 0) return LSDF_OK;
    if (!params || !points || !out) return fail(LSDF_E_INVALID_ARG, "mlp_eval: NULL device pointer");
    EvalArgs a{};
    int rc = make_domain(*domain, 0, &a.d);
    if (rc != LSDF_OK) return rc;
    const int cus = device_cus();
    if (cus <= 0) return fail(LSDF_E_DEVICE, "mlp_eval: cannot read the device's compute-unit count");
    a.params = params;
    a.points = points;
    a.out = out;
    a.N = N;
    a.tiles = (N + TILE - 1) / TILE;
    const int64_t blocks = std::min<int64_t>((int64_t)cus * kBlocksPerCu, (a.tiles + kWaves - 1) / kWaves);
    hipLaunchKernelGGL(mlp_eval_kernel, dim3((unsigned)blocks), dim3(kBlock), 0, as_stream(stream), a);
    return check_launch("mlp_eval");
}

LSDF_API int lsdf_query_min_distance_mlp(const float* link_T, int32_t C, int32_t L, const lsdf_grid* grids,
                                         const void* grid_buf, const float* mlp_params, const lsdf_mlp_domain* domains,
                                         float margin, const float* points, int64_t M, float* out_dist,
                                         int32_t* out_link, float* out_link_dist, uint32_t flags, void* workspace,
                                         size_t ws_bytes, void* stream) {
    clear_error();
    if (flags != 0) return fail(LSDF_E_UNSUPPORTED, "query_mlp: unsupported flags 0x%x", flags);
    if (C < 0 || M < 0) return fail(LSDF_E_SHAPE, "query_mlp: negative size");
    if (L < 1 || L > LSDF_MAX_LINKS) return fail(LSDF_E_SHAPE, "query_mlp: L = %d out of [1, %d]", (int)L, LSDF_MAX_LINKS);
    if (!grids || !domains) return fail(LSDF_E_INVALID_ARG, "query_mlp: grids or domains is NULL");
    if (std::isnan(margin)) return fail(LSDF_E_INVALID_ARG, "query_mlp: margin is NaN");
    if (C == 0) return LSDF_OK;
    if (!link_T || !grid_buf || !mlp_params || !out_dist || !out_link || !workspace)
        return fail(LSDF_E_INVALID_ARG, "query_mlp: NULL device pointer");
    if (M > 0 && !points) return fail(LSDF_E_INVALID_ARG, "query_mlp: points is NULL");
    if ((reinterpret_cast<uintptr_t>(workspace) & 255) != 0)
        return fail(LSDF_E_INVALID_ARG, "query_mlp: workspace is not 256-byte aligned");
    size_t need = 0;
    int rc = lsdf_query_workspace_size(C, L, M, flags, &need);
    if (rc != LSDF_OK) return rc;
    if (ws_bytes < need) return fail(LSDF_E_SHAPE, "query_mlp: workspace has %zu bytes, needs %zu", ws_bytes, need);
    QueryMlpArgs a{};
    bool cubic = true;
    const int dtype = grids[0].dtype;
    for (int i = 0; i < L; ++i) {
        if ((rc = prepare_link_grid(grids[i], i, &a.link[i])) != LSDF_OK) return rc;
        if ((rc = make_domain(domains[i], i, &a.dom[i])) != LSDF_OK) return rc;
        if (grids[i].dtype != dtype) return fail(LSDF_E_UNSUPPORTED, "query_mlp: grids of one query must share a dtype");
        cubic = cubic && a.link[i].cubic;
    }
    hipStream_t s = as_stream(stream);
    a.link_T = link_T;
    a.params = mlp_params;
    a.grid = grid_buf;
    a.points = points;
    a.keys = static_cast<uint32_t*>(workspace);
    a.M = M;
    a.C = C;
    a.L = L;
    a.margin = margin;
    const int64_t chunks = (int64_t)C * ((M + kChunkPts - 1) / kChunkPts);
    if (chunks > 0) {
        const int cus = device_cus();
        if (cus <= 0) return fail(LSDF_E_DEVICE, "query_mlp: cannot read the device's compute-unit count");
        // one workgroup per CU (each takes every link in turn), no more than
        // the chunks of one link need
        const dim3 grid((unsigned)std::max<int64_t>(1, std::min<int64_t>(cus, (chunks + kQueryWaves - 1) / kQueryWaves)));
        if ((rc = launch_zero_words(a.keys, (int64_t)C * L, s)) != LSDF_OK) return rc;
        // a wave comes back for more about 8 times, so that the last ones taken
        // even the waves out (big batches of chunks cost less each: 8 a time
        // 3.74 ms, 4 or 16 4.0 and 3.9 ms for 500 x 100,000 x 7)
        a.take = (int32_t)std::max<int64_t>(1, std::min<int64_t>(kMaxTake, chunks / (8 * kQueryWaves * (int64_t)grid.x)));
        bool bounded = false;
        for (int i = 0; i < L; ++i) bounded = bounded || a.dom[i].inv_bound != 0.0f;
        if (bounded) {
            // the upper bounds, after the keys in the workspace (which holds
            // the plain query's tables too, far more than C L words)
            float* ub = reinterpret_cast<float*>(static_cast<char*>(workspace) + ((size_t)C * L * 4 + 255) / 256 * 256);
            // then the chunk spheres and the seed chunks
            const int64_t nt = (M + TILE - 1) / TILE;
            float4* csph = reinterpret_cast<float4*>(reinterpret_cast<char*>(ub) + ((size_t)C * L * 4 + 255) / 256 * 256);
            int32_t* seed = reinterpret_cast<int32_t*>(csph + (nt + kTileChunk - 1) / kTileChunk);
            const size_t used = static_cast<size_t>(reinterpret_cast<char*>(seed + 2 * (int64_t)C * L) -
                                                    static_cast<char*>(workspace));
            if (used > need) return fail(LSDF_E_SHAPE, "query_mlp: workspace layout exceeds %zu bytes", need);
            BoundArgs b{};
            for (int i = 0; i < L; ++i) b.dom[i] = a.dom[i];
            b.link_T = link_T;
            b.points = points;
            b.ubound = ub;
            b.seed = seed;
            b.M = M;
            b.C = C;
            b.L = L;
            b.margin = margin;
            hipLaunchKernelGGL(mlp_bound_kernel, dim3((unsigned)((C + kBoundConfigs - 1) / kBoundConfigs), L),
                               dim3(kBoundBlock), 0, s, b);
            if ((rc = check_launch("query_min_distance_mlp bounds")) != LSDF_OK) return rc;
            hipLaunchKernelGGL(mlp_sphere_kernel, dim3((unsigned)((nt + 255) / 256)), dim3(256), 0, s, points, M, csph);
            if ((rc = check_launch("query_min_distance_mlp spheres")) != LSDF_OK) return rc;
            a.ubound = ub;
            a.chunk_sph = csph;
            a.seed = seed;
        }
        hipEvent_t ev0, ev1;
        take_kernel_events(&ev0, &ev1);
        if (ev0 && hipEventRecord(ev0, s) != hipSuccess) return fail(LSDF_E_DEVICE, "query_mlp: event record failed");
        switch (dtype * 2 + (cubic ? 1 : 0)) {
            case LSDF_F32 * 2 + 1: hipLaunchKernelGGL((query_mlp_kernel<true, LSDF_F32>), grid, dim3(kQueryBlock), 0, s, a); break;
            case LSDF_F32 * 2: hipLaunchKernelGGL((query_mlp_kernel<false, LSDF_F32>), grid, dim3(kQueryBlock), 0, s, a); break;
            case LSDF_BF16 * 2 + 1: hipLaunchKernelGGL((query_mlp_kernel<true, LSDF_BF16>), grid, dim3(kQueryBlock), 0, s, a); break;
            case LSDF_BF16 * 2: hipLaunchKernelGGL((query_mlp_kernel<false, LSDF_BF16>), grid, dim3(kQueryBlock), 0, s, a); break;
            case LSDF_F16 * 2 + 1: hipLaunchKernelGGL((query_mlp_kernel<true, LSDF_F16>), grid, dim3(kQueryBlock), 0, s, a); break;
            default: hipLaunchKernelGGL((query_mlp_kernel<false, LSDF_F16>), grid, dim3(kQueryBlock), 0, s, a); break;
        }
        if ((rc = check_launch("query_min_distance_mlp")) != LSDF_OK) return rc;
        if (ev1 && hipEventRecord(ev1, s) != hipSuccess) return fail(LSDF_E_DEVICE, "query_mlp: event record failed");
    }
    return lsdf::launch_query_finalize(chunks > 0 ? a.keys : nullptr, out_dist, out_link, out_link_dist, C, L,
                                       s);
}

LSDF_API int lsdf_mlp_train_workspace_size(int32_t L, int32_t B, size_t* bytes) {
    clear_error();
    if (!bytes) return fail(LSDF_E_INVALID_ARG, "mlp_train_workspace_size: bytes is NULL");
    int rc = check_train_sizes(L, B, 1);
    if (rc != LSDF_OK) return rc;
    *bytes = train_layout(L, B, nullptr, nullptr);
    return LSDF_OK;
}

LSDF_API int lsdf_mlp_loss_grad(const float* params, const lsdf_mlp_domain* domains, int32_t L, const float* samples,
                                const float* labels, int64_t N, const int32_t* batch_index, int32_t B, float* loss_out,
                                float* grad_out, void* workspace, size_t ws_bytes, void* stream) {
    clear_error();
    if (!grad_out) return fail(LSDF_E_INVALID_ARG, "mlp_loss_grad: grad_out is NULL");
    return train_common(params, nullptr, nullptr, 0, 0.f, 0.f, 0.f, 0.f, false, domains, L, samples, labels, N,
                        batch_index, B, loss_out, grad_out, workspace, ws_bytes, stream);
}

LSDF_API int lsdf_mlp_train_step(float* params, float* adam_m, float* adam_v, int64_t t, float lr, float beta1,
                                 float beta2, float eps, const lsdf_mlp_domain* domains, int32_t L,
                                 const float* samples, const float* labels, int64_t N, const int32_t* batch_index,
                                 int32_t B, float* loss_out, float* grad_out, void* workspace, size_t ws_bytes,
                                 void* stream) {
    clear_error();
    return train_common(params, adam_m, adam_v, t, lr, beta1, beta2, eps, true, domains, L, samples, labels, N,
                        batch_index, B, loss_out, grad_out, workspace, ws_bytes, stream);
}
