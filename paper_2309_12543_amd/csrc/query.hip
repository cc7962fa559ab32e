// Batched clearance query (Sec. III-A): per configuration c, the minimum over
// obstacle points and links of link i's grid SDF read at the point moved into
// link i's frame.
//
// Work layout:
//   * a wave tests one link i and 64 consecutive configurations (one per
//     lane, a tile); each lane holds the world-to-grid affine map of its pose
//     (the inverse pose of Eq. 4 with the grid scaling folded in) in 12 VGPRs;
//   * obstacle points and their bounds are wave-uniform: they stream through
//     scalar loads into SGPRs, so mapping a point is 9 FMAs with no
//     cross-lane traffic;
//   * points are culled by boxes: a first small kernel bounds every block of
//     8 consecutive points and every group of 8 blocks by an axis-aligned
//     box, and a wave skips a group or block when no lane's grid box can hold
//     any of its points (the box centre is mapped with the lane's own map; the
//     test widens the grid box by the box's half extents times the map's
//     magnitudes plus a bound on FP32 rounding, so the skip is exact).
//     Consecutive points of a voxel grid lie on a line, which a sphere bounds
//     badly: 500 waypoints against 20,000 such points left 7,700 to 9,000
//     blocks to test with spheres and leave 300 to 3,900 with boxes, and half
//     to a tenth of the groups;
//   * a block that survives is recorded in a list in the workgroup's LDS;
//     after a barrier the workgroup's waves share out the listed blocks, and
//     so on until no chunk is left;
//   * a listed block's points are tested one by one; the pairs (point,
//     configuration) inside a grid box, a quarter of the lanes where there is
//     one, wait in a queue of the wave's, from which 64 at a time gather their
//     8 corners and interpolate, whichever block and tile they came from.
//     Their minima go to a table of the workgroup's tiles in LDS (an atomic
//     max per pair), and from there to global memory once per list (one
//     atomic max per pair straight to global memory took longer than all of
//     the rest);
//   * a call may hold many trajectories, each a range of configurations
//     checked against its own range of points (a re-planned path against
//     its latest cloud); a plain query is the one-trajectory case.  The
//     ranges come from device arrays, and the plan that turns them into
//     work (chunk counts and their prefix sums) is built on the device by
//     the first kernel, so that no call reads anything back to the host and
//     a whole step can be captured once in a graph and replayed with new
//     ranges;
//   * the first kernel also writes, per (link, configuration), the lane's
//     map and culling thresholds into a field-major table (one coalesced
//     load per field per chunk) and zeroes the keys;
//   * the iteration space (trajectory, link, 64-configuration tile, point)
//     is cut into chunks of a tunable number of 8-point blocks (a chunk takes
//     every n-th group of its trajectory's cloud, or a part of one group),
//     dealt to the waves over the whole grid or inside per-XCD slices
//     (blocks b = x mod 8 take a contiguous slice, which keeps an XCD on one
//     or two links' grids in its L2); the four waves of a workgroup take
//     chunks from four different parts of the order;
//   * per-pair minima merge across workgroups with one unsigned atomic max on
//     a complemented order-preserving key; a last small kernel turns the keys
//     into the outputs (the kernel boundary orders it after every atomic,
//     with no device fence).
// Bound by the VALU and by the latency of its dependent loads.  GPU time of a
// call on one MI355X, all three kernels, before (spheres, a gather per point
// and lane, minima straight to global memory) and now: 50 waypoints, 2,000
// points 17.3 -> 14.9 us; 500, 20,000 31 -> 24 us; 500, 100,000, 128^3 bf16
// 77 -> 46 us; 333, 12,345 all near the arm 191 -> 70 us; 64 paths of 50 to
// 1,000 with clouds of 5,000 to 200,000 2.16 -> 1.46 ms.
#include <algorithm>
#include <atomic>
#include <mutex>

#include "fk_chain.hpp"
#include "grid_sample.hpp"

namespace {

using lsdf::GridT;
using lsdf::LinkGrid;
using lsdf::inside;

#ifndef LSDF_QUERY_BLOCK
#define LSDF_QUERY_BLOCK 256         // threads per workgroup of the query kernel
#endif
constexpr int kBlock = LSDF_QUERY_BLOCK;
constexpr int kWavesPerBlock = kBlock / 64;
constexpr int kXcds = 8;
constexpr float kFar = 1e30f;       // centred coordinate of unused lanes: never inside

constexpr int kBlockPts = 8;        // points per block, the smallest unit culled by a box
constexpr int kGroupBlocks = 8;     // blocks per group, the unit a chunk is made of
constexpr int kGroupPts = kBlockPts * kGroupBlocks;
#ifndef LSDF_QUERY_GROUP_BATCH
#define LSDF_QUERY_GROUP_BATCH 4    // groups of a chunk loaded and tested together
#endif
constexpr int kGroupBatch = LSDF_QUERY_GROUP_BATCH;

// Default tiling: as many workgroups per CU as can be resident at once (so
// that no wave of the persistent grid waits for another to finish; 8 if
// the runtime cannot say), chunks dealt over the whole grid, one chunk per
// wave of the grid at most: the fewest groups per chunk that give no more
// chunks than waves for the call's sizes (with offset arrays, the capacities C
// and M, as if every trajectory had its share of both), as the waves with two
// chunks would end last (C = 500, M = 100,000, L = 7: 11 groups 45.7 us, 8
// groups and 1.3 chunks a wave 48.6).  Where that takes more than 16, 8 (16
// paths: 101 us, with 16 groups 110), and 16 where the chunks are dealt (64
// paths: 1.46 ms, with 8 groups 1.60); a quarter of a group where the call is
// so small that an eighth of the waves would have a group (C = 50, M = 2,000:
// 15.1 us with quarters, 16.3 with halves, 18.2 with whole ones; C = 200, M =
// 8,000 near the arm, halves where the rule takes whole groups: 59 us, not 49).
constexpr int kDefaultBlocksPerCu = 8;
constexpr int kDefaultSchedule = LSDF_SCHED_INTERLEAVED;

// From this many chunks per wave on, all but each wave's first are dealt as
// the workgroups come for them: 64 paths, 55 chunks a wave, 1.43 ms against
// 1.72 dealt beforehand; 16 paths, 2 chunks a wave, 120 us against 111.
constexpr int kDealChunks = 16;

int default_chunk_blocks(int64_t K, int64_t C, int64_t L, int64_t M, int64_t waves) {
    const int64_t tiles = L * std::max(K, (C + 63) / 64), groups = ((M + K - 1) / K + kGroupPts - 1) / kGroupPts;
    if (tiles * groups * kGroupBlocks <= waves) return kGroupBlocks / 4;
    if (tiles * groups >= kDealChunks * 16 * waves) return 16 * kGroupBlocks;
    const int64_t most = K == 1 ? 16 : 8;   // (the trajectories of a batch differ: 12 groups 107 us, 8 101)
    int64_t g = std::max<int64_t>(1, tiles * groups / waves);
    while (g <= most && tiles * ((groups + g - 1) / g) > waves) ++g;
    return (int)(g <= most ? g : 8) * kGroupBlocks;
}
constexpr int kRunsPerBlock = 24;   // runs of chunks a workgroup comes for, about (8: 1.62 ms, 16: 1.48)
constexpr int kMaxRun = 64;         // chunks of a run, at most
constexpr int kMaxChunkPoints = 8192;
constexpr int kMaxBlocksPerCu = 16;

// Work plan of one trajectory, built on the device.  Entry K (one past the
// last trajectory) is a PlanEnd.
struct TrajPlan {
    int64_t chunk_start;       // first chunk of this trajectory
    int64_t m_lo, m_hi;        // points [m_lo, m_hi) of the concatenated cloud
    int32_t c_lo, c_n;         // configurations [c_lo, c_lo + c_n)
    int32_t cgroups;           // ceil(c_n / 64)
    int32_t chunks_per_group;  // ceil(groups of 64 points touched / chunk_groups)
    int32_t pad[2];
};
struct PlanEnd {
    int64_t chunk_start;       // the total chunk count
    int32_t next[kXcds];       // runs of chunks dealt so far, per XCD
    int32_t pad[2];
};
static_assert(sizeof(TrajPlan) == 48 && sizeof(PlanEnd) == sizeof(TrajPlan), "plan entry layout");

// A block of 8 points some lane's box may reach, handed from the wave that
// found it to whichever wave of the workgroup takes it.
struct Block {
    uint32_t index;            // in the concatenated cloud
    uint32_t tile_points;      // its tile, and from bit 16 its points that are the trajectory's
};
// A link and 64 configurations that blocks of the list were found for.
struct Tile {
    int32_t link;
    int32_t c0, n;             // configurations [c0, c0 + n), one per lane
};
// A wave looks for room before each batch of groups and may add all its
// blocks and one tile.
constexpr int kListFull = 512;
constexpr int kListCap = kListFull + kWavesPerBlock * kGroupBatch * kGroupBlocks;
constexpr int kTilesFull = 12;
constexpr int kTileCap = kTilesFull + kWavesPerBlock;
constexpr int kLongList = 64, kTake = 4;
constexpr int kQueueCap = 128;     // pairs waiting: below 64, and the 64 of one point

// A link's grid as the evaluation of mixed pairs reads it, from LDS.
struct GridView {
    float half[3];
    int32_t n[3];
    int64_t offset;
};

struct QueryArgs {
    LinkGrid link[LSDF_MAX_LINKS];
    const float* maps;       // [L][kMapFields][C]
    uint32_t* keys;          // [C][L] complemented ordered keys, 0 = empty
    int64_t M;
    int32_t C;
    int32_t K;               // trajectories
    int32_t L;
    int32_t split;           // a chunk is a 2^-split share of a group (0: whole groups)
    int32_t blocks_per_xcd;
    int32_t schedule;        // LSDF_SCHED_*
};

// Per (link, configuration): the world-to-grid map and the culling
// thresholds, stored field-major ([L][kMapFields][C]) so that a wave's 64
// consecutive configurations read each field with one coalesced load.
constexpr int kMapFields = 15;   // M (9, row-major), w (3), k_a (3)

// A box that holds 64 (a group's) points, widened (see box_of).
struct Box {
    float cx, cy, cz, hx, hy, hz;
};
// The same for 8 points in 16 bytes: the half extents as bytes (x, y, z from
// the low byte) times the power of two whose exponent is the high byte.
struct PackedBox {
    float cx, cy, cz;
    uint32_t h;
};

struct PrepArgs {
    LinkGrid link[LSDF_MAX_LINKS];
    lsdf::DhTable dh;        // used when q != NULL
    const float* q;          // joint angles [C][dof], or NULL: poses come from link_T
    float* link_T_out;       // poses computed from q are stored here when not NULL
    const float* link_T;
    const float* points;
    PackedBox* blocks;       // [ceil(M / 8)]
    Box* groups;             // [ceil(M / 64)]
    TrajPlan* plan;          // [K + 1]
    float* maps;             // [L][kMapFields][C]
    uint32_t* keys;          // [C][L], zeroed here
    const int32_t* c_off;    // device [K + 1] or NULL (one trajectory of all C)
    const int64_t* m_off;    // device [K + 1] or NULL (one trajectory of all M)
    int64_t M;
    int64_t box_base;        // first thread of the box job: C L rounded up to the wave size
    int32_t C;
    int32_t K;
    int32_t L;
    int32_t chunk_groups;    // groups of 64 points per chunk
    int32_t split;           // parts a group is cut into, as a power of two
};

struct FinalizeArgs {
    const uint32_t* keys;    // [C][L], or NULL
    float* out_dist;
    int32_t* out_link;
    float* out_link_dist;
    int32_t C;
    int32_t L;
};

// A 64-bit value that every lane holds alike, moved to scalar registers.
__device__ __forceinline__ int64_t uniform64(int64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// This lane's map v = M [x; y; z] + w (centred grid coordinates) and culling
// thresholds for (link i, configuration c0 + lane), from the table the first
// kernel built; lanes from n on get a map that sends every point far outside
// the box.
struct Map {
    float m00, m01, m02, w0, m10, m11, m12, w1, m20, m21, m22, w2, k0, k1, k2;
};
__device__ __forceinline__ void load_map(const QueryArgs& p, int i, int c0, int n, int lane, Map& m) {
    m = Map{0.f, 0.f, 0.f, kFar, 0.f, 0.f, 0.f, kFar, 0.f, 0.f, 0.f, kFar, 0.f, 0.f, 0.f};
    if (lane < n) {
        const float* f = p.maps + (int64_t)i * kMapFields * p.C + c0;   // wave-uniform
        auto field = [&](int k) { return (f + (int64_t)k * p.C)[(uint32_t)lane]; };
        m.m00 = field(0); m.m01 = field(1); m.m02 = field(2);
        m.m10 = field(3); m.m11 = field(4); m.m12 = field(5);
        m.m20 = field(6); m.m21 = field(7); m.m22 = field(8);
        m.w0 = field(9); m.w1 = field(10); m.w2 = field(11);
        m.k0 = field(12); m.k1 = field(13); m.k2 = field(14);
    }
}
__device__ __forceinline__ void map_point(const Map& m, float x, float y, float z, float& v0, float& v1, float& v2) {
    v0 = fmaf(m.m00, x, fmaf(m.m01, y, fmaf(m.m02, z, m.w0)));
    v1 = fmaf(m.m10, x, fmaf(m.m11, y, fmaf(m.m12, z, m.w1)));
    v2 = fmaf(m.m20, x, fmaf(m.m21, y, fmaf(m.m22, z, m.w2)));
}

// Orders one wave's accesses to its queue (the hardware keeps them in order;
// this keeps the compiler from moving them).
__device__ __forceinline__ void queue_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// What the workgroup holds in LDS: the blocks its waves found (one list, added
// to by all), each wave's queue of pairs, and the links' grids.
struct QueryShared {
    Block block[kListCap];
    float4 pair[kWavesPerBlock][kQueueCap];    // centred grid coordinates; 64 tile + lane
    uint32_t best[kTileCap][64];               // complemented ordered keys, 0 = empty
    Tile tile[kTileCap];
    GridView grid[LSDF_MAX_LINKS];
    int listed;     // blocks in the list
    int tiles;
    int64_t run_q, run_step;   // the workgroup's run of chunks: the first, the distance to the next,
    int run, taken;            // how many, how many of them are taken
    int open;       // waves that left a chunk begun
};

// Where a wave stands: the chunk it has begun or is to begin, and its next group.
struct Walk {
    int64_t q, q_end, q_step;   // (the last two: of chunks dealt beforehand)
    int32_t gb;
    int32_t k;      // the trajectory of chunk q, or an earlier one
    bool has;       // there is a chunk q
    bool fresh;     // it is not begun
};

// Tests chunks until the list is full or the workgroup's run of chunks is
// through.  The boxes of a chunk's groups are tested against every lane's grid
// box, then their blocks'; a block some lane may reach goes to the list.
template <bool DEAL>
__device__ __forceinline__ void collect(const QueryArgs& p, const PackedBox* __restrict__ blocks,
                                        const Box* __restrict__ groups, const TrajPlan* __restrict__ plan, Walk& w,
                                        int lane, QueryShared& sh) {
    auto room = [&] {
        return (__hip_atomic_load(&sh.listed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < kListFull) &
               (__hip_atomic_load(&sh.tiles, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < kTilesFull);
    };
    for (;;) {
        if (!w.has) {
            if (!DEAL) return;
            int n = 0;
            if (lane == 0) n = atomicAdd(&sh.taken, 1);
            n = __builtin_amdgcn_readfirstlane(n);
            if (n >= __builtin_amdgcn_readfirstlane(sh.run)) return;
            w.q = uniform64(sh.run_q) + n * uniform64(sh.run_step);
            w.has = w.fresh = true;
        }
        if (DEAL && w.q < plan[w.k].chunk_start) w.k = 0;
        if (w.q >= plan[w.k + 1].chunk_start) {
            // its trajectory: the last entry whose start is <= q
            int hi = p.K - 1;
            ++w.k;
            while (w.k < hi) {
                const int mid = (w.k + hi + 1) >> 1;
                if (plan[mid].chunk_start <= w.q) w.k = mid; else hi = mid - 1;
            }
        }
        const TrajPlan& t = plan[w.k];
        const int64_t m_lo = t.m_lo, m_hi = t.m_hi;
        const int cgroups = t.cgroups, cpg = t.chunks_per_group;
        // (plain 32-bit and unsigned arithmetic: a small call is bound by the issue of
        // the some 400 mostly scalar instructions each wave needs to reach its
        // boxes; 363 x 8,248 x 7 that meet nothing 12.5 us with signed 64-bit
        // quotients and a modulo in mix_slot, 12.2 so)
        const int64_t local = w.q - t.chunk_start;
        uint32_t g, mc;   // tile (at most L C / 64 of them) and chunk of it
        if (local < ((int64_t)1 << 32)) {
            g = (uint32_t)local / (uint32_t)cpg;
            mc = (uint32_t)local - g * (uint32_t)cpg;
        } else {
            g = (uint32_t)((uint64_t)local / (uint32_t)cpg);
            mc = (uint32_t)(local - (int64_t)g * cpg);
        }
        // places are turned by 0.618 cpg from tile to tile: a workgroup's waves take
        // chunks half a grid or more apart, which would test the same part of the
        // cloud where that is near a multiple of cpg (500 x 100,000 on 128^3 grids
        // beside a table, 2,008 workgroups, cpg 143: 67 us, 53 with the turn; the
        // geometric mean over 12 other scenes is 44.3 us without it and 45.0 with it)
        mc += __umulhi(g * 2654435769u, (uint32_t)cpg);   // both below cpg < 2^31
        if (mc >= (uint32_t)cpg) mc -= (uint32_t)cpg;
        const int i = (int)(g / (uint32_t)cgroups);
        const int cb = (int)(g - (uint32_t)i * (uint32_t)cgroups);
        const int c0 = t.c_lo + cb * 64, cn = min(t.c_n - cb * 64, 64);
        // the trajectory's points lie in groups of 8 blocks of 8 (aligned in the
        // concatenated cloud); chunk mc takes every cpg-th group from the
        // trajectory's group mc, so that points near a link, which lie together
        // in the cloud, spread over the chunks rather than piling onto a few
        // waves
        const int64_t group0 = (uint64_t)m_lo / kGroupPts;
        const int ngroup = (int)((uint64_t)(m_hi + kGroupPts - 1) / kGroupPts - group0);
        const Box* const gbox = groups + group0;
        // blocks of the trajectory, counted from its first group's
        const uint32_t blk0 = ((uint32_t)m_lo & (kGroupPts - 1)) / kBlockPts;
        const uint32_t blk1 = (uint32_t)((uint64_t)(m_hi - group0 * kGroupPts + kBlockPts - 1) / kBlockPts);
        // the share of a group's blocks that is the chunk's (all, or a part)
        const int part = (int)(mc & ((1u << p.split) - 1)), gstep = cpg >> p.split;
        const uint32_t share = ((1u << (kGroupBlocks >> p.split)) - 1) << (part * (kGroupBlocks >> p.split));
        Map m;
        load_map(p, i, c0, cn, lane, m);
        int tile = -1;   // its number, once a block is found for it
        // kGroupBatch groups of the chunk at a time: their boxes are loaded
        // together and tested (one round trip for the batch); only the groups
        // some lane may reach go on to their blocks' boxes
        if (w.fresh) w.gb = (int)(mc >> p.split);
        w.fresh = false;
        for (; w.gb < ngroup; w.gb += kGroupBatch * gstep) {
            if (!room()) return;
            Box bx[kGroupBatch];
#pragma unroll
            for (int k = 0; k < kGroupBatch; ++k)   // past the trajectory's groups: its last one, not tested
                bx[k] = gbox[min(w.gb + k * gstep, ngroup - 1)];
            uint32_t gnear = 0;
            auto test = [&](int k) {
                const Box& b = bx[k];
                float s0, s1, s2;
                map_point(m, b.cx, b.cy, b.cz, s0, s1, s2);
                const float r0 = fmaf(fabsf(m.m00), b.hx, fmaf(fabsf(m.m01), b.hy, fmaf(fabsf(m.m02), b.hz, m.k0)));
                const float r1 = fmaf(fabsf(m.m10), b.hx, fmaf(fabsf(m.m11), b.hy, fmaf(fabsf(m.m12), b.hz, m.k1)));
                const float r2 = fmaf(fabsf(m.m20), b.hx, fmaf(fabsf(m.m21), b.hy, fmaf(fabsf(m.m22), b.hz, m.k2)));
                const bool near = (fabsf(s0) <= r0) & (fabsf(s1) <= r1) & (fabsf(s2) <= r2);
                if (__ballot(near)) gnear |= 1u << k;
            };
            // a full batch with no branch between its tests; of the last one, which
            // is all a small call's wave has, only the groups there are (363 x 8,248
            // x 7 that meet nothing, a group a wave: 13.0 us with all four tested,
            // 12.5; 1,000 x 100,000 x 7, 12 a wave, 25.8 and 25.2)
            if (w.gb + (kGroupBatch - 1) * gstep < ngroup) {
#pragma unroll
                for (int k = 0; k < kGroupBatch; ++k) test(k);
            } else {
#pragma unroll
                for (int k = 0; k < kGroupBatch - 1; ++k) {
                    if (w.gb + k * gstep >= ngroup) break;
                    test(k);
                }
            }
            while (gnear) {   // wave-uniform
                const int kg = __builtin_ctz(gnear);
                gnear &= gnear - 1;
                // a box bounds all points of its group or block, so also the
                // trajectory's share of one it shares with its neighbour
                const uint32_t b0 = kGroupBlocks * (uint32_t)(w.gb + kg * gstep);
                uint32_t valid = share;
                if (b0 < blk0) valid &= ~0u << (blk0 - b0);
                if (b0 + kGroupBlocks > blk1) valid &= (1u << (blk1 - b0)) - 1;
                uint32_t near_mask = 0;
                // (past the last block the array is followed by the groups' boxes
                // and the plan; what is read there is masked out)
                const PackedBox* const pb = blocks + (group0 * kGroupBlocks + b0);
#pragma unroll
                for (int u = 0; u < kGroupBlocks; ++u) {
                    const PackedBox& b = pb[u];
                    float s0, s1, s2;
                    map_point(m, b.cx, b.cy, b.cz, s0, s1, s2);
                    const float unit = __uint_as_float(b.h >> 24 << 23);
                    const float hx = (float)(b.h & 255u), hy = (float)(b.h >> 8 & 255u), hz = (float)(b.h >> 16 & 255u);
                    const float r0 = fmaf(fmaf(fabsf(m.m00), hx, fmaf(fabsf(m.m01), hy, fabsf(m.m02) * hz)), unit, m.k0);
                    const float r1 = fmaf(fmaf(fabsf(m.m10), hx, fmaf(fabsf(m.m11), hy, fabsf(m.m12) * hz)), unit, m.k1);
                    const float r2 = fmaf(fmaf(fabsf(m.m20), hx, fmaf(fabsf(m.m21), hy, fabsf(m.m22) * hz)), unit, m.k2);
                    const bool near = (fabsf(s0) <= r0) & (fabsf(s1) <= r1) & (fabsf(s2) <= r2);
                    if (__ballot(near)) near_mask |= 1u << u;
                }
                near_mask &= valid;
                if (near_mask) {
                    if (tile < 0) {
                        if (lane == 0) tile = atomicAdd(&sh.tiles, 1);
                        tile = __builtin_amdgcn_readfirstlane(tile);
                        if (lane == 0) sh.tile[tile] = Tile{i, c0, cn};
                        sh.best[tile][lane] = 0;
                    }
                    int slot = 0;
                    if (lane == 0) slot = atomicAdd(&sh.listed, __builtin_popcount(near_mask));
                    slot = __builtin_amdgcn_readfirstlane(slot);
                    // lane u writes block u
                    if (lane < kGroupBlocks && (near_mask >> lane & 1)) {
                        const int64_t index = group0 * kGroupBlocks + b0 + lane, j = index * kBlockPts;
                        uint32_t pts = (1u << kBlockPts) - 1;   // the trajectory's points of the block
                        if (j < m_lo) pts &= pts << (m_lo - j);
                        if (j + kBlockPts > m_hi) pts &= (1u << (m_hi - j)) - 1;
                        sh.block[slot + __builtin_popcount(near_mask & ((1u << lane) - 1))] =
                            Block{(uint32_t)index, (uint32_t)tile | pts << 16};
                    }
                }
            }
        }
        if (DEAL) {
            w.has = false;
        } else {
            w.q += w.q_step;
            w.has = w.q < w.q_end;
            w.fresh = true;
        }
    }
}

// Slot of workgroup b (of n) for its wave w: waves 2 and 3 shift by half
// the grid and odd waves count from the other end, so that a workgroup's
// four chunks come from four different parts of the chunk order (early and
// late links, early and late configuration groups).  A bijection of [0, n)
// for each w.
__device__ __forceinline__ int mix_slot(int b, int n, int w) {
    int s = (w & 2) ? b + n / 2 : b;
    if (s >= n) s -= n;
    return (w & 1) ? n - 1 - s : s;
}

// (80 SGPRs let 8 workgroups be resident per CU; with the 106 it would take it
// is 6, though the runtime's occupancy says 7, so that the grid's last seventh
// began when the others ended: 64 paths 1.94 ms.  What spills goes to VGPR
// lanes.)
template <bool CUBIC, int DT, bool DEAL>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_num_sgpr(80))) void query_kernel(
    QueryArgs p, const float* __restrict__ points, const typename GridT<DT>::T* __restrict__ grid,
    const PackedBox* __restrict__ blocks, const Box* __restrict__ groups, TrajPlan* __restrict__ plan) {
    __shared__ QueryShared sh;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t total = plan[p.K].chunk_start;
    // The waves of one workgroup start a grid's (or slice's) width apart, on
    // different links or tiles, so that the shared list evens them out.  From
    // there every wave takes every n-th chunk, or (DEAL) the workgroups take the
    // rest in runs from a counter per XCD.
    const int xcd = blockIdx.x % kXcds;
    const bool slices = p.schedule == LSDF_SCHED_XCD_SLICES;   // each XCD (blocks b = x mod 8) its own range of chunks
    const int64_t lo = slices ? total * xcd / kXcds : 0, hi = slices ? total * (xcd + 1) / kXcds : total;
    const int n0 = slices ? p.blocks_per_xcd : (int)gridDim.x;
    Walk w{};
    w.q = lo + (int64_t)wave * n0 + mix_slot(slices ? (int)blockIdx.x / kXcds : (int)blockIdx.x, n0, wave);
    w.q_end = hi;
    w.q_step = (int64_t)n0 * kWavesPerBlock;
    w.has = w.fresh = w.q < hi;
    // run r is chunks given + r, given + r + nruns, ...: far apart, as the
    // chunks near a link, which cost the most, come together
    const int64_t given = lo + w.q_step;
    const int64_t run = DEAL ? min((int64_t)kMaxRun, max((int64_t)kWavesPerBlock, (hi - given) / (kRunsPerBlock * n0))) : 1;
    const int64_t nruns = DEAL ? (hi - given + run - 1) / run : 0;
    if (threadIdx.x == 0) {
        sh.listed = sh.tiles = sh.open = 0;
        if (DEAL) {
            sh.run = sh.taken = 0;
            sh.run_step = nruns;
        }
    }
    __syncthreads();

    float4* const queue = sh.pair[wave];
    int waiting = 0;   // pairs in the wave's queue
    // the grid values of the queue's last n pairs, one per lane
    auto evaluate = [&](int n) {
        queue_fence();
        waiting -= n;
        if (lane < n) {
            const float4 e = queue[waiting + lane];
            const int at = __float_as_int(e.w);
            const GridView gv = sh.grid[sh.tile[at >> 6].link];
            LinkGrid lg;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                lg.half[a] = gv.half[a];
                lg.n[a] = gv.n[a];
            }
            const float val = lsdf::cell_value<DT>(grid + gv.offset, lg, e.x, e.y, e.z);
            if (val < INFINITY) atomicMax(&sh.best[at >> 6][at & 63], ~lsdf::ordered_bits(val));
        }
        queue_fence();
    };

    for (;;) {
        collect<DEAL>(p, blocks, groups, plan, w, lane, sh);
        if (w.has && lane == 0) atomicAdd(&sh.open, 1);
        __syncthreads();
        const int nd = sh.listed, nt = sh.tiles;
        const bool left = sh.open > 0;
        const bool dry = DEAL && sh.taken >= sh.run;   // the run is through
        if (nd == 0 && !left && (!DEAL || (dry && given >= hi))) break;
        if (threadIdx.x < (unsigned)p.L) {
            const LinkGrid& lg = p.link[threadIdx.x];
            sh.grid[threadIdx.x] =
                GridView{{lg.half[0], lg.half[1], lg.half[2]}, {lg.n[0], lg.n[1], lg.n[2]}, (int64_t)lg.offset};
        }
        __syncthreads();
        int64_t next_q = hi;
        if (dry && given < hi && threadIdx.x == 0) {   // fetched while the list is worked off
            const int64_t n = atomicAdd(&reinterpret_cast<PlanEnd*>(&plan[p.K])->next[xcd], 1);
            next_q = given + (slices ? n : n * kXcds + xcd);
        }
        // the list's blocks, dealt to the workgroup's waves in runs; a long
        // list's runs are longer, so that its map is loaded once for several
        const int take = nd >= kLongList ? kTake : 1;
        int tile = -1;
        Tile t{};
        Map m;
        for (int r = wave * take; r < nd; r += kWavesPerBlock * take) {
            for (int it = r; it < min(r + take, nd); ++it) {
                const uint32_t index = __builtin_amdgcn_readfirstlane(sh.block[it].index);
                const uint32_t tp = __builtin_amdgcn_readfirstlane(sh.block[it].tile_points);
                if ((int)(tp & 0xffffu) != tile) {
                    tile = (int)(tp & 0xffffu);
                    t.link = __builtin_amdgcn_readfirstlane(sh.tile[tile].link);
                    t.c0 = __builtin_amdgcn_readfirstlane(sh.tile[tile].c0);
                    t.n = __builtin_amdgcn_readfirstlane(sh.tile[tile].n);
                    load_map(p, t.link, t.c0, t.n, lane, m);
                }
                const LinkGrid& lg = p.link[t.link];
                const int64_t j = (int64_t)index * kBlockPts;
                uint32_t any = (1u << kBlockPts) - 1;   // the points inside some lane's box
                // the block's coordinates, one per lane
                const float* const at = points + 3 * j;
                const float xl = at[(uint32_t)min(lane, j + kBlockPts <= p.M ? 3 * kBlockPts - 1 : 3 * (int)(p.M - j) - 1)];
                if (j + kBlockPts <= p.M) {
                    any = 0;
#pragma unroll
                    for (int u = 0; u < kBlockPts; ++u) {
                        float v0, v1, v2;
                        map_point(m, at[3 * u], at[3 * u + 1], at[3 * u + 2], v0, v1, v2);
                        if (__ballot(inside<CUBIC>(lg, v0, v1, v2))) any |= 1u << u;
                    }
                }
                any &= tp >> 16;
                while (any) {   // wave-uniform
                    const int u = 3 * __builtin_ctz(any);
                    any &= any - 1;
                    auto coord = [&](int k) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(xl), k)); };
                    float v0, v1, v2;
                    map_point(m, coord(u), coord(u + 1), coord(u + 2), v0, v1, v2);
                    const bool is = inside<CUBIC>(lg, v0, v1, v2);
                    const uint64_t lanes = __ballot(is);
                    if (is)
                        queue[waiting + __builtin_amdgcn_mbcnt_hi((uint32_t)(lanes >> 32),
                                                                  __builtin_amdgcn_mbcnt_lo((uint32_t)lanes, 0))] =
                            make_float4(v0, v1, v2, __int_as_float(64 * tile + lane));
                    waiting += __builtin_popcountll(lanes);
                    if (waiting >= 64) evaluate(64);
                }
            }
        }
        if (waiting > 0) evaluate(waiting);
        __syncthreads();
        for (int g = wave; g < nt; g += kWavesPerBlock) {
            const uint32_t kv = sh.best[g][lane];
            if (kv) atomicMax(&p.keys[(int64_t)(sh.tile[g].c0 + lane) * p.L + sh.tile[g].link], kv);
        }
        if (!left && (!DEAL || (dry && given >= hi))) break;
        __syncthreads();   // the list, the table and the counters are read
        if (threadIdx.x == 0) {
            sh.listed = sh.tiles = sh.open = 0;
            if (DEAL && dry) {
                sh.run_q = next_q;
                sh.run = next_q < min(given + nruns, hi) ? (int)((hi - next_q + nruns - 1) / nruns) : 0;
                sh.taken = 0;
            }
        }
        __syncthreads();
        if (DEAL && dry && sh.run == 0 && !left) break;
    }
}

// The widened box of points in [lo, hi]: its half extents grow by a relative
// 1e-5, by 1e-4 of the largest coordinate magnitude on their axis (which
// bounds FP32 rounding of the mapped coordinates many times over) and by
// 1e-6 m.  Where that is not finite the box is one that reaches everything.
__device__ __forceinline__ Box box_of(const float (&lo)[3], const float (&hi)[3]) {
    float c[3], h[3];
    bool finite = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        c[a] = 0.5f * lo[a] + 0.5f * hi[a];
        const float r = fmaxf(hi[a] - c[a], c[a] - lo[a]);
        h[a] = fmaf(r, 1.00001f, fmaf(1e-4f, fabsf(c[a]) + r, 1e-6f));
        finite &= h[a] < 1e30f;   // false for NaN
    }
    if (!finite) return Box{0.f, 0.f, 0.f, 1e30f, 1e30f, 1e30f};
    return Box{c[0], c[1], c[2], h[0], h[1], h[2]};
}

__device__ __forceinline__ PackedBox pack_box(const Box& b) {
    // the power of two from hmax / 255 up, and the half extents in units of it,
    // rounded up (hmax >= 1e-6 keeps both it and its inverse normal)
    const float hmax = fmaxf(b.hx, fmaxf(b.hy, b.hz));
    const uint32_t unit = (__float_as_uint(hmax * (1.0001f / 255.0f)) + 0x7fffffu) & 0x7f800000u;
    const float inv = __uint_as_float((254u << 23) - unit);
    const uint32_t x = (uint32_t)ceilf(b.hx * inv), y = (uint32_t)ceilf(b.hy * inv), z = (uint32_t)ceilf(b.hz * inv);
    return PackedBox{b.cx, b.cy, b.cz, unit << 1 | z << 16 | y << 8 | x};
}

// The boxes of block b (8 points from 8 b) and, for b = 8 g, of group g
// (blocks 8 g to 8 g + 7), from the thread of block b; the eight threads of a
// group are adjacent lanes and combine their boxes by shuffles.  Past the end
// of the cloud the last point repeats, which changes no box; NaN coordinates
// are left out (such a point is inside no grid's box).  Every lane of a group
// must call this together.
__device__ __forceinline__ void block_and_group_boxes(const float* __restrict__ points, int64_t b, int64_t M,
                                                      PackedBox* block_out, Box* group_out) {
    float x[kBlockPts][3];
#pragma unroll
    for (int k = 0; k < kBlockPts; ++k) {
        const int64_t j = min(b * kBlockPts + k, M - 1);
#pragma unroll
        for (int a = 0; a < 3; ++a) x[k][a] = points[3 * j + a];
    }
    float lo[3], hi[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = hi[a] = x[0][a];
#pragma unroll
        for (int k = 1; k < kBlockPts; ++k) {
            lo[a] = fminf(lo[a], x[k][a]);
            hi[a] = fmaxf(hi[a], x[k][a]);
        }
    }
    if (b * kBlockPts < M) *block_out = pack_box(box_of(lo, hi));
#pragma unroll
    for (int o = 1; o < kGroupBlocks; o <<= 1) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            lo[a] = fminf(lo[a], __shfl_xor(lo[a], o, 64));
            hi[a] = fmaxf(hi[a], __shfl_xor(hi[a], o, 64));
        }
    }
    if ((b & (kGroupBlocks - 1)) == 0) *group_out = box_of(lo, hi);
}

// The plan of the batched queries (in one workgroup of 256 threads).
__device__ __forceinline__ void build_plan(const PrepArgs& a) {
    __shared__ int64_t scan[256];
    const int t = threadIdx.x;
    int64_t carry = 0;
    for (int base = 0; base < a.K; base += 256) {
        const int k = base + t;
        TrajPlan e{};
        int64_t n = 0;
        if (k < a.K) {
            const int32_t c0 = a.c_off ? min(max(a.c_off[k], 0), a.C) : 0;
            const int32_t c1 = a.c_off ? min(max(a.c_off[k + 1], c0), a.C) : a.C;
            const int64_t m0 = a.m_off ? min(max(a.m_off[k], (int64_t)0), a.M) : 0;
            const int64_t m1 = a.m_off ? min(max(a.m_off[k + 1], m0), a.M) : a.M;
            e.m_lo = m0;
            e.m_hi = m1;
            e.c_lo = c0;
            e.c_n = c1 - c0;
            e.cgroups = (e.c_n + 63) / 64;
            // the groups (aligned in the concatenated cloud) that hold a point of [m0, m1)
            const int64_t ng = m1 > m0 ? (m1 + kGroupPts - 1) / kGroupPts - m0 / kGroupPts : 0;
            e.chunks_per_group = (int32_t)((ng + a.chunk_groups - 1) / a.chunk_groups) << a.split;
            n = (int64_t)a.L * e.cgroups * e.chunks_per_group;
        }
        scan[t] = n;
        __syncthreads();
        for (int off = 1; off < 256; off <<= 1) {   // inclusive Hillis-Steele scan
            const int64_t v = t >= off ? scan[t - off] : 0;
            __syncthreads();
            scan[t] += v;
            __syncthreads();
        }
        if (k < a.K) {
            e.chunk_start = carry + scan[t] - n;
            a.plan[k] = e;
        }
        carry += scan[255];
        __syncthreads();
    }
    if (t == 0) {
        PlanEnd e{};
        e.chunk_start = carry;
        *reinterpret_cast<PlanEnd*>(&a.plan[a.K]) = e;
    }
}

// First kernel of a query, three independent jobs on separate threads so
// that their latencies overlap.  Thread t < C L zeroes key t and writes the
// map table entry of (link t / C, configuration t mod C), from the given pose
// or, in the fused form, from the pose it computes from the joint angles.
// Thread box_base + s bounds block s of 8 consecutive points of the
// concatenated cloud by a box, and with its group's seven other lanes group
// s / 8 by another (box_base is a multiple of the wave size, so every wave
// holds whole groups).  The last
// workgroup builds the plan: each trajectory's ranges clamped into [0, C)
// and [0, M) (so a bad offset table gives wrong ranges, never an access out
// of bounds), its chunk count and the exclusive prefix sum of the counts.
__global__ __launch_bounds__(256) void prep_kernel(PrepArgs a) {
    const int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (blockIdx.x == gridDim.x - 1) {
        build_plan(a);
        return;
    }
    if (b >= a.box_base) {
        const int64_t sb = b - a.box_base;
        // uniform over the eight lanes of a group
        if (sb / kGroupBlocks * kGroupPts < a.M)
            block_and_group_boxes(a.points, sb, a.M, &a.blocks[sb], &a.groups[sb / kGroupBlocks]);
        return;
    }
    if (b < (int64_t)a.C * a.L) {
        a.keys[b] = 0u;
        // map of link i at configuration c: row a of R^T scaled by invh_a,
        // offset -invh_a (R^T t)_a + cen_a (the inverse pose of Eq. 4 with
        // the grid scaling folded in); then the culling thresholds: half_a
        // plus a bound on FP32 rounding
        const int i = (int)(b / a.C);
        const int64_t c = b - (int64_t)i * a.C;
        const LinkGrid& lg = a.link[i];
        float T[12];
        if (a.q) {
            // the pose from the joint angles, with the kinematics kernel's
            // arithmetic (same bits as lsdf_fk_batch)
            lsdf::chain_pose(a.dh, a.q + c * a.dh.dof, i, T);
            if (a.link_T_out) {
                float* o = a.link_T_out + (c * a.L + i) * 12;
#pragma unroll
                for (int k = 0; k < 12; ++k) o[k] = T[k];
            }
        } else {
            const float* src = a.link_T + (c * a.L + i) * 12;
#pragma unroll
            for (int k = 0; k < 12; ++k) T[k] = src[k];
        }
        const float r00 = T[0], r01 = T[1], r02 = T[2], t0 = T[3];
        const float r10 = T[4], r11 = T[5], r12 = T[6], t1 = T[7];
        const float r20 = T[8], r21 = T[9], r22 = T[10], t2 = T[11];
        float f[kMapFields];
        f[0] = lg.invh[0] * r00; f[1] = lg.invh[0] * r10; f[2] = lg.invh[0] * r20;
        f[3] = lg.invh[1] * r01; f[4] = lg.invh[1] * r11; f[5] = lg.invh[1] * r21;
        f[6] = lg.invh[2] * r02; f[7] = lg.invh[2] * r12; f[8] = lg.invh[2] * r22;
        f[9] = fmaf(-lg.invh[0], fmaf(r00, t0, fmaf(r10, t1, r20 * t2)), lg.cen[0]);
        f[10] = fmaf(-lg.invh[1], fmaf(r01, t0, fmaf(r11, t1, r21 * t2)), lg.cen[1]);
        f[11] = fmaf(-lg.invh[2], fmaf(r02, t0, fmaf(r12, t1, r22 * t2)), lg.cen[2]);
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) f[12 + ax] = lg.half[ax] + fmaf(1e-4f, fabsf(f[9 + ax]), 1e-3f);
        float* out = a.maps + (int64_t)i * kMapFields * a.C + c;
#pragma unroll
        for (int k = 0; k < kMapFields; ++k) out[(int64_t)k * a.C] = f[k];
    }
}

// Keys -> outputs, one lane per configuration (keys == NULL: no pair was
// evaluated, every configuration gets +inf and -1).
__global__ __launch_bounds__(kBlock) void finalize_kernel(FinalizeArgs p) {
    const int c = blockIdx.x * kBlock + threadIdx.x;
    if (c >= p.C) return;
    uint32_t k[LSDF_MAX_LINKS];
#pragma unroll
    for (int i = 0; i < LSDF_MAX_LINKS; ++i)
        if (i < p.L) k[i] = p.keys ? p.keys[(int64_t)c * p.L + i] : 0u;
    uint32_t bestk = 0;
    int arg = -1;
#pragma unroll
    for (int i = 0; i < LSDF_MAX_LINKS; ++i) {
        if (i < p.L) {
            if (p.out_link_dist) p.out_link_dist[(int64_t)c * p.L + i] = k[i] ? lsdf::from_ordered_bits(~k[i]) : INFINITY;
            if (k[i] > bestk) {   // strict: ties keep the lowest link
                bestk = k[i];
                arg = i;
            }
        }
    }
    p.out_dist[c] = bestk ? lsdf::from_ordered_bits(~bestk) : INFINITY;
    p.out_link[c] = arg;
}

// Zeroes n words (the learned query's keys before its main kernel).
__global__ __launch_bounds__(kBlock) void zero_kernel(uint32_t* w, int64_t n) {
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (t < n) w[t] = 0u;
}

}  // namespace

int lsdf::launch_query_finalize(const uint32_t* keys, float* out_dist, int32_t* out_link, float* out_link_dist, int32_t C,
                                int32_t L, hipStream_t s) {
    FinalizeArgs f{keys, out_dist, out_link, out_link_dist, C, L};
    hipLaunchKernelGGL(finalize_kernel, dim3((unsigned)((C + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, f);
    return check_launch("query finalize");
}

int lsdf::launch_zero_words(uint32_t* w, int64_t n, hipStream_t s) {
    if (n <= 0) return LSDF_OK;
    hipLaunchKernelGGL(zero_kernel, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, w, n);
    return check_launch("zero words");
}

namespace {

size_t keys_bytes(int64_t C, int64_t L) { return ((size_t)(C * L) * 4 + 255) / 256 * 256; }
// The blocks' boxes (16 bytes each), then the groups' (24), in 80 bytes per 32
// points: callers hold workspaces of that size and the scratch array's limit
// follows from it, so it stays; with q = ceil(M / 32) the boxes take at most
// 64 q + 24 ceil(q / 2) bytes, no more than that but for q = 1, whose 88 bytes
// round up to the same 256.
int64_t block_count(int64_t M) { return (M + kBlockPts - 1) / kBlockPts; }
int64_t group_count(int64_t M) { return (M + kGroupPts - 1) / kGroupPts; }
size_t box_bytes(int64_t M) { return ((size_t)((M + 31) / 32) * 80 + 255) / 256 * 256; }
size_t plan_bytes(int64_t K) { return ((size_t)(K + 1) * sizeof(TrajPlan) + 255) / 256 * 256; }
// (72 bytes per link and configuration likewise; the map table takes 60)
size_t map_bytes(int64_t C, int64_t L) { return ((size_t)(C * L) * 72 + 255) / 256 * 256; }
static_assert(kMapFields * 4 <= 72, "the map table's share of the workspace");

// Workspace: keys | block and group boxes | plan | maps, each 256-byte aligned.
size_t workspace_bytes(int64_t K, int64_t C, int64_t L, int64_t M) {
    return keys_bytes(C, L) + box_bytes(M) + plan_bytes(K) + map_bytes(C, L);
}

// Workgroups of the query kernel variant that fit on one CU at once.
template <bool CUBIC, int DT, bool DEAL>
int resident_blocks_of() {
    static std::atomic<int> cached{0};
    int v = cached.load(std::memory_order_relaxed);
    if (v > 0) return v;
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, query_kernel<CUBIC, DT, DEAL>, kBlock, 0) != hipSuccess || n < 1)
        n = kDefaultBlocksPerCu;
    n = std::min(n, kMaxBlocksPerCu);
    cached.store(n, std::memory_order_relaxed);
    return n;
}

// Calls f with the kernel's template arguments.
template <bool CUBIC, int DT, bool DEAL>
struct Variant {
    static constexpr bool cubic = CUBIC, deal = DEAL;
    static constexpr int dtype = DT;
};
template <bool CUBIC, int DT, class F>
auto with_deal(bool deal, F&& f) {
    return deal ? f(Variant<CUBIC, DT, true>{}) : f(Variant<CUBIC, DT, false>{});
}
template <class F>
auto with_variant(int dtype, bool cubic, bool deal, F&& f) {
    switch (dtype * 2 + (cubic ? 1 : 0)) {
        case LSDF_F32 * 2 + 1: return with_deal<true, LSDF_F32>(deal, f);
        case LSDF_F32 * 2: return with_deal<false, LSDF_F32>(deal, f);
        case LSDF_BF16 * 2 + 1: return with_deal<true, LSDF_BF16>(deal, f);
        case LSDF_BF16 * 2: return with_deal<false, LSDF_BF16>(deal, f);
        case LSDF_F16 * 2 + 1: return with_deal<true, LSDF_F16>(deal, f);
        default: return with_deal<false, LSDF_F16>(deal, f);
    }
}

int device_cus() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    return cus;
}

// (chunk_blocks and blocks_per_cu: 0 where the call's sizes are to choose)
int check_tuning(const char* who, const lsdf_query_tuning* t, int* chunk_blocks, int* blocks_per_cu,
                 int* schedule) {
    using lsdf::fail;
    *chunk_blocks = 0;
    *blocks_per_cu = 0;
    *schedule = kDefaultSchedule;
    if (!t) return LSDF_OK;
    if (t->chunk_points != 0) {
        if (t->chunk_points < kBlockPts || t->chunk_points > kMaxChunkPoints || t->chunk_points % kBlockPts != 0)
            return fail(LSDF_E_INVALID_ARG, "%s: chunk_points = %d is not a multiple of 8 in [8, %d]", who,
                        (int)t->chunk_points, kMaxChunkPoints);
        *chunk_blocks = t->chunk_points / kBlockPts;
    }
    if (t->blocks_per_cu != 0) {
        if (t->blocks_per_cu < 1 || t->blocks_per_cu > kMaxBlocksPerCu)
            return fail(LSDF_E_INVALID_ARG, "%s: blocks_per_cu = %d out of [1, %d]", who, (int)t->blocks_per_cu,
                        kMaxBlocksPerCu);
        *blocks_per_cu = t->blocks_per_cu;
    }
    if (t->schedule != LSDF_SCHED_DEFAULT) {
        if (t->schedule != LSDF_SCHED_XCD_SLICES && t->schedule != LSDF_SCHED_INTERLEAVED)
            return fail(LSDF_E_INVALID_ARG, "%s: unknown schedule %d", who, (int)t->schedule);
        *schedule = t->schedule;
    }
    if (t->reserved != 0) return fail(LSDF_E_INVALID_ARG, "%s: tuning.reserved must be 0", who);
    return LSDF_OK;
}

// Shared body of the plain (K = 1, no offset arrays) and batched queries.
// With dh != NULL the poses are computed from the joint angles q in the
// first kernel (and stored in link_T when it is not NULL).
int run_query(const char* who, int32_t K, const int32_t* c_off, const int64_t* m_off, const float* link_T, int32_t C,
              int32_t L, const lsdf_grid* grids, const void* grid_buf, const float* points, int64_t M, float* out_dist,
              int32_t* out_link, float* out_link_dist, const lsdf_query_tuning* tuning, uint32_t flags,
              void* workspace, size_t ws_bytes, void* stream, const lsdf::DhTable* dh = nullptr,
              const float* q = nullptr) {
    using namespace lsdf;
    if (flags != 0) return fail(LSDF_E_UNSUPPORTED, "%s: unsupported flags 0x%x", who, flags);
    if (C < 0 || M < 0 || M > LSDF_MAX_POINTS)
        return fail(LSDF_E_SHAPE, "%s: size out of range (C = %d, M = %lld)", who, (int)C, (long long)M);
    if (L < 1 || L > LSDF_MAX_LINKS) return fail(LSDF_E_SHAPE, "%s: L = %d out of [1, %d]", who, (int)L, LSDF_MAX_LINKS);
    if (K < 1 || K > LSDF_MAX_TRAJECTORIES)
        return fail(LSDF_E_SHAPE, "%s: K = %d out of [1, %d]", who, (int)K, LSDF_MAX_TRAJECTORIES);
    if (!grids) return fail(LSDF_E_INVALID_ARG, "%s: grids is NULL", who);
    int chunk_blocks = 0, blocks_per_cu = 0, schedule = 0;
    int rc = check_tuning(who, tuning, &chunk_blocks, &blocks_per_cu, &schedule);
    if (rc != LSDF_OK) return rc;
    if (C == 0) return LSDF_OK;
    if ((!dh && !link_T) || (dh && !q) || !grid_buf || !out_dist || !out_link || !workspace)
        return fail(LSDF_E_INVALID_ARG, "%s: NULL device pointer", who);
    if (dh && L != dh->dof + 1)
        return fail(LSDF_E_SHAPE, "%s: %d grids for a %d-joint arm (needs dof + 1)", who, (int)L, (int)dh->dof);
    if (M > 0 && !points) return fail(LSDF_E_INVALID_ARG, "%s: points is NULL", who);
    if ((reinterpret_cast<uintptr_t>(workspace) & 255) != 0)
        return fail(LSDF_E_INVALID_ARG, "%s: workspace is not 256-byte aligned", who);
    const size_t need = workspace_bytes(K, C, L, M);
    if (ws_bytes < need) return fail(LSDF_E_SHAPE, "%s: workspace has %zu bytes, needs %zu", who, ws_bytes, need);

    QueryArgs p{};
    bool cubic = true;
    const int dtype = grids[0].dtype;
    for (int i = 0; i < L; ++i) {
        rc = prepare_link_grid(grids[i], i, &p.link[i]);
        if (rc != LSDF_OK) return rc;
        if (grids[i].dtype != dtype) return fail(LSDF_E_UNSUPPORTED, "%s: grids of one query must share a dtype", who);
        cubic = cubic && p.link[i].cubic;
    }
    const int cus = device_cus();
    if (cus <= 0) return fail(LSDF_E_DEVICE, "%s: cannot read the device's compute-unit count", who);
    auto resident = [&](bool deal) {
        return with_variant(dtype, cubic, deal, [](auto v) {
            using V = decltype(v);
            return resident_blocks_of<V::cubic, V::dtype, V::deal>();
        });
    };
    const bool fill_device = blocks_per_cu == 0;
    if (fill_device) blocks_per_cu = resident(false);
    if (chunk_blocks == 0)   // from the capacities C and M when offsets are given
        chunk_blocks = default_chunk_blocks(K, C, L, M, (int64_t)cus * blocks_per_cu * kWavesPerBlock);
    const bool deal = (double)L * ((C + 63) / 64) * ((M + kBlockPts * chunk_blocks - 1) / (kBlockPts * chunk_blocks)) >=
                      (double)K * kDealChunks * cus * blocks_per_cu * kWavesPerBlock;
    if (fill_device && deal) blocks_per_cu = resident(true);
    hipStream_t s = as_stream(stream);
    char* ws = static_cast<char*>(workspace);
    PackedBox* block_box = reinterpret_cast<PackedBox*>(ws + keys_bytes(C, L));
    Box* group_box = reinterpret_cast<Box*>(block_box + block_count(M));
    TrajPlan* plan = reinterpret_cast<TrajPlan*>(ws + keys_bytes(C, L) + box_bytes(M));
    float* maps = reinterpret_cast<float*>(ws + keys_bytes(C, L) + box_bytes(M) + plan_bytes(K));
    p.maps = maps;
    p.keys = reinterpret_cast<uint32_t*>(ws);
    p.M = M;
    p.C = C;
    p.K = K;
    p.L = L;
    // chunks of whole groups, or of a half or quarter of one
    const int chunk_groups = (chunk_blocks + kGroupBlocks - 1) / kGroupBlocks;
    p.split = chunk_blocks >= kGroupBlocks ? 0 : chunk_blocks >= kGroupBlocks / 2 ? 1 : 2;
    p.schedule = schedule;
    // the first kernel runs when there are points to test, or when poses
    // computed from joint angles are asked for
    if (M > 0 || (dh && link_T)) {
        PrepArgs a{};
        for (int i = 0; i < L; ++i) a.link[i] = p.link[i];
        if (dh) {
            a.dh = *dh;
            a.q = q;
            a.link_T_out = const_cast<float*>(link_T);   // an output in the fused form
        }
        a.link_T = link_T;
        a.points = points;
        a.blocks = block_box;
        a.groups = group_box;
        a.plan = plan;
        a.maps = maps;
        a.keys = p.keys;
        a.c_off = c_off;
        a.m_off = m_off;
        a.M = M;
        a.C = C;
        a.K = K;
        a.L = L;
        a.chunk_groups = chunk_groups;
        a.split = p.split;
        // map threads, then (from a wave boundary) one thread per block of
        // every group, then the plan's workgroup
        a.box_base = ((int64_t)C * L + 63) / 64 * 64;
        const int64_t threads = a.box_base + kGroupBlocks * group_count(M);
        hipLaunchKernelGGL(prep_kernel, dim3((unsigned)((threads + 255) / 256 + 1)), dim3(256), 0, s, a);
        rc = check_launch(who);
        if (rc != LSDF_OK) return rc;
    }
    if (M > 0) {
        // persistent grid: blocks_per_cu workgroups per CU, a multiple of
        // the XCD count; when the chunk count is known here (one trajectory
        // given by C and M), no more waves than chunks
        int64_t blocks = (int64_t)cus * blocks_per_cu;
        if (!c_off) {
            const int64_t chunks = (int64_t)L * ((C + 63) / 64) * (((group_count(M) + chunk_groups - 1) / chunk_groups) << p.split);
            blocks = std::min<int64_t>(blocks, (chunks + kWavesPerBlock - 1) / kWavesPerBlock);
        }
        blocks = (blocks + kXcds - 1) / kXcds * kXcds;
        p.blocks_per_xcd = (int32_t)(blocks / kXcds);
        const PackedBox* bb = block_box;
        const Box* gb = group_box;
        TrajPlan* pl = plan;
        const dim3 gd((unsigned)blocks), bd(kBlock);
        hipEvent_t ev0, ev1;
        take_kernel_events(&ev0, &ev1);
        if (ev0 && hipEventRecord(ev0, s) != hipSuccess) return fail(LSDF_E_DEVICE, "%s: event record failed", who);
        with_variant(dtype, cubic, deal, [&](auto v) {
            using V = decltype(v);
            hipLaunchKernelGGL((query_kernel<V::cubic, V::dtype, V::deal>), gd, bd, 0, s, p, points,
                               static_cast<const typename GridT<V::dtype>::T*>(grid_buf), bb, gb, pl);
        });
        rc = check_launch(who);
        if (rc != LSDF_OK) return rc;
        if (ev1 && hipEventRecord(ev1, s) != hipSuccess) return fail(LSDF_E_DEVICE, "%s: event record failed", who);
    }
    // M = 0: no prep kernel ran and no key is meaningful; every
    // configuration gets +inf and -1
    return launch_query_finalize(M > 0 ? p.keys : nullptr, out_dist, out_link, out_link_dist, C, L, s);
}

}  // namespace

LSDF_API int lsdf_query_workspace_size(int32_t C, int32_t L, int64_t M, uint32_t flags, size_t* bytes) {
    lsdf::clear_error();
    if (flags != 0) return lsdf::fail(LSDF_E_UNSUPPORTED, "query_workspace_size: unsupported flags 0x%x", flags);
    return lsdf_query_batched_workspace_size(1, C, L, M, bytes);
}

LSDF_API int lsdf_query_batched_workspace_size(int32_t K, int32_t C, int32_t L, int64_t M, size_t* bytes) {
    using namespace lsdf;
    clear_error();
    if (!bytes) return fail(LSDF_E_INVALID_ARG, "query_workspace_size: bytes is NULL");
    if (C < 0 || M < 0 || M > LSDF_MAX_POINTS) return fail(LSDF_E_SHAPE, "query_workspace_size: size out of range");
    if (L < 1 || L > LSDF_MAX_LINKS) return fail(LSDF_E_SHAPE, "query_workspace_size: L = %d out of [1, %d]", (int)L, LSDF_MAX_LINKS);
    if (K < 1 || K > LSDF_MAX_TRAJECTORIES)
        return fail(LSDF_E_SHAPE, "query_workspace_size: K = %d out of [1, %d]", (int)K, LSDF_MAX_TRAJECTORIES);
    *bytes = workspace_bytes(K, C, L, M);
    return LSDF_OK;
}

LSDF_API int lsdf_query_min_distance(const float* link_T, int32_t C, int32_t L, const lsdf_grid* grids,
                                     const void* grid_buf, const float* points, int64_t M, float* out_dist,
                                     int32_t* out_link, float* out_link_dist, uint32_t flags, void* workspace,
                                     size_t ws_bytes, void* stream) {
    lsdf::clear_error();
    return run_query("query", 1, nullptr, nullptr, link_T, C, L, grids, grid_buf, points, M, out_dist, out_link,
                     out_link_dist, nullptr, flags, workspace, ws_bytes, stream);
}

namespace {

// Workspace of lsdf_query_min_distance_noalloc: one copy per GPU, loaded with
// the code object.  Host code never names the array itself (on the host it
// is only a stand-in for the symbol); it takes the device address that
// hipGetSymbolAddress gives for the current device, once per device.
constexpr size_t kNoAllocScratch = LSDF_QUERY_NOALLOC_SCRATCH;
constexpr int kMaxDevices = 64;
static __device__ __align__(256) unsigned char scratch[kNoAllocScratch];

std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

int noalloc_scratch(void** out) {
    using namespace lsdf;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return fail(LSDF_E_DEVICE, "query_noalloc: no current device");
    if (dev < 0 || dev >= kMaxDevices)
        return fail(LSDF_E_DEVICE, "query_noalloc: device %d beyond the %d the library tracks", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(LSDF_E_DEVICE, "query_noalloc: hipGetSymbolAddress of the scratch array failed (%s)",
                        hipGetErrorString(e));
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return LSDF_OK;
}

}  // namespace

LSDF_API int lsdf_query_min_distance_noalloc(const float* link_T, int32_t C, int32_t L, const lsdf_grid* grids,
                                             const void* grid_buf, const float* points, int64_t M, float* out_dist,
                                             int32_t* out_link, float* out_link_dist, uint32_t flags, void* stream) {
    using namespace lsdf;
    clear_error();
    if (flags != 0) return fail(LSDF_E_UNSUPPORTED, "query_noalloc: unsupported flags 0x%x", flags);
    if (C < 0 || M < 0 || M > LSDF_MAX_POINTS)
        return fail(LSDF_E_SHAPE, "query_noalloc: size out of range (C = %d, M = %lld)", (int)C, (long long)M);
    if (L < 1 || L > LSDF_MAX_LINKS)
        return fail(LSDF_E_SHAPE, "query_noalloc: L = %d out of [1, %d]", (int)L, LSDF_MAX_LINKS);
    if (C == 0) return LSDF_OK;
    const size_t need = workspace_bytes(1, C, L, M);
    if (need > kNoAllocScratch)
        return fail(LSDF_E_SHAPE,
                    "query_noalloc: C = %d, L = %d, M = %lld needs %zu bytes of workspace; the library holds %zu "
                    "(use lsdf_query_min_distance with a workspace of your own)",
                    (int)C, (int)L, (long long)M, need, kNoAllocScratch);
    void* ws = nullptr;
    const int rc = noalloc_scratch(&ws);
    if (rc != LSDF_OK) return rc;
    return run_query("query_noalloc", 1, nullptr, nullptr, link_T, C, L, grids, grid_buf, points, M, out_dist,
                     out_link, out_link_dist, nullptr, 0, ws, kNoAllocScratch, stream);
}

LSDF_API int lsdf_query_min_distance_batched(int32_t K, const int32_t* traj_c_offset, const int64_t* traj_m_offset,
                                             const float* link_T, int32_t C, int32_t L, const lsdf_grid* grids,
                                             const void* grid_buf, const float* points, int64_t M, float* out_dist,
                                             int32_t* out_link, float* out_link_dist,
                                             const lsdf_query_tuning* tuning, uint32_t flags, void* workspace,
                                             size_t ws_bytes, void* stream) {
    using namespace lsdf;
    clear_error();
    if (!traj_c_offset || !traj_m_offset) return fail(LSDF_E_INVALID_ARG, "query_batched: NULL offset array");
    return run_query("query_batched", K, traj_c_offset, traj_m_offset, link_T, C, L, grids, grid_buf, points, M,
                     out_dist, out_link, out_link_dist, tuning, flags, workspace, ws_bytes, stream);
}

LSDF_API int lsdf_query_from_joints(const lsdf_dh* dh, int32_t dof, const float* base_T, const float* q,
                                    int32_t K, const int32_t* traj_c_offset, const int64_t* traj_m_offset,
                                    int32_t C, const lsdf_grid* grids, const void* grid_buf, const float* points,
                                    int64_t M, float* link_T, float* out_dist, int32_t* out_link,
                                    float* out_link_dist, const lsdf_query_tuning* tuning, uint32_t flags,
                                    void* workspace, size_t ws_bytes, void* stream) {
    using namespace lsdf;
    clear_error();
    DhTable t;
    int rc = make_dh_table("query_from_joints", dh, dof, base_T, &t);
    if (rc != LSDF_OK) return rc;
    if ((traj_c_offset == nullptr) != (traj_m_offset == nullptr))
        return fail(LSDF_E_INVALID_ARG, "query_from_joints: give both offset arrays or neither");
    if (!traj_c_offset && K != 1)
        return fail(LSDF_E_SHAPE, "query_from_joints: K = %d without offset arrays (must be 1)", (int)K);
    return run_query("query_from_joints", K, traj_c_offset, traj_m_offset, link_T, C, dof + 1, grids, grid_buf,
                     points, M, out_dist, out_link, out_link_dist, tuning, flags, workspace, ws_bytes, stream, &t, q);
}

LSDF_API int lsdf_query_autotune(int32_t K, const int32_t* traj_c_offset, const int64_t* traj_m_offset,
                                 const float* link_T, int32_t C, int32_t L, const lsdf_grid* grids,
                                 const void* grid_buf, const float* points, int64_t M, float* out_dist,
                                 int32_t* out_link, const lsdf_query_tuning* candidates, int32_t n_candidates,
                                 int32_t reps, void* workspace, size_t ws_bytes, void* stream,
                                 lsdf_query_tuning* best, float* best_ms) {
    using namespace lsdf;
    clear_error();
    if (!traj_c_offset || !traj_m_offset) return fail(LSDF_E_INVALID_ARG, "query_autotune: NULL offset array");
    if (!best) return fail(LSDF_E_INVALID_ARG, "query_autotune: best is NULL");
    if (reps < 1 || reps > 1000) return fail(LSDF_E_INVALID_ARG, "query_autotune: reps = %d out of [1, 1000]", (int)reps);
    // the default tiling first (so the pick is never a tiling measured
    // slower than it), then chunk sizes over the resident grid, a smaller
    // grid, and the per-XCD slices
    static const lsdf_query_tuning kGrid[] = {
        {0, 0, LSDF_SCHED_DEFAULT, 0},        {64, 0, LSDF_SCHED_INTERLEAVED, 0},
        {128, 0, LSDF_SCHED_INTERLEAVED, 0},  {256, 0, LSDF_SCHED_INTERLEAVED, 0},
        {512, 0, LSDF_SCHED_INTERLEAVED, 0},  {1024, 0, LSDF_SCHED_INTERLEAVED, 0},
        {2048, 0, LSDF_SCHED_INTERLEAVED, 0}, {4096, 0, LSDF_SCHED_INTERLEAVED, 0},
        {256, 4, LSDF_SCHED_INTERLEAVED, 0},  {1024, 4, LSDF_SCHED_INTERLEAVED, 0},
        {256, 0, LSDF_SCHED_XCD_SLICES, 0},   {1024, 0, LSDF_SCHED_XCD_SLICES, 0},
    };
    if (!candidates) {
        candidates = kGrid;
        n_candidates = (int32_t)(sizeof(kGrid) / sizeof(kGrid[0]));
    }
    if (n_candidates < 1) return fail(LSDF_E_INVALID_ARG, "query_autotune: no candidates");
    for (int32_t c = 0; c < n_candidates; ++c) {
        int cb = 0, bpc = 0, sch = 0;
        int rc = check_tuning("query_autotune", &candidates[c], &cb, &bpc, &sch);
        if (rc != LSDF_OK) return rc;
    }
    hipStream_t s = as_stream(stream);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
        if (e0) (void)hipEventDestroy(e0);
        return fail(LSDF_E_DEVICE, "query_autotune: cannot create events");
    }
    int rc = LSDF_OK;
    float best_t = INFINITY;
    int32_t best_i = -1;
    for (int32_t c = 0; c < n_candidates && rc == LSDF_OK; ++c) {
        // one untimed call, then reps timed calls between two events
        rc = run_query("query_autotune", K, traj_c_offset, traj_m_offset, link_T, C, L, grids, grid_buf, points, M,
                       out_dist, out_link, nullptr, &candidates[c], 0, workspace, ws_bytes, stream);
        if (rc != LSDF_OK) break;
        if (hipEventRecord(e0, s) != hipSuccess) { rc = fail(LSDF_E_DEVICE, "query_autotune: event record failed"); break; }
        for (int32_t r = 0; r < reps && rc == LSDF_OK; ++r)
            rc = run_query("query_autotune", K, traj_c_offset, traj_m_offset, link_T, C, L, grids, grid_buf, points,
                           M, out_dist, out_link, nullptr, &candidates[c], 0, workspace, ws_bytes, stream);
        if (rc != LSDF_OK) break;
        float ms = 0.0f;
        if (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
            hipEventElapsedTime(&ms, e0, e1) != hipSuccess) {
            rc = fail(LSDF_E_DEVICE, "query_autotune: event timing failed");
            break;
        }
        ms /= (float)reps;
        if (ms < best_t) {
            best_t = ms;
            best_i = c;
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc != LSDF_OK) return rc;
    if (best_i < 0) return fail(LSDF_E_DEVICE, "query_autotune: no candidate could be timed");
    *best = candidates[best_i];
    if (best_ms) *best_ms = best_t;
    return LSDF_OK;
}

