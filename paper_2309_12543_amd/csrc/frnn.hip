// The paper's tiny network for the Euclidean grid transformation
// (Sec. III-B-1, Eq. 4-5): f(R) ~ R^T P, the rotated normalised centres of
// the (2m)^3 voxels of a transformed Link SDF block, from the 9 entries of
// the rotation; two fully connected layers with a ReLU between them,
// trained with an L1 loss and Adam (Sec. IV-B).
//
//   x = R row-major (9), h = ReLU(W1 x + b1) (32), out = W2 h + b2 (3 V),
//   V = (2m)^3, output o = 3 j + a, voxel j = (j_z 2m + j_y) 2m + j_x,
//   target_o = sum_b R[b][a] P_j[b],  P_j = (j + 1/2) / m - 1 per axis.
//   Parameters: W1[32][9], b1[32], W2[3V][32], b2[3V] (FP32).
//
// Training step (all FP32, deterministic: no floating-point atomics), three
// kernels, every sum in the order of the rows or rotations it runs over (a step
// from other bits, an ulp in a parameter, now and then turns a sign of the next
// step's errors):
//   step kernel    every wave takes blocks of 128 outputs, 16 at a time: their
//                  values, their errors against the exact target, dW2 and db2 and
//                  their Adam update, the wave's share of the loss and the block's
//                  of dh = sum_o g_o W2[o] (g_o = sign(error) / (B 3V)), with every
//                  product on FP32 MFMA (of few blocks the row kernel takes them, a
//                  thread per output, and an Adam kernel at the end: takes_rows);
//   slice kernel   sums the blocks' shares of dh in 64 interleaved slices;
//   finish kernel  a workgroup per hidden unit sums the slices, then dW1, db1
//                  through the ReLU and their Adam update; one more the loss.
// Max-error kernel: max |f(R) - R^T P| over rotations and outputs (the
// paper's 10^7-transformation test), one thread per output row, rotations
// in tiles of 64 whose hidden layers are computed once per workgroup.
#include <algorithm>

#include "lsdf_internal.hpp"

namespace {

constexpr int kH = LSDF_FRNN_HIDDEN;
constexpr int kRows = 128;          // output rows per workgroup of the row and max-error kernels
constexpr int kMaxB = 64;           // rotations per training step
constexpr int kTile = 64;           // rotations per tile in the max-error kernel
constexpr int kStepBlock = 256;     // threads of the step kernel's workgroups
constexpr int kStepGroups = 512;    // its workgroups at most: two a CU
constexpr int kBlockUnits = 8;      // units of 16 outputs whose share of dh is summed by itself
constexpr int kSlices = 64;         // first level of the sum of these shares

struct Layout {
    int64_t V, O;                   // voxels, outputs (3 V)
    int64_t w1, b1, w2, b2, n;      // offsets into the parameter vector, count
};

Layout layout(int32_t m) {
    Layout l{};
    l.V = (int64_t)(2 * m) * (2 * m) * (2 * m);
    l.O = 3 * l.V;
    l.w1 = 0;
    l.b1 = l.w1 + kH * 9;
    l.w2 = l.b1 + kH;
    l.b2 = l.w2 + l.O * kH;
    l.n = l.b2 + l.O;
    return l;
}

// Target of output o for rotation r (row-major 3x3).
__device__ inline float frnn_target(const float* r, int64_t o, int m) {
    const int64_t j = o / 3;
    const int a = (int)(o - 3 * j);
    const int w = 2 * m;
    const int jx = (int)(j % w), jy = (int)((j / w) % w), jz = (int)(j / ((int64_t)w * w));
    const float inv = 1.0f / (float)m;
    const float px = fmaf((float)jx + 0.5f, inv, -1.0f);
    const float py = fmaf((float)jy + 0.5f, inv, -1.0f);
    const float pz = fmaf((float)jz + 0.5f, inv, -1.0f);
    return fmaf(r[0 * 3 + a], px, fmaf(r[1 * 3 + a], py, r[2 * 3 + a] * pz));
}

struct TrainArgs {
    float* params;
    const float* R;          // [B][9]
    float* grad;             // [n]
    float* adam_m;           // [n], or NULL: the gradient only
    float* adam_v;
    float* part_dh;          // [blocks][kH][B]
    float* slice_dh;         // [kSlices][kH][B]
    float* part_loss;        // [groups], or [blocks] of the row kernel
    float* loss_out;         // [1] or NULL
    Layout lay;
    int32_t m;
    int32_t B;
    int32_t blocks;          // of 128 outputs
    int32_t groups;          // workgroups of the step kernel, or of the row kernel
    float lr, b1, b2, eps, c1, c2, r1, r2;   // c1 = 1 - b1^t, c2 = 1 - b2^t, r1 = 1 / c1, r2 = 1 / c2
};

typedef float f32x4 __attribute__((ext_vector_type(4)));
// four floats at any element: a vector load needs no alignment beyond one's
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

struct AdamState {
    float p, m, v;
};
// x / c, rounded as a division, from r = 1 / c rounded (Markstein): the quotient's
// error is exact in one multiply-add, and adding it times r rounds once (below
// 2^-102 that error underflows, and the quotient is within one unit in the last
// place).  Where that is not finite the product stands.
__device__ inline float divide(float x, float c, float r) {
    const float q = x * r, t = fmaf(fmaf(-q, c, x), r, q);
    return t == t ? t : q;
}
__device__ inline AdamState adam(const TrainArgs& a, AdamState s, float g) {
    const float m = fmaf(a.b1, s.m, (1.0f - a.b1) * g);
    const float v = fmaf(a.b2, s.v, (1.0f - a.b2) * g * g);
    return {s.p - a.lr * divide(m, a.c1, a.r1) / (sqrtf(divide(v, a.c2, a.r2)) + a.eps), m, v};
}

// Gradient g of parameter k, and its Adam update when there are moments.
__device__ inline void update(const TrainArgs& a, int64_t k, float g) {
    a.grad[k] = g;
    if (!a.adam_m) return;
    const AdamState s = adam(a, {a.params[k], a.adam_m[k], a.adam_v[k]}, g);
    a.params[k] = s.p;
    a.adam_m[k] = s.m;
    a.adam_v[k] = s.v;
}

// Pre-activation of hidden unit u at rotation r.
__device__ inline float hidden(const TrainArgs& a, int u, const float* r) {
    const float* W1 = a.params + a.lay.w1 + u * 9;
    float acc = a.params[a.lay.b1 + u];
#pragma unroll
    for (int k = 0; k < 9; ++k) acc = fmaf(W1[k], r[k], acc);
    return acc;
}

__device__ inline float masked(float e, uint32_t mask) { return __uint_as_float(__float_as_uint(e) & mask); }
__device__ inline float sign_of(float e) { return e > 0.0f ? 1.0f : (e < 0.0f ? -1.0f : 0.0f); }

// Row or column i of a product stands for output or rotation turned(i) of its
// 16, so that the four values a lane holds (rows 4 g + r) are those of 4 r + g: the
// next product takes one from each g, 4 r, 4 r + 1, .. in order.
__device__ inline int turned(int i) { return 4 * (i & 3) + (i >> 2); }

// What a wave reads of its 16 outputs (lane: c, g as below): for the products,
// a unit ahead, and for Adam, at its unit's start.
struct Unit {
    float wo[kH / 4];         // W2[o][4 s + g], o the unit's output turned(c)
    float wu[4][2];           // W2[output 4 r + g][16 ut + c]
    float bias;               // b2[o]
};
__device__ inline Unit load_unit(const TrainArgs& a, int q, int c, int g) {
    const float* W2 = a.params + a.lay.w2;
    const int64_t last = a.lay.O - 1, o = min((int64_t)16 * q + turned(c), last);
    Unit u;
#pragma unroll
    for (int s = 0; s < kH / 4; ++s) u.wo[s] = W2[o * kH + 4 * s + g];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t ok = min((int64_t)16 * q + 4 * r + g, last);
#pragma unroll
        for (int ut = 0; ut < 2; ++ut) u.wu[r][ut] = W2[ok * kH + 16 * ut + c];
    }
    u.bias = a.params[a.lay.b2 + o];
    return u;
}
struct UnitState {
    f32x4 p[2], m[2], v[2];   // W2[o][16 ut + 4 g ..] and its moments
    float bias_m, bias_v;
};
__device__ inline UnitState load_state(const TrainArgs& a, int64_t o, int g) {
    UnitState u;
    u.bias_m = a.adam_m[a.lay.b2 + o];
    u.bias_v = a.adam_v[a.lay.b2 + o];
#pragma unroll
    for (int ut = 0; ut < 2; ++ut) {
        const int64_t k = a.lay.w2 + o * kH + 16 * ut + 4 * g;
        u.p[ut] = *reinterpret_cast<const f32x4_any*>(a.params + k);
        u.m[ut] = *reinterpret_cast<const f32x4_any*>(a.adam_m + k);
        u.v[ut] = *reinterpret_cast<const f32x4_any*>(a.adam_v + k);
    }
    return u;
}

// The step kernel.  Products run on v_mfma_f32_16x16x4 (lane l, c = l mod 16,
// g = l / 16: A row c and B column c at k = 4 step + g; D column c, rows 4 g +
// r), which is one chain of fused multiply-adds per output in the order of k:
// the outputs' K = 32 runs in the units' order, so an error and its sign are
// those of a scalar loop.  The errors are wanted with the rotations along K
// (for dW2) and with the outputs along K (for dh); rather than transposed
// through LDS they are formed both ways, from the same registers: W H^T gives
// lane l the outputs 4 g + r at rotation c, H W^T the output c at rotations
// 4 g + r, each already in the next product's operand layout (its K index
// permuted on both sides so that it runs in order: turned()).
// Two waves a SIMD (256 registers) share 30 us of MFMA, about as much VALU and
// the memory traffic (parameters and moments read and written, the gradient
// written: 236 MB at 44^3 voxels, 42 us at the rate the separate Adam kernel
// reached; 16 MB of shares), which overlap in part: 98 us for a step of 64
// rotations, back to back with the slice and finish kernels 107 us.  Separate kernels for the
// hidden layer, the outputs (FP32 VALU, 107 us), two levels of sums and Adam (42
// us) took 154 us a step.  With dh summed over all of a wave's outputs, signs
// for g and reciprocals for Adam's quotients it was 88 us, but in other bits:
// in 3 of 20 second steps an error's sign differed.  At 3 and 4 waves a SIMD
// (spills) 105 to 184 us; the gradient's stores past the caches 1 to 7 us faster.
template <bool ADAM>
__global__ __launch_bounds__(kStepBlock, 2) void frnn_step_kernel(TrainArgs a) {
    constexpr int kTilesB = kMaxB / 16, kSteps = kH / 4, kStride = kH + 1;
    __shared__ float hs[kMaxB][kStride];                // hidden layer, 0 past the batch
    __shared__ __align__(16) float rt[9][kMaxB];        // rotations, transposed; place 16 bt + i holds 16 bt + turned(i)
    __shared__ float share_loss[kStepBlock / 64];
    const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int B = a.B;
    const int O = (int)a.lay.O, w = 2 * a.m;
    const int units = (O + 15) / 16;
    int blk = blockIdx.x * (kStepBlock / 64) + wave;
    Unit u = load_unit(a, min(kBlockUnits * blk, units - 1), c, g);   // on its way during the hidden layer
    for (int k = tid; k < 9 * kMaxB; k += kStepBlock) {
        const int b = k % kMaxB / 16 * 16 + turned(k % 16);
        rt[k / kMaxB][k % kMaxB] = b < B ? a.R[b * 9 + k / kMaxB] : 0.0f;
    }
    __syncthreads();
    {
        // thread t: unit t mod 32 at rotations t / 32, t / 32 + 8, ..
        const int u = tid % kH;
        const float* W1 = a.params + a.lay.w1 + u * 9;
        float w1[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) w1[k] = W1[k];
        const float b1 = a.params[a.lay.b1 + u];
        for (int b = tid / kH; b < kMaxB; b += kStepBlock / kH) {
            float acc = b1;
#pragma unroll
            for (int k = 0; k < 9; ++k) acc = fmaf(w1[k], rt[k][b / 16 * 16 + turned(b % 16)], acc);
            hs[b][u] = b < B ? fmaxf(acc, 0.0f) : 0.0f;
        }
    }
    __syncthreads();
    f32x4 dh[2][kTilesB];   // units 16 ut + 4 g + r, rotation 16 bt + turned(c)
    const float scale = 1.0f / ((float)B * (float)a.lay.O);
    const float inv = 1.0f / (float)a.m;
    float loss = 0.0f;
    const int stride = gridDim.x * (kStepBlock / 64);
    for (; blk < a.blocks; blk += stride)
    for (int q = kBlockUnits * blk; q < min(kBlockUnits * (blk + 1), units); ++q) {
        if (q == kBlockUnits * blk) {
#pragma unroll
            for (int bt = 0; bt < kTilesB; ++bt) dh[0][bt] = dh[1][bt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
        // the next unit's rows are on their way while this one's are used
        const bool last = q + 1 == min(kBlockUnits * (blk + 1), units);
        UnitState st;
        if (ADAM) st = load_state(a, min((int64_t)16 * q + turned(c), a.lay.O - 1), g);
        const Unit next = load_unit(a, min(last ? kBlockUnits * (blk + stride) : q + 1, units - 1), c, g);
        // this lane's output with the outputs along columns or rows (turned(c)),
        // and with them along K (4 r + g); past the last one that stands in, its
        // signs 0 where sums are formed
        const int of = 16 * q + turned(c), o = min(of, O - 1), j = o / 3, comp = o - 3 * j;
        const uint32_t live = of < O ? ~0u : 0u;
        const float bias = u.bias;
        const int jz = j / (w * w), jy = (j - jz * w * w) / w, jx = j - (jz * w + jy) * w;
        const float px = fmaf((float)jx + 0.5f, inv, -1.0f), py = fmaf((float)jy + 0.5f, inv, -1.0f),
                    pz = fmaf((float)jz + 0.5f, inv, -1.0f);
        f32x4 bias_k, px_k, py_k, pz_k;
        uint32_t live_k[4];
        int comp_k[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            live_k[r] = 16 * q + 4 * r + g < O ? ~0u : 0u;
            comp_k[r] = (uint32_t)(16 * q + 4 * r + g) % 3u;
            bias_k[r] = __shfl(bias, 4 * g + r, 64);
            px_k[r] = __shfl(px, 4 * g + r, 64);
            py_k[r] = __shfl(py, 4 * g + r, 64);
            pz_k[r] = __shfl(pz, 4 * g + r, 64);
        }
        f32x4 dw[3] = {};   // dW2[o][16 ut + 4 g + r]; db2[o] in every row
        // the outputs of rotations 16 bt .., rotations along columns (y) and along K (z)
        auto outputs = [&](int bt, f32x4& y, f32x4& z) {
            y = bias_k;
            z = f32x4{bias, bias, bias, bias};
#pragma unroll
            for (int s = 0; s < kSteps; ++s) {
                const float h = hs[16 * bt + turned(c)][4 * s + g];
                y = __builtin_amdgcn_mfma_f32_16x16x4f32(u.wo[s], h, y, 0, 0, 0);
                z = __builtin_amdgcn_mfma_f32_16x16x4f32(h, u.wo[s], z, 0, 0, 0);
            }
        };
        f32x4 y, z, yn, zn;
        outputs(0, y, z);
#pragma unroll
        for (int bt = 0; bt < kTilesB; ++bt) {
            if (16 * bt >= B) break;
            // the next rotations' products run under this one's errors
            if (bt + 1 < kTilesB) outputs(bt + 1, yn, zn);
            const int at = 16 * bt + c, b = 16 * bt + turned(c);
            const f32x4 r0 = *reinterpret_cast<const f32x4*>(&rt[comp][16 * bt + 4 * g]);
            const f32x4 r1 = *reinterpret_cast<const f32x4*>(&rt[3 + comp][16 * bt + 4 * g]);
            const f32x4 r2 = *reinterpret_cast<const f32x4*>(&rt[6 + comp][16 * bt + 4 * g]);
            const uint32_t in_c = b < B ? ~0u : 0u;   // masks, not conditions: no branches between the products
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                // outputs along K: dh
                const float ty = fmaf(rt[comp_k[r]][at], px_k[r], fmaf(rt[3 + comp_k[r]][at], py_k[r], rt[6 + comp_k[r]][at] * pz_k[r]));
                const float gy = sign_of(masked(y[r] - ty, live_k[r] & in_c)) * scale;
                // rotations along K: the loss, dW2 and db2
                const uint32_t in_k = 16 * bt + 4 * r + g < B ? ~0u : 0u;
                const float tz = fmaf(r0[r], px, fmaf(r1[r], py, r2[r] * pz));
                const float e = masked(z[r] - tz, in_k);
                loss += fabsf(masked(e, live));
                const float gz = sign_of(e) * scale;
                dw[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(1.0f, gz, dw[2], 0, 0, 0);
#pragma unroll
                for (int ut = 0; ut < 2; ++ut) {
                    dh[ut][bt] = __builtin_amdgcn_mfma_f32_16x16x4f32(u.wu[r][ut], gy, dh[ut][bt], 0, 0, 0);
                    dw[ut] = __builtin_amdgcn_mfma_f32_16x16x4f32(hs[16 * bt + 4 * r + g][16 * ut + c], gz, dw[ut], 0, 0, 0);
                }
            }
            y = yn;
            z = zn;
        }
        const float db = dw[2][0];
        // no branches from here to the next unit: a wait for its rows then only
        // counts the stores behind them instead of waiting for those too
        // (lanes past the block hold the last voxel's values, and the four
        // lanes of a b2 the same one: they store alike)
#pragma unroll
        for (int ut = 0; ut < 2; ++ut) {
            const int64_t k = a.lay.w2 + (int64_t)o * kH + 16 * ut + 4 * g;
            const f32x4 gr = dw[ut];
            __builtin_nontemporal_store(gr, reinterpret_cast<f32x4_any*>(a.grad + k));
            if (ADAM) {
                f32x4 p4, m4, v4;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const AdamState x = adam(a, {st.p[ut][r], st.m[ut][r], st.v[ut][r]}, gr[r]);
                    p4[r] = x.p;
                    m4[r] = x.m;
                    v4[r] = x.v;
                }
                *reinterpret_cast<f32x4_any*>(a.params + k) = p4;
                *reinterpret_cast<f32x4_any*>(a.adam_m + k) = m4;
                *reinterpret_cast<f32x4_any*>(a.adam_v + k) = v4;
            }
        }
        a.grad[a.lay.b2 + o] = db;
        if (ADAM) {
            const AdamState x = adam(a, {u.bias, st.bias_m, st.bias_v}, db);
            a.params[a.lay.b2 + o] = x.p;
            a.adam_m[a.lay.b2 + o] = x.m;
            a.adam_v[a.lay.b2 + o] = x.v;
        }
        u = next;
        if (last) {
            // the block's share of dh
#pragma unroll
            for (int ut = 0; ut < 2; ++ut)
#pragma unroll
                for (int bt = 0; bt < kTilesB; ++bt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int b = 16 * bt + turned(c);
                        if (b < B) a.part_dh[((int64_t)blk * kH + 16 * ut + 4 * g + r) * B + b] = dh[ut][bt][r];
                    }
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) loss += __shfl_xor(loss, off, 64);
    if (lane == 0) share_loss[wave] = loss;
    __syncthreads();
    if (tid == 0) {
        float s = 0.0f;
        for (int v = 0; v < kStepBlock / 64; ++v) s += share_loss[v];
        a.part_loss[blockIdx.x] = s;
    }
}

// The step of a network of few blocks (takes_rows): one thread per output row, a
// workgroup per block, on FP32 VALU; the step kernel's sums in the step kernel's
// order.  Latency bounds both.  A wave of the step kernel takes the 8 units of a
// block one after another, a chain of 29 to 61 us, longer by 8 for every 16
// rotations begun, where there are too few blocks to hide it; here two waves
// share a block and Adam follows as a kernel of its own, whose traffic grows with
// the blocks.  A training step (us, step kernel and this one):
//   outputs (blocks)         1 rotation    16            17            33            64
//     5,184 (41)             37.2  20.8    38.4  26.1                                61.7  42.0
//    24,000 (188)            38.9  24.8    40.5  30.4                                64.0  46.5
//    52,728 (412)            41.2  35.6    43.6  41.1    51.7  41.2    60.0  47.0    67.6  58.4
//    65,856 (515)            40.8  37.7    43.1  43.3    50.7  43.7    58.9  49.5    67.6  61.4
//    81,000 (633)            41.4  42.4    43.7  48.3    50.1  48.3    60.3  54.9    68.8  67.1
//    98,304 (768)            42.1  48.0    44.3  53.0    52.4  52.4    61.2  58.9    69.8  71.8
//   117,912 (922)            43.4  53.9    45.9  59.7    53.2  59.0    62.4  65.2    70.6  79.2
inline bool takes_rows(int64_t blocks, int B) { return blocks < (B <= 16 ? 576 : 704); }

__global__ __launch_bounds__(kRows) void frnn_row_kernel(TrainArgs a) {
    static_assert(kRows == (kMaxB / 4) * (kH / 4), "one 4 x 4 tile of dh per thread");
    __shared__ float hs[kMaxB][kH];
    __shared__ float rs[kMaxB][9];
    // sign of g[row][b] (g is +scale, -scale or 0), transposed: rows contiguous,
    // the pad staggers the rotations over the banks
    __shared__ __align__(16) int8_t sgT[kMaxB][kRows + 4];
    __shared__ float4 ws4[kRows][kH / 4];       // W2 rows in 16 B chunks, chunk c stored at c ^ (row mod 8)
    __shared__ float ls[kRows / 64];
    const int tid = threadIdx.x;
    const int B = a.B;
    for (int k = tid; k < B * kH; k += kRows) hs[k / kH][k % kH] = fmaxf(hidden(a, k % kH, a.R + k / kH * 9), 0.0f);
    for (int k = tid; k < B * 9; k += kRows) rs[k / 9][k % 9] = a.R[k];
    const int64_t o = (int64_t)blockIdx.x * kRows + tid;
    const bool live = o < a.lay.O;
    float wrow[kH];
    const float* W2 = a.params + a.lay.w2;
#pragma unroll
    for (int u = 0; u < kH; ++u) wrow[u] = live ? W2[o * kH + u] : 0.0f;
#pragma unroll
    for (int c = 0; c < kH / 4; ++c)
        ws4[tid][c ^ (tid & 7)] = make_float4(wrow[4 * c], wrow[4 * c + 1], wrow[4 * c + 2], wrow[4 * c + 3]);
    const float bias = live ? a.params[a.lay.b2 + o] : 0.0f;
    // this row's block voxel and component (the target is R^T P_j, component a)
    int comp = 0;
    float px = 0.0f, py = 0.0f, pz = 0.0f;
    if (live) {
        const int64_t j = o / 3;
        comp = (int)(o - 3 * j);
        const int w = 2 * a.m;
        const int jx = (int)(j % w), jy = (int)((j / w) % w), jz = (int)(j / ((int64_t)w * w));
        const float inv = 1.0f / (float)a.m;
        px = fmaf((float)jx + 0.5f, inv, -1.0f);
        py = fmaf((float)jy + 0.5f, inv, -1.0f);
        pz = fmaf((float)jz + 0.5f, inv, -1.0f);
    }
    __syncthreads();
    const float scale = 1.0f / ((float)B * (float)a.lay.O);
    float dw[kH];
#pragma unroll
    for (int u = 0; u < kH; ++u) dw[u] = 0.0f;
    float db = 0.0f, loss = 0.0f;
    for (int b = 0; b < B; ++b) {
        float y = bias;
#pragma unroll
        for (int u = 0; u < kH; ++u) y = fmaf(wrow[u], hs[b][u], y);
        float g = 0.0f;
        int8_t sg = 0;
        if (live) {
            const float* r = rs[b];
            const float t = fmaf(r[comp], px, fmaf(r[3 + comp], py, r[6 + comp] * pz));
            const float e = y - t;
            loss += fabsf(e);
            sg = e > 0.0f ? 1 : (e < 0.0f ? -1 : 0);
            g = e > 0.0f ? scale : (e < 0.0f ? -scale : 0.0f);
        }
        sgT[b][tid] = sg;
#pragma unroll
        for (int u = 0; u < kH; ++u) dw[u] = fmaf(g, hs[b][u], dw[u]);
        db += g;
    }
    if (live) {
        float* gW2 = a.grad + a.lay.w2 + o * kH;
#pragma unroll
        for (int u = 0; u < kH; ++u) gW2[u] = dw[u];
        a.grad[a.lay.b2 + o] = db;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) loss += __shfl_xor(loss, off, 64);
    if ((tid & 63) == 0) ls[tid >> 6] = loss;
    __syncthreads();
    // this workgroup's share of dh[b][u] = sum over its rows of g W2[o][u],
    // rows in order; thread t holds b = 4 (t / 8) + i, u = 4 (t mod 8) + k
    const int bt = tid >> 3, ut = tid & 7;
    float acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[i][k] = 0.0f;
    for (int r0 = 0; r0 < kRows; r0 += 4) {
        uint32_t sg4[4];   // the signs of rows r0 .. r0 + 3, one byte each
#pragma unroll
        for (int i = 0; i < 4; ++i) sg4[i] = *reinterpret_cast<const uint32_t*>(&sgT[4 * bt + i][r0]);
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const float4 wv = ws4[r0 + rr][ut ^ ((r0 + rr) & 7)];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                // g itself, rebuilt exactly from its sign
                const float gi = (float)(int8_t)(sg4[i] >> (8 * rr)) * scale;
                acc[i][0] = fmaf(gi, wv.x, acc[i][0]);
                acc[i][1] = fmaf(gi, wv.y, acc[i][1]);
                acc[i][2] = fmaf(gi, wv.z, acc[i][2]);
                acc[i][3] = fmaf(gi, wv.w, acc[i][3]);
            }
        }
    }
    float* pd = a.part_dh + (int64_t)blockIdx.x * kH * B;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int b = 4 * bt + i;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (b < B) pd[(4 * ut + k) * B + b] = acc[i][k];
    }
    if (tid == 0) a.part_loss[blockIdx.x] = ls[0] + ls[1];
}

// Adam of the output layer, after the row kernel.
__global__ __launch_bounds__(256) void frnn_adam_kernel(TrainArgs a) {
    const int64_t k = a.lay.w2 + (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k < a.lay.n) update(a, k, a.grad[k]);
}

// First level of the sum of the blocks' shares of dh: slice sl sums blocks sl,
// sl + kSlices, .. in order.
__global__ __launch_bounds__(256) void frnn_slice_kernel(TrainArgs a) {
    const int sl = blockIdx.y, n = a.B * kH, p = blockIdx.x * 256 + threadIdx.x;
    if (p >= n) return;
    float s = 0.0f;
#pragma unroll 8
    for (int k = sl; k < a.blocks; k += kSlices) s += a.part_dh[(int64_t)k * n + p];
    a.slice_dh[(int64_t)sl * n + p] = s;
}

// The finish kernel: workgroup u < kH sums dh of hidden unit u over the slices
// in order and forms dW1[u], db1[u] through the ReLU, the rotations in order;
// workgroup kH sums the loss.
__global__ __launch_bounds__(64) void frnn_finish_kernel(TrainArgs a) {
    static_assert(kMaxB == 64, "a lane per rotation");
    __shared__ float dz[kMaxB];
    __shared__ float rs[kMaxB * 9];
    const int u = blockIdx.x, b = threadIdx.x;
    if (u == kH) {
        float l = 0.0f;
        for (int k = b; k < a.groups; k += 64) l += a.part_loss[k];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off, 64);
        if (b == 0 && a.loss_out) a.loss_out[0] = l / ((float)a.B * (float)a.lay.O);
        return;
    }
    const int n = a.B * kH, bb = min(b, a.B - 1);
    for (int k = b; k < a.B * 9; k += 64) rs[k] = a.R[k];
    float s = 0.0f;
#pragma unroll
    for (int sl = 0; sl < kSlices; ++sl) s += a.slice_dh[(int64_t)sl * n + u * a.B + bb];
    dz[b] = hidden(a, u, a.R + bb * 9) > 0.0f ? s : 0.0f;
    __syncthreads();
    if (b < 10) {
        float t = 0.0f;
        for (int k = 0; k < a.B; ++k) t = b < 9 ? fmaf(dz[k], rs[k * 9 + b], t) : t + dz[k];
        update(a, b < 9 ? a.lay.w1 + u * 9 + b : a.lay.b1 + u, t);
    }
}

struct EvalArgs {
    const float* params;
    const float* R;          // [N][9]
    int64_t N;
    Layout lay;
    int32_t m;
    uint32_t* out_max;       // float bits of a non-negative maximum
};

__global__ __launch_bounds__(kRows) void frnn_max_error_kernel(EvalArgs a) {
    __shared__ float hs[kTile][kH];
    __shared__ float rs[kTile][9];
    __shared__ float red[kRows];
    const int tid = threadIdx.x;
    const int64_t o = (int64_t)blockIdx.x * kRows + tid;
    const bool live = o < a.lay.O;
    float wrow[kH];
#pragma unroll
    for (int u = 0; u < kH; ++u) wrow[u] = live ? a.params[a.lay.w2 + o * kH + u] : 0.0f;
    const float bias = live ? a.params[a.lay.b2 + o] : 0.0f;
    const float* W1 = a.params + a.lay.w1;
    float worst = 0.0f;
    for (int64_t t0 = (int64_t)blockIdx.y * kTile; t0 < a.N; t0 += (int64_t)gridDim.y * kTile) {
        const int nt = (int)min<int64_t>(kTile, a.N - t0);
        __syncthreads();
        for (int k = tid; k < nt * 9; k += kRows) rs[k / 9][k % 9] = a.R[t0 * 9 + k];
        __syncthreads();
        for (int p = tid; p < nt * kH; p += kRows) {
            const int b = p / kH, u = p - b * kH;
            float acc = a.params[a.lay.b1 + u];
#pragma unroll
            for (int k = 0; k < 9; ++k) acc = fmaf(W1[u * 9 + k], rs[b][k], acc);
            hs[b][u] = fmaxf(acc, 0.0f);
        }
        __syncthreads();
        if (live) {
            for (int b = 0; b < nt; ++b) {
                float y = bias;
#pragma unroll
                for (int u = 0; u < kH; ++u) y = fmaf(wrow[u], hs[b][u], y);
                worst = fmaxf(worst, fabsf(y - frnn_target(rs[b], o, a.m)));
            }
        }
    }
    red[tid] = worst;
    __syncthreads();
    if (tid == 0) {
        float mx = 0.0f;
        for (int r = 0; r < kRows; ++r) mx = fmaxf(mx, red[r]);
        atomicMax(a.out_max, __float_as_uint(mx));   // non-negative: bit order = value order
    }
}

__global__ void frnn_zero_kernel(uint32_t* w) { *w = 0u; }

int check_m(const char* who, int32_t m) {
    if (m < 1 || m > LSDF_FRNN_MAX_HALF)
        return lsdf::fail(LSDF_E_SHAPE, "%s: m = %d out of [1, %d]", who, (int)m, LSDF_FRNN_MAX_HALF);
    return LSDF_OK;
}

size_t align256(size_t b) { return (b + 255) / 256 * 256; }

// Blocks of 128 outputs, and workgroups of the step kernel: a wave per block,
// two workgroups a CU at most.
int64_t step_blocks(const Layout& l) { return (l.O + 16 * kBlockUnits - 1) / (16 * kBlockUnits); }
int64_t step_groups(const Layout& l) {
    const int64_t waves = kStepBlock / 64;
    return std::min<int64_t>(kStepGroups, (step_blocks(l) + waves - 1) / waves);
}

}  // namespace

LSDF_API int lsdf_frnn_nparam(int32_t m, int64_t* n) {
    using namespace lsdf;
    clear_error();
    int rc = check_m("frnn_nparam", m);
    if (rc != LSDF_OK) return rc;
    if (!n) return fail(LSDF_E_INVALID_ARG, "frnn_nparam: n is NULL");
    *n = layout(m).n;
    return LSDF_OK;
}

LSDF_API int lsdf_frnn_train_workspace_size(int32_t m, int32_t B, size_t* bytes) {
    using namespace lsdf;
    clear_error();
    int rc = check_m("frnn_train_workspace_size", m);
    if (rc != LSDF_OK) return rc;
    if (B < 1 || B > kMaxB) return fail(LSDF_E_SHAPE, "frnn_train_workspace_size: B = %d out of [1, %d]", (int)B, kMaxB);
    if (!bytes) return fail(LSDF_E_INVALID_ARG, "frnn_train_workspace_size: bytes is NULL");
    const Layout l = layout(m);
    *bytes = align256((size_t)step_blocks(l) * kH * B * 4) + align256((size_t)kSlices * kH * B * 4) +
             align256((size_t)step_blocks(l) * 4);
    return LSDF_OK;
}

LSDF_API int lsdf_frnn_train_step(float* params, float* adam_m, float* adam_v, int64_t t, float lr, float beta1,
                                  float beta2, float eps, int32_t m, const float* R, int32_t B, float* loss_out,
                                  float* grad, void* workspace, size_t ws_bytes, void* stream) {
    using namespace lsdf;
    clear_error();
    size_t need = 0;
    int rc = lsdf_frnn_train_workspace_size(m, B, &need);
    if (rc != LSDF_OK) return rc;
    if (!params || !R || !grad || !workspace) return fail(LSDF_E_INVALID_ARG, "frnn_train_step: NULL device pointer");
    if ((adam_m == nullptr) != (adam_v == nullptr))
        return fail(LSDF_E_INVALID_ARG, "frnn_train_step: give both Adam moments or neither");
    if (adam_m && t < 1) return fail(LSDF_E_INVALID_ARG, "frnn_train_step: step t must be >= 1");
    if (adam_m && !(std::isfinite(lr) && lr >= 0.0f && beta1 >= 0.0f && beta1 < 1.0f && beta2 >= 0.0f &&
                    beta2 < 1.0f && eps > 0.0f))
        return fail(LSDF_E_INVALID_ARG, "frnn_train_step: bad Adam hyper-parameters");
    if ((reinterpret_cast<uintptr_t>(workspace) & 255) != 0)
        return fail(LSDF_E_INVALID_ARG, "frnn_train_step: workspace is not 256-byte aligned");
    if (ws_bytes < need) return fail(LSDF_E_SHAPE, "frnn_train_step: workspace has %zu bytes, needs %zu", ws_bytes, need);
    TrainArgs a{};
    a.lay = layout(m);
    a.params = params;
    a.R = R;
    a.grad = grad;
    a.adam_m = adam_m;
    a.adam_v = adam_v;
    a.loss_out = loss_out;
    a.m = m;
    a.B = B;
    a.groups = (int32_t)step_groups(a.lay);
    a.blocks = (int32_t)step_blocks(a.lay);
    char* ws = static_cast<char*>(workspace);
    a.part_dh = reinterpret_cast<float*>(ws);
    ws += align256((size_t)a.blocks * kH * B * 4);
    a.slice_dh = reinterpret_cast<float*>(ws);
    ws += align256((size_t)kSlices * kH * B * 4);
    a.part_loss = reinterpret_cast<float*>(ws);
    a.lr = lr;
    a.b1 = beta1;
    a.b2 = beta2;
    a.eps = eps;
    a.c1 = (float)(1.0 - std::pow((double)beta1, (double)t));
    a.c2 = (float)(1.0 - std::pow((double)beta2, (double)t));
    a.r1 = (float)(1.0 / (double)a.c1);
    a.r2 = (float)(1.0 / (double)a.c2);
    hipStream_t s = as_stream(stream);
    static_assert(kRows == 16 * kBlockUnits, "a row workgroup's share is a block's");
    const bool rows = takes_rows(a.blocks, B);
    if (rows) {
        a.groups = a.blocks;
        hipLaunchKernelGGL(frnn_row_kernel, dim3((unsigned)a.blocks), dim3(kRows), 0, s, a);
    } else if (adam_m) {
        hipLaunchKernelGGL(frnn_step_kernel<true>, dim3((unsigned)a.groups), dim3(kStepBlock), 0, s, a);
    } else {
        hipLaunchKernelGGL(frnn_step_kernel<false>, dim3((unsigned)a.groups), dim3(kStepBlock), 0, s, a);
    }
    if ((rc = check_launch("frnn_train_step (step)")) != LSDF_OK) return rc;
    hipLaunchKernelGGL(frnn_slice_kernel, dim3((unsigned)((B * kH + 255) / 256), kSlices), dim3(256), 0, s, a);
    if ((rc = check_launch("frnn_train_step (slices)")) != LSDF_OK) return rc;
    hipLaunchKernelGGL(frnn_finish_kernel, dim3(kH + 1), dim3(64), 0, s, a);
    if ((rc = check_launch("frnn_train_step (finish)")) != LSDF_OK || !rows || !adam_m) return rc;
    hipLaunchKernelGGL(frnn_adam_kernel, dim3((unsigned)((a.lay.n - a.lay.w2 + 255) / 256)), dim3(256), 0, s, a);
    return check_launch("frnn_train_step (adam)");
}

LSDF_API int lsdf_frnn_max_error(const float* params, int32_t m, const float* R, int64_t N, float* out_max,
                                 void* stream) {
    using namespace lsdf;
    clear_error();
    int rc = check_m("frnn_max_error", m);
    if (rc != LSDF_OK) return rc;
    if (N < 0) return fail(LSDF_E_SHAPE, "frnn_max_error: N < 0");
    if (!params || !out_max || (N > 0 && !R)) return fail(LSDF_E_INVALID_ARG, "frnn_max_error: NULL device pointer");
    EvalArgs a{};
    a.params = params;
    a.R = R;
    a.N = N;
    a.lay = layout(m);
    a.m = m;
    a.out_max = reinterpret_cast<uint32_t*>(out_max);
    hipStream_t s = as_stream(stream);
    hipLaunchKernelGGL(frnn_zero_kernel, dim3(1), dim3(1), 0, s, a.out_max);
    if ((rc = check_launch("frnn_max_error (zero)")) != LSDF_OK) return rc;
    if (N == 0) return LSDF_OK;
    // rows across x, rotation tiles dealt over y: about 8192 workgroups
    const int64_t xb = (a.lay.O + kRows - 1) / kRows;
    const int64_t tiles = (N + kTile - 1) / kTile;
    const int64_t yb = std::max<int64_t>(1, std::min<int64_t>({tiles, 8192 / xb, 65535}));
    hipLaunchKernelGGL(frnn_max_error_kernel, dim3((unsigned)xb, (unsigned)yb), dim3(kRows), 0, s, a);
    return check_launch("frnn_max_error");
}
