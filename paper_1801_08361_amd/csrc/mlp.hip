// Learned proposal on the GPU: a 24-64-64-1 MLP (ReLU, ReLU, sigmoid) that
// predicts, per pixel, the probability that its hypothesis pick (a mode drawn
// among the colour-consistent modes of its leaves) lies within 5 cm of its
// true world point. Its output becomes integer pick weights for
// the three pixel picks of every hypothesis try; uniform preemptive scoring
// stays the judge.
//
// Matrix products run on the gfx950 matrix cores (v_mfma_f32_16x16x32_bf16:
// bfloat16 operands, FP32 accumulation). In training a workgroup owns a tile
// of 64 rows: forward (two MFMA layers and an FP32 output dot), loss, and
// backward (weight gradients and the hidden-layer input gradient are MFMA as
// well); the per-tile gradient partials are summed in a fixed order by the
// Adam step, which updates the FP32 master weights and their bfloat16 copies.
//
// Also here: the per-pixel inputs and the inlier labeller that trains the MLP
// from poses accepted by the depth-difference check of Sec. 3.3.1, Eqs. 3-4
// (verify.hip).
#include <math.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <vector>

#include "mlp_dev.h"

namespace rl {

int update_modes(Forest *f, hipStream_t s);
int frame_from(const Forest *f, const uint16_t *depth, const uint8_t *rgb, const reloc_intrinsics *K, Frame &fr);

}  // namespace rl

struct reloc_mlp {
    float *w = nullptr;          // [NP] FP32 master weights
    float *m = nullptr, *v = nullptr;
    float *grad = nullptr;       // [NP + 1]: gradient, then the loss
    float *partial = nullptr;    // [cap_tiles][NP + 1]
    int cap_tiles = 0;
    uint16_t *q = nullptr;       // [NQ] bfloat16 copies
    float *loss = nullptr;       // [cap_loss] loss sums of the epochs' last minibatches
    int cap_loss = 0;
    int step = 0;
};

namespace rl {

// one 16x32 by 32x16 product of host-given tiles, with the operand loads and the
// result's places of the training and inference kernels (checks the lane layout)
__global__ void __launch_bounds__(64) k_mfma_probe(const uint16_t *__restrict__ A, const uint16_t *__restrict__ Bt,
                                                   float *__restrict__ C)
{
    floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tile_operand(A, 32), tile_operand(Bt, 32), acc, 0, 0, 0);
    const int l = __lane_id();
    for (int i = 0; i < 4; ++i) C[(4 * (l >> 4) + i) * 16 + (l & 15)] = acc[i];
}

// ---------------------------------------------------------------------------
// initialisation and bfloat16 copies
// ---------------------------------------------------------------------------

// Glorot-uniform weights from Philox (key (seed, 5), counter (k, 0, 0, 0)),
// zero biases
__global__ void k_mlp_init(float *__restrict__ w, uint64_t seed)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= NP) return;
    int fi = 0, fo = 0;
    if (k < OB1) { fi = 24; fo = 64; }
    else if (k >= OW2 && k < OB2) { fi = 64; fo = 64; }
    else if (k >= OW3 && k < OB3) { fi = 64; fo = 1; }
    if (!fi) {
        w[k] = 0.0f;
        return;
    }
    const float a = sqrtf(6.0f / (float)(fi + fo));
    const U4 u = philox((uint64_t)k, 0, 0, 0, seed, TAG_MLP_INIT);
    const float r = (float)(u.x[0] >> 40) / 16777216.0f;
    w[k] = (2.0f * r - 1.0f) * a;
}

__global__ void k_mlp_pack(const float *__restrict__ w, uint16_t *__restrict__ q)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < 64 * 32) {
        const int j = k / 32, i = k % 32;
        q[QW1 + k] = i < 24 ? f2bf(w[OW1 + j * 24 + i]) : (uint16_t)0;
    }
    if (k < 64 * 64) {
        const int j = k / 64, i = k % 64;
        const uint16_t h = f2bf(w[OW2 + k]);
        q[QW2 + k] = h;
        q[QW2T + i * 64 + j] = h;
    }
    if (k < 64) q[QW3 + k] = f2bf(w[OW3 + k]);
}

// ---------------------------------------------------------------------------
// training: one 64-row tile per workgroup
// ---------------------------------------------------------------------------

constexpr int TS = 72;   // row stride of a tile's arrays: 16-byte rows, off the banks' period

struct __align__(16) TrainTile {
    uint16_t XT[32 * TS];                  // [input][row]
    uint16_t H1[ROWS * TS], H1T[64 * TS];  // [row][unit], [unit][row]
    uint16_t H2[ROWS * TS];
    uint16_t D2[ROWS * TS], D2T[64 * TS];  // loss gradient of layer 2's sums
    uint16_t D1T[64 * TS];                 // and of layer 1's
    float dz[5][ROWS];
};

// column sums of a 4-row-per-lane tile value over the 4 row groups of a wave
__device__ __forceinline__ float col_sum(float s)
{
    s += __shfl_xor(s, 16, 64);
    s += __shfl_xor(s, 32, 64);
    return s;
}

// four values rounded to bfloat16, as two pairs
__device__ __forceinline__ uint2 round4(const float v[4])
{
    return make_uint2(bf16_pair(v[0], v[1]), bf16_pair(v[2], v[3]));
}

__device__ __forceinline__ uint16_t half_of(const uint2 &p, int i)
{
    return (uint16_t)((i & 2 ? p.y : p.x) >> (16 * (i & 1)));
}

// where a minibatch's rows come from: all rows in order (n_rows = 0), or drawn
// uniformly with replacement by Philox (key (seed, 6), counter (epoch, step,
// j, 0))
struct RowDraw {
    uint64_t seed;
    int32_t n_rows, epoch, step;
};

// Gradient partial (NP values) and loss sum (entry NP) of one tile's rows:
// forward, loss and backward. Wavefronts 0-3 have 16 units each of every layer
// and hold the weights they multiply by in registers from the start (loaded
// one by one inside the layers they were most of a launch's 34 us on a single
// wavefront per tile; 64 tiles take 8.5 us this way, the chain of draws,
// gathers and three exchanges); wavefront 4 stages the transposed inputs and
// computes the output layer's gradient and the loss meanwhile. All wavefronts
// compute the logits (lane = row), so that only the layers' activations and
// layer 2's gradient pass between them. Every sum has the order of the
// single-wavefront form: a product's k in two steps of 32, the logit over the
// units, dw3 and db3 over the rows, biases over (16-row group, row) and then
// the four row groups. The target of label q is q / 255 and
// dz = (sigmoid(z) - q / 255) * inv_n.
__global__ void __launch_bounds__(320) k_mlp_fwd_bwd(const uint16_t *__restrict__ X, const uint8_t *__restrict__ Y,
                                                     RowDraw draw, int n, float inv_n, const uint16_t *__restrict__ q,
                                                     const float *__restrict__ w, float *__restrict__ partial)
{
    __shared__ TrainTile S;
    const int tile = blockIdx.x, wave = threadIdx.x >> 6, l = __lane_id();
    const int col = l & 15, r0 = (l >> 4) * 4, kb = (l >> 4) * 8, c = 16 * (wave & 3) + col;
    float *out = partial + (int64_t)tile * (NP + 1);
    // lane's row of the tile, -1 past the minibatch's end
    int32_t src = tile * ROWS + l < n ? tile * ROWS + l : -1;
    if (draw.n_rows && src >= 0) {
        const U4 u = philox((uint64_t)draw.epoch, (uint64_t)draw.step, (uint64_t)src, 0, draw.seed, TAG_MLP_BATCH);
        src = (int32_t)uniform_int(u.x[0], (uint64_t)draw.n_rows);
    }
    const uint8_t label = src >= 0 ? Y[src] : (uint8_t)0;
    const bf16x8 zero8 = __builtin_bit_cast(bf16x8, make_uint4(0u, 0u, 0u, 0u));
    bf16x8 xa[4], w1b, w2b[2], w2tb[2];
    float b1c = 0.0f, b2c = 0.0f, w3c = 0.0f;
    if (wave < 4) {
#pragma unroll
        for (int ti = 0; ti < 4; ++ti) {
            const int32_t row = __shfl(src, 16 * ti + col, 64);
            xa[ti] = row >= 0 ? load8(X + (int64_t)row * 32 + kb) : zero8;
        }
        w1b = tile_operand(q + QW1 + 16 * wave * 32, 32);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            w2b[k] = tile_operand(q + QW2 + 16 * wave * 64 + 32 * k, 64);
            w2tb[k] = tile_operand(q + QW2T + 16 * wave * 64 + 32 * k, 64);
        }
        b1c = w[OB1 + c];
        b2c = w[OB2 + c];
        w3c = bf2f(q[QW3 + c]);
    } else {
        uint4 x[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            x[k] = src >= 0 ? *(const uint4 *)(X + (int64_t)src * 32 + 8 * k) : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t v[4] = {x[k].x, x[k].y, x[k].z, x[k].w};
#pragma unroll
            for (int e = 0; e < 8; ++e) S.XT[(8 * k + e) * TS + l] = (uint16_t)(v[e >> 1] >> (16 * (e & 1)));
        }
    }
    const float b3 = w[OB3];
    uint32_t on1 = 0u, on2 = 0u;   // the lane's 16 activations above 0, bit 4 ti + i
    if (wave < 4) {
        // layer 1: H1 = relu(X W1^T + b1)
#pragma unroll
        for (int ti = 0; ti < 4; ++ti) {
            floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[ti], w1b, acc, 0, 0, 0);
            float hv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                hv[i] = acc[i] + b1c;
                hv[i] = hv[i] > 0.0f ? hv[i] : 0.0f;
            }
            const uint2 h = round4(hv);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                on1 |= half_of(h, i) ? 1u << (4 * ti + i) : 0u;
                S.H1[(16 * ti + r0 + i) * TS + c] = half_of(h, i);
            }
            *(uint2 *)(S.H1T + c * TS + 16 * ti + r0) = h;
        }
    }
    __syncthreads();
    if (wave < 4) {
        // layer 2: H2 = relu(H1 W2^T + b2)
#pragma unroll
        for (int ti = 0; ti < 4; ++ti) {
            floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int k = 0; k < 2; ++k)
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tile_operand(S.H1 + 16 * ti * TS + 32 * k, TS), w2b[k], acc,
                                                              0, 0, 0);
            float hv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                hv[i] = acc[i] + b2c;
                hv[i] = hv[i] > 0.0f ? hv[i] : 0.0f;
            }
            const uint2 h = round4(hv);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                on2 |= half_of(h, i) ? 1u << (4 * ti + i) : 0u;
                S.H2[(16 * ti + r0 + i) * TS + c] = half_of(h, i);
            }
        }
    }
    __syncthreads();
    // output: z = w3 . h2 + b3 (FP32, lane = row), loss and its gradient
    float z = 0.0f;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint4 h = *(const uint4 *)(S.H2 + l * TS + 8 * k), v = *(const uint4 *)(q + QW3 + 8 * k);
        const uint32_t hw[4] = {h.x, h.y, h.z, h.w}, vw[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            z = fmaf(__uint_as_float(vw[e] << 16), __uint_as_float(hw[e] << 16), z);
            z = fmaf(__uint_as_float(vw[e] & 0xFFFF0000u), __uint_as_float(hw[e] & 0xFFFF0000u), z);
        }
    }
    z = z + b3;
    const bool valid = tile * ROWS + l < n;
    const float y = (float)label / 255.0f;
    S.dz[wave][l] = valid ? (1.0f / (1.0f + expf(-z)) - y) * inv_n : 0.0f;
    wave_lds_sync();
    const float *dz = S.dz[wave];
    if (wave == 4) {
        float loss = valid ? fmaxf(z, 0.0f) - z * y + log1pf(expf(-fabsf(z))) : 0.0f;
        for (int o = 32; o >= 1; o >>= 1) loss += __shfl_xor(loss, o, 64);
        if (l == 0) out[NP] = loss;
        // dw3[j] = sum_rows dz h2 (lane = j), db3 = sum dz
        float g = 0.0f, b = 0.0f;
#pragma unroll 16
        for (int row = 0; row < ROWS; ++row) {
            g = fmaf(dz[row], bf2f(S.H2[row * TS + l]), g);
            b += dz[row];
        }
        out[OW3 + l] = g;
        if (l == 0) out[OB3] = b;
    } else {
        // dH2 = dz w3 [h2 > 0]; db2 = column sums
        float bs = 0.0f;
#pragma unroll
        for (int ti = 0; ti < 4; ++ti) {
            const float4 dr = *(const float4 *)(dz + 16 * ti + r0);
            const float drow[4] = {dr.x, dr.y, dr.z, dr.w};
            float d[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                d[i] = (on2 >> (4 * ti + i)) & 1u ? drow[i] * w3c : 0.0f;
                bs += d[i];
            }
            const uint2 h = round4(d);
#pragma unroll
            for (int i = 0; i < 4; ++i) S.D2[(16 * ti + r0 + i) * TS + c] = half_of(h, i);
            *(uint2 *)(S.D2T + c * TS + 16 * ti + r0) = h;
        }
        bs = col_sum(bs);
        if (l < 16) out[OB2 + c] = bs;
        wave_lds_sync();
        // dW2 = dH2^T H1: this wavefront's units (its own rows of D2T) by all of layer 1's
        bf16x8 a[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) a[k] = tile_operand(S.D2T + 16 * wave * TS + 32 * k, TS);
#pragma unroll
        for (int tj = 0; tj < 4; ++tj) {
            floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int k = 0; k < 2; ++k)
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[k], tile_operand(S.H1T + 16 * tj * TS + 32 * k, TS), acc, 0,
                                                              0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) out[OW2 + (16 * wave + r0 + i) * 64 + 16 * tj + col] = acc[i];
        }
    }
    __syncthreads();
    if (wave == 4) return;
    // dH1 = dH2 W2 [h1 > 0]; db1 = column sums
    float bs = 0.0f;
#pragma unroll
    for (int ti = 0; ti < 4; ++ti) {
        floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < 2; ++k)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tile_operand(S.D2 + 16 * ti * TS + 32 * k, TS), w2tb[k], acc, 0, 0,
                                                          0);
        float d[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            d[i] = (on1 >> (4 * ti + i)) & 1u ? acc[i] : 0.0f;
            bs += d[i];
        }
        *(uint2 *)(S.D1T + c * TS + 16 * ti + r0) = round4(d);
    }
    bs = col_sum(bs);
    if (l < 16) out[OB1 + c] = bs;
    wave_lds_sync();
    // dW1 = dH1^T X (input columns 24..31 are padding)
    bf16x8 a[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) a[k] = tile_operand(S.D1T + 16 * wave * TS + 32 * k, TS);
#pragma unroll
    for (int tj = 0; tj < 2; ++tj) {
        floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < 2; ++k)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[k], tile_operand(S.XT + 16 * tj * TS + 32 * k, TS), acc, 0, 0, 0);
        const int x = 16 * tj + col;
        if (x < 24)
#pragma unroll
            for (int i = 0; i < 4; ++i) out[OW1 + (16 * wave + r0 + i) * 24 + x] = acc[i];
    }
}

// sum over the tiles of one gradient entry, in tile order (the additions wait
// for one another, so a batch's loads are issued ahead of them)
__device__ __forceinline__ float tile_sum(const float *__restrict__ partial, int tiles, int k)
{
    constexpr int B = 32;
    float s = 0.0f;
    for (int t0 = 0; t0 < tiles; t0 += B) {
        float v[B];
#pragma unroll
        for (int t = 0; t < B; ++t) v[t] = partial[(int64_t)min(t0 + t, tiles - 1) * (NP + 1) + k];
#pragma unroll
        for (int t = 0; t < B; ++t)
            if (t0 + t < tiles) s += v[t];
    }
    return s;
}

__global__ void __launch_bounds__(64) k_mlp_reduce(const float *__restrict__ partial, int tiles, float *__restrict__ grad)
{
    const int k = blockIdx.x * 64 + threadIdx.x;
    if (k <= NP) grad[k] = tile_sum(partial, tiles, k);
}

// One Adam step from the tiles' partials: the entry's sum, its moments, the
// FP32 weight and its bfloat16 copies; the thread past the parameters writes
// the minibatch's loss sum to *loss where one is wanted. (Sum, Adam and copies
// as three kernels took 16.0 + 4.7 + 4.6 us a step of 64 tiles; this takes 3.8.)
__global__ void __launch_bounds__(64) k_mlp_update(const float *__restrict__ partial, int tiles, float *__restrict__ w,
                                                   float *__restrict__ m, float *__restrict__ v, uint16_t *__restrict__ q,
                                                   float lr, float c1, float c2, float *__restrict__ loss)
{
    const int k = blockIdx.x * 64 + threadIdx.x;
    if (k > NP) return;
    if (k == NP) {
        if (loss) *loss = tile_sum(partial, tiles, k);
        return;
    }
    const float m0 = m[k], v0 = v[k], w0 = w[k];
    const float g = tile_sum(partial, tiles, k);
    const float mk = 0.9f * m0 + 0.1f * g;
    const float vk = 0.999f * v0 + 0.001f * g * g;
    m[k] = mk;
    v[k] = vk;
    const float wk = w0 - lr * (mk / c1) / (sqrtf(vk / c2) + 1e-8f);
    w[k] = wk;
    const uint16_t h = f2bf(wk);
    if (k < OB1) {
        q[QW1 + (k / 24) * 32 + k % 24] = h;
    } else if (k >= OW2 && k < OB2) {
        const int e = k - OW2;
        q[QW2 + e] = h;
        q[QW2T + (e & 63) * 64 + (e >> 6)] = h;
    } else if (k >= OW3 && k < OB3) {
        q[QW3 + k - OW3] = h;
    }
}

__global__ void __launch_bounds__(64) k_mlp_logits(const uint16_t *__restrict__ X, int n,
                                                   const uint16_t *__restrict__ q, const float *__restrict__ w,
                                                   float *__restrict__ z)
{
    __shared__ InTile S;
    const int r0 = blockIdx.x * ROWS, l = __lane_id();
    uint4 *d = (uint4 *)(S.X + l * 32);
    if (r0 + l < n) {
        const uint4 *src = (const uint4 *)(X + (int64_t)(r0 + l) * 32);
        for (int k = 0; k < 4; ++k) d[k] = src[k];
    } else {
        for (int k = 0; k < 4; ++k) d[k] = make_uint4(0, 0, 0, 0);
    }
    stage_head(S, q, w);
    __syncthreads();
    const float zl = tile_forward_regs(S, q, w);
    if (r0 + l < n) z[r0 + l] = zl;
}

// ---------------------------------------------------------------------------
// per-pixel inputs, labels, verification
// ---------------------------------------------------------------------------

constexpr int PIX_THREADS = 128;
constexpr int MAX_TREES = 16;   // (checked when a forest is created)

// Bound by the chains and gathers of its walks (traverse_trees): 320 x 240,
// depth 10, half of the pixels 51 to 31 us, 640 x 480, depth 15 116 to 78
// against walking tree after tree.
// VEC: X and XF are 16-byte aligned (as torch's tensors are); their rows of 64
// and 96 bytes then go out in 16-byte stores, 10 where single values take 56
template <bool VEC>
__global__ void __launch_bounds__(PIX_THREADS) k_pixel_features(FeatArgs A, const int32_t *__restrict__ pix, int n,
                                                                uint16_t *__restrict__ X, float *__restrict__ XF)
{
    __shared__ int32_t leaf[MAX_TREES][PIX_THREADS];
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int p = pix[i];
    float x[24];
    if (p >= 0 && p < A.fr.W * A.fr.H) pixel_features(A, p, &leaf[0][threadIdx.x], PIX_THREADS, x);
    else
        for (int k = 0; k < 24; ++k) x[k] = 0.0f;
    if constexpr (VEC) {
        uint4 *in = (uint4 *)(X + (int64_t)i * 32);
        auto pair = [&](int k) { return (uint32_t)f2bf(x[k]) | ((uint32_t)f2bf(x[k + 1]) << 16); };
#pragma unroll
        for (int k = 0; k < 24; k += 8) in[k / 8] = make_uint4(pair(k), pair(k + 2), pair(k + 4), pair(k + 6));
        in[3] = make_uint4(0u, 0u, 0u, 0u);
        if (XF) {
            float4 *row = (float4 *)(XF + (int64_t)i * 24);
#pragma unroll
            for (int k = 0; k < 6; ++k) row[k] = make_float4(x[4 * k], x[4 * k + 1], x[4 * k + 2], x[4 * k + 3]);
        }
    } else {
        for (int k = 0; k < 32; ++k) X[(int64_t)i * 32 + k] = k < 24 ? f2bf(x[k]) : (uint16_t)0;
        if (XF)
            for (int k = 0; k < 24; ++k) XF[(int64_t)i * 24 + k] = x[k];
    }
}

struct PoseF {
    float R[9], t[3];
};

// The probability that the pixel's hypothesis pick is correct under the
// pose: among the modes of the pixel's leaves whose colour passes the pick's
// colour test (|mode - pixel| <= rgb_tol in every channel), the fraction that
// lie within 5 cm of y = R c + t (FP32, the scoring transform), as
// round(255 good / candidates) (0 without candidates). The walks advance
// together and a leaf's modes are loaded four at a time: 320 x 240, depth 10,
// half of the pixels 57 to 32 us, 640 x 480, depth 15 121 to 97.
__global__ void __launch_bounds__(PIX_THREADS) k_label(FeatArgs A, PoseF P, int rgb_tol, const int32_t *__restrict__ pix, int n,
                        uint8_t *__restrict__ lab)
{
    __shared__ int32_t leaves[MAX_TREES][PIX_THREADS];
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int p = pix[i];
    uint32_t cand = 0, good = 0;
    if (p >= 0 && p < A.fr.W * A.fr.H) {
        const uint32_t d = A.fr.depth[p];
        if (valid_depth(A.fr, d)) {
            const int u = p % A.fr.W, v = p / A.fr.W;
            float c[3];
            cam_point(A.fr, u, v, d, c);
            float y[3];
            for (int k = 0; k < 3; ++k)
                y[k] = fmaf(P.R[k * 3 + 0], c[0], fmaf(P.R[k * 3 + 1], c[1], fmaf(P.R[k * 3 + 2], c[2], P.t[k])));
            const int pr = A.fr.rgb[(int64_t)p * 3], pg = A.fr.rgb[(int64_t)p * 3 + 1], pb = A.fr.rgb[(int64_t)p * 3 + 2];
            const float lim = 0.05f * 0.05f;
            int32_t *leaf = &leaves[0][threadIdx.x];
            traverse_trees(A.nodes, A.T, A.L, A.fr, u, v, (int32_t)d, pixel_den(A.fr, (int32_t)d), leaf, PIX_THREADS);
            for (int t = 0; t < A.T; ++t) {
                const int64_t li = (int64_t)t * A.L + leaf[t * PIX_THREADS];
                const int nm = A.nmodes[li];
                // four modes' loads at a time; past the leaf's last they read it again
                for (int m0 = 0; m0 < nm; m0 += 4) {
                    float mu[4][3];
                    uint32_t rgb[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const Mode &md = A.modes[li * A.M + min(m0 + e, nm - 1)];
                        for (int k = 0; k < 3; ++k) mu[e][k] = md.mu[k];
                        rgb[e] = md.rgb;
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int mr = (int)(rgb[e] & 255u), mg = (int)((rgb[e] >> 8) & 255u), mb = (int)((rgb[e] >> 16) & 255u);
                        const float d0 = y[0] - mu[e][0], d1 = y[1] - mu[e][1], d2 = y[2] - mu[e][2];
                        const bool is = m0 + e < nm && abs(mr - pr) <= rgb_tol && abs(mg - pg) <= rgb_tol && abs(mb - pb) <= rgb_tol;
                        cand += is ? 1u : 0u;
                        good += is && (d0 * d0 + d1 * d1) + d2 * d2 <= lim ? 1u : 0u;
                    }
                }
            }
        }
    }
    lab[i] = cand ? (uint8_t)((255u * good + cand / 2u) / cand) : (uint8_t)0;
}

// every pixel of a frame: inputs, forward, pick weight floor(sigma 65536) + 1
// for valid pixels, 0 otherwise
__global__ void __launch_bounds__(64) k_mlp_pixels(FeatArgs A, const uint16_t *__restrict__ q,
                                                   const float *__restrict__ w, uint32_t *__restrict__ weights,
                                                   float *__restrict__ prob)
{
    __shared__ InTile S;
    __shared__ int32_t leaf[MAX_TREES][ROWS];
    const int P = A.fr.W * A.fr.H;
    const int l = __lane_id();
    const int p = blockIdx.x * ROWS + l;
    float x[24];
    if (p < P) pixel_features(A, p, &leaf[0][l], ROWS, x);
    else
        for (int k = 0; k < 24; ++k) x[k] = 0.0f;
    store_row(S.X, x);
    stage_head(S, q, w);
    __syncthreads();
    const float zl = tile_forward_regs(S, q, w);
    if (p < P) {
        const bool ok = valid_depth(A.fr, A.fr.depth[p]);
        float sg = 0.0f;
        const uint32_t wt = pick_weight(zl, &sg);
        weights[p] = ok ? wt : 0u;
        if (prob) prob[p] = ok ? sg : 0.0f;
    }
}

static FeatArgs feat_args(const Forest *f, const Frame &fr)
{
    FeatArgs A;
    A.fr = fr;
    A.nodes = f->nodes;
    A.nmodes = f->nmodes;
    A.modes = f->modes;
    A.leaf_in = f->leaf_in;
    A.packed = nullptr;
    A.xnodes = nullptr;
    A.T = f->T; A.L = f->L; A.M = f->M; A.R = f->R;
    return A;
}

static int ensure_tiles(reloc_mlp *m, int tiles)
{
    if (tiles <= m->cap_tiles) return RELOC_OK;
    if (m->partial) (void)hipFree(m->partial);
    m->partial = nullptr;
    m->cap_tiles = 0;
    RL_HIP(device_malloc((void **)&m->partial, (size_t)tiles * (NP + 1) * sizeof(float)));
    m->cap_tiles = tiles;
    return RELOC_OK;
}

static int ensure_loss(reloc_mlp *m, int n)
{
    if (n <= m->cap_loss) return RELOC_OK;
    if (m->loss) (void)hipFree(m->loss);
    m->loss = nullptr;
    m->cap_loss = 0;
    RL_HIP(device_malloc((void **)&m->loss, (size_t)n * sizeof(float)));
    m->cap_loss = n;
    return RELOC_OK;
}

// the tiles' gradient partials of the mean loss over n rows into m->partial
static int mlp_partials(reloc_mlp *m, const uint16_t *X, const uint8_t *Y, const RowDraw &draw, int n, int *tiles,
                        hipStream_t s)
{
    *tiles = (n + ROWS - 1) / ROWS;
    int rc = ensure_tiles(m, *tiles);
    if (rc) return rc;
    RL_LAUNCH("k_mlp_fwd_bwd", k_mlp_fwd_bwd, dim3(*tiles), dim3(320), 0, s, X, Y, draw, n, 1.0f / (float)n, m->q, m->w,
              m->partial);
    return RELOC_OK;
}

// Valid pixels of a frame (the depth test of the features and of the
// relocaliser's pool) as indices v W + u in raster order: per block of
// VP_BLOCK pixels a count, one workgroup's exclusive scan of the counts, then
// each block's indices at its offset. Each of VP_THREADS threads takes
// pixels t + j VP_THREADS of its block, so its wavefront's 64-pixel chunks
// c = j (VP_THREADS / 64) + wave run in raster order.
constexpr int VP_BLOCK = 1024, VP_THREADS = 256, VP_CH = VP_BLOCK / 64;

__global__ void __launch_bounds__(VP_THREADS) k_valid_count(Frame fr, int P, int32_t *__restrict__ cnt)
{
    __shared__ int32_t wc[VP_THREADS / 64];
    const int b = blockIdx.x, t = threadIdx.x;
    int n = 0;
    for (int j = 0; j < VP_BLOCK / VP_THREADS; ++j) {
        const int p = b * VP_BLOCK + j * VP_THREADS + t;
        n += __popcll(__ballot(p < P && valid_depth(fr, fr.depth[p])));
    }
    if (__lane_id() == 0) wc[t >> 6] = n;
    __syncthreads();
    if (t == 0) {
        int s = 0;
        for (int w = 0; w < VP_THREADS / 64; ++w) s += wc[w];
        cnt[b] = s;
    }
}

// exclusive scan of nb counts in place; the total to cnt[nb]
__global__ void __launch_bounds__(1024) k_valid_scan(int32_t *__restrict__ cnt, int nb)
{
    __shared__ int32_t ws[16];
    __shared__ int32_t carry;
    const int lane = __lane_id(), wave = threadIdx.x >> 6;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int base = 0; base < nb; base += 1024) {
        const int i = base + (int)threadIdx.x;
        const int v = i < nb ? cnt[i] : 0;
        int x = v;
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) ws[wave] = x;
        __syncthreads();
        int off = carry;
        for (int w = 0; w < wave; ++w) off += ws[w];
        __syncthreads();
        if (i < nb) cnt[i] = off + x - v;
        if (threadIdx.x == 1023) carry = off + x;
        __syncthreads();
    }
    if (threadIdx.x == 0) cnt[nb] = carry;
}

__global__ void __launch_bounds__(VP_THREADS) k_valid_emit(Frame fr, int P, const int32_t *__restrict__ off,
                                                           int32_t *__restrict__ pix)
{
    __shared__ int32_t wc[VP_CH];
    const int b = blockIdx.x, t = threadIdx.x, wave = t >> 6;
    constexpr int J = VP_BLOCK / VP_THREADS;
    bool ok[J];
    uint64_t m[J];
    for (int j = 0; j < J; ++j) {
        const int p = b * VP_BLOCK + j * VP_THREADS + t;
        ok[j] = p < P && valid_depth(fr, fr.depth[p]);
        m[j] = __ballot(ok[j]);
        if (__lane_id() == 0) wc[j * (VP_THREADS / 64) + wave] = __popcll(m[j]);
    }
    __syncthreads();
    for (int j = 0; j < J; ++j) {
        const int c = j * (VP_THREADS / 64) + wave;
        int o = off[b];
        for (int k = 0; k < c; ++k) o += wc[k];
        if (ok[j]) pix[o + __popcll(m[j] & ((1ull << __lane_id()) - 1ull))] = b * VP_BLOCK + j * VP_THREADS + t;
    }
}

static int mlp_pack(reloc_mlp *m, hipStream_t s)
{
    RL_LAUNCH("k_mlp_pack", k_mlp_pack, dim3(16), dim3(256), 0, s, m->w, m->q);
    RL_HIP(hipGetLastError());
    return RELOC_OK;
}

}  // namespace rl

using namespace rl;

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------

const uint16_t *rl_mlp_q(const reloc_mlp *m) { return m->q; }
const float *rl_mlp_w(const reloc_mlp *m) { return m->w; }

static void mlp_free(reloc_mlp *m)
{
    (void)hipFree(m->w);
    (void)hipFree(m->m);
    (void)hipFree(m->v);
    (void)hipFree(m->grad);
    (void)hipFree(m->partial);
    (void)hipFree(m->q);
    (void)hipFree(m->loss);
}

extern "C" int reloc_mlp_create(uint64_t seed, void *stream, reloc_mlp **out)
{
    if (!out) return RELOC_E_ARG;
    *out = nullptr;
    hipStream_t s = (hipStream_t)stream;
    reloc_mlp *m = new (std::nothrow) reloc_mlp();
    if (!m) return RELOC_E_NOMEM;
    if (device_malloc((void **)&m->w, NP * 4) != hipSuccess || device_malloc((void **)&m->m, NP * 4) != hipSuccess ||
        device_malloc((void **)&m->v, NP * 4) != hipSuccess || device_malloc((void **)&m->grad, (NP + 1) * 4) != hipSuccess ||
        device_malloc((void **)&m->q, NQ * 2) != hipSuccess) {
        mlp_free(m);
        delete m;
        return RELOC_E_NOMEM;
    }
    if (hipMemsetAsync(m->m, 0, NP * 4, s) != hipSuccess || hipMemsetAsync(m->v, 0, NP * 4, s) != hipSuccess) {
        mlp_free(m);
        delete m;
        return RELOC_E_HIP;
    }
    RL_LAUNCH("k_mlp_init", k_mlp_init, dim3((NP + 255) / 256), dim3(256), 0, s, m->w, seed);
    if (mlp_pack(m, s)) {
        mlp_free(m);
        delete m;
        return RELOC_E_HIP;
    }
    *out = m;
    return RELOC_OK;
}

extern "C" int reloc_mlp_destroy(reloc_mlp *m)
{
    if (!m) return RELOC_E_ARG;
    (void)hipDeviceSynchronize();
    mlp_free(m);
    delete m;
    return RELOC_OK;
}

extern "C" int reloc_mlp_get_weights(const reloc_mlp *m, float *w_host)
{
    if (!m || !w_host) return RELOC_E_ARG;
    RL_HIP(hipDeviceSynchronize());
    RL_HIP(hipMemcpy(w_host, m->w, NP * 4, hipMemcpyDeviceToHost));
    return RELOC_OK;
}

extern "C" int reloc_mlp_set_weights(reloc_mlp *m, const float *w_host)
{
    if (!m || !w_host) return RELOC_E_ARG;
    RL_HIP(hipDeviceSynchronize());
    RL_HIP(hipMemcpy(m->w, w_host, NP * 4, hipMemcpyHostToDevice));
    int rc = mlp_pack(m, 0);
    if (rc) return rc;
    RL_HIP(hipDeviceSynchronize());
    return RELOC_OK;
}

extern "C" int reloc_mlp_gradient(reloc_mlp *m, const uint16_t *x_dev, const uint8_t *y_dev, int32_t n,
                                  float *grad_host, float *loss_host, void *stream)
{
    if (!m || !x_dev || !y_dev || n < 1 || !grad_host || ((uintptr_t)x_dev & 15)) return RELOC_E_ARG;
    hipStream_t s = (hipStream_t)stream;
    int tiles = 0;
    int rc = mlp_partials(m, x_dev, y_dev, RowDraw{0, 0, 0, 0}, n, &tiles, s);
    if (rc) return rc;
    RL_LAUNCH("k_mlp_reduce", k_mlp_reduce, dim3((NP + 1 + 63) / 64), dim3(64), 0, s, m->partial, tiles, m->grad);
    RL_HIP(hipGetLastError());
    std::vector<float> g(NP + 1);
    RL_HIP(hipMemcpyAsync(g.data(), m->grad, (NP + 1) * 4, hipMemcpyDeviceToHost, s));
    RL_HIP(hipStreamSynchronize(s));
    memcpy(grad_host, g.data(), NP * 4);
    if (loss_host) *loss_host = g[NP] / (float)n;
    return RELOC_OK;
}

extern "C" int reloc_mlp_train(reloc_mlp *m, const uint16_t *x_dev, const uint8_t *y_dev, int32_t n_rows,
                               int32_t epochs, int32_t batch_rows, float lr, uint64_t seed, float *epoch_loss_host,
                               void *stream)
{
    if (!m || !x_dev || !y_dev || n_rows < 1 || epochs < 0 || batch_rows < 1 || !(lr > 0.0f) ||
        ((uintptr_t)x_dev & 15))
        return RELOC_E_ARG;
    hipStream_t s = (hipStream_t)stream;
    // (without losses nothing is allocated but the minibatch's tiles, once)
    int rc = epoch_loss_host ? ensure_loss(m, epochs) : RELOC_OK;
    if (rc) return rc;
    const int steps = std::max(1, n_rows / batch_rows);
    for (int e = 0; e < epochs; ++e) {
        for (int st = 0; st < steps; ++st) {
            int tiles = 0;
            rc = mlp_partials(m, x_dev, y_dev, RowDraw{seed, n_rows, e, st}, batch_rows, &tiles, s);
            if (rc) return rc;
            m->step++;
            const float c1 = 1.0f - powf(0.9f, (float)m->step), c2 = 1.0f - powf(0.999f, (float)m->step);
            RL_LAUNCH("k_mlp_update", k_mlp_update, dim3((NP + 1 + 63) / 64), dim3(64), 0, s, m->partial, tiles, m->w, m->m,
                      m->v, m->q, lr, c1, c2, epoch_loss_host && st == steps - 1 ? m->loss + e : nullptr);
        }
    }
    RL_HIP(hipGetLastError());
    if (epoch_loss_host && epochs > 0) {
        RL_HIP(hipMemcpyAsync(epoch_loss_host, m->loss, (size_t)epochs * sizeof(float), hipMemcpyDeviceToHost, s));
        RL_HIP(hipStreamSynchronize(s));
        for (int e = 0; e < epochs; ++e) epoch_loss_host[e] = (float)(epoch_loss_host[e] / (double)batch_rows);
    }
    return RELOC_OK;
}

extern "C" int reloc_mlp_logits(reloc_mlp *m, const uint16_t *x_dev, int32_t n, float *z_dev, void *stream)
{
    if (!m || !x_dev || !z_dev || n < 1 || ((uintptr_t)x_dev & 15)) return RELOC_E_ARG;
    RL_LAUNCH("k_mlp_logits", k_mlp_logits, dim3((n + ROWS - 1) / ROWS), dim3(64), 0, (hipStream_t)stream, x_dev, n,
              m->q, m->w, z_dev);
    RL_HIP(hipGetLastError());
    return RELOC_OK;
}

extern "C" int reloc_mlp_pixel_weights(reloc_mlp *m, reloc_forest *f, const uint16_t *depth_dev,
                                       const uint8_t *rgb_dev, const reloc_intrinsics *K, uint32_t *weights_dev,
                                       float *prob_dev, void *stream)
{
    if (!m || !f || !weights_dev) return RELOC_E_ARG;
    Frame fr;
    int rc = frame_from(f, depth_dev, rgb_dev, K, fr);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    rc = update_modes(f, s);
    if (rc) return rc;
    const int P = fr.W * fr.H;
    RL_LAUNCH("k_mlp_pixels", k_mlp_pixels, dim3((P + ROWS - 1) / ROWS), dim3(64), 0, s, feat_args(f, fr), m->q, m->w,
              weights_dev, prob_dev);
    RL_HIP(hipGetLastError());
    return RELOC_OK;
}

extern "C" int reloc_pixel_features(reloc_forest *f, const uint16_t *depth_dev, const uint8_t *rgb_dev,
                                    const reloc_intrinsics *K, const int32_t *pix_dev, int32_t n, uint16_t *x_dev,
                                    float *xf_dev, void *stream)
{
    if (!f || n < 0 || (n > 0 && (!pix_dev || !x_dev))) return RELOC_E_ARG;
    Frame fr;
    int rc = frame_from(f, depth_dev, rgb_dev, K, fr);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    rc = update_modes(f, s);
    if (rc) return rc;
    if (n == 0) return RELOC_OK;
    auto kernel = (((uintptr_t)x_dev | (uintptr_t)xf_dev) & 15) ? k_pixel_features<false> : k_pixel_features<true>;
    RL_LAUNCH("k_pixel_features", kernel, dim3((n + PIX_THREADS - 1) / PIX_THREADS), dim3(PIX_THREADS), 0, s, feat_args(f, fr),
              pix_dev, n, x_dev, xf_dev);
    RL_HIP(hipGetLastError());
    return RELOC_OK;
}

extern "C" int reloc_valid_pixels(reloc_forest *f, const uint16_t *depth_dev, const uint8_t *rgb_dev,
                                  const reloc_intrinsics *K, int32_t *pix_dev, int32_t *n_out, void *stream)
{
    if (!f || !pix_dev || !n_out) return RELOC_E_ARG;
    Frame fr;
    int rc = frame_from(f, depth_dev, rgb_dev, K, fr);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    const int P = fr.W * fr.H, nb = (P + VP_BLOCK - 1) / VP_BLOCK;
    int32_t *cnt = nullptr;
    const size_t bytes = (size_t)(nb + 1) * 4;
    // (a kept block: 37 us a call, 62 with an allocation in stream order)
    if (block_take((void **)&cnt, bytes) != hipSuccess) return RELOC_E_NOMEM;
    RL_LAUNCH("k_valid_count", k_valid_count, dim3(nb), dim3(VP_THREADS), 0, s, fr, P, cnt);
    RL_LAUNCH("k_valid_scan", k_valid_scan, dim3(1), dim3(1024), 0, s, cnt, nb);
    RL_LAUNCH("k_valid_emit", k_valid_emit, dim3(nb), dim3(VP_THREADS), 0, s, fr, P, cnt, pix_dev);
    int32_t n = 0;
    if (hipGetLastError() != hipSuccess || hipMemcpyAsync(&n, cnt + nb, 4, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        rc = RELOC_E_HIP;
    // (the stream is done with it; if the wait failed, hipFree's own is left)
    block_return(cnt, bytes, f->device, rc ? 0 : KEEP_BYTES);
    if (rc) return rc;
    *n_out = n;
    return RELOC_OK;
}

extern "C" int reloc_label_pixels(reloc_forest *f, const uint16_t *depth_dev, const uint8_t *rgb_dev,
                                  const reloc_intrinsics *K, const double pose_c2w[16], const int32_t *pix_dev,
                                  int32_t n, uint8_t *label_dev, void *stream)
{
    if (!f || !pose_c2w || n < 0 || (n > 0 && (!pix_dev || !label_dev))) return RELOC_E_ARG;
    Frame fr;
    int rc = frame_from(f, depth_dev, rgb_dev, K, fr);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    rc = update_modes(f, s);
    if (rc) return rc;
    if (n == 0) return RELOC_OK;
    PoseF P;
    for (int r = 0; r < 3; ++r) {
        for (int c = 0; c < 3; ++c) P.R[r * 3 + c] = (float)pose_c2w[r * 4 + c];
        P.t[r] = (float)pose_c2w[r * 4 + 3];
    }
    RL_LAUNCH("k_label", k_label, dim3((n + PIX_THREADS - 1) / PIX_THREADS), dim3(PIX_THREADS), 0, s, feat_args(f, fr), P, f->p.rgb_tol, pix_dev,
              n, label_dev);
    RL_HIP(hipGetLastError());
    return RELOC_OK;
}


__global__ void k_bf16_probe(const float *__restrict__ x, int n, uint16_t *__restrict__ y)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (2 * i + 1 < n) {
        const uint32_t p = bf16_pair(x[2 * i], x[2 * i + 1]);
        y[2 * i] = (uint16_t)(p & 0xFFFFu);
        y[2 * i + 1] = (uint16_t)(p >> 16);
    } else if (2 * i < n) {
        y[2 * i] = (uint16_t)(bf16_pair(x[2 * i], 0.0f) & 0xFFFFu);
    }
}

extern "C" int reloc_debug_bf16(const float *x_host, int32_t n, uint16_t *y_host)
{
    if (n < 0 || (n > 0 && (!x_host || !y_host))) return RELOC_E_ARG;
    if (n == 0) return RELOC_OK;
    float *x = nullptr;
    uint16_t *y = nullptr;
    if (device_malloc((void **)&x, (size_t)n * 4) != hipSuccess) return RELOC_E_NOMEM;
    if (device_malloc((void **)&y, (size_t)n * 2) != hipSuccess) {
        (void)hipFree(x);
        return RELOC_E_NOMEM;
    }
    int rc = RELOC_OK;
    if (hipMemcpy(x, x_host, (size_t)n * 4, hipMemcpyHostToDevice) != hipSuccess) rc = RELOC_E_HIP;
    if (!rc) {
        const int pairs = (n + 1) / 2;
        hipLaunchKernelGGL(k_bf16_probe, dim3((pairs + 255) / 256), dim3(256), 0, 0, x, n, y);
        if (hipDeviceSynchronize() != hipSuccess || hipMemcpy(y_host, y, (size_t)n * 2, hipMemcpyDeviceToHost) != hipSuccess)
            rc = RELOC_E_HIP;
    }
    (void)hipFree(x);
    (void)hipFree(y);
    return rc;
}

extern "C" int reloc_debug_mfma_probe(const uint16_t *a_host, const uint16_t *bt_host, float *c_host)
{
    if (!a_host || !bt_host || !c_host) return RELOC_E_ARG;
    uint16_t *a = nullptr, *b = nullptr;
    float *c = nullptr;
    if (device_malloc((void **)&a, 16 * 32 * 2) != hipSuccess) return RELOC_E_NOMEM;
    if (device_malloc((void **)&b, 16 * 32 * 2) != hipSuccess || device_malloc((void **)&c, 256 * 4) != hipSuccess) {
        (void)hipFree(a);
        (void)hipFree(b);
        return RELOC_E_NOMEM;
    }
    int rc = RELOC_OK;
    if (hipMemcpy(a, a_host, 16 * 32 * 2, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(b, bt_host, 16 * 32 * 2, hipMemcpyHostToDevice) != hipSuccess)
        rc = RELOC_E_HIP;
    if (!rc) {
        hipLaunchKernelGGL(k_mfma_probe, dim3(1), dim3(64), 0, 0, a, b, c);
        if (hipDeviceSynchronize() != hipSuccess || hipMemcpy(c_host, c, 256 * 4, hipMemcpyDeviceToHost) != hipSuccess)
            rc = RELOC_E_HIP;
    }
    (void)hipFree(a);
    (void)hipFree(b);
    (void)hipFree(c);
    return rc;
}
