// MLP closure kernels: fused forward (and backward) of a tile of rows per
// workgroup on the 16x16x32 BF16 matrix cores with FP32 accumulation.
//
// Precision contract: inputs, weights, hidden activations fed to the next
// layer and pre-activation gradients fed to a product are bfloat16 (round
// to nearest even); products accumulate in FP32; biases, pre-activations,
// SiLU, bias gradients and the optimiser run in FP32.
//
// Eight waves per workgroup; wave w owns features 16w..16w+15 of every hidden
// layer for all rows of the tile, so that its weights are read once, ahead of
// the first product, and the time of a tile is that of a short chain:
//   forward    H_l^T = silu(W_l^T H_{l-1}^T + b_l)   K = 32 or 128
//   backward   dH_{l-1}^T = W_l dZ_l^T               contraction over the outputs
//              dW_l^T = dZ_l^T H_{l-1}               contraction over the 32 rows
// The products are formed transposed (features down, rows across), so that a
// lane holds four consecutive features of a row and the row-major tile that
// feeds the next product takes them in one 8-byte write.  Copies with the
// rows contiguous (H_l and dZ_l by feature) feed the weight gradients, so
// every matrix-core operand is one 16-byte LDS read.
#include <cmath>

#include "mlp.h"

namespace dsmcx {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kSA = 136;  // row stride (elements) of row-major tiles [32][128 + 8]
constexpr int kST = 40;   // row stride of transposed tiles [features][32 + 8]
constexpr int kSX = 40;   // row stride of the input tile [rows][32 + 8]
constexpr int kThreads = 512;
constexpr int kReduceThreads = 64;
constexpr int64_t kMlpSmallRows = 32768;
constexpr int64_t kMlpGrid = 512;
constexpr int kParamBlocks = (kMlpParams + kReduceThreads - 1) / kReduceThreads;

constexpr int kOffWf1 = 0, kOffWf2 = kOffWf1 + 128 * 32, kOffWf3 = kOffWf2 + 128 * 128, kOffWf4 = kOffWf3 + 128 * 128,
              kOffWb2 = kOffWf4 + 16 * 128, kOffWb3 = kOffWb2 + 128 * 128, kOffWb4 = kOffWb3 + 128 * 128;

__device__ __forceinline__ uint32_t pack2(float a, float b) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

__device__ __forceinline__ uint16_t to_bf16(float f) { return (uint16_t)pack2(f, 0.0f); }

__device__ __forceinline__ f32x4 mfma(uint4 a, uint4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                   0, 0, 0);
}

// 1 / (1 + exp(-z)).  The reciprocal of d = (1 + exp(-z)) / 4, at least 1/4 and
// a normal number wherever it is finite, from the hardware's by one Newton
// step: equal to the quotient for every float z > -87.33; below, where the
// result is denormal, within its last bit (all 2^32 compared).  Half of the
// instructions of a division.
__device__ __forceinline__ float sigmoidf(float z) {
    const float d = __builtin_fmaf(0.25f, expf(-z), 0.25f);
    float r = __builtin_amdgcn_rcpf(d);
    r = __builtin_fmaf(__builtin_fmaf(-d, r, 1.0f), r, r);
    return 0.25f * __builtin_amdgcn_div_fixupf(r, d, 1.0f);
}

// This lane's matrix-core operands of row `row` of a [rows][32 KS] matrix.
template <int KS>
__device__ __forceinline__ void operand(const uint16_t* M, int ld, int row, uint4* o) {
    const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) o[ks] = *(const uint4*)(M + (size_t)row * ld + ks * 32 + 8 * g);
}

// acc[b] = W (this wave's 16 features) times the rows 16b.. of the row-major
// tile T: lane (r, g) gets features 4g.. of row 16b + r.
template <int KS, int RB>
__device__ __forceinline__ void mm(const uint4* W, const uint16_t* T, int ld, f32x4* acc) {
    const int r = threadIdx.x & 15, g = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int b = 0; b < RB; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int b = 0; b < RB; ++b)
            acc[b] = mfma(W[ks], *(const uint4*)(T + (16 * b + r) * ld + ks * 32 + 8 * g), acc[b]);
}

// Hidden-layer epilogue: z = acc + b, h = silu(z) (bf16) into the next
// row-major tile and (training) the tile by features; z and its sigmoid kept
// for the backward.
template <bool TRAIN, int RB>
__device__ __forceinline__ void hidden_out(const f32x4* acc, f32x4 bias, uint16_t* Hn, uint16_t* Ht, f32x4* zkeep,
                                           f32x4* skeep) {
    const int r = threadIdx.x & 15, g = (threadIdx.x & 63) >> 4, f0 = 16 * (threadIdx.x >> 6) + 4 * g;
#pragma unroll
    for (int b = 0; b < RB; ++b) {
        float h[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float z = acc[b][i] + bias[i];
            const float s = sigmoidf(z);
            if (TRAIN) {
                zkeep[b][i] = z;
                skeep[b][i] = s;
            }
            h[i] = z * s;
        }
        uint2 pk;
        pk.x = pack2(h[0], h[1]);
        pk.y = pack2(h[2], h[3]);
        *(uint2*)(Hn + (16 * b + r) * kSA + f0) = pk;
        if (TRAIN) {
            uint16_t* t = Ht + f0 * kST + 16 * b + r;
            t[0] = (uint16_t)pk.x;
            t[kST] = (uint16_t)(pk.x >> 16);
            t[2 * kST] = (uint16_t)pk.y;
            t[3 * kST] = (uint16_t)(pk.y >> 16);
        }
    }
}

// Value of lane K of each group of four.
template <int K>
__device__ __forceinline__ float quad(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), K * 0x55, 0xf, 0xf, true));
}

// dZ = dH * silu'(z) (FP32), stored bf16 by rows (D, unless null) and by
// features (Dt); the FP32 sums over the rows of this wave's features go to
// bias_grad.
__device__ __forceinline__ void grad_out(const f32x4* dh, const f32x4* z, const f32x4* sg, uint16_t* D, uint16_t* Dt,
                                         float* bias_grad) {
    const int r = threadIdx.x & 15, g = (threadIdx.x & 63) >> 4, f0 = 16 * (threadIdx.x >> 6) + 4 * g;
    float s[2][4];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        float d[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            d[i] = dh[b][i] * (sg[b][i] * (1.0f + z[b][i] * (1.0f - sg[b][i])));
            // rows in fours, then the fours
            float q = (((0.f + quad<0>(d[i])) + quad<1>(d[i])) + quad<2>(d[i])) + quad<3>(d[i]);
            q += __shfl_xor(q, 4, 64);
            q += __shfl_xor(q, 8, 64);
            s[b][i] = q;
        }
        uint2 pk;
        pk.x = pack2(d[0], d[1]);
        pk.y = pack2(d[2], d[3]);
        if (D) *(uint2*)(D + (16 * b + r) * kSA + f0) = pk;
        uint16_t* t = Dt + f0 * kST + 16 * b + r;
        t[0] = (uint16_t)pk.x;
        t[kST] = (uint16_t)(pk.x >> 16);
        t[2 * kST] = (uint16_t)pk.y;
        t[3 * kST] = (uint16_t)(pk.y >> 16);
    }
    if (r == 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) bias_grad[f0 + i] = s[0][i] + s[1][i];
    }
}

// Weight gradient W[k][n] (flat, in-major) = sum_r dZ[r][n] H[r][k] for the 16
// features n of this wave: rows n of Dt (its own, so that no other wave has to
// be waited for), rows k of Ht.
template <int NKT>
__device__ __forceinline__ void weight_grad(const uint16_t* Dt, const uint16_t* Ht, int kvalid, float* out) {
    const int r = threadIdx.x & 15, g = (threadIdx.x & 63) >> 4, n0 = 16 * (threadIdx.x >> 6);
    uint4 a;
    operand<1>(Dt, kST, n0 + r, &a);
    f32x4 acc[NKT];
#pragma unroll
    for (int t = 0; t < NKT; ++t) {
        uint4 b;
        operand<1>(Ht, kST, 16 * t + r, &b);
        acc[t] = mfma(a, b, f32x4{0.f, 0.f, 0.f, 0.f});
    }
#pragma unroll
    for (int t = 0; t < NKT; ++t)
        if (16 * t + r < kvalid) *(f32x4*)(out + (size_t)(16 * t + r) * kMlpHid + n0 + 4 * g) = acc[t];
}

// The output layer of rows 16b.. (one wave): lane (r, g) gets output r of rows
// 4g...
__device__ __forceinline__ f32x4 output_layer(const MlpDev& m, const uint16_t* H, int b) {
    const int r = threadIdx.x & 15;
    uint4 a[4], w[4];
    operand<4>(m.wf4, 128, r, w);
    operand<4>(H, kSA, 16 * b + r, a);
    f32x4 out = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) out = mfma(a[ks], w[ks], out);
    return out;
}

__device__ __forceinline__ f32x4 bias4(const float* b) {
    const int f0 = 16 * (threadIdx.x >> 6) + 4 * ((threadIdx.x & 63) >> 4);
    return f32x4{b[f0], b[f0 + 1], b[f0 + 2], b[f0 + 3]};
}

// Forward of tiles of 16 RB rows, the workgroups striding over them with the
// weights in registers.  Bounded by the vector instructions of the SiLUs (some
// 25 each, 384 a row).  A call with its synchronisation, against two waves of
// 16 rows by all features each: 30 rows 18 us (26), 48,000 31 (47), 400,000 141
// (275).
template <int RB>
__global__ __launch_bounds__(kThreads) void k_mlp_forward(MlpDev m, const float* x, int64_t n, float* y) {
    constexpr int kRows = 16 * RB;
    __shared__ __attribute__((aligned(16))) uint16_t X[kRows * kSX];
    __shared__ __attribute__((aligned(16))) uint16_t HA[kRows * kSA];
    __shared__ __attribute__((aligned(16))) uint16_t HB[kRows * kSA];
    const int tid = threadIdx.x, w = tid >> 6, r = tid & 15, g = (tid & 63) >> 4;
    uint4 w1, w2[4], w3[4];
    operand<1>(m.wf1, 32, 16 * w + r, &w1);
    operand<4>(m.wf2, 128, 16 * w + r, w2);
    operand<4>(m.wf3, 128, 16 * w + r, w3);
    const f32x4 b1 = bias4(m.params + kMlpB1), b2 = bias4(m.params + kMlpB2), b3 = bias4(m.params + kMlpB3);
    const float b4 = r < kMlpOut ? m.params[kMlpB4 + r] : 0.f;
    for (int e = tid; e < kRows * kSX; e += kThreads) X[e] = 0;
    constexpr int kLoads = (kRows * kMlpIn + kThreads - 1) / kThreads;
    float in[kLoads];
    auto load = [&](int64_t tile) {
#pragma unroll
        for (int k = 0; k < kLoads; ++k) {
            const int e = tid + kThreads * k;
            const int64_t at = tile * kRows * kMlpIn + e;
            in[k] = e < kRows * kMlpIn && at < n * kMlpIn ? x[at] : 0.f;
        }
    };
    const int64_t tiles = (n + kRows - 1) / kRows;
    load(blockIdx.x);
    __syncthreads();
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
#pragma unroll
        for (int k = 0; k < kLoads; ++k) {
            const int e = tid + kThreads * k;
            if (e < kRows * kMlpIn) X[e / kMlpIn * kSX + e % kMlpIn] = to_bf16(in[k]);
        }
        __syncthreads();
        if (tile + gridDim.x < tiles) load(tile + gridDim.x);
        f32x4 acc[RB];
        mm<1, RB>(&w1, X, kSX, acc);
        hidden_out<false, RB>(acc, b1, HB, nullptr, nullptr, nullptr);
        __syncthreads();
        mm<4, RB>(w2, HB, kSA, acc);
        hidden_out<false, RB>(acc, b2, HA, nullptr, nullptr, nullptr);
        __syncthreads();
        mm<4, RB>(w3, HA, kSA, acc);
        hidden_out<false, RB>(acc, b3, HB, nullptr, nullptr, nullptr);
        __syncthreads();
        if (w < RB) {
            const f32x4 out = output_layer(m, HB, w);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t row = tile * kRows + 16 * w + 4 * g + i;
                if (row < n && r < kMlpOut) y[row * kMlpOut + r] = out[i] + b4;
            }
        }
    }
}

// Forward and backward of a tile of 32 rows, given or (batch.on) drawn from the
// n rows with replacement (purpose 8); the tile's share of the gradient and of
// the loss to partial and loss_partial.  Bounded by the chain of the seven
// products with their barriers and, over many tiles, by the writes of the
// partial gradients.  With the reduction, against two waves per tile: 397 rows
// 20 us (35), 4,096 rows 30 (75).
__global__ __launch_bounds__(kThreads) void k_mlp_tile(MlpDev m, const float* x, const float* tgt, MlpBatch batch,
                                                       int64_t n, float scale, float* partial, float* loss_partial) {
    __shared__ __attribute__((aligned(16))) uint16_t HA[kMlpTile * kSA];
    __shared__ __attribute__((aligned(16))) uint16_t HB[kMlpTile * kSA];
    __shared__ __attribute__((aligned(16))) uint16_t X[kMlpTile * kSX];
    __shared__ __attribute__((aligned(16))) uint16_t Ht0[32 * kST];
    __shared__ __attribute__((aligned(16))) uint16_t Ht1[128 * kST];
    __shared__ __attribute__((aligned(16))) uint16_t Ht2[128 * kST];
    __shared__ __attribute__((aligned(16))) uint16_t Ht3[128 * kST];
    __shared__ __attribute__((aligned(16))) uint16_t Dt[128 * kST];
    __shared__ __attribute__((aligned(16))) uint16_t Dt4[16 * kST];
    __shared__ int32_t src[kMlpTile];
    __shared__ float bsum[2 * 16];
    __shared__ float lsum[2];

    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, r = l & 15, g = l >> 4;
    const int64_t base = (int64_t)blockIdx.x * kMlpTile;

    // the wave's weights of every product
    uint4 w1, w2[4], w3[4], v4, v3[4], v2[4];
    operand<1>(m.wf1, 32, 16 * w + r, &w1);
    operand<4>(m.wf2, 128, 16 * w + r, w2);
    operand<4>(m.wf3, 128, 16 * w + r, w3);
    operand<1>(m.wb4, 32, 16 * w + r, &v4);
    operand<4>(m.wb3, 128, 16 * w + r, v3);
    operand<4>(m.wb2, 128, 16 * w + r, v2);
    const f32x4 b1 = bias4(m.params + kMlpB1), b2 = bias4(m.params + kMlpB2), b3 = bias4(m.params + kMlpB3);

    // rows of the tile, 13 features padded to 32
    if (tid < kMlpTile) {
        int32_t s = (int32_t)(base + tid);
        if (batch.on && base + tid < n) {
            const Rand4 q = draw(batch.key, (uint32_t)((base + tid) & 0xFFFFFFFF), batch.step, kPurposeMlp, 0);
            s = (int32_t)pick(q.w[0], (uint32_t)batch.rows);
        }
        src[tid] = s;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kMlpTile * 32 / kThreads; ++k) {
        const int e = tid + kThreads * k, rr = e >> 5, f = e & 31;
        const uint16_t b = to_bf16(base + rr < n && f < kMlpIn ? x[(int64_t)src[rr] * kMlpIn + f] : 0.f);
        X[rr * kSX + f] = b;
        Ht0[f * kST + rr] = b;
    }
    // targets of the output layer's waves
    float t4[4] = {0.f, 0.f, 0.f, 0.f};
    if (w < 2 && r < kMlpOut) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int rr = 16 * w + 4 * g + i;
            if (base + rr < n) t4[i] = tgt[(int64_t)src[rr] * kMlpOut + r];
        }
    }
    __syncthreads();

    f32x4 acc[2], z1[2], z2[2], z3[2], s1[2], s2[2], s3[2];
    mm<1, 2>(&w1, X, kSX, acc);
    hidden_out<true, 2>(acc, b1, HB, Ht1, z1, s1);
    __syncthreads();
    mm<4, 2>(w2, HB, kSA, acc);
    hidden_out<true, 2>(acc, b2, HA, Ht2, z2, s2);
    __syncthreads();
    mm<4, 2>(w3, HA, kSA, acc);
    hidden_out<true, 2>(acc, b3, HB, Ht3, z3, s3);
    __syncthreads();

    // ---- backward ------------------------------------------------------
    // dY = scale (y - t); bf16 copies: row-major [32][32] in HA (columns
    // >= 9 zero), by outputs [16][32] in Dt4.  Waves 0 and 1, 16 rows each;
    // the others clear the columns 16..31 of HA.
    if (w < 2) {
        const f32x4 out = output_layer(m, HB, w);
        const float b4 = r < kMlpOut ? m.params[kMlpB4 + r] : 0.f;
        float dz[4], loss = 0.f, s4 = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t row = base + 16 * w + 4 * g + i;
            float d = 0.f;
            if (row < n && r < kMlpOut) {
                const float e = (out[i] + b4) - t4[i];
                loss += e * e;
                d = scale * e;
            }
            dz[i] = d;
            s4 += d;
        }
        uint2 pk;
        pk.x = pack2(dz[0], dz[1]);
        pk.y = pack2(dz[2], dz[3]);
        *(uint2*)(Dt4 + r * kST + 16 * w + 4 * g) = pk;
        uint16_t* h = HA + (16 * w + 4 * g) * kSA + r;
        h[0] = (uint16_t)pk.x;
        h[kSA] = (uint16_t)(pk.x >> 16);
        h[2 * kSA] = (uint16_t)pk.y;
        h[3 * kSA] = (uint16_t)(pk.y >> 16);
        s4 += __shfl_xor(s4, 16, 64);
        s4 += __shfl_xor(s4, 32, 64);
        if (g == 0) bsum[w * 16 + r] = s4;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) loss += __shfl_xor(loss, o, 64);
        if (l == 0) lsum[w] = loss;
    } else if (tid < 128 + 64) {
        const int e = tid - 128;
        *(uint4*)(HA + (e >> 1) * kSA + 16 + 8 * (e & 1)) = uint4{0, 0, 0, 0};
    }
    __syncthreads();
    float* P = partial + (size_t)blockIdx.x * kMlpPartial;
    if (tid < kMlpOut) P[kMlpB4 + tid] = bsum[tid] + bsum[16 + tid];
    if (tid == 0) loss_partial[blockIdx.x] = lsum[0] + lsum[1];
    // dH3 = dZ4 W4^T (contraction over the 9 outputs padded to 32)
    mm<1, 2>(&v4, HA, kSA, acc);
    grad_out(acc, z3, s3, HB, Dt, P + kMlpB3);
    // dW4 (16 output rows of which 9 are real): wave w takes inputs 16w..
    {
        uint4 a, b;
        operand<1>(Dt4, kST, r, &a);
        operand<1>(Ht3, kST, 16 * w + r, &b);
        const f32x4 a4 = mfma(a, b, f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (4 * g + i < kMlpOut) P[kMlpW4 + (16 * w + r) * kMlpOut + 4 * g + i] = a4[i];
    }
    __syncthreads();
    mm<4, 2>(v3, HB, kSA, acc);
    weight_grad<8>(Dt, Ht2, 128, P + kMlpW3);
    grad_out(acc, z2, s2, HA, Dt, P + kMlpB2);
    __syncthreads();
    mm<4, 2>(v2, HA, kSA, acc);
    weight_grad<8>(Dt, Ht1, 128, P + kMlpW2);
    grad_out(acc, z1, s1, nullptr, Dt, P + kMlpB1);
    __syncthreads();
    weight_grad<2>(Dt, Ht0, kMlpIn, P + kMlpW1);
}

// Sum of parameter p's partials over the tiles, in their order; the loads of
// sixteen tiles are in flight at a time.
__device__ __forceinline__ float partial_sum(const float* partial, int64_t nblk, int p) {
    const float* q = partial + p;
    float s = 0.f;
    int64_t b = 0;
    for (; b + 16 <= nblk; b += 16) {
        float v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = q[(size_t)(b + k) * kMlpPartial];
#pragma unroll
        for (int k = 0; k < 16; ++k) s += v[k];
    }
    for (; b < nblk; ++b) s += q[(size_t)b * kMlpPartial];
    return s;
}

// The loss over the tiles in their order (one wave: loads by all lanes).
__device__ __forceinline__ void loss_sum(const float* loss_partial, int64_t nblk, double* loss, double denom) {
    __shared__ float v[64];
    const int l = threadIdx.x;
    double s = 0.0;
    for (int64_t b0 = 0; b0 < nblk; b0 += 64) {
        if (b0 + l < nblk) v[l] = loss_partial[b0 + l];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const int m = (int)(nblk - b0 < 64 ? nblk - b0 : 64);
        if (l == 0)
            for (int k = 0; k < m; ++k) s += (double)v[k];
        __builtin_amdgcn_wave_barrier();
    }
    if (l == 0) *loss = s / denom;
}

// grad[p] = sum over tiles of the partials (fixed order); the last workgroup
// adds the loss.
__global__ __launch_bounds__(kReduceThreads) void k_mlp_reduce(const float* partial, const float* loss_partial,
                                                               int64_t nblk, float* grad, double* loss, double denom) {
    if (blockIdx.x == kParamBlocks) {
        if (threadIdx.x < 64) loss_sum(loss_partial, nblk, loss, denom);
        return;
    }
    const int p = blockIdx.x * kReduceThreads + threadIdx.x;
    if (p < kMlpParams) grad[p] = partial_sum(partial, nblk, p);
}

// Parameter p of the FP32 weights into its bf16 operand copies.
__device__ __forceinline__ void pack_param(int p, float v, uint16_t* out) {
    const uint16_t b = to_bf16(v);
    if (p < kMlpB1) {
        const int q = p - kMlpW1, k = q >> 7, nn = q & 127;
        out[kOffWf1 + nn * 32 + k] = b;
    } else if (p >= kMlpW2 && p < kMlpB2) {
        const int q = p - kMlpW2, k = q >> 7, nn = q & 127;
        out[kOffWf2 + nn * 128 + k] = b;
        out[kOffWb2 + q] = b;
    } else if (p >= kMlpW3 && p < kMlpB3) {
        const int q = p - kMlpW3, k = q >> 7, nn = q & 127;
        out[kOffWf3 + nn * 128 + k] = b;
        out[kOffWb3 + q] = b;
    } else if (p >= kMlpW4 && p < kMlpB4) {
        const int q = p - kMlpW4, k = q / kMlpOut, j = q - k * kMlpOut;
        out[kOffWf4 + j * 128 + k] = b;
        out[kOffWb4 + k * 32 + j] = b;
    }
}

__device__ __forceinline__ float adam(float* params, float* m, float* v, int p, float g, MlpAdam a) {
    const float mm_ = a.b1 * m[p] + (1.0f - a.b1) * g;
    const float vv = a.b2 * v[p] + (1.0f - a.b2) * g * g;
    m[p] = mm_;
    v[p] = vv;
    const float x = params[p] - a.lr * (mm_ / a.c1) / (sqrtf(vv / a.c2) + a.eps);
    params[p] = x;
    return x;
}

// Optimiser step from a given gradient, with the operand copies.
__global__ void k_mlp_adam(float* params, const float* grad, float* m, float* v, MlpAdam a, uint16_t* packed) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < kMlpParams) pack_param(p, adam(params, m, v, p, grad[p], a), packed);
}

// A training step after its tiles: the gradient (not kept), the optimiser, the
// operand copies, and by the last workgroup the loss; one launch where there
// were three.  A step on 4,096 of 48,000 rows: tiles 23 us and this 8, where
// draw, tiles, reduction, optimiser and copies took 93.
__global__ __launch_bounds__(kReduceThreads) void k_mlp_step(const float* partial, const float* loss_partial,
                                                             int64_t nblk, double* loss, float* params, float* m,
                                                             float* v, MlpAdam a, uint16_t* packed) {
    if (blockIdx.x == kParamBlocks) {
        if (threadIdx.x < 64) loss_sum(loss_partial, nblk, loss, 1.0);
        return;
    }
    const int p = blockIdx.x * kReduceThreads + threadIdx.x;
    if (p < kMlpParams) pack_param(p, adam(params, m, v, p, partial_sum(partial, nblk, p), a), packed);
}

// bf16 operand copies of the FP32 weights (zero padding).
__global__ void k_mlp_pack(const float* P, uint16_t* out) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= kMlpPackTotal) return;
    float v = 0.f;
    if (e < kOffWf2) {  // wf1[n][k], k < 32
        const int q = e - kOffWf1, nn = q >> 5, k = q & 31;
        if (k < kMlpIn) v = P[kMlpW1 + k * 128 + nn];
    } else if (e < kOffWf3) {
        const int q = e - kOffWf2, nn = q >> 7, k = q & 127;
        v = P[kMlpW2 + k * 128 + nn];
    } else if (e < kOffWf4) {
        const int q = e - kOffWf3, nn = q >> 7, k = q & 127;
        v = P[kMlpW3 + k * 128 + nn];
    } else if (e < kOffWb2) {  // wf4[j][k], j < 16
        const int q = e - kOffWf4, j = q >> 7, k = q & 127;
        if (j < kMlpOut) v = P[kMlpW4 + k * kMlpOut + j];
    } else if (e < kOffWb3) {  // wb2[k][n]
        v = P[kMlpW2 + (e - kOffWb2)];
    } else if (e < kOffWb4) {
        v = P[kMlpW3 + (e - kOffWb3)];
    } else {  // wb4[k][j], j < 32
        const int q = e - kOffWb4, k = q >> 5, j = q & 31;
        if (j < kMlpOut) v = P[kMlpW4 + k * kMlpOut + j];
    }
    out[e] = to_bf16(v);
}

// Initial weights uniform in (-1, 1)/sqrt(fan_in) (purpose 8, block 1,
// subject = parameter index), biases zero.
__global__ void k_mlp_init(float* P, RngKey key) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= kMlpParams) return;
    int fan = 0;
    if (p < kMlpB1) fan = kMlpIn;
    else if (p >= kMlpW2 && p < kMlpB2) fan = kMlpHid;
    else if (p >= kMlpW3 && p < kMlpB3) fan = kMlpHid;
    else if (p >= kMlpW4 && p < kMlpB4) fan = kMlpHid;
    if (!fan) {
        P[p] = 0.f;
        return;
    }
    const Rand4 r = draw(key, (uint32_t)p, 0u, kPurposeMlp, 1);
    P[p] = (float)((2.0 * u01(r.w[0], r.w[1]) - 1.0) / sqrt((double)fan));
}

}  // namespace

MlpDev mlp_dev_view(const float* params, const uint16_t* packed) {
    MlpDev d;
    d.wf1 = packed + kOffWf1;
    d.wf2 = packed + kOffWf2;
    d.wf3 = packed + kOffWf3;
    d.wf4 = packed + kOffWf4;
    d.wb2 = packed + kOffWb2;
    d.wb3 = packed + kOffWb3;
    d.wb4 = packed + kOffWb4;
    d.params = params;
    return d;
}

void launch_mlp_pack(hipStream_t s, const float* params, uint16_t* packed) {
    hipLaunchKernelGGL(k_mlp_pack, dim3((kMlpPackTotal + 255) / 256), dim3(256), 0, s, params, packed);
}

int64_t mlp_blocks(int64_t n) { return (n + kMlpTile - 1) / kMlpTile; }

void launch_mlp_forward(hipStream_t s, const MlpDev& m, const float* x, int64_t n, float* y) {
    if (n <= 0) return;
    // 64-row tiles where there are enough to fill the card (half of the LDS
    // reads and of the workgroups' starts per row; 100,000 rows: 51 us against
    // 53, 48,000: 31 against 34), 32-row ones below, a shorter chain (24,000
    // rows: 25 us against 26, 8,192: 18 against 21)
    if (n > kMlpSmallRows) {
        const int64_t tiles = (n + 63) / 64;
        hipLaunchKernelGGL(k_mlp_forward<4>, dim3((unsigned)(tiles < kMlpGrid ? tiles : kMlpGrid)), dim3(kThreads), 0,
                           s, m, x, n, y);
    } else {
        hipLaunchKernelGGL(k_mlp_forward<2>, dim3((unsigned)((n + 31) / 32)), dim3(kThreads), 0, s, m, x, n, y);
    }
}

void launch_mlp_grad(hipStream_t s, const MlpDev& m, const float* x, const float* t, const MlpBatch& batch, int64_t n,
                     float* partial, float* loss_partial) {
    if (n <= 0) return;
    const float scale = (float)(2.0 / ((double)n * kMlpOut));
    hipLaunchKernelGGL(k_mlp_tile, dim3((unsigned)mlp_blocks(n)), dim3(kThreads), 0, s, m, x, t, batch, n, scale,
                       partial, loss_partial);
}

void launch_mlp_reduce(hipStream_t s, const float* partial, const float* loss_partial, int64_t nblk, float* grad,
                       double* loss, double denom) {
    hipLaunchKernelGGL(k_mlp_reduce, dim3(kParamBlocks + 1), dim3(kReduceThreads), 0, s, partial, loss_partial, nblk,
                       grad, loss, denom);
}

MlpAdam mlp_adam(int step, float lr, float b1, float b2, float eps) {
    const auto c = [step](float b) { return (float)(1.0 - std::pow((double)b, step)); };
    return MlpAdam{lr, b1, b2, eps, c(b1), c(b2)};
}

void launch_mlp_adam(hipStream_t s, float* params, const float* grad, float* m, float* v, const MlpAdam& a,
                     uint16_t* packed) {
    hipLaunchKernelGGL(k_mlp_adam, dim3((kMlpParams + 255) / 256), dim3(256), 0, s, params, grad, m, v, a, packed);
}

void launch_mlp_step(hipStream_t s, const float* partial, const float* loss_partial, int64_t nblk, double* loss,
                     float* params, float* m, float* v, const MlpAdam& a, uint16_t* packed) {
    hipLaunchKernelGGL(k_mlp_step, dim3(kParamBlocks + 1), dim3(kReduceThreads), 0, s, partial, loss_partial, nblk,
                       loss, params, m, v, a, packed);
}

void launch_mlp_init(hipStream_t s, float* params, RngKey key) {
    hipLaunchKernelGGL(k_mlp_init, dim3((kMlpParams + 255) / 256), dim3(256), 0, s, params, key);
}

}  // namespace dsmcx
