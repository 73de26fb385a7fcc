// Device code of the learned swap proposal's network: per-node features
// (8) -> 128 -> 128 -> 1 logit on the matrix cores (v_mfma_f32_16x16x32_bf16,
// gfx950's K = 32 BF16 instruction), FP32 accumulation, FP32 biases.
//
// Precision: the weights are BF16 (W1, W2, w3 rounded to nearest even from
// the FP32 master copy).  Activations are not rounded to BF16: every
// activation operand x enters the matrix cores as two BF16 numbers, hi =
// bf16(x) and lo = bf16(x - hi), whose sum carries 16 significant bits
// (relative error <= 2^-17), and both halves are multiplied by the same
// weight.  The sums over rows in the backward pass (weight gradients) cancel
// strongly -- the loss gradient w.r.t. the logits sums to zero over the nodes
// -- so a single BF16 rounding of the activations (2^-9) would show up
// amplified in the gradients; with the split it stays below FP32 accumulation
// noise.
//
// MFMA 16x16x32 operand layout (one wavefront, lane l, g = l / 16):
//   A (16 x 32, row i, column k):  lane holds A[l % 16][8 g + j], j = 0..7
//   B (32 x 16, row k, column c):  lane holds B[8 g + j][l % 16]
//   D (16 x 16):                   lane holds D[4 g + r][l % 16],  r = 0..3
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace bnos {

constexpr int kH = 128;          // hidden width
constexpr int kF = 8;            // features per node
constexpr int kRows = 64;        // rows (nodes) of one sample, padded
constexpr int kHP = kH + 8;      // LDS row pitch of hidden activations (bf16): breaks the 256-byte row stride
constexpr int kNParam = kH * kF + kH + kH * kH + kH + kH + 1;   // 17,793
// offsets in the flat parameter vector W1 [128][8], b1, W2 [128][128], b2, w3, b3
constexpr int kOffW1 = 0;
constexpr int kOffB1 = kOffW1 + kH * kF;
constexpr int kOffW2 = kOffB1 + kH;
constexpr int kOffB2 = kOffW2 + kH * kH;
constexpr int kOffW3 = kOffB2 + kH;
constexpr int kOffB3 = kOffW3 + kH;

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

// float -> bf16 bits, round to nearest even (finite inputs)
__device__ __host__ __forceinline__ uint16_t f2bf(float x)
{
    uint32_t u;
    __builtin_memcpy(&u, &x, 4);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __host__ __forceinline__ float bf2f(uint16_t b)
{
    uint32_t u = (uint32_t)b << 16;
    float x;
    __builtin_memcpy(&x, &u, 4);
    return x;
}

// x = hi + lo + O(2^-17 |x|) for two values; x - hi is exact in FP32.  The operands come packed, x0's
// in the low halves: the card converts two values at a time.
__device__ __forceinline__ uint32_t pack_bf(float x0, float x1)
{
    typedef float v2f __attribute__((ext_vector_type(2)));
    typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f){x0, x1}, v2bf));
}
__device__ __forceinline__ void split2_bf(float x0, float x1, uint32_t &hi, uint32_t &lo)
{
    hi = pack_bf(x0, x1);
    lo = pack_bf(x0 - __builtin_bit_cast(float, hi << 16), x1 - __builtin_bit_cast(float, hi & 0xffff0000u));
}

// The same for one value.
__device__ __forceinline__ void split_bf(float x, uint16_t &hi, uint16_t &lo)
{
    uint32_t h, l;
    split2_bf(x, 0.f, h, l);
    hi = (uint16_t)h;
    lo = (uint16_t)l;
}

// Splits the four values of consecutive rows of a column and stores the operands in the rows of hi
// and lo (pitch kHP); h, l: the packed operands, rows 0 and 1, then 2 and 3.
__device__ __forceinline__ void split4_rows(const float (&x)[4], uint16_t *hi, uint16_t *lo, uint32_t (&h)[2],
                                            uint32_t (&l)[2])
{
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        split2_bf(x[2 * i], x[2 * i + 1], h[i], l[i]);
        hi[(2 * i) * kHP] = (uint16_t)h[i];
        hi[(2 * i + 1) * kHP] = (uint16_t)(h[i] >> 16);
        lo[(2 * i) * kHP] = (uint16_t)l[i];
        lo[(2 * i + 1) * kHP] = (uint16_t)(l[i] >> 16);
    }
}

// What the kernels read: BF16 weights (W2 also transposed, for the backward
// pass), w3 as the BF16-rounded floats, FP32 biases, feature normalisation.
struct MlpView {
    const uint16_t *W1b;     // [128][8]
    const uint16_t *W2b;     // [128][128]  W2[u][k]
    const uint16_t *W2tb;    // [128][128]  W2[u][k] at [k][u]
    const float *w3r;        // [128] bf16-rounded values
    const float *b1, *b2, *b3;
    const float *norm;       // [16]: mu[8], 1/sd[8]
};

__device__ __forceinline__ v4f mfma32(v4u a, v4u b, v4f c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0,
                                                   0, 0);
}

// Eight consecutive bf16 values (16-byte aligned) as one operand register set.
__device__ __forceinline__ v4u ld8(const uint16_t *p) { return *reinterpret_cast<const v4u *>(p); }

// LDS of one forward pass (16-byte aligned: operands are read with 16-byte LDS loads).
struct alignas(16) MlpLds {
    uint16_t z[kRows][16];          // normalised features: hi in columns 0..7, lo in 8..15
    uint16_t h1[2][kRows][kHP];     // relu(layer 1): [0] hi, [1] lo
    float part[kRows][8];           // per column-tile partial logits
    float logit[kRows];
};

// x[0] w[0] + ... + x[15] w[15] over the lanes of a row of 16, in the row's lane 0 (other lanes: not
// the sum): neighbours first, the even lane's product taken unrounded, then by twos, fours and eights.
template <int CTRL>
__device__ __forceinline__ float row_moved_f32(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float row_dot_f32(float x, float w)
{
    float v = fmaf(x, w, row_moved_f32<0xb1>(x * w));    // quad_perm: lane ^ 1
    v = v + row_moved_f32<0x4e>(v);                      // lane ^ 2
    v = v + row_moved_f32<0x104>(v);                     // row_shl: lane + 4
    return v + row_moved_f32<0x108>(v);                  // lane + 8
}

// A wavefront's share of the weights: the 16 hidden units of column tile wave % 8 in both layers, as
// the operands the matrix cores take.  Loaded once for as many samples as the caller has (a
// tile's operands requested where they were used made every tile wait for L2).
struct MlpRegs {
    v4u w1, w2[4];
    float b1, b2, w3;
};

__device__ __forceinline__ MlpRegs mlp_load(const MlpView &P, int wave, int lane)
{
    const int li = lane & 15, g = lane >> 4, u = (wave & 7) * 16 + li;
    MlpRegs R;
    R.w1 = (v4u){0u, 0u, 0u, 0u};
    if (g < 2) R.w1 = ld8(P.W1b + u * kF);
#pragma unroll
    for (int q = 0; q < 4; ++q) R.w2[q] = ld8(P.W2b + u * kH + q * 32 + 8 * g);
    R.b1 = P.b1[u];
    R.b2 = P.b2[u];
    R.w3 = P.w3r[u];
    return R;
}

// Forward pass of one sample (rows <= 64 nodes) by a block of 8, 16, 24 or 32 wavefronts: wavefront w
// takes the columns of tile w % 8 for the row tiles w / 8, w / 8 + waves / 8, ... that hold rows.
// zraw: raw features [rows][8] (LDS or global).  The logits land in L.logit[0..rows).  Fixed
// reduction orders: deterministic.
__device__ __forceinline__ void mlp_forward_block(const MlpView &P, const MlpRegs &R, const float *zraw, int rows,
                                                  MlpLds &L)
{
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int nw = blockDim.x >> 6;
    const int tiles = (rows + 15) >> 4;
    for (int e = tid; e < tiles * 16 * kF; e += blockDim.x) {
        const int r = e / kF, k = e % kF;
        float v = 0.f;
        if (r < rows) v = (zraw[r * kF + k] - P.norm[k]) * P.norm[kF + k];
        split_bf(v, L.z[r][k], L.z[r][kF + k]);
    }
    __syncthreads();
    const int li = lane & 15, g = lane >> 4, ct = wave & 7, u = ct * 16 + li;
    // layer 1: one K = 32 step per tile: A = [z_hi | z_lo | 0 | 0], B = [W1^T; W1^T; 0; 0], so
    // the product is (z_hi + z_lo) W1^T
    for (int rt = wave >> 3; rt < tiles; rt += nw >> 3) {
        v4u a = {0u, 0u, 0u, 0u};
        if (g < 2) a = ld8(&L.z[rt * 16 + li][8 * g]);
        const v4f d = mfma32(a, R.w1, (v4f){0.f, 0.f, 0.f, 0.f});
        float h[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float x = d[r] + R.b1;
            h[r] = x > 0.f ? x : 0.f;
        }
        uint32_t hh[2], hl[2];
        split4_rows(h, &L.h1[0][rt * 16 + 4 * g][u], &L.h1[1][rt * 16 + 4 * g][u], hh, hl);
    }
    __syncthreads();
    // layer 2: K = 128 inputs, taken twice (hi, then lo), each against W2; then
    // the layer-3 dot products per column tile
    for (int rt = wave >> 3; rt < tiles; rt += nw >> 3) {
        v4f d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 8; ++s)
            d = mfma32(ld8(&L.h1[s >> 2][rt * 16 + li][(s & 3) * 32 + 8 * g]), R.w2[s & 3], d);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float x = d[r] + R.b2;
            const float q = row_dot_f32(x > 0.f ? x : 0.f, R.w3);
            if (li == 0) L.part[rt * 16 + 4 * g + r][ct] = q;
        }
    }
    __syncthreads();
    if (tid < kRows) {
        float s = P.b3[0];
#pragma unroll
        for (int c = 0; c < 8; ++c) s += L.part[tid][c];
        L.logit[tid] = s;                    // (past the row tiles: unused)
    }
    __syncthreads();
}

// ln q({a,b}) from logits (FP64 softmax of the FP32 logits), eps mixing weight.
__device__ __forceinline__ double pair_logq_dev(const float *logit, int n, int a, int b, double eps)
{
    double mx = -1e300;
    for (int i = 0; i < n; ++i) mx = logit[i] > mx ? logit[i] : mx;
    double s = 0.0;
    for (int i = 0; i < n; ++i) s += exp((double)logit[i] - mx);
    const double pa = exp((double)logit[a] - mx) / s, pb = exp((double)logit[b] - mx) / s;
    const double Q = pa * pb * (1.0 / (1.0 - pa) + 1.0 / (1.0 - pb));
    return log((1.0 - eps) * Q + eps * 2.0 / ((double)n * (n - 1)));
}

// host side (mlp.hip)
MlpView mlp_view(const void *mlp_handle);
bool mlp_handle_live(const void *mlp_handle);

}  // namespace bnos
