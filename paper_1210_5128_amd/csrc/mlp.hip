// The learned swap proposal's network on the device: parameters (FP32
// master + BF16 copies), forward pass, loss gradient by hand-written
// MFMA backward GEMMs, deterministic reductions and Adam.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <mutex>
#include <set>
#include <string>
#include <vector>

#include "bnos_internal.h"
#include "mlp_device.h"
#include "score_device.h"

namespace bnos {

struct MlpT {
    uint32_t magic = 0;
    int device = 0;
    float *d_master = nullptr;   // [kNParam]
    float *d_m = nullptr;        // Adam first moment
    float *d_v = nullptr;        // Adam second moment
    uint16_t *d_W1b = nullptr;   // [128][8]
    uint16_t *d_W2b = nullptr;   // [128][128]
    uint16_t *d_W2tb = nullptr;  // [128][128], transposed
    float *d_w3r = nullptr;      // [128]
    float *d_norm = nullptr;     // [16]: mu, 1/sd
    double *d_normpart = nullptr;   // [kNormBlocks][16]: per-block feature sums
    float h_mu[kF], h_sd[kF];
    int64_t adam_t = 0;
};

constexpr uint32_t kMlpMagic = 0x3E7A11CEu;
static std::mutex g_mlp_mu;
static std::set<const MlpT *> g_mlps;

static bool mlp_live(const MlpT *m)
{
    std::lock_guard<std::mutex> lk(g_mlp_mu);
    return m && g_mlps.count(m) && m->magic == kMlpMagic;
}

MlpView mlp_view(const void *h)
{
    const MlpT *m = reinterpret_cast<const MlpT *>(h);
    MlpView P;
    P.W1b = m->d_W1b;
    P.W2b = m->d_W2b;
    P.W2tb = m->d_W2tb;
    P.w3r = m->d_w3r;
    P.b1 = m->d_master + kOffB1;
    P.b2 = m->d_master + kOffB2;
    P.b3 = m->d_master + kOffB3;
    P.norm = m->d_norm;
    return P;
}

bool mlp_handle_live(const void *h) { return mlp_live(reinterpret_cast<const MlpT *>(h)); }

// ------------------------------------------------------------------ kernels

// BF16 copies of the weights from the FP32 master (W2 also transposed).
__global__ void k_mlp_refresh(const float *__restrict__ master, uint16_t *__restrict__ W1b,
                              uint16_t *__restrict__ W2b, uint16_t *__restrict__ W2tb, float *__restrict__ w3r)
{
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g < kH * kF) {
        W1b[g] = f2bf(master[kOffW1 + g]);
    } else if (g < kH * kF + kH * kH) {
        const int e = g - kH * kF;
        const uint16_t b = f2bf(master[kOffW2 + e]);
        W2b[e] = b;
        W2tb[(e % kH) * kH + e / kH] = b;
    } else if (g < kH * kF + kH * kH + kH) {
        const int e = g - kH * kF - kH * kH;
        w3r[e] = bf2f(f2bf(master[kOffW3 + e]));
    }
}

// Logits of R samples of n nodes from raw features [R][n][8]: block b takes the samples b,
// b + blocks, ... with the weights in registers.
__global__ __launch_bounds__(1024) void k_mlp_forward(MlpView P, const float *__restrict__ feats, int R, int n,
                                                      float *__restrict__ logits)
{
    __shared__ MlpLds L;
    const MlpRegs W = mlp_load(P, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), threadIdx.x & 63);
    for (int s = blockIdx.x; s < R; s += gridDim.x) {
        mlp_forward_block(P, W, feats + (int64_t)s * n * kF, n, L);
        if (threadIdx.x < n) logits[(int64_t)s * n + threadIdx.x] = L.logit[threadIdx.x];
    }
}

// Per-feature mean and population standard deviation over `rows` rows (FP64,
// fixed reduction trees, so the result does not depend on scheduling); sd
// below 1e-6 is replaced by 1.  Block b of kNormBlocks sums rows b, b + G, ...
// (G = grid threads) per thread, then a tree over its threads; the last
// kernel adds the block sums in block order.
constexpr int kNormBlocks = 256;
constexpr int kNormThreads = 256;
__global__ __launch_bounds__(kNormThreads) void k_feat_norm_part(const float *__restrict__ feats, int64_t rows,
                                                                  double *__restrict__ part)
{
    __shared__ double s1[kF][kNormThreads], s2[kF][kNormThreads];
    double a[kF], b[kF];
#pragma unroll
    for (int k = 0; k < kF; ++k) a[k] = b[k] = 0.0;
    const float4 *f4 = reinterpret_cast<const float4 *>(feats);
    const int64_t stride = (int64_t)gridDim.x * kNormThreads;
    for (int64_t r = (int64_t)blockIdx.x * kNormThreads + threadIdx.x; r < rows; r += stride) {
        const float4 lo = f4[2 * r], hi = f4[2 * r + 1];
        const float v[kF] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
        for (int k = 0; k < kF; ++k) {
            a[k] += (double)v[k];
            b[k] += (double)v[k] * (double)v[k];
        }
    }
#pragma unroll
    for (int k = 0; k < kF; ++k) {
        s1[k][threadIdx.x] = a[k];
        s2[k][threadIdx.x] = b[k];
    }
    __syncthreads();
    for (int w = kNormThreads / 2; w >= 1; w >>= 1) {
        if (threadIdx.x < w)
#pragma unroll
            for (int k = 0; k < kF; ++k) {
                s1[k][threadIdx.x] += s1[k][threadIdx.x + w];
                s2[k][threadIdx.x] += s2[k][threadIdx.x + w];
            }
        __syncthreads();
    }
    if (threadIdx.x < kF) {
        part[(int64_t)blockIdx.x * 2 * kF + threadIdx.x] = s1[threadIdx.x][0];
        part[(int64_t)blockIdx.x * 2 * kF + kF + threadIdx.x] = s2[threadIdx.x][0];
    }
}

__global__ void k_feat_norm_final(const double *__restrict__ part, int blocks, int64_t rows,
                                  float *__restrict__ norm)
{
    const int k = threadIdx.x;
    if (k >= kF) return;
    double t1 = 0.0, t2 = 0.0;
    for (int b = 0; b < blocks; ++b) {
        t1 += part[(int64_t)b * 2 * kF + k];
        t2 += part[(int64_t)b * 2 * kF + kF + k];
    }
    const double mu = rows ? t1 / (double)rows : 0.0;
    const double var = rows ? t2 / (double)rows - mu * mu : 1.0;
    double sd = var > 0 ? sqrt(var) : 0.0;
    if (!(sd > 1e-6)) sd = 1.0;
    norm[k] = (float)mu;
    norm[kF + k] = (float)(1.0 / sd);
}

constexpr int kRP = kRows + 8;       // LDS row pitch of arrays with the nodes along a row (bf16)
constexpr int kFP = kRows + 4;       // and of such a float array
struct alignas(16) GradLds {
    uint16_t z[kRows][16];          // normalised features: hi in columns 0..7, lo in 8..15
    uint16_t zt[16][kRP];           // the same, transposed
    uint16_t h1[2][kRows][kHP];     // relu(layer 1) as hi / lo operands; then dL/dpre2
    uint16_t h1t[2][kH][kRP];       // relu(layer 1), transposed
    uint16_t d2t[2][kH][kRP];       // dL/dpre2, transposed
    float ft[kH][kFP];              // relu(layer 2), transposed; then dL/dpre1
    float part[kRows][8];
    alignas(16) float dl[kRows];
};
static_assert(sizeof(GradLds) <= 160 * 1024, "one block per compute unit");

// Sample index of position j of the epoch's visiting order (affine bijection).
__device__ __forceinline__ int64_t visit(int64_t j, int64_t count, int64_t stride, int64_t offset)
{
    // j < 2^31 and stride < count <= 2^31: the product fits in 64 bits
    return (int64_t)(((uint64_t)j * (uint64_t)stride + (uint64_t)offset) % (uint64_t)count);
}

// Largest value of a wavefront, in every lane.
__device__ __forceinline__ double wave_max_f64(double v)
{
    v = fmax(v, dpp_f64<0xb1>(v));       // lane ^ 1
    v = fmax(v, dpp_f64<0x4e>(v));       // lane ^ 2
    v = fmax(v, dpp_f64<0x141>(v));      // row_half_mirror
    v = fmax(v, dpp_f64<0x140>(v));      // row_mirror
    return fmax(fmax(readlane_f64(v, 0), readlane_f64(v, 16)), fmax(readlane_f64(v, 32), readlane_f64(v, 48)));
}

// op folded over the rows of a column and of the logit gradients, in order from zero, as far as the
// row tiles that hold nodes (a row past the nodes has gradient zero and adds zero); both are read
// 16 rows at a time (one element at a time, every row waited for its own LDS read).
template <typename Op>
__device__ __forceinline__ float rows_in_order(int n, const float *col, const float *dl, Op op)
{
    typedef __attribute__((address_space(3))) const v4f lds4;
    lds4 *pc = (lds4 *)(col), *pd = (lds4 *)(dl);
    asm("" : "+v"(pc), "+v"(pd));       // (else every address is kept across samples, and spills)
    float s = 0.f;
#pragma unroll
    for (int r0 = 0; r0 < kRows; r0 += 16) {
        if (r0 >= n) break;
        v4f c[4], d[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            c[i] = pc[r0 / 4 + i];
            d[i] = pd[r0 / 4 + i];
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) s = op(s, c[i / 4][i % 4], d[i / 4][i % 4]);
    }
    return s;
}

// Block per chunk of `spb` samples: forward, gradient of -ln q(pair) w.r.t.
// the logits, backward through both layers with MFMA GEMMs (the weight
// gradients accumulate in matrix-core accumulators across the chunk), then
// one partial gradient (+ loss sum at index kNParam) per block.  Every
// activation operand is a hi/lo BF16 pair (see mlp_device.h); products of two
// activations take hi*hi + hi*lo + lo*hi.
//
// A chunk is serial and its samples' phases depend on each other, so a sample's latency bounds
// the kernel (about 18,800 cycles at 60 nodes; the matrix cores are busy for 2,600 of
// them): the weights stay in registers for the whole chunk, the next sample's features are
// requested a sample ahead, and every operand is one 16-byte LDS read (activations that the
// gradients contract over the nodes are kept transposed too).  Wavefront w takes 2 x 2 tiles
// of each product (row tiles 2 (w / 4) + i, column tiles 2 (w % 4) + c; 2 x 4 of gW2), which
// halves the LDS reads of one column tile by all rows, and keeps its part of layer 2 and of
// layer 1's relu in registers until their gradients are formed.  The bias and w3 sums run
// over the nodes in order, one column per thread.  60 nodes, 1,024 samples, with the
// reduction: 290 us with operands gathered from row-major arrays and weights read where used,
// 185 us with transposed arrays, 152 us with the row sums read 16 at a time and the weights
// kept, 130 us with 2 x 2 tiles and two values split per conversion (8,192 samples: 1,420,
// 881, 747 and 640 us).
constexpr int kGradWaves = 8;

__global__ __launch_bounds__(kGradWaves * 64) void k_mlp_grad(MlpView P, const float *__restrict__ feats,
                                                   const int32_t *__restrict__ pairs, int64_t count, int64_t first,
                                                   int64_t nsamples, int64_t stride, int64_t offset, int n, int spb,
                                                   double eps, float *__restrict__ part)
{
    __shared__ GradLds G;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, g = lane >> 4;
    const int rp = wave >> 2, cp = wave & 3;
    v4f accW2[2][4];                // gW2 tiles (row tile 2 cp + c, column tile 4 rp + q)
    v4f accW1 = {0.f, 0.f, 0.f, 0.f};
    float gw3 = 0.f, gb2 = 0.f, gb1 = 0.f;      // column tid, tid - 128, tid - 256
    float gb3 = 0.f;
    double loss = 0.0;
    const MlpRegs R[2] = {mlp_load(P, 2 * cp, lane), mlp_load(P, 2 * cp + 1, lane)};
    v4u w2t[2][4];                  // W2^T rows of these column tiles
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            accW2[c][q] = (v4f){0.f, 0.f, 0.f, 0.f};
            w2t[c][q] = ld8(P.W2tb + ((2 * cp + c) * 16 + li) * kH + q * 32 + 8 * g);
        }
    const float w3c = tid < 2 * kH ? P.w3r[tid & (kH - 1)] : 0.f;
    const float b3 = P.b3[0], mu = P.norm[tid % kF], isd = P.norm[kF + tid % kF];
    const int64_t j0 = (int64_t)blockIdx.x * spb;
    const int last = (int)(nsamples - j0 < spb ? nsamples - j0 : spb) - 1;
    // one feature of one node per thread and the pair, requested a sample ahead
    const int fr = tid / kF, fk = tid % kF;
    const int64_t fo = (int64_t)(fr < n ? fr : 0) * kF + fk;
    int64_t smp = visit(first + j0, count, stride, offset);
    float x0 = feats[smp * n * kF + fo];
    int pa0 = pairs[smp * 2], pb0 = pairs[smp * 2 + 1];
    for (int si = 0; si <= last; ++si) {
        {
            float v = 0.f;
            if (fr < n) v = (x0 - mu) * isd;
            uint16_t hi, lo;
            split_bf(v, hi, lo);
            G.z[fr][fk] = hi;
            G.z[fr][kF + fk] = lo;
            G.zt[fk][fr] = hi;
            G.zt[kF + fk][fr] = lo;
        }
        const int a = pa0, b = pb0;
        if (si < last) {                // visit() of the next position
            smp += stride;
            if (smp >= count) smp -= count;
        }
        x0 = feats[smp * n * kF + fo];
        pa0 = pairs[smp * 2];
        pb0 = pairs[smp * 2 + 1];
        __syncthreads();
        // layer 1 (as mlp_forward_block)
        uint32_t on = 0;                // bit 8 i + 4 c + r: this element of layer 1 passed its relu
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int rt = 2 * rp + i;
            v4u a1 = {0u, 0u, 0u, 0u};
            if (g < 2) a1 = ld8(&G.z[rt * 16 + li][8 * g]);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int u = (2 * cp + c) * 16 + li, row = rt * 16 + 4 * g;
                const v4f d = mfma32(a1, R[c].w1, (v4f){0.f, 0.f, 0.f, 0.f});
                float h[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float x = d[r] + R[c].b1;
                    h[r] = x > 0.f ? x : 0.f;
                }
                uint32_t hh[2], hl[2];
                split4_rows(h, &G.h1[0][row][u], &G.h1[1][row][u], hh, hl);
                *reinterpret_cast<uint2 *>(&G.h1t[0][u][row]) = make_uint2(hh[0], hh[1]);
                *reinterpret_cast<uint2 *>(&G.h1t[1][u][row]) = make_uint2(hl[0], hl[1]);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if ((uint16_t)(hh[r >> 1] >> (16 * (r & 1)))) on |= 1u << (8 * i + 4 * c + r);
            }
        }
        __syncthreads();
        // layer 2, its outputs kept in registers too, and the layer-3 dot products
        v4f h2[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int c = 0; c < 2; ++c) h2[i][c] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const v4u x = ld8(&G.h1[s >> 2][(2 * rp + i) * 16 + li][(s & 3) * 32 + 8 * g]);
#pragma unroll
                for (int c = 0; c < 2; ++c) h2[i][c] = mfma32(x, R[c].w2[s & 3], h2[i][c]);
            }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int row = (2 * rp + i) * 16 + 4 * g;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float x = h2[i][c][r] + R[c].b2;
                    h2[i][c][r] = x > 0.f ? x : 0.f;
                    const float q = row_dot_f32(h2[i][c][r], R[c].w3);
                    if (li == 0) G.part[row + r][2 * cp + c] = q;
                }
                *reinterpret_cast<v4f *>(&G.ft[(2 * cp + c) * 16 + li][row]) = h2[i][c];
            }
        __syncthreads();
        // dL/dlogit for L = -ln q({a,b})
        if (wave == 0) {
            float s = b3;
#pragma unroll
            for (int c = 0; c < 8; ++c) s += G.part[lane][c];
            const double l = lane < n ? (double)s : -1e300;
            const double mx = wave_max_f64(l);
            double e = lane < n ? exp(l - mx) : 0.0;
            const double p = e / wave_sum_f64(e);
            const double pa = readlane_f64(p, a & 63), pb = readlane_f64(p, b & 63);
            const double Q = pa * pb * (1.0 / (1.0 - pa) + 1.0 / (1.0 - pb));
            const double q = (1.0 - eps) * Q + eps * 2.0 / ((double)n * (n - 1));
            const double ga = pa * pb * (1.0 / ((1.0 - pa) * (1.0 - pa)) + 1.0 / (1.0 - pb));
            const double gb = pb * pa * (1.0 / ((1.0 - pb) * (1.0 - pb)) + 1.0 / (1.0 - pa));
            double dQ = -p * (ga + gb) + (lane == a ? ga : 0.0) + (lane == b ? gb : 0.0);
            G.dl[lane] = lane < n ? (float)(-(1.0 - eps) * dQ / q) : 0.f;
            loss += -log(q);
        }
        __syncthreads();
        // dL/dpre2 = relu'(pre2) * dl * w3 (hi/lo operands, both ways; h1's rows are done with)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int row = (2 * rp + i) * 16 + 4 * g;
            const v4f dl = *reinterpret_cast<const v4f *>(&G.dl[row]);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int u = (2 * cp + c) * 16 + li;
                float d[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) d[r] = h2[i][c][r] > 0.f ? dl[r] * R[c].w3 : 0.f;
                uint32_t dh[2], dlo[2];
                split4_rows(d, &G.h1[0][row][u], &G.h1[1][row][u], dh, dlo);
                *reinterpret_cast<uint2 *>(&G.d2t[0][u][row]) = make_uint2(dh[0], dh[1]);
                *reinterpret_cast<uint2 *>(&G.d2t[1][u][row]) = make_uint2(dlo[0], dlo[1]);
            }
        }
        // w3 / layer-2 bias / b3 gradients (rows in order)
        if (tid < kH) {
            gw3 += rows_in_order(n, &G.ft[tid][0], &G.dl[0], [](float s, float h, float d) { return fmaf(d, h, s); });
        } else if (tid < 2 * kH) {
            gb2 += rows_in_order(n, &G.ft[tid - kH][0], &G.dl[0],
                                 [w3c](float s, float h, float d) { return s + (h > 0.f ? d * w3c : 0.f); });
        } else if (tid == 2 * kH) {
            gb3 += rows_in_order(n, &G.dl[0], &G.dl[0], [](float s, float, float d) { return s + d; });
        }
        __syncthreads();
        // gW2[u][k] += sum_r d2[r][u] h1[r][k]: A[u][r] = d2, B[r][k] = h1, K = 64 rows in two
        // steps of 32, for the products (d2 hi, h1 hi), (d2 hi, h1 lo), (d2 lo, h1 hi)
        {
            v4u x[2][2][2];
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int pd = 0; pd < 2; ++pd)
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks) x[c][pd][ks] = ld8(&G.d2t[pd][(2 * cp + c) * 16 + li][ks * 32 + 8 * g]);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v4u y[2][2];
#pragma unroll
                for (int ph = 0; ph < 2; ++ph)
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks) y[ph][ks] = ld8(&G.h1t[ph][(4 * rp + q) * 16 + li][ks * 32 + 8 * g]);
#pragma unroll
                for (int pr = 0; pr < 3; ++pr)
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                        for (int c = 0; c < 2; ++c) accW2[c][q] = mfma32(x[c][pr == 2][ks], y[pr == 1][ks], accW2[c][q]);
                __builtin_amdgcn_sched_barrier(0);    // (with every read moved to the front, registers spill)
            }
        }
        // dh1[r][k] = sum_u d2[r][u] W2[u][k] (K = 128, hi then lo); dpre1 = relu'(pre1) dh1
        {
            v4f d[2][2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int c = 0; c < 2; ++c) d[i][c] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < 8; ++s)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const v4u x = ld8(&G.h1[s >> 2][(2 * rp + i) * 16 + li][(s & 3) * 32 + 8 * g]);
#pragma unroll
                    for (int c = 0; c < 2; ++c) d[i][c] = mfma32(x, w2t[c][s & 3], d[i][c]);
                }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const int row = (2 * rp + i) * 16 + 4 * g;
                    v4f v;
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] = (row + r < n && (on >> (8 * i + 4 * c + r) & 1u)) ? d[i][c][r] : 0.f;
                    *reinterpret_cast<v4f *>(&G.ft[(2 * cp + c) * 16 + li][row]) = v;
                }
        }
        __syncthreads();
        // gW1[u][k] += sum_r dpre1[r][u] z[r][k]: A[u][r] = dpre1 (hi, then lo), B[r][c] = the
        // z row (columns 0..7 hi, 8..15 lo); columns c and c + 8 are added at the end, so the
        // tile sums hi*hi + hi*lo + lo*hi + lo*lo (8 tiles of 16 hidden units)
        {
            v4u x[2][2];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const v4f e = *reinterpret_cast<const v4f *>(&G.ft[wave * 16 + li][ks * 32 + 8 * g]);
                const v4f f = *reinterpret_cast<const v4f *>(&G.ft[wave * 16 + li][ks * 32 + 8 * g + 4]);
                uint32_t h[4], l[4];
                split2_bf(e[0], e[1], h[0], l[0]);
                split2_bf(e[2], e[3], h[1], l[1]);
                split2_bf(f[0], f[1], h[2], l[2]);
                split2_bf(f[2], f[3], h[3], l[3]);
                x[0][ks] = (v4u){h[0], h[1], h[2], h[3]};
                x[1][ks] = (v4u){l[0], l[1], l[2], l[3]};
            }
#pragma unroll
            for (int s = 0; s < 4; ++s) accW1 = mfma32(x[s >> 1][s & 1], ld8(&G.zt[li][(s & 1) * 32 + 8 * g]), accW1);
        }
        if (tid >= 2 * kH && tid < 3 * kH) {
            gb1 += rows_in_order(n, &G.ft[tid - 2 * kH][0], &G.dl[0], [](float s, float x, float) { return s + x; });
        }
        __syncthreads();
    }
    // partial gradient of this block
    float *out = part + (int64_t)blockIdx.x * (kNParam + 1);
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                out[kOffW2 + ((2 * cp + c) * 16 + 4 * g + r) * kH + (4 * rp + q) * 16 + li] = accW2[c][q][r];
    {
        // column li + 8 holds the products with z_lo of column li
        float hi8[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) hi8[r] = __shfl(accW1[r], (lane & ~15) | ((li + 8) & 15), 64);
        if (li < kF)
#pragma unroll
            for (int r = 0; r < 4; ++r) out[kOffW1 + (wave * 16 + 4 * g + r) * kF + li] = accW1[r] + hi8[r];
    }
    if (tid < kH) out[kOffW3 + tid] = gw3;
    else if (tid < 2 * kH) out[kOffB2 + tid - kH] = gb2;
    else if (tid < 3 * kH) out[kOffB1 + tid - 2 * kH] = gb1;
    if (tid == 2 * kH) out[kOffB3] = gb3;
    if (tid == 0) out[kNParam] = (float)loss;
}

// Sum of one parameter's partials over the blocks, in block order (FP64), 16 loads in flight.
__device__ __forceinline__ double partial_sum(const float *__restrict__ part, int blocks, int p)
{
    double s = 0.0;
    int b = 0;
    for (; b + 16 <= blocks; b += 16) {
        float v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = part[(int64_t)(b + i) * (kNParam + 1) + p];
#pragma unroll
        for (int i = 0; i < 16; ++i) s += v[i];
    }
    for (; b < blocks; ++b) s += part[(int64_t)b * (kNParam + 1) + p];
    return s;
}

// grad[p] = (sum over blocks, in block order) / count; loss likewise.
__global__ void k_grad_reduce(const float *__restrict__ part, int blocks, double inv, float *__restrict__ grad,
                              double *__restrict__ loss)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p > kNParam) return;
    const double s = partial_sum(part, blocks, p);
    if (p < kNParam) grad[p] = (float)(s * inv);
    else if (loss) *loss = s * inv;
}

// One training step after the partials: the gradient as k_grad_reduce forms it, Adam (Kingma & Ba
// 2015) on the FP32 master weights, and the BF16 copies as k_mlp_refresh makes them.  Bound by the
// latency of the partials' reads: 6 us for 128 blocks, where the three kernels took 30 us.
__global__ void k_train_step(const float *__restrict__ part, int blocks, double inv, float *__restrict__ loss_slot,
                             float *__restrict__ w, float *__restrict__ m, float *__restrict__ v, float lr, float b1,
                             float b2, float eps, float c1, float c2, uint16_t *__restrict__ W1b,
                             uint16_t *__restrict__ W2b, uint16_t *__restrict__ W2tb, float *__restrict__ w3r)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p > kNParam) return;
    const double s = partial_sum(part, blocks, p);
    if (p == kNParam) {
        if (loss_slot) *loss_slot = (float)(s * inv);
        return;
    }
    const float gp = (float)(s * inv);
    const float mp = b1 * m[p] + (1.f - b1) * gp;
    const float vp = b2 * v[p] + (1.f - b2) * gp * gp;
    m[p] = mp;
    v[p] = vp;
    const float x = w[p] - lr * (mp / c1) / (sqrtf(vp / c2) + eps);
    w[p] = x;
    if (p < kOffB1) {
        W1b[p] = f2bf(x);
    } else if (p >= kOffW2 && p < kOffB2) {
        const int e = p - kOffW2;
        const uint16_t b = f2bf(x);
        W2b[e] = b;
        W2tb[(e % kH) * kH + e / kH] = b;
    } else if (p >= kOffW3 && p < kOffB3) {
        w3r[p - kOffW3] = bf2f(f2bf(x));
    }
}

static void refresh(MlpT *m, hipStream_t st)
{
    const int total = kH * kF + kH * kH + kH;
    hipLaunchKernelGGL(k_mlp_refresh, dim3((total + 255) / 256), dim3(256), 0, st, m->d_master, m->d_W1b,
                       m->d_W2b, m->d_W2tb, m->d_w3r);
}

static void free_mlp(MlpT *m)
{
    hipFree(m->d_master);
    hipFree(m->d_m);
    hipFree(m->d_v);
    hipFree(m->d_W1b);
    hipFree(m->d_W2b);
    hipFree(m->d_W2tb);
    hipFree(m->d_w3r);
    hipFree(m->d_norm);
    hipFree(m->d_normpart);
}

constexpr int kSamplesPerBlock = 8;
static int grad_blocks(int64_t nsamples) { return (int)((nsamples + kSamplesPerBlock - 1) / kSamplesPerBlock); }

// The blocks' partial gradients of samples first .. first + nsamples of an epoch's order.
static bnos_status launch_grad(MlpT *m, const float *feats, const int32_t *pairs, int64_t count, int64_t first,
                               int64_t nsamples, int64_t stride, int64_t offset, int n, double eps, float *part,
                               hipStream_t st)
{
    hipLaunchKernelGGL(k_mlp_grad, dim3(grad_blocks(nsamples)), dim3(kGradWaves * 64), 0, st, mlp_view(m), feats, pairs,
                       count, first, nsamples, stride, offset, n, kSamplesPerBlock, eps, part);
    BNOS_HIP(hipGetLastError());
    return BNOS_OK;
}

}  // namespace bnos

using namespace bnos;

extern "C" bnos_status bnos_mlp_create(bnos_mlp *out)
{
    if (!out) { set_error("out is NULL"); return BNOS_E_INVALID; }
    MlpT *m = new (std::nothrow) MlpT();
    if (!m) { set_error("host allocation failed"); return BNOS_E_NOMEM; }
    hipError_t e;
    if ((e = hipGetDevice(&m->device)) != hipSuccess) { delete m; set_error(hipGetErrorString(e)); return BNOS_E_DEVICE; }
#define ALLOC(p, bytes) if ((e = hipMalloc((void **)&(p), (bytes))) != hipSuccess) { free_mlp(m); delete m; set_error(std::string("hipMalloc: ") + hipGetErrorString(e)); return e == hipErrorOutOfMemory ? BNOS_E_NOMEM : BNOS_E_DEVICE; }
    ALLOC(m->d_master, sizeof(float) * kNParam);
    ALLOC(m->d_m, sizeof(float) * kNParam);
    ALLOC(m->d_v, sizeof(float) * kNParam);
    ALLOC(m->d_W1b, sizeof(uint16_t) * kH * kF);
    ALLOC(m->d_W2b, sizeof(uint16_t) * kH * kH);
    ALLOC(m->d_W2tb, sizeof(uint16_t) * kH * kH);
    ALLOC(m->d_normpart, sizeof(double) * kNormBlocks * 2 * kF);
    ALLOC(m->d_w3r, sizeof(float) * kH);
    ALLOC(m->d_norm, sizeof(float) * 2 * kF);
#undef ALLOC
    std::vector<float> zero(kNParam, 0.f);
    float norm[2 * kF];
    for (int k = 0; k < kF; ++k) {
        m->h_mu[k] = 0.f;
        m->h_sd[k] = 1.f;
        norm[k] = 0.f;
        norm[kF + k] = 1.f;
    }
    bool ok = hipMemcpy(m->d_master, zero.data(), sizeof(float) * kNParam, hipMemcpyHostToDevice) == hipSuccess &&
              hipMemcpy(m->d_m, zero.data(), sizeof(float) * kNParam, hipMemcpyHostToDevice) == hipSuccess &&
              hipMemcpy(m->d_v, zero.data(), sizeof(float) * kNParam, hipMemcpyHostToDevice) == hipSuccess &&
              hipMemcpy(m->d_norm, norm, sizeof norm, hipMemcpyHostToDevice) == hipSuccess;
    if (!ok) { free_mlp(m); delete m; set_error("hipMemcpy failed"); return BNOS_E_DEVICE; }
    refresh(m, nullptr);
    if (hipDeviceSynchronize() != hipSuccess) { free_mlp(m); delete m; set_error("refresh failed"); return BNOS_E_DEVICE; }
    m->magic = kMlpMagic;
    {
        std::lock_guard<std::mutex> lk(g_mlp_mu);
        g_mlps.insert(m);
    }
    *out = reinterpret_cast<bnos_mlp>(m);
    return BNOS_OK;
}

extern "C" void bnos_mlp_free(bnos_mlp h)
{
    MlpT *m = reinterpret_cast<MlpT *>(h);
    if (!mlp_live(m)) return;
    {
        std::lock_guard<std::mutex> lk(g_mlp_mu);
        g_mlps.erase(m);
    }
    hipDeviceSynchronize();
    m->magic = 0;
    free_mlp(m);
    delete m;
}

extern "C" bnos_status bnos_mlp_set_params(bnos_mlp h, const float *params, const float *mu, const float *sd)
{
    MlpT *m = reinterpret_cast<MlpT *>(h);
    if (!mlp_live(m)) { set_error("invalid network handle"); return BNOS_E_STATE; }
    if (params)
        for (int p = 0; p < kNParam; ++p)
            if (!std::isfinite(params[p])) { set_error("non-finite parameter"); return BNOS_E_INVALID; }
    if ((mu && !sd) || (!mu && sd)) { set_error("mu and sd go together"); return BNOS_E_INVALID; }
    if (sd)
        for (int k = 0; k < kF; ++k)
            if (!(sd[k] > 0.f) || !std::isfinite(sd[k]) || !std::isfinite(mu[k])) { set_error("sd must be > 0, finite"); return BNOS_E_INVALID; }
    BNOS_HIP(hipSetDevice(m->device));
    if (params) {
        std::vector<float> zero(kNParam, 0.f);
        BNOS_HIP(hipMemcpy(m->d_master, params, sizeof(float) * kNParam, hipMemcpyHostToDevice));
        BNOS_HIP(hipMemcpy(m->d_m, zero.data(), sizeof(float) * kNParam, hipMemcpyHostToDevice));
        BNOS_HIP(hipMemcpy(m->d_v, zero.data(), sizeof(float) * kNParam, hipMemcpyHostToDevice));
        m->adam_t = 0;
        refresh(m, nullptr);
        BNOS_HIP(hipGetLastError());
    }
    if (mu) {
        float norm[2 * kF];
        for (int k = 0; k < kF; ++k) {
            m->h_mu[k] = mu[k];
            m->h_sd[k] = sd[k];
            norm[k] = mu[k];
            norm[kF + k] = 1.f / sd[k];
        }
        BNOS_HIP(hipMemcpy(m->d_norm, norm, sizeof norm, hipMemcpyHostToDevice));
    }
    BNOS_HIP(hipDeviceSynchronize());
    return BNOS_OK;
}

extern "C" bnos_status bnos_mlp_get_params(bnos_mlp h, float *params, float *mu, float *sd)
{
    MlpT *m = reinterpret_cast<MlpT *>(h);
    if (!mlp_live(m)) { set_error("invalid network handle"); return BNOS_E_STATE; }
    BNOS_HIP(hipSetDevice(m->device));
    BNOS_HIP(hipDeviceSynchronize());
    if (params) BNOS_HIP(hipMemcpy(params, m->d_master, sizeof(float) * kNParam, hipMemcpyDeviceToHost));
    if (mu || sd) {
        float norm[2 * kF];
        BNOS_HIP(hipMemcpy(norm, m->d_norm, sizeof norm, hipMemcpyDeviceToHost));
        for (int k = 0; k < kF; ++k) {
            if (mu) mu[k] = norm[k];
            if (sd) sd[k] = 1.f / norm[kF + k];
        }
    }
    return BNOS_OK;
}

extern "C" bnos_status bnos_mlp_fit_norm(bnos_mlp h, const float *feats, int64_t rows, void *stream)
{
    MlpT *m = reinterpret_cast<MlpT *>(h);
    if (!mlp_live(m)) { set_error("invalid network handle"); return BNOS_E_STATE; }
    if (!feats || rows < 1) { set_error("need at least one feature row"); return BNOS_E_INVALID; }
    if (reinterpret_cast<uintptr_t>(feats) % 16) { set_error("feats must be 16-byte aligned"); return BNOS_E_INVALID; }
    BNOS_HIP(hipSetDevice(m->device));
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    int64_t want = (rows + kNormThreads - 1) / kNormThreads;
    const int blocks = (int)(want < kNormBlocks ? want : kNormBlocks);
    hipLaunchKernelGGL(k_feat_norm_part, dim3(blocks), dim3(kNormThreads), 0, st, feats, rows, m->d_normpart);
    BNOS_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_feat_norm_final, dim3(1), dim3(64), 0, st, m->d_normpart, blocks, rows, m->d_norm);
    BNOS_HIP(hipGetLastError());
    return BNOS_OK;
}

extern "C" bnos_status bnos_mlp_forward(bnos_mlp h, const float *feats, int32_t R, int32_t n, float *logits,
                                        void *stream)
{
    MlpT *m = reinterpret_cast<MlpT *>(h);
    if (!mlp_live(m)) { set_error("invalid network handle"); return BNOS_E_STATE; }
    if (!feats || !logits) { set_error("NULL argument"); return BNOS_E_INVALID; }
    if (R < 1 || n < 2 || n > 64) { set_error("need R >= 1 and 2 <= n <= 64"); return BNOS_E_RANGE; }
    BNOS_HIP(hipSetDevice(m->device));
    hipLaunchKernelGGL(k_mlp_forward, dim3(R < 512 ? R : 512), dim3(1024), 0, reinterpret_cast<hipStream_t>(stream),
                       mlp_view(m), feats, R, n, logits);
    BNOS_HIP(hipGetLastError());
    return BNOS_OK;
}

extern "C" bnos_status bnos_mlp_grad(bnos_mlp h, const float *feats, const int32_t *pairs, int32_t R, int32_t n,
                                     float eps, float *grad, double *loss, void *stream)
{
    MlpT *m = reinterpret_cast<MlpT *>(h);
    if (!mlp_live(m)) { set_error("invalid network handle"); return BNOS_E_STATE; }
    if (!feats || !pairs || !grad) { set_error("NULL argument"); return BNOS_E_INVALID; }
    if (R < 1 || n < 2 || n > 64) { set_error("need R >= 1 and 2 <= n <= 64"); return BNOS_E_RANGE; }
    if (!(eps >= 0.f && eps <= 1.f)) { set_error("eps outside [0, 1]"); return BNOS_E_RANGE; }
    BNOS_HIP(hipSetDevice(m->device));
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    const int blocks = grad_blocks(R);
    float *part = nullptr;
    BNOS_HIP(hipMalloc((void **)&part, sizeof(float) * (size_t)blocks * (kNParam + 1)));
    bnos_status s = launch_grad(m, feats, pairs, R, 0, R, 1, 0, n, eps, part, st);
    if (s == BNOS_OK) {
        hipLaunchKernelGGL(k_grad_reduce, dim3((kNParam + 1 + 255) / 256), dim3(256), 0, st, part, blocks,
                           1.0 / (double)R, grad, loss);
        if (hipGetLastError() != hipSuccess) { s = BNOS_E_DEVICE; set_error("gradient launch failed"); }
    }
    hipError_t e = hipStreamSynchronize(st);
    hipFree(part);
    if (s != BNOS_OK) return s;
    if (e != hipSuccess) { set_error(hipGetErrorString(e)); return BNOS_E_DEVICE; }
    return BNOS_OK;
}

static uint64_t host_mix(uint64_t z)
{
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

static int64_t gcd64(int64_t a, int64_t b)
{
    while (b) {
        int64_t t = a % b;
        a = b;
        b = t;
    }
    return a;
}

extern "C" bnos_status bnos_mlp_train(bnos_mlp h, const float *feats, const int32_t *pairs, int64_t count, int32_t n,
                                      float eps, int32_t epochs, int32_t batch, float lr, uint64_t seed,
                                      float *loss_trace, void *stream)
{
    MlpT *m = reinterpret_cast<MlpT *>(h);
    if (!mlp_live(m)) { set_error("invalid network handle"); return BNOS_E_STATE; }
    if (!feats || !pairs) { set_error("NULL argument"); return BNOS_E_INVALID; }
    if (count < 1 || n < 2 || n > 64 || epochs < 0 || batch < 1) { set_error("bad sizes"); return BNOS_E_RANGE; }
    if (!(eps >= 0.f && eps <= 1.f) || !(lr > 0.f)) { set_error("bad eps or lr"); return BNOS_E_RANGE; }
    BNOS_HIP(hipSetDevice(m->device));
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    const int64_t bsz = batch < count ? batch : count;
    float *part = nullptr;
    BNOS_HIP(hipMalloc((void **)&part, sizeof(float) * (size_t)grad_blocks(bsz) * (kNParam + 1)));
    const int64_t steps_per_epoch = (count + bsz - 1) / bsz;
    int64_t step = 0;
    bnos_status s = BNOS_OK;
    for (int ep = 0; ep < epochs && s == BNOS_OK; ++ep) {
        // visiting order of this epoch: j -> (offset + j * stride) mod count, stride coprime to count
        uint64_t r = host_mix(seed ^ host_mix(0x5EEDull + (uint64_t)ep));
        int64_t stride = 1 + (int64_t)(r % (uint64_t)count);
        while (gcd64(stride, count) != 1) stride = stride % count + 1;
        const int64_t offset = (int64_t)(host_mix(r) % (uint64_t)count);
        for (int64_t b = 0; b < steps_per_epoch && s == BNOS_OK; ++b) {
            const int64_t first = b * bsz;
            const int64_t ns = (first + bsz <= count) ? bsz : count - first;
            s = launch_grad(m, feats, pairs, count, first, ns, stride, offset, n, eps, part, st);
            if (s != BNOS_OK) break;
            ++m->adam_t;
            const float b1 = 0.9f, b2 = 0.999f;
            const float c1 = 1.f - powf(b1, (float)m->adam_t), c2 = 1.f - powf(b2, (float)m->adam_t);
            hipLaunchKernelGGL(k_train_step, dim3((kNParam + 1 + 127) / 128), dim3(128), 0, st, part, grad_blocks(ns),
                               1.0 / (double)ns, loss_trace ? loss_trace + step : nullptr, m->d_master, m->d_m, m->d_v,
                               lr, b1, b2, 1e-8f, c1, c2, m->d_W1b, m->d_W2b, m->d_W2tb, m->d_w3r);
            if (hipGetLastError() != hipSuccess) { s = BNOS_E_DEVICE; set_error("training launch failed"); }
            ++step;
        }
    }
    hipError_t e = hipStreamSynchronize(st);
    hipFree(part);
    if (s != BNOS_OK) return s;
    if (e != hipSuccess) { set_error(hipGetErrorString(e)); return BNOS_E_DEVICE; }
    return BNOS_OK;
}
