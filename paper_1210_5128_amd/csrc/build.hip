// Local-score table build on the device: data ingest, parent-set
// enumeration, contingency counting in LDS and the BDeu + pairwise-prior
// score (Sec. II Eq. (3); Sec. III.A Eq. (4); Sec. IV Eq. (9)-(10)).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <set>
#include <string>
#include <vector>

#include "bnos_internal.h"

namespace bnos {

// ------------------------------------------------------------------ errors, handles

static thread_local std::string g_err;
static std::mutex g_handles_mu;
static std::set<const TableT *> g_handles;

void set_error(const std::string &msg) { g_err = msg; }

bool handle_live(const TableT *t)
{
    std::lock_guard<std::mutex> lk(g_handles_mu);
    return t && g_handles.count(t) && t->magic == kMagic;
}

void register_handle(TableT *t)
{
    std::lock_guard<std::mutex> lk(g_handles_mu);
    g_handles.insert(t);
}

bool unregister_handle(TableT *t)
{
    std::lock_guard<std::mutex> lk(g_handles_mu);
    g_handles.erase(t);
    return g_handles.empty();
}

int64_t TableT::device_bytes() const
{
    return (int64_t)n * S_pad * (int64_t)(sizeof(uint64_t) + sizeof(float)) + (int64_t)n * N_pad +
           (int64_t)n * (int64_t)(sizeof(int32_t) + n * sizeof(double) + 5 * sizeof(double)) + 64 * 8 * 8 +
           part_bytes + kpart_bytes + (int64_t)n * (S_pad / 256) * 8 + (int64_t)n * (S_pad / 64) * 8 +
           (int64_t)n * (S_pad / 4) * 8 + (int64_t)n * (S_pad / 256) * 4 + (int64_t)n * kBoundSlots * 12 +
           (d_kmask ? kept_bytes() : 0);
}

// ------------------------------------------------------------------ device helpers

// Orders LDS traffic of one wavefront between phases (zero / count / read).
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
}

// Mask over the n-1 candidate slots -> mask over node ids: a zero bit is
// inserted at position `node` (slot s < node is node s, slot s >= node is s+1).
__device__ __forceinline__ uint64_t slot_to_node_mask(uint64_t m, int node)
{
    uint64_t lo = m & ((1ull << node) - 1ull);
    uint64_t hi = (node >= 63) ? 0ull : ((m >> node) << (node + 1));
    return hi | lo;
}

// The e-th mask, in ascending numeric order, among masks over `bits` bits with
// at most K set bits.  nsets[b*8 + k] = number of masks over b bits with <= k
// set bits; the masks whose top bit is clear come first.
__device__ __forceinline__ uint64_t unrank_ascending(int64_t e, int bits, int K,
                                                      const int64_t *__restrict__ nsets)
{
    uint64_t m = 0;
    int k = K;
    for (int b = bits - 1; b >= 0 && k > 0; --b) {
        int64_t c = nsets[b * 8 + k];
        if (e >= c) {
            m |= 1ull << b;
            e -= c;
            --k;
        }
    }
    return m;
}

__device__ __forceinline__ double wave_sum_f64(double v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Parent members of a node mask, ascending, with the cell weights of the
// counting layout: cell = x_child + r_child * sum_t x_{m_t} * prod_{t'>t} r_{m_t'}.
struct Members {
    int id[kMaxK];
    int w[kMaxK];
    int cnt;
    int q;
};

__device__ __forceinline__ Members decode_members(uint64_t mask, int r_child,
                                                  const int32_t *__restrict__ ar)
{
    Members M;
    M.cnt = 0;
    uint64_t m = mask;
#pragma unroll
    for (int t = 0; t < kMaxK; ++t) {
        M.id[t] = 0;
        M.w[t] = 0;
        if (m) {
            int b = __builtin_ctzll(m);
            m &= m - 1;
            M.id[t] = b;
            M.cnt = t + 1;
        }
    }
    int acc = r_child;
#pragma unroll
    for (int t = kMaxK - 1; t >= 0; --t) {
        if (t < M.cnt) {
            M.w[t] = acc;
            acc *= ar[M.id[t]];
        }
    }
    M.q = acc / r_child;
    return M;
}

// Histogram of the N samples into hist[0 .. q*r) (one wavefront; hist is this
// wavefront's private LDS region).  Each lane takes 4 consecutive samples per
// step from 32-bit loads of the column-major data.
__device__ __forceinline__ void wave_count(const uint8_t *__restrict__ data, int64_t N, int64_t N_pad,
                                           int child, const Members &M, int cells, uint32_t *hist,
                                           int lane)
{
    for (int c = lane; c < cells; c += 64) hist[c] = 0u;
    wave_lds_sync();
    const uint32_t *colc = reinterpret_cast<const uint32_t *>(data + (int64_t)child * N_pad);
    const uint32_t *colm[kMaxK];
#pragma unroll
    for (int t = 0; t < kMaxK; ++t)
        colm[t] = reinterpret_cast<const uint32_t *>(data + (int64_t)M.id[t] * N_pad);
    for (int64_t base = (int64_t)lane * 4; base < N; base += 256) {
        uint32_t xc = colc[base >> 2];
        uint32_t xm[kMaxK];
#pragma unroll
        for (int t = 0; t < kMaxK; ++t) xm[t] = (t < M.cnt) ? colm[t][base >> 2] : 0u;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            int cell = (int)((xc >> (8 * b)) & 0xffu);
#pragma unroll
            for (int t = 0; t < kMaxK; ++t) cell += M.w[t] * (int)((xm[t] >> (8 * b)) & 0xffu);
            if (base + b < N) atomicAdd(&hist[cell], 1u);
        }
    }
    wave_lds_sync();
}

// ------------------------------------------------------------------ kernels

// Row-major int8 [N][n] -> column-major uint8 [n][N_pad] (padding already zero).
__global__ void k_ingest(const int8_t *__restrict__ src, int64_t N, int n, int64_t N_pad,
                         uint8_t *__restrict__ dst)
{
    int64_t total = N * n;
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < total;
         g += (int64_t)gridDim.x * blockDim.x) {
        int64_t t = g / n;
        int v = (int)(g - t * n);
        dst[(int64_t)v * N_pad + t] = (uint8_t)src[g];
    }
}

// Device-resident input: counts the states outside [0, arity) (the host input
// is checked on the host instead).
__global__ void k_check_states(const int8_t *__restrict__ src, int64_t N, int n, const int32_t *__restrict__ ar,
                               unsigned *__restrict__ bad)
{
    const int64_t total = N * n;
    unsigned c = 0;
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < total;
         g += (int64_t)gridDim.x * blockDim.x) {
        const int x = src[g];
        const int v = (int)(g % n);
        c += (x < 0 || x >= ar[v]) ? 1u : 0u;
    }
    if (c) atomicAdd(bad, c);
}

// Prior term in nats per (child i, parent m): ln(10) * 100 * (R - 0.5)^3 (Eq. (10),
// a log10 quantity in Eq. (9)); R = (1 + w)/2 in mode 0, R given in mode 1.
__global__ void k_prior(const float *__restrict__ src, int n, int mode, double *__restrict__ dst)
{
    int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n * n) return;
    int i = g / n, m = g - (g / n) * n;
    double v = 0.0;
    if (src && i != m) {
        double x = (double)src[g];
        double R = (mode == 0) ? 0.5 * (1.0 + x) : x;
        double d = R - 0.5;
        v = 2.302585092994045684 * 100.0 * d * d * d;
    }
    dst[g] = v;
}

// lut[row][c] = lnG(c + a) - lnG(a), a = ess / den[row], c = 0..N (FP64 ocml lgamma); with
// scale > 0 as 64-bit integers, the nearest to scale times that (see lut_scale).
__global__ void k_lut(const int32_t *__restrict__ den, int rows, int64_t N, double ess, double scale,
                      double *__restrict__ lut)
{
    const int64_t total = (int64_t)rows * (N + 1);
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < total; g += (int64_t)gridDim.x * blockDim.x) {
        const int row = (int)(g / (N + 1));
        const int64_t c = g - (int64_t)row * (N + 1);
        const double a = ess / (double)den[row];
        const double v = lgamma((double)c + a) - lgamma(a);
        lut[g] = scale > 0.0 ? __builtin_bit_cast(double, (int64_t)rint(v * scale)) : v;
    }
}

// Rank of a mask among the masks over `bits` bits with at most K set bits, in
// ascending numeric order (the inverse of unrank_ascending).
__device__ __forceinline__ int64_t rank_ascending(uint64_t m, int bits, int K, const int64_t *__restrict__ nsets)
{
    int64_t r = 0;
    int k = K;
    for (int b = bits - 1; b >= 0; --b)
        if ((m >> b) & 1ull) {
            r += nsets[b * 8 + k];
            --k;
        }
    return r;
}

// A node subset U (|U| <= K+1) as the joint histogram sees it: members
// ascending, their arities, and the stride of each member's digit in the joint
// cell index (the last member fastest).
struct Subset {
    int u[kMaxK + 1], r[kMaxK + 1], stride[kMaxK + 1];
    uint32_t magic[kMaxK + 1];   // floor(2^32 / r) + 1: quotients by r of cell indices (<= 2^14) by multiply-high
    int j;        // members
    int cells;    // product of the members' arities
};

// q = x / r and x - q r for 0 <= x <= 2^14 and 1 <= r <= 255: with m = floor(2^32/r) + 1,
// x m / 2^32 exceeds x / r by less than x / 2^32 <= 2^-18, too little to carry a
// fraction of at most (r - 1) / r past the next integer.  q r <= x fits a 24-bit multiply.
__device__ __forceinline__ void divmod_small(int x, int r, uint32_t magic, int &q, int &rem)
{
    q = (r == 1) ? x : (int)__umulhi((uint32_t)x, magic);
    rem = x - (int)__umul24((uint32_t)q, (uint32_t)r);
}

// (ar: the n arities, then their magic numbers.)
__device__ __forceinline__ Subset decode_subset(uint64_t U, const int32_t *__restrict__ ar, int n)
{
    Subset S;
    S.j = 0;
    uint64_t m = U;
#pragma unroll
    for (int t = 0; t <= kMaxK; ++t) {
        S.u[t] = 0;
        S.r[t] = 1;
        S.magic[t] = 0u;
        if (m) {
            S.u[t] = __builtin_ctzll(m);
            m &= m - 1;
            S.r[t] = ar[S.u[t]];
            S.magic[t] = (uint32_t)ar[n + S.u[t]];
            S.j = t + 1;
        }
    }
    int cells = 1;
#pragma unroll
    for (int t = kMaxK; t >= 0; --t) {
        S.stride[t] = cells;
        if (t < S.j) cells *= S.r[t];
    }
    S.cells = cells;
    return S;
}

// Joint histogram of U's variables over the N samples into hist[0 .. cells)
// (one wavefront, its private LDS region); each lane takes 4 consecutive
// samples per step from 32-bit loads of the column-major data.  A cell's byte
// offset is the sum of each member's state times its stride in bytes: states
// are below 256 and cells number at most 2^14, so every product and the sum
// fit 24-bit multiplies.  Whole 256-sample steps need no per-sample check;
// only the last, partial step tests each sample against N.
// (J = the number of members, a constant of the instance.)
template <int J>
__device__ __forceinline__ void joint_histogram_j(const uint8_t *__restrict__ data, int64_t N, int64_t N_pad,
                                                  const Subset &S, uint32_t *hist, int lane)
{
    const uint32_t *col[J];
    uint32_t st4[J];
#pragma unroll
    for (int t = 0; t < J; ++t) {
        col[t] = reinterpret_cast<const uint32_t *>(data + (int64_t)S.u[t] * N_pad);
        st4[t] = (uint32_t)S.stride[t] * 4u;
    }
    char *hb = reinterpret_cast<char *>(hist);
    auto offset_of = [&](const uint32_t (&x)[J], int b) -> uint32_t {
        uint32_t off = 0;
#pragma unroll
        for (int t = 0; t < J; ++t) off += __umul24((x[t] >> (8 * b)) & 0xffu, st4[t]);
        return off;
    };
    const int64_t whole = N & ~(int64_t)255;
    for (int64_t base = (int64_t)lane * 4; base < whole; base += 256) {
        uint32_t x[J];
#pragma unroll
        for (int t = 0; t < J; ++t) x[t] = col[t][base >> 2];
#pragma unroll
        for (int b = 0; b < 4; ++b) atomicAdd(reinterpret_cast<uint32_t *>(hb + offset_of(x, b)), 1u);
    }
    const int64_t base = whole + (int64_t)lane * 4;
    if (base < N) {
        uint32_t x[J];
#pragma unroll
        for (int t = 0; t < J; ++t) x[t] = col[t][base >> 2];
#pragma unroll
        for (int b = 0; b < 4; ++b)
            if (base + b < N) atomicAdd(reinterpret_cast<uint32_t *>(hb + offset_of(x, b)), 1u);
    }
}

__device__ __forceinline__ void joint_histogram(const uint8_t *__restrict__ data, int64_t N, int64_t N_pad,
                                                const Subset &S, uint32_t *hist, int lane)
{
    for (int c = lane; c < S.cells; c += 64) hist[c] = 0u;
    wave_lds_sync();
    switch (S.j) {                 // uniform: one subset per wavefront
    case 1: joint_histogram_j<1>(data, N, N_pad, S, hist, lane); break;
    case 2: joint_histogram_j<2>(data, N, N_pad, S, hist, lane); break;
    case 3: joint_histogram_j<3>(data, N, N_pad, S, hist, lane); break;
    case 4: joint_histogram_j<4>(data, N, N_pad, S, hist, lane); break;
    case 5: joint_histogram_j<5>(data, N, N_pad, S, hist, lane); break;
    case 6: joint_histogram_j<6>(data, N, N_pad, S, hist, lane); break;
    default: joint_histogram_j<kMaxK + 1>(data, N, N_pad, S, hist, lane); break;
    }
    wave_lds_sync();
}

// Member c of U as the child of the family (u_c, U \ {u_c}): its id, arity,
// digit stride and the family's number of parent configurations (the cells
// divided by the arity), selected without indexing the arrays by c.
__device__ __forceinline__ void subset_member(const Subset &S, int c, int &node, int &ri, int &sci, int &q)
{
    node = 0;
    ri = 1;
    sci = 1;
    uint32_t mag = 0;
#pragma unroll
    for (int t = 0; t <= kMaxK; ++t)
        if (t == c) {
            node = S.u[t];
            ri = S.r[t];
            sci = S.stride[t];
            mag = S.magic[t];
        }
    int rem;
    divmod_small(S.cells, ri, mag, q, rem);
}

// Joint cell of parent configuration k of the family whose child is member c,
// with the child's state 0: k's digits run over the parents ascending, the
// last one fastest (the lowest id most significant, as in the per-family
// count layout); the child's state x adds x * (c's stride).
__device__ __forceinline__ int family_base(const Subset &S, int c, int k)
{
    int rest = k, J = 0;
#pragma unroll
    for (int t = kMaxK; t >= 0; --t) {
        if (t < S.j && t != c) {
            int q, d;
            divmod_small(rest, S.r[t], S.magic[t], q, d);
            J += (int)__umul24((uint32_t)d, (uint32_t)S.stride[t]);
            rest = q;
        }
    }
    return J;
}

// One wavefront per node subset U, |U| = 1 .. K+1 (U's rank + 1 among the
// masks over n bits with at most K+1 bits): the joint histogram of U's
// variables over the N samples, then for every member i of U the local score
// of the family (i, U \ {i}) from it -- that family's N_ijk are the joint
// counts with i's state as the child state -- stored at U \ {i}'s entry of i's
// row.  Counting once per U instead of once per family cuts the sample visits
// by the mean family size (about 5x at K = 4).

// The lookup's terms as integers: the families of U share the sum of the N_ijk terms, which
// depend only on U's cells (alpha_ijk = ess / cells for every child), and each subtracts the
// terms of its own N_ik.  64-bit integers add up to the same total in any order, so the shared
// sum, k_build's order over one family's cells and any lane assignment store the same score,
// bit for bit.  lut_scale picks the unit: a family's sum stays below 2^62 of them, and a term,
// rounded to the nearest, is closer to its FP64 value than FP64 additions of the family's
// terms keep it (n = 60, N = 5,000: units of 2^-45).

// Adds this lane's cells (c, c + 64, ...) of the joint histogram: the N_ijk terms to `all`,
// and to of[t] the N_ik terms of the family whose child is member t, each taken at the cell
// with that member's state 0.  (J = the number of members, a constant of the instance.)
template <int J>
__device__ __forceinline__ void subset_terms_j(const Subset &S, const uint32_t *hist, int lane,
                                               const int32_t *__restrict__ lut_row,
                                               const int64_t *__restrict__ lut, int64_t stride, uint64_t &all,
                                               uint64_t (&of)[kMaxK + 1])
{
    const int64_t *Lijk = lut + lut_row[S.cells] * stride;
    const int64_t *Lik[J];
#pragma unroll
    for (int t = 0; t < J; ++t) {
        int q, rem;
        divmod_small(S.cells, S.r[t], S.magic[t], q, rem);
        Lik[t] = lut + lut_row[q] * stride;
    }
    for (int c = lane; c < S.cells; c += 64) {
        const uint32_t cnt = hist[c];
        all += (uint64_t)Lijk[cnt];
        int rest = c;
#pragma unroll
        for (int t = J - 1; t >= 0; --t) {
            int d = rest;
            if (t > 0) {
                int q;
                divmod_small(rest, S.r[t], S.magic[t], q, d);
                rest = q;
            }
            if (d == 0) {
                uint32_t nik = cnt;
                for (int x = 1, at = c + S.stride[t]; x < S.r[t]; ++x, at += S.stride[t]) nik += hist[at];
                of[t] += (uint64_t)Lik[t][nik];
            }
        }
    }
}

// What bounded it: scalar instructions.  The families' ranks were looked up bit by bit over 59
// slots, U unranked over 60 nodes, seven 64-bit divisions formed the magic numbers, for every
// subset, and every family summed the N_ijk terms again: 56 ms at n = 60 for 200 samples and for
// 5,000 alike.  A wavefront now takes `run` consecutive subsets, each the successor of the one
// before, lane t finishes the family of member t, and what is left is the histogram.
template <int WAVES>
__global__ __launch_bounds__(WAVES * 64) void k_build_joint(
    const uint8_t *__restrict__ data, int64_t N, int64_t N_pad, const int32_t *__restrict__ ar,
    const double *__restrict__ prior, const int64_t *__restrict__ nsets, int n, int K, double unit,
    double log_gamma, int64_t n_subsets, int run, int64_t S_pad, int cells_cap, const int32_t *__restrict__ lut_row,
    const int64_t *__restrict__ lut, uint64_t *__restrict__ masks, float *__restrict__ scores)
{
    extern __shared__ uint32_t lds_hist[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // uniform: the subset's decode stays scalar
    const int lane = threadIdx.x & 63;
    uint32_t *hist = lds_hist + wave * cells_cap;
    const int64_t g0 = ((int64_t)blockIdx.x * WAVES + wave) * run;
    if (g0 >= n_subsets) return;
    uint64_t U = unrank_ascending(g0 + 1, n, K + 1, nsets);
    for (int64_t g = g0; g < g0 + run && g < n_subsets; ++g) {
        const Subset Sb = decode_subset(U, ar, n);
        joint_histogram(data, N, N_pad, Sb, hist, lane);
        uint64_t all = 0ull, of[kMaxK + 1];
#pragma unroll
        for (int t = 0; t <= kMaxK; ++t) of[t] = 0ull;
        switch (Sb.j) {                // uniform
        case 1: subset_terms_j<1>(Sb, hist, lane, lut_row, lut, N + 1, all, of); break;
        case 2: subset_terms_j<2>(Sb, hist, lane, lut_row, lut, N + 1, all, of); break;
        case 3: subset_terms_j<3>(Sb, hist, lane, lut_row, lut, N + 1, all, of); break;
        case 4: subset_terms_j<4>(Sb, hist, lane, lut_row, lut, N + 1, all, of); break;
        case 5: subset_terms_j<5>(Sb, hist, lane, lut_row, lut, N + 1, all, of); break;
        case 6: subset_terms_j<6>(Sb, hist, lane, lut_row, lut, N + 1, all, of); break;
        default: subset_terms_j<kMaxK + 1>(Sb, hist, lane, lut_row, lut, N + 1, all, of); break;
        }
        all = wave_sum_u64(all);
        uint64_t sum = 0ull;           // lane t: the family of member t
        int node = 0;
#pragma unroll
        for (int t = 0; t <= kMaxK; ++t)
            if (t < Sb.j) {            // uniform
                const uint64_t o = wave_sum_u64(of[t]);
                sum = lane == t ? all - o : sum;
                node = lane == t ? Sb.u[t] : node;
            }
        if (lane < Sb.j) {
            double sc = fma((double)(Sb.j - 1), log_gamma, (double)(int64_t)sum * unit);   // unit: a power of two
            // the rank of U without the node: its members from the highest down, at places
            // K, K - 1, ..., those above the node one slot lower
            int64_t e = (int64_t)node * S_pad;
#pragma unroll
            for (int t = 0; t <= kMaxK; ++t)
                if (t < Sb.j && t != lane) {
                    sc += prior[(int64_t)node * n + Sb.u[t]];
                    const int above = Sb.j - 1 - t - (lane > t ? 1 : 0), slot = Sb.u[t] - (lane < t ? 1 : 0);
                    e += nsets[slot * 8 + (K - above)];
                }
            masks[e] = U & ~(1ull << node);
            scores[e] = (float)sc;     // round to nearest even
        }
        wave_lds_sync();   // every lane has read hist before the next subset clears it
        U += (__popcll(U) <= K) ? 1ull : (U & (0ull - U));   // the next mask of at most K + 1 members
    }
}

// The same with FP64 terms, a family after the other (where no integer unit serves: see
// lut_scale): the BDeu terms are summed in the same order as in k_build (parent configurations k
// by lane, the lowest id most significant; child states in order; the same butterfly), so the
// stored scores are the same, bit for bit.
template <int WAVES>
__global__ __launch_bounds__(WAVES * 64) void k_build_joint_fp(
    const uint8_t *__restrict__ data, int64_t N, int64_t N_pad, const int32_t *__restrict__ ar,
    const double *__restrict__ prior, const int64_t *__restrict__ nsets, int n, int K, double ess,
    double log_gamma, int64_t n_subsets, int64_t S_pad, int cells_cap, const int32_t *__restrict__ lut_row,
    const double *__restrict__ lut, uint64_t *__restrict__ masks, float *__restrict__ scores)
{
    extern __shared__ uint32_t lds_hist[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // uniform: the subset's decode stays scalar
    const int lane = threadIdx.x & 63;
    uint32_t *hist = lds_hist + wave * cells_cap;
    for (int64_t g = (int64_t)blockIdx.x * WAVES + wave; g < n_subsets; g += (int64_t)gridDim.x * WAVES) {
        const uint64_t U = unrank_ascending(g + 1, n, K + 1, nsets);
        const Subset Sb = decode_subset(U, ar, n);
        const int j = Sb.j, cells = Sb.cells;
        joint_histogram(data, N, N_pad, Sb, hist, lane);
        // one family per member
        for (int c = 0; c < j; ++c) {
            int node, ri, sci, q;
            subset_member(Sb, c, node, ri, sci, q);
            const double *L_ijk = lut + (int64_t)lut_row[cells] * (N + 1);
            const double *L_ik = lut + (int64_t)lut_row[q] * (N + 1);
            double acc = 0.0;
            for (int k = lane; k < q; k += 64) {
                const int J = family_base(Sb, c, k);
                uint32_t nik = 0;
                double part = 0.0;
                for (int x = 0; x < ri; ++x) {
                    const uint32_t cnt = hist[J + (int)__umul24((uint32_t)x, (uint32_t)sci)];
                    nik += cnt;
                    if (cnt) part += L_ijk[cnt];
                }
                if (nik) part += -L_ik[nik];
                acc += part;
            }
            acc = wave_sum_f64(acc);
            if (lane == 0) {
                const uint64_t pm = U & ~(1ull << node);
                double sc = acc + (double)(j - 1) * log_gamma;
#pragma unroll
                for (int t = 0; t <= kMaxK; ++t)
                    if (t < j && t != c) sc += prior[(int64_t)node * n + Sb.u[t]];
                const uint64_t slot = (pm & ((1ull << node) - 1ull)) | (node >= 63 ? 0ull : ((pm >> (node + 1)) << node));
                const int64_t e = (int64_t)node * S_pad + rank_ascending(slot, n - 1, K, nsets);
                masks[e] = pm;
                scores[e] = (float)sc;   // round to nearest even
            }
        }
        wave_lds_sync();   // every lane has read hist before the next subset clears it
    }
}

// Padding entries e in [S, S_pad) of every row: (~0, -inf), which no
// predecessor set can contain.
__global__ void k_pad_rows(int n, int64_t S, int64_t S_pad, uint64_t *__restrict__ masks, float *__restrict__ scores)
{
    const int64_t per = S_pad - S;
    const int64_t total = (int64_t)n * per;
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < total; g += (int64_t)gridDim.x * blockDim.x) {
        const int64_t node = g / per;
        const int64_t e = node * S_pad + S + (g - node * per);
        masks[e] = ~0ull;
        scores[e] = -INFINITY;
    }
}

// One wavefront per (node, entry): enumerate the entry's parent set, count
// N_ijk in LDS, reduce the BDeu terms in FP64, add the structure penalty and
// the prior terms, store (mask, FP32 score).  Padding entries get (~0, -inf),
// which no predecessor set can contain.
template <int WAVES>
__global__ __launch_bounds__(WAVES * 64) void k_build(
    const uint8_t *__restrict__ data, int64_t N, int64_t N_pad, const int32_t *__restrict__ ar,
    const double *__restrict__ prior, const int64_t *__restrict__ nsets, int n, int K, double ess,
    double unit, double log_gamma, int64_t S, int64_t S_pad, int cells_cap, const int32_t *__restrict__ lut_row,
    const double *__restrict__ lut, uint64_t *__restrict__ masks, float *__restrict__ scores)
{
    extern __shared__ uint32_t lds_hist[];
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    uint32_t *hist = lds_hist + wave * cells_cap;
    const int64_t total = (int64_t)n * S_pad;
    for (int64_t g = (int64_t)blockIdx.x * WAVES + wave; g < total; g += (int64_t)gridDim.x * WAVES) {
        const int node = (int)(g / S_pad);
        const int64_t e = g - (int64_t)node * S_pad;
        if (e >= S) {
            if (lane == 0) {
                masks[g] = ~0ull;
                scores[g] = -INFINITY;
            }
            continue;
        }
        const uint64_t mask = slot_to_node_mask(unrank_ascending(e, n - 1, K, nsets), node);
        const int r = ar[node];
        Members M = decode_members(mask, r, ar);
        const int cells = M.q * r;
        wave_count(data, N, N_pad, node, M, cells, hist, lane);

        const double a_ijk = ess / (double)cells;
        const double a_ik = ess / (double)M.q;
        double acc = 0.0;
        if (lut && unit > 0.0) {      // integer terms
            const int64_t *L_ijk = reinterpret_cast<const int64_t *>(lut) + (int64_t)lut_row[cells] * (N + 1);
            const int64_t *L_ik = reinterpret_cast<const int64_t *>(lut) + (int64_t)lut_row[M.q] * (N + 1);
            uint64_t sum = 0ull;
            for (int k = lane; k < M.q; k += 64) {
                uint32_t nik = 0;
                for (int j = 0; j < r; ++j) {
                    const uint32_t c = hist[k * r + j];
                    nik += c;
                    sum += (uint64_t)L_ijk[c];
                }
                sum -= (uint64_t)L_ik[nik];
            }
            acc = (double)(int64_t)wave_sum_u64(sum) * unit;
        } else if (lut) {
            // lnG(c + a) - lnG(a) looked up per count (same FP64 values as computed below)
            const double *L_ijk = lut + (int64_t)lut_row[cells] * (N + 1);
            const double *L_ik = lut + (int64_t)lut_row[M.q] * (N + 1);
            for (int k = lane; k < M.q; k += 64) {
                uint32_t nik = 0;
                double part = 0.0;
                for (int j = 0; j < r; ++j) {
                    const uint32_t c = hist[k * r + j];
                    nik += c;
                    if (c) part += L_ijk[c];
                }
                if (nik) part += -L_ik[nik];
                acc += part;
            }
        } else {
            const double lg_ijk = lgamma(a_ijk);
            const double lg_ik = lgamma(a_ik);
            for (int k = lane; k < M.q; k += 64) {
                uint32_t nik = 0;
                double part = 0.0;
                for (int j = 0; j < r; ++j) {
                    const uint32_t c = hist[k * r + j];
                    nik += c;
                    if (c) part += lgamma((double)c + a_ijk) - lg_ijk;
                }
                if (nik) part += -(lgamma(a_ik + (double)nik) - lg_ik);
                acc += part;
            }
        }
        if (!(lut && unit > 0.0)) acc = wave_sum_f64(acc);
        wave_lds_sync();   // every lane has read hist before the next entry clears it
        if (lane == 0) {
            double s = fma((double)M.cnt, log_gamma, acc);
#pragma unroll
            for (int t = 0; t < kMaxK; ++t)
                if (t < M.cnt) s += prior[(int64_t)node * n + M.id[t]];
            masks[g] = mask;
            scores[g] = (float)s;   // round to nearest even
        }
    }
}

// Per-node static features of the learned proposal: prior terms summed as
// child (row) and as parent (column), and max, mean and population standard
// deviation of the node's stored FP32 scores (FP64 sums, fixed tree).  One block per row, each thread
// adds its entries in order: bound by the loads it has in flight (60
// nodes, 489,406 entries: 352 us one at a time, 86 us with 16).
constexpr int kStatLoads = 16;
template <typename Op>
__device__ __forceinline__ void stat_entries(const float *__restrict__ row, int64_t S, int tid, Op op)
{
    int64_t e = tid;
    for (; e + 1024 * (kStatLoads - 1) < S; e += 1024 * kStatLoads) {
        float v[kStatLoads];
#pragma unroll
        for (int i = 0; i < kStatLoads; ++i) v[i] = row[e + 1024 * i];
#pragma unroll
        for (int i = 0; i < kStatLoads; ++i) op((double)v[i]);
    }
    for (; e < S; e += 1024) op((double)row[e]);
}

__global__ __launch_bounds__(1024) void k_node_stats(const float *__restrict__ scores, int64_t S, int64_t S_pad,
                                                     const double *__restrict__ prior, int n,
                                                     double *__restrict__ out)
{
    __shared__ double s_a[1024], s_b[1024];
    const int node = blockIdx.x;
    const int tid = threadIdx.x;
    const float *row = scores + (int64_t)node * S_pad;
    double mx = -INFINITY, sum = 0.0;
    stat_entries(row, S, tid, [&](double v) {
        mx = v > mx ? v : mx;
        sum += v;
    });
    s_a[tid] = mx;
    s_b[tid] = sum;
    __syncthreads();
    for (int w = 512; w >= 1; w >>= 1) {
        if (tid < w) {
            s_a[tid] = s_a[tid + w] > s_a[tid] ? s_a[tid + w] : s_a[tid];
            s_b[tid] += s_b[tid + w];
        }
        __syncthreads();
    }
    const double gmax = s_a[0];
    const double mean = s_b[0] / (double)S;
    __syncthreads();
    double sq = 0.0;
    stat_entries(row, S, tid, [&](double v) {
        const double d = v - mean;
        sq += d * d;
    });
    s_b[tid] = sq;
    __syncthreads();
    for (int w = 512; w >= 1; w >>= 1) {
        if (tid < w) s_b[tid] += s_b[tid + w];
        __syncthreads();
    }
    if (tid == 0) {
        double rs = 0.0, cs = 0.0;
        for (int m = 0; m < n; ++m) {
            if (m == node) continue;
            rs += prior[(int64_t)node * n + m];
            cs += prior[(int64_t)m * n + node];
        }
        double *o = out + (int64_t)node * 5;
        o[0] = rs;
        o[1] = cs;
        o[2] = gmax;
        o[3] = mean;
        o[4] = sqrt(s_b[0] / (double)S);
    }
}

// AND of the masks of every 256-entry tile and of its four 64-entry sub-tiles,
// and the tile's largest score (one wavefront per tile), stored at the tile's
// summary place (summary_pos: row_tiles tiles per row, in sum_chunks chunks of
// sum_steps steps).
__global__ __launch_bounds__(256) void k_tile_and(const uint64_t *__restrict__ masks,
                                                  const float *__restrict__ scores, int64_t tiles,
                                                  int64_t row_tiles, int64_t sum_chunks, int sum_steps,
                                                  uint64_t *__restrict__ tand, uint64_t *__restrict__ tsub,
                                                  float *__restrict__ tmax)
{
    const int64_t tile = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (tile >= tiles) return;                       // uniform per wavefront
    const int64_t row = tile / row_tiles, r = tile - row * row_tiles;
    const int64_t at = row * row_tiles + summary_pos(r >> 2, (int)(r & 3), sum_chunks, sum_steps);
    const uint64_t *p = masks + tile * 256 + lane * 4;
    const float *q = scores + tile * 256 + lane * 4;
    uint64_t v = p[0] & p[1] & p[2] & p[3];
    float x = fmaxf(fmaxf(q[0], q[1]), fmaxf(q[2], q[3]));
    // lanes 16s .. 16s+15 hold sub-tile s (entries 64s .. 64s+63)
#pragma unroll
    for (int off = 1; off <= 8; off <<= 1) v &= (uint64_t)__shfl_xor((unsigned long long)v, off, 64);
    if ((lane & 15) == 0) tsub[at * 4 + (lane >> 4)] = v;
#pragma unroll
    for (int off = 16; off <= 32; off <<= 1) v &= (uint64_t)__shfl_xor((unsigned long long)v, off, 64);
#pragma unroll
    for (int off = 1; off <= 32; off <<= 1) x = fmaxf(x, __shfl_xor(x, off, 64));
    if (lane == 0) {
        tand[at] = v;
        tmax[at] = x;
    }
}

// Index in a row of the singleton {slot s}: every mask below 1 << s, i.e.
// every set of at most K slots below s, comes first.
__device__ __forceinline__ int64_t singleton_index(int s, int K)
{
    int64_t c = 1, tot = 1;
    for (int k = 1; k <= K; ++k) {
        c = c * (s - k + 1) / k;
        tot += c;
    }
    return tot;
}

// The score bound's candidates of each row (one block per node), in
// kBoundSlots slots: slot s < n - 1 the singleton of slot s (K >= 1), slot 63
// the empty set, then the listed top entries: with M the row's largest score
// among the sets of two or more members, the entries of those sets within b
// quarter-nats of M, for the largest b that keeps them to at most
// kBoundCands.  Unused slots hold (~0, -inf), which no order can use.  The
// list's order is that of the appends and does not matter: only the entries'
// values are used.
constexpr int kBoundBins = 1024;
__global__ __launch_bounds__(1024) void k_bound_cands(const uint64_t *__restrict__ masks,
                                                      const float *__restrict__ scores, int n, int K, int64_t S,
                                                      int64_t S_pad, uint64_t *__restrict__ cmask,
                                                      float *__restrict__ cscore)
{
    __shared__ float s_max[1024 / 64];
    __shared__ unsigned s_hist[kBoundBins];
    __shared__ unsigned s_cut, s_cnt;
    const int node = blockIdx.x;
    const int tid = threadIdx.x;
    const uint64_t *mr = masks + (int64_t)node * S_pad;
    const float *sr = scores + (int64_t)node * S_pad;
    float mx = -INFINITY;
    for (int64_t e = tid; e < S; e += 1024)
        if (__popcll(mr[e]) >= 2) mx = fmaxf(mx, sr[e]);
#pragma unroll
    for (int off = 1; off <= 32; off <<= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    if ((tid & 63) == 0) s_max[tid >> 6] = mx;
    for (int i = tid; i < kBoundBins; i += 1024) s_hist[i] = 0u;
    __syncthreads();
    float M = s_max[0];
    for (int w = 1; w < 1024 / 64; ++w) M = fmaxf(M, s_max[w]);
    for (int64_t e = tid; e < S; e += 1024) {
        if (__popcll(mr[e]) < 2) continue;
        const float d = (M - sr[e]) * 4.0f;
        if (d < (float)kBoundBins) atomicAdd(&s_hist[(int)d], 1u);
    }
    __syncthreads();
    if (tid == 0) {
        unsigned acc = 0u;
        int b = 0;
        while (b < kBoundBins && acc + s_hist[b] <= (unsigned)kBoundCands) acc += s_hist[b++];
        s_cut = (unsigned)b;
        s_cnt = 0u;
    }
    __syncthreads();
    const float cut = (float)s_cut;
    if (tid < 64) {
        uint64_t fm = ~0ull;
        float fx = -INFINITY;
        if (tid == 63) {
            fm = 0ull;
            fx = sr[0];
        } else if (tid < n - 1 && K >= 1) {
            fm = 1ull << (tid < node ? tid : tid + 1);
            fx = sr[singleton_index(tid, K)];
        }
        cmask[(int64_t)node * kBoundSlots + tid] = fm;
        cscore[(int64_t)node * kBoundSlots + tid] = fx;
    }
    uint64_t *cm = cmask + (int64_t)node * kBoundSlots + 64;
    float *cs = cscore + (int64_t)node * kBoundSlots + 64;
    for (int64_t e = tid; e < S; e += 1024) {
        const uint64_t m = mr[e];
        if (__popcll(m) < 2) continue;
        const float x = sr[e];
        if ((M - x) * 4.0f < cut) {
            const unsigned k = atomicAdd(&s_cnt, 1u);
            cm[k] = m;
            cs[k] = x;
        }
    }
    __syncthreads();
    for (int k = (int)s_cnt + tid; k < kBoundCands; k += 1024) {
        cm[k] = ~0ull;
        cs[k] = -INFINITY;
    }
}

// The slot-space mask (the node's own bit removed: slot s is node s below the
// node, node s + 1 above it) of the first entry of every 4-entry group of each
// row, for the scoring pass that computes the other masks; for padding, the
// mask of slot n - 1, which no row holds and no step from it leaves.
__global__ __launch_bounds__(256) void k_anchor(const uint64_t *__restrict__ masks, int n, int64_t S_pad,
                                                uint64_t *__restrict__ anchor)
{
    const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t per_row = S_pad / 4;
    if (g >= (int64_t)n * per_row) return;
    const int node = (int)(g / per_row);
    const uint64_t m = masks[g * 4];
    const uint64_t low = (1ull << node) - 1ull;
    anchor[g] = (m == ~0ull) ? (1ull << (n - 1)) : ((m & low) | ((m >> 1) & ~low));
}

// ---- kept entries (see kept_mean)
//
// Subset records: sub[node][r], r the rank of a set among those of at most K - 1
// members, holds (the largest score among the set's subsets and itself, its own
// score).  A set of j members takes its j immediate subsets' records, so the
// passes run over j = 0, 1, ... K - 1.

struct SubRec {
    float top, own;
};

// This block's copy of nsets as 32-bit numbers (ranks are below 2^31: a row has fewer entries).
__device__ __forceinline__ void load_nsets32(const int64_t *__restrict__ nsets, int *s_ns)
{
    for (int i = threadIdx.x; i < 512; i += blockDim.x) s_ns[i] = (int)nsets[i];
    __syncthreads();
}

// The largest score among a set's proper subsets, and the second largest of its
// immediate subsets' own scores and the empty set's (distinct entries for two or more
// members), for slot-space mask m (at least one member).  The rank of m without member
// t is the sum of the weights of the members above t at their own places and of those
// below t one place up; places count down from `k`, the size limit of the ranks' space.
__device__ __forceinline__ void subset_bounds(uint64_t m, int k, const int *__restrict__ s_ns,
                                              const SubRec *__restrict__ sub, float empty, float &top, float &sec)
{
    int below = 0;                                 // members below the removed one, one place up
    {
        int t = 0;
        for (uint64_t x = m; x; ++t) {
            const int b = 63 - __builtin_clzll(x);
            x &= ~(1ull << b);
            if (t > 0) below += s_ns[b * 8 + (k - t + 1)];
        }
    }
    int above = 0, t = 0;
    top = -INFINITY;
    float s1 = empty, s2 = -INFINITY;
    for (uint64_t x = m; x; ++t) {
        const int b = 63 - __builtin_clzll(x);
        x &= ~(1ull << b);
        if (t > 0) below -= s_ns[b * 8 + (k - t + 1)];
        const SubRec r = sub[above + below];
        top = fmaxf(top, r.top);
        s2 = fmaxf(s2, fminf(s1, r.own));
        s1 = fmaxf(s1, r.own);
        if (k - t >= 0) above += s_ns[b * 8 + (k - t)];
    }
    sec = s2;
}

// The e-th mask over `bits` bits with at most k members, from the block's copy of nsets.
__device__ __forceinline__ uint64_t unrank32(int e, int bits, int k, const int *__restrict__ s_ns)
{
    uint64_t m = 0;
    for (int b = bits - 1; b >= 0 && k > 0; --b) {
        const int c = s_ns[b * 8 + k];
        if (e >= c) {
            m |= 1ull << b;
            e -= c;
            --k;
        }
    }
    return m;
}

// Records of one node's sets of at most K - 1 members, one block per node, the sets of j
// members after those of j - 1.
__global__ __launch_bounds__(1024) void k_keep_subsets(const float *__restrict__ scores,
                                                       const int64_t *__restrict__ nsets, int n, int K,
                                                       int64_t S_pad, int64_t sub_row, SubRec *sub)
{
    __shared__ int s_ns[512];
    load_nsets32(nsets, s_ns);
    const int node = blockIdx.x;
    const float *row = scores + (int64_t)node * S_pad;
    SubRec *out = sub + (int64_t)node * sub_row;
    for (int j = 0; j < K; ++j) {
        const int sets = s_ns[(n - 1) * 8 + j];                      // of at most j members
        for (int g = threadIdx.x; g < sets; g += 1024) {
            const uint64_t m = unrank32(g, n - 1, j, s_ns);
            if (__popcll(m) != j) continue;
            int full = 0, mine = 0, t = 0;         // ranks in the row and among the sets of at most K - 1
            for (uint64_t x = m; x; ++t) {
                const int b = 63 - __builtin_clzll(x);
                x &= ~(1ull << b);
                full += s_ns[b * 8 + (K - t)];
                mine += s_ns[b * 8 + (K - 1 - t)];
            }
            const float own = row[full];
            float top = own;
            if (j > 0) {
                float below, sec;
                subset_bounds(m, K - 1, s_ns, out, row[0], below, sec);
                top = fmaxf(top, below);
            }
            out[mine] = {top, own};
        }
        __syncthreads();
    }
}

// b - kBoundGap, or -inf where FP32 cannot hold that gap below b or rounds it towards b: the entries
// below b are all kept then (the scans' gap_below is lowered instead).
__device__ __forceinline__ float keep_gap_below(float b)
{
    const float g = b - kBoundGap;
    return (b - g >= kBoundGap) ? g : -INFINITY;
}

// Where a row's kept entries sit: rows follow one another, padded to whole steps of a scan.
// By one wavefront; *fits tells whether all rows have room.
__device__ __forceinline__ int kept_place_of(const int32_t *klen, int n, int node, int64_t cap, bool *fits)
{
    const int lane = threadIdx.x & 63;
    constexpr int kStep = 64 * kKeptTiles;
    const int len = lane < n ? klen[lane] : 0;
    int64_t sum = (len + kStep - 1) / kStep * kStep;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int64_t o = __shfl_up(sum, off, 64);
        if (lane >= off) sum += o;
    }
    *fits = __shfl(sum, 63, 64) <= cap && __ballot(len > kKeptCap) == 0ull;
    return node > 0 ? (int)__shfl(sum, node - 1, 64) : 0;
}

// One thread per 4-entry group of a row: which of its entries are kept (the byte of
// `kept`), and the rows' numbers of them.
__global__ __launch_bounds__(256) void k_keep_entries(const uint64_t *__restrict__ masks,
                                                      const float *__restrict__ scores,
                                                      const int64_t *__restrict__ nsets, int n, int K, int64_t S,
                                                      int64_t S_pad, int64_t sub_row, const SubRec *__restrict__ sub,
                                                      uint8_t *__restrict__ kept, int32_t *__restrict__ klen)
{
    __shared__ int s_ns[512];
    load_nsets32(nsets, s_ns);
    const int node = blockIdx.y;
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;       // the row's 4-entry group (S_pad / 4 is a multiple of 256)
    const int64_t row = (int64_t)node * S_pad;
    const SubRec *srow = sub + (int64_t)node * sub_row;
    const float empty = scores[row];
    uint32_t bits = 0u;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int64_t at = 4 * q + e;
        if (at >= S) continue;
        const float x = scores[row + at];
        const uint64_t nm = masks[row + at];
        const uint64_t low = (1ull << node) - 1ull;
        const uint64_t m = (nm & low) | ((nm >> 1) & ~low);          // slot space
        bool keep = true;
        if (__popcll(m) >= 2) {
            float top, sec;
            subset_bounds(m, K - 1, s_ns, srow, empty, top, sec);
            keep = !(x < keep_gap_below(top) && x < sec);
        }
        bits |= keep ? (1u << e) : 0u;
    }
    kept[row / 4 + q] = (uint8_t)bits;
    int mine = __popc(bits);
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) mine += __shfl_xor(mine, off, 64);
    if ((threadIdx.x & 63) == 0 && mine != 0) atomicAdd(&klen[node], mine);
}

// A sort key for each kept entry, appended to its row's list (in any order: the sort fixes
// it).  A key's high half falls as the score rises, its low half is the place in the row, so
// ascending keys list descending scores and, among equal ones, ascending masks.  klen also
// receives the rows' first entries, and holds the lists' cursors (zero at first).  60 nodes: 363 us with
// one byte of the bits per lane and round, 210 us with four (the cursors' updates bound it).
__global__ __launch_bounds__(256) void k_keep_keys(const float *__restrict__ scores, int n, int64_t S_pad,
                                                   const uint8_t *__restrict__ kept, int64_t cap,
                                                   uint64_t *__restrict__ keys, int32_t *klen)
{
    const int node = blockIdx.y;
    const int lane = threadIdx.x & 63;
    bool fits;
    const int first = kept_place_of(klen, n, node, cap, &fits);
    if (!fits) return;                                               // uniform over the grid
    if (blockIdx.x == 0 && threadIdx.x == 0) klen[2 * n + node] = first;
    const int64_t row = (int64_t)node * S_pad;
    // four bytes of the bits, 16 entries, per lane (S_pad is a multiple of 1024)
    const uint32_t *words = reinterpret_cast<const uint32_t *>(kept + row / 4);
    for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < S_pad / 16; q += (int64_t)gridDim.x * 256) {
        const uint32_t bits = words[q];
        const int mine = __popc(bits);
        int before = mine;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(before, off, 64);
            if (lane >= off) before += o;
        }
        const int total = __shfl(before, 63, 64);
        if (total == 0) continue;                                    // uniform per wavefront
        int base = 0;
        if (lane == 0) base = atomicAdd(&klen[3 * n + node], total); // one update per wavefront
        base = first + __shfl(base, 0, 64) + before - mine;
        for (uint32_t x = bits; x; x &= x - 1) {                     // bit 8 b + e: entry 4 b + e of the 16
            const int p = __builtin_ctz(x);
            const int64_t at = 16 * q + 4 * (p >> 3) + (p & 7);
            const uint32_t u = __float_as_uint(scores[row + at] + 0.0f);          // -0 sorts as +0
            const uint32_t up = (u >> 31) ? ~u : (u | 0x80000000u);               // rises with the score
            keys[base++] = ((uint64_t)~up << 32) | (uint32_t)at;
        }
    }
}

// The kept row's entry `place` from its key.
__device__ __forceinline__ void keep_entry(const uint64_t *masks, const float *scores, int64_t row, uint64_t key,
                                           uint64_t *kmask, float *kscore, int64_t place)
{
    const int64_t at = row + (uint32_t)key;
    kmask[place] = masks[at];
    kscore[place] = scores[at];
}

// Sort of one run of a row's keys (bitonic, in LDS); a row of one run goes straight to its kept
// entries.
__global__ __launch_bounds__(1024) void k_keep_sort(const uint64_t *__restrict__ masks,
                                                    const float *__restrict__ scores, int n, int64_t S_pad,
                                                    int64_t cap, const int32_t *__restrict__ klen, uint64_t *keys,
                                                    uint64_t *__restrict__ kmask, float *__restrict__ kscore)
{
    __shared__ uint64_t s_key[kKeptRun];
    const int node = blockIdx.x;
    const int tid = threadIdx.x;
    const int all = klen[node], begin = blockIdx.y * kKeptRun;
    if (begin >= all) return;                                        // uniform
    bool fits;
    const int64_t first = kept_place_of(klen, n, node, cap, &fits);
    if (!fits) return;                                               // uniform
    const int len = all - begin < kKeptRun ? all - begin : kKeptRun;
    int P = 64;
    while (P < len) P <<= 1;                                         // P <= kKeptRun
    uint64_t *run = keys + first + begin;
    for (int i = tid; i < P; i += 1024) s_key[i] = i < len ? run[i] : ~0ull;
    __syncthreads();
    for (int k = 2; k <= P; k <<= 1)
        for (int j = k >> 1; j >= 1; j >>= 1) {
            for (int i = tid; i < P / 2; i += 1024) {
                const int a = 2 * i - (i & (j - 1)), b = a + j;       // the i-th pair at distance j
                const uint64_t x = s_key[a], y = s_key[b];
                const bool up = (a & k) == 0;
                if ((x > y) == up) {
                    s_key[a] = y;
                    s_key[b] = x;
                }
            }
            __syncthreads();
        }
    for (int i = tid; i < len; i += 1024) {
        if (all <= kKeptRun) keep_entry(masks, scores, (int64_t)node * S_pad, s_key[i], kmask, kscore, first + i);
        else run[i] = s_key[i];
    }
}

// The kept entries of a row of several sorted runs: a key's place is its place in its own run
// plus the smaller keys of the other runs (keys are distinct).  One thread per key.
__global__ __launch_bounds__(1024) void k_keep_merge(const uint64_t *__restrict__ masks,
                                                     const float *__restrict__ scores, int n, int64_t S_pad,
                                                     int64_t cap, const int32_t *__restrict__ klen,
                                                     const uint64_t *__restrict__ keys,
                                                     uint64_t *__restrict__ kmask, float *__restrict__ kscore)
{
    const int node = blockIdx.x;
    const int len = klen[node], i = blockIdx.y * 1024 + threadIdx.x;
    if (len <= kKeptRun || blockIdx.y * 1024 >= (unsigned)len) return;   // uniform
    bool fits;
    const int64_t first = kept_place_of(klen, n, node, cap, &fits);
    if (!fits || i >= len) return;
    const uint64_t *k = keys + first;
    const uint64_t key = k[i];
    const int own = i / kKeptRun;
    int place = i - own * kKeptRun;
    for (int r = 0; r * kKeptRun < len; ++r) {
        if (r == own) continue;
        int lo = r * kKeptRun, hi = lo + kKeptRun < len ? lo + kKeptRun : len;
        const int lo0 = lo;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (k[mid] < key) lo = mid + 1;
            else hi = mid;
        }
        place += lo - lo0;
    }
    keep_entry(masks, scores, (int64_t)node * S_pad, key, kmask, kscore, first + place);
}

// One block per kept row: its padding, the largest kept score among the sets holding each node
// (the first place that holds it), the row's score-bound candidates (as k_bound_cands lists
// them, but the top kept entries), and its place among the rows in descending length.
__global__ __launch_bounds__(1024) void k_keep_top(int n, int64_t cap, int32_t *klen, uint64_t *kmask, float *kscore,
                                                   float *__restrict__ kpm, uint64_t *__restrict__ cmask,
                                                   float *__restrict__ cscore)
{
    __shared__ int s_first[64];
    const int node = blockIdx.x;
    const int tid = threadIdx.x;
    const int len = klen[node];
    bool fits;
    const int64_t first = kept_place_of(klen, n, node, cap, &fits);
    if (!fits) return;                                               // uniform
    uint64_t *krow = kmask + first, *cm = cmask + (int64_t)node * kBoundSlots;
    float *xrow = kscore + first, *cs = cscore + (int64_t)node * kBoundSlots;
    if (tid < 64) {
        s_first[tid] = 0x7fffffff;
        const int o = tid < n ? klen[tid] : -1;
        const int before = __popcll(__ballot(o > len || (o == len && tid < node)));
        if (tid == 0) klen[n + before] = node;
    }
    if (tid < kBoundSlots) {
        cm[tid] = ~0ull;
        cs[tid] = -INFINITY;
    }
    constexpr int kStep = 64 * kKeptTiles;
    const int padded = (len + kStep - 1) / kStep * kStep;
    for (int i = len + tid; i < padded; i += 1024) {
        krow[i] = ~0ull;
        xrow[i] = -INFINITY;
    }
    __syncthreads();
    for (int i = tid; i < len; i += 1024) {
        const uint64_t m = krow[i];
        for (uint64_t r = m; r; r &= r - 1) {
            const int b = __builtin_ctzll(r);
            if (i < s_first[b]) atomicMin(&s_first[b], i);
        }
        if (__popcll(m) < 2) {                                       // the empty set and the singletons
            const int b = m ? __builtin_ctzll(m) : 64;
            const int to = m == 0ull ? 63 : (b < node ? b : b - 1);
            cm[to] = m;
            cs[to] = xrow[i];
        }
    }
    __syncthreads();
    if (tid < n) {
        const int f = s_first[tid];
        kpm[(int64_t)node * n + tid] = f < len ? xrow[f] : -INFINITY;
    }
    if (tid < 64) {                                                  // one wavefront
        int at = 64;
        for (int i0 = 0; i0 < len && at < kBoundSlots; i0 += 64) {   // uniform
            const int i = i0 + tid;
            const uint64_t m = i < len ? krow[i] : ~0ull;
            const float x = i < len ? xrow[i] : -INFINITY;
            const bool list = i < len && __popcll(m) >= 2;
            const uint64_t bal = __ballot(list);
            const int to = at + __popcll(bal & ((1ull << tid) - 1ull));
            if (list && to < kBoundSlots) {
                cm[to] = m;
                cs[to] = x;
            }
            at += __popcll(bal);
        }
    }
}

// Counts for explicit (node, parent mask) queries, with the build's counting code.
template <int WAVES>
__global__ __launch_bounds__(WAVES * 64) void k_counts(
    const uint8_t *__restrict__ data, int64_t N, int64_t N_pad, const int32_t *__restrict__ ar,
    int Q, const int32_t *__restrict__ qnode, const uint64_t *__restrict__ qmask,
    const int64_t *__restrict__ qoff, int cells_cap, uint32_t *__restrict__ out)
{
    extern __shared__ uint32_t lds_hist[];
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    uint32_t *hist = lds_hist + wave * cells_cap;
    for (int qi = blockIdx.x * WAVES + wave; qi < Q; qi += gridDim.x * WAVES) {
        const int node = qnode[qi];
        const int r = ar[node];
        Members M = decode_members(qmask[qi], r, ar);
        const int cells = M.q * r;
        wave_count(data, N, N_pad, node, M, cells, hist, lane);
        for (int c = lane; c < cells; c += 64) out[qoff[qi] + c] = hist[c];
        wave_lds_sync();
    }
}

// The same queries answered by the joint-histogram path of the default build
// (k_build_joint): the histogram of U = parents + node, read out as the
// family's cells (parent configuration k, the lowest id most significant, then
// the child state).
template <int WAVES>
__global__ __launch_bounds__(WAVES * 64) void k_counts_joint(
    const uint8_t *__restrict__ data, int64_t N, int64_t N_pad, const int32_t *__restrict__ ar, int n,
    int Q, const int32_t *__restrict__ qnode, const uint64_t *__restrict__ qmask,
    const int64_t *__restrict__ qoff, int cells_cap, uint32_t *__restrict__ out)
{
    extern __shared__ uint32_t lds_hist[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // uniform: the subset's decode stays scalar
    const int lane = threadIdx.x & 63;
    uint32_t *hist = lds_hist + wave * cells_cap;
    for (int qi = blockIdx.x * WAVES + wave; qi < Q; qi += gridDim.x * WAVES) {
        const int child = qnode[qi];
        const uint64_t U = qmask[qi] | (1ull << child);
        const Subset Sb = decode_subset(U, ar, n);
        joint_histogram(data, N, N_pad, Sb, hist, lane);
        const int c = __popcll(U & ((1ull << child) - 1ull));       // the child's place among U's members
        int node, ri, sci, q;
        subset_member(Sb, c, node, ri, sci, q);
        for (int k = lane; k < q; k += 64) {
            const int J = family_base(Sb, c, k);
            for (int x = 0; x < ri; ++x)
                out[qoff[qi] + (int64_t)k * ri + x] = hist[J + (int)__umul24((uint32_t)x, (uint32_t)sci)];
        }
        wave_lds_sync();
    }
}

// ------------------------------------------------------------------ host side

static int64_t binom_host(int a, int b)
{
    if (b < 0 || a < 0 || b > a) return 0;
    int64_t r = 1;
    for (int t = 1; t <= b; ++t) r = r * (a - b + t) / t;
    return r;
}

static int64_t sets_upto(int m, int K)
{
    int64_t s = 0;
    for (int j = 0; j <= K && j <= m; ++j) s += binom_host(m, j);
    return s;
}

static int waves_for_cells(int cells_cap) { return cells_cap <= 4096 ? 4 : 1; }

// Units per nat of an integer lookup (a power of two), or 0 where FP64 terms serve: alpha = ess / d
// runs from ess / max_cells to ess, so with N samples no term's magnitude passes N (ln(N + ess + 1) + 1)
// + |ln alpha| + 1, a family has at most min(N, cells) terms that start at ln alpha, and its sums
// stay below the bound formed here; outside these ess the differences of lgamma lose their digits.
static double lut_scale(double ess, int64_t N, int max_cells)
{
    if (!(ess >= 1e-6 && ess <= 1e6)) return 0.0;
    const double starts = (double)std::min<int64_t>(N + 1, max_cells);
    const double bound = 2.0 * ((double)(N + 1) * (std::log((double)N + ess + 2.0) + 1.0) +
                                starts * (std::fabs(std::log(ess / (double)max_cells)) + std::fabs(std::log(ess)) + 2.0));
    int s = 62;
    for (double b = bound; b >= 1.0; b *= 0.5) --s;
    return s < 1 ? 0.0 : std::ldexp(1.0, s < 50 ? s : 50);
}

template <int W>
static hipError_t launch_build(TableT *t, hipStream_t st, int cells_cap, const int32_t *lut_row, const double *lut,
                               double scale)
{
    int64_t total = (int64_t)t->n * t->S_pad;
    int64_t blocks = (total + W - 1) / W;
    if (blocks > (1 << 22)) blocks = 1 << 22;
    size_t lds = (size_t)W * cells_cap * sizeof(uint32_t);
    hipLaunchKernelGGL(k_build<W>, dim3((unsigned)blocks), dim3(W * 64), lds, st, t->d_data, t->N,
                       t->N_pad, t->d_ar, t->d_prior, t->d_nsets, t->n, t->K, t->ess,
                       scale > 0.0 ? 1.0 / scale : 0.0, t->log_gamma,
                       t->S, t->S_pad, cells_cap, lut_row, lut, t->d_masks, t->d_scores);
    return hipGetLastError();
}

template <int W>
static hipError_t launch_build_joint(TableT *t, hipStream_t st, int cells_cap, const int32_t *lut_row,
                                     const double *lut, double scale)
{
    const int64_t subsets = sets_upto(t->n, t->K + 1) - 1;
    size_t lds = (size_t)W * cells_cap * sizeof(uint32_t);
    if (scale > 0.0) {
        // runs long enough to spread the first subset's unranking, short enough to leave 16 wavefronts
        // to each SIMD of the card
        const int run = (int)std::max<int64_t>(1, std::min<int64_t>(32, subsets / 16384));
        const int64_t waves = (subsets + run - 1) / run, blocks = (waves + W - 1) / W;
        if (blocks > INT32_MAX) return hipErrorInvalidValue;
        hipLaunchKernelGGL(k_build_joint<W>, dim3((unsigned)blocks), dim3(W * 64), lds, st, t->d_data, t->N,
                           t->N_pad, t->d_ar, t->d_prior, t->d_nsets, t->n, t->K, 1.0 / scale, t->log_gamma, subsets,
                           run, t->S_pad, cells_cap, lut_row, reinterpret_cast<const int64_t *>(lut), t->d_masks,
                           t->d_scores);
    } else {
        int64_t blocks = (subsets + W - 1) / W;
        if (blocks > (1 << 22)) blocks = 1 << 22;
        hipLaunchKernelGGL(k_build_joint_fp<W>, dim3((unsigned)blocks), dim3(W * 64), lds, st, t->d_data, t->N,
                           t->N_pad, t->d_ar, t->d_prior, t->d_nsets, t->n, t->K, t->ess, t->log_gamma, subsets,
                           t->S_pad, cells_cap, lut_row, lut, t->d_masks, t->d_scores);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || t->S_pad == t->S) return e;
    const int64_t pad = (int64_t)t->n * (t->S_pad - t->S);
    hipLaunchKernelGGL(k_pad_rows, dim3((unsigned)std::min<int64_t>((pad + 255) / 256, 1 << 16)), dim3(256), 0, st,
                       t->n, t->S, t->S_pad, t->d_masks, t->d_scores);
    return hipGetLastError();
}

static int cells_cap_for(int max_cells)
{
    int c = 64;
    while (c < max_cells) c <<= 1;
    return c;
}

static void free_kept(TableT *t)
{
    hipFree(t->d_kmask);                           // one allocation holds all of them
    t->d_kmask = nullptr;
    t->d_kscore = nullptr;
    t->d_klen = nullptr;
    t->d_kpm = nullptr;
    t->d_kept = nullptr;
}

// Lists the table's kept rows after its rows are built (waits for the stream).  A table
// without them (more kept entries than kept_mean per row, a memory cap they would pass, no
// memory for them) is served by the streaming pass, so nothing here fails the build but a
// device error.
static hipError_t list_kept(TableT *t, hipStream_t st, int64_t max_bytes)
{
    const int n = t->n, K = t->K;
    const int64_t sub_row = K >= 1 ? sets_upto(n - 1, K - 1) : 1;
    if (sub_row * n > kKeptSubsetCap) return hipSuccess;
    constexpr int64_t kStep = 64 * kKeptTiles;
    const int64_t row_cap = std::min<int64_t>((t->S + kStep - 1) / kStep * kStep, kKeptCap);
    t->kept_cap = n * std::min<int64_t>(row_cap, kept_mean(t->S));
    if (max_bytes > 0 && t->device_bytes() + t->kept_bytes() > max_bytes) return hipSuccess;
    // one allocation for the table (kept_bytes() of it) and one for the build's passes
    const int64_t cells = t->kept_cap;
    char *own = nullptr, *tmp = nullptr;
    if (hipMalloc((void **)&own, (size_t)t->kept_bytes()) != hipSuccess ||
        hipMalloc((void **)&tmp, (size_t)(cells * 8 + sub_row * n * (int64_t)sizeof(SubRec))) != hipSuccess) {
        (void)hipGetLastError();
        hipFree(own);
        return hipSuccess;
    }
    t->d_kmask = reinterpret_cast<uint64_t *>(own);
    t->d_kscore = reinterpret_cast<float *>(own + cells * 8);
    t->d_kpm = reinterpret_cast<float *>(own + cells * 12);
    t->d_klen = reinterpret_cast<int32_t *>(own + cells * 12 + (int64_t)n * n * 4);
    t->d_kept = reinterpret_cast<uint8_t *>(own + cells * 12 + (int64_t)n * n * 4 + (int64_t)n * 16);
    uint64_t *keys = reinterpret_cast<uint64_t *>(tmp);
    SubRec *sub = reinterpret_cast<SubRec *>(tmp + cells * 8);
    std::vector<int32_t> len(n);
    hipError_t e = hipMemsetAsync(t->d_klen, 0, sizeof(int32_t) * 4 * n, st);
    if (e == hipSuccess) {
        const unsigned groups = (unsigned)(t->S_pad / 1024), longest = (unsigned)std::min<int64_t>(row_cap, cells);
        hipLaunchKernelGGL(k_keep_subsets, dim3(n), dim3(1024), 0, st, t->d_scores, t->d_nsets, n, K, t->S_pad,
                           sub_row, sub);
        hipLaunchKernelGGL(k_keep_entries, dim3(groups, (unsigned)n), dim3(256), 0, st, t->d_masks, t->d_scores,
                           t->d_nsets, n, K, t->S, t->S_pad, sub_row, sub, t->d_kept, t->d_klen);
        hipLaunchKernelGGL(k_keep_keys, dim3(std::min((groups + 3) / 4, 128u), (unsigned)n), dim3(256), 0, st, t->d_scores, n,
                           t->S_pad, t->d_kept, cells, keys, t->d_klen);
        hipLaunchKernelGGL(k_keep_sort, dim3(n, (longest + kKeptRun - 1) / kKeptRun), dim3(1024), 0, st, t->d_masks,
                           t->d_scores, n, t->S_pad, cells, t->d_klen, keys, t->d_kmask, t->d_kscore);
        if (longest > (unsigned)kKeptRun)
            hipLaunchKernelGGL(k_keep_merge, dim3(n, (longest + 1023) / 1024), dim3(1024), 0, st, t->d_masks,
                               t->d_scores, n, t->S_pad, cells, t->d_klen, keys, t->d_kmask, t->d_kscore);
        hipLaunchKernelGGL(k_keep_top, dim3(n), dim3(1024), 0, st, n, cells, t->d_klen, t->d_kmask, t->d_kscore,
                           t->d_kpm, t->d_cmask, t->d_cscore);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpyAsync(len.data(), t->d_klen, sizeof(int32_t) * n, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    hipFree(tmp);
    if (e != hipSuccess) return e;
    bool fits = true;
    for (int i = 0; i < n; ++i) {
        const int64_t steps = (len[i] + kStep - 1) / kStep;
        fits = fits && len[i] <= kKeptCap;
        t->kept_total += len[i];
        t->kept_steps += steps;
        t->kept_steps_max = std::max(t->kept_steps_max, (int)steps);
    }
    if (!fits || t->kept_steps * kStep > cells) free_kept(t);
    return hipSuccess;
}

static void free_device(TableT *t)
{
    hipFree(t->d_data);
    hipFree(t->d_prior);
    hipFree(t->d_nsets);
    hipFree(t->d_masks);
    hipFree(t->d_scores);
    hipFree(t->d_nstat);
    hipFree(t->d_tand);
    hipFree(t->d_tsub);
    hipFree(t->d_anchor);
    hipFree(t->d_tmax);
    hipFree(t->d_cmask);
    hipFree(t->d_cscore);
    hipFree(t->d_part);
    hipFree(t->d_kpart);
    free_kept(t);
    for (auto e : t->ev_start) hipEventDestroy(e);
    for (auto e : t->ev_stop) hipEventDestroy(e);
}

}  // namespace bnos

using namespace bnos;

extern "C" const char *bnos_last_error(void) { return g_err.c_str(); }

extern "C" int32_t bnos_version(void) { return 100; }

extern "C" bnos_status bnos_build_score_table(const int8_t *data, int64_t N, int32_t n,
                                              const int32_t *arities, int32_t K, double ess,
                                              const float *prior, const bnos_build_opts *opts,
                                              void *stream, bnos_table *out)
{
    if (!out) { set_error("out is NULL"); return BNOS_E_INVALID; }
    if (!arities) { set_error("arities is NULL"); return BNOS_E_INVALID; }
    if (N < 0 || N > 2147483647LL) { set_error("N outside [0, 2^31-1]"); return BNOS_E_RANGE; }
    if (N > 0 && !data) { set_error("data is NULL"); return BNOS_E_INVALID; }
    if (n < 1 || n > 64) { set_error("n outside [1, 64]"); return BNOS_E_RANGE; }
    if (K < 0 || K > n - 1 || K > kMaxK) { set_error("K outside [0, min(n-1, 6)]"); return BNOS_E_RANGE; }
    if (!(ess > 0.0) || !std::isfinite(ess)) { set_error("ess must be finite and > 0"); return BNOS_E_INVALID; }
    bnos_build_opts o;
    std::memset(&o, 0, sizeof(o));
    if (opts) o = *opts;
    for (int r = 0; r < 4; ++r)
        if (o.reserved[r] != 0) { set_error("opts.reserved must be zero"); return BNOS_E_INVALID; }
    if (o.data_on_device != 0 && o.data_on_device != 1) { set_error("data_on_device must be 0 or 1"); return BNOS_E_INVALID; }
    const bool dev_data = o.data_on_device == 1;
    if (o.prior_mode != 0 && o.prior_mode != 1) { set_error("prior_mode must be 0 or 1"); return BNOS_E_INVALID; }
    if (o.count_mode != 0 && o.count_mode != 1) { set_error("count_mode must be 0 or 1"); return BNOS_E_INVALID; }
    if (!std::isfinite(o.log_gamma)) { set_error("log_gamma must be finite"); return BNOS_E_INVALID; }
    for (int v = 0; v < n; ++v)
        if (arities[v] < 1 || arities[v] > 255) { set_error("arity outside [1, 255]"); return BNOS_E_RANGE; }
    for (int64_t t = 0; t < (dev_data ? 0 : N); ++t)        // device data: checked on the device
        for (int v = 0; v < n; ++v) {
            int x = data[t * n + v];
            if (x < 0 || x >= arities[v]) {
                char buf[128];
                std::snprintf(buf, sizeof buf, "state %d of node %d in sample %lld is outside [0, %d)", x, v,
                              (long long)t, arities[v]);
                set_error(buf);
                return BNOS_E_INVALID;
            }
        }
    if (prior) {
        for (int i = 0; i < n; ++i)
            for (int m = 0; m < n; ++m) {
                if (i == m) continue;
                float x = prior[i * n + m];
                bool ok = std::isfinite(x) && (o.prior_mode == 0 ? (x >= -1.f && x <= 1.f) : (x >= 0.f && x <= 1.f));
                if (!ok) { set_error("prior entry NaN or out of range"); return BNOS_E_INVALID; }
            }
    }
    // Largest contingency table: r_i times the K largest arities among the other nodes.
    int max_cells = 1;
    for (int i = 0; i < n; ++i) {
        std::vector<int> o2;
        for (int m = 0; m < n; ++m) if (m != i) o2.push_back(arities[m]);
        std::sort(o2.rbegin(), o2.rend());
        int64_t c = arities[i];
        for (int j = 0; j < K && j < (int)o2.size(); ++j) c *= o2[j];
        if (c > kMaxCells) { set_error("q_i * r_i above 16384"); return BNOS_E_RANGE; }
        if (c > max_cells) max_cells = (int)c;
    }

    TableT *t = new (std::nothrow) TableT();
    if (!t) { set_error("host allocation failed"); return BNOS_E_NOMEM; }
    t->n = n;
    t->K = K;
    t->N = N;
    t->N_pad = ((N + 255) / 256) * 256;
    if (t->N_pad == 0) t->N_pad = 256;
    t->S = sets_upto(n - 1, K);
    {
        // Rows are padded to a multiple of P * 1024 entries, P the smallest power
        // of two >= the row's 1024-entry steps (and >= a requested chunk
        // length), at most 16; chunk lengths are the powers of two dividing P.
        const int64_t node_steps = (t->S + kEntriesPerStep - 1) / kEntriesPerStep;
        int st = o.chunk_steps;
        if (st != 0 && (st < 1 || st > kMaxStepsPerChunk || (st & (st - 1)) != 0)) {
            set_error("chunk_steps must be 0 or a power of two <= 16");
            delete t;
            return BNOS_E_RANGE;
        }
        int P = 1;
        while (P < kMaxStepsPerChunk && (P < node_steps || P < st)) P <<= 1;
        t->pad_steps = P;
        t->S_pad = ((node_steps + P - 1) / P) * P * kEntriesPerStep;
        if (const char *cap_s = std::getenv("BNOS_MAX_DEVICE_BYTES")) {
            const long long cap = std::atoll(cap_s);
            if (cap > 0 && t->device_bytes() > cap) {
                char buf[160];
                std::snprintf(buf, sizeof buf, "table needs %lld device bytes, above BNOS_MAX_DEVICE_BYTES = %lld",
                              (long long)t->device_bytes(), cap);
                set_error(buf);
                delete t;
                return BNOS_E_NOMEM;
            }
        }
        if (st == 0) {
            // automatic: the length that best fills whole rounds of resident blocks
            // (8 blocks of 256 threads per compute unit) for a single-order pass
            int cus = 256;
            int dev = 0;
            if (hipGetDevice(&dev) == hipSuccess) {
                int v = 0;
                if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
                    cus = v;
            }
            const int64_t slots = (int64_t)cus * 8;
            const int64_t steps_pad = t->S_pad / kEntriesPerStep;
            double best_eff = -1.0;
            st = 1;
            for (int c = 1; c <= P; c <<= 1) {
                const int64_t blocks = (int64_t)n * (steps_pad / c);
                const int64_t rounds = (blocks + slots - 1) / slots;
                const double eff = (double)(n * node_steps) / (double)(rounds * slots * c);
                if (eff >= best_eff - 1e-12) {
                    best_eff = eff;
                    st = c;
                }
            }
        }
        t->chunk_entries = st * kEntriesPerStep;
        t->chunks = (int)(t->S_pad / t->chunk_entries);
    }
    t->max_cells = max_cells;
    t->ess = ess;
    t->log_gamma = o.log_gamma;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);

    auto fail = [&](bnos_status s) {
        free_device(t);
        delete t;
        return s;
    };
    hipError_t e;
    if ((e = hipGetDevice(&t->device)) != hipSuccess) { set_error(std::string("hipGetDevice: ") + hipGetErrorString(e)); return fail(BNOS_E_DEVICE); }
    constexpr size_t kNsetsBytes = sizeof(int64_t) * 64 * 8;
#define ALLOC(ptr, bytes)                                                               \
    if ((e = hipMalloc((void **)&(ptr), (bytes))) != hipSuccess) {                      \
        set_error(std::string("hipMalloc " #ptr ": ") + hipGetErrorString(e));          \
        return fail(e == hipErrorOutOfMemory ? BNOS_E_NOMEM : BNOS_E_DEVICE);           \
    }
    ALLOC(t->d_data, (size_t)n * t->N_pad);
    ALLOC(t->d_nsets, kNsetsBytes + kHostResult + sizeof(int32_t) * (2 * n + 64));   // with the arities, uploaded together
    t->d_ar = reinterpret_cast<int32_t *>(reinterpret_cast<char *>(t->d_nsets) + kNsetsBytes);
    t->d_order = t->d_ar + 2 * n;
    t->d_result = reinterpret_cast<double *>(t->d_order + 64);
    ALLOC(t->d_prior, sizeof(double) * n * n);
    ALLOC(t->d_masks, sizeof(uint64_t) * (size_t)n * t->S_pad);
    ALLOC(t->d_scores, sizeof(float) * (size_t)n * t->S_pad);
    ALLOC(t->d_nstat, sizeof(double) * (size_t)n * 5);
    ALLOC(t->d_tand, sizeof(uint64_t) * (size_t)n * (t->S_pad / 256));
    ALLOC(t->d_tsub, sizeof(uint64_t) * (size_t)n * (t->S_pad / 64));
    ALLOC(t->d_anchor, sizeof(uint64_t) * (size_t)n * (t->S_pad / 4));
    ALLOC(t->d_tmax, sizeof(float) * (size_t)n * (t->S_pad / 256));
    ALLOC(t->d_cmask, sizeof(uint64_t) * (size_t)n * kBoundSlots);
    ALLOC(t->d_cscore, sizeof(float) * (size_t)n * kBoundSlots);
#undef ALLOC
    int8_t *d_rows = nullptr;
    float *d_prior_in = nullptr;
    int32_t *d_lut_row = nullptr, *d_den = nullptr;          // these two after d_lut in its allocation
    double *d_lut = nullptr;
    std::vector<int64_t> nsets(64 * 8, 0);
    for (int b = 0; b < 64; ++b)
        for (int k = 0; k < 8; ++k) nsets[b * 8 + k] = sets_upto(b, k);
#define CK(call)                                                                         \
    if ((e = (call)) != hipSuccess) {                                                     \
        set_error(std::string(#call) + ": " + hipGetErrorString(e));                      \
        hipFree(d_rows); hipFree(d_prior_in);                                             \
        hipFree(d_lut);                                                                   \
        return fail(BNOS_E_DEVICE);                                                       \
    }
    if (N > 0 && !dev_data) CK(hipMalloc((void **)&d_rows, (size_t)N * n));
    if (prior) CK(hipMalloc((void **)&d_prior_in, sizeof(float) * n * n));
    CK(hipMemsetAsync(t->d_data, 0, (size_t)n * t->N_pad, st));
    if (N > 0 && !dev_data) CK(hipMemcpyAsync(d_rows, data, (size_t)N * n, hipMemcpyHostToDevice, st));
    if (prior) CK(hipMemcpyAsync(d_prior_in, prior, sizeof(float) * n * n, hipMemcpyHostToDevice, st));
    std::vector<int32_t> ar_magic(arities, arities + n);     // the arities, then their magic numbers (divmod_small)
    for (int v = 0; v < n; ++v) ar_magic.push_back(arities[v] > 1 ? (int32_t)(uint32_t)(0x100000000ull / arities[v] + 1) : 0);
    nsets.resize(64 * 8 + n);
    std::memcpy(nsets.data() + 64 * 8, ar_magic.data(), sizeof(int32_t) * 2 * n);
    CK(hipMemcpyAsync(t->d_nsets, nsets.data(), kNsetsBytes + sizeof(int32_t) * 2 * n, hipMemcpyHostToDevice, st));
    if (N > 0) {
        int64_t tot = N * n;
        int blocks = (int)std::min<int64_t>((tot + 255) / 256, 1 << 16);
        if (dev_data) {                          // the caller's device rows: check their states first
            unsigned *d_bad = nullptr;
            unsigned bad = 0;
            CK(hipMalloc((void **)&d_bad, sizeof(unsigned)));
            hipError_t e2 = hipMemsetAsync(d_bad, 0, sizeof(unsigned), st);
            if (e2 == hipSuccess) {
                hipLaunchKernelGGL(k_check_states, dim3(blocks), dim3(256), 0, st, data, N, n, t->d_ar, d_bad);
                e2 = hipGetLastError();
            }
            if (e2 == hipSuccess) e2 = hipMemcpyAsync(&bad, d_bad, sizeof(unsigned), hipMemcpyDeviceToHost, st);
            if (e2 == hipSuccess) e2 = hipStreamSynchronize(st);
            hipFree(d_bad);
            CK(e2);
            if (bad) {
                char buf[128];
                std::snprintf(buf, sizeof buf, "%u states of the device data are outside their node's arity", bad);
                set_error(buf);
                hipFree(d_prior_in);
                return fail(BNOS_E_INVALID);
            }
        }
        hipLaunchKernelGGL(k_ingest, dim3(blocks), dim3(256), 0, st, dev_data ? data : d_rows, N, n, t->N_pad,
                           t->d_data);
        CK(hipGetLastError());
    }
    hipLaunchKernelGGL(k_prior, dim3((n * n + 255) / 256), dim3(256), 0, st, d_prior_in, n, o.prior_mode,
                       t->d_prior);
    CK(hipGetLastError());
    // lnGamma lookup: the BDeu terms only take alpha = ess / d for d = q (a
    // product of at most K parent arities) and d = q * r_i; every such d up to
    // the largest q * r_i gets a row of lnG(c + alpha) - lnG(alpha), c = 0..N,
    // unless that would take more than kLutBytes (then lgamma is called inline).
    const double scale = lut_scale(ess, N, max_cells);
    {
        std::vector<char> isq(max_cells + 1, 0), isd(max_cells + 1, 0);
        std::vector<int> ar_set;
        for (int v = 0; v < n; ++v)
            if (std::find(ar_set.begin(), ar_set.end(), arities[v]) == ar_set.end()) ar_set.push_back(arities[v]);
        std::vector<int> qs = {1};
        isq[1] = 1;
        for (int depth = 0; depth < K; ++depth) {
            const size_t m = qs.size();
            for (size_t i = 0; i < m; ++i)
                for (int a : ar_set) {
                    const int64_t q = (int64_t)qs[i] * a;
                    if (q <= max_cells && !isq[q]) { isq[q] = 1; qs.push_back((int)q); }
                }
        }
        std::vector<int32_t> den, row(max_cells + 1, 0);
        for (int q : qs) {
            isd[q] = 1;
            for (int a : ar_set)
                if ((int64_t)q * a <= max_cells) isd[(int64_t)q * a] = 1;
        }
        for (int d = 1; d <= max_cells; ++d)
            if (isd[d]) { row[d] = (int32_t)den.size(); den.push_back(d); }
        constexpr int64_t kLutBytes = 256ll << 20;
        if ((int64_t)den.size() * (N + 1) * 8 <= kLutBytes) {
            const int64_t tot = (int64_t)den.size() * (N + 1);
            const int dens = (int)den.size();
            den.insert(den.end(), row.begin(), row.end());
            CK(hipMalloc((void **)&d_lut, sizeof(double) * (size_t)tot + sizeof(int32_t) * den.size()));
            d_den = reinterpret_cast<int32_t *>(d_lut + tot);
            d_lut_row = d_den + dens;
            CK(hipMemcpyAsync(d_den, den.data(), sizeof(int32_t) * den.size(), hipMemcpyHostToDevice, st));
            hipLaunchKernelGGL(k_lut, dim3((unsigned)std::min<int64_t>((tot + 255) / 256, 1 << 16)), dim3(256), 0, st,
                               d_den, dens, N, ess, scale, d_lut);
            CK(hipGetLastError());
        }
    }
    int cap = cells_cap_for(max_cells);
    t->count_mode = (d_lut && o.count_mode == 0) ? 0 : 1;
    if (t->count_mode == 0) {                    // one joint histogram per node subset
        if (waves_for_cells(cap) == 4) { CK(launch_build_joint<4>(t, st, cap, d_lut_row, d_lut, scale)); }
        else { CK(launch_build_joint<1>(t, st, cap, d_lut_row, d_lut, scale)); }
    } else {                                     // one histogram per family
        if (waves_for_cells(cap) == 4) { CK(launch_build<4>(t, st, cap, d_lut_row, d_lut, scale)); }
        else { CK(launch_build<1>(t, st, cap, d_lut_row, d_lut, scale)); }
    }
    hipLaunchKernelGGL(k_node_stats, dim3(n), dim3(1024), 0, st, t->d_scores, t->S, t->S_pad, t->d_prior, n,
                       t->d_nstat);
    CK(hipGetLastError());
    {
        const int64_t tiles = (int64_t)n * (t->S_pad / 256);
        const int64_t row_tiles = t->S_pad / 256;
        hipLaunchKernelGGL(k_tile_and, dim3((unsigned)((tiles + 3) / 4)), dim3(256), 0, st, t->d_masks,
                           t->d_scores, tiles, row_tiles, row_tiles / (4 * (int64_t)t->pad_steps), t->pad_steps,
                           t->d_tand, t->d_tsub, t->d_tmax);
        CK(hipGetLastError());
        const int64_t groups = (int64_t)n * (t->S_pad / 4);
        hipLaunchKernelGGL(k_anchor, dim3((unsigned)((groups + 255) / 256)), dim3(256), 0, st, t->d_masks, n,
                           t->S_pad, t->d_anchor);
        CK(hipGetLastError());
        const char *cap_s = std::getenv("BNOS_MAX_DEVICE_BYTES");
        CK(list_kept(t, st, cap_s ? std::atoll(cap_s) : 0));
        if (!t->d_kmask) {                       // else the kept rows gave the candidates
            hipLaunchKernelGGL(k_bound_cands, dim3(n), dim3(1024), 0, st, t->d_masks, t->d_scores, n, K, t->S,
                               t->S_pad, t->d_cmask, t->d_cscore);
            CK(hipGetLastError());
        }
    }
    CK(hipStreamSynchronize(st));
    hipFree(d_rows);
    hipFree(d_prior_in);
    hipFree(d_lut);
#undef CK
    t->magic = kMagic;
    register_handle(t);
    *out = reinterpret_cast<bnos_table>(t);
    return BNOS_OK;
}

extern "C" void bnos_table_free(bnos_table h)
{
    TableT *t = reinterpret_cast<TableT *>(h);
    if (!t || !handle_live(t)) return;
    const bool last = unregister_handle(t);
    hipDeviceSynchronize();
    t->magic = 0;
    free_device(t);
    delete t;
    if (last) trim_result_buffers();
}

extern "C" bnos_status bnos_table_info(bnos_table h, int32_t *n, int32_t *K, int64_t *S, int64_t *bytes)
{
    TableT *t = reinterpret_cast<TableT *>(h);
    if (!handle_live(t)) { set_error("invalid table handle"); return BNOS_E_STATE; }
    if (n) *n = t->n;
    if (K) *K = t->K;
    if (S) *S = t->S;
    if (bytes) *bytes = t->device_bytes();
    return BNOS_OK;
}

extern "C" bnos_status bnos_table_kept(bnos_table h, int64_t *entries)
{
    TableT *t = reinterpret_cast<TableT *>(h);
    if (!handle_live(t)) { set_error("invalid table handle"); return BNOS_E_STATE; }
    if (!entries) { set_error("NULL argument"); return BNOS_E_INVALID; }
    *entries = t->d_kmask ? t->kept_total : 0;
    return BNOS_OK;
}

extern "C" bnos_status bnos_table_export(bnos_table h, int32_t node, uint64_t *masks, float *scores, int64_t cap)
{
    TableT *t = reinterpret_cast<TableT *>(h);
    if (!handle_live(t)) { set_error("invalid table handle"); return BNOS_E_STATE; }
    if (!masks || !scores) { set_error("output is NULL"); return BNOS_E_INVALID; }
    if (node < 0 || node >= t->n) { set_error("node out of range"); return BNOS_E_RANGE; }
    if (cap < t->S) { set_error("cap below entries per node"); return BNOS_E_RANGE; }
    BNOS_HIP(hipSetDevice(t->device));
    BNOS_HIP(hipMemcpy(masks, t->d_masks + (int64_t)node * t->S_pad, sizeof(uint64_t) * t->S, hipMemcpyDeviceToHost));
    BNOS_HIP(hipMemcpy(scores, t->d_scores + (int64_t)node * t->S_pad, sizeof(float) * t->S, hipMemcpyDeviceToHost));
    return BNOS_OK;
}

extern "C" bnos_status bnos_counts(bnos_table h, int32_t Q, const int32_t *nodes, const uint64_t *masks,
                                   uint32_t *counts, int64_t cap)
{
    TableT *t = reinterpret_cast<TableT *>(h);
    if (!handle_live(t)) { set_error("invalid table handle"); return BNOS_E_STATE; }
    if (Q < 0) { set_error("Q < 0"); return BNOS_E_RANGE; }
    if (Q == 0) return BNOS_OK;
    if (!nodes || !masks || !counts) { set_error("NULL argument"); return BNOS_E_INVALID; }
    std::vector<int32_t> ar(t->n);
    BNOS_HIP(hipSetDevice(t->device));
    BNOS_HIP(hipMemcpy(ar.data(), t->d_ar, sizeof(int32_t) * t->n, hipMemcpyDeviceToHost));
    std::vector<int64_t> off(Q);
    int64_t tot = 0;
    int maxc = 1;
    for (int q = 0; q < Q; ++q) {
        int v = nodes[q];
        if (v < 0 || v >= t->n) { set_error("query node out of range"); return BNOS_E_RANGE; }
        uint64_t m = masks[q];
        if (t->n < 64 && (m >> t->n)) { set_error("query mask names a node >= n"); return BNOS_E_INVALID; }
        if ((m >> v) & 1ull) { set_error("query mask contains its own node"); return BNOS_E_INVALID; }
        if (__builtin_popcountll(m) > t->K) { set_error("query mask has more than K members"); return BNOS_E_RANGE; }
        int64_t c = ar[v];
        for (int b = 0; b < t->n; ++b) if ((m >> b) & 1ull) c *= ar[b];
        off[q] = tot;
        tot += c;
        if (c > maxc) maxc = (int)c;
    }
    if (tot > cap) { set_error("cap below total cells"); return BNOS_E_RANGE; }
    int32_t *d_nodes = nullptr;
    uint64_t *d_masks = nullptr;
    int64_t *d_off = nullptr;
    uint32_t *d_out = nullptr;
    hipError_t e = hipSuccess;
    auto cleanup = [&]() { hipFree(d_nodes); hipFree(d_masks); hipFree(d_off); hipFree(d_out); };
#define CK(call) if ((e = (call)) != hipSuccess) { set_error(std::string(#call) + ": " + hipGetErrorString(e)); cleanup(); return BNOS_E_DEVICE; }
    CK(hipMalloc((void **)&d_nodes, sizeof(int32_t) * Q));
    CK(hipMalloc((void **)&d_masks, sizeof(uint64_t) * Q));
    CK(hipMalloc((void **)&d_off, sizeof(int64_t) * Q));
    CK(hipMalloc((void **)&d_out, sizeof(uint32_t) * tot));
    CK(hipMemcpy(d_nodes, nodes, sizeof(int32_t) * Q, hipMemcpyHostToDevice));
    CK(hipMemcpy(d_masks, masks, sizeof(uint64_t) * Q, hipMemcpyHostToDevice));
    CK(hipMemcpy(d_off, off.data(), sizeof(int64_t) * Q, hipMemcpyHostToDevice));
    int cap_cells = cells_cap_for(maxc);
    int blocks = (int)std::min<int64_t>((Q + 3) / 4, 1 << 16);
    // the counting code of the table's own build: joint histograms (count_mode 0) or per family
    const bool four = waves_for_cells(cap_cells) == 4;
    const dim3 grid((unsigned)(four ? blocks : blocks * 4)), block(four ? 256 : 64);
    const size_t lds = (four ? 4 : 1) * cap_cells * sizeof(uint32_t);
    if (t->count_mode == 0) {
        if (four) hipLaunchKernelGGL(k_counts_joint<4>, grid, block, lds, 0, t->d_data, t->N, t->N_pad, t->d_ar, t->n, Q,
                                     d_nodes, d_masks, d_off, cap_cells, d_out);
        else hipLaunchKernelGGL(k_counts_joint<1>, grid, block, lds, 0, t->d_data, t->N, t->N_pad, t->d_ar, t->n, Q,
                                d_nodes, d_masks, d_off, cap_cells, d_out);
    } else {
        if (four) hipLaunchKernelGGL(k_counts<4>, grid, block, lds, 0, t->d_data, t->N, t->N_pad, t->d_ar, Q,
                                     d_nodes, d_masks, d_off, cap_cells, d_out);
        else hipLaunchKernelGGL(k_counts<1>, grid, block, lds, 0, t->d_data, t->N, t->N_pad, t->d_ar, Q, d_nodes,
                                d_masks, d_off, cap_cells, d_out);
    }
    CK(hipGetLastError());
    CK(hipMemcpy(counts, d_out, sizeof(uint32_t) * tot, hipMemcpyDeviceToHost));
#undef CK
    cleanup();
    return BNOS_OK;
}

extern "C" bnos_status bnos_table_node_features(bnos_table h, double *out)
{
    TableT *t = reinterpret_cast<TableT *>(h);
    if (!handle_live(t)) { set_error("invalid table handle"); return BNOS_E_STATE; }
    if (!out) { set_error("out is NULL"); return BNOS_E_INVALID; }
    BNOS_HIP(hipSetDevice(t->device));
    BNOS_HIP(hipMemcpy(out, t->d_nstat, sizeof(double) * 5 * t->n, hipMemcpyDeviceToHost));
    return BNOS_OK;
}
