// Internal declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>
#include <string>
#include <vector>

#include "bnos.h"

namespace bnos {

// Largest contingency table (q_i * r_i cells) a build supports; the counting
// kernel keeps one such histogram per wavefront in LDS.
constexpr int kMaxCells = 16384;
constexpr int kMaxK = 6;

// Order-scoring geometry: 256 threads, 4 entries per thread per step, so a
// block consumes 1024 entries per step; a chunk is 1..16 steps, taken from a
// node's row at a stride of `chunks` steps (chunk c: steps c, c + chunks, ...).
constexpr int kScoreThreads = 256;
constexpr int kEntriesPerStep = 1024;
constexpr int kMaxStepsPerChunk = 16;

// Place of the summaries (tile AND, sub-tile ANDs, tile maximum) of tile w of
// step s of a row inside that row's summary arrays.  The row's steps form C
// chunks of the longest chunk length P (the row padding), chunk c holding steps
// c, c + C, c + 2C, ... as the scoring blocks take them; a chunk's summaries are
// stored together (its i-th step's tile w at (c P + i) 4 + w), so the blocks of
// that launch shape read theirs from one run of memory.  A permutation of the
// row's tiles: only where the summaries sit changes, not what they hold.
__host__ __device__ inline int64_t summary_pos(int64_t s, int w, int64_t C, int P)
{
    return ((s % C) * P + s / C) * 4 + w;
}

// Score bound of the streaming pass: a block first takes, for each of its
// orders, lower bounds on the best and the second-best consistent entry of its
// node from entries it knows the order can use (the empty set, the singletons
// of the predecessors, and kBoundCands listed top entries of the row with two
// or more members), then leaves out for that order every tile whose largest
// score is below both the second-best bound and the best bound minus
// kBoundGap nats.  Such a tile holds neither the argmax nor the second best,
// and each of its terms is below e^-60 of the largest term of the node's sum.
constexpr int kBoundCands = 192;
constexpr int kBoundSlots = 64 + kBoundCands;   // per node: slot s < 63 {slot s}, 63 the empty set, then the list
constexpr float kBoundGap = 60.0f;

// Kept entries.  A parent set m of a row can be left out of every order's
// result at build when its own subsets already rule it out: an order that can
// use m can use every subset of m, so if one of them scores kBoundGap nats
// above m and two of them score above m, m is neither the best nor the second
// best of any order that can use it and its term is below e^-kBoundGap of the
// largest one -- the score bound's own criterion, from subsets instead of
// candidates, once for all orders.  A build therefore lists each row's other
// entries, the kept ones, apart: at n = 60, K = 4, N = 5,000 they are 1,200 to
// 6,200 of 489,406 per row on average, depending on the data, with single rows
// of 100,000.  A table that keeps more than kept_mean() per row on average (few
// samples of binary variables: nearly all of them) stays with the streaming pass,
// which shares each streamed tile between orders.  The lines, from 1,044 tables of 16 to
// 60 nodes drawn below them, scored both ways: with up to 6,144 kept entries per row
// one order takes 0.68 times the streamed time (geometric mean; over 5% more on 15 of 906
// tables), 256 orders 0.25 times; whole rows cross over near there (256 orders: 5,036 of 5,036
// entries kept 29 / 28 us, 6,018 of 6,018 38 to 49 / 40 to 44, 7,547 of 7,547 43 / 36).
// Above it rows are long enough to be streamed in many tiles: with 6,144 to 16,384, at most a
// sixteenth of the row, 0.43 times for one order and 0.23 for 256 (over 5% more on 11
// and none of 138; eight orders on 19, up to 2.3 times: tables with one row of 400 steps and
// more); 18,184 of 231,526 entries 30 / 30 and 134 / 512 us, 39,150 of 489,406 68 / 91 and 245 / 857.
constexpr int kKeptMeanLow = 6144, kKeptMeanHigh = 16384;
constexpr int64_t kept_mean(int64_t S)
{
    return S / 16 < kKeptMeanLow ? kKeptMeanLow : (S / 16 > kKeptMeanHigh ? kKeptMeanHigh : S / 16);
}
// Steps of all kept rows up to which uniform chains run on them, from S entries per row; see
// chains_fold_kept.
constexpr int64_t kept_chain_steps(int C, int64_t S)
{
    if (C >= 16) return INT64_MAX;
    const int64_t least = C < 4 ? 600 : 1600, share = S / (C < 4 ? 256 : 100);
    return least > share ? least : share;
}
constexpr int kKeptCap = 1 << 19;         // entries of one row
constexpr int kKeptRun = 16384;           // sort keys of one block: 128 KB of LDS
constexpr int kKeptTiles = 4;             // 64-entry tiles a wavefront takes per step; rows are padded to whole steps
constexpr int64_t kKeptSubsetCap = (int64_t)1 << 26;   // (node, subset) records of the build's pass over subsets

// Partial-reduction record written by each scoring block (one per order).
struct Partial {
    float m, s;          // running max and sum of exp(x - m) over consistent entries
    float best, second;  // top-1 score and best score among the others
    uint64_t bmask;      // mask of the top-1 entry
};

struct TableT {
    uint32_t magic = 0;
    int n = 0, K = 0;
    int64_t N = 0, N_pad = 0;
    int64_t S = 0, S_pad = 0;       // entries per node before / after padding
    int chunk_entries = 0;          // entries per scoring block
    int chunks = 0;                 // scoring blocks per node = S_pad / chunk_entries
    int pad_steps = 1;              // rows are padded to a multiple of pad_steps * 1024 entries
    int max_cells = 0;
    int count_mode = 0;             // counting code the build used: 0 joint histograms, 1 per family
    double ess = 1.0, log_gamma = 0.0;
    int device = 0;

    uint8_t *d_data = nullptr;      // column-major [n][N_pad]
    int32_t *d_ar = nullptr;        // [n]
    double *d_prior = nullptr;      // [n][n] prior term in nats (0 where none)
    int64_t *d_nsets = nullptr;     // [64][8] number of masks over `bit` bits with <= k members
    uint64_t *d_masks = nullptr;    // [n][S_pad]
    float *d_scores = nullptr;      // [n][S_pad]
    double *d_nstat = nullptr;      // [n][5]: prior row sum, prior column sum, max, mean, sd of the row
    uint64_t *d_tand = nullptr;     // [n * S_pad / 256]: AND of the masks of each 256-entry tile
    uint64_t *d_tsub = nullptr;     // [n * S_pad / 64]: AND of the masks of each 64-entry sub-tile
    bool tile_skip = true;
    uint64_t *d_anchor = nullptr;   // [n * S_pad / 4]: slot-space mask of every 4th entry
    bool computed_masks = true;     // one-order blocks compute masks from the anchors
    float *d_tmax = nullptr;        // [n * S_pad / 256]: largest score of each tile
    uint64_t *d_cmask = nullptr;    // [n][kBoundSlots]: bound candidates (node-space mask; ~0 for none)
    float *d_cscore = nullptr;      // [n][kBoundSlots]: their scores (-inf for none)
    bool score_bound = true;        // one-order blocks skip tiles by the score bound

    // kept entries (null when the table has none listed): row i's klen[i] sit from entry
    // klen[2 n + i] on, in descending score, equal scores in ascending mask order, padded with
    // (~0, -inf) to a multiple of 64 * kKeptTiles
    uint64_t *d_kmask = nullptr;    // [kept_cap]
    float *d_kscore = nullptr;      // [kept_cap]
    int32_t *d_klen = nullptr;      // [4][n]: kept entries, the nodes in descending order of them, first entries, -
    float *d_kpm = nullptr;         // [n][n]: largest kept score of row i among the sets holding node m
    uint8_t *d_kept = nullptr;      // [n * S_pad / 4]: bit e of byte g set when entry 4 g + e is kept
    int64_t kept_cap = 0;           // entries the arrays hold
    int64_t kept_total = 0;         // kept entries of all rows
    int64_t kept_steps = 0;         // scan steps of all kept rows
    int kept_steps_max = 0;         // and of the longest one

    // bnos_score_order's buffers, held by one call at a time, after the arities
    std::mutex host_mu;
    int32_t *d_order = nullptr;     // [64]
    double *d_result = nullptr;     // two sums, then a mask per node

    // order-scoring workspace: per (order, node, chunk) partial reductions
    void *d_part = nullptr;
    int64_t part_bytes = 0;         // capacity in bytes
    void *d_kpart = nullptr;        // and of the kept rows: per (order, node) one
    int64_t kpart_bytes = 0;

    // kernel timing: a ring of kEventRing event pairs, created when timing is
    // first enabled; launches in flight occupy ev_count slots from ev_head on
    static constexpr size_t kEventRing = 256;
    bool timing = false;
    int timing_every = 1;           // every timing_every-th launch carries events
    int64_t timing_seen = 0;        // scoring launches since timing was enabled
    std::vector<hipEvent_t> ev_start, ev_stop;
    size_t ev_head = 0, ev_count = 0;
    double timed_ms = 0.0;
    int64_t timed_launches = 0;
    std::vector<int64_t> ev_passes;     // table passes of the launch in each slot
    int64_t timed_passes = 0;

    // autotuned per batch-size bucket (1, 2-3, 4-7, 8-15, 16+); 0 = default
    int tuned_bt[5] = {0, 0, 0, 0, 0};   // orders per scoring block
    int tuned_cs[5] = {0, 0, 0, 0, 0};   // chunk length in 1024-entry steps
    int tuned_gather[5] = {0, 0, 0, 0, 0};   // 1: score by enumerating the consistent sets (K <= 4)

    int64_t device_bytes() const;
    static int bucket(int B) { return B >= 16 ? 4 : (B >= 8 ? 3 : (B >= 4 ? 2 : (B >= 2 ? 1 : 0))); }
    // Chunk length (entries) and chunks per node used for a launch of B orders:
    // the autotuned length of B's bucket; else for 8+ orders the longest chunk
    // (a block's fixed cost -- tile summaries, predecessor masks, the per-order
    // reductions -- is then spread over the most entries, and the orders
    // already fill the grid); else the length chosen at build time.
    int chunk_entries_for(int B) const
    {
        const int cs = tuned_cs[bucket(B)];
        if (cs > 0) return cs * 1024;
        return B >= 8 ? pad_steps * 1024 : chunk_entries;
    }
    int chunks_for(int B) const { return (int)(S_pad / chunk_entries_for(B)); }
    // Chain sweeps of C chains have their own launch shape (bnos_chains_autotune /
    // bnos_chains_set_launch) per chain-count bucket; 0 = the scoring shape of a
    // batch of C orders, except that the orders per block follow pick_bt.
    int chain_bt[5] = {0, 0, 0, 0, 0};
    int chain_cs[5] = {0, 0, 0, 0, 0};
    int chain_chunk_entries_for(int C) const
    {
        const int cs = chain_cs[bucket(C)];
        return cs > 0 ? cs * 1024 : chunk_entries_for(C);
    }
    int chain_chunks_for(int C) const { return (int)(S_pad / chain_chunk_entries_for(C)); }
    // partials of one launch: [B][chunks][n], with n slots per order in gather mode; a chain
    // sweep of B chains writes [B][chain chunks][n]
    int64_t partial_bytes_for(int B) const
    {
        int c = chunks_for(B) > n ? chunks_for(B) : n;
        if (chain_chunks_for(B) > c) c = chain_chunks_for(B);
        c += d_kmask ? 1 : 0;                    // the kept entries' slot
        return (int64_t)B * n * c * (int64_t)sizeof(Partial);
    }
    // the partials, then (256-byte aligned) each order's score-bound cut per node
    int64_t cuts_offset_for(int B) const { return (partial_bytes_for(B) + 255) & ~(int64_t)255; }
    int64_t workspace_bytes_for(int B) const { return cuts_offset_for(B) + (int64_t)B * n * (int64_t)sizeof(float); }
    bool gather_for(int B) const { return K <= 4 && tuned_gather[bucket(B)] != 0; }
    // the kept rows alone serve scoring and chains (with the score bound off, the streaming pass
    // adds the other entries)
    bool kept_rows() const { return d_kmask != nullptr && score_bound && tile_skip; }
    // whether C chains fold their kept rows apart from the other entries, with the score bound on (where
    // they need nothing else) and off alike, so that both add FP32 sums in the same order.  An
    // iteration on kept rows takes the longer the more steps they have, and little more for more
    // chains; streamed, it takes the longer the longer the rows, and the more chains.  Kept / streamed us
    // per iteration: 57 nodes, 1,665 steps, 1 chain 48 / 31, 4 chains 48 / 44, 16 48 / 79, 256 52 / 314;
    // 45 nodes and 14,235 entries per row, 753 steps, 26 / 21, 28 / 25, 28 / 37, 31 / 62; 60 nodes, 1,480 steps,
    // 1 chain 30 / 61.  Of the 1,044 tables of kept_mean(), on this side of the lines 1 (table, count) pair
    // is over 5% slower kept for 1 to 3 chains and 24 (of 3,132) are for 4 to 15; with one line of 1,600
    // steps below 4 chains and none above it was 65 and 39.  16 chains and more always take them: 7 of
    // 3,132 are slower, up to 1.6 times, and a call on many tables waits for those it streams (32 tables
    // of 20 to 60 nodes, 64 chains: 61 us per iteration, 114 with the longest few streamed).  The learned
    // proposal's streamed step takes 40 to 60 us alone: on 347 tables of 500 kept steps and more, one
    // chain is slower kept on 8.
    bool chains_fold_kept(int C, bool learned) const
    {
        return d_kmask != nullptr && (learned || kept_steps <= kept_chain_steps(C, S));
    }
    // whether they run on the kept rows alone
    bool kept_chains(int C, bool learned) const { return kept_rows() && chains_fold_kept(C, learned); }
    int64_t kept_bytes() const
    {
        return kept_cap * 12 + (int64_t)n * 16 + (int64_t)n * n * 4 + (int64_t)n * (S_pad / 4);
    }
};

// Wavefront reductions on the data-parallel-primitive (DPP) lane network:
// quad permutes (lane ^ 1, lane ^ 2), row shifts by 4 and 8 and the two row
// broadcasts (lane 15 of a row to the next row, lane 31 to rows 2 and 3) leave
// the reduction of all 64 lanes in lane 63, one VALU instruction per level; a
// lane whose source does not exist reads the identity.  The association is
// fixed, so the result does not depend on scheduling; readlane makes it uniform.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v, uint32_t identity)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)identity, (int)v, CTRL, 0xf, 0xf, false);
}

// Sum of a 64-bit integer over the wavefront, uniform.
template <int CTRL>
__device__ __forceinline__ uint64_t dpp_u64(uint64_t v)
{
    return ((uint64_t)dpp_u32<CTRL>((uint32_t)(v >> 32), 0u) << 32) | dpp_u32<CTRL>((uint32_t)v, 0u);
}
__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v)
{
    v += dpp_u64<0xb1>(v);
    v += dpp_u64<0x4e>(v);
    v += dpp_u64<0x114>(v);
    v += dpp_u64<0x118>(v);
    v += dpp_u64<0x142>(v);
    v += dpp_u64<0x143>(v);
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), 63) << 32) |
           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 63);
}

constexpr size_t kHostResult = sizeof(double) * 2 + sizeof(uint64_t) * 64;
constexpr uint32_t kMagic = 0xB0A5C0DEu;

void set_error(const std::string &msg);
bool handle_live(const TableT *t);
void register_handle(TableT *t);
bool unregister_handle(TableT *t);     // true when it was the last one
void trim_result_buffers();            // after that: see take_result_buffer

}  // namespace bnos

#define BNOS_HIP(call)                                                               \
    do {                                                                             \
        hipError_t e_ = (call);                                                      \
        if (e_ != hipSuccess) {                                                      \
            bnos::set_error(std::string(#call) + ": " + hipGetErrorString(e_));     \
            return BNOS_E_DEVICE;                                                    \
        }                                                                            \
    } while (0)
