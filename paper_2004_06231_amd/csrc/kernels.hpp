// Launchers of the HIP kernels (device code: leaf_forward, einsum_forward, einsum_backward, statistics, update and
// sampling .hip).  All pointers
// are device pointers; every launcher only enqueues work on `stream`.
#pragma once
#include <hip/hip_runtime.h>
#include <algorithm>
#include <cstdint>

#include "../../include/einet.h"

namespace einet_impl {

// Index tables of the plan: one int32 vector each on the host (Plan) and one
// pointer each into the bound workspace on the device (DevTables).  leaf_logc holds
// the float32 bit patterns of log C(N, v), v = 0..N, for binomial leaves.
#define EINET_TABLES(X)                                                                                    \
    X(ein_left) X(ein_right) X(ein_out) X(ein_kout) X(ein_woff) X(ein_part)                                  \
    X(ein_rec) X(ein_brec) X(leaf_gsrc)                                                                               \
    X(mix_node) X(mix_kout) X(mix_cptr) X(mix_child) X(mix_voff) X(mix_rec)                                \
    X(leaf_node) X(leaf_replica) X(leaf_sptr) X(leaf_var) X(lv_leaf) X(lv_var)                             \
    X(rb_pblk) X(row_off) X(row_len) X(leaf_logc)                         \
    X(sr_node) X(sr_pptr) X(sr_item) X(sr_mix) X(sr_layer_ptr) X(rb_rec) X(sr_rec) X(root_rec)

struct DevTables {
#define X(name) const int32_t* name;
    EINET_TABLES(X)
#undef X
};

struct Dims {
    int B, D, C, R, K, T, TD, family;
    int P;   // leaf parameter: trials of a binomial leaf (1 for Bernoulli), values of a categorical leaf
    int nodes;   // nodes of the activation arena
};

void launch_leaf_derive(const float* phi, float* theta, const Dims& d, hipStream_t s);
// A [node][B][K] float32 holds residuals, Off [node][B] float64 the offsets: log-density = Off + A
void launch_leaf_forward(const DevTables& t, int n_leaves, int max_scope, const float* x, const uint8_t* mask,
                         int mask_mode, const float* theta, float* A, double* Off, const Dims& d, hipStream_t s);
// logp (may be NULL): the launch that produces the root value also writes it there.  full_k: every item of the
// launch has K output entries (all layers but the root's).
void launch_einsum_forward(const DevTables& t, int first, int count, bool full_k, const float* params, float* A,
                           double* Off, float* amax, float* logp, const Dims& d, hipStream_t s);
// Every einsum item also has a record of EIN_REC_INTS ints in ein_rec, which a kernel gets with one scalar load: left node,
// right node, node of its output, offset of W.
constexpr int EIN_REC_INTS = 4;
// A mixing item with at most MIX_REC_CHILDREN partitions also has a record of MIX_REC_INTS ints in mix_rec:
// node, entries, offset of its weights, number of partitions, then the nodes of the partitions.  The kernel gets
// all of it with one request instead of walking three tables one after the other.
constexpr int MIX_REC_CHILDREN = 8, MIX_REC_INTS = 16;
// max_children: the largest number of partitions of a region of these items
void launch_mixing_forward(const DevTables& t, int first, int count, int max_children, const float* params, float* A,
                           double* Off, float* logp, const Dims& d, hipStream_t s);

// The top of the circuit in one launch each way.  The top einsum layer holds exactly the partitions of the root (a
// single output entry each); root_rec lists them: number of partitions, the root's node, the offset of its mixing
// weights (-1: one partition), unused, then ROOT_REC_STRIDE ints per partition: einsum item, left node, right node,
// node of the partition's own output (the root's node when it is the only one), offset of W, position among the
// root's mixing weights, first of its posterior blocks.
constexpr int ROOT_REC_STRIDE = 7;
// Row stride (floats) of the LDS copies of these kernels: a multiple of 4 whose quarter is odd, so that 16-byte reads
// of eight consecutive rows fall into different banks.
#if defined(__HIPCC__)
__host__ __device__
#endif
inline int root_row_stride(int K) {
    const int k4 = (K + 3) & ~3;
    return ((k4 >> 2) & 1) ? k4 : k4 + 4;
}
// LDS of the bottom-up kernel: per wave a copy of W [K][stride] and of eR [samples][stride], then offset (float64) and
// residual of every partition for the workgroup's samples, and the mixing weight of every partition.
constexpr int ROOT_FWD_WAVES = 8, ROOT_FWD_SAMPLES = 4;
inline size_t root_forward_lds_bytes(int K, int n_partitions) {
    const size_t ks = (size_t)root_row_stride(K);
    return sizeof(float) * ROOT_FWD_WAVES * (K * ks + ROOT_FWD_SAMPLES * ks) +
           (sizeof(double) + sizeof(float)) * (size_t)n_partitions * ROOT_FWD_SAMPLES + sizeof(float) * (size_t)n_partitions;
}
// The kernel serves the top layer whenever it fits the 160 KB of LDS of a compute unit (a few
// hundred partitions at K = 64); beyond that the general einsum and mixing kernels run.
inline bool root_kernels_apply(int n_partitions, int K) {
    return n_partitions > 0 && root_forward_lds_bytes(K, n_partitions) <= 160 * 1024;
}
// Bottom-up: S~, shifts and offsets of every partition (Eq. 3-5), then the root's mixture (App. B) and log P.
void launch_root_forward(const DevTables& t, int n_partitions, const float* params, float* A, double* Off, float* amax,
                         float* logp, const Dims& d, hipStream_t s);
struct PartialSumList;   // statistics left for the end of a top-down pass (below)
// Top-down: weight statistics (Eq. 6) and child posteriors of the root's partitions; the root's posterior is 1 and its
// mixing step is folded in.  Writes posterior blocks like launch_einsum_backward (root_bwd_groups_per_item workgroups and
// right-child blocks per item).  e_woff: the weight offsets of the layer's items in order.  part: root_bwd_partial_bound
// floats of scratch for the statistics blocks of shares of the chunks, or null (then the chunks are always walked in turn);
// with shares the sum of the blocks is appended to *list, not launched.
void launch_root_backward(const DevTables& t, int n_partitions, const int32_t* e_woff, float* part, PartialSumList* jobs,
                          bool accumulate, const float* params, float* stats,
                          const float* A, const double* Off, const float* amax, float* Gp, const Dims& d, hipStream_t s);

// Every top-down region also has a record of RB_REC_INTS ints in rb_rec: node, entries, number of parent blocks,
// position of its list in rb_pblk, then the first RB_REC_BLOCKS blocks, two ints each (the rest, if any, only in the list):
// block number, and the code that says whether the block is written (bwd_block_limit), in the order of their codes; at
// RB_REC_ALWAYS the number of blocks that are always written.
constexpr int RB_REC_INTS = 64, RB_REC_BLOCKS = 28, RB_REC_ALWAYS = 60;
void launch_region_assemble(const DevTables& t, int first, int count, bool is_root_layer, float* G, const float* Gp,
                            const Dims& d, hipStream_t s);

// Posterior blocks ([B][K] floats each) of an einsum item in Gp: one for its left child, then one per workgroup that takes some of
// its slices for its right child; reserved are those of the smallest batch.  A record names an item's first block.
constexpr int PS_SAMPLES = 64;       // samples of a workgroup of the top-down kernel for K up to 16
// Workgroups per (item, chunk of 128 samples) of the top-down kernel for a layer of `count` items: the slices of an item are
// spread over several workgroups where the launch would otherwise have fewer than bwd_workgroups of them (one per compute
// unit, two where they have more than one chunk's work), see bwd_whole_items.
// Workgroup grp takes slices grp*KQ/groups .. (grp+1)*KQ/groups - 1 and writes right-child block 1+grp of the item.  Larger
// batches need fewer groups: a block list holds those of the smallest, each with its code.
#if defined(__HIPCC__)
__host__ __device__
#endif
inline int bwd_workgroups(int nchunks) { return nchunks == 1 ? 256 : 512; }
// K up to 16: a workgroup that forms no statistics (beyond PS_SAMPLES samples), or has no more than two slices, has too little
// to share.  EM step of trees, K = 16, 112 items, 1000 samples, whole items and split ones: 124 and 140 us; K = 8, 64 samples, 4
// and 112 items: 38 and 42, 55 and 59.
#if defined(__HIPCC__)
__host__ __device__
#endif
inline bool bwd_whole_items(int K, int B) { return K <= 8 || (K <= 16 && B > PS_SAMPLES); }
#if defined(__HIPCC__)
__host__ __device__
#endif
inline int bwd_groups_per_item(int count, int K, int B) {
    const int kq = (K + 3) / 4, nchunks = (B + 127) / 128;
    if (bwd_whole_items(K, B)) return 1;
    const long long n = (long long)(count > 0 ? count : 1) * nchunks;
    const int target = bwd_workgroups(nchunks), g = n >= target ? 1 : target / (int)n;
    return g > kq ? kq : g;
}
// Code of right-child block 1 + q of an item in a layer of `count` items: the block is written when q < groups, that is
// when (q + 1) * count * nchunks is at most bwd_workgroups(nchunks); 0: always.  So the blocks in use are those whose code is at
// most bwd_block_limit(K, B) (one comparison per block in the kernel that adds them up; with the product in its place EM
// steps of 32x32 images, six such launches each, took 1 to 2 % longer: K = 25, one sample 167 us and 165, K = 40: 221 and 219).
inline int32_t bwd_block_code(int count, int q) { return q == 0 ? 0 : (q + 1) * count; }
inline int32_t bwd_block_limit(int K, int B) {
    const int nchunks = (B + 127) / 128;
    return bwd_whole_items(K, B) ? 0 : bwd_workgroups(nchunks) / nchunks;
}
// The top-down kernel above K = 16 (K8 = ceil(K / 8), EXACT: K is 8 K8) brings in post_slices(K8) slices of an item's weights
// at a time, whether or not the workgroup has that many left.  Row i of W that row r (0 .. 4 post_slices - 1) of the stage from
// slice `it` on is read from, and the first of the four left entries read for slice `it`: in range for slices that do not exist.
#if defined(__HIPCC__)
__host__ __device__
#endif
constexpr int post_slices(int K8) { return K8 == 3 ? 3 : K8 == 4 ? 2 : 1; }
template <int K8, bool EXACT>
#if defined(__HIPCC__)
__host__ __device__
#endif
inline int post_weight_row(int it, int r, int K) {
    const int i = 4 * it + r;
    return (EXACT && post_slices(K8) == 1) || i < K ? i : K - 1;
}
template <int K8, bool EXACT>
#if defined(__HIPCC__)
__host__ __device__
#endif
inline int post_left_entry(int it, int K) {
    const int i = 4 * it;
    return (EXACT && post_slices(K8) == 1) || i < K - 4 ? i : K - 4;
}
// Workgroups per item of the root's layer (its kernel takes all chunks in one workgroup).
inline int root_bwd_groups_per_item(int count, int K) {
    const int kq = (K + 3) / 4;
    const int g = 256 / (count > 0 ? count : 1);
    return g < 1 ? 1 : (g > kq ? kq : g);
}
// A region with one partition and one parent partition (every inner region of a random binary tree) has its
// posterior in consecutive blocks of Gp, written by that parent.  The kernel that reads the posterior of such a region adds
// them up itself, which saves the launch that would assemble G.  The source of a posterior is two ints: first block (-1:
// it is in G) and how many there are: n > 0: those of the right child of an item in a layer of n items, n <= 0: -n.
constexpr int GSRC_MAX_BLOCKS = 6;
#if defined(__HIPCC__)
__host__ __device__
#endif
inline int bwd_source_blocks(int32_t n, int K, int B) { return n > 0 ? bwd_groups_per_item(n, K, B) : -n; }

// (K = 16, few items: their posteriors have up to four blocks, which the statistics would add up again for every sample.  EM step
// of trees, 4 items, assembled and read from the blocks: 1000 samples 68.6 and 74.9 us, 300 samples 54.1 and 54.4; but 64 samples
// 39.5 and 37.4.)
inline bool bwd_reads_blocks(int count, int K) { return K != 16 || count >= 32; }

// Every einsum item has a record of EIN_BREC_INTS ints in ein_brec for the top-down pass: left node, right node, node of its
// output, its region, offset of W, offset and stride of its mixing weights (offset -1: one partition), source of its
// region's posterior (two ints), first of its own posterior blocks, unused.
constexpr int EIN_BREC_INTS = 12;
// Above K = 16 the top-down kernel also leaves the operands of an item's weight statistics in memory, sample-major:
// EIN_IMAGES images of 4 ceil(K / 4) rows of ein_image_stride(B) floats each, Q, then eR, then eL (rows beyond K and samples
// beyond the batch hold anything).
constexpr int EIN_IMAGES = 3;
#if defined(__HIPCC__)
__host__ __device__
#endif
inline int ein_image_stride(int B) { return (B + 31) & ~31; }

// What the end of a top-down pass still has to do for the statistics of the weights.  They are not needed before the
// M-step, so the launches of a pass only note it down.
// Per job (a launch whose batch was split into shares with statistics blocks of their own):
//   stats[e_woff[item] + r] (+)= sum over v < vper of part[(v * count + item) * block + r], r < block.
constexpr int PARTIAL_SUM_JOBS = 2;      // the root's layer, the layers below
struct PartialSumJob {
    const int32_t* e_woff;
    const float* part;
    int count, vper, block;
};
struct PartialSumJobs {
    PartialSumJob job[PARTIAL_SUM_JOBS];
};
// Einsum items first .. first + count - 1 (rec, woff: ein_brec and ein_woff of the first), whose weight statistics are formed
// at once.  part: ein_stat_partial_bound floats of scratch.
struct EinStatsWork {
    const int32_t *rec, *woff;
    float* part;
    const float *params, *A, *amax, *G, *Gp, *img;
    const double* Off;
    int first, count, B, K;
    int total;                       // items of all layers below the root's
    bool formed;                     // chunk by chunk, in `part`: only to be added up
};
// Few items with several chunks of 128 samples: the batch is split into shares (of whole chunks), as many as give every wave of
// the chip work of its own; above K = 16 a wave takes about three row tiles of a slice there.  Up to K = 16 the workgroups walk the
// batch 128 samples at a time (about 2 us), which a sum of blocks is worth from four chunks on: K = 16, 28 items, 1000 samples:
// 21.8 us in one share, 11.0 in four and 3.9 for the sum.
inline long long ein_stat_units(int count, int K) {
    const int kq = (K + 3) / 4;
    return (long long)count * kq * (K <= 16 ? 1 : (kq + 2) / 3);
}
inline long long ein_stat_most_shares(int count, int K, int B) {
    const long long units = ein_stat_units(count, K), nchunks = (B + 127) / 128;
    if (units == 0 || nchunks < (K <= 16 ? 4 : 2) || units > (K <= 16 ? 384 : 1024)) return 1;
    return std::min<long long>((K <= 16 ? 768 : 2048) / units, nchunks);
}
inline int ein_stat_shares(int count, int K, int B) {
    const int nchunks = (B + 127) / 128, v = (int)ein_stat_most_shares(count, K, B);
    const int cpv = v < 1 ? nchunks : (nchunks + v - 1) / v;
    return cpv < 1 ? 1 : (nchunks + cpv - 1) / cpv;
}
inline int ein_stat_share(int nshare, int B) {       // samples of a share
    const int nchunks = (B + 127) / 128;
    return nshare == 1 ? B : 128 * ((nchunks + nshare - 1) / nshare);
}
// Above K = 16 the layers take one of two forms: posteriors and statistics in one launch per layer (k_einsum_backward_fused), or
// posteriors per layer and the statistics of all layers at the end.  total: items of all layers below the root's (all layers of a model take the same
// form).  Us of an EM step, one launch per layer and the other form:
//   one chunk, 28 / 112 / 194 / 496 items: K = 22, 128 samples: 92 / 111 / 172 / 210 and 109 / 126 / 189 / 219; K = 32, 64: 89 / 100 /
//     180 / 225 and 95 / 111 / 182 / 224, 128: 101 / 123 / 208 / 282 and 107 / 132 / 201 / 252; K = 40, 16: 97 / 125 / 208 / 296 and
//     107 / 141 / 222 / 340, 128: 123 / 186 / 281 / 473 and 124 / 181 / 258 / 437;
//   256 samples, a block per chunk, 8 / 24 items: K = 20 53 / 66 and 65 / 78, K = 32 62 / 91 and 70 / 99, K = 40 77 / 109 and 85 / 119;
//     both chunks in turn, 112 / 194 items: K = 28 172 / 266 and 191 / 264, K = 36 279 / 414 and 244 / 336;
//   640 samples, a block per chunk, 4 / 8 / 16 items: K = 24 61 / 64 / 83 and 71 / 74 / 96, K = 40 75 / 103 / 143 and 82 / 106 / 143.
// More blocks than the statistics' own launch is cut into (FUSED_UNITS: up to 35 MB) pay up to K = 24 for any number of items, above for
// few:
//   200 samples, 194 / 240 items: K = 20 179 / 154 and in turn 187 / 164, K = 22 216 / 197 and 248 / 213, K = 23 223 / 206 and 254 / 219,
//     K = 24 213 / 181 and 218 / 182; 160 samples, K = 24 210 / 182 and 210 / 176;
//   500 samples, 24 / 28 / 64 items: K = 22 - / - / 132 and - / - / 145, K = 28 - / 122 / - and - / 138 / -, K = 32 103 / 133 / 168 and
//     118 / 138 / 161; 1000 samples, 24 / 28 items: K = 24 160 / 119 and 176 / 129, K = 32 141 / 166 and 156 / 161;
//   300 samples, 24 / 28 items: K = 36 121 / 145 and 127 / 145, K = 40 124 / 154 and 128 / 137, K = 44 178 / 194 and 191 / 190, K = 48 - / 227
//     and - / 207; 16 items, K = 44 142 and 157.
constexpr long long FUSED_UNITS = 6144;
inline bool fused_more_blocks(int total, int K, int nchunks) {
    const long long n = ein_stat_units(total, K) * nchunks;
    if (n == 0 || n > FUSED_UNITS) return false;
    if (K == 24) return n <= 5400;                        // (whole pieces of eight: the other form is the faster of its neighbours)
    if (K <= 32) return K < 24 || total <= 24 || (total <= 32 && n <= 4096);
    return K <= 44 && (K & 3) == 0 && total <= 24 && nchunks <= 3;
}
inline bool einsum_backward_fused(int total, int K, int B) {
    const bool quads = (K & 3) == 0;                      // (rows of other K are staged entry by entry, from registers that spill)
    if (K <= 16 || K > 48 || (K > 40 && !quads)) return false;
    const int nchunks = (B + 127) / 128;
    if (nchunks > 1) {
        if (fused_more_blocks(total, K, nchunks)) return true;
        if (ein_stat_shares(total, K, B) == nchunks) return K <= 32 || nchunks == 2 || total <= 8 || (nchunks == 3 && total <= 16);
        return nchunks == 2 && K == 28 && total <= 128;
    }
    if (total <= 32 || K <= 24) return true;
    if (total <= 128) return K <= 32 || B <= 64;
    return (K <= 28 && total <= 256) || B <= 32 || (B <= 64 && quads);
}
// Shares of the chunks in one launch per layer: as many as chunks, or all chunks in turn where that is not worth their blocks.
inline int fused_shares(int total, int K, int B) {
    const int nchunks = (B + 127) / 128;
    return nchunks > 1 && (fused_more_blocks(total, K, nchunks) || ein_stat_shares(total, K, B) == nchunks) ? nchunks : 1;
}
// Floats of scratch for the blocks of statistics of either form, for batches of up to max_B: ein_stat_shares never has more of them
// than ein_stat_most_shares for a larger batch.
inline size_t ein_stat_partial_bound(int count, int K, int max_B) {
    long long v = ein_stat_most_shares(count, K, max_B);
    if (K > 16)
        for (int n = 2; n <= (max_B + 127) / 128 && ein_stat_units(count, K) * n <= FUSED_UNITS; ++n)
            if (fused_more_blocks(count, K, n) && einsum_backward_fused(count, K, 128 * n)) v = std::max<long long>(v, n);
    return v < 2 ? 0 : (size_t)v * count * K * K * K;
}

// Floats of images (EIN_IMAGES) for batches of up to max_B, of which some take the other form
inline size_t ein_image_floats(int total, int K, int max_B) {
    int B = K <= 16 ? 0 : max_B;
    while (B > 0 && einsum_backward_fused(total, K, B)) --B;
    return (size_t)total * EIN_IMAGES * (4 * ((K + 3) / 4)) * ein_image_stride(B);
}
struct PartialSumList {
    int n = 0;
    PartialSumJobs jobs;
    EinStatsWork ein{};
};
void launch_sum_partial_stats(const PartialSumList& list, float* stats, bool accumulate, hipStream_t s);
// Posteriors of the children of a layer's items (every layer but the root's: all items have K output entries).  Notes the
// items down in *list for their statistics: the layers of a pass come from the top, so their items are one range.
// img: ein_image_floats floats; part: as in EinStatsWork, is kept in *list by the caller.
// direct: the posterior of every item's region is not in G; the kernel adds up the parent's blocks itself, as
// ein_brec says (only layers with Plan::ein_layer_direct set; then no launch_region_assemble for their regions).
void launch_einsum_backward(const DevTables& t, int first, int count, bool accumulate,
                            const float* params, float* stats, const float* A, const double* Off, const float* amax,
                            const float* G, float* Gp, float* img, PartialSumList* list, bool direct, const Dims& d,
                            hipStream_t s);
// The root's layer (n_partitions items of K^2 weights, root_bwd_groups_per_item workgroups each): a layer of so few items
// that its workgroups leave more than half of the compute units idle, with a batch of several chunks of 128 samples, is
// launched with several shares of the chunks per item.  Each writes its statistics to a block of its own, which a later
// launch adds up in a fixed order.  That launch costs about 4 us, so the split is taken only where the chunks a workgroup
// no longer walks are worth twice that: a workgroup spends roughly half of root_bwd_unit_us(K) on one chunk of one slice.
constexpr float BWD_SPLIT_PAYS_US = 8.f;
inline float root_bwd_unit_us(int K) { return 1.f + 9.f * (float)(K * K) / 1600.f; }
inline int root_bwd_virtual_items(int n_partitions, int K, int B) {
    const int groups = root_bwd_groups_per_item(n_partitions, K), wgs = n_partitions * groups, nchunks = (B + 127) / 128;
    if (wgs <= 0 || wgs > 128 || nchunks < 2) return 1;
    int v = 256 / wgs;
    if (v > nchunks) v = nchunks;
    const int cpv = (nchunks + v - 1) / v;
    const int slices = ((K + 3) / 4 + groups - 1) / groups;      // per workgroup
    if ((float)((nchunks - cpv) * slices) * 0.5f * root_bwd_unit_us(K) < BWD_SPLIT_PAYS_US) return 1;
    return (nchunks + cpv - 1) / cpv;
}
// floats of scratch that its launch needs for the blocks with any batch up to max_B (0: never split)
inline size_t root_bwd_partial_bound(int n_partitions, int K, int max_B) {
    const int wgs = n_partitions * root_bwd_groups_per_item(n_partitions, K), nchunks = (max_B + 127) / 128;
    if (wgs <= 0 || wgs > 128 || nchunks < 2) return 0;
    const int v = 256 / wgs < nchunks ? 256 / wgs : nchunks;
    return (size_t)v * n_partitions * K * K;
}
// leaf statistics and mixing statistics (independent of each other) in one launch
// direct: the leaves' posteriors are not in G; the kernels add up the parents' blocks of Gp themselves, as leaf_gsrc says
// (only with Plan::leaves_direct).
void launch_tail_backward(const DevTables& t, int n_lv, int n_leaves, int max_scope, int n_mix, int max_children,
                          const float* x, const uint8_t* mask, int mask_mode, const float* params, const float* A,
                          const double* Off, const float* G, const float* Gp, bool direct, float* stats,
                          int64_t phi_off, int64_t den_off, int64_t tot_off, const Dims& d, hipStream_t s);
// the whole M-step in one launch; the statistics of the first n_lazy_rows weight rows are left as they
// are (the next E-step overwrites them); when no E-step has run since they were last consumed
// (lazy_rows_are_zero) those rows count as zero and their weights are kept
void launch_em_update(const DevTables& t, int n_rows, int n_lazy_rows, bool lazy_rows_are_zero, float* params,
                      float* stats, float* theta,
                      int64_t phi_off, int64_t den_off, int64_t tot_off, float step, float min_var, float max_var,
                      float w_floor, const Dims& d, hipStream_t s);
void launch_fill(float* p, float value, int64_t n, hipStream_t s);
void launch_init_params(const DevTables& t, int n_rows, float* params, int64_t phi_off, uint64_t seed, float lo,
                        float hi, const Dims& d, hipStream_t s);

// ---- top-down sampling.  sel [B][nodes rounded up to a multiple of four], a byte each, holds the entry every sample uses
// at a region, -1 where the sample does not visit it (`sel` has room for an int32 per sample and node).
// u [num_partitions + num_regions][B]: the uniforms of the choices.
// evidence = false: no forward pass has run, the choices follow the weights alone.
// A sampling item (sum region) with at most SR_REC_PARTS partitions also has a record of SR_REC_INTS ints in
// sr_rec: node, number of partitions, offset of its mixing weights (-1: one partition), unused, then per partition
// SR_REC_STRIDE ints: einsum item, left node, right node, offset of W, partition number, node of the partition's
// own output (-1: the region itself), unused.  Regions with more partitions have nparts only (the kernel then walks
// the tables).
constexpr int SR_REC_INTS = 64, SR_REC_PARTS = 8, SR_REC_STRIDE = 7;
// The choices: for every region that a sample reaches, that of a partition (regions with several) and then of a pair of
// child entries.  One launch per sum layer, or one for all; layer_ptr, reach: Plan::sr_layer_ptr and Plan::sr_reach.
void launch_sample_regions(const DevTables& t, const int32_t* layer_ptr, const int32_t* reach, int num_layers,
                           int num_partitions, bool evidence, const float* params, const float* A, const double* Off,
                           const float* amax, const float* u, int num_nodes, int32_t* sel, const Dims& d, hipStream_t s);
void launch_sample_leaves(const DevTables& t, int n_lv, const float* x, const uint8_t* mask, int mask_mode,
                          const float* phi, const float* noise, const int32_t* sel, float* out, const Dims& d,
                          hipStream_t s);
// Device address, on the current device, of the library's fixed arena of EINET_STATIC_SCRATCH_BYTES bytes
// (256-byte aligned).  No allocation: the arena is part of the loaded code object.
hipError_t static_scratch_address(void** ptr);

// Streaming-copy rate (GB/s, read + written) and register-resident fp32 MFMA rates (TFLOP/s: 32x32x2; 16x16x4 with one
// and with four waves per SIMD) of the current device, best of `reps` launches each; dst also receives the loops'
// results (it needs at least EINET_PEAKS_MIN_BYTES bytes).
hipError_t measure_peaks(const void* src, void* dst, size_t bytes, int reps, double* out, hipStream_t s);

void launch_mixture_logp(const float* lp, const float* log_coef, int n_components, int B, float* out, hipStream_t s);

}  // namespace einet_impl
