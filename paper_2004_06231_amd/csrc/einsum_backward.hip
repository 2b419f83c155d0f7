// Top-down pass: posterior of the regions and of the children of the einsum items.  The weight statistics of the items
// (Eq. 6) are formed by einsum_statistics.hip, in one launch for all layers, when the posteriors of all regions are known;
// small batches have them here, with the posteriors.
#include "bf16x6.hpp"

#include <mutex>

namespace einet_impl {

namespace {

// ------------------------------------------------------------------ top-down pass, regions
// G[region][b][k] = sum of the posterior blocks its parent partitions wrote (1 at
// the root).  Element-wise, one thread per (region, b, k); summing here instead of
// scattering from the producers keeps the pass free of atomics.
__global__ void k_region_assemble(const int32_t* __restrict__ r_rec, const int32_t* __restrict__ r_pblk, int is_root,
                                  float* __restrict__ G, const float* __restrict__ Gp, int limit, int B, int K) {
    // the region's record: node, entries, number of parent blocks, start of its block list, first blocks (block number,
    // code: used if at most limit), in the order of their codes
    const int32_t* rec = r_rec + (size_t)blockIdx.x * RB_REC_INTS;
    const int node = rec[0], kout = rec[1], cnt = limit == 0 ? rec[RB_REC_ALWAYS] : rec[2];
    const int e = blockIdx.y * blockDim.x + threadIdx.x;
    if (e >= B * kout) return;
    const int b = e / kout, k = e - b * kout;
    const size_t blk = (size_t)B * K, o = (size_t)b * K + k;
    float g = is_root ? 1.f : 0.f;
    // Fourteen blocks per round, all requested before the first is added: a region of a Poon-Domingos structure
    // has a few dozen parent blocks, and one memory latency per block would be the whole kernel.  The numbers of
    // the first 28 blocks come with the record, so that the blocks are the second request, not the third.
    constexpr int RND = RB_REC_BLOCKS / 2;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        if (r * RND < cnt && (r == 0 || rec[4 + 2 * r * RND + 1] <= limit)) {
            float v[RND];
#pragma unroll
            for (int q = 0; q < RND; ++q) {
                const int32_t* en = rec + 4 + 2 * (r * RND + q);
                v[q] = r * RND + q < cnt && en[1] <= limit ? Gp[(size_t)en[0] * blk + o] : 0.f;
            }
#pragma unroll
            for (int q = 0; q < RND; ++q) g += v[q];
        }
    }
    const int32_t* list = r_pblk + 2 * rec[3];
    for (int p0 = RB_REC_BLOCKS; p0 < cnt && list[2 * p0 + 1] <= limit; p0 += 16) {   // the rest of a very long list
        float v[16];
#pragma unroll
        for (int q = 0; q < 16; ++q)
            v[q] = p0 + q < cnt && list[2 * (p0 + q) + 1] <= limit ? Gp[(size_t)list[2 * (p0 + q)] * blk + o] : 0.f;
#pragma unroll
        for (int q = 0; q < 16; ++q) g += v[q];
    }
    G[(size_t)node * blk + o] = g;
}

// ------------------------------------------------------------------ top-down pass, posteriors of the children
// For one einsum item, with Q[b,k] = G_out[b,k] / S~[b,k] (S~ the shifted sum of Eq. 4):
//   U[b,i,j]       = sum_k Q[b,k] W[k,i,j]
//   Gp_left[b,i]   = eL[b,i] sum_j U[b,i,j] eR[b,j]
//   Gp_right[b,j]  = eR[b,j] sum_i U[b,i,j] eL[b,i]
// G_out is the posterior of the item's region s times, for a region with several
// partitions, the mixing weight and S^c/S; S^c cancels against S~ (the residual of the
// item's own output is log S~), leaving
//   Q = G[s] * v * exp((Off[out] - Off[s]) - A[s])        (Off[out] = Off[s] for a single partition).
//
// U is a product with contraction k, on the bfloat16 matrix pipe at float32 precision (bf16x6.hpp).  Posteriors range over
// all exponents (Q is large where S~ is small), so the Q of a sample are multiplied by the power of two that brings the
// largest near 2^60 before they are split: entries 2^-162 below the largest keep all their bits, and the sums stay below
// 2^96 for rows of weights that add up to 1.
//
// A workgroup of four waves takes one item, 128 samples (32 per wave, two sets of 16) and a run of slices, a slice being
// four consecutive left entries i; everything but the weights is private to a wave, so the slices W[:, 4 i .., :] are
// all that goes through LDS, SG of them at a time (transposed on the way: the contraction runs along k), the next ones
// in flight in registers.  A tile has 16 rows, four j (lane group kg holds j = 4 t + kg) x four i (the accumulators of a
// lane), so both reductions are in-lane: the right child's entries stay in registers over the workgroup's slices, the
// left child's four meet once per slice over the four lane groups.
// The items of a short launch are cut into several workgroups (bwd_groups_per_item): each writes the left child's entries of its
// slices and a block of its own with its share of the right child's, which the reader adds up.
//
// Bound by latency: at two waves per SIMD the counters show the matrix pipes busy 11 to 15 % of a launch of 128 samples and waves
// that wait for something 42 % of their time (at 1000 samples 27 to 34 % and 37 to 40 %); a wave's products wait for its splits and
// its loads.  Us of a launch (in brackets: kernel that formed the statistics in the same launch, float32 matrix instructions): K = 40, 128 samples,
// 20 / 40 / 50 / 60 items: 12.8 / 16.8 / 17.8 / 21.9 (16.8 / 29.3 / 30.8 / 40.2), K = 40, 1000 samples: 33.8 / 66.9 / 70.6 / 72.5
// (104 / 200 / 207 / 278); K = 30, 100 samples, 20 / 40 / 80 items: 12.8 / 14.0 / 18.0 (15.6 / 25.4 / 37.8).
template <int K8>
struct PostLayout {
    using X = X6<K8>;
    static constexpr int KP = X::KP, NT = X::NT;
    static constexpr int SG = post_slices(K8);            // slices per stage
    static constexpr int TU = X::UNITS + 1;               // 16-byte units of a tile: consecutive tiles in different banks
    static constexpr int SLICE = NT * TU;                 // units of a slice
    static constexpr int NBUF = 2 * SG * SLICE * 16 <= 160 * 1024 ? 2 : 1;
    static constexpr size_t LDS_BYTES = (size_t)NBUF * SG * SLICE * 16;
    static constexpr int NI = SG * K8 * 4 * NT;           // work items of a stage: (slice, octet of k, i, four j)
    static constexpr int NL = (NI + 255) / 256;
    static constexpr int NO = X::NQ + X::R2 + X::R1;      // octets of Q that a lane's operand needs
    static constexpr int NP = (NT + 3) / 4;               // 16-byte pieces of a row that a lane loads
    static constexpr int WAVES = K8 <= 5 ? 2 : 1;   // per SIMD, so that no register spills
};

// ------------------------------------------------------------------ the same, K up to 16
// A whole item fits a workgroup and its launches are bound by their chain of requests and by the instructions that a
// compute unit fetches once, so this kernel is kept short: float32 operands on v_mfma_f32_16x16x4_f32 (nothing to split or
// to scale), a wave per 16 samples, the weights of the workgroup's slices in LDS as they are in memory.  Rows come in as one 16-byte
// piece per lane (lane group g: entries 4 g .. 4 g + 3) and are transposed over the lane groups into the operand layout,
// outputs leave the same way.
// Us of a launch (in brackets as above): K = 10, 100 samples, 20 / 80 / 160 / 320 / 640 / 1280 items: 5.6 / 5.5 / 6.5 / 8.0 / 10.4 /
// 16.7 (8.2 / 8.2 / 14.4 / 17.2 / 27.5 / 43.0); K = 16, 256 samples, 40 items: 6.1.
// Few items: their slices over several workgroups as above.  EM step of 32x32 images (five layers of 20 to 60 items), one / 64
// samples, K = 10: 99 / 111 us, K = 13: 104 / 115, K = 16: 94 / 108; with a workgroup per item 104 / 113, 114 / 123, 104 / 114 (99 / 111,
// 100 / 113, 98 / 106).
// QUADS: K is 4 KQ (see load_piece).
template <int KQ>
struct PostSmall {
    static constexpr int KP = 4 * KQ;
    static constexpr int SI = 20;                         // row stride: 20 modulo 32, so that four rows i of four entries j ..
    static constexpr int S = KP * SI + (KP * SI % 32 == 16 ? 0 : 16);   // .. and two k, 16 modulo 32 apart, hit 32 banks
};

// STATS (batches of PS_SAMPLES at most): the workgroup has all operands of its item's weight statistics (Eq. 6) and forms
// them too, which saves their launch: a wave contracts its 16 samples, the four waves' sums meet in LDS.
// SPLIT: several workgroups per item (with STATS only, see bwd_groups_per_item).
template <int KQ, bool QUADS, bool STATS, bool ACCUM, bool SPLIT>
__global__ __launch_bounds__(256, STATS && KQ > 2 ? 2 : 4) void k_einsum_posterior_small(
    const int32_t* __restrict__ e_rec, const float* __restrict__ params, float* __restrict__ stats, const float* __restrict__ A,
    const double* __restrict__ Off, const float* __restrict__ amax, const float* __restrict__ G, float* Gp, int item0,
    int nchunks, int ngr_, int direct, int B, int K_) {
    using LY = PostSmall<KQ>;
    constexpr int SI = LY::SI, S = LY::S, KP = LY::KP;
    __shared__ __attribute__((aligned(16))) float wl[KP * S];
    // a wave's rows of Q, eR and eL ([16 samples][16]), later the waves' sums of KQ tiles
    __shared__ __attribute__((aligned(16))) float sx[STATS ? 4 * (KQ > 3 ? KQ : 3) * 256 : 4];
    float* sQ = sx + (STATS ? (threadIdx.x >> 6) * 3 * 256 : 0);
    const int K = QUADS ? KP : K_;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c16 = lane & 15, g = lane >> 4;
    const int vb = xcd_contiguous_block();
    const int ngr = SPLIT ? ngr_ : 1, grp = vb % ngr, chunk = (vb / ngr) % nchunks, li = vb / (ngr * nchunks);
    const int it0 = SPLIT ? grp * KQ / ngr : 0, it1 = SPLIT ? (grp + 1) * KQ / ngr : KQ;       // blocks of four left entries
    const int32_t* rec = e_rec + (size_t)li * EIN_BREC_INTS;
    const int left = rec[0], right = rec[1], out = rec[2], reg = rec[3], voff = rec[5], vstr = rec[6], src = rec[7], srcn = rec[8];
    const size_t blk = (size_t)B * K;
    const float* W = params + rec[4];

    // ---- the weights: pieces of rows (k, i), consecutive threads consecutive pieces; what does not exist is zeros
    constexpr int NW = (KP * KP * KQ + 255) / 256;
    const int ni = 4 * (it1 - it0), npiece = KP * ni * KQ;
    const float rni = 1.f / (float)ni;
    auto piece_of = [&](int f, int& k, int& i, int& p) {
        const int r = f / KQ;
        p = f - r * KQ;
        k = SPLIT ? (int)(((float)r + 0.5f) * rni) : r / KP;          // r / ni (r < 256)
        i = 4 * it0 + r - k * ni;
    };
    float w[NW][4];
#pragma unroll
    for (int x = 0; x < NW; ++x) {
        if (256 * x < npiece) {
            int k, i, p;
            piece_of(min(tid + 256 * x, npiece - 1), k, i, p);
            const int row = QUADS ? k * K + i : min(k, K - 1) * K + min(i, K - 1);
            load_piece<KQ, QUADS>(W + (size_t)row * K, p, K, w[x]);
        }
    }
    // ---- this lane's piece of its sample's rows
    const int b = chunk * PS_SAMPLES + 16 * wave + c16, bc = min(b, B - 1);
    const bool active = chunk * PS_SAMPLES + 16 * wave < B;
    const int gp = min(g, KQ - 1);
    float q[4], er[4], el[KP];
    if (active) {
        const size_t row = (size_t)bc * K;
        const float* Gs = (direct ? Gp + (size_t)src * blk : G + (size_t)reg * blk) + row;
        float a[4], lp[KQ][4], v[4] = {1.f, 1.f, 1.f, 1.f};
        load_piece<KQ, QUADS>(Gs, gp, K, q);
        load_piece<KQ, QUADS>(A + (size_t)reg * blk + row, gp, K, a);
        load_piece<KQ, QUADS>(A + (size_t)right * blk + row, gp, K, er);
#pragma unroll
        for (int p = 0; p < KQ; ++p) load_piece<KQ, QUADS>(A + (size_t)left * blk + row, p, K, lp[p]);
        const float al = amax[(size_t)(item0 + li) * 2 * B + bc], ar = amax[((size_t)(item0 + li) * 2 + 1) * B + bc];
        const double* Oo = Off + (size_t)out * B;
        const double* Os = Off + (size_t)reg * B;
        const float dd = (float)(Oo[bc] - Os[bc]);
        if (voff >= 0) {
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = params[voff + min(4 * gp + c, K - 1) * vstr];
        }
        // (a posterior may be in several blocks, at most KQ)
        const int gcnt = direct ? bwd_source_blocks(srcn, K, B) : 1;
        float more[KQ][4];
#pragma unroll
        for (int x = 1; x < KQ; ++x)
            if (x < gcnt) load_piece<KQ, QUADS>(Gs + x * blk, gp, K, more[x]);
#pragma unroll
        for (int x = 1; x < KQ; ++x)
            if (x < gcnt) {
#pragma unroll
                for (int c = 0; c < 4; ++c) q[c] += more[x][c];
            }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const bool in = (QUADS && KQ == 4) || (4 * g + c < K);
            const float qv = q[c] * v[c] * __expf(dd - a[c]);
            q[c] = in && q[c] != 0.f && b < B ? qv : 0.f;
            er[c] = in ? __expf(er[c] - ar) : 0.f;
        }
#pragma unroll
        for (int p = 0; p < KQ; ++p)
#pragma unroll
            for (int c = 0; c < 4; ++c) el[4 * p + c] = QUADS || 4 * p + c < K ? __expf(lp[p][c] - al) : 0.f;
        if constexpr (STATS) {
            if (g < KQ) {
                *reinterpret_cast<floatx4*>(sQ + c16 * 16 + 4 * g) = floatx4{q[0], q[1], q[2], q[3]};
                *reinterpret_cast<floatx4*>(sQ + 256 + c16 * 16 + 4 * g) = floatx4{er[0], er[1], er[2], er[3]};
            }
            if (g == 0) {
#pragma unroll
                for (int p = 0; p < KQ; ++p)
                    *reinterpret_cast<floatx4*>(sQ + 512 + c16 * 16 + 4 * p) = floatx4{el[4 * p], el[4 * p + 1], el[4 * p + 2], el[4 * p + 3]};
            }
        }
        transpose_groups(q);                              // q[s]: entry k = 4 s + g, er[t]: entry j = 4 t + g
        transpose_groups(er);
    }
#pragma unroll
    for (int x = 0; x < NW; ++x) {
        int k, i, p;
        piece_of(tid + 256 * x, k, i, p);
        if (tid + 256 * x < npiece) {
            floatx4 v;
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = QUADS || (k < K && i < K && 4 * p + c < K) ? w[x][c] : 0.f;
            *reinterpret_cast<floatx4*>(wl + k * S + i * SI + 4 * p) = v;
        }
    }
    __syncthreads();
    if (active) {
        const float* wr = wl + g * S + (c16 & 3) * SI + (c16 >> 2);   // tile row m = 4 (j % 4) + i % 4
        float gr[4] = {0.f, 0.f, 0.f, 0.f}, glf[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int it = 0; it < KQ; ++it) {
            if (it < it0 || it >= it1) continue;
            float gl[4] = {0.f, 0.f, 0.f, 0.f};
            floatx4 acc[KQ];
#pragma unroll
            for (int jt = 0; jt < KQ; ++jt) acc[jt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < KQ; ++s)
#pragma unroll
                for (int jt = 0; jt < KQ; ++jt)
                    acc[jt] = __builtin_amdgcn_mfma_f32_16x16x4f32(wr[4 * s * S + 4 * it * SI + 4 * jt], q[s], acc[jt], 0, 0, 0);
            // acc[jt][c] = U[b][i = 4 it + c][j = 4 jt + g]
#pragma unroll
            for (int jt = 0; jt < KQ; ++jt)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    gl[c] = fmaf(acc[jt][c], er[jt], gl[c]);
                    gr[jt] = fmaf(acc[jt][c], el[4 * it + c], gr[jt]);
                }
            transpose_groups(gl);                             // summed over the lane groups: entry 4 it + g
            const float mine = g == 0 ? el[4 * it] : g == 1 ? el[4 * it + 1] : g == 2 ? el[4 * it + 2] : el[4 * it + 3];
            glf[it] = ((gl[0] + gl[1]) + (gl[2] + gl[3])) * mine;
        }
#pragma unroll
        for (int jt = 0; jt < KQ; ++jt) gr[jt] *= er[jt];
        if (QUADS) {
            transpose_groups(glf);
            transpose_groups(gr);
        }
        float* gleft = Gp + (size_t)rec[9] * blk + (size_t)b * K;
        float* gright = gleft + (size_t)(1 + grp) * blk;
        if (QUADS) {
            if (g >= it0 && g < it1 && b < B) *reinterpret_cast<floatx4*>(gleft + 4 * g) = floatx4{glf[0], glf[1], glf[2], glf[3]};
            if (g < KQ && b < B) *reinterpret_cast<floatx4*>(gright + 4 * g) = floatx4{gr[0], gr[1], gr[2], gr[3]};
        } else {
#pragma unroll
            for (int t = 0; t < KQ; ++t)
                if (4 * t + g < K && b < B) {
                    if (t >= it0 && t < it1) gleft[4 * t + g] = glf[t];
                    gright[4 * t + g] = gr[t];
                }
        }
    }
    if constexpr (STATS) {
        // rows (k, i), columns j, contraction over the wave's samples: lane group g takes the samples s + g.  Entries beyond K
        // are rows and columns that nobody reads; samples beyond the batch have Q = 0.
        floatx4 acc[KQ][KQ];
#pragma unroll
        for (int it = 0; it < KQ; ++it)
#pragma unroll
            for (int kt = 0; kt < KQ; ++kt) acc[it][kt] = floatx4{0.f, 0.f, 0.f, 0.f};
        if (active) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int s = 0; s < 16; s += 4) {
                const float* row = sQ + (s + g) * 16;
                const float rb = row[256 + c16];
                float qa[KQ];
#pragma unroll
                for (int kt = 0; kt < KQ; ++kt) qa[kt] = row[4 * kt + (c16 >> 2)];
#pragma unroll
                for (int it = 0; it < KQ; ++it) {
                    if (it < it0 || it >= it1) continue;
                    const float la = row[512 + 4 * it + (c16 & 3)];
#pragma unroll
                    for (int kt = 0; kt < KQ; ++kt) acc[it][kt] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[kt] * la, rb, acc[it][kt], 0, 0, 0);
                }
            }
        }
        // tile (it, kt) is finished by wave kt: acc[c]: k = 4 kt + g, i = 4 it + c, j = c16
        float* Nw = stats + rec[4];
        floatx4* red = reinterpret_cast<floatx4*>(sx);    // [wave][kt][lane]
#pragma unroll
        for (int it = 0; it < KQ; ++it) {
            if (it < it0 || it >= it1) continue;
            const int k = 4 * wave + g;
            const bool own = wave < KQ && k < K && c16 < K;
            float old[4] = {0.f, 0.f, 0.f, 0.f};
            if (ACCUM && own) {
#pragma unroll
                for (int c = 0; c < 4; ++c) old[c] = Nw[(k * K + min(4 * it + c, K - 1)) * K + c16];
            }
            __syncthreads();                              // rows, or the sums of the block before, have been read
#pragma unroll
            for (int kt = 0; kt < KQ; ++kt) red[(wave * KQ + kt) * 64 + lane] = acc[it][kt];
            __syncthreads();
            if (own) {
                floatx4 sum = red[wave * 64 + lane];
#pragma unroll
                for (int x = 1; x < 4; ++x) sum += red[(x * KQ + wave) * 64 + lane];
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (4 * it + c < K) Nw[(k * K + 4 * it + c) * K + c16] = old[c] + wl[k * S + (4 * it + c) * SI + c16] * sum[c];
            }
        }
    }
}

// EXACT: K is 8 K8 (no entry to leave out or to clamp, which keeps the kernel short).
template <int K8, bool EXACT>
__global__ __launch_bounds__(256, PostLayout<K8>::WAVES) void k_einsum_posterior(
    const int32_t* __restrict__ e_rec, const float* __restrict__ params, const float* __restrict__ A,
    const double* __restrict__ Off, const float* __restrict__ amax, const float* __restrict__ G, float* Gp, float* __restrict__ img,
    int item0, int nchunks, int ngr, int direct, int B, int K_) {
    const int K = EXACT ? 8 * K8 : K_;
    using LY = PostLayout<K8>;
    using X = X6<K8>;
    constexpr int NT = LY::NT, SG = LY::SG, TU = LY::TU, SLICE = LY::SLICE, NL = LY::NL, NO = LY::NO, NP = LY::NP;
    extern __shared__ __attribute__((aligned(16))) uint32x4 wl[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c16 = lane & 15, kg = lane >> 4;
    const int vb = xcd_contiguous_block();
    const int grp = vb % ngr, chunk = (vb / ngr) % nchunks, li = vb / (ngr * nchunks);
    const int32_t* rec = e_rec + (size_t)li * EIN_BREC_INTS;
    const int left = rec[0], right = rec[1], out = rec[2], reg = rec[3], voff = rec[5], vstr = rec[6];
    const int nte = (K + 3) >> 2;                         // tiles per slice, slices per item
    const int it0 = grp * nte / ngr, it1 = (grp + 1) * nte / ngr;   // this workgroup's slices
    const size_t blk = (size_t)B * K;
    const float* W = params + rec[4];
    const bool quads = EXACT || (K & 3) == 0;                      // rows of 16-byte groups

    // ---- W: thread t takes every 256th work item (consecutive threads consecutive j); rows k beyond K are zeros; the last
    // octet of k starts at K - 8, its first entries, which the octet before holds already, are zeros
    auto start_of = [&](int o) { return EXACT ? 8 * o : min(8 * o, K - 8); };
    floatx4 wv[NL][8];
    int wsrc[NL], wil[NL], wj[NL], wpo[NL], wsl[NL];
#pragma unroll
    for (int x = 0; x < NL; ++x) {
        const int f = tid + 256 * x;
        const int jp = f % nte, q = f / nte, o = (q >> 2) % K8, sl = (q >> 2) / K8;
        wil[x] = 4 * sl + (q & 3);
        wsl[x] = sl;
        wpo[x] = o;
        wj[x] = EXACT ? 4 * jp : min(4 * jp, K - 4);
        wsrc[x] = start_of(o) * K * K + wj[x];
    }
    auto fetch_w = [&](int it) {                          // slices it .. it + SG - 1
#pragma unroll
        for (int x = 0; x < NL; ++x) {
            if (wsl[x] < SG) {
            const float* p = W + wsrc[x] + (size_t)post_weight_row<K8, EXACT>(it, wil[x], K) * K;
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) {
                wv[x][kk] = *reinterpret_cast<const floatx4u*>(p + kk * K * K);
            }
            }
        }
    };
    auto store_w = [&](int it, uint32x4* dst) {
#pragma unroll
        for (int x = 0; x < NL; ++x) {
            const int o = wpo[x], il = wil[x] & 3;
            const bool row = 4 * it + wil[x] < K;
            const int k0 = 8 * o - start_of(o);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int j = wj[x] + c;
                float v[8];
#pragma unroll
                for (int kk = 0; kk < 8; ++kk) {
                    v[kk] = EXACT || (row && kk >= k0) ? wv[x][kk][c] * X6_SCALE : 0.f;
                }
                uint32x4 part[3];
                split_octet(v, part[0], part[1], part[2]);
                if (wsl[x] < SG) {
                    uint32x4* d = dst + wsl[x] * SLICE + (j >> 2) * TU;
#pragma unroll
                    for (int p = 0; p < 3; ++p) d[x6_unit<K8>(p, o, 4 * (j & 3) + il)] = part[p];
                }
            }
        }
    };
    fetch_w(it0);

    // ---- rows of this lane's samples
    const int b0 = chunk * 128 + 32 * wave;
    const bool active = b0 < B;                           // (a wave beyond the batch only brings weights in)
    uint32x4 q[2][X::NR];
    float er[2][4 * NP], gr[2][4 * NP], al[2], unscale[2];
    floatx4 lraw[2][SG];
    const float* Lp[2];
#pragma unroll
    for (int s = 0; s < 2; ++s)
        Lp[s] = A + (size_t)left * blk + (size_t)min(b0 + 16 * s + c16, B - 1) * K;
    auto fetch_l = [&](int it) {                          // the left entries of slices it .. it + SG - 1
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int sl = 0; sl < SG; ++sl) {
                const int i = 4 * (it + sl);
                if (quads) {
                    lraw[s][sl] = *reinterpret_cast<const floatx4u*>(Lp[s] + post_left_entry<K8, EXACT>(it + sl, K));
                } else {
#pragma unroll
                    for (int c = 0; c < 4; ++c) lraw[s][sl][c] = Lp[s][min(i + c, K - 1)];
                }
            }
    };
    // (the images for the weight statistics: rows k, j, i at Bp, lanes of a group consecutive samples)
    const int Bp = ein_image_stride(B);
    float* iQ = img + (size_t)(item0 + li) * EIN_IMAGES * (4 * nte) * Bp;
    float* iR = iQ + (size_t)(4 * nte) * Bp;
    float* iL = iR + (size_t)(4 * nte) * Bp;
    if (active) {
        const int gcnt = direct ? bwd_source_blocks(rec[8], K, B) : 1;
        const float* Gs = direct ? Gp + (size_t)rec[7] * blk : G + (size_t)reg * blk;
        const float* As = A + (size_t)reg * blk;
        fetch_l(it0);
        float g8[2][NO][8], a8[2][NO][8], v8[NO][8], ar[2], dd[2];
        auto oct_of = [&](int z) { return z < X::NQ ? 4 * z + kg : X::R2 && z == X::NQ ? 4 * X::NQ + (kg & 1) : K8 - 1; };
        auto load8 = [&](const float* p, float (&v)[8]) {
            {
                const floatx4 v0 = *reinterpret_cast<const floatx4u*>(p), v1 = *reinterpret_cast<const floatx4u*>(p + 4);
#pragma unroll
                for (int c = 0; c < 4; ++c) { v[c] = v0[c]; v[4 + c] = v1[c]; }
            }
        };
        float4 rraw[2][NP];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int b = min(b0 + 16 * s + c16, B - 1);
            const float* Rp = A + (size_t)right * blk + (size_t)b * K;
#pragma unroll
            for (int z = 0; z < NO; ++z) {
                const size_t o = (size_t)b * K + start_of(oct_of(z));
                load8(Gs + o, g8[s][z]);
                load8(As + o, a8[s][z]);
            }
            al[s] = amax[(size_t)(item0 + li) * 2 * B + b];
            ar[s] = amax[((size_t)(item0 + li) * 2 + 1) * B + b];
            dd[s] = (float)(Off[(size_t)out * B + b] - Off[(size_t)reg * B + b]);
            // right entries: lane group kg requests the pieces 4 p + kg, transposed below
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                if (quads) {
                    rraw[s][p] = *reinterpret_cast<const float4*>(Rp + 4 * min(4 * p + kg, nte - 1));
                } else {
                    float* e = &rraw[s][p].x;
#pragma unroll
                    for (int c = 0; c < 4; ++c) e[c] = Rp[min(16 * p + 4 * c + kg, K - 1)];
                }
            }
        }
        if (voff >= 0) {
#pragma unroll
            for (int z = 0; z < NO; ++z)
#pragma unroll
                for (int c = 0; c < 8; ++c) v8[z][c] = params[voff + min(start_of(oct_of(z)) + c, K - 1) * vstr];
        }
        for (int x = 1; x < gcnt; ++x) {                  // the other blocks of the parent
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int b = min(b0 + 16 * s + c16, B - 1);
#pragma unroll
                for (int z = 0; z < NO; ++z) {
                    float more[8];
                    load8(Gs + x * blk + (size_t)b * K + start_of(oct_of(z)), more);
#pragma unroll
                    for (int c = 0; c < 8; ++c) g8[s][z][c] += more[c];
                }
            }
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            float top = 0.f;
#pragma unroll
            for (int z = 0; z < NO; ++z) {
                const int o = oct_of(z);
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const bool in = EXACT || c >= 8 * o - start_of(o);
                    const float g = g8[s][z][c];
                    const float e = __expf(dd[s] - a8[s][z][c]);
                    const float qv = (voff >= 0 ? g * v8[z][c] : g) * e;
                    g8[s][z][c] = in && g != 0.f ? qv : 0.f;
                    top = fmaxf(top, g8[s][z][c]);
                }
                const bool own = z < X::NQ || (X::R2 && z == X::NQ ? kg < 2 : kg == 0);     // (lanes share the last octets)
                if (grp == 0 && own && b0 + 16 * s + c16 < B) {
#pragma unroll
                    for (int c = 0; c < 8; ++c)
                        if (EXACT || c >= 8 * o - start_of(o)) iQ[(size_t)(start_of(o) + c) * Bp + b0 + 16 * s + c16] = g8[s][z][c];
                }
            }
            top = fmaxf(top, __shfl_xor(top, 16, 64));
            top = fmaxf(top, __shfl_xor(top, 32, 64));
            // the power of two f that brings the largest near 2^60 (at most 2^126, so that 1 / f is a normal number)
            const int ex = (int)(__builtin_bit_cast(uint32_t, top) >> 23) - 127;
            const int fx = top > 0.f ? min(60 - ex, 126) : 0;
            const float f = __builtin_bit_cast(float, (uint32_t)(fx + 127) << 23);
            unscale[s] = __builtin_bit_cast(float, (uint32_t)(127 - fx) << 23);
            int z = 0;
            x6_sample_operand<K8>(kg, [&](int, float* v) {          // (called for the octets in the order of oct_of)
#pragma unroll
                for (int c = 0; c < 8; ++c) v[c] = g8[s][z][c] * f;
                ++z;
            }, q[s]);
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                float r[4] = {rraw[s][p].x, rraw[s][p].y, rraw[s][p].z, rraw[s][p].w};
                if (quads) transpose_groups(r);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const bool in = 16 * p + 4 * c + kg < K;
                    er[s][4 * p + c] = in ? __expf(r[c] - ar[s]) : 0.f;
                    gr[s][4 * p + c] = 0.f;
                    if (grp == ngr - 1 && in && b0 + 16 * s + c16 < B) iR[(size_t)(16 * p + 4 * c + kg) * Bp + b0 + 16 * s + c16] = er[s][4 * p + c];
                }
            }
        }
    }
    // rows j of the last tile that do not exist: zeros, in every buffer (no other store reaches them)
    if (!quads) {
        const int miss = 4 * nte - K;                     // 1 .. 3
        for (int f = tid; f < LY::NBUF * SG * 3 * K8 * 4 * miss; f += 256) {
            const int il = f & 3, j = 4 - miss + (f >> 2) % miss, po = (f >> 2) / miss % (3 * K8), sl = (f >> 2) / miss / (3 * K8);
            wl[sl * SLICE + (nte - 1) * TU + po * 16 + ((4 * j + il) ^ (po & 3))] = uint32x4{0u, 0u, 0u, 0u};
        }
    }
    int unit[X::NR];
#pragma unroll
    for (int a = 0; a < X::NR; ++a) unit[a] = x6_row_unit<K8>(a, kg, c16);
    float* gleft = Gp + (size_t)rec[9] * blk;
    float* gright = gleft + (size_t)(1 + grp) * blk;

    int buf = 0;
    for (int it = it0; it < it1; it += SG) {
        uint32x4* cur = wl + buf * (SG * SLICE);
        if (LY::NBUF == 1 && it > it0) __syncthreads();   // readers of the previous stage are done
        store_w(it, cur);
        floatx4 el[2][SG];
        if (active) {
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int sl = 0; sl < SG; ++sl)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        el[s][sl][c] = EXACT || 4 * (it + sl) + c < K ? __expf(lraw[s][sl][c] - al[s]) : 0.f;
        }
        __syncthreads();
        if (it + SG < it1) {
            fetch_w(it + SG);
            if (active) fetch_l(it + SG);
        }
        if (active) {
#pragma unroll
            for (int sl = 0; sl < SG; ++sl) {
                if (it + sl < it1) {
                    const uint32x4* wt = cur + sl * SLICE;
                    floatx4 gl[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        if (EXACT || t < nte) {
                            uint32x4 a[X::NR];
#pragma unroll
                            for (int z = 0; z < X::NR; ++z) a[z] = wt[t * TU + unit[z]];
                            floatx4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
                            x6_tile<K8, 2>(a, q, acc);
                            // acc[s][c] = U[b][i = 4 (it + sl) + c][j = 4 t + kg]
#pragma unroll
                            for (int s = 0; s < 2; ++s)
#pragma unroll
                                for (int c = 0; c < 4; ++c) {
                                    gl[s][c] = fmaf(acc[s][c], er[s][t], gl[s][c]);
                                    gr[s][t] = fmaf(acc[s][c], el[s][sl][c], gr[s][t]);
                                }
                            if (EXACT) __builtin_amdgcn_sched_barrier(0);    // (more tiles at once would spill)
                        }
                    }
#pragma unroll
                    for (int s = 0; s < 2; ++s) {
                        // sum over the lane groups; lane group kg ends up with entry i = 4 (it + sl) + kg
                        float r[4] = {gl[s][0], gl[s][1], gl[s][2], gl[s][3]};
                        transpose_groups(r);
                        const float sum = ((r[0] + r[1]) + (r[2] + r[3])) * (1.f / X6_SCALE) * unscale[s];
                        const floatx4 e = el[s][sl];
                        const float mine = kg == 0 ? e[0] : kg == 1 ? e[1] : kg == 2 ? e[2] : e[3];
                        const int b = b0 + 16 * s + c16, i = 4 * (it + sl) + kg;
                        if (b < B && i < K) {
                            gleft[(size_t)b * K + i] = sum * mine;
                            iL[(size_t)i * Bp + b] = mine;
                        }
                    }
                }
            }
        }
        if (LY::NBUF == 2) buf ^= 1;
    }
    if (!active) return;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int b = b0 + 16 * s + c16;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            float r[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) r[c] = gr[s][4 * p + c] * (1.f / X6_SCALE) * unscale[s] * er[s][4 * p + c];
            if (quads) {
                transpose_groups(r);
                if (b < B && 4 * p + kg < nte)
                    *reinterpret_cast<floatx4*>(gright + (size_t)b * K + 4 * (4 * p + kg)) = floatx4{r[0], r[1], r[2], r[3]};
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (b < B && 16 * p + 4 * c + kg < K) gright[(size_t)b * K + 16 * p + 4 * c + kg] = r[c];
            }
        }
    }
}

template <int KQ>
void launch_posterior_small(const DevTables& t, int first, int count, bool with_stats, bool accumulate, const float* params,
                            float* stats, const float* A, const double* Off, const float* amax, const float* G, float* Gp,
                            bool direct, const Dims& d, hipStream_t s) {
    const int nchunks = (d.B + PS_SAMPLES - 1) / PS_SAMPLES, ngr = bwd_groups_per_item(count, d.K, d.B);
#define EINET_LAUNCH(Q, ST, ACC, SP)                                                                                         \
    hipLaunchKernelGGL((k_einsum_posterior_small<KQ, Q, ST, ACC, SP>), dim3(count * nchunks * ngr), dim3(256), 0, s,              \
                       t.ein_brec + (size_t)first * EIN_BREC_INTS, params, stats, A, Off, amax, G, Gp, first, nchunks, ngr,   \
                       direct ? 1 : 0, d.B, d.K)
#define EINET_LAUNCH_Q(Q)                                                     \
    do {                                                                      \
        if (!with_stats) EINET_LAUNCH(Q, false, false, false);                \
        else if (KQ > 2 && ngr > 1 && accumulate) EINET_LAUNCH(Q, true, true, (KQ > 2)); \
        else if (KQ > 2 && ngr > 1) EINET_LAUNCH(Q, true, false, (KQ > 2));   \
        else if (accumulate) EINET_LAUNCH(Q, true, true, false);              \
        else EINET_LAUNCH(Q, true, false, false);                             \
    } while (0)
    if (d.K == 4 * KQ) EINET_LAUNCH_Q(true);
    else EINET_LAUNCH_Q(false);
#undef EINET_LAUNCH_Q
#undef EINET_LAUNCH
}

template <int K8>
void launch_posterior_k8(const DevTables& t, int first, int count, const float* params, const float* A, const double* Off,
                         const float* amax, const float* G, float* Gp, float* img, bool direct, const Dims& d, hipStream_t s) {
    const size_t lds = PostLayout<K8>::LDS_BYTES;
    if (lds > 64 * 1024) {
        static std::once_flag attr_set[EINET_MAX_DEVICES];
        int dev = 0;
        (void)hipGetDevice(&dev);
        std::call_once(attr_set[dev % EINET_MAX_DEVICES], [&] { 
            allow_dynamic_lds(&k_einsum_posterior<K8, true>, lds);
            allow_dynamic_lds(&k_einsum_posterior<K8, false>, lds);
        });
    }
    const int nchunks = (d.B + 127) / 128, ngr = bwd_groups_per_item(count, d.K, d.B);
#define EINET_LAUNCH(EX)                                                                                              \
    hipLaunchKernelGGL((k_einsum_posterior<K8, EX>), dim3(count * nchunks * ngr), dim3(256), lds, s,                    \
                       t.ein_brec + (size_t)first * EIN_BREC_INTS, params, A, Off, amax, G, Gp, img, first, nchunks, ngr, \
                       direct ? 1 : 0, d.B, d.K)
    if (d.K == 8 * K8) EINET_LAUNCH(true);
    else EINET_LAUNCH(false);
#undef EINET_LAUNCH
}

// ------------------------------------------------------------------ posteriors and statistics in one launch
// Batches of one chunk (128 samples) with few entries or few items: the launches are chains of requests, and one more of
// them for the statistics costs more than what the split operands save (einsum_backward_fused).  One workgroup per (item,
// share of the chunks, run of slices of four left entries): eR^T and Q^T are staged once, sample-major, the slices W[:, 4 i .., :] stream
// through LDS with the next in flight in registers; both products, statistics (contraction over the batch) and posteriors (over
// k), read the slice.  The right child's posterior is summed over the workgroup's slices in LDS and written to a block of its
// own.  With several chunks a workgroup walks `cpv` of them; nshare > 1: every share's statistics go to blocks of their own in
// `part`, which a later launch adds up.
template <int KQ>
struct BwdLayout {
    static constexpr int KP = 4 * KQ;
    static constexpr int SI = ((KP + 7) / 16) * 16 + 8;   // stride between the slice's i rows: 8 mod 16
    static constexpr int S = 4 * SI + 4;                  // stride between k rows: 4 mod 32
    static constexpr int NJ = (KP + 15) / 16;             // column tiles of GEMM-1
    static constexpr int BC = 128;                        // samples per pass over the batch
    static constexpr int ST = BC + 4;                     // row stride of the sample-major operand copies: 4 mod 32
    static constexpr int OFF_R = KP * S;                  // eR^T [16 NJ][ST]
    static constexpr int OFF_Q = OFF_R + 16 * NJ * ST;    // Q^T  [KP][ST]
    static constexpr int OFF_L = OFF_Q + KP * ST;         // eL^T [4][ST] of the current slice
    static constexpr int OFF_G = OFF_L + 4 * ST;          // Gp_right of the workgroup's slices [BC][KP]
    static constexpr int LDS_FLOATS = OFF_G + BC * KP;
    static_assert(LDS_FLOATS <= 40960, "160 KB of LDS");
    static constexpr int MAXU = (NJ * KQ + 7) / 8;        // GEMM-1 tiles per wave
    static constexpr int NW4 = (KP * 4 * KQ + 511) / 512; // float4 per thread of one W slice
    static constexpr int NW1 = (KP * 4 * KP + 511) / 512; // floats per thread when K is not a multiple of 4
};

// GEMM-1 over one pass of the batch for NU tiles of this wave.  The operands are kept
// sample-major in LDS (eR^T, Q^T, eL^T) and lane group g contracts samples g*RG .. g*RG+RG-1,
// so that one 16-byte LDS read feeds four consecutive MFMA steps.
template <int KQ, int NU>
__device__ __forceinline__ void bwd_gemm1(floatx4* acc1, const float* const* qcol, const float* const* rcol,
                                          const float* elcol, int rg) {
    // operands of the next four samples are requested before the MFMAs of the current four are issued
    float4 e = *reinterpret_cast<const float4*>(elcol);
    float4 qa[NU], rb[NU];
#pragma unroll
    for (int q = 0; q < NU; ++q) {
        qa[q] = *reinterpret_cast<const float4*>(qcol[q]);
        rb[q] = *reinterpret_cast<const float4*>(rcol[q]);
    }
    for (int s = 0; s < rg; s += 4) {
        const int sn = min(s + 4, rg - 4);           // the last round reads its own operands again
        const float4 en = *reinterpret_cast<const float4*>(elcol + sn);
        float4 qn[NU], rn[NU];
#pragma unroll
        for (int q = 0; q < NU; ++q) {
            qn[q] = *reinterpret_cast<const float4*>(qcol[q] + sn);
            rn[q] = *reinterpret_cast<const float4*>(rcol[q] + sn);
        }
#pragma unroll
        for (int q = 0; q < NU; ++q) acc1[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[q].x * e.x, rb[q].x, acc1[q], 0, 0, 0);
#pragma unroll
        for (int q = 0; q < NU; ++q) acc1[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[q].y * e.y, rb[q].y, acc1[q], 0, 0, 0);
#pragma unroll
        for (int q = 0; q < NU; ++q) acc1[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[q].z * e.z, rb[q].z, acc1[q], 0, 0, 0);
#pragma unroll
        for (int q = 0; q < NU; ++q) acc1[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[q].w * e.w, rb[q].w, acc1[q], 0, 0, 0);
        e = en;
#pragma unroll
        for (int q = 0; q < NU; ++q) {
            qa[q] = qn[q];
            rb[q] = rn[q];
        }
    }
}

// LOOP: cpv is more than one (the loop costs registers).
template <int KQ, bool VEC, bool ACCUM, bool DIRECT, bool LOOP>
__global__ __launch_bounds__(512, 2) void k_einsum_backward_fused(
    const int32_t* __restrict__ e_rec,
    const float* __restrict__ params, float* __restrict__ stats, const float* __restrict__ A,
    const double* __restrict__ Off, const float* __restrict__ amax, const float* __restrict__ G, float* Gp,
    int item0, int ngroups, int nshare, int cpv, int total, float* __restrict__ part, int B, int K) {
    using LY = BwdLayout<KQ>;
    constexpr int KP = LY::KP, SI = LY::SI, S = LY::S, ST = LY::ST, BC = LY::BC, MAXU = LY::MAXU;
    extern __shared__ float lds[];
    float* Wl = lds;
    float* sR = lds + LY::OFF_R;
    float* sQ = lds + LY::OFF_Q;
    float* sL = lds + LY::OFF_L;
    float* sG = lds + LY::OFF_G;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int vb = xcd_contiguous_block();
    const int grp = vb % ngroups, share = (vb / ngroups) % nshare, li = vb / (ngroups * nshare);
    const int it0 = grp * KQ / ngroups, it1 = (grp + 1) * KQ / ngroups;     // this workgroup's slices
    const bool multi = it1 - it0 > 1;   // several slices: their shares of Gp_right are summed in LDS first
    const int item = item0 + li;
    const int32_t* rec = e_rec + (size_t)li * EIN_BREC_INTS;
    const size_t blk = (size_t)B * K;
    const float* Lp = A + (size_t)rec[0] * blk;
    const float* Rp = A + (size_t)rec[1] * blk;
    const float* As = A + (size_t)rec[3] * blk;
    // posterior of the item's region: assembled in G, or (DIRECT) the sum of gcnt consecutive blocks that the
    // region's only parent wrote to Gp, added up in the order the assembly launch would take
    const int gcnt = DIRECT ? bwd_source_blocks(rec[8], K, B) : 0;
    const float* Gs = DIRECT ? Gp + (size_t)rec[7] * blk : G + (size_t)rec[3] * blk;
    float* gleft = Gp + (size_t)rec[9] * blk;
    float* gright = gleft + (size_t)(1 + grp) * blk;
    const float* W = params + rec[4];
    const size_t wbase = (size_t)rec[4];
    const int voff = rec[5], vstr = rec[6];
    const float* aL = amax + (size_t)item * 2 * B;
    const float* aR = aL + B;
    const double* Oo = Off + (size_t)rec[2] * B;
    const double* Os = Off + (size_t)rec[3] * B;

    // registers that carry the next W slice
    float4 w4[VEC ? LY::NW4 : 1];
    float w1[VEC ? 1 : LY::NW1];
    auto fetch_w = [&](int it) {
        if constexpr (VEC) {
#pragma unroll
            for (int n = 0; n < LY::NW4; ++n) {
                const int q = tid + 512 * n;
                const int j4 = q % KQ, il = (q / KQ) & 3, k = q / (4 * KQ);
                w4[n] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (k < K) w4[n] = *reinterpret_cast<const float4*>(W + ((size_t)k * K + 4 * it + il) * K + 4 * j4);
            }
        } else {
#pragma unroll
            for (int n = 0; n < LY::NW1; ++n) {
                const int q = tid + 512 * n;
                const int j = q % KP, il = (q / KP) & 3, k = q / (4 * KP);
                const int i = 4 * it + il;
                w1[n] = (k < K && i < K && j < K) ? W[((size_t)k * K + i) * K + j] : 0.f;
            }
        }
    };
    auto store_w = [&]() {
        if constexpr (VEC) {
#pragma unroll
            for (int n = 0; n < LY::NW4; ++n) {
                const int q = tid + 512 * n;
                const int j4 = q % KQ, il = (q / KQ) & 3, k = q / (4 * KQ);
                if (k < KP) *reinterpret_cast<float4*>(Wl + k * S + il * SI + 4 * j4) = w4[n];
            }
        } else {
#pragma unroll
            for (int n = 0; n < LY::NW1; ++n) {
                const int q = tid + 512 * n;
                const int j = q % KP, il = (q / KP) & 3, k = q / (4 * KP);
                if (k < KP) Wl[k * S + il * SI + j] = w1[n];
            }
        }
    };
    fetch_w(it0);

    const int c = lane & 15, g = lane >> 4;
    const int gm = c >> 2, rm = c & 3;
    // GEMM-1 tiles of this wave: u = jt * KQ + kt
    constexpr int U = LY::NJ * KQ;
    const int u0 = wave * U / 8, nu = (wave + 1) * U / 8 - u0;
    const float* qcol[MAXU];
    const float* rcol[MAXU];
    int uoff[MAXU], uwl[MAXU];        // offset of (k, i = 0, j) in W / Nw, and in the LDS slice
    bool uok[MAXU];
#pragma unroll
    for (int q = 0; q < MAXU; ++q) {
        const int u = min(u0 + q, U - 1);
        const int jt = u / KQ, ukt = u - jt * KQ;
        qcol[q] = sQ + (4 * ukt + gm) * ST;     // + g*RG + s
        rcol[q] = sR + (16 * jt + c) * ST;
        const int k = 4 * ukt + g, j = 16 * jt + c;
        uok[q] = q < nu && k < K && j < K;
        uoff[q] = uok[q] ? (k * K) * K + j : 0;
        uwl[q] = uok[q] ? k * S + j : 0;
    }
    float* Nw = nshare > 1 ? part + ((size_t)share * total + item) * ((size_t)K * K * K) : stats + wbase;

    // staging of eR and Q
    const int srow = tid >> 2, sq = tid & 3;
    constexpr int NF = (BC * KQ + 511) / 512;      // float4 of a [BC][K] block per thread

    const int bfirst = share * (LOOP ? cpv : 1) * BC, bend = min(bfirst + (LOOP ? cpv : 1) * BC, B);
    for (int b0 = bfirst; LOOP ? b0 < bend : b0 == bfirst; b0 += BC) {
        const int nb = min(BC, B - b0);
        const int rg = (((nb + 3) >> 2) + 3) & ~3;         // samples per lane group in GEMM-1, multiple of 4
        const bool rok = srow < nb;
        const int ro = (b0 + min(srow, nb - 1)) * K;       // a valid row even for the idle tail threads
        const float al = aL[b0 + min(srow, nb - 1)];
        if (LOOP && b0 > bfirst) __syncthreads();                  // readers of the chunk before are done
        if constexpr (VEC) {
            // the [nb][K] blocks are contiguous: 16-byte loads, consecutive threads consecutive addresses
            float4 r4[NF], g4[NF], a4[NF], v4[NF];
            float arn[NF], ddn[NF];
#pragma unroll
            for (int n = 0; n < NF; ++n) {
                const int f = min(tid + 512 * n, nb * KQ - 1);
                const int row = f / KQ, k4 = f - row * KQ;
                r4[n] = *reinterpret_cast<const float4*>(Rp + (size_t)(b0 + row) * K + 4 * k4);
                g4[n] = *reinterpret_cast<const float4*>(Gs + (size_t)(b0 + row) * K + 4 * k4);
                if (DIRECT && gcnt > 1) {
                    float4 gx[GSRC_MAX_BLOCKS - 1];
#pragma unroll
                    for (int x = 1; x < GSRC_MAX_BLOCKS; ++x)
                        gx[x - 1] = x < gcnt ? *reinterpret_cast<const float4*>(Gs + x * blk + (size_t)(b0 + row) * K + 4 * k4)
                                             : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                    for (int x = 1; x < GSRC_MAX_BLOCKS; ++x)
                        if (x < gcnt) {
                            g4[n].x += gx[x - 1].x;
                            g4[n].y += gx[x - 1].y;
                            g4[n].z += gx[x - 1].z;
                            g4[n].w += gx[x - 1].w;
                        }
                }
                a4[n] = *reinterpret_cast<const float4*>(As + (size_t)(b0 + row) * K + 4 * k4);
                arn[n] = aR[b0 + row];
                ddn[n] = (float)(Oo[b0 + row] - Os[b0 + row]);
                v4[n] = make_float4(1.f, 1.f, 1.f, 1.f);
                if (voff >= 0) {
                    v4[n].x = params[voff + min(4 * k4 + 0, K - 1) * vstr];
                    v4[n].y = params[voff + min(4 * k4 + 1, K - 1) * vstr];
                    v4[n].z = params[voff + min(4 * k4 + 2, K - 1) * vstr];
                    v4[n].w = params[voff + min(4 * k4 + 3, K - 1) * vstr];
                }
            }
#pragma unroll
            for (int n = 0; n < NF; ++n) {
                const int f = tid + 512 * n;
                if (f < BC * KQ) {
                    const int row = f / KQ, k4 = f - row * KQ;
                    const bool in = row < nb;
                    const float rr[4] = {r4[n].x, r4[n].y, r4[n].z, r4[n].w};
                    const float gg[4] = {g4[n].x, g4[n].y, g4[n].z, g4[n].w};
                    const float aa[4] = {a4[n].x, a4[n].y, a4[n].z, a4[n].w};
                    const float vv[4] = {v4[n].x, v4[n].y, v4[n].z, v4[n].w};
#pragma unroll
                    for (int c4 = 0; c4 < 4; ++c4) {
                        const int k = 4 * k4 + c4;
                        const float e = __expf(rr[c4] - arn[n]);
                        const float q = gg[c4] * vv[c4] * __expf(ddn[n] - aa[c4]);
                        sR[k * ST + row] = in ? e : 0.f;
                        sQ[k * ST + row] = (in && k < K && gg[c4] != 0.f) ? q : 0.f;
                    }
                }
            }
            for (int j = KP + sq; j < 16 * LY::NJ; j += 4) sR[j * ST + srow] = 0.f;   // rows beyond the padded K
            if (multi)
                for (int u = 0; u < KQ; ++u) sG[srow * KP + sq * KQ + u] = 0.f;
        } else {
            const float ar = aR[b0 + min(srow, nb - 1)];
            const float dd = (float)(Oo[b0 + min(srow, nb - 1)] - Os[b0 + min(srow, nb - 1)]);
            float rv[KQ], gv[KQ], av[KQ];
#pragma unroll
            for (int u = 0; u < KQ; ++u) {
                const int k = sq * KQ + u;
                const int kc = min(k, K - 1);
                rv[u] = Rp[ro + kc];
                gv[u] = Gs[ro + min(kc, K - 1)];
                if (DIRECT && gcnt > 1) {
                    float gx[GSRC_MAX_BLOCKS - 1];
#pragma unroll
                    for (int x = 1; x < GSRC_MAX_BLOCKS; ++x) gx[x - 1] = x < gcnt ? Gs[x * blk + ro + min(kc, K - 1)] : 0.f;
#pragma unroll
                    for (int x = 1; x < GSRC_MAX_BLOCKS; ++x)
                        if (x < gcnt) gv[u] += gx[x - 1];
                }
                av[u] = As[ro + min(kc, K - 1)];
            }
#pragma unroll
            for (int u = 0; u < KQ; ++u) {
                const int k = sq * KQ + u;
                const float vw = (voff >= 0 && k < K) ? params[voff + k * vstr] : 1.f;
                const float e = __expf(rv[u] - ar);
                const float q = gv[u] * vw * __expf(dd - av[u]);
                sR[k * ST + srow] = (rok && k < K) ? e : 0.f;
                sQ[k * ST + srow] = (rok && k < K && gv[u] != 0.f) ? q : 0.f;
            }
            for (int j = KP + sq; j < 16 * LY::NJ; j += 4) sR[j * ST + srow] = 0.f;   // rows beyond the padded K
            if (multi)
                for (int u = 0; u < KQ; ++u) sG[srow * KP + sq * KQ + u] = 0.f;
        }

        for (int it = it0; it < it1; ++it) {
            if (it != it0) __syncthreads();                // readers of the previous slice are done
            store_w();
            {
                const float e = __expf(Lp[ro + min(4 * it + sq, K - 1)] - al);
                sL[sq * ST + srow] = (rok && 4 * it + sq < K) ? e : 0.f;
            }
            __syncthreads();
            // the next slice, or the first one for the next chunk, goes in flight now
            if (it + 1 < it1) fetch_w(it + 1);
            else if (LOOP && b0 + BC < bend) fetch_w(it0);

            // statistics this wave will update, fetched early (not needed when they are known to be zero)
            float nw[MAXU][4];
#pragma unroll
            for (int q = 0; q < MAXU; ++q)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int i = VEC ? 4 * it + r : min(4 * it + r, K - 1);
                    // (units that are not ours read a valid dummy; later chunks always add)
                    nw[q][r] = ACCUM || (LOOP && b0 > bfirst) ? Nw[uoff[q] + i * K] : 0.f;
                }

            // ---- GEMM-1
            floatx4 acc1[MAXU];
#pragma unroll
            for (int q = 0; q < MAXU; ++q) acc1[q] = floatx4{0.f, 0.f, 0.f, 0.f};
            {
                const float* elcol = sL + rm * ST + g * rg;
                const float* qc[MAXU];
                const float* rc[MAXU];
#pragma unroll
                for (int q = 0; q < MAXU; ++q) {
                    qc[q] = qcol[q] + g * rg;
                    rc[q] = rcol[q] + g * rg;
                }
                if (nu == MAXU) bwd_gemm1<KQ, MAXU>(acc1, qc, rc, elcol, rg);
                else if (MAXU > 1 && nu == MAXU - 1)
                    bwd_gemm1<KQ, (MAXU > 1 ? MAXU - 1 : 1)>(acc1, qc, rc, elcol, rg);
                else
                    for (int q = 0; q < nu; ++q) bwd_gemm1<KQ, 1>(acc1 + q, qc + q, rc + q, elcol, rg);
            }

            // ---- GEMM-2: one tile of 16 samples per wave
            if (wave * 16 < nb) {
                const int bl = wave * 16 + c;
                const bool ok = bl < nb;
                float erg[KQ];
#pragma unroll
                for (int s = 0; s < KQ; ++s) erg[s] = sR[(4 * s + g) * ST + bl];
                const float* qrow = sQ + g * ST + bl;
                const float4 e4 = make_float4(sL[bl], sL[ST + bl], sL[2 * ST + bl], sL[3 * ST + bl]);
                const float* wl = Wl + g * S + rm * SI + gm;      // row 4*gm+rm of a tile = (j = 4jt+gm, i = 4it+rm)
                floatx4 acc[KQ];
#pragma unroll
                for (int jt = 0; jt < KQ; ++jt) acc[jt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
                for (int s = 0; s < KQ; ++s) {
                    const float qs = qrow[4 * s * ST];
#pragma unroll
                    for (int jt = 0; jt < KQ; ++jt)
                        acc[jt] = __builtin_amdgcn_mfma_f32_16x16x4f32(wl[4 * s * S + 4 * jt], qs, acc[jt], 0, 0, 0);
                }
                // acc[jt][r] = U[b][i = 4it+r][j = 4jt+g]
                float gl0 = 0.f, gl1 = 0.f, gl2 = 0.f, gl3 = 0.f;
                float* right = gright + (size_t)(b0 + bl) * K;
                float* racc = sG + bl * KP;
#pragma unroll
                for (int jt = 0; jt < KQ; ++jt) {
                    const float t = acc[jt][0] * e4.x + acc[jt][1] * e4.y + acc[jt][2] * e4.z + acc[jt][3] * e4.w;
                    // this lane owns the entry in every slice: no race
                    if (multi) racc[4 * jt + g] += erg[jt] * t;
                    else if (ok && 4 * jt + g < K) right[4 * jt + g] = erg[jt] * t;
                    gl0 = fmaf(acc[jt][0], erg[jt], gl0);
                    gl1 = fmaf(acc[jt][1], erg[jt], gl1);
                    gl2 = fmaf(acc[jt][2], erg[jt], gl2);
                    gl3 = fmaf(acc[jt][3], erg[jt], gl3);
                }
                gl0 += __shfl_xor(gl0, 16, 64); gl0 += __shfl_xor(gl0, 32, 64);
                gl1 += __shfl_xor(gl1, 16, 64); gl1 += __shfl_xor(gl1, 32, 64);
                gl2 += __shfl_xor(gl2, 16, 64); gl2 += __shfl_xor(gl2, 32, 64);
                gl3 += __shfl_xor(gl3, 16, 64); gl3 += __shfl_xor(gl3, 32, 64);
                const float glr = g == 0 ? gl0 * e4.x : (g == 1 ? gl1 * e4.y : (g == 2 ? gl2 * e4.z : gl3 * e4.w));
                if (ok && 4 * it + g < K) gleft[(size_t)(b0 + bl) * K + 4 * it + g] = glr;
            }

            // ---- GEMM-1 epilogue: Nw += W * acc
#pragma unroll
            for (int q = 0; q < MAXU; ++q) {
                if (uok[q]) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int i = 4 * it + r;
                        if (VEC || i < K) Nw[uoff[q] + i * K] = nw[q][r] + Wl[uwl[q] + r * SI] * acc1[q][r];
                    }
                }
            }
        }
        if (multi) {                        // Gp_right of the workgroup's slices, row by row
            __syncthreads();
            float* right = gright + (size_t)b0 * K;
            for (int e = tid; e < nb * K; e += 512) {
                const int b = e / K, j = e - b * K;
                right[e] = sG[b * KP + j];
            }
        }
    }
}

}  // namespace

void launch_region_assemble(const DevTables& t, int first, int count, bool is_root_layer, float* G, const float* Gp,
                            const Dims& d, hipStream_t s) {
    if (count == 0) return;
    dim3 grid(count, (d.B * d.K + 255) / 256);
    hipLaunchKernelGGL(k_region_assemble, grid, dim3(256), 0, s, t.rb_rec + (size_t)first * RB_REC_INTS, t.rb_pblk,
                       is_root_layer ? 1 : 0, G, Gp, bwd_block_limit(d.K, d.B), d.B, d.K);
}

template <int KQ>
static void launch_backward_fused(const DevTables& t, int first, int count, bool accumulate, const float* params, float* stats,
                                  const float* A, const double* Off, const float* amax, const float* G, float* Gp, float* part, int total,
                                  bool direct, const Dims& d, hipStream_t s) {
    constexpr size_t lds = sizeof(float) * BwdLayout<KQ>::LDS_FLOATS;
    constexpr bool ENTRIES = KQ <= 10, TURNS = KQ == 7;       // forms that einsum_backward_fused asks for
    const int ngroups = bwd_groups_per_item(count, d.K, d.B), nchunks = (d.B + 127) / 128;
    const int nshare = fused_shares(total, d.K, d.B), cpv = (nchunks + nshare - 1) / nshare;
    const bool adds = accumulate && nshare == 1;                          // (blocks of shares are written, not added to)
#define EINET_LAUNCH_L(V, ACC, DIR, L)                                                                                      \
    do {                                                                                                                    \
        if (lds > 64 * 1024) {                                                                                              \
            static std::once_flag attr_set[EINET_MAX_DEVICES];                                                              \
            int dev = 0;                                                                                                    \
            (void)hipGetDevice(&dev);                                                                                       \
            std::call_once(attr_set[dev % EINET_MAX_DEVICES],                                                               \
                           [&] { allow_dynamic_lds(&k_einsum_backward_fused<KQ, V, ACC, DIR, L>, lds); });                  \
        }                                                                                                                   \
        hipLaunchKernelGGL((k_einsum_backward_fused<KQ, V, ACC, DIR, L>), dim3(count * nshare * ngroups), dim3(512), lds, s, \
                           t.ein_brec + (size_t)first * EIN_BREC_INTS, params, stats, A, Off, amax, G, Gp, first, ngroups,  \
                           nshare, cpv, total, part, d.B, d.K);                                                             \
    } while (0)
#define EINET_LAUNCH_A(V, DIR, L)                              \
    do {                                                       \
        if (adds) EINET_LAUNCH_L(V, true, DIR, L);             \
        else EINET_LAUNCH_L(V, false, DIR, L);                 \
    } while (0)
#define EINET_LAUNCH(V)                                        \
    do {                                                       \
        if (TURNS && cpv > 1 && direct) EINET_LAUNCH_A(V, true, TURNS);       \
        else if (TURNS && cpv > 1) EINET_LAUNCH_A(V, false, TURNS);           \
        else if (direct) EINET_LAUNCH_A(V, true, false);       \
        else EINET_LAUNCH_A(V, false, false);                  \
    } while (0)
    if ((d.K & 3) == 0) {
        EINET_LAUNCH(true);
    } else if constexpr (ENTRIES) {
        EINET_LAUNCH(false);
    }
#undef EINET_LAUNCH
#undef EINET_LAUNCH_A
#undef EINET_LAUNCH_L
}

void launch_einsum_backward(const DevTables& t, int first, int count, bool accumulate, const float* params, float* stats, const float* A,
                            const double* Off, const float* amax, const float* G, float* Gp, float* img, PartialSumList* list,
                            bool direct, const Dims& d, hipStream_t s) {
    if (count == 0) return;
    // (one workgroup per item: it takes the statistics with it)
    EinStatsWork& w = list->ein;
    const bool fused = einsum_backward_fused(w.total, d.K, d.B);
    const bool with_stats = fused || (d.K <= 16 && d.B <= PS_SAMPLES);
    if (fused) {
        switch ((d.K + 3) / 4) {
#define EINET_CASE(J) \
    case J: launch_backward_fused<J>(t, first, count, accumulate, params, stats, A, Off, amax, G, Gp, w.part, w.total, direct, d, s); break;
            EINET_CASE(5) EINET_CASE(6) EINET_CASE(7) EINET_CASE(8) EINET_CASE(9) EINET_CASE(10) EINET_CASE(11) EINET_CASE(12)
#undef EINET_CASE
        }
    } else if (d.K <= 16) {
        switch ((d.K + 3) / 4) {
#define EINET_CASE(J) \
    case J: launch_posterior_small<J>(t, first, count, with_stats, accumulate, params, stats, A, Off, amax, G, Gp, direct, d, s); break;
            EINET_CASE(1) EINET_CASE(2) EINET_CASE(3) EINET_CASE(4)
#undef EINET_CASE
        }
    } else {
        switch ((d.K + 7) / 8) {
#define EINET_CASE(J) \
    case J: launch_posterior_k8<J>(t, first, count, params, A, Off, amax, G, Gp, img, direct, d, s); break;
            EINET_CASE(3) EINET_CASE(4) EINET_CASE(5) EINET_CASE(6) EINET_CASE(7) EINET_CASE(8)
#undef EINET_CASE
        }
    }
    if (with_stats && (!fused || fused_shares(w.total, d.K, d.B) == 1)) return;
    w = EinStatsWork{t.ein_brec + (size_t)first * EIN_BREC_INTS, t.ein_woff + first, w.part, params, A, amax, G, Gp, img, Off, first,
                     w.count + count, d.B, d.K, w.total, fused};
}

}  // namespace einet_impl
