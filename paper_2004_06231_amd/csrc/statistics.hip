// End of the top-down pass: statistics of the mixing weights and of the leaves (Eq. 6-7).
#include "bf16x6.hpp"

#include <mutex>

namespace einet_impl {

namespace {

// Statistics of the mixing weights (App. B, Eq. 6): Nv[s,k,c] += v[s,k,c] * sum_b G[s][b,k] * S^c[b,k] / S[b,k].
// One workgroup per (mixing item, child); a reduction over the batch through LDS.  Runs in the same
// launch as the leaf statistics (k_tail_backward): the two are independent.  The workgroup is a chain of memory
// requests: the item's record (node, entries, weight offset, partitions: one request instead of four tables one after the
// other), then the rows of four samples per thread at once together with the weight and its old statistic.
template <int TPB>
__device__ __forceinline__ void mixing_stats_body(int item, int c, const int32_t* __restrict__ m_rec,
                                                  const int32_t* __restrict__ m_cptr,
                                                  const int32_t* __restrict__ m_child, const float* __restrict__ params,
                                                  float* __restrict__ stats, const float* __restrict__ A,
                                                  const double* __restrict__ Off, const float* __restrict__ G, int B,
                                                  int K) {
    __shared__ float red[TPB];
    const int tid = threadIdx.x;
    const int32_t* rec = m_rec + (size_t)item * MIX_REC_INTS;
    const int node = rec[0], kout = rec[1], voff = rec[2], nc = rec[3];
    if (c >= nc) return;
    const int child = c < MIX_REC_CHILDREN ? rec[4 + c] : m_child[m_cptr[item] + c];
    const int nbl = TPB / kout, k = tid % kout, bl = tid / kout;
    const float* As = A + (size_t)node * B * K;
    const float* Ac = A + (size_t)child * B * K;
    const float* Gs = G + (size_t)node * B * K;
    const double* Os = Off + (size_t)node * B;
    const double* Oc = Off + (size_t)child * B;
    const size_t so = (size_t)voff + (size_t)min(tid, kout - 1) * nc + c;
    const float pv = params[so], sv = stats[so];       // (used by the first kout threads at the end)
    float part = 0.f;
    if (bl < nbl)
        for (int b0 = bl; b0 < B; b0 += 4 * nbl) {
            float g[4], ac[4], as[4];
            double dd[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int b = min(b0 + u * nbl, B - 1);
                const size_t o = (size_t)b * K + k;
                g[u] = Gs[o];
                ac[u] = Ac[o];
                as[u] = As[o];
                dd[u] = Oc[b] - Os[b];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (b0 + u * nbl < B && g[u] != 0.f) part += g[u] * expf((float)dd[u] + ac[u] - as[u]);
        }
    red[tid] = part;
    __syncthreads();
    // A sum with few entries (the root has one) has hundreds of sample groups: 32 threads per entry first add every 32nd
    // group, so that no thread walks more than a few dozen values.
    int ngr = nbl;
    if (nbl > 64) {
        constexpr int J = 32;
        float t = 0.f;
        const int kk = tid % kout, j = tid / kout;
        if (j < J)
            for (int l = j; l < nbl; l += J) t += red[l * kout + kk];
        __syncthreads();
        if (j < J) red[j * kout + kk] = t;
        __syncthreads();
        ngr = J;
    }
    if (tid < kout) {
        float t4[4] = {0.f, 0.f, 0.f, 0.f};
        int l = 0;
        for (; l + 4 <= ngr; l += 4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) t4[u] += red[(l + u) * kout + tid];
        }
        for (; l < ngr; ++l) t4[0] += red[l * kout + tid];
        stats[so] = sv + pv * ((t4[0] + t4[1]) + (t4[2] + t4[3]));
    }
}

// ------------------------------------------------------------------ top-down pass, leaves
// Posterior-weighted sufficient statistics (Eq. 6-7).  A workgroup of 1024 threads
// owns 1024/NCH consecutive statistics entries (leaf variable, channel, k); its NCH
// parts each walk every NCH-th sample and the partial sums meet in LDS.
// DIRECT: the leaf's posterior is not in G; it is the sum of the blocks of Gp that leaf_gsrc names (two ints per leaf, see
// GSRC_MAX_BLOCKS), added up in the order the assembly launch would take.
template <int NCH, bool DIRECT>
__device__ __forceinline__ void leaf_backward_body(
    int block, const int32_t* __restrict__ lv_leaf, const int32_t* __restrict__ lv_var, const int32_t* __restrict__ leaf_node,
    const int32_t* __restrict__ leaf_replica, int n_lv, const float* __restrict__ x,
    const uint8_t* __restrict__ mask, int mask_mode, const float* __restrict__ G, const float* __restrict__ Gp,
    const int32_t* __restrict__ leaf_gsrc, float* __restrict__ stats,
    int64_t phi_off, int64_t den_off, int64_t tot_off, Dims d) {
    constexpr int NO = 1024 / NCH;
    __shared__ float red[NCH][4][NO];
    const int lo = threadIdx.x % NO, part_id = threadIdx.x / NO;
    const int idx = block * NO + lo;
    const bool valid = idx < n_lv * d.C * d.K;
    const int k = valid ? idx % d.K : 0, c = valid ? (idx / d.K) % d.C : 0, e = valid ? idx / (d.K * d.C) : 0;
    const int leaf = lv_leaf[e], var = lv_var[e], r = leaf_replica[leaf];
    const size_t gblk = (size_t)d.B * d.K;
    const int gsrc = DIRECT ? leaf_gsrc[2 * leaf] : 0;
    const int gcnt = DIRECT ? bwd_source_blocks(leaf_gsrc[2 * leaf + 1], d.K, d.B) : 1;
    const float* Gl = (DIRECT ? Gp + (size_t)gsrc * gblk : G + (size_t)leaf_node[leaf] * gblk) + k;
    const float* xp = x + (size_t)var * d.C + c;
    const bool shared_obs = mask_mode != EINET_MASK_SHARED || mask[var] != 0;
    float n1 = 0.f, n2 = 0.f, den = 0.f, tot = 0.f;
#pragma unroll 4
    for (int b = part_id; b < d.B; b += NCH) {
        float p = Gl[(size_t)b * d.K];
        if (DIRECT && gcnt > 1) {
            float px[GSRC_MAX_BLOCKS - 1];
#pragma unroll
            for (int q = 1; q < GSRC_MAX_BLOCKS; ++q) px[q - 1] = q < gcnt ? Gl[q * gblk + (size_t)b * d.K] : 0.f;
#pragma unroll
            for (int q = 1; q < GSRC_MAX_BLOCKS; ++q)
                if (q < gcnt) p += px[q - 1];
        }
        bool obs = shared_obs;
        if (mask_mode == EINET_MASK_PER_SAMPLE) obs = mask[(size_t)b * d.D + var] != 0;
        const float xv = xp[(size_t)b * d.D * d.C];
        const float pm = obs ? p : 0.f;
        tot += p;
        den += pm;
        n1 = fmaf(pm, xv, n1);
        n2 = fmaf(pm * xv, xv, n2);
    }
    red[part_id][0][lo] = n1;
    red[part_id][1][lo] = n2;
    red[part_id][2][lo] = den;
    red[part_id][3][lo] = tot;
    __syncthreads();
    if (part_id || !valid) return;
#pragma unroll
    for (int q = 1; q < NCH; ++q) {
        n1 += red[q][0][lo];
        n2 += red[q][1][lo];
        den += red[q][2][lo];
        tot += red[q][3][lo];
    }
    const size_t ph = phi_off + ((size_t)(var * d.C + c) * d.R + r) * d.T * d.K + k;
    stats[ph] += n1;
    if (d.T == 2) stats[ph + d.K] += n2;
    if (c == 0) {
        const size_t o = ((size_t)var * d.R + r) * d.K + k;
        stats[den_off + o] += den;
        stats[tot_off + o] += tot;
    }
}

// Categorical leaves: the sufficient statistic is the indicator of the value, so num[v][k] = sum_b [x_b = v] p[b][k] is a
// product of a one-hot matrix [V x B] with the leaf's posterior block [B x K], here on v_mfma_f32_16x16x32_bf16: the
// one-hot entries are exact in bfloat16 and a posterior is the exact sum of three bfloat16 numbers (hi, mid, lo: 24 bits),
// so three products accumulated in float32 give the float32 sum, in a fixed order.  A workgroup of four waves takes one
// leaf, 16 of the K entries and four of the leaf's (variable, channel) pairs, one pair per wave; per pass over 128 samples
// it stages the posteriors (split, sample-major) and the pairs' values in LDS.  A wave forms the operand of 16 values x 32
// samples by comparisons and keeps its V x 16 sums in registers over all passes (RT tiles of 16 values, V <= 16 RT).
// A marginalised variable's value is staged as 0xffff, which is no value; den is the sum over the observed samples.
// Bound by the posteriors' comparisons (20 vector instructions per three MFMAs) and by the read-modify-write of the table:
// 784 pairs, V = 256, K = 16, 200 samples: 18 us, where one wave per pair, a lane per entry walking the samples one
// after the other with its column of a histogram in LDS, took 125 us.
constexpr int CAT_BC = 128;                            // samples per pass
constexpr int CAT_ST = CAT_BC + 8;                     // row stride (16-bit entries): rows 16 bytes apart modulo 128
constexpr float CAT_SCALE = 0x1p+100f;                 // keeps the rests of the smallest posteriors above the smallest bfloat16
constexpr int CAT_PAIRS = 4;                           // pairs per workgroup, one per wave

template <int RT>
__global__ __launch_bounds__(256) void k_leaf_backward_categorical(
    const int32_t* __restrict__ leaf_node, const int32_t* __restrict__ leaf_replica, const int32_t* __restrict__ leaf_sptr,
    const int32_t* __restrict__ leaf_var, int chunks_per_leaf, const float* __restrict__ x, const uint8_t* __restrict__ mask,
    int mask_mode, const float* __restrict__ G, float* __restrict__ stats, int64_t phi_off, int64_t den_off,
    int64_t tot_off, Dims d) {
    __shared__ __attribute__((aligned(16))) uint16_t gs[3][16][CAT_ST];       // [part][entry][sample]
    __shared__ __attribute__((aligned(16))) uint16_t xs[CAT_PAIRS][CAT_ST];   // values
    __shared__ float red[16][17];
    const int leaf = blockIdx.x / chunks_per_leaf, p0 = (blockIdx.x - leaf * chunks_per_leaf) * CAT_PAIRS, k0 = blockIdx.y * 16;
    const int s0 = leaf_sptr[leaf], npairs = (leaf_sptr[leaf + 1] - s0) * d.C;
    if (p0 >= npairs) return;                          // (whole workgroup) this leaf has fewer chunks
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c16 = lane & 15, kg = lane >> 4;
    const int V = d.P;
    const float* Gl = G + (size_t)leaf_node[leaf] * d.B * d.K + k0;
    // staging: thread (entry sk, sample slot sb) of the posteriors; thread (pair, slot) of the values
    const int sk = tid & 15, sb = tid >> 4;
    const bool kin = k0 + sk < d.K;
    const int wpair = min(p0 + wave, npairs - 1), wvar = leaf_var[s0 + wpair / d.C], wc = wpair - wpair / d.C * d.C;
    const bool wshared = mask_mode != EINET_MASK_SHARED || mask[wvar] != 0;
    floatx4 acc[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    float tot = 0.f;                                   // thread (sk, sb): its share of sum_b p[b][k]
    for (int b0 = 0; b0 < d.B; b0 += CAT_BC) {
        const int nb = min(CAT_BC, d.B - b0);
        float g[8];
        float xv[2];
        bool ob[2];
#pragma unroll
        for (int q = 0; q < 8; ++q) g[q] = kin && 8 * sb + q < nb ? Gl[(size_t)(b0 + 8 * sb + q) * d.K + sk] : 0.f;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int b = b0 + min(lane + 64 * q, nb - 1);
            xv[q] = x[((size_t)b * d.D + wvar) * d.C + wc];
            ob[q] = lane + 64 * q < nb && wshared;
            if (mask_mode == EINET_MASK_PER_SAMPLE) ob[q] = ob[q] && mask[(size_t)b * d.D + wvar] != 0;
        }
        if (b0 > 0) __syncthreads();                   // readers of the previous pass are done
        uint32_t hi[4], mid[4], lo[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) split_bf16x3(g[2 * q] * CAT_SCALE, g[2 * q + 1] * CAT_SCALE, hi[q], mid[q], lo[q]);
        *reinterpret_cast<uint32x4*>(&gs[0][sk][8 * sb]) = uint32x4{hi[0], hi[1], hi[2], hi[3]};
        *reinterpret_cast<uint32x4*>(&gs[1][sk][8 * sb]) = uint32x4{mid[0], mid[1], mid[2], mid[3]};
        *reinterpret_cast<uint32x4*>(&gs[2][sk][8 * sb]) = uint32x4{lo[0], lo[1], lo[2], lo[3]};
        tot += ((g[0] + g[1]) + (g[2] + g[3])) + ((g[4] + g[5]) + (g[6] + g[7]));
#pragma unroll
        for (int q = 0; q < 2; ++q)
            xs[wave][lane + 64 * q] = ob[q] ? (uint16_t)min(max((int)xv[q], 0), V - 1) : (uint16_t)0xffffu;
        __syncthreads();
        for (int s = 0; s < nb; s += 32) {             // (posteriors beyond the batch are zero, their values 0xffff)
            const uint32x4 xq = *reinterpret_cast<const uint32x4*>(&xs[wave][s + 8 * kg]);
            bf16x8 bg[3];
#pragma unroll
            for (int p = 0; p < 3; ++p) bg[p] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint32x4*>(&gs[p][c16][s + 8 * kg]));
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                const uint32_t v = 16 * t + c16;       // this lane's row of the one-hot operand
                uint32x4 one;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    one[q] = ((xq[q] & 0xffffu) == v ? 0x3f80u : 0u) | ((xq[q] >> 16) == v ? 0x3f800000u : 0u);
                const bf16x8 a = __builtin_bit_cast(bf16x8, one);
#pragma unroll
                for (int p = 0; p < 3; ++p) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bg[p], acc[t], 0, 0, 0);
            }
        }
    }
    const int r = leaf_replica[leaf], k = k0 + c16;
    // acc[t][q]: value 16 t + 4 kg + q, entry k0 + c16
    const bool own = p0 + wave < npairs && k < d.K;
    float den = 0.f;
#pragma unroll
    for (int t = 0; t < RT; ++t) acc[t] *= 1.f / CAT_SCALE;
    if (own) {
        const size_t ph = phi_off + ((size_t)(wvar * d.C + wc) * d.R + r) * V * d.K + k;
        // (the old statistics are requested before the first store: one memory latency, not one per value)
        float nold[RT][4];
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) nold[t][q] = stats[ph + (size_t)min(16 * t + 4 * kg + q, V - 1) * d.K];
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int v = 16 * t + 4 * kg + q;
                den += acc[t][q];                      // (rows beyond V are zero)
                if (v < V) stats[ph + (size_t)v * d.K] = nold[t][q] + acc[t][q];
            }
    }
    den += __shfl_xor(den, 16, 64);
    den += __shfl_xor(den, 32, 64);
    red[sk][sb] = tot;
    __syncthreads();
    if (own && wc == 0 && kg == 0) {
        float t4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 16; ++q) t4[q & 3] += red[c16][q];
        const size_t o = ((size_t)wvar * d.R + r) * d.K + k;
        stats[den_off + o] += den;
        stats[tot_off + o] += (t4[0] + t4[1]) + (t4[2] + t4[3]);
    }
}

// The same statistics for leaves of at least 16 (variable, channel) pairs (image cells and strips, long variable lists):
// num[pair][k] = sum_b x[b][pair] p[b][k], the same with x^2 for Gaussian leaves (SQ) and with the observation flags (MASK),
// is a product with the batch as contraction, on the bfloat16 matrix pipe at float32 precision (bf16x6.hpp).  A wave takes
// 16 pairs (the rows) and all entries k; a lane's operand, eight samples of its pair, comes straight from memory (a load
// reads 16 pairs side by side) and is requested a step of 64 samples ahead; the flags are exact in bfloat16.  (Posteriors times
// 2^24, so that the third part of a small one is a normal number; values and flags times 2^-24.  Squares below 2^-85 would
// lose bits by that: a wave that has met such values forms its sums again, see leaf_sums_float32.)  The leaf's
// posteriors, which all waves share, are split into bfloat16 parts once per workgroup and step and go through LDS.
// tot = sum_b p[b][k] is summed on the side.
// Runs in one launch with the mixing statistics, hence the eight waves; `waves` of them have pairs.
// Bound by the loads of the values, which no other workgroup reads: strips of 128 x 128 x 3 images, K = 40, 500 samples:
// 51 us, with the values staged through LDS for float32 matrix instructions and the batch cut into groups 91 + 10 us.
constexpr int LX_THREADS = 512;
constexpr int LX_STEP = 64, LX_RB = LX_STEP + 8;       // samples per step; row stride (bfloat16) of the posteriors
// Smallest of `least` and of the values that are not zero, as twice its bits less one.
__device__ __forceinline__ uint32_t smallest_value(uint32_t least, const float (&v)[8]) {
#pragma unroll
    for (int c = 0; c < 8; ++c) least = min(least, (__builtin_bit_cast(uint32_t, v[c]) << 1) - 1u);
    return least;
}
__device__ __forceinline__ bool squares_lose_bits(uint32_t least) {
    return __any(least < (__builtin_bit_cast(uint32_t, 0x1p-42f) << 1) - 1u);
}
// The sums of x p and x^2 p of a wave's 16 pairs once more, in float32 throughout: samples first .. first + run - 1 and every
// `stride` on.  Only waves with values between 0 and 2^-42 come here.  xp, mp: the lane's pair; Gl: the leaf's gcnt blocks.
template <bool MASK, int NJ>
__device__ __forceinline__ void leaf_sums_float32(floatx4 (&sum)[2][NJ], int first, int run, int stride, const float* xp,
                                               size_t xstride, const uint8_t* mp, size_t mstride, const float* Gl, int gcnt, int B,
                                               int K) {
    const int lane = threadIdx.x & 63, c16 = lane & 15, kg = lane >> 4;
    const size_t gblk = (size_t)B * K;
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int jt = 0; jt < NJ; ++jt) sum[q][jt] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int s = first; s < B; s += stride)
        for (int u = 0; u < run && s + u < B; u += 4) {
            const int b = s + u + kg, bc = min(b, B - 1);      // lane group kg: one of four samples
            const float x = !MASK || mp[bc * mstride] ? xp[bc * xstride] : 0.f;
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt) {
                const int k = 16 * jt + c16;
                float p = 0.f;
                for (int y = 0; y < gcnt; ++y) p += b < B && k < K ? Gl[y * gblk + (size_t)bc * K + k] : 0.f;
                sum[0][jt] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, p, sum[0][jt], 0, 0, 0);
                sum[1][jt] = __builtin_amdgcn_mfma_f32_16x16x4f32(x * x, p, sum[1][jt], 0, 0, 0);
            }
        }
}
template <bool SQ, bool MASK, int NJ, bool DIRECT>
__device__ __forceinline__ void leaf_stats_body(
    int block, int chunks_per_leaf, int waves, const int32_t* __restrict__ leaf_node, const int32_t* __restrict__ leaf_replica,
    const int32_t* __restrict__ leaf_sptr, const int32_t* __restrict__ leaf_var, const float* __restrict__ x,
    const uint8_t* __restrict__ mask, int mask_mode, const float* __restrict__ G, const float* __restrict__ Gp,
    const int32_t* __restrict__ leaf_gsrc, float* __restrict__ stats, int64_t phi_off, int64_t den_off, int64_t tot_off,
    const Dims& d) {
    constexpr int NR = 16 * NJ;                        // columns, padded
    __shared__ __attribute__((aligned(16))) uint16_t ps[2][3][NR][LX_RB];
    constexpr int NG = LX_STEP / 4, NI = (NR * NG + LX_THREADS - 1) / LX_THREADS;     // groups of four samples; items per thread
    __shared__ float red[NG][NR];
    const int leaf = block / chunks_per_leaf, chunk = block - leaf * chunks_per_leaf;
    const int s0 = leaf_sptr[leaf], npairs = (leaf_sptr[leaf + 1] - s0) * d.C;
    if (16 * waves * chunk >= npairs) return;          // (whole workgroup) this leaf has fewer chunks
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c16 = lane & 15, kg = lane >> 4;
    const size_t gblk = (size_t)d.B * d.K;
    const float* Gl = DIRECT ? Gp + (size_t)leaf_gsrc[2 * leaf] * gblk : G + (size_t)leaf_node[leaf] * gblk;
    const int gcnt = DIRECT ? bwd_source_blocks(leaf_gsrc[2 * leaf + 1], d.K, d.B) : 1;
    // this lane's pair
    const int tile = chunk * waves + wave, pair = 16 * tile + c16;
    const bool work = wave < waves && 16 * tile < npairs;
    const int pv = min(pair, npairs - 1), var = leaf_var[s0 + pv / d.C];
    const size_t xstride = (size_t)d.D * d.C;
    const float* xp = x + (size_t)var * d.C + (pv - pv / d.C * d.C);
    const uint8_t* mp = MASK ? mask + var : nullptr;
    // staging: item (entry, four samples) of the posteriors
    float g[NI][4], xv[LX_STEP / 32][8];
    uint8_t ob[LX_STEP / 32][8];
    auto fetch = [&](int s) {
#pragma unroll
        for (int x = 0; x < NI; ++x) {
            const int f = tid + LX_THREADS * x, k = f % NR, b = s + 4 * (f / NR);
            const float* src = Gl + (size_t)b * d.K + k;
#pragma unroll
            for (int q = 0; q < 4; ++q) g[x][q] = k < d.K && f < NR * NG && b + q < d.B ? src[(size_t)q * d.K] : 0.f;
            for (int y = 1; y < gcnt; ++y) {
                float m[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) m[q] = k < d.K && f < NR * NG && b + q < d.B ? src[y * gblk + (size_t)q * d.K] : 0.f;
#pragma unroll
                for (int q = 0; q < 4; ++q) g[x][q] += m[q];
            }
        }
        if (work) {
#pragma unroll
            for (int u = 0; u < LX_STEP / 32; ++u)
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int b = min(s + 32 * u + 8 * kg + q, d.B - 1);       // (beyond the batch the posteriors are zero)
                    xv[u][q] = xp[(size_t)b * xstride];
                    if (MASK) ob[u][q] = mp[mask_mode == EINET_MASK_PER_SAMPLE ? (size_t)b * d.D : 0];
                }
        }
    };
    float tot[NI];
#pragma unroll
    for (int x = 0; x < NI; ++x) tot[x] = 0.f;
    auto stage = [&](int buf) {
#pragma unroll
        for (int x = 0; x < NI; ++x) {
            const int f = tid + LX_THREADS * x;
            if (f >= NR * NG) continue;
            uint32_t p0[3], p1[3];
            split_bf16x3(g[x][0] * X6_SCALE, g[x][1] * X6_SCALE, p0[0], p0[1], p0[2]);
            split_bf16x3(g[x][2] * X6_SCALE, g[x][3] * X6_SCALE, p1[0], p1[1], p1[2]);
#pragma unroll
            for (int p = 0; p < 3; ++p) *reinterpret_cast<uint2*>(&ps[buf][p][f % NR][4 * (f / NR)]) = make_uint2(p0[p], p1[p]);
            tot[x] += (g[x][0] + g[x][1]) + (g[x][2] + g[x][3]);
        }
    };
    constexpr int NK = 1 + (SQ ? 1 : 0) + (MASK ? 1 : 0);
    floatx4 acc[NK][NJ];
#pragma unroll
    for (int q = 0; q < NK; ++q)
#pragma unroll
        for (int jt = 0; jt < NJ; ++jt) acc[q][jt] = floatx4{0.f, 0.f, 0.f, 0.f};
    uint32_t least = ~0u;
    fetch(0);
    stage(0);
    for (int s = 0, buf = 0; s < d.B; s += LX_STEP, buf ^= 1) {
        float xc[LX_STEP / 32][8];
        uint32x4 one[LX_STEP / 32];
#pragma unroll
        for (int u = 0; u < LX_STEP / 32; ++u) {
#pragma unroll
            for (int q = 0; q < 8; ++q) xc[u][q] = !MASK || ob[u][q] ? xv[u][q] : 0.f;
            if (SQ && work) least = smallest_value(least, xc[u]);
            if (MASK) {
#pragma unroll
                for (int q = 0; q < 4; ++q) one[u][q] = (ob[u][2 * q] ? 0x3380u : 0u) | (ob[u][2 * q + 1] ? 0x33800000u : 0u);
            }
        }
        __syncthreads();                               // the step is staged; readers of the other buffer are done
        const bool more = s + LX_STEP < d.B;
        if (more) fetch(s + LX_STEP);
#pragma unroll
        for (int u = 0; u < LX_STEP / 32; ++u) {
            if (!work || s + 32 * u >= d.B) continue;
            constexpr int NQ = SQ ? 2 : 1, PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};     // (small parts first)
            uint32x4 a[NQ][3];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                float w[8];
#pragma unroll
                for (int c = 0; c < 8; ++c) w[c] = xc[u][c] * (q == 0 ? 1.f : xc[u][c]) * (1.f / X6_SCALE);
                split_octet(w, a[q][0], a[q][1], a[q][2]);
            }
            // (a column tile at a time and its sums added afterwards: few registers, and one rounding of the sums per step)
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt) {
                uint32x4 pb[3];
                floatx4 t[NK];
#pragma unroll
                for (int p = 0; p < 3; ++p) pb[p] = *reinterpret_cast<const uint32x4*>(&ps[buf][p][16 * jt + c16][32 * u + 8 * kg]);
#pragma unroll
                for (int q = 0; q < NK; ++q) t[q] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int p = 0; p < 6; ++p)
#pragma unroll
                    for (int q = 0; q < NQ; ++q) t[q] = mfma_bf16(a[q][PA[p]], pb[PB[p]], t[q]);
                if constexpr (MASK) {
#pragma unroll
                    for (int p = 2; p >= 0; --p) t[NK - 1] = mfma_bf16(one[u], pb[p], t[NK - 1]);
                }
#pragma unroll
                for (int q = 0; q < NK; ++q) acc[q][jt] += t[q];
            }
        }
        if (more) stage(buf ^ 1);
    }
#pragma unroll
    for (int x = 0; x < NI; ++x) {
        const int f = tid + LX_THREADS * x;
        if (f < NR * NG) red[f / NR][f % NR] = tot[x];
    }
    __syncthreads();
    if (!work) return;
    if constexpr (SQ) {
        if (squares_lose_bits(least)) {
            floatx4 sum[2][NJ];
            leaf_sums_float32<MASK, NJ>(sum, 0, d.B, d.B, xp, xstride, mp, mask_mode == EINET_MASK_PER_SAMPLE ? d.D : 0, Gl, gcnt, d.B, d.K);
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int jt = 0; jt < NJ; ++jt) acc[q][jt] = sum[q][jt];
        }
    }
    // acc[q][jt][v]: pair 16 tile + 4 kg + v, entry 16 jt + c16
    const int r = leaf_replica[leaf];
#pragma unroll
    for (int jt = 0; jt < NJ; ++jt) {
        const int k = 16 * jt + c16;
        float t = 0.f;
#pragma unroll
        for (int h = 0; h < NG; ++h) t += red[h][k];
        // (the old statistics of the four pairs are requested before the first store)
        size_t ph[4], o[4];
        float old[4][4];
        bool first[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int p = 16 * tile + 4 * kg + v, pc = min(p, npairs - 1);
            const int vv = leaf_var[s0 + pc / d.C], c = pc - pc / d.C * d.C;
            first[v] = c == 0;
            ph[v] = phi_off + ((size_t)(vv * d.C + c) * d.R + r) * d.T * d.K + k;
            o[v] = ((size_t)vv * d.R + r) * d.K + k;
            if (p < npairs && k < d.K) {
                old[v][0] = stats[ph[v]];
                if (SQ) old[v][1] = stats[ph[v] + d.K];
                if (first[v]) old[v][2] = stats[den_off + o[v]], old[v][3] = stats[tot_off + o[v]];
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if (16 * tile + 4 * kg + v >= npairs || k >= d.K) continue;
            stats[ph[v]] = old[v][0] + acc[0][jt][v];
            if (SQ) stats[ph[v] + d.K] = old[v][1] + acc[SQ ? 1 : 0][jt][v];
            if (first[v]) {
                stats[den_off + o[v]] = old[v][2] + (MASK ? acc[NK - 1][jt][v] : t);
                stats[tot_off + o[v]] = old[v][3] + t;
            }
        }
    }
}

// The same for models with few tiles of 16 pairs: a workgroup takes one tile and deals the batch to its eight waves, 32 samples
// at a time; every wave splits the posteriors of its own samples, so nothing is shared before the waves' sums meet at the end.
// With mixing statistics, us of the launch (in brackets: both operands staged through LDS, a thread per (pair, entry)): 32x32x3
// images in cells of 8 x 8, K = 40: 13.3 for 128 samples (14.7), 47 for 1000 (80); 28x28 in cells, K = 16, 256 samples, with flags:
// 8.0 (18.0); lists of variables, K = 20, 200 samples: 9.3 (16.8).
template <bool SQ, bool MASK, int NJ>
struct LeafTileLds {
    static constexpr int NR = 16 * NJ, NK = 1 + (SQ ? 1 : 0) + (MASK ? 1 : 0);
    static constexpr int RB = 40;                      // row stride (bfloat16) of a wave's 32 samples
    static constexpr int WAVE = 3 * NR * RB * 2;       // bytes of a wave's posteriors
    static constexpr int SUMS = NK * NJ * 1024 + 8 * NR * 4;      // .. of its sums: [kind][jt][lane][4], tot [8][NR]
    static constexpr int BYTES = 8 * (WAVE > SUMS ? WAVE : SUMS);
};
template <bool SQ, bool MASK, int NJ, bool DIRECT>
__device__ __forceinline__ void leaf_tile_body(
    int block, int tiles_per_leaf, char* lds, const int32_t* __restrict__ leaf_node, const int32_t* __restrict__ leaf_replica,
    const int32_t* __restrict__ leaf_sptr, const int32_t* __restrict__ leaf_var, const float* __restrict__ x,
    const uint8_t* __restrict__ mask, int mask_mode, const float* __restrict__ G, const float* __restrict__ Gp,
    const int32_t* __restrict__ leaf_gsrc, float* __restrict__ stats, int64_t phi_off, int64_t den_off, int64_t tot_off,
    const Dims& d) {
    using LY = LeafTileLds<SQ, MASK, NJ>;
    constexpr int NR = LY::NR, NK = LY::NK, NI = NR * 8 / 64;        // items (entry, four samples) per lane
    const int leaf = block / tiles_per_leaf, tile = block - leaf * tiles_per_leaf;
    const int s0 = leaf_sptr[leaf], npairs = (leaf_sptr[leaf + 1] - s0) * d.C;
    if (16 * tile >= npairs) return;                   // (whole workgroup) this leaf has fewer tiles
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c16 = lane & 15, kg = lane >> 4;
    const size_t gblk = (size_t)d.B * d.K;
    const float* Gl = DIRECT ? Gp + (size_t)leaf_gsrc[2 * leaf] * gblk : G + (size_t)leaf_node[leaf] * gblk;
    const int gcnt = DIRECT ? bwd_source_blocks(leaf_gsrc[2 * leaf + 1], d.K, d.B) : 1;
    const int pv = min(16 * tile + c16, npairs - 1), var = leaf_var[s0 + pv / d.C];
    const size_t xstride = (size_t)d.D * d.C;
    const float* xp = x + (size_t)var * d.C + (pv - pv / d.C * d.C);
    const uint8_t* mp = MASK ? mask + var : nullptr;
    uint16_t* ps = reinterpret_cast<uint16_t*>(lds + wave * LY::WAVE);      // [part][entry][RB]
    floatx4 acc[NK][NJ];
    float tot[NI];
#pragma unroll
    for (int q = 0; q < NK; ++q)
#pragma unroll
        for (int jt = 0; jt < NJ; ++jt) acc[q][jt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int y = 0; y < NI; ++y) tot[y] = 0.f;
    uint32_t least = ~0u;
    for (int s = 32 * wave; s < d.B; s += 256) {
        float g[NI][4], xv[8];
        uint8_t ob[8];
#pragma unroll
        for (int y = 0; y < NI; ++y) {
            const int f = lane + 64 * y, k = f % NR, b = s + 4 * (f / NR);
            const float* src = Gl + (size_t)b * d.K + k;
#pragma unroll
            for (int q = 0; q < 4; ++q) g[y][q] = k < d.K && b + q < d.B ? src[(size_t)q * d.K] : 0.f;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int b = min(s + 8 * kg + q, d.B - 1);           // (samples beyond the batch: their posteriors are zero)
            xv[q] = xp[(size_t)b * xstride];
            if (MASK) ob[q] = mp[mask_mode == EINET_MASK_PER_SAMPLE ? (size_t)b * d.D : 0];
        }
        for (int z = 1; z < gcnt; ++z) {
#pragma unroll
            for (int y = 0; y < NI; ++y) {
                const int f = lane + 64 * y, k = f % NR, b = s + 4 * (f / NR);
                const float* src = Gl + z * gblk + (size_t)b * d.K + k;
#pragma unroll
                for (int q = 0; q < 4; ++q) g[y][q] += k < d.K && b + q < d.B ? src[(size_t)q * d.K] : 0.f;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");    // (the LDS serves a wave's requests in order)
#pragma unroll
        for (int y = 0; y < NI; ++y) {
            const int f = lane + 64 * y;
            uint32_t p0[3], p1[3];
            split_bf16x3(g[y][0] * X6_SCALE, g[y][1] * X6_SCALE, p0[0], p0[1], p0[2]);
            split_bf16x3(g[y][2] * X6_SCALE, g[y][3] * X6_SCALE, p1[0], p1[1], p1[2]);
#pragma unroll
            for (int p = 0; p < 3; ++p)
                *reinterpret_cast<uint2*>(ps + (p * NR + f % NR) * LY::RB + 4 * (f / NR)) = make_uint2(p0[p], p1[p]);
            tot[y] += (g[y][0] + g[y][1]) + (g[y][2] + g[y][3]);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        uint32x4 pb[NJ][3];
#pragma unroll
        for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
            for (int p = 0; p < 3; ++p) pb[jt][p] = *reinterpret_cast<const uint32x4*>(ps + (p * NR + 16 * jt + c16) * LY::RB + 8 * kg);
        constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};     // (small parts first)
        if (MASK) {
#pragma unroll
            for (int c = 0; c < 8; ++c) xv[c] = ob[c] ? xv[c] : 0.f;
        }
        if (SQ) least = smallest_value(least, xv);
#pragma unroll
        for (int q = 0; q < (SQ ? 2 : 1); ++q) {
            float w[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) w[c] = xv[c] * (q == 0 ? 1.f : xv[c]) * (1.f / X6_SCALE);
            uint32x4 a[3];
            split_octet(w, a[0], a[1], a[2]);
            floatx4 t[NJ];
#pragma unroll
            for (int p = 0; p < 6; ++p)
#pragma unroll
                for (int jt = 0; jt < NJ; ++jt)
                    t[jt] = mfma_bf16(a[PA[p]], pb[jt][PB[p]], p == 0 ? floatx4{0.f, 0.f, 0.f, 0.f} : t[jt]);
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt) acc[q][jt] += t[jt];
        }
        if constexpr (MASK) {
            uint32x4 one;
#pragma unroll
            for (int q = 0; q < 4; ++q) one[q] = (ob[2 * q] ? 0x3380u : 0u) | (ob[2 * q + 1] ? 0x33800000u : 0u);
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt) {              // (small parts first, one rounding of the sums per step)
                floatx4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int p = 2; p >= 0; --p) t = mfma_bf16(one, pb[jt][p], t);
                acc[NK - 1][jt] += t;
            }
        }
    }
    if constexpr (SQ) {
        if (squares_lose_bits(least)) {
            floatx4 sum[2][NJ];
            leaf_sums_float32<MASK, NJ>(sum, 32 * wave, 32, 256, xp, xstride, mp, mask_mode == EINET_MASK_PER_SAMPLE ? d.D : 0, Gl, gcnt,
                                        d.B, d.K);
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int jt = 0; jt < NJ; ++jt) acc[q][jt] = sum[q][jt];
        }
    }
    __syncthreads();                                   // every wave is done with its posteriors
    {
        floatx4* out = reinterpret_cast<floatx4*>(lds + wave * LY::SUMS);
#pragma unroll
        for (int q = 0; q < NK; ++q)
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt) out[(q * NJ + jt) * 64 + lane] = acc[q][jt];
        float* t = reinterpret_cast<float*>(lds + wave * LY::SUMS + NK * NJ * 1024);
#pragma unroll
        for (int y = 0; y < NI; ++y) t[lane + 64 * y] = tot[y];       // [sample group][entry]
    }
    __syncthreads();
    // block (q, jt) of the sums is finished by one wave: pair 16 tile + 4 kg + v, entry 16 jt + c16
    const int r = leaf_replica[leaf];
    for (int blk = wave; blk < NK * NJ; blk += 8) {
        const int q = blk / NJ, k = 16 * (blk - q * NJ) + c16;
        floatx4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 8; ++w) sum += reinterpret_cast<const floatx4*>(lds + w * LY::SUMS)[blk * 64 + lane];
        float t = 0.f;
        if (q == 0 || q == NK - 1)
#pragma unroll 2
            for (int w = 0; w < 8; ++w)                // (all at once would take 64 registers)
#pragma unroll
                for (int h = 0; h < 8; ++h) t += reinterpret_cast<const float*>(lds + w * LY::SUMS + NK * NJ * 1024)[h * NR + k];
        // (the old statistics are requested before the first store)
        size_t ph[4], o[4];
        float old[4][3];
        bool in[4], first[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int p = 16 * tile + 4 * kg + v, pc = min(p, npairs - 1);
            const int vv = leaf_var[s0 + pc / d.C], c = pc - pc / d.C * d.C;
            in[v] = p < npairs && k < d.K;
            first[v] = in[v] && c == 0;
            ph[v] = phi_off + (((size_t)(vv * d.C + c) * d.R + r) * d.T + q) * d.K + k;
            o[v] = ((size_t)vv * d.R + r) * d.K + k;
            if (in[v] && q < (SQ ? 2 : 1)) old[v][0] = stats[ph[v]];
            if (first[v] && q == 0) old[v][1] = stats[tot_off + o[v]];
            if (first[v] && q == NK - 1) old[v][2] = stats[den_off + o[v]];
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if (in[v] && q < (SQ ? 2 : 1)) stats[ph[v]] = old[v][0] + sum[v];
            if (first[v] && q == 0) stats[tot_off + o[v]] = old[v][1] + t;
            if (first[v] && q == NK - 1) stats[den_off + o[v]] = old[v][2] + (MASK ? sum[v] : t);
        }
    }
}

// Last launch of the top-down pass: leaf statistics in the first n_leaf_blocks workgroups, mixing
// statistics in the others (item = idx / max_children, child = idx % max_children).
template <int NCH, bool DIRECT>
__global__ __launch_bounds__(1024) void k_tail_backward(
    int n_leaf_blocks, int max_children, const int32_t* __restrict__ lv_leaf, const int32_t* __restrict__ lv_var,
    const int32_t* __restrict__ leaf_node, const int32_t* __restrict__ leaf_replica, int n_lv,
    const float* __restrict__ x, const uint8_t* __restrict__ mask, int mask_mode, const float* __restrict__ G,
    const float* __restrict__ Gp, const int32_t* __restrict__ leaf_gsrc,
    float* __restrict__ stats, int64_t phi_off, int64_t den_off, int64_t tot_off, const int32_t* __restrict__ m_rec,
    const int32_t* __restrict__ m_cptr, const int32_t* __restrict__ m_child, const float* __restrict__ params,
    const float* __restrict__ A, const double* __restrict__ Off, Dims d) {
    const int blk = blockIdx.x;
    if (blk < n_leaf_blocks) {
        leaf_backward_body<NCH, DIRECT>(blk, lv_leaf, lv_var, leaf_node, leaf_replica, n_lv, x, mask, mask_mode, G, Gp,
                                        leaf_gsrc, stats, phi_off, den_off, tot_off, d);
    } else {
        const int idx = blk - n_leaf_blocks;
        mixing_stats_body<1024>(idx / max_children, idx % max_children, m_rec, m_cptr, m_child, params, stats, A, Off, G,
                                d.B, d.K);
    }
}

// The same with the leaves' statistics as matrix products (TILE: a tile per workgroup).
template <bool SQ, bool MASK, int NJ, bool DIRECT, bool TILE>
__global__ __launch_bounds__(LX_THREADS, TILE || MASK || NJ > 3 ? 2 : 4) void k_tail_backward_matrix(
    int n_leaf_blocks, int chunks_per_leaf, int waves, int max_children, const int32_t* __restrict__ leaf_node,
    const int32_t* __restrict__ leaf_replica, const int32_t* __restrict__ leaf_sptr, const int32_t* __restrict__ leaf_var,
    const float* __restrict__ x, const uint8_t* __restrict__ mask, int mask_mode, const float* __restrict__ G,
    const float* __restrict__ Gp, const int32_t* __restrict__ leaf_gsrc, float* __restrict__ stats, int64_t phi_off,
    int64_t den_off, int64_t tot_off, const int32_t* __restrict__ m_rec, const int32_t* __restrict__ m_cptr,
    const int32_t* __restrict__ m_child, const float* __restrict__ params, const float* __restrict__ A,
    const double* __restrict__ Off, Dims d) {
    const int blk = blockIdx.x;
    if (blk < n_leaf_blocks) {
        if constexpr (TILE) {
            extern __shared__ __attribute__((aligned(16))) char tile_lds[];
            leaf_tile_body<SQ, MASK, NJ, DIRECT>(blk, chunks_per_leaf, tile_lds, leaf_node, leaf_replica, leaf_sptr, leaf_var, x,
                                                 mask, mask_mode, G, Gp, leaf_gsrc, stats, phi_off, den_off, tot_off, d);
        } else {
            leaf_stats_body<SQ, MASK, NJ, DIRECT>(blk, chunks_per_leaf, waves, leaf_node, leaf_replica, leaf_sptr, leaf_var, x,
                                                  mask, mask_mode, G, Gp, leaf_gsrc, stats, phi_off, den_off, tot_off, d);
        }
    } else {
        const int idx = blk - n_leaf_blocks;
        mixing_stats_body<LX_THREADS>(idx / max_children, idx % max_children, m_rec, m_cptr, m_child, params, stats, A, Off, G,
                                d.B, d.K);
    }
}

}  // namespace

void launch_tail_backward(const DevTables& t, int n_lv, int n_leaves, int max_scope, int n_mix, int max_children,
                          const float* x, const uint8_t* mask, int mask_mode, const float* params, const float* A,
                          const double* Off, const float* G, const float* Gp, bool direct, float* stats,
                          int64_t phi_off, int64_t den_off, int64_t tot_off, const Dims& d, hipStream_t s) {
    const int total = n_lv * d.C * d.K;
    const bool categorical = d.family == EINET_LEAF_CATEGORICAL;
    if (categorical) {   // indicator statistics: a kernel of their own (at most 256 values)
        const int cpl = (max_scope * d.C + CAT_PAIRS - 1) / CAT_PAIRS;
        const dim3 grid(n_leaves * cpl, (d.K + 15) / 16);
#define EINET_CAT(RT)                                                                                              \
    hipLaunchKernelGGL(k_leaf_backward_categorical<RT>, grid, dim3(256), 0, s, t.leaf_node, t.leaf_replica,          \
                       t.leaf_sptr, t.leaf_var, cpl, x, mask, mask_mode, G, stats, phi_off, den_off, tot_off, d)
        if (d.P <= 16) EINET_CAT(1);
        else if (d.P <= 32) EINET_CAT(2);
        else if (d.P <= 64) EINET_CAT(4);
        else if (d.P <= 128) EINET_CAT(8);
        else EINET_CAT(16);
#undef EINET_CAT
    }
    const int mc = max_children > 0 ? max_children : 1, n_mix_blocks = n_mix * max_children;
    // Scopes that fill a tile of 16 pairs: on the matrix pipe, from the batch on that an instruction contracts half of.  Eight
    // waves with a tile each, which split the posteriors once for all, where that makes enough workgroups and a workgroup of one
    // tile would give most of its waves no samples (up to 64) or there are many tiles; otherwise a tile per workgroup, whose waves
    // share the batch.  Us of an EM step, a thread per entry / one tile / eight tiles: 128 leaves of 32 pairs, K = 40, 16 samples
    // 143 / 144 / 141, 64 samples 170 / 159 / 157, 128 samples 201 / 182 / 186; 64 leaves of 192 pairs, K = 20, 4 samples 159 / 166 /
    // 161, 64 samples 198 / 187 / 183, 400 samples 433 / 405 / 406; 8 leaves of 128 pairs, K = 40, 16 samples 53 / 55 / 58, 64 samples 58 /
    // 59 / 63, 200 samples 79 / 78 / 89; 16 leaves of 64 pairs with flags, K = 10, 64 samples 114 / 113 / 112, 128 samples 121 / 117 / 118.
    const int tiles = (max_scope * d.C + 15) / 16, waves = LX_THREADS / 64, eights = (tiles + waves - 1) / waves;
    const bool tile = (int64_t)n_leaves * eights < 64 || (d.B > 64 && (int64_t)n_leaves * tiles <= 2 * EINET_NUM_CUS);
    const bool matrix = max_scope * d.C >= 16 && d.B > (tile ? 16 : 8);
    if (!categorical && matrix) {
        const int chunks = tile ? tiles : eights;
        const int n_leaf_blocks = n_leaves * chunks;
#define EINET_LAUNCH_T(SQ, MASK, NJ, DIR, TILE)                                                                         \
    do {                                                                                                                \
        const size_t lds = TILE ? LeafTileLds<SQ, MASK, NJ>::BYTES : 0;                                                 \
        if (lds > 64 * 1024) {                                                                                          \
            static std::once_flag attr_set[EINET_MAX_DEVICES];                                                          \
            int dev = 0;                                                                                                \
            (void)hipGetDevice(&dev);                                                                                   \
            std::call_once(attr_set[dev % EINET_MAX_DEVICES],                                                           \
                           [&] { allow_dynamic_lds(&k_tail_backward_matrix<SQ, MASK, NJ, DIR, TILE>, lds); });          \
        }                                                                                                               \
        hipLaunchKernelGGL((k_tail_backward_matrix<SQ, MASK, NJ, DIR, TILE>), dim3(n_leaf_blocks + n_mix_blocks),       \
                           dim3(LX_THREADS), lds, s, n_leaf_blocks, chunks, waves, mc, t.leaf_node, t.leaf_replica,     \
                           t.leaf_sptr, t.leaf_var, x, mask, mask_mode, G, Gp, t.leaf_gsrc, stats, phi_off, den_off,    \
                           tot_off, t.mix_rec, t.mix_cptr, t.mix_child, params, A, Off, d);                             \
    } while (0)
#define EINET_LAUNCH_D(SQ, MASK, NJ, DIR)                    \
    do {                                                     \
        if (tile) EINET_LAUNCH_T(SQ, MASK, NJ, DIR, true);   \
        else EINET_LAUNCH_T(SQ, MASK, NJ, DIR, false);       \
    } while (0)
#define EINET_LAUNCH_M(SQ, MASK, NJ)                         \
    do {                                                     \
        if (direct) EINET_LAUNCH_D(SQ, MASK, NJ, true);      \
        else EINET_LAUNCH_D(SQ, MASK, NJ, false);            \
    } while (0)
#define EINET_LAUNCH(NJ)                                                      \
    do {                                                                      \
        const bool masked = mask_mode != EINET_MASK_NONE;                     \
        if (d.T == 2 && masked) EINET_LAUNCH_M(true, true, NJ);               \
        else if (d.T == 2) EINET_LAUNCH_M(true, false, NJ);                   \
        else if (masked) EINET_LAUNCH_M(false, true, NJ);                     \
        else EINET_LAUNCH_M(false, false, NJ);                                \
    } while (0)
        switch ((d.K + 15) / 16) {
            case 1: EINET_LAUNCH(1); break;
            case 2: EINET_LAUNCH(2); break;
            case 3: EINET_LAUNCH(3); break;
            default: EINET_LAUNCH(4); break;
        }
#undef EINET_LAUNCH
#undef EINET_LAUNCH_M
#undef EINET_LAUNCH_D
#undef EINET_LAUNCH_T
        return;
    }
    // short scopes: a thread per statistic, straight from memory (eight parts of the batch from 64 samples on: 17.4 -> 15.5 us
    // for 2560 leaves of three variables and 100 samples; sixteen: 21.6 us)
    const int nch = d.B >= 64 ? 8 : d.B >= 16 ? 4 : 1;
    const int n_leaf_blocks = categorical ? 0 : (total + 1024 / nch - 1) / (1024 / nch);
    const int blocks = n_leaf_blocks + n_mix_blocks;
    if (blocks == 0) return;
#define EINET_LAUNCH_D(N, DIR)                                                                                       \
    hipLaunchKernelGGL((k_tail_backward<N, DIR>), dim3(blocks), dim3(1024), 0, s, n_leaf_blocks, mc, t.lv_leaf, t.lv_var, \
                       t.leaf_node, t.leaf_replica, n_lv, x, mask, mask_mode, G, Gp, t.leaf_gsrc, stats, phi_off, den_off, \
                       tot_off, t.mix_rec, t.mix_cptr, t.mix_child, params, A, Off, d)
#define EINET_LAUNCH(N)                       \
    do {                                      \
        if (direct) EINET_LAUNCH_D(N, true);  \
        else EINET_LAUNCH_D(N, false);        \
    } while (0)
    if (nch == 8) EINET_LAUNCH(8);
    else if (nch == 4) EINET_LAUNCH(4);
    else EINET_LAUNCH(1);
#undef EINET_LAUNCH
#undef EINET_LAUNCH_D
}

}  // namespace einet_impl
