// Top-down sampling (Sec. 2, Sec. 4.2, App. D).
#include "device_common.hpp"

namespace einet_impl {

namespace {

// ------------------------------------------------------------------ top-down sampling (Sec. 2, Sec. 4.2, App. D)
// sel[b][node]: entry of the node that sample b uses, -1 if the sample does not reach the node (one byte: K is at most
// 64).  In a decomposable circuit a sample reaches a region at most once (two paths to it would sit under two
// children of one product, whose scopes are disjoint), so the writes below never collide.
__host__ __device__ inline int sample_sel_stride(int num_nodes) { return (num_nodes + 3) & ~3; }
// Choices of a sample are kept in LDS up to this many nodes, beyond it in its row of `sel` itself.
constexpr int SAMPLE_LDS_NODES = 60 * 1024;

// A choice from unnormalised weights w_0..w_{n-1} with a uniform u is the first index whose running sum
// exceeds u times the total.
//
// Region with several partitions: partition c has weight v[k][c] * S^c[k] / S[k] given the evidence
// (App. B), v[k][c] without.  Every lane of the wave walks the few partitions; all get the same answer.
__device__ __forceinline__ int sample_partition(int mi, int s, int k, int b, const int32_t* __restrict__ m_cptr,
                                                const int32_t* __restrict__ m_child,
                                                const int32_t* __restrict__ m_voff, int evidence,
                                                const float* __restrict__ params, const float* __restrict__ A,
                                                const double* __restrict__ Off, const float* __restrict__ u,
                                                int num_partitions, int B, int K) {
    const int c0 = m_cptr[mi], nc = m_cptr[mi + 1] - c0;
    const float* v = params + m_voff[mi] + (size_t)k * nc;
    const size_t srow = (size_t)s * B + b;
    float total = 0.f;
    for (int c = 0; c < nc; ++c) {
        const size_t row = (size_t)m_child[c0 + c] * B + b;
        total += evidence ? v[c] * expf((float)(Off[row] - Off[srow]) + A[row * K + k] - A[srow * K + k]) : v[c];
    }
    const float tau = u[(size_t)(num_partitions + s) * B + b] * total;
    float run = 0.f;
    int pick = -1, last = 0;
    for (int c = 0; c < nc; ++c) {
        const size_t row = (size_t)m_child[c0 + c] * B + b;
        const float w = evidence ? v[c] * expf((float)(Off[row] - Off[srow]) + A[row * K + k] - A[srow * K + k]) : v[c];
        run += w;
        if (w > 0.f) last = c;
        if (pick < 0 && run > tau) pick = c;
    }
    return pick < 0 ? last : pick;                   // u so close to 1 that rounding ate the last interval
}

// Inclusive sums over the lanes of a wave.
__device__ __forceinline__ float wave_scan(float v, int lane) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const float up = __shfl_up(v, o, 64);
        if (lane >= o) v += up;
    }
    return v;
}

// First lane whose running sum exceeds tau among the lanes with non-zero weight; u so close to 1 that rounding ate the
// last interval: the last lane of non-zero weight (lane 0 if there is none).
__device__ __forceinline__ int wave_choice(float w, float incl, float tau) {
    const unsigned long long some = __ballot(w > 0.f), hit = __ballot(w > 0.f && incl > tau);
    if (hit != 0ull) return __ffsll((long long)hit) - 1;
    return some != 0ull ? 63 - __clzll((long long)some) : 0;
}

// All choices of a sample, the root's first: a workgroup takes one sample through the sum layers top-down, a barrier
// between two layers.  In a layer of at most 64 regions every wave looks at all of them, one per lane, and those that the
// sample reaches are dealt to the waves in turn; in a larger one a wave looks at every (waves)-th region (those
// that a sample reaches are then many and consecutive) and works on what it finds, one after the other.
//
// Region with several partitions: the partition first (as above).  Partition: the pair (i, j) has weight
// W[k][i][j] * eL[i] * eR[j] given the evidence (the posterior of Eq. 6 for the chosen output entry k), W[k][i][j]
// without; pairs are numbered i * K + j.  The first index whose running sum exceeds the threshold is found in two steps
// without forming the products one by one: lane i holds row i of W in registers and its sum, a scan over the rows finds i
// and what is left of the threshold, a scan over row i finds j.
//
// Bound by the chain of requests per layer (choice -> record -> rows and weights -> row i), which is why the weights
// are requested before the evidence is there, and why the layers share a launch: a sample meets 15 partitions of
// a 32x32x3 image in six layers.  With 128 samples, K = 40: 38 us for all choices (44 with every (waves)-th region for
// each wave in small layers too); a launch per layer, with a wave for every (region, sample) of the layer and the K*K
// products of a pair in LDS, took 81.
template <bool IN_LDS>
__global__ __launch_bounds__(1024) void k_sample_regions(
    const int32_t* __restrict__ layer_ptr, int num_layers, const int32_t* __restrict__ sr_node,
    const int32_t* __restrict__ sr_rec, const int32_t* __restrict__ sr_pptr, const int32_t* __restrict__ sr_item,
    const int32_t* __restrict__ sr_mix, const int32_t* __restrict__ m_cptr, const int32_t* __restrict__ m_child,
    const int32_t* __restrict__ m_voff, const int32_t* __restrict__ e_left, const int32_t* __restrict__ e_right,
    const int32_t* __restrict__ e_woff, const int32_t* __restrict__ e_part, int evidence,
    const float* __restrict__ params, const float* __restrict__ A, const double* __restrict__ Off,
    const float* __restrict__ amax, const float* __restrict__ u, int num_partitions, int8_t* sel_all, int num_nodes,
    int B, int K) {
    extern __shared__ int32_t sel_lds[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
    const int b = blockIdx.x, stride = sample_sel_stride(num_nodes);
    int32_t* row_out = reinterpret_cast<int32_t*>(sel_all + (size_t)b * stride);
    int32_t* words = IN_LDS ? sel_lds : row_out;
    volatile int8_t* sel = reinterpret_cast<int8_t*>(words);
    for (int i = threadIdx.x; i < stride >> 2; i += blockDim.x) words[i] = i == 0 ? (int32_t)0xffffff00 : -1;   // (the root's
    __syncthreads();                                                                       // single entry; nothing else)
    const int KK = K * K;
    for (int l = num_layers - 1; l >= 0; --l) {
        const int first = layer_ptr[l], count = layer_ptr[l + 1] - first;
        const bool dealt = count <= 64;
        const int step = dealt ? 1 : nwaves;
        int turn = 0;
        for (int r0 = dealt ? 0 : wave; r0 < count; r0 += 64 * nwaves) {
            const int mine = r0 + lane * step;
            const int k_mine = mine < count ? sel[sr_node[first + mine]] : -1;
            unsigned long long reached = __ballot(k_mine >= 0);
            while (reached != 0ull) {
                const int ln = __ffsll((long long)reached) - 1;
                reached &= reached - 1;
                if (dealt && (turn++ & (nwaves - 1)) != wave) continue;
                const int k = __builtin_amdgcn_readlane(k_mine, ln);
                const int ri = first + r0 + ln * step;
                // the region's record: node, partitions, mixing weights, and per partition its einsum item and nodes
                const int32_t* rec = sr_rec + (size_t)ri * SR_REC_INTS;
                const int s = rec[0], nparts = rec[1];
                int item, left, right, woff, upart;
                if (nparts <= SR_REC_PARTS) {
                    int c = 0;
                    if (nparts > 1) {
                        // partition c has weight v[k][c] * S^c[k] / S[k] given the evidence (App. B), v[k][c] without;
                        // every lane walks the few partitions and gets the same answer
                        const float* v = params + rec[2] + (size_t)k * nparts;
                        const size_t srow = (size_t)s * B + b;
                        float w[SR_REC_PARTS];
#pragma unroll
                        for (int q = 0; q < SR_REC_PARTS; ++q) {
                            w[q] = 0.f;
                            if (q < nparts) {
                                w[q] = v[q];
                                if (evidence) {
                                    const size_t crow = (size_t)rec[4 + q * SR_REC_STRIDE + 5] * B + b;
                                    w[q] *= expf((float)(Off[crow] - Off[srow]) + A[crow * K + k] - A[srow * K + k]);
                                }
                            }
                        }
                        float total = 0.f;
#pragma unroll
                        for (int q = 0; q < SR_REC_PARTS; ++q)
                            if (q < nparts) total += w[q];
                        const float tau = u[(size_t)(num_partitions + s) * B + b] * total;
                        float run = 0.f;
                        int pick = -1, last = 0;
#pragma unroll
                        for (int q = 0; q < SR_REC_PARTS; ++q)
                            if (q < nparts) {
                                run += w[q];
                                if (w[q] > 0.f) last = q;
                                if (pick < 0 && run > tau) pick = q;
                            }
                        c = pick < 0 ? last : pick;          // u so close to 1 that rounding ate the last interval
                    }
                    c = __builtin_amdgcn_readfirstlane(c);
                    const int32_t* q = rec + 4 + c * SR_REC_STRIDE;
                    item = q[0], left = q[1], right = q[2], woff = q[3], upart = q[4];
                } else {
                    const int c = sample_partition(sr_mix[ri], s, k, b, m_cptr, m_child, m_voff, evidence, params, A, Off, u,
                                                   num_partitions, B, K);
                    item = __builtin_amdgcn_readfirstlane(sr_item[sr_pptr[ri] + c]);
                    left = e_left[item], right = e_right[item], woff = e_woff[item], upart = e_part[item];
                }
                const int lc = min(lane, K - 1);
                const float* wk = params + woff + (size_t)k * KK;
                const float* row = wk + (size_t)lc * K;
                floatx4 w[16];                               // row `lane` of W (any multiple of four bytes)
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    if (4 * q + 4 <= K) {
                        w[q] = *reinterpret_cast<const floatx4u*>(row + 4 * q);
                    } else {
#pragma unroll
                        for (int c = 0; c < 4; ++c) w[q][c] = 4 * q + c < K ? row[4 * q + c] : 0.f;
                    }
                }
                float el = lane < K ? 1.f : 0.f, er = el;
                if (evidence) {
                    const float al = amax[(size_t)item * 2 * B + b], ar = amax[((size_t)item * 2 + 1) * B + b];
                    const float vl = A[((size_t)left * B + b) * K + lc], vr = A[((size_t)right * B + b) * K + lc];
                    el *= __expf(vl - al);
                    er *= __expf(vr - ar);
                }
                const float uu = u[(size_t)upart * B + b];
                float sum = 0.f;
#pragma unroll
                for (int q = 0; q < 16; ++q)
                    if (4 * q < K) {
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            sum = fmaf(w[q][c], __int_as_float(__builtin_amdgcn_readlane(__float_as_int(er), 4 * q + c)), sum);
                    }
                const float wi = sum * el, incl = wave_scan(wi, lane);
                const float tau = uu * __shfl(incl, 63, 64);
                const int i = __builtin_amdgcn_readfirstlane(wave_choice(wi, incl, tau));
                const float wj = wk[(size_t)i * K + lc] * er;
                const float rest = (tau - __shfl(incl - wi, i, 64)) / __shfl(el, i, 64);
                const int j = wave_choice(wj, wave_scan(wj, lane), rest);
                if (lane == 0) {
                    sel[left] = (int8_t)i;
                    sel[right] = (int8_t)j;
                }
            }
        }
        __syncthreads();                             // the choices of this layer are there for the next one
    }
    if (IN_LDS)
        for (int i = threadIdx.x; i < stride >> 2; i += blockDim.x) row_out[i] = sel_lds[i];
}

// Leaves: one thread per (leaf variable, sample).  An observed variable keeps its value; the others take the
// mean of the chosen entry (noise == NULL), mean + sd * noise (Gaussian, noise standard normal) or
// noise < p (Bernoulli, noise uniform).
__global__ void k_sample_leaves(const int32_t* __restrict__ lv_leaf, const int32_t* __restrict__ lv_var,
                                const int32_t* __restrict__ leaf_node, const int32_t* __restrict__ leaf_replica,
                                int n_lv, const float* __restrict__ x, const uint8_t* __restrict__ mask, int mask_mode,
                                const float* __restrict__ phi, const float* __restrict__ noise,
                                const int32_t* __restrict__ logc, const int8_t* __restrict__ sel,
                                float* __restrict__ out, Dims d) {
    const int lv = blockIdx.x * blockDim.x + threadIdx.x, b = blockIdx.y;
    if (lv >= n_lv) return;
    const int leaf = lv_leaf[lv], var = lv_var[lv];
    const int k = sel[(size_t)b * sample_sel_stride(d.nodes) + leaf_node[leaf]];
    if (k < 0) return;
    bool obs = false;
    if (mask_mode == EINET_MASK_SHARED) obs = mask[var] != 0;
    if (mask_mode == EINET_MASK_PER_SAMPLE) obs = mask[(size_t)b * d.D + var] != 0;
    const int r = leaf_replica[leaf];
    for (int c = 0; c < d.C; ++c) {
        const size_t o = ((size_t)b * d.D + var) * d.C + c;
        if (obs) {
            out[o] = x[o];
            continue;
        }
        const float* ph = phi + (((size_t)var * d.C + c) * d.R + r) * d.T * d.K + k;
        const float mean = ph[0];
        float val = mean;
        if (d.family == EINET_LEAF_CATEGORICAL) {
            float total = 0.f, ev = 0.f;
            for (int v = 0; v < d.P; ++v) {
                total += ph[(size_t)v * d.K];
                ev = fmaf((float)v, ph[(size_t)v * d.K], ev);
            }
            val = ev;                                                    // E[x]
            if (noise) {
                const float tau = noise[o] * total;
                float run = 0.f;
                int pick = -1, last = 0;
                for (int v = 0; v < d.P; ++v) {
                    const float w = ph[(size_t)v * d.K];
                    run += w;
                    if (w > 0.f) last = v;
                    if (pick < 0 && run > tau) pick = v;
                }
                val = (float)(pick < 0 ? last : pick);
            }
        } else if (d.family == EINET_LEAF_BINOMIAL) {
            if (noise) {
                const float p = mean / (float)d.P;
                const float lp = logf(p), l1p = log1pf(-p);
                float total = 0.f;
                for (int v = 0; v <= d.P; ++v)
                    total += expf(__int_as_float(logc[v]) + (float)v * lp + (float)(d.P - v) * l1p);
                const float tau = noise[o] * total;
                float run = 0.f;
                int pick = -1, last = 0;
                for (int v = 0; v <= d.P; ++v) {
                    const float w = expf(__int_as_float(logc[v]) + (float)v * lp + (float)(d.P - v) * l1p);
                    run += w;
                    if (w > 0.f) last = v;
                    if (pick < 0 && run > tau) pick = v;
                }
                val = (float)(pick < 0 ? last : pick);
            }
        } else if (noise) {
            if (d.family == EINET_LEAF_GAUSSIAN) val = mean + sqrtf(fmaxf(ph[d.K] - mean * mean, 0.f)) * noise[o];
            else val = noise[o] < mean ? 1.f : 0.f;
        }
        out[o] = val;
    }
}

}  // namespace

void launch_sample_regions(const DevTables& t, int num_layers, int num_partitions, bool evidence, const float* params,
                           const float* A, const double* Off, const float* amax, const float* u, int num_nodes,
                           int32_t* sel, const Dims& d, hipStream_t s) {
    // Up to 256 samples (one workgroup per compute unit): sixteen waves, so that the regions of a layer run side by side;
    // beyond that four waves, so that samples do.
    const int threads = d.B <= EINET_NUM_CUS ? 1024 : 256;
    const int stride = sample_sel_stride(num_nodes);
#define EINET_LAUNCH(L, BYTES)                                                                                        \
    hipLaunchKernelGGL((k_sample_regions<L>), dim3(d.B), dim3(threads), BYTES, s, t.sr_layer_ptr, num_layers, t.sr_node, \
                       t.sr_rec, t.sr_pptr, t.sr_item, t.sr_mix, t.mix_cptr, t.mix_child, t.mix_voff, t.ein_left,     \
                       t.ein_right, t.ein_woff, t.ein_part, evidence ? 1 : 0, params, A, Off, amax, u, num_partitions, \
                       reinterpret_cast<int8_t*>(sel), num_nodes, d.B, d.K)
    if (stride <= SAMPLE_LDS_NODES) {
        EINET_LAUNCH(true, (size_t)stride);
    } else {
        EINET_LAUNCH(false, 0);
    }
#undef EINET_LAUNCH
}

void launch_sample_leaves(const DevTables& t, int n_lv, const float* x, const uint8_t* mask, int mask_mode,
                          const float* phi, const float* noise, const int32_t* sel, float* out, const Dims& d,
                          hipStream_t s) {
    hipLaunchKernelGGL(k_sample_leaves, dim3((n_lv + 255) / 256, d.B), dim3(256), 0, s, t.lv_leaf, t.lv_var,
                       t.leaf_node, t.leaf_replica, n_lv, x, mask, mask_mode, phi, noise, t.leaf_logc,
                       reinterpret_cast<const int8_t*>(sel), out, d);
}

}  // namespace einet_impl
