// Top-down sampling (Sec. 2, Sec. 4.2, App. D).
#include "device_common.hpp"

#include <mutex>

namespace einet_impl {

namespace {

// ------------------------------------------------------------------ top-down sampling (Sec. 2, Sec. 4.2, App. D)
// sel[b][node]: entry of the node that sample b uses, -1 if the sample does not reach the node (one byte: K is at most
// 64).  In a decomposable circuit a sample reaches a region at most once (two paths to it would sit under two
// children of one product, whose scopes are disjoint), so the writes below never collide.
__host__ __device__ inline int sample_sel_stride(int num_nodes) { return (num_nodes + 3) & ~3; }
// One launch for all layers keeps the choices of a sample in LDS: models of at most this many nodes.
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

// The partition that a sample takes at a region from entry k: its einsum item, its children's nodes, the offset of its
// weights and its number.  ri: the region's place in the sampling tables.
struct SamplePartition {
    int item, left, right, woff, number;
};
__device__ __forceinline__ SamplePartition sample_region(
    int ri, int k, int b, const int32_t* __restrict__ sr_rec, const int32_t* __restrict__ sr_pptr,
    const int32_t* __restrict__ sr_item, const int32_t* __restrict__ sr_mix, const int32_t* __restrict__ m_cptr,
    const int32_t* __restrict__ m_child, const int32_t* __restrict__ m_voff, const int32_t* __restrict__ e_left,
    const int32_t* __restrict__ e_right, const int32_t* __restrict__ e_woff, const int32_t* __restrict__ e_part, int evidence,
    const float* __restrict__ params, const float* __restrict__ A, const double* __restrict__ Off,
    const float* __restrict__ u, int num_partitions, int B, int K) {
    // the region's record: node, partitions, mixing weights, and per partition its einsum item and nodes
    const int32_t* rec = sr_rec + (size_t)ri * SR_REC_INTS;
    const int s = rec[0], nparts = rec[1];
    if (nparts > SR_REC_PARTS) {
        const int c = sample_partition(sr_mix[ri], s, k, b, m_cptr, m_child, m_voff, evidence, params, A, Off, u,
                                       num_partitions, B, K);
        const int item = __builtin_amdgcn_readfirstlane(sr_item[sr_pptr[ri] + c]);
        return SamplePartition{item, e_left[item], e_right[item], e_woff[item], e_part[item]};
    }
    int c = 0;
    if (nparts > 1) {
        // partition c has weight v[k][c] * S^c[k] / S[k] given the evidence (App. B), v[k][c] without; every
        // lane walks the few partitions and gets the same answer
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
        c = pick < 0 ? last : pick;                  // u so close to 1 that rounding ate the last interval
    }
    c = __builtin_amdgcn_readfirstlane(c);
    const int32_t* q = rec + 4 + c * SR_REC_STRIDE;
    return SamplePartition{q[0], q[1], q[2], q[3], q[4]};
}

// Partition: the pair (i, j) has weight W[k][i][j] * eL[i] * eR[j] given the evidence (the posterior of
// Eq. 6 for the chosen output entry k), W[k][i][j] without; pairs are numbered i * K + j.  The K*K weights go to LDS (the
// wave's own part), every lane sums a run of consecutive pairs, a wave scan of the run sums finds the run that holds the
// threshold and its lane walks it.
__device__ __forceinline__ int sample_pos(int t) { return t + (t >> 5); }   // padded: runs start in different banks
__host__ __device__ inline int sample_pair_floats(int K) { return K * K + ((K * K) >> 5) + 1 + 128; }   // LDS of a wave

__device__ __forceinline__ int sample_pair(const SamplePartition& p, int k, int b, int lane, float* wl, int evidence,
                                           const float* __restrict__ params, const float* __restrict__ A,
                                           const float* __restrict__ amax, const float* __restrict__ u, int B, int K) {
    const int KK = K * K;
    float* el = wl + sample_pos(KK) + 1;
    float* er = el + 64;
    __builtin_amdgcn_wave_barrier();                 // (the reads of a region before are done)
    if (evidence) {
        const float al = amax[(size_t)p.item * 2 * B + b], ar = amax[((size_t)p.item * 2 + 1) * B + b];
        el[lane] = lane < K ? __expf(A[((size_t)p.left * B + b) * K + lane] - al) : 0.f;
        er[lane] = lane < K ? __expf(A[((size_t)p.right * B + b) * K + lane] - ar) : 0.f;
        __builtin_amdgcn_wave_barrier();
    }
    const float* row = params + p.woff + (size_t)k * KK;
    for (int t0 = lane; t0 < KK; t0 += 8 * 64) {      // eight loads in flight per lane
        float w[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) w[q] = t0 + 64 * q < KK ? row[t0 + 64 * q] : 0.f;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int t = t0 + 64 * q;
            if (t < KK) {
                if (evidence) {
                    const int i = t / K, j = t - i * K;
                    w[q] *= el[i] * er[j];
                }
                wl[sample_pos(t)] = w[q];
            }
        }
    }
    __builtin_amdgcn_wave_barrier();                 // a wave reads back only its own part of LDS
    const int chunk = (KK + 63) >> 6;
    const int t0 = min(lane * chunk, KK), t1 = min(t0 + chunk, KK);
    float part = 0.f;
    for (int t = t0; t < t1; ++t) part += wl[sample_pos(t)];
    float incl = part;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const float up = __shfl_up(incl, o, 64);
        if (lane >= o) incl += up;
    }
    const float total = __shfl(incl, 63, 64);
    const float tau = u[(size_t)p.number * B + b] * total;
    const unsigned long long hit = __ballot(incl > tau && t1 > t0);
    int pick = -1;
    if (hit != 0ull) {
        const int owner = __ffsll((long long)hit) - 1;
        if (lane == owner) {
            float run = incl - part;
            int last = t0;
            for (int t = t0; t < t1; ++t) {
                const float w = wl[sample_pos(t)];
                run += w;
                if (w > 0.f) last = t;
                if (pick < 0 && run > tau) pick = t;
            }
            if (pick < 0) pick = last;               // the run's own sum exceeded tau, its walk did not: rounding
        }
        pick = __shfl(pick, owner, 64);
    } else {
        // u so close to 1 that rounding ate the last interval: the last pair of non-zero weight
        int last = -1;
        for (int t = t0; t < t1; ++t)
            if (wl[sample_pos(t)] > 0.f) last = t;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) last = max(last, __shfl_xor(last, o, 64));
        pick = max(last, 0);
    }
    return pick;
}

// The choices of one sum layer: a wave per (region, sample).  The launch of the root's layer (clear) first marks all other
// nodes of its samples as not reached.  MANY: for layers with many more regions than a sample can reach, a wave takes
// every `slots`-th region, looks at 64 of them at once, one per lane, and works on those that its sample reaches.
// Bound by the chain of requests of a region (entry and record -> partition -> weights), then by the walk over the products
// in LDS: 2.4 us per layer for K = 4, 7 for K = 40, 15 for K = 64, few samples; see the rule at the launch.
constexpr int SAMPLE_WAVES = 4;
template <bool MANY>
__global__ __launch_bounds__(64 * SAMPLE_WAVES) void k_sample_layer(
    const int32_t* __restrict__ sr_node, int count, int slots, const int32_t* __restrict__ sr_rec,
    const int32_t* __restrict__ sr_pptr, const int32_t* __restrict__ sr_item, const int32_t* __restrict__ sr_mix,
    const int32_t* __restrict__ m_cptr, const int32_t* __restrict__ m_child, const int32_t* __restrict__ m_voff,
    const int32_t* __restrict__ e_left, const int32_t* __restrict__ e_right, const int32_t* __restrict__ e_woff,
    const int32_t* __restrict__ e_part, int evidence, const float* __restrict__ params, const float* __restrict__ A,
    const double* __restrict__ Off, const float* __restrict__ amax, const float* __restrict__ u, int num_partitions,
    int8_t* sel_all, int num_nodes, int clear, int B, int K) {
    extern __shared__ float lds[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int b = blockIdx.y * SAMPLE_WAVES + wave;
    if (b >= B) return;                              // whole waves leave: no barrier below
    const int stride = sample_sel_stride(num_nodes);
    int8_t* sel = sel_all + (size_t)b * stride;
    float* wl = lds + wave * sample_pair_floats(K);
    auto choose = [&](int ri, int k) {
        const SamplePartition p = sample_region(ri, k, b, sr_rec, sr_pptr, sr_item, sr_mix, m_cptr, m_child, m_voff, e_left,
                                                e_right, e_woff, e_part, evidence, params, A, Off, u, num_partitions, B, K);
        const int pick = sample_pair(p, k, b, lane, wl, evidence, params, A, amax, u, B, K);
        if (!MANY && clear) __threadfence_block();   // the row's -1 are written before the choices
        if (lane == 0) {
            if (!MANY && clear) sel[0] = 0;
            const int i = pick / K;
            sel[p.left] = (int8_t)i;
            sel[p.right] = (int8_t)(pick - i * K);
        }
    };
    if constexpr (MANY) {
        for (int r0 = blockIdx.x; r0 < count; r0 += 64 * slots) {
            const int mine = r0 + lane * slots;
            const int k_mine = mine < count ? sel[sr_node[mine]] : -1;
            unsigned long long reached = __ballot(k_mine >= 0);
            while (reached != 0ull) {
                const int ln = __ffsll((long long)reached) - 1;
                reached &= reached - 1;
                choose(r0 + ln * slots, __builtin_amdgcn_readlane(k_mine, ln));
            }
        }
    } else {
        if (clear) {                                 // (the root's layer is the root alone, node 0, with its single entry)
            typedef int32_t int32x4u __attribute__((ext_vector_type(4), aligned(4)));
            int32_t* words = reinterpret_cast<int32_t*>(sel);
            const int n = stride >> 2, n4 = n & ~3;
            for (int i = 4 * lane; i < n4; i += 256) *reinterpret_cast<int32x4u*>(words + i) = int32x4u{-1, -1, -1, -1};
            if (lane < n - n4) words[n4 + lane] = -1;
        }
        const int k = clear ? 0 : sel[sr_rec[(size_t)blockIdx.x * SR_REC_INTS]];
        if (k >= 0) choose(blockIdx.x, k);
    }
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

// Waves of a workgroup of the kernel below.  Up to 256 samples (one workgroup per compute unit): sixteen, so that the
// regions of a layer run side by side; beyond that four, so that samples do.
constexpr int sample_waves(int B) { return B <= EINET_NUM_CUS ? 16 : 4; }

// All choices of a sample in one launch, the root's first: a workgroup takes one sample through the sum layers top-down, a
// barrier between two layers.  In a layer of at most 64 regions every wave looks at all of them, one per lane, and those
// that the sample reaches are dealt to the waves in turn; in a larger one a wave looks at every (waves)-th region (those
// that a sample reaches are then many and consecutive) and works on what it finds, one after the other.
//
// The choices are those of k_sample_layer.  The first pair whose running sum exceeds the threshold is found in two steps
// without forming the products one by one: lane i holds row i of W in registers and its sum, a scan over the rows finds i
// and what is left of the threshold, a scan over row i finds j.
//
// Bound by the chain of requests per region (choice -> record -> rows and weights -> row i), which is why the weights
// are requested before the evidence is there.  32x32x3 images, 128 samples, K = 40: 29 us without evidence for the choices
// and the leaves, 59 with a launch per layer; with evidence the choices took 38 us, 44 before the regions of small layers
// were dealt to the waves.
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
    volatile int8_t* sel = reinterpret_cast<int8_t*>(sel_lds);
    for (int i = threadIdx.x; i < stride >> 2; i += blockDim.x) sel_lds[i] = i == 0 ? (int32_t)0xffffff00 : -1;   // (the
    __syncthreads();                                                                  // root's single entry; nothing else)
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
                const SamplePartition p = sample_region(ri, k, b, sr_rec, sr_pptr, sr_item, sr_mix, m_cptr, m_child, m_voff,
                                                        e_left, e_right, e_woff, e_part, evidence, params, A, Off, u,
                                                        num_partitions, B, K);
                const int lc = min(lane, K - 1);
                const float* wk = params + p.woff + (size_t)k * KK;
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
                    const float al = amax[(size_t)p.item * 2 * B + b], ar = amax[((size_t)p.item * 2 + 1) * B + b];
                    const float vl = A[((size_t)p.left * B + b) * K + lc], vr = A[((size_t)p.right * B + b) * K + lc];
                    el *= __expf(vl - al);
                    er *= __expf(vr - ar);
                }
                const float uu = u[(size_t)p.number * B + b];
                float sum = 0.f;
#pragma unroll
                for (int q = 0; q < 16; ++q)
                    if (4 * q < K) {
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            sum = fmaf(w[q][c], __int_as_float(__builtin_amdgcn_readlane(__float_as_int(er), 4 * q + c)), sum);
                    }
                const float wi = sum * el, incl = wave_scan(wi, lane);
                const float total = __shfl(incl, 63, 64), tau = uu * total;
                const int i = __builtin_amdgcn_readfirstlane(wave_choice(wi, incl, tau));
                const float wj = wk[(size_t)i * K + lc] * er;
                const float rest = (tau - __shfl(incl - wi, i, 64)) / __shfl(el, i, 64);
                // (no pair of non-zero weight: the first one)
                const int j = total > 0.f ? wave_choice(wj, wave_scan(wj, lane), rest) : 0;
                if (lane == 0) {
                    sel[p.left] = (int8_t)i;
                    sel[p.right] = (int8_t)j;
                }
            }
        }
        __syncthreads();                             // the choices of this layer are there for the next one
    }
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

// Layers with at least eight times as many regions as a sample can reach (the replicas of random trees) and more waves
// than fill the chip: one wave per region that can be reached instead of one per region (1024 variables, depth 9, R = 40,
// K = 4, 1000 samples: 418 us instead of 1340).  Below that the wave that looks at a single region is the faster one, because
// it has its region's record before it knows the entry (R = 1, 1 sample: 30 us instead of 33).
static bool sample_layer_is_sparse(int count, int reach, int B) {
    return count >= 8 * reach && (int64_t)count * B > 16384;
}

// One launch for all layers, or one per layer?  In one launch the regions of a layer that do not find a wave of their own
// wait for each other: a step of a wave takes 3.4 us, more where the rows of W come from memory (K^3).  A launch per layer
// costs 3.4 us (the call from the host; the kernel 2.4) and the walk over the K^2 products, then the waves' time
// where they are more than the chip holds.  The constants are fitted to 1812 cases, launched from the host: 1 to 1000
// samples, K 4 to 64, trees of depth 2 to 9 with 1 to 40 replicas, images; on average the form that is chosen takes 0.7 %
// longer than the faster one (replayed from a graph 2.5 %: there a launch costs less).  One launch against a launch per layer: 32x32x3 images,
// 128 samples, K = 40: 29 and 59 us, K = 4: 30 and 27; 1024 variables, depth 9, 16 samples, K = 4: 133 and 33 us, K = 40: 165
// and 93.
static bool sample_in_one_launch(int num_layers, const int32_t* layer_ptr, const int32_t* reach, int num_nodes,
                                 const Dims& d) {
    if (sample_sel_stride(num_nodes) > SAMPLE_LDS_NODES) return false;
    const double K = d.K, K3 = K * K * K;
    const int waves = sample_waves(d.B);
    int64_t steps = 0, choices = 0, looked_at = 0;
    for (int l = 0; l < num_layers; ++l) {
        const int count = layer_ptr[l + 1] - layer_ptr[l];
        steps += (reach[l] + waves - 1) / waves;
        choices += reach[l];
        looked_at += sample_layer_is_sparse(count, reach[l], d.B) ? reach[l] : count;
    }
    const double one = (3.4 + 2e-5 * K3) * (double)steps;
    const double each = num_layers * (3.4 + 3e-3 * K * K) +
                        d.B * ((5.5e-5 + 1.2e-10 * K3 * K) * (double)looked_at + (3e-4 + 2e-8 * K3) * (double)choices);
    return one < each;
}

void launch_sample_regions(const DevTables& t, const int32_t* layer_ptr, const int32_t* reach, int num_layers,
                           int num_partitions, bool evidence, const float* params, const float* A, const double* Off,
                           const float* amax, const float* u, int num_nodes, int32_t* sel, const Dims& d, hipStream_t s) {
    int8_t* sel8 = reinterpret_cast<int8_t*>(sel);
    const int ev = evidence ? 1 : 0;
    if (sample_in_one_launch(num_layers, layer_ptr, reach, num_nodes, d)) {
        hipLaunchKernelGGL(k_sample_regions, dim3(d.B), dim3(64 * sample_waves(d.B)), (size_t)sample_sel_stride(num_nodes), s,
                           t.sr_layer_ptr, num_layers, t.sr_node, t.sr_rec, t.sr_pptr, t.sr_item, t.sr_mix, t.mix_cptr,
                           t.mix_child, t.mix_voff, t.ein_left, t.ein_right, t.ein_woff, t.ein_part, ev, params, A, Off, amax,
                           u, num_partitions, sel8, num_nodes, d.B, d.K);
        return;
    }
    const size_t lds = sizeof(float) * SAMPLE_WAVES * sample_pair_floats(d.K);   // at most 68 KB (K = 64)
    if (lds > 64 * 1024) {
        static std::once_flag attr_set[EINET_MAX_DEVICES];
        int dev = 0;
        (void)hipGetDevice(&dev);
        std::call_once(attr_set[dev % EINET_MAX_DEVICES], [&] {
            allow_dynamic_lds(&k_sample_layer<false>, 72 * 1024);
            allow_dynamic_lds(&k_sample_layer<true>, 72 * 1024);
        });
    }
    for (int l = num_layers - 1; l >= 0; --l) {
        const int first = layer_ptr[l], count = layer_ptr[l + 1] - first;
        const bool clear = l == num_layers - 1;
        const bool many = !clear && sample_layer_is_sparse(count, reach[l], d.B);
        const int slots = many ? reach[l] : count;
#define EINET_LAUNCH(M)                                                                                                   \
    hipLaunchKernelGGL((k_sample_layer<M>), dim3(slots, (d.B + SAMPLE_WAVES - 1) / SAMPLE_WAVES), dim3(64 * SAMPLE_WAVES),\
                       lds, s, t.sr_node + first, count, slots, t.sr_rec + (size_t)first * SR_REC_INTS,                   \
                       t.sr_pptr + first, t.sr_item, t.sr_mix + first, t.mix_cptr, t.mix_child, t.mix_voff, t.ein_left,   \
                       t.ein_right, t.ein_woff, t.ein_part, ev, params, A, Off, amax, u, num_partitions, sel8, num_nodes, \
                       clear ? 1 : 0, d.B, d.K)
        if (many) EINET_LAUNCH(true);
        else EINET_LAUNCH(false);
#undef EINET_LAUNCH
    }
}

void launch_sample_leaves(const DevTables& t, int n_lv, const float* x, const uint8_t* mask, int mask_mode,
                          const float* phi, const float* noise, const int32_t* sel, float* out, const Dims& d,
                          hipStream_t s) {
    hipLaunchKernelGGL(k_sample_leaves, dim3((n_lv + 255) / 256, d.B), dim3(256), 0, s, t.lv_leaf, t.lv_var,
                       t.leaf_node, t.leaf_replica, n_lv, x, mask, mask_mode, phi, noise, t.leaf_logc,
                       reinterpret_cast<const int8_t*>(sel), out, d);
}

}  // namespace einet_impl
