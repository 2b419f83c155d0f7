// End of the top-down pass: statistics of the einsum weights (Eq. 6), for the items of all layers below the root's in one
// launch.  They need the posteriors of the regions, which the top-down launches have left, and are needed by the M-step
// only: nothing waits for them, so no layer's launch carries them.
#include "bf16x6.hpp"

#include <mutex>

namespace einet_impl {

namespace {

//   Nw[k,i,j] (+)= W[k,i,j] * sum_b Q[b,k] eL[b,i] eR[b,j],      Q = G[s] * v * exp((Off[out] - Off[s]) - A[s])
// (Q as in the top-down kernel): a product with the batch as contraction, rows (k, i) in tiles of 4 x 4, columns j in tiles
// of 16.  Rows are staged in LDS; the operand of a row tile, Q * eL, is formed on the fly.  The sums stay in registers over
// the whole batch.

// Rows of one item, as the workgroup needs them.
struct StatRows {
    const float *L, *R, *As, *Gs, *aL, *aR;
    const double *Oo, *Os;
    const float* v;                                    // mixing weights of the item's region, null: one partition
    int vstr, gcnt;                                    // blocks (B * K floats apart) that add up to the region's posterior
};

__device__ __forceinline__ StatRows stat_rows(const int32_t* rec, int item, const float* params, const float* A,
                                              const double* Off, const float* amax, const float* G, const float* Gp, int B, int K) {
    const size_t blk = (size_t)B * K;
    StatRows r;
    r.L = A + (size_t)rec[0] * blk;
    r.R = A + (size_t)rec[1] * blk;
    r.As = A + (size_t)rec[3] * blk;
    r.Oo = Off + (size_t)rec[2] * B;
    r.Os = Off + (size_t)rec[3] * B;
    r.v = rec[5] >= 0 ? params + rec[5] : nullptr;
    r.vstr = rec[6];
    r.Gs = rec[7] >= 0 ? Gp + (size_t)rec[7] * blk : G + (size_t)rec[3] * blk;
    r.gcnt = rec[7] >= 0 ? bwd_source_blocks(rec[8], K, B) : 1;
    r.aL = amax + (size_t)item * 2 * B;
    r.aR = r.aL + B;
    return r;
}

// ------------------------------------------------------------------ K up to 16
// One column tile: the split of a bfloat16 operand would take longer than what the faster instruction saves, so this is
// v_mfma_f32_16x16x4_f32.  The batch is dealt to the four waves of a workgroup, 32 samples at a time, and a wave takes all
// row tiles of its samples: rows come in as 16-byte pieces (lane = (sample, piece)), pass through a wave-private LDS
// tile, [sample][16] as they are in memory, and only the sums of the four waves meet at the end.  Entries beyond K are
// rows and columns of the product that nobody reads; samples beyond the batch have Q = 0.  The row tiles of an item
// (blocks of four left entries) are spread over nsplit workgroups where there are few items, and the batch over nshare where
// that is not enough (statistics in blocks of their own, [nshare][count][K^3], which a later launch adds up).
// Bound by the instructions besides the matrix ones (rows to operands).  K = 10, 2540 items, 100 samples: 29.8 us; K = 16, 388
// items, 256 samples: 18.4 us.  (Sum of the top-down launches with it 87.9 us, with the statistics in every launch 126.6.)
template <int KQ, bool QUADS, bool ACCUM>
__global__ __launch_bounds__(256, 3) void k_einsum_stats_small(const int32_t* __restrict__ e_rec, const float* __restrict__ params,
                                                             float* __restrict__ stats, const float* __restrict__ A,
                                                             const double* __restrict__ Off, const float* __restrict__ amax,
                                                             const float* __restrict__ G, const float* __restrict__ Gp,
                                                             int item0, int count, int nsplit, int nshare, int share,
                                                             float* __restrict__ part_blocks, int B, int K_) {
    constexpr int KP = 4 * KQ, WT = 32 * 16;           // floats of a wave's tile
    __shared__ __attribute__((aligned(16))) float lds[4 * 3 * WT];
    const int K = QUADS ? KP : K_;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c16 = lane & 15, g = lane >> 4;
    const int vb = xcd_contiguous_block();
    const int part = vb % nsplit, sh = (vb / nsplit) % nshare, li = vb / (nsplit * nshare);
    const int bs = sh * share, be = min(bs + share, B);       // this workgroup's samples
    const int i0 = part * KQ / nsplit, i1 = (part + 1) * KQ / nsplit;
    const int32_t* rec = e_rec + (size_t)li * EIN_BREC_INTS;
    const StatRows rows = stat_rows(rec, item0 + li, params, A, Off, amax, G, Gp, B, K);
    const size_t blk = (size_t)B * K;
    float* sR = lds + wave * 3 * WT;
    float* sQ = sR + WT;
    float* sL = sQ + WT;
    const int ls = lane >> 2, lp = lane & 3, pc = min(lp, KQ - 1);       // loads: sample of 16, piece
    float v[4] = {1.f, 1.f, 1.f, 1.f};
    if (rows.v) {
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = rows.v[min(4 * pc + c, K - 1) * rows.vstr];
    }
    float r4[2][4], l4[2][4], g4[2][4], a4[2][4], al[2], ar[2], dd[2];
    auto fetch = [&](int b0) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int b = min(b0 + 16 * u + ls, B - 1);
            const size_t o = (size_t)b * K;
            load_piece<KQ, QUADS>(rows.R + o, pc, K, r4[u]);
            load_piece<KQ, QUADS>(rows.L + o, pc, K, l4[u]);
            load_piece<KQ, QUADS>(rows.Gs + o, pc, K, g4[u]);
            load_piece<KQ, QUADS>(rows.As + o, pc, K, a4[u]);
            for (int x = 1; x < rows.gcnt; ++x) {
                float more[4];
                load_piece<KQ, QUADS>(rows.Gs + x * blk + o, pc, K, more);
#pragma unroll
                for (int c = 0; c < 4; ++c) g4[u][c] += more[c];
            }
            al[u] = rows.aL[b];
            ar[u] = rows.aR[b];
            dd[u] = (float)(rows.Oo[b] - rows.Os[b]);
        }
    };
    floatx4 acc[KQ][KQ];
#pragma unroll
    for (int it = 0; it < KQ; ++it)
#pragma unroll
        for (int kt = 0; kt < KQ; ++kt) acc[it][kt] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (bs + 32 * wave < be) fetch(bs + 32 * wave);
    for (int b0 = bs + 32 * wave; b0 < be; b0 += 128) {
        __builtin_amdgcn_wave_barrier();               // (the LDS serves a wave's requests in order)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const bool in = b0 + 16 * u + ls < be;
            floatx4 q, r, l;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                q[c] = in && g4[u][c] != 0.f ? g4[u][c] * v[c] * __expf(dd[u] - a4[u][c]) : 0.f;
                r[c] = __expf(r4[u][c] - ar[u]);
                l[c] = __expf(l4[u][c] - al[u]);
            }
            const int o = (16 * u + ls) * 16 + 4 * lp;
            if (lp < KQ) {
                *reinterpret_cast<floatx4*>(sQ + o) = q;
                *reinterpret_cast<floatx4*>(sR + o) = r;
                *reinterpret_cast<floatx4*>(sL + o) = l;
            }
        }
        if (b0 + 128 < be) fetch(b0 + 128);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const int steps = min(32, be - b0);
        for (int s = 0; s < steps; s += 4) {           // lane group g: sample s + g
            const float* q0 = sQ + (s + g) * 16 + (c16 >> 2);
            const float* l0 = sL + (s + g) * 16 + (c16 & 3);
            const float rb = sR[(s + g) * 16 + c16];
            float qa[KQ];
#pragma unroll
            for (int kt = 0; kt < KQ; ++kt) qa[kt] = q0[4 * kt];
#pragma unroll
            for (int it = 0; it < KQ; ++it) {
                if (it >= i0 && it < i1) {
                    const float la = l0[4 * it];
#pragma unroll
                    for (int kt = 0; kt < KQ; ++kt)    // rows m = 4 (k % 4) + i % 4
                        acc[it][kt] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[kt] * la, rb, acc[it][kt], 0, 0, 0);
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    // The four waves' sums of the tiles of one block of left entries at a time; wave w finishes tile kt = w:
    // acc[it][kt][c]: k = 4 kt + g, i = 4 it + c, j = c16
    const float* W = params + rec[4];
    float* Nw = nshare > 1 ? part_blocks + ((size_t)sh * count + li) * (K * K * K) : stats + rec[4];
    floatx4* red = reinterpret_cast<floatx4*>(lds);    // [wave][kt][lane]
    static_assert(4 * KQ * 64 * 4 <= 4 * 3 * WT, "the sums fit where the rows were");
#pragma unroll
    for (int it = 0; it < KQ; ++it) {
        if (it >= i0 && it < i1) {
            const int k = 4 * wave + g;
            float w[4] = {0.f, 0.f, 0.f, 0.f}, old[4] = {0.f, 0.f, 0.f, 0.f};
            if (k < K && c16 < K) {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int o = (k * K + min(4 * it + c, K - 1)) * K + c16;
                    w[c] = W[o];
                    if (ACCUM) old[c] = Nw[o];
                }
            }
            __syncthreads();                           // rows, or the sums of the block before, have been read
#pragma unroll
            for (int kt = 0; kt < KQ; ++kt) red[(wave * KQ + kt) * 64 + lane] = acc[it][kt];
            __syncthreads();
            if (wave < KQ) {
                floatx4 sum = red[wave * 64 + lane];
#pragma unroll
                for (int x = 1; x < 4; ++x) sum += red[(x * KQ + wave) * 64 + lane];
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (k < K && c16 < K && 4 * it + c < K) Nw[(k * K + 4 * it + c) * K + c16] = old[c] + w[c] * sum[c];
            }
        }
    }
}

template <int KQ>
void launch_stats_small(const EinStatsWork& w, bool accumulate, float* stats, hipStream_t s) {
    // three workgroups per compute unit
    const int want = (3 * EINET_NUM_CUS + w.count - 1) / w.count, nsplit = want > KQ ? KQ : want;
    const int nshare = ein_stat_shares(w.count, w.K, w.B), share = ein_stat_share(nshare, w.B);
#define EINET_LAUNCH(Q, ACC)                                                                                          \
    hipLaunchKernelGGL((k_einsum_stats_small<KQ, Q, ACC>), dim3(w.count * nsplit * nshare), dim3(256), 0, s, w.rec, w.params, \
                       stats, w.A, w.Off, w.amax, w.G, w.Gp, w.first, w.count, nsplit, nshare, share, w.part, w.B, w.K)
    const bool adds = accumulate && nshare == 1;       // (blocks of shares are written, not added to)
    if (w.K == 4 * KQ) {
        if (adds) EINET_LAUNCH(true, true);
        else EINET_LAUNCH(true, false);
    } else {
        if (adds) EINET_LAUNCH(false, true);
        else EINET_LAUNCH(false, false);
    }
#undef EINET_LAUNCH
}

// ------------------------------------------------------------------ K from 17
// Several column tiles share a row operand: bfloat16 parts (bf16x6.hpp, six instructions of 32 samples per tile).  The
// top-down kernel leaves Q, eR and eL of every item sample-major in memory (EinImages), so that staging is a copy; eR is
// split on the way.  Q * eL is formed in float32 and split for every row tile, which is most of the kernel's vector work: a
// wave owns whole row tiles with all their columns, so that every product is formed once.
//
// A wave takes a unit, the row tiles of one slice (four left entries i; NH units per slice where its registers do not hold
// the sums of all k, or where there are few items); a workgroup of eight waves takes `per` consecutive units and stages the
// items that they touch (NSLOT at most).  One workgroup per compute unit, so nothing else hides its waits: the rows of the
// next 32 samples are requested before the products of the current ones and go to the other half of the LDS after them.
//
// Scales: eR and eL carry 2^24 each, so that the bits of their smallest normal numbers survive the split.  A row k of Q whose
// largest value in the first step that has one is outside 2^-40 .. 2^40 is multiplied by a power of two that brings it to 1, and
// by a smaller one (the sums with it) from the step on whose values would pass 2^40; so sums stay below 2^96.  The threads that
// stage a row choose its factor from the values as they are in memory, before they multiply: times the factor of the steps
// before, a value may be beyond the largest float32.
// K = 40, 194 items: 37 us for 128 samples, 202 us for 1000.  The counters show the matrix pipes busy 33 and 42 % of that time, waves
// that wait for something 28 to 31 % of theirs and for an instruction to issue another 31 to 33 %: one wave's products wait for its
// own splits.  K = 30, 140 items, 100 samples: 23 us.
// STEP: samples that are staged at once.  32, the contraction of one instruction, or ST_WHOLE: the whole of a short batch.
constexpr int ST_WHOLE = 128;
template <int KQ, int NH, int STEP>
struct StatLayout {
    static constexpr int KP = 4 * KQ, NJ = (KP + 15) / 16;        // column tiles
    static constexpr int NRT = (KQ + NH - 1) / NH;        // row tiles of a wave
    static constexpr int RB = STEP + 8, RF = STEP + 4;    // row strides: bfloat16, float
    static constexpr int OFF_Q = 3 * 16 * NJ * RB * 2;    // a slot: eR [3 parts][16 NJ][RB] bfloat16, Q [4 NRT NH][RF]
    static constexpr int SLOT = OFF_Q + 4 * NRT * NH * RF * 4;
    // items that a workgroup's units can touch (its units are few enough)
    static constexpr bool SEQ = STEP == ST_WHOLE;         // the units of a slice one after the other
    static constexpr int UI = KQ * (SEQ ? 1 : NH);        // units per item (SEQ: those of a slice counted as one)
    static constexpr int NSLOT = UI < 7 ? 3 : 2, PER = 8; // most units of a workgroup
    static constexpr int NBUF = SEQ ? 1 : 2;
    static constexpr int OFF_L = NSLOT * SLOT;            // eL [8 waves][4][RF]
    static constexpr int OFF_M = OFF_L + 8 * 4 * RF * 4;  // per slot: what the factors of Q changed by with the step [64]
    static constexpr int BUF = OFF_M + NSLOT * 64 * 4;
    static constexpr int OFF_F = NBUF * BUF;              // per slot: factors of the rows of Q [64]
    static constexpr int LDS_BYTES = OFF_F + NSLOT * 64 * 4;
    static constexpr int ROUNDS = (NSLOT * 2 * KP * 8 + 511) / 512;      // pieces of STEP / 8 samples per thread and step
    static_assert(LDS_BYTES <= 160 * 1024, "the rows fit the LDS of a compute unit");
};

// Factor of a row of Q, a power of two: top is the largest value of the step, old the factor so far, 0 where all values so far were
// zero.
__device__ __forceinline__ float stat_row_factor(float top, float old) {
    if (top == 0.f) return old;
    const int ex = (int)(__builtin_bit_cast(uint32_t, top) >> 23) - 127, exo = (int)(__builtin_bit_cast(uint32_t, old) >> 23) - 127;
    const bool keep = old == 0.f ? top >= 0x1p-40f && top <= 0x1p+40f : ex + exo < 40;
    if (keep) return old == 0.f ? 1.f : old;
    return __builtin_bit_cast(float, (uint32_t)(127 - min(max(ex, -125), 125)) << 23);
}

// Short batches (STEP = ST_WHOLE): the units of a slice are taken one after the other by the same wave, so that the weights of
// a unit's rows are requested before its products and the statistics of one unit are stored while the next is multiplied.
template <int KQ, int NH, int STEP, bool ACCUM>
__global__ __launch_bounds__(512, 2) void k_einsum_stats(const int32_t* __restrict__ e_rec, const float* __restrict__ params,
                                                       float* __restrict__ stats, const float* __restrict__ img,
                                                       int item0, int count, int per, int nshare, int share,
                                                       float* __restrict__ part, int B, int K) {
    using LY = StatLayout<KQ, NH, STEP>;
    constexpr int KP = LY::KP, NJ = LY::NJ, NRT = LY::NRT, RB = LY::RB, RF = LY::RF, UI = LY::UI;
    constexpr bool SEQ = LY::SEQ;
    constexpr int NU = SEQ ? 1 : NH, Q4 = STEP / 32, PS = STEP / 8;      // units per slice, 16-byte groups and samples of a piece
    extern __shared__ __attribute__((aligned(16))) char lds_c[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c16 = lane & 15, kg = lane >> 4;
    float* sF = reinterpret_cast<float*>(lds_c + LY::OFF_F);
    const int Bp = ein_image_stride(B);
    const size_t isz = (size_t)EIN_IMAGES * KP * Bp;   // floats of an item's images
    // Units v0 .. v0 + n - 1 of this workgroup: unit v of an item: slice v / NU, row tiles NRT (v % NU) ..  A batch in nshare
    // shares of `share` samples: every item counts as nshare virtual ones, numbered item-major; their statistics go to
    // blocks of their own in `part` ([nshare][count][K^3]), which a later launch adds up.
    const long long first = (long long)xcd_contiguous_block() * per;
    const int vi0 = (int)(first / UI), v0 = (int)(first - (long long)vi0 * UI);
    const int n = (int)min((long long)per, (long long)count * nshare * UI - first);
    const int nslot = (v0 + n - 1) / UI + 1;           // virtual items touched
    const bool work = wave < n;
    const int v = v0 + min(wave, n - 1), slot = v / UI, vi = v - slot * UI;
    const int it = vi / NU, li = (vi0 + slot) / nshare, sh = vi0 + slot - li * nshare;
    int kt0 = NRT * (vi % NU);
    auto image_of = [&](int sl) {                      // first sample of the first image of virtual item vi0 + sl
        const int q = vi0 + sl, item = q / nshare;
        return img + (size_t)(item0 + item) * isz + (size_t)(q - item * nshare) * share;
    };
    auto samples_of = [&](int sl) { return min(share, B - (vi0 + sl) % nshare * share); };

    // ---- staging: piece f = (row, STEP / 8 samples) of Q and of eR of the items; rows beyond K, samples beyond the batch: zero
    floatx4 x4[LY::ROUNDS][Q4], l4[Q4];
    float fac[LY::ROUNDS];                             // of the row, if it is one of Q; 0: all its values so far were zero
#pragma unroll
    for (int x = 0; x < LY::ROUNDS; ++x) fac[x] = 0.f;
    auto fetch = [&](int s) {
#pragma unroll
        for (int x = 0; x < LY::ROUNDS; ++x) {
            const int f = tid + 512 * x, b = s + PS * (f & 7), row = f >> 3, sl = row / (2 * KP), y = row - sl * 2 * KP;
            const float* src = image_of(sl) + (size_t)y * Bp + b;
            const int nsl = samples_of(sl);
#pragma unroll
            for (int q = 0; q < Q4; ++q) {
                x4[x][q] = floatx4{0.f, 0.f, 0.f, 0.f};
                if (sl < nslot && (y >= KP ? y - KP : y) < K && b + 4 * q < nsl) x4[x][q] = *reinterpret_cast<const floatx4*>(src + 4 * q);
            }
        }
        const int i = 4 * it + ((lane >> 3) & 3), b = s + PS * (lane & 7);     // this wave's four rows of eL: lanes 0 .. 31
        const float* src = image_of(slot) + (size_t)(2 * KP + i) * Bp + b;
        const int nsl = samples_of(slot);
#pragma unroll
        for (int q = 0; q < Q4; ++q) {
            l4[q] = floatx4{0.f, 0.f, 0.f, 0.f};
            if (work && lane < 32 && i < K && b + 4 * q < nsl) l4[q] = *reinterpret_cast<const floatx4*>(src + 4 * q);
        }
    };
    auto stage = [&](int s, char* buf) {
#pragma unroll
        for (int x = 0; x < LY::ROUNDS; ++x) {
            const int f = tid + 512 * x, b = PS * (f & 7), row = f >> 3, sl = row / (2 * KP), y = row - sl * 2 * KP;
            if (sl < nslot) {
                char* dst = buf + sl * LY::SLOT;
                const int nsl = samples_of(sl);
                floatx4 v[Q4];
#pragma unroll
                for (int q = 0; q < Q4; ++q)
#pragma unroll
                    for (int c = 0; c < 4; ++c) v[q][c] = s + b + 4 * q + c < nsl ? x4[x][q][c] : 0.f;
                if (y >= KP) {
#pragma unroll
                    for (int q = 0; q < Q4; ++q) {
                        uint32_t p0[3], p1[3];
                        split_bf16x3(v[q][0] * X6_SCALE, v[q][1] * X6_SCALE, p0[0], p0[1], p0[2]);
                        split_bf16x3(v[q][2] * X6_SCALE, v[q][3] * X6_SCALE, p1[0], p1[1], p1[2]);
                        uint16_t* d = reinterpret_cast<uint16_t*>(dst) + (y - KP) * RB + b + 4 * q;
#pragma unroll
                        for (int p = 0; p < 3; ++p) *reinterpret_cast<uint2*>(d + p * 16 * NJ * RB) = make_uint2(p0[p], p1[p]);
                    }
                } else {
                    float top = 0.f;
#pragma unroll
                    for (int q = 0; q < Q4; ++q) top = fmaxf(fmaxf(fmaxf(top, v[q][0]), fmaxf(v[q][1], v[q][2])), v[q][3]);
                    top = fmaxf(top, __shfl_xor(top, 1, 64));       // (the eight lanes of a row)
                    top = fmaxf(top, __shfl_xor(top, 2, 64));
                    top = fmaxf(top, __shfl_xor(top, 4, 64));
                    const float old = fac[x], now = stat_row_factor(top, old);
                    fac[x] = now;
                    if (b == 0) {
                        reinterpret_cast<float*>(buf + LY::OFF_M)[sl * 64 + y] = now == old || old == 0.f ? 1.f : now * (1.f / old);
                        sF[sl * 64 + y] = now == 0.f ? 1.f : now;
                    }
#pragma unroll
                    for (int q = 0; q < Q4; ++q)
                        *reinterpret_cast<floatx4*>(reinterpret_cast<float*>(dst + LY::OFF_Q) + y * RF + b + 4 * q) = v[q] * now;
                }
            }
        }
        if (lane < 32) {
            const int b = PS * (lane & 7), nsl = samples_of(slot);
#pragma unroll
            for (int q = 0; q < Q4; ++q) {
#pragma unroll
                for (int c = 0; c < 4; ++c) l4[q][c] = s + b + 4 * q + c < nsl ? l4[q][c] * X6_SCALE : 0.f;
                *reinterpret_cast<floatx4*>(reinterpret_cast<float*>(buf + LY::OFF_L) + wave * 4 * RF + (lane >> 3) * RF + b + 4 * q) = l4[q];
            }
        }
    };

    floatx4 acc[NRT][NJ];
    auto clear = [&] {
#pragma unroll
        for (int r = 0; r < NRT; ++r)
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt) acc[r][jt] = floatx4{0.f, 0.f, 0.f, 0.f};
    };
    clear();
    // the sums of 32 samples, s .. of a step; lane group kg contracts the samples s + 8 kg .. + 7.  Small parts first, and the
    // sums over the batch grow by one rounded addition per step: with all six products added to them the root mean square error
    // of Nw grew with the batch (500 samples, K = 40: 2.6e-7 of a value).
    auto products = [&](const char* buf, int s) {
        const char* mine = buf + slot * LY::SLOT;
        const uint16_t* rp = reinterpret_cast<const uint16_t*>(mine) + c16 * RB + 8 * kg + s;
        const float* qp = reinterpret_cast<const float*>(mine + LY::OFF_Q) + (4 * kt0 + (c16 >> 2)) * RF + 8 * kg + s;
        const float* lp = reinterpret_cast<const float*>(buf + LY::OFF_L) + wave * 4 * RF + (c16 & 3) * RF + 8 * kg + s;
        uint32x4 rb[NJ][3];
#pragma unroll
        for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
            for (int p = 0; p < 3; ++p) rb[jt][p] = *reinterpret_cast<const uint32x4*>(rp + (p * 16 * NJ + 16 * jt) * RB);
        const floatx4 la = *reinterpret_cast<const floatx4*>(lp), lb = *reinterpret_cast<const floatx4*>(lp + 4);
#pragma unroll
        for (int r = 0; r < NRT; ++r) {
            const floatx4 qa = *reinterpret_cast<const floatx4*>(qp + 4 * r * RF);
            const floatx4 qb = *reinterpret_cast<const floatx4*>(qp + 4 * r * RF + 4);
            float w[8];
#pragma unroll
            for (int c = 0; c < 4; ++c) { w[c] = qa[c] * la[c]; w[4 + c] = qb[c] * lb[c]; }
            uint32x4 a[3];
            split_octet(w, a[0], a[1], a[2]);
            constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};
            floatx4 t[NJ];
#pragma unroll
            for (int p = 0; p < 6; ++p)
#pragma unroll
                for (int jt = 0; jt < NJ; ++jt)
                    t[jt] = mfma_bf16(a[PA[p]], rb[jt][PB[p]], p == 0 ? floatx4{0.f, 0.f, 0.f, 0.f} : t[jt]);
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt) acc[r][jt] += t[jt];
        }
    };
    // acc[r][jt][c]: k = 4 (kt0 + r) + kg, i = 4 it + c, j = 16 jt + c16
    const int32_t woff = e_rec[(size_t)li * EIN_BREC_INTS + 4];
    const float* W = params + woff;
    float* Nw = nshare > 1 ? part + ((size_t)sh * count + li) * ((size_t)K * K * K) : stats + woff;
    float wr[NRT][NJ][4];
    auto fetch_w = [&] {
#pragma unroll
        for (int r = 0; r < NRT; ++r)
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    wr[r][jt][c] = W[(min(4 * (kt0 + r) + kg, K - 1) * K + min(4 * it + c, K - 1)) * K + min(16 * jt + c16, K - 1)];
    };
    auto store_unit = [&] {
#pragma unroll
        for (int r = 0; r < NRT; ++r) {
            const int k = 4 * (kt0 + r) + kg;
            const float inv = 1.f / sF[slot * 64 + min(k, KP - 1)];
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int j = 16 * jt + c16;
                    if (k < K && 4 * it + c < K && j < K) {
                        float* dst = Nw + (k * K + 4 * it + c) * K + j;
                        *dst = (ACCUM ? *dst : 0.f) + wr[r][jt][c] * (acc[r][jt][c] * X6_UNSCALE * inv);
                    }
                }
        }
    };

    constexpr bool EARLY = !SEQ && NRT <= 4;            // (registers to spare: the weights come in with the first rows)
    fetch(0);
    if (EARLY && work) fetch_w();
    stage(0, lds_c);
    int buf = 0;
#pragma unroll 1
    for (int s = 0; s < share; s += STEP) {
        __syncthreads();                               // the step is staged; readers of the other buffer are done
        char* here = lds_c + buf * LY::BUF;
        if (!SEQ && s > 0 && work) {                   // (s = 0: no sums yet)
            const float* change = reinterpret_cast<const float*>(here + LY::OFF_M) + slot * 64;
            if (__any(lane < KP && change[min(lane, KP - 1)] != 1.f)) {
#pragma unroll
                for (int r = 0; r < NRT; ++r) {
                    const float ch = change[min(4 * (kt0 + r) + kg, KP - 1)];
#pragma unroll
                    for (int jt = 0; jt < NJ; ++jt) acc[r][jt] *= ch;
                }
            }
        }
        if constexpr (SEQ) {
            if (work) {
#pragma unroll 1
                for (int h = 0; h < NH; ++h, kt0 += NRT) {
                    fetch_w();
                    if (h > 0) clear();
#pragma unroll 1
                    for (int u = 0; u < B; u += 32) products(here, u);
                    store_unit();
                }
            }
        } else {
            const bool more = s + STEP < share;
            if (more) fetch(s + STEP);
            if (work) products(here, 0);
            if (more) stage(s + STEP, lds_c + (buf ^ 1) * LY::BUF);
            buf ^= 1;
        }
    }
    if (!SEQ && work) {
        if (!EARLY) fetch_w();
        store_unit();
    }
}

// stats[item][r] (+)= sum over the vper blocks of part[.][item][r], job blockIdx.y of the list
__global__ void k_sum_partial_stats(PartialSumJobs jobs, float* __restrict__ stats, int accumulate) {
    const PartialSumJob& j = jobs.job[blockIdx.y];
    const size_t n = (size_t)j.count * j.block;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const int li = (int)(i / j.block);
        float* dst = stats + (size_t)j.e_woff[li] + (i - (size_t)li * j.block);
        float sum = accumulate ? *dst : 0.f;
        for (int v = 0; v < j.vper; ++v) sum += j.part[(size_t)v * n + i];
        *dst = sum;
    }
}

template <int KQ, int NH, int STEP>
void launch_stats_units(const EinStatsWork& w, bool accumulate, float* stats, hipStream_t s) {
    using LY = StatLayout<KQ, NH, STEP>;
    static std::once_flag attr_set[EINET_MAX_DEVICES];
    int dev = 0;
    (void)hipGetDevice(&dev);
    std::call_once(attr_set[dev % EINET_MAX_DEVICES], [&] {
        allow_dynamic_lds(&k_einsum_stats<KQ, NH, STEP, true>, LY::LDS_BYTES);
        allow_dynamic_lds(&k_einsum_stats<KQ, NH, STEP, false>, LY::LDS_BYTES);
    });
    const int nshare = STEP == ST_WHOLE ? 1 : ein_stat_shares(w.count, w.K, w.B), share = ein_stat_share(nshare, w.B);
    const long long units = (long long)w.count * nshare * LY::UI;
    const int per = (int)std::min<long long>(LY::PER, (units + EINET_NUM_CUS - 1) / EINET_NUM_CUS);
    const long long wgs = (units + per - 1) / per;
#define EINET_LAUNCH(ACC)                                                                                                    \
    hipLaunchKernelGGL((k_einsum_stats<KQ, NH, STEP, ACC>), dim3((unsigned)wgs), dim3(512), LY::LDS_BYTES, s, w.rec, w.params, \
                       stats, w.img, w.first, w.count, per, nshare, share, w.part, w.B, w.K)
    if (accumulate && nshare == 1) EINET_LAUNCH(true);
    else EINET_LAUNCH(false);                          // (blocks of shares are written, not added to)
#undef EINET_LAUNCH
}

template <int KQ>
void launch_stats_kq(const EinStatsWork& w, bool accumulate, float* stats, hipStream_t s) {
    // a wave takes a whole slice where that gives every compute unit four waves; otherwise about three row tiles of it (K = 40, 7
    // items, 500 samples: 15.7 us, with whole slices 34.8).  Batches of ST_WHOLE at most in one step: K = 40, 194 items, 128
    // samples: 40.9 us, in steps of 32 samples 49.2; K = 30, 140 items, 100 samples: 23.1 and 25.4
    constexpr int BIG = KQ > 12 ? 2 : 1, SMALL = (KQ + 2) / 3;
    if ((long long)w.count * KQ < 4 * EINET_NUM_CUS) {
        launch_stats_units<KQ, SMALL, 32>(w, accumulate, stats, s);
        return;
    }
    if constexpr (KQ <= 12) {
        if (w.B <= ST_WHOLE) {
            launch_stats_units<KQ, 2, ST_WHOLE>(w, accumulate, stats, s);
            return;
        }
    }
    launch_stats_units<KQ, BIG, 32>(w, accumulate, stats, s);
}

void launch_statistics(const EinStatsWork& w, bool accumulate, float* stats, hipStream_t s) {
    if (w.K <= 16) {
        switch ((w.K + 3) / 4) {
#define EINET_CASE(J) case J: launch_stats_small<J>(w, accumulate, stats, s); break;
            EINET_CASE(1) EINET_CASE(2) EINET_CASE(3) EINET_CASE(4)
#undef EINET_CASE
        }
        return;
    }
    switch ((w.K + 3) / 4) {
#define EINET_CASE(J) case J: launch_stats_kq<J>(w, accumulate, stats, s); break;
        EINET_CASE(5) EINET_CASE(6) EINET_CASE(7) EINET_CASE(8) EINET_CASE(9) EINET_CASE(10) EINET_CASE(11) EINET_CASE(12)
        EINET_CASE(13) EINET_CASE(14) EINET_CASE(15) EINET_CASE(16)
#undef EINET_CASE
    }
}

}  // namespace

void launch_sum_partial_stats(const PartialSumList& list, float* stats, bool accumulate, hipStream_t s) {
    PartialSumJobs jobs = list.jobs;
    int n = list.n;
    if (list.ein.count > 0) {
        const EinStatsWork& w = list.ein;
        if (!w.formed) launch_statistics(w, accumulate, stats, s);
        const int nshare = w.formed ? fused_shares(w.count, w.K, w.B) : ein_stat_shares(w.count, w.K, w.B);
        if (nshare > 1) jobs.job[n++] = PartialSumJob{w.woff, w.part, w.count, nshare, w.K * w.K * w.K};
    }
    if (n == 0) return;
    size_t most = 0;
    for (int i = 0; i < n; ++i) most = std::max(most, (size_t)jobs.job[i].count * jobs.job[i].block);
    const unsigned bx = (unsigned)std::min<size_t>((most + 255) / 256, 1024);
    hipLaunchKernelGGL(k_sum_partial_stats, dim3(bx, n), dim3(256), 0, s, jobs, stats, accumulate ? 1 : 0);
}

}  // namespace einet_impl
