// Bottom-up pass: einsum layers (Eq. 3-5) and mixing layers (App. B).
#include "bf16x6.hpp"

#include <mutex>

namespace einet_impl {

namespace {

// ------------------------------------------------------------------ einsum layer, forward
// With eL = exp(L - a), eR = exp(R - a') (a, a' the row maxima; Eq. 4) the layer needs
//     S~[b,k] = sum_i eL[b,i] * T[(k,i), b],   T[(k,i), b] = sum_j W[k,i,j] eR[b,j].
// T is a dense GEMM (rows (k,i), columns b, contraction j) on v_mfma_f32_16x16x4_f32;
// one MFMA tile holds 4 outputs k (one per 16-lane group) x 4 inputs i (one per
// accumulator register), so the i-reduction of Eq. 4 is four in-lane FMAs per tile
// and the K x K outer product of Sec. 3.2 is never formed.
//
// One workgroup per (einsum item, tile of 4 outputs k).  Its slice W[4 k][K][K] is
// contiguous in memory; it is staged once in LDS, zero-padded to multiples of 4,
// with row strides chosen so that the A-operand reads of a half-wave hit 32
// distinct banks (i-stride = 8 mod 16, k-stride = 2 mod 32, lane groups read
// consecutive j).  Every wave then takes tiles of 16 samples: eR (the B operand)
// lives in registers, eL in a wave-private LDS tile, and each tile costs KQ*KQ
// MFMAs (KQ = ceil(K/4)).
template <int KQ>
struct FwdLayout {
    static constexpr int KP = 4 * KQ;
    static constexpr int SJ = ((KP + 7) / 16) * 16 + 8;   // smallest value >= KP that is 8 mod 16
    static constexpr int SK = KP * SJ + 2;
    static constexpr int LDS_W = ((4 * SK + 3) / 4) * 4;  // W slice, rounded so the eL tiles stay 16-byte aligned
    static constexpr int SE = KP + 4;                     // row stride of a wave's eL tile
    static constexpr int LDS_FLOATS = LDS_W + 8 * 16 * SE;
};

// Orders the LDS traffic of one wave: what its lanes wrote before is visible to all its lanes after (the LDS
// serves the requests of a wave in order; this keeps the compiler from moving accesses across).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int KQ>
__global__ __launch_bounds__(512, KQ >= 14 ? 2 : 4) void k_einsum_forward(const int32_t* __restrict__ e_left,
                                                        const int32_t* __restrict__ e_right,
                                                        const int32_t* __restrict__ e_out,
                                                        const int32_t* __restrict__ e_kout,
                                                        const int32_t* __restrict__ e_woff,
                                                        const float* __restrict__ params, float* __restrict__ A,
                                                        double* __restrict__ Off, float* __restrict__ amax,
                                                        float* __restrict__ logp, int item0, int B, int K, int nkt) {
    using LY = FwdLayout<KQ>;
    constexpr int KP = LY::KP, SJ = LY::SJ, SK = LY::SK;
    extern __shared__ float Wl[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nwaves = blockDim.x >> 6;
    const int vb = xcd_contiguous_block();
    const int li = vb / nkt, kt = vb - li * nkt;
    const int item = item0 + li;
    const int kout = e_kout[li];
    if (4 * kt >= kout) return;                        // root items have a single output entry
    const float* Lp = A + (size_t)e_left[li] * B * K;
    const float* Rp = A + (size_t)e_right[li] * B * K;
    const float* W = params + e_woff[li];

    const int c = lane & 15, g = lane >> 4;          // sample column of the tile, lane group
    const int gm = c >> 2, rm = c & 3;               // as A-operand lane: row 4*gm+rm = (k = 4kt+gm, i = 4it+rm)
    const int n_btiles = (B + 15) >> 4;
    // stage W[4kt .. 4kt+3][.][.]
    if ((K & 3) == 0) {
        // four 16-byte loads per thread in flight before the first goes to LDS
        for (int q0 = tid; q0 < 4 * KP * KQ; q0 += 4 * blockDim.x) {
            float4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int q = q0 + u * blockDim.x;
                const int j4 = q % KQ, i = (q / KQ) % KP, kl = q / (KQ * KP);
                v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (q < 4 * KP * KQ && 4 * kt + kl < kout && i < K)
                    v[u] = *reinterpret_cast<const float4*>(W + ((size_t)(4 * kt + kl) * K + i) * K + 4 * j4);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int q = q0 + u * blockDim.x;
                if (q < 4 * KP * KQ) {
                    const int j4 = q % KQ, i = (q / KQ) % KP, kl = q / (KQ * KP);
                    float* dst = Wl + kl * SK + i * SJ + 4 * j4;
                    *reinterpret_cast<float2*>(dst) = make_float2(v[u].x, v[u].y);
                    *reinterpret_cast<float2*>(dst + 2) = make_float2(v[u].z, v[u].w);
                }
            }
        }
    } else {
        for (int q0 = tid; q0 < 4 * KP * KP; q0 += 8 * blockDim.x) {     // eight loads in flight, as above
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int q = q0 + u * blockDim.x;
                const int j = q % KP, i = (q / KP) % KP, kl = q / (KP * KP);
                v[u] = 0.f;
                if (q < 4 * KP * KP && 4 * kt + kl < kout && i < K && j < K) v[u] = W[((size_t)(4 * kt + kl) * K + i) * K + j];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int q = q0 + u * blockDim.x;
                if (q < 4 * KP * KP) Wl[(q / (KP * KP)) * SK + ((q / KP) % KP) * SJ + q % KP] = v[u];
            }
        }
    }
    __syncthreads();

    const float* wl = Wl + gm * SK + rm * SJ + g;    // + it*4*SJ + 4*s : contraction index j = 4s + g
    float* elw = Wl + LY::LDS_W + wave * (16 * LY::SE);   // this wave's eL tile [16][SE]
    for (int bt0 = 0; bt0 < n_btiles; bt0 += nwaves) {
        const int bt = bt0 + wave;
        const int b = bt * 16 + c;
        const bool ok = bt < n_btiles && b < B;
        // offsets of the children, needed only when the result is stored: requested now, used at the end
        double off_children = 0.0;
        if (ok && kt == 0 && g == 0)
            off_children = Off[(size_t)e_left[li] * B + b] + Off[(size_t)e_right[li] * B + b];
        // lane (c, g) holds entries 4s+g of row b of both inputs
        float er[KQ], el[KQ];
        float mr = -INFINITY, ml = -INFINITY;
        if ((K & 3) == 0) {
            // The 16 rows of the tile are contiguous in memory: they are fetched with 16-byte loads, consecutive
            // lanes consecutive addresses, and reach the operand layout through the wave's LDS tile.
            constexpr int NFW = (16 * KQ + 63) / 64;
            const int rows = bt < n_btiles ? min(16, B - 16 * bt) : 0;
            float4 rawR[NFW], rawL[NFW];
#pragma unroll
            for (int n = 0; n < NFW; ++n) {
                const int f = min(lane + 64 * n, max(rows, 1) * KQ - 1);
                rawR[n] = rawL[n] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (rows > 0) {
                    rawR[n] = *reinterpret_cast<const float4*>(Rp + (size_t)16 * bt * K + 4 * f);
                    rawL[n] = *reinterpret_cast<const float4*>(Lp + (size_t)16 * bt * K + 4 * f);
                }
            }
            wave_lds_sync();                         // the previous tile's reads of eL are done
#pragma unroll
            for (int n = 0; n < NFW; ++n) {
                const int f = lane + 64 * n;
                if (f < 16 * KQ) *reinterpret_cast<float4*>(elw + (f / KQ) * LY::SE + 4 * (f % KQ)) = rawR[n];
            }
            wave_lds_sync();
#pragma unroll
            for (int s = 0; s < KQ; ++s) er[s] = ok ? elw[c * LY::SE + 4 * s + g] : -INFINITY;
            wave_lds_sync();
#pragma unroll
            for (int n = 0; n < NFW; ++n) {
                const int f = lane + 64 * n;
                if (f < 16 * KQ) *reinterpret_cast<float4*>(elw + (f / KQ) * LY::SE + 4 * (f % KQ)) = rawL[n];
            }
            wave_lds_sync();
#pragma unroll
            for (int s = 0; s < KQ; ++s) el[s] = ok ? elw[c * LY::SE + 4 * s + g] : -INFINITY;
        } else {
#pragma unroll
            for (int s = 0; s < KQ; ++s) {
                const int j = 4 * s + g;
                const bool in = ok && j < K;
                er[s] = in ? Rp[(size_t)b * K + j] : -INFINITY;
                el[s] = in ? Lp[(size_t)b * K + j] : -INFINITY;
            }
            wave_lds_sync();                         // the previous tile's reads of eL are done
        }
#pragma unroll
        for (int s = 0; s < KQ; ++s) {
            mr = fmaxf(mr, er[s]);
            ml = fmaxf(ml, el[s]);
        }
        mr = fmaxf(mr, __shfl_xor(mr, 16, 64));
        mr = fmaxf(mr, __shfl_xor(mr, 32, 64));
        ml = fmaxf(ml, __shfl_xor(ml, 16, 64));
        ml = fmaxf(ml, __shfl_xor(ml, 32, 64));
        if (mr == -INFINITY) mr = 0.f;               // an all-zero input vector: exp(-inf) = 0, no NaN
        if (ml == -INFINITY) ml = 0.f;
        // (the tile is private to the wave, and every lane overwrites the entries it has read itself)
#pragma unroll
        for (int s = 0; s < KQ; ++s) {
            er[s] = __expf(er[s] - mr);              // stays in registers: the B operand
            elw[c * LY::SE + 4 * s + g] = __expf(el[s] - ml);
        }
        wave_lds_sync();
        float sacc = 0.f;
#pragma unroll
        for (int it = 0; it < KQ; ++it) {
            floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < KQ; ++s)
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wl[it * 4 * SJ + 4 * s], er[s], acc, 0, 0, 0);
            const float4 e4 = *reinterpret_cast<const float4*>(elw + c * LY::SE + 4 * it);
            sacc += acc[0] * e4.x + acc[1] * e4.y + acc[2] * e4.z + acc[3] * e4.w;
        }
        const int k = 4 * kt + g;
        const float res = __logf(sacc);                // residual against Off[left] + Off[right] + ml + mr
        if (ok && k < kout) A[((size_t)e_out[li] * B + b) * K + k] = res;
        if (ok && kt == 0 && g == 0) {
            const double off = off_children + (double)ml + (double)mr;
            Off[(size_t)e_out[li] * B + b] = off;
            if (logp && e_out[li] == 0) logp[b] = (float)(off + (double)res);   // node 0: the root region, one entry
            amax[((size_t)item * 2) * B + b] = ml;     // the shifts, kept for the top-down pass
            amax[((size_t)item * 2 + 1) * B + b] = mr;
        }
    }
}

// ------------------------------------------------------------------ einsum layer, forward, K = 24 and 48
// The same factorisation on v_mfma_f32_32x32x2_f32 (the fp32 shape that issues at the full rate of the matrix
// pipe), as one workgroup per compute unit that walks a run of work units.  A tile of the product T has 32 rows
// (k, i) and 32 samples; with i fastest, groups of 8 rows stay inside one k, and a lane holds four consecutive i of
// four such groups, so the i-reduction is again in-lane: 16 FMAs per tile.  K / 8 tiles hold exactly four k.
typedef float floatx16 __attribute__((ext_vector_type(16)));

template <int K8>
struct FwdSLayout {
    static constexpr int K = 8 * K8;
    static constexpr int RS = K + 4;                 // row stride (floats): RS/4 odd -> 16-byte operand reads of 8 lanes hit 32 banks
    static constexpr int SLICE = 4 * K * RS;         // W[4 k][K i][RS]
    static constexpr int OFF_E = 2 * SLICE;          // eR, eL of the four sample tiles: [tile][2][K8][64 lanes][4]
    static constexpr int OFF_S = OFF_E + 4 * 2 * K8 * 256;   // sums of a unit: [2 slots][tile][64 lanes][4]
    static constexpr int LDS_FLOATS = OFF_S + 2 * 4 * 256;
    static constexpr int NQ4 = 4 * K * (K / 4);      // float4 of a slice
    static constexpr int NL = (NQ4 + 255) / 256;     // per producer thread
};

// A workgroup owns a run of units; a unit is (item, batch chunk of 128 samples, 4 outputs k) = K8 tiles of 32 rows
// (k, i) of the product W[(k,i), j] eR[j, b].  Waves 0-3 only run the matrix pipe: wave w owns samples 32 w .. 32 w + 31
// of the chunk, reads its operands from LDS and leaves four sums per lane in LDS.  Waves 4-7 do everything else: they
// bring the W slices and the child rows in, form exp(x - max), and turn the sums of the previous unit into log values.
template <int K8>
__global__ __launch_bounds__(512, 1) void k_einsum_forward_s(const int32_t* __restrict__ e_left,
                                                           const int32_t* __restrict__ e_right,
                                                           const int32_t* __restrict__ e_out,
                                                           const int32_t* __restrict__ e_woff,
                                                           const float* __restrict__ params, float* __restrict__ A,
                                                           double* __restrict__ Off, float* __restrict__ amax,
                                                           int item0, int count, int B) {
    using LY = FwdSLayout<K8>;
    constexpr int K = LY::K, RS = LY::RS, NQ = K / 4, NL = LY::NL;
    extern __shared__ float lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 31, h = lane >> 5;
    const int nt = wave & 3;                          // sample tile of this wave (both roles)
    const int nchunks = (B + 127) >> 7;
    const int U = count * nchunks * NQ;              // unit = (item, chunk, quad), quad fastest
    const int g = xcd_contiguous_block();
    const int u0 = (int)((long long)g * U / gridDim.x), u1 = (int)((long long)(g + 1) * U / gridDim.x);
    if (u0 >= u1) return;
    // position of the first unit
    int quad = u0 % NQ, chunk = (u0 / NQ) % nchunks, li = u0 / (NQ * nchunks);
    float* erl = lds + LY::OFF_E + nt * (2 * K8 * 256) + lane * 4;       // + (2 * which + t) * 256 ... see below

    if (wave >= 4) {
        // ------------------------------------------------------------ producer waves
        const int pt = tid - 256;
        floatx4 wv[NL];
#define FETCH_W(li_, quad_)                                                                \
    {                                                                                      \
        const float* W_ = params + e_woff[li_] + (size_t)(quad_) * 4 * K * K;              \
        _Pragma("unroll") for (int q = 0; q < NL; ++q) {                                   \
            const int f = min(pt + 256 * q, LY::NQ4 - 1);                                  \
            wv[q] = *reinterpret_cast<const floatx4*>(W_ + (size_t)4 * f);                 \
        }                                                                                  \
    }
#define STORE_W(buf_)                                                                      \
    {                                                                                      \
        _Pragma("unroll") for (int q = 0; q < NL; ++q) {                                   \
            const int f = pt + 256 * q;                                                    \
            const int row = f / (K / 4), c4 = f - row * (K / 4);                           \
            if (f < LY::NQ4) *reinterpret_cast<floatx4*>((buf_) + row * RS + 4 * c4) = wv[q]; \
        }                                                                                  \
    }
        // rows of (item, chunk): lane (n, h) of tile nt takes entries 8 t + 4 h .. + 3 of sample 32 nt + n; exp(x - max)
        // goes to LDS for the matrix wave of the same tile; the item's first unit also owns the offsets and shifts
        auto rows = [&](int rli, int rchunk, bool owner) {
            const int b = rchunk * 128 + nt * 32 + n;
            const int bc = min(b, B - 1);              // rows beyond the batch read the last one again
            const int left = e_left[rli], right = e_right[rli];
            const float* Lp = A + ((size_t)left * B + bc) * K + 4 * h;
            const float* Rp = A + ((size_t)right * B + bc) * K + 4 * h;
            floatx4 rawR[K8], rawL[K8];
#pragma unroll
            for (int t = 0; t < K8; ++t) {
                rawR[t] = *reinterpret_cast<const floatx4*>(Rp + 8 * t);
                rawL[t] = *reinterpret_cast<const floatx4*>(Lp + 8 * t);
            }
            double off_children = 0.0;
            if (owner && h == 0) off_children = Off[(size_t)left * B + bc] + Off[(size_t)right * B + bc];
            float xr = -INFINITY, xl = -INFINITY;
#pragma unroll
            for (int t = 0; t < K8; ++t) {
                xr = fmaxf(fmaxf(xr, fmaxf(rawR[t][0], rawR[t][1])), fmaxf(rawR[t][2], rawR[t][3]));
                xl = fmaxf(fmaxf(xl, fmaxf(rawL[t][0], rawL[t][1])), fmaxf(rawL[t][2], rawL[t][3]));
            }
            xr = fmaxf(xr, __shfl_xor(xr, 32, 64));
            xl = fmaxf(xl, __shfl_xor(xl, 32, 64));
            if (xr == -INFINITY) xr = 0.f;             // an all-zero input vector: exp(-inf) = 0, no NaN
            if (xl == -INFINITY) xl = 0.f;
#pragma unroll
            for (int t = 0; t < K8; ++t) {
                floatx4 er, el;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    er[c] = __expf(rawR[t][c] - xr);
                    el[c] = __expf(rawL[t][c] - xl);
                }
                *reinterpret_cast<floatx4*>(erl + t * 256) = er;
                *reinterpret_cast<floatx4*>(erl + (K8 + t) * 256) = el;
            }
            if (owner && h == 0 && b < B) {
                const int out = e_out[rli];
                Off[(size_t)out * B + b] = off_children + (double)xl + (double)xr;
                amax[((size_t)(item0 + rli) * 2) * B + b] = xl;
                amax[((size_t)(item0 + rli) * 2 + 1) * B + b] = xr;
            }
        };
        // sums of a finished unit -> residuals log S~
        auto finish = [&](int fli, int fchunk, int fquad, int slot) {
            const float* sp = lds + LY::OFF_S + (slot * 4 + nt) * 256 + n * 4;
            const floatx4 s0 = *reinterpret_cast<const floatx4*>(sp);
            const floatx4 s1 = *reinterpret_cast<const floatx4*>(sp + 128);
            const int b = fchunk * 128 + nt * 32 + n;
            if (h == 0 && b < B) {
                floatx4 r;
#pragma unroll
                for (int c = 0; c < 4; ++c) r[c] = __logf(s0[c] + s1[c]);
                *reinterpret_cast<floatx4*>(A + ((size_t)e_out[fli] * B + b) * K + 4 * fquad) = r;
            }
        };
        rows(li, chunk, quad == 0);                     // (the matrix waves bring the first slice in)
        // position of the unit whose slice is in flight
        int lq = quad, lc = chunk, lli = li;
        auto advance = [&](int& q_, int& c_, int& i_) {
            if (++q_ == NQ) { q_ = 0; if (++c_ == nchunks) { c_ = 0; ++i_; } }
        };
        advance(lq, lc, lli);
        if (u0 + 1 < u1) FETCH_W(lli, lq)
        __syncthreads();                                // B0: slice u0 and the first rows are in LDS
        __syncthreads();                                // X: the matrix waves hold the rows in registers
        int pq = quad, pc = chunk, pli = li;            // previous unit
        for (int u = u0; u < u1; ++u) {
            // the matrix waves work on unit u = (li, chunk, quad)
            if (u + 1 < u1) {
                STORE_W(lds + ((u + 1 - u0) & 1) * LY::SLICE)
                int q2 = lq, c2 = lc, i2 = lli;
                advance(q2, c2, i2);
                if (u + 2 < u1) FETCH_W(i2, q2)
            }
            if (u > u0) finish(pli, pc, pq, (u - 1 - u0) & 1);
            const bool new_rows = u + 1 < u1 && quad == NQ - 1;
            if (new_rows) rows(lli, lc, true);
            pq = quad; pc = chunk; pli = li;
            quad = lq; chunk = lc; li = lli;
            advance(lq, lc, lli);
            __syncthreads();                            // B(u+1)
            if (new_rows) __syncthreads();              // X
        }
        finish(pli, pc, pq, (u1 - 1 - u0) & 1);
    } else {
        // ------------------------------------------------------------ matrix waves
        float er[4 * K8], el[K8][4];
        const bool active = chunk * 128 + nt * 32 < B || nchunks > 1;     // (a tile beyond a short batch does nothing)
        {
            // the first W slice, while the producer waves fetch and shift the first rows
            const float* W_ = params + e_woff[li] + (size_t)quad * 4 * K * K;
            floatx4 w0[NL];
#pragma unroll
            for (int q = 0; q < NL; ++q) w0[q] = *reinterpret_cast<const floatx4*>(W_ + (size_t)4 * min(tid + 256 * q, LY::NQ4 - 1));
#pragma unroll
            for (int q = 0; q < NL; ++q) {
                const int f = tid + 256 * q;
                const int row = f / (K / 4), c4 = f - row * (K / 4);
                if (f < LY::NQ4) *reinterpret_cast<floatx4*>(lds + row * RS + 4 * c4) = w0[q];
            }
        }
        __syncthreads();                                // B0
        bool load_rows = true;
        for (int u = u0; u < u1; ++u) {
            if (load_rows) {
#pragma unroll
                for (int t = 0; t < K8; ++t) {
                    const floatx4 r = *reinterpret_cast<const floatx4*>(erl + t * 256);
                    const floatx4 l = *reinterpret_cast<const floatx4*>(erl + (K8 + t) * 256);
#pragma unroll
                    for (int c = 0; c < 4; ++c) { er[4 * t + c] = r[c]; el[t][c] = l[c]; }
                }
                __syncthreads();                        // X
            }
            const float* wrow = lds + ((u - u0) & 1) * LY::SLICE + n * RS + 4 * h;
            float sk[4] = {0.f, 0.f, 0.f, 0.f};
            if (active) {
                floatx4 a[2][K8];
                floatx16 acc[2];
#pragma unroll
                for (int t = 0; t < K8; ++t) a[0][t] = *reinterpret_cast<const floatx4*>(wrow + 8 * t);
#pragma unroll
                for (int m = 0; m <= K8; ++m) {
                    if (m + 1 < K8) {
#pragma unroll
                        for (int t = 0; t < K8; ++t)
                            a[(m + 1) & 1][t] = *reinterpret_cast<const floatx4*>(wrow + 32 * (m + 1) * RS + 8 * t);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if (m < K8) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[m & 1][r] = 0.f;
#pragma unroll
                        for (int t = 0; t < K8; ++t) {
#pragma unroll
                            for (int c = 0; c < 4; ++c)
                                acc[m & 1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[m & 1][t][c], er[4 * t + c], acc[m & 1], 0, 0, 0);
                        }
                    }
                    if (m > 0) {
                        // acc[4 a + c]: row 8 a + 4 h + c of tile m - 1; group g = 4 (m - 1) + a: k = g / K8, i = 8 (g % K8) + 4 h + c
#pragma unroll
                        for (int a4 = 0; a4 < 4; ++a4) {
                            const int gg = 4 * (m - 1) + a4, kq = gg / K8, uu = gg % K8;
#pragma unroll
                            for (int c = 0; c < 4; ++c) sk[kq] = fmaf(acc[(m - 1) & 1][4 * a4 + c], el[uu][c], sk[kq]);
                        }
                    }
                }
            }
            floatx4 sv = {sk[0], sk[1], sk[2], sk[3]};
            *reinterpret_cast<floatx4*>(lds + LY::OFF_S + (((u - u0) & 1) * 4 + nt) * 256 + lane * 4) = sv;
            load_rows = u + 1 < u1 && quad == NQ - 1;
            if (++quad == NQ) quad = 0;
            __syncthreads();                            // B(u+1)
        }
    }
#undef FETCH_W
#undef STORE_W
}

// ------------------------------------------------------------------ einsum layer, forward, K from 17 to 40
// The same factorisation on the bfloat16 matrix pipe at float32 precision (bf16x6.hpp), as one workgroup per compute unit
// that walks a run of work units.  A unit is (item, chunk of 128 samples, 4 outputs k).  A tile of the product T has 16
// rows (four left entries i x four outputs k) and 16 samples; with row m = 4 (i % 4) + k % 4 the lane group kg holds the
// left entries i = 4 t + kg and its four accumulators the four outputs, so the i-reduction of Eq. 4 is four in-lane FMAs
// per tile and the four lane groups' shares are added when the sums are turned into logarithms.
//
// Waves 0-3 only run the matrix pipe: wave w owns samples 32 w .. 32 w + 31 of the chunk as two sets of 16, keeps the
// operand of eR (split into bfloat16 octets) and eL in registers, reads the operand of the W rows from LDS (16 bytes per
// lane and register, each used for both sets) and leaves its sums in LDS.  Waves 4-7 do everything else: they bring the W
// slices in and split them (the slice of the next unit, requested one unit ahead), bring the rows of the next item in
// (also requested one unit ahead), form exp(x - max), and turn the sums of the previous unit into log values.
// K need not be a multiple of 8: entries beyond K are zeros in the operands (EXACT = false; rows of W and of A then start
// at any multiple of four bytes).  kout: output entries of every item of the launch (K, or 1 in the root's layer).
//
// At K = 40 a unit is 160 instructions of 16 cycles per matrix wave (2560 cycles, the float32 shape needed 6400); with 128
// samples a launch is bound by its start (tables, rows, first slice) and by the W slices coming in, with many chunks by the
// matrix pipe and the vector instructions beside it.  Layers of 24 / 50 / 60 / 40 / 20 items, K = 40: 8 / 12 / 14 / 12 / 8 us
// with 128 samples (9 / 13.5 / 17 / 13 / 8 on v_mfma_f32_32x32x2_f32), 23 / 41 / 48 / 34 / 21 us with 1000 (34 / 64 / 74 / 52 /
// 31).  Spreading the producers' work over eight matrix waves, so that it interleaves with their instructions, was slower
// (56 us for the layer of 60): reading the W operand for half of the tiles by twice as many waves costs more LDS time.
template <int K8>
struct FwdXLayout {
    using X = X6<K8>;
    static constexpr int KP = X::KP, NT = X::NT;
    static constexpr int SLICE = NT * X::BYTES;      // bytes of a W slice
    static constexpr int RS = KP + 4;                     // row stride (floats) of eR, eL: RS/4 odd
    static constexpr int OFF_E = 2 * SLICE;               // eR [128][RS], eL [128][RS]
    static constexpr int OFF_S = OFF_E + 2 * 128 * RS * 4;   // sums: [2 slots][4 waves][2 sets][64 lanes][4]
    static constexpr int LDS_BYTES = OFF_S + 2 * 4 * 2 * 1024;
    static constexpr int NI = 4 * KP * K8;           // octets of a slice
    static constexpr int NL = (NI + 255) / 256;           // per producer thread
};

template <int K8, bool EXACT>
__global__ __launch_bounds__(512, 1) void k_einsum_forward_x(const int32_t* __restrict__ e_rec, const float* __restrict__ params,
                                                           float* __restrict__ A, double* __restrict__ Off,
                                                           float* __restrict__ amax, int item0, int count, int B, int K_, int kout) {
    using LY = FwdXLayout<K8>;
    using X = X6<K8>;
    constexpr int KP = LY::KP, NT = LY::NT, RS = LY::RS, NL = LY::NL;
    extern __shared__ __attribute__((aligned(16))) char lds_c[];
    const int K = EXACT ? KP : K_;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nt = wave & 3;                          // sample tile (32 samples) of this wave (both roles)
    const int nchunks = (B + 127) >> 7;
    const int NG = (kout + 3) / 4;    // groups of outputs per item
    const int U = count * nchunks * NG;               // unit = (item, chunk, group), group fastest
    const int wg = xcd_contiguous_block();
    const int u0 = (int)((long long)wg * U / gridDim.x), u1 = (int)((long long)(wg + 1) * U / gridDim.x);
    if (u0 >= u1) return;
    struct Pos { int g, c, li; };
    auto advance = [&](Pos& q) {
        if (++q.g == NG) { q.g = 0; if (++q.c == nchunks) { q.c = 0; ++q.li; } }
    };
    Pos pos{u0 % NG, (u0 / NG) % nchunks, u0 / (NG * nchunks)};
    float* eRl = reinterpret_cast<float*>(lds_c + LY::OFF_E);
    float* eLl = eRl + 128 * RS;
    float* sums = reinterpret_cast<float*>(lds_c + LY::OFF_S);

    // W octets of a unit: thread t of 256 takes every 256th octet (row (k, i), octet of j; consecutive threads consecutive
    // addresses; threads beyond the last octet repeat it: the same values to the same place); entries that do not exist
    // are zero.  When K is not a multiple of 8 the last octet of a row starts at K - 8, so that it too is two 16-byte
    // loads: its first entries, which the octet before holds already, are zeros in W, and the operand of eR starts its
    // last octet there as well.
    floatx4 wv[NL][2];
    int wsrc[NL], wdst[NL][3], wk[NL];
    uint32_t wlive[NL];                               // entries of the octet that count, a bit each
#pragma unroll
    for (int x = 0; x < NL; ++x) {
        const int f = min((tid & 255) + 256 * x, LY::NI - 1);
        const int o = f % K8, i = (f / K8) % KP, kl = f / (K8 * KP), start = EXACT ? 8 * o : min(8 * o, K - 8);
        wk[x] = kl;
        wsrc[x] = (kl * K + min(i, K - 1)) * K + start;
        wlive[x] = i >= K ? 0u : (0xffu << (8 * o - start)) & 0xffu;
#pragma unroll
        for (int p = 0; p < 3; ++p)                   // (the rows of the three parts are swizzled differently)
            wdst[x][p] = (i >> 2) * X::UNITS + x6_unit<K8>(p, o, 4 * (i & 3) + kl);
    }
    auto fetch_w = [&](const Pos& q) {
        const float* W = params + e_rec[q.li * EIN_REC_INTS + 3] + (size_t)q.g * 4 * K * K;
#pragma unroll
        for (int x = 0; x < NL; ++x) {
            const float* p = W + wsrc[x];
            if (!EXACT && 4 * q.g + wk[x] >= kout) p -= wk[x] * K * K;     // (outputs beyond the last one)
            wv[x][0] = *reinterpret_cast<const floatx4u*>(p);
            wv[x][1] = *reinterpret_cast<const floatx4u*>(p + 4);
        }
    };
    auto store_w = [&](int buf, int g) {
        uint32x4* dst = reinterpret_cast<uint32x4*>(lds_c + buf * LY::SLICE);
#pragma unroll
        for (int x = 0; x < NL; ++x) {
            const uint32_t live = 4 * g + wk[x] < kout ? wlive[x] : 0u;
            float v[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) v[c] = EXACT || ((live >> c) & 1) ? wv[x][c >> 2][c & 3] * X6_SCALE : 0.f;
            uint32x4 part[3];
            split_octet(v, part[0], part[1], part[2]);
#pragma unroll
            for (int p = 0; p < 3; ++p) dst[wdst[x][p]] = part[p];
        }
    };

    if (wave >= 4) {
        // ------------------------------------------------------------ producer waves
        const int n = lane & 31, h = lane >> 5;
        // rows of (item, chunk): lane (n, h) of tile nt takes entries 8 t + 4 h .. + 3 of sample 32 nt + n; exp(x - max)
        // goes to LDS for the matrix waves; the item's first unit also owns the offsets and shifts
        floatx4 rawR[K8], rawL[K8];
        double off_children = 0.0;
        auto fetch_rows = [&](const Pos& q) {
            const int32_t* rec = e_rec + q.li * EIN_REC_INTS;
            const int bc = min(q.c * 128 + nt * 32 + n, B - 1);    // rows beyond the batch read the last one again
            const size_t rl = (size_t)rec[0] * B + bc, rr = (size_t)rec[1] * B + bc;
            const float* Lp = A + rl * K;
            const float* Rp = A + rr * K;
#pragma unroll
            for (int t = 0; t < K8; ++t) {
                const int e = 8 * t + 4 * h;
                if (EXACT) {
                    rawR[t] = *reinterpret_cast<const floatx4*>(Rp + e);
                    rawL[t] = *reinterpret_cast<const floatx4*>(Lp + e);
                } else if (e + 4 <= K) {
                    rawR[t] = *reinterpret_cast<const floatx4u*>(Rp + e);
                    rawL[t] = *reinterpret_cast<const floatx4u*>(Lp + e);
                } else {
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        rawR[t][c] = Rp[min(e + c, K - 1)];
                        rawL[t][c] = Lp[min(e + c, K - 1)];
                    }
                }
            }
            if (q.g == 0 && h == 0) off_children = Off[rl] + Off[rr];
        };
        auto stage_rows = [&](const Pos& q) {
            float xr = -INFINITY, xl = -INFINITY;
#pragma unroll
            for (int t = 0; t < K8; ++t) {
                if (!EXACT) {
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if (8 * t + 4 * h + c >= K) rawR[t][c] = rawL[t][c] = -INFINITY;
                }
                xr = fmaxf(fmaxf(xr, fmaxf(rawR[t][0], rawR[t][1])), fmaxf(rawR[t][2], rawR[t][3]));
                xl = fmaxf(fmaxf(xl, fmaxf(rawL[t][0], rawL[t][1])), fmaxf(rawL[t][2], rawL[t][3]));
            }
            xr = fmaxf(xr, __shfl_xor(xr, 32, 64));
            xl = fmaxf(xl, __shfl_xor(xl, 32, 64));
            if (xr == -INFINITY) xr = 0.f;             // an all-zero input vector: exp(-inf) = 0, no NaN
            if (xl == -INFINITY) xl = 0.f;
#pragma unroll
            for (int t = 0; t < K8; ++t) {
                floatx4 er, el;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    er[c] = __expf(rawR[t][c] - xr) * X6_SCALE;
                    el[c] = __expf(rawL[t][c] - xl);
                }
                *reinterpret_cast<floatx4*>(eRl + (nt * 32 + n) * RS + 8 * t + 4 * h) = er;
                *reinterpret_cast<floatx4*>(eLl + (nt * 32 + n) * RS + 8 * t + 4 * h) = el;
            }
            const int b = q.c * 128 + nt * 32 + n;
            if (q.g == 0 && h == 0 && b < B) {
                Off[(size_t)e_rec[q.li * EIN_REC_INTS + 2] * B + b] = off_children + (double)xl + (double)xr;
                amax[((size_t)(item0 + q.li) * 2) * B + b] = xl;
                amax[((size_t)(item0 + q.li) * 2 + 1) * B + b] = xr;
            }
        };
        // sums of a finished unit -> residuals log S~ of sample 32 nt + n
        auto finish = [&](const Pos& q, int slot) {
            const int b = q.c * 128 + nt * 32 + n;
            const float* sp = sums + ((slot * 4 + nt) * 2 + (n >> 4)) * 256 + (n & 15) * 4;
            if (h != 0 || b >= B) return;
            floatx4 r = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kg = 0; kg < 4; ++kg) r += *reinterpret_cast<const floatx4*>(sp + kg * 64);
#pragma unroll
            for (int c = 0; c < 4; ++c) r[c] = __logf(r[c] * X6_UNSCALE);
            const int k = 4 * q.g;
            float* out = A + ((size_t)e_rec[q.li * EIN_REC_INTS + 2] * B + b) * K + k;
            if (EXACT) *reinterpret_cast<floatx4*>(out) = r;
            else
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (k + c < kout) out[c] = r[c];
        };
        fetch_rows(pos);
        stage_rows(pos);                                // (the matrix waves bring the first slice in)
        Pos nxt = pos;                                  // unit whose slice is in flight
        advance(nxt);
        if (u0 + 1 < u1) {
            fetch_w(nxt);
            if (nxt.g == 0) fetch_rows(nxt);
        }
        __syncthreads();                                // B0: slice u0 and the first rows are in LDS
        __syncthreads();                                // X: the matrix waves hold the rows in registers
        Pos prev = pos;
        for (int u = u0; u < u1; ++u) {
            // the matrix waves work on unit u = pos
            const bool more = u + 1 < u1, new_rows = more && nxt.g == 0;
            Pos n2 = nxt;
            advance(n2);
            if (more) store_w((u + 1 - u0) & 1, nxt.g);
            if (new_rows) stage_rows(nxt);
            if (u + 2 < u1) {
                fetch_w(n2);
                if (n2.g == 0) fetch_rows(n2);
            }
            if (u > u0) finish(prev, (u - 1 - u0) & 1);
            prev = pos;
            pos = nxt;
            nxt = n2;
            __syncthreads();                            // B(u+1)
            if (new_rows) __syncthreads();              // X
        }
        finish(prev, (u1 - 1 - u0) & 1);
    } else {
        // ------------------------------------------------------------ matrix waves
        const int c16 = lane & 15, kg = lane >> 4;
        fetch_w(pos);                                   // the first slice, while the producers fetch and shift the first rows
        store_w(0, pos.g);
        int unit[X::NR];
#pragma unroll
        for (int a = 0; a < X::NR; ++a) unit[a] = x6_row_unit<K8>(a, kg, c16);
        uint32x4 er[2][X::NR];
        float el[NT][2];
        const bool active = pos.c * 128 + nt * 32 < B || nchunks > 1;    // (a tile beyond a short batch does nothing)
        __syncthreads();                                // B0
        bool load_rows = true;
        for (int u = u0; u < u1; ++u) {
            if (load_rows) {
                if (active) {
#pragma unroll
                    for (int s = 0; s < 2; ++s) {
                        const float* row = eRl + (nt * 32 + 16 * s + c16) * RS;
                        x6_sample_operand<K8>(kg, [&](int o, float* v) {
                            if constexpr (!EXACT) {
#pragma unroll
                                for (int c = 0; c < 8; ++c) v[c] = row[min(8 * o, K - 8) + c];
                                return;
                            }
                            const floatx4 v0 = *reinterpret_cast<const floatx4*>(row + 8 * o);
                            const floatx4 v1 = *reinterpret_cast<const floatx4*>(row + 8 * o + 4);
#pragma unroll
                            for (int c = 0; c < 4; ++c) { v[c] = v0[c]; v[4 + c] = v1[c]; }
                        }, er[s]);
#pragma unroll
                        for (int t = 0; t < NT; ++t) el[t][s] = eLl[(nt * 32 + 16 * s + c16) * RS + 4 * t + kg];
                    }
                }
                __syncthreads();                        // X
            }
            const uint32x4* wt = reinterpret_cast<const uint32x4*>(lds_c + ((u - u0) & 1) * LY::SLICE);
            if (active) {
                uint32x4 a[2][X::NR];
                floatx4 sk[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
                floatx4 acc[2][2];
#pragma unroll
                for (int z = 0; z < X::NR; ++z) a[0][z] = wt[unit[z]];
#pragma unroll
                for (int t = 0; t <= NT; ++t) {
                    if (t + 1 < NT) {
#pragma unroll
                        for (int z = 0; z < X::NR; ++z) a[(t + 1) & 1][z] = wt[(t + 1) * X::UNITS + unit[z]];
                    }
                    if (t < NT) {
                        acc[t & 1][0] = floatx4{0.f, 0.f, 0.f, 0.f};
                        acc[t & 1][1] = floatx4{0.f, 0.f, 0.f, 0.f};
                        x6_tile<K8, 2>(a[t & 1], er, acc[t & 1]);
                    }
                    if (t > 0) {
                        // (the tile before: its accumulators are ready while this one's instructions run)
#pragma unroll
                        for (int s = 0; s < 2; ++s)
#pragma unroll
                            for (int c = 0; c < 4; ++c) sk[s][c] = fmaf(acc[(t - 1) & 1][s][c], el[t - 1][s], sk[s][c]);
                    }
                }
                float* sp = sums + (((u - u0) & 1) * 4 + nt) * 512 + lane * 4;
                *reinterpret_cast<floatx4*>(sp) = sk[0];
                *reinterpret_cast<floatx4*>(sp + 256) = sk[1];
            }
            load_rows = u + 1 < u1 && pos.g == NG - 1;
            advance(pos);
            __syncthreads();                            // B(u+1)
        }
    }
}

// ------------------------------------------------------------------ einsum layer, forward, K up to 16 and K = 20
// A whole item fits a workgroup, and its launches are bound by their chain of requests and by the instructions that a compute
// unit fetches once, so this kernel is kept short: float32 operands on v_mfma_f32_16x16x4_f32 (nothing to split), a wave
// per 16 samples, all weights of the item in LDS as they are in memory.  A tile of the product T has the rows (four outputs
// k) x (four left entries i); row m = 4 (k % 4) + i % 4, so lane group g holds output 4 kt + g and its accumulators four left
// entries: the sum of Eq. 4 is in-lane.  The contraction runs over j = KQ g + s: lane group g needs KQ consecutive entries
// of its sample's row, which are one load, and of the rows of W, which are one LDS read.
// A workgroup walks `cpg` chunks of 64 samples and takes all outputs or, where there are few items, a share of them.
// Microseconds of a launch, against a kernel with operands split into bfloat16 parts (14 KB of instructions) and, for one
// sample or K = 4, the kernel above: K = 10, 1000 samples, 1280 / 640 / 320 / 160 / 80 / 40 / 20 items: 77.6 / 43.8 / 28.4 / 15.5 /
// 10.0 / 7.4 / 6.4 (84 / 47.5 / 27 / 17.5 / 11 / 8 / 6.4); K = 16, 256 samples, 48 / 100 / 120 / 80 / 40 items: 4.6 / 5.4 / 5.4 / 5.4 /
// 4.6 (5.3 / 6.8 / 7.0 / 6.6 / 5.1); one sample: 3.6 to 4.0 (4.2); K = 4, 64 samples, 2 and 1 items: 3.2 and 2.6 (3.9 and 3.8).
template <int KQ>
struct FwdCompact {
    static constexpr int KP = 4 * KQ;
    static constexpr int SI = 20;                         // row stride of W in LDS; with S 16 modulo 32 the reads of eight lanes
    static constexpr int S = KP * SI + (KP * SI % 32 == 16 ? 0 : 16);   // .. (two k, four i) hit different banks
};

template <int KQ, bool QUADS>
__global__ __launch_bounds__(256, 4) void k_einsum_forward_compact(const int32_t* __restrict__ e_rec, const float* __restrict__ params,
                                                                 float* __restrict__ A, double* __restrict__ Off,
                                                                 float* __restrict__ amax, int item0, int ngrp, int cpg,
                                                                 int nsplit, int B, int K_) {
    using LY = FwdCompact<KQ>;
    constexpr int KP = LY::KP, SI = LY::SI, S = LY::S;
    __shared__ __attribute__((aligned(16))) float wl[KP * S];
    const int K = QUADS ? KP : K_;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c16 = lane & 15, g = lane >> 4;
    const int vb = xcd_contiguous_block();
    const int part = vb % nsplit, grp = (vb / nsplit) % ngrp, li = vb / (nsplit * ngrp);
    const int q0 = part * KQ / nsplit, q1 = (part + 1) * KQ / nsplit;      // groups of four outputs
    const int32_t* rec = e_rec + (size_t)li * EIN_REC_INTS;
    const int left = rec[0], right = rec[1], out = rec[2];
    const float* W = params + rec[3] + (size_t)4 * q0 * K * K;
    const int npiece = min(4 * (q1 - q0), K - 4 * q0) * K * KQ;
    const size_t blk = (size_t)B * K;

    // ---- the weights: pieces of rows (k, i), consecutive threads consecutive pieces
    constexpr int NW = (KP * KP * KQ + 255) / 256;
    float w[NW][4];
#pragma unroll
    for (int x = 0; x < NW; ++x) {
        if (256 * x >= npiece) break;
        const int f = min(tid + 256 * x, npiece - 1);
        load_piece<KQ, QUADS>(W + (size_t)(f / KQ) * K, f % KQ, K, w[x]);
    }
    // ---- rows of this lane's sample: KQ right entries from KQ g on, all left entries
    float er[KQ], lp[KQ][4];
    double off_children = 0.0;
    auto fetch_rows = [&](int chunk) {
        const int b = min(chunk * 64 + 16 * wave + c16, B - 1);
        const float* Rp = A + (size_t)right * blk + (size_t)b * K;
        const float* Lp = A + (size_t)left * blk + (size_t)b * K;
#pragma unroll
        for (int s = 0; s < KQ; ++s) er[s] = Rp[QUADS ? KQ * g + s : min(KQ * g + s, K - 1)];
#pragma unroll
        for (int p = 0; p < KQ; ++p) load_piece<KQ, QUADS>(Lp, p, K, lp[p]);
        off_children = Off[(size_t)left * B + b] + Off[(size_t)right * B + b];
    };
    const int c0 = grp * cpg, c1 = min(c0 + cpg, (B + 63) >> 6);
    fetch_rows(c0);
    if constexpr (!QUADS) {                               // entries that do not exist are zeros
        for (int f = tid; f < KP * S / 4; f += 256) *reinterpret_cast<floatx4*>(wl + 4 * f) = floatx4{0.f, 0.f, 0.f, 0.f};
        __syncthreads();
    }
#pragma unroll
    for (int x = 0; x < NW; ++x) {
        const int f = tid + 256 * x, r = f / KQ, p = f % KQ, k = r / K, i = r - k * K;
        if (f < npiece) {
            float* dst = wl + (4 * q0 + k) * S + i * SI + 4 * p;
            if constexpr (QUADS) {
                *reinterpret_cast<floatx4*>(dst) = floatx4{w[x][0], w[x][1], w[x][2], w[x][3]};
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (4 * p + c < K) dst[c] = w[x][c];
            }
        }
    }
    __syncthreads();
    const float* wr = wl + (c16 >> 2) * S + (c16 & 3) * SI + KQ * g;
    for (int chunk = c0; chunk < c1; ++chunk) {
        const int b = chunk * 64 + 16 * wave + c16;
        if (b - c16 >= B) break;                          // (whole waves: no barrier follows)
        float xr = -INFINITY, xl = -INFINITY, el[KP];
#pragma unroll
        for (int s = 0; s < KQ; ++s) {
            if (!QUADS && KQ * g + s >= K) er[s] = -INFINITY;
            xr = fmaxf(xr, er[s]);
        }
        xr = fmaxf(xr, __shfl_xor(xr, 16, 64));
        xr = fmaxf(xr, __shfl_xor(xr, 32, 64));
#pragma unroll
        for (int p = 0; p < KQ; ++p)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                el[4 * p + c] = QUADS || 4 * p + c < K ? lp[p][c] : -INFINITY;
                xl = fmaxf(xl, el[4 * p + c]);
            }
        if (xr == -INFINITY) xr = 0.f;                    // an all-zero input vector: exp(-inf) = 0, no NaN
        if (xl == -INFINITY) xl = 0.f;
#pragma unroll
        for (int s = 0; s < KQ; ++s) er[s] = __expf(er[s] - xr);
#pragma unroll
        for (int i = 0; i < KP; ++i) el[i] = __expf(el[i] - xl);
        if (part == 0 && g == 0 && b < B) {
            Off[(size_t)out * B + b] = off_children + (double)xl + (double)xr;
            amax[(size_t)(item0 + li) * 2 * B + b] = xl;
            amax[((size_t)(item0 + li) * 2 + 1) * B + b] = xr;
        }
        float erc[KQ];
#pragma unroll
        for (int s = 0; s < KQ; ++s) erc[s] = er[s];
        if (chunk + 1 < c1) fetch_rows(chunk + 1);
        float sk[KQ > 4 ? KQ : 4] = {};
#pragma unroll
        for (int kt = 0; kt < KQ; ++kt) {
            if (kt >= q0 && kt < q1) {
                floatx4 acc[KQ];
#pragma unroll
                for (int it = 0; it < KQ; ++it) acc[it] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < KQ; ++s)
#pragma unroll
                    for (int it = 0; it < KQ; ++it)
                        acc[it] = __builtin_amdgcn_mfma_f32_16x16x4f32(wr[4 * kt * S + 4 * it * SI + s], erc[s], acc[it], 0, 0, 0);
#pragma unroll
                for (int it = 0; it < KQ; ++it)
#pragma unroll
                    for (int c = 0; c < 4; ++c) sk[kt] = fmaf(acc[it][c], el[4 * it + c], sk[kt]);
            }
        }
        // lane group g holds the outputs k = 4 kt + g
#pragma unroll
        for (int kt = 0; kt < KQ; ++kt) sk[kt] = __logf(sk[kt]);
        float* row = A + (size_t)out * blk + (size_t)min(b, B - 1) * K;
        if constexpr (QUADS && KQ <= 4) {
            transpose_groups(sk);                         // .. now 4 g .. 4 g + 3
            if (b < B && g >= q0 && g < q1) *reinterpret_cast<floatx4*>(row + 4 * g) = floatx4{sk[0], sk[1], sk[2], sk[3]};
        } else {
#pragma unroll
            for (int kt = 0; kt < KQ; ++kt)
                if (b < B && kt >= q0 && kt < q1 && 4 * kt + g < K) row[4 * kt + g] = sk[kt];
        }
    }
}

// ------------------------------------------------------------------ einsum layer, forward, K from 13 to 16, large launches
// Small items are bound by the chain of requests in front of their arithmetic, so many small workgroups per compute unit
// take them: four waves per (item, group of chunks), a chunk being 128 samples, 32 per wave.  The whole item's weights are
// split into LDS once (at most 24 KB); a lane loads the rows of its own samples straight from memory, so nothing but the
// weights is shared.  Same tiles as above with row m = 4 (k % 4) + i % 4: lane group kg holds output k = 4 q + kg of group
// q, its four accumulators four consecutive left entries, so a sum of Eq. 4 is complete in one lane.
// Against the short kernel below: see einsum_forward_kernel.  Registers must not spill: with
// 128 instead of 168 of them and 28 spilled every launch took 4 us longer.
struct FwdSmallLayout {
    using X = X6<2>;
    static constexpr int KP = X::KP, NT = X::NT;
    static constexpr int LDS_BYTES = NT * NT * X::BYTES;  // NT groups of four outputs x NT tiles
    static constexpr int NI = KP * KP * 2;                // octets of the weights
    static constexpr int NL = (NI + 255) / 256;
};

__global__ __launch_bounds__(256, 3) void k_einsum_forward_small(const int32_t* __restrict__ e_rec, const float* __restrict__ params,
                                                               float* __restrict__ A, double* __restrict__ Off,
                                                               float* __restrict__ amax, int item0, int ngrp, int cpg, int nsplit,
                                                               int B, int K, int kout) {
    using LY = FwdSmallLayout;
    using X = LY::X;
    constexpr int K8 = 2;
    constexpr int KP = LY::KP, NT = LY::NT, NL = LY::NL;
    extern __shared__ __attribute__((aligned(16))) char lds_c[];
    uint32x4* wl = reinterpret_cast<uint32x4*>(lds_c);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c16 = lane & 15, kg = lane >> 4;
    const int vb = xcd_contiguous_block();
    const int part = vb % nsplit, grp = (vb / nsplit) % ngrp, li = vb / (nsplit * ngrp);
    const int NG = (kout + 3) >> 2, q0 = part * NG / nsplit, q1 = (part + 1) * NG / nsplit;   // groups of four outputs
    const int ni = (q1 - q0) * 4 * KP * K8;           // octets of their weights
    const int32_t* rec = e_rec + li * EIN_REC_INTS;
    const int left = rec[0], right = rec[1], out = rec[2];
    const int nchunks = (B + 127) >> 7, c0 = grp * cpg, c1 = min(c0 + cpg, nchunks);
    const float* W = params + rec[3];

    floatx4 wv[NL][2];
#pragma unroll
    for (int x = 0; x < NL; ++x) {
        if (256 * x >= ni) break;
        const int f = min(tid + 256 * x, ni - 1);
        const int o = f % K8, i = (f / K8) % KP, k = 4 * q0 + f / (K8 * KP);
        const float* p = W + ((size_t)min(k, kout - 1) * K + min(i, K - 1)) * K;
        p += min(8 * o, K - 8);                       // (the last octet of a row starts at K - 8, as above)
        wv[x][0] = *reinterpret_cast<const floatx4u*>(p);
        wv[x][1] = *reinterpret_cast<const floatx4u*>(p + 4);
    }
    // rows of this lane's samples (two sets of 16): one octet of R, all of L
    float rr[2][8], rl[2][KP];
    double off_children[2];
    auto fetch_rows = [&](int chunk) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int b = min(chunk * 128 + 32 * wave + 16 * s + c16, B - 1);
            const float* Lp = A + ((size_t)left * B + b) * K;
            const float* Rp = A + ((size_t)right * B + b) * K;
            const int st = (kg & 1) ? K - 8 : 0;
            const floatx4 r0 = *reinterpret_cast<const floatx4u*>(Rp + st), r1 = *reinterpret_cast<const floatx4u*>(Rp + st + 4);
            const floatx4 l0 = *reinterpret_cast<const floatx4u*>(Lp), l1 = *reinterpret_cast<const floatx4u*>(Lp + 4);
            // (the left entries of the tiles 2 and 3 are the row's last eight, those below 8 among them: their weights
            // are zeros there)
            const floatx4 l2 = *reinterpret_cast<const floatx4u*>(Lp + K - 8), l3 = *reinterpret_cast<const floatx4u*>(Lp + K - 4);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                rr[s][c] = r0[c]; rr[s][4 + c] = r1[c];
                rl[s][c] = l0[c]; rl[s][4 + c] = l1[c]; rl[s][8 + c] = l2[c]; rl[s][12 + c] = l3[c];
            }
            off_children[s] = Off[(size_t)left * B + b] + Off[(size_t)right * B + b];
        }
    };
    fetch_rows(c0);
#pragma unroll
    for (int x = 0; x < NL; ++x) {
        const int f = tid + 256 * x;
        const int o = f % K8, i = (f / K8) % KP, kl = f / (K8 * KP), k = 4 * q0 + kl;
        if (f < ni) {
            float v[8];
            const bool row = k < kout && i < K;
#pragma unroll
            for (int c = 0; c < 8; ++c) v[c] = row && (o == 0 || c >= 16 - K) ? wv[x][c >> 2][c & 3] * X6_SCALE : 0.f;
            uint32x4 part[3];
            split_octet(v, part[0], part[1], part[2]);
            // row slot of the tiles: left entry i < 8 in slot i, i >= 8 in slot 8 + (i - (K - 8)); the slots in between have
            // no left entry of their own and get the zeros of the rows i >= K
            const int slot = i < 8 ? i : i < K ? i + 16 - K : 8 + i - K;
            uint32x4* d = wl + ((kl >> 2) * NT + (slot >> 2)) * X::UNITS;
#pragma unroll
            for (int p = 0; p < 3; ++p) d[x6_unit<K8>(p, o, 4 * (kl & 3) + (slot & 3))] = part[p];
        }
    }
    int unit[X::NR];
#pragma unroll
    for (int a = 0; a < X::NR; ++a) unit[a] = x6_row_unit<K8>(a, kg, c16);
    __syncthreads();
    for (int chunk = c0; chunk < c1; ++chunk) {
        if (chunk > c0) fetch_rows(chunk);            // (the other workgroups of the compute unit hide the wait)
        uint32x4 er[2][X::NR];
        float el[2][KP];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            float xr = rr[s][0], xl = rl[s][0];
#pragma unroll
            for (int c = 1; c < 8; ++c) xr = fmaxf(xr, rr[s][c]);
            xr = fmaxf(xr, __shfl_xor(xr, 16, 64));
#pragma unroll
            for (int c = 1; c < KP; ++c) xl = fmaxf(xl, rl[s][c]);
            if (xr == -INFINITY) xr = 0.f;            // an all-zero input vector: exp(-inf) = 0, no NaN
            if (xl == -INFINITY) xl = 0.f;
            float e8[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) e8[c] = __expf(rr[s][c] - xr) * X6_SCALE;
            x6_sample_operand<K8>(kg, [&](int, float* v) {
#pragma unroll
                for (int c = 0; c < 8; ++c) v[c] = e8[c];
            }, er[s]);
#pragma unroll
            for (int c = 0; c < KP; ++c) el[s][c] = __expf(rl[s][c] - xl);
            const int b = chunk * 128 + 32 * wave + 16 * s + c16;
            if (kg == 0 && b < B && part == 0) {
                Off[(size_t)out * B + b] = off_children[s] + (double)xl + (double)xr;
                amax[((size_t)(item0 + li) * 2) * B + b] = xl;
                amax[((size_t)(item0 + li) * 2 + 1) * B + b] = xr;
            }
        }
#pragma unroll
        for (int ql = 0; ql < NT; ++ql) {
            if (q0 + ql >= q1) break;
            float sk[2] = {0.f, 0.f};
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                uint32x4 a[X::NR];
#pragma unroll
                for (int z = 0; z < X::NR; ++z) a[z] = wl[(ql * NT + t) * X::UNITS + unit[z]];
                floatx4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
                x6_tile<K8, 2>(a, er, acc);
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int c = 0; c < 4; ++c) sk[s] = fmaf(acc[s][c], el[s][4 * t + c], sk[s]);
            }
            const int k = 4 * (q0 + ql) + kg;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int b = chunk * 128 + 32 * wave + 16 * s + c16;
                if (b < B && k < kout) A[((size_t)out * B + b) * K + k] = __logf(sk[s] * X6_UNSCALE);
            }
        }
    }
}

// ------------------------------------------------------------------ einsum layer, forward, K from 17 to 31, short launches
// A launch with about one unit per compute unit is the chain of requests in front of its arithmetic; the persistent
// kernel's producer waves and barriers only lengthen it.  Here a workgroup of four waves takes one (item, chunk of 128
// samples, four outputs), every lane loads the rows of its own samples, and only the W slice goes through LDS.  The tiles
// and the lane layout are those of the persistent kernel.
// K = 30, 160 / 80 / 40 items, 100 samples: 9.8 / 7.8 / 6.0 us; the float32 kernel took 15.8 / 11.3 / 8.6 us.
template <int K8>
__global__ __launch_bounds__(256, 2) void k_einsum_forward_direct(const int32_t* __restrict__ e_rec, const float* __restrict__ params,
                                                                float* __restrict__ A, double* __restrict__ Off,
                                                                float* __restrict__ amax, int item0, int nchunks, int B, int K,
                                                                int kout) {
    using X = X6<K8>;
    constexpr int KP = X::KP, NT = X::NT, NI = 4 * KP * K8, NL = (NI + 255) / 256, NO = X::NQ + X::R2 + X::R1;
    __shared__ __attribute__((aligned(16))) uint32x4 wl[NT * X::UNITS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c16 = lane & 15, kg = lane >> 4;
    const int NG = (kout + 3) >> 2;
    const int vb = xcd_contiguous_block();
    const int g = vb % NG, chunk = (vb / NG) % nchunks, li = vb / (NG * nchunks);
    const int32_t* rec = e_rec + li * EIN_REC_INTS;
    const int left = rec[0], right = rec[1], out = rec[2];
    const float* W = params + rec[3] + (size_t)g * 4 * K * K;
    // the octets of R that this lane's operand needs, the left entries 4 t + kg, of its two samples
    float rr[2][NO][8], rl[2][NT];
    double off_children[2];
    auto oct_of = [&](int z) { return z < X::NQ ? 4 * z + kg : X::R2 && z == X::NQ ? 4 * X::NQ + (kg & 1) : K8 - 1; };
    auto start_of = [&](int o) { return min(8 * o, K - 8); };
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int b = min(chunk * 128 + 32 * wave + 16 * s + c16, B - 1);
        const float* Lp = A + ((size_t)left * B + b) * K;
        const float* Rp = A + ((size_t)right * B + b) * K;
#pragma unroll
        for (int z = 0; z < NO; ++z) {
            const int st = start_of(oct_of(z));
            const floatx4 r0 = *reinterpret_cast<const floatx4u*>(Rp + st), r1 = *reinterpret_cast<const floatx4u*>(Rp + st + 4);
#pragma unroll
            for (int c = 0; c < 4; ++c) { rr[s][z][c] = r0[c]; rr[s][z][4 + c] = r1[c]; }
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) rl[s][t] = Lp[min(4 * t + kg, K - 1)];
        off_children[s] = Off[(size_t)left * B + b] + Off[(size_t)right * B + b];
    }
    floatx4 wv[NL][2];
#pragma unroll
    for (int x = 0; x < NL; ++x) {
        const int f = min(tid + 256 * x, NI - 1);
        const int o = f % K8, i = (f / K8) % KP, kl = f / (K8 * KP);
        const float* p = W + ((size_t)min(kl, kout - 1 - 4 * g) * K + min(i, K - 1)) * K + start_of(o);
        wv[x][0] = *reinterpret_cast<const floatx4u*>(p);
        wv[x][1] = *reinterpret_cast<const floatx4u*>(p + 4);
    }
    // (entries that do not exist, and those that the octet before holds already, are zeros)
#pragma unroll
    for (int x = 0; x < NL; ++x) {
        const int f = min(tid + 256 * x, NI - 1);
        const int o = f % K8, i = (f / K8) % KP, kl = f / (K8 * KP);
        const int first = i < K && 4 * g + kl < kout ? 8 * o - start_of(o) : 8;
        float v[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) v[c] = c >= first ? wv[x][c >> 2][c & 3] * X6_SCALE : 0.f;
        uint32x4 part[3];
        split_octet(v, part[0], part[1], part[2]);
#pragma unroll
        for (int p = 0; p < 3; ++p) wl[(i >> 2) * X::UNITS + x6_unit<K8>(p, o, 4 * (i & 3) + kl)] = part[p];
    }
    uint32x4 er[2][X::NR];
    float el[2][NT];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        float xr = -INFINITY, xl = -INFINITY;
#pragma unroll
        for (int z = 0; z < NO; ++z)
#pragma unroll
            for (int c = 0; c < 8; ++c) xr = fmaxf(xr, rr[s][z][c]);
#pragma unroll
        for (int t = 0; t < NT; ++t) xl = fmaxf(xl, rl[s][t]);
        xr = fmaxf(xr, __shfl_xor(xr, 16, 64));
        xl = fmaxf(xl, __shfl_xor(xl, 16, 64));
        xr = fmaxf(xr, __shfl_xor(xr, 32, 64));
        xl = fmaxf(xl, __shfl_xor(xl, 32, 64));
        if (xr == -INFINITY) xr = 0.f;                // an all-zero input vector: exp(-inf) = 0, no NaN
        if (xl == -INFINITY) xl = 0.f;
        int z = 0;
        x6_sample_operand<K8>(kg, [&](int, float* v) {          // (called for the octets in the order of oct_of)
#pragma unroll
            for (int c = 0; c < 8; ++c) v[c] = __expf(rr[s][z][c] - xr) * X6_SCALE;
            ++z;
        }, er[s]);
#pragma unroll
        for (int t = 0; t < NT; ++t) el[s][t] = __expf(rl[s][t] - xl);
        const int b = chunk * 128 + 32 * wave + 16 * s + c16;
        if (kg == 0 && b < B && g == 0) {
            Off[(size_t)out * B + b] = off_children[s] + (double)xl + (double)xr;
            amax[((size_t)(item0 + li) * 2) * B + b] = xl;
            amax[((size_t)(item0 + li) * 2 + 1) * B + b] = xr;
        }
    }
    int unit[X::NR];
#pragma unroll
    for (int a = 0; a < X::NR; ++a) unit[a] = x6_row_unit<K8>(a, kg, c16);
    __syncthreads();
    floatx4 sk[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        uint32x4 a[X::NR];
#pragma unroll
        for (int z = 0; z < X::NR; ++z) a[z] = wl[t * X::UNITS + unit[z]];
        floatx4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
        x6_tile<K8, 2>(a, er, acc);
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int c = 0; c < 4; ++c) sk[s][c] = fmaf(acc[s][c], el[s][t], sk[s][c]);
    }
    // the lane groups' shares: afterwards every lane holds the four sums of its sample, lane group kg stores output kg
#pragma unroll
    for (int s = 0; s < 2; ++s) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            sk[s][c] += __shfl_xor(sk[s][c], 16, 64);
            sk[s][c] += __shfl_xor(sk[s][c], 32, 64);
        }
        const float mine = kg == 0 ? sk[s][0] : kg == 1 ? sk[s][1] : kg == 2 ? sk[s][2] : sk[s][3];
        const int b = chunk * 128 + 32 * wave + 16 * s + c16, k = 4 * g + kg;
        if (b < B && k < kout) A[((size_t)out * B + b) * K + k] = __logf(mine * X6_UNSCALE);
    }
}

// ------------------------------------------------------------------ mixing layer, forward (App. B)
// Offset of the output: the largest offset of the children (their residuals are at most 0, so no term
// exceeds its weight); residual: log sum_c v[c] exp((Off[c] - Off[out]) + A[c]).
constexpr int MIX_UNROLL = MIX_REC_CHILDREN;
__global__ void k_mixing_forward(const int32_t* __restrict__ m_rec, const float* __restrict__ params,
                                 float* __restrict__ A, double* __restrict__ Off, float* __restrict__ logp, int B,
                                 int K) {
    // the item's record: node, entries, weight offset, number of partitions, partition nodes
    const int32_t* rec = m_rec + (size_t)blockIdx.x * MIX_REC_INTS;
    const int node = rec[0], kout = rec[1], nc = rec[3];
    int child[MIX_UNROLL];
#pragma unroll
    for (int c = 0; c < MIX_UNROLL; ++c) child[c] = rec[4 + c];
    const int e = blockIdx.y * blockDim.x + threadIdx.x;
    if (e >= B * kout) return;
    const int b = e / kout, k = e - b * kout;
    const float* v = params + rec[2] + (size_t)k * nc;
    double m = -INFINITY;
    float s = 0.f;
    {
        // offsets, residuals and weights of all children are requested together: one memory latency, not two
        double off[MIX_UNROLL];
        float a[MIX_UNROLL], w[MIX_UNROLL];
#pragma unroll
        for (int c = 0; c < MIX_UNROLL; ++c) {
            off[c] = 0.0;
            a[c] = w[c] = 0.f;
            if (c < nc) {
                const size_t row = (size_t)child[c] * B + b;
                off[c] = Off[row];
                a[c] = A[row * K + k];
                w[c] = v[c];
            }
        }
#pragma unroll
        for (int c = 0; c < MIX_UNROLL; ++c)
            if (c < nc) m = fmax(m, off[c]);
#pragma unroll
        for (int c = 0; c < MIX_UNROLL; ++c)
            if (c < nc) s += w[c] * expf((float)(off[c] - m) + a[c]);
    }
    const float res = logf(s);
    const size_t row = (size_t)node * B + b;
    A[row * K + k] = res;
    if (k == 0) {
        Off[row] = m;
        if (logp && node == 0) logp[b] = (float)(m + (double)res);   // node 0: the root region, one entry
    }
}

// The same for regions with many partitions (the root over R replicas of random binary trees): one wave per
// output element, the children spread over the lanes, maximum and sum by wave reductions.
__global__ __launch_bounds__(256) void k_mixing_forward_many(
    const int32_t* __restrict__ m_node, const int32_t* __restrict__ m_kout, const int32_t* __restrict__ m_cptr,
    const int32_t* __restrict__ m_child, const int32_t* __restrict__ m_voff, const float* __restrict__ params,
    float* __restrict__ A, double* __restrict__ Off, float* __restrict__ logp, int B, int K) {
    const int item = blockIdx.x;
    const int kout = m_kout[item];
    const int lane = threadIdx.x & 63;
    const int e = blockIdx.y * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (e >= B * kout) return;                       // whole waves leave
    const int b = e / kout, k = e - b * kout;
    const int c0 = m_cptr[item], nc = m_cptr[item + 1] - c0;
    const float* v = params + m_voff[item] + (size_t)k * nc;
    double m = -INFINITY;
    for (int c = lane; c < nc; c += 64) m = fmax(m, Off[(size_t)m_child[c0 + c] * B + b]);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
    float s = 0.f;
    for (int c = lane; c < nc; c += 64) {
        const size_t row = (size_t)m_child[c0 + c] * B + b;
        s += v[c] * expf((float)(Off[row] - m) + A[row * K + k]);
    }
    s = wave_sum(s);
    if (lane == 0) {
        const float res = logf(s);
        const size_t row = (size_t)m_node[item] * B + b;
        A[row * K + k] = res;
        if (k == 0) {
            Off[row] = m;
            if (logp && m_node[item] == 0) logp[b] = (float)(m + (double)res);
        }
    }
}

}  // namespace

template <int KQ>
static void launch_einsum_forward_kq(const DevTables& t, int first, int count, const float* params, float* A,
                                     double* Off, float* amax, float* logp, const Dims& d, hipStream_t s) {
    const int nkt = (d.K + 3) / 4;
    const int n_btiles = (d.B + 15) / 16;
    const int nw_max = count * nkt >= 1024 ? 4 : 8;    // many small workgroups: more of them per compute unit
    const int nw = n_btiles < nw_max ? n_btiles : nw_max;
    const size_t lds = sizeof(float) * FwdLayout<KQ>::LDS_FLOATS;
    if (lds > 64 * 1024) {
        static std::once_flag attr_set[EINET_MAX_DEVICES];
        int dev = 0;
        (void)hipGetDevice(&dev);
        std::call_once(attr_set[dev % EINET_MAX_DEVICES], [&] { allow_dynamic_lds(&k_einsum_forward<KQ>, lds); });
    }
    hipLaunchKernelGGL(k_einsum_forward<KQ>, dim3(count * nkt), dim3(64 * nw), lds, s, t.ein_left + first,
                       t.ein_right + first, t.ein_out + first, t.ein_kout + first, t.ein_woff + first, params, A, Off,
                       amax, logp, first, d.B, d.K, nkt);
}

template <int K8>
static void launch_einsum_forward_s(const DevTables& t, int first, int count, const float* params, float* A,
                                     double* Off, float* amax, const Dims& d, hipStream_t s) {
    using LY = FwdSLayout<K8>;
    const size_t lds = sizeof(float) * LY::LDS_FLOATS;
    static std::once_flag attr_set[EINET_MAX_DEVICES];
    int dev = 0;
    (void)hipGetDevice(&dev);
    std::call_once(attr_set[dev % EINET_MAX_DEVICES], [&] { allow_dynamic_lds(&k_einsum_forward_s<K8>, lds); });
    const int units = count * ((d.B + 127) / 128) * (LY::K / 4);
    hipLaunchKernelGGL(k_einsum_forward_s<K8>, dim3(units < EINET_NUM_CUS ? units : EINET_NUM_CUS), dim3(512), lds, s,
                       t.ein_left + first, t.ein_right + first, t.ein_out + first, t.ein_woff + first, params, A, Off,
                       amax, first, count, d.B);
}

template <int K8>
static void launch_einsum_forward_x(const DevTables& t, int first, int count, int kout, const float* params, float* A,
                                    double* Off, float* amax, const Dims& d, hipStream_t s) {
    const size_t lds = FwdXLayout<K8>::LDS_BYTES;
    static std::once_flag attr_set[EINET_MAX_DEVICES];
    int dev = 0;
    (void)hipGetDevice(&dev);
    std::call_once(attr_set[dev % EINET_MAX_DEVICES], [&] {
        allow_dynamic_lds(&k_einsum_forward_x<K8, true>, lds);
        allow_dynamic_lds(&k_einsum_forward_x<K8, false>, lds);
    });
    const int nchunks = (d.B + 127) / 128, units = count * nchunks * ((kout + 3) / 4);
    const dim3 grid(units < EINET_NUM_CUS ? units : EINET_NUM_CUS);
    const int32_t* rec = t.ein_rec + (size_t)first * EIN_REC_INTS;
    if (d.K == 8 * K8 && kout == d.K) {
        hipLaunchKernelGGL((k_einsum_forward_x<K8, true>), grid, dim3(512), lds, s, rec, params, A, Off, amax, first, count,
                           d.B, d.K, kout);
        return;
    }
    hipLaunchKernelGGL((k_einsum_forward_x<K8, false>), grid, dim3(512), lds, s, rec, params, A, Off, amax, first, count, d.B,
                       d.K, kout);
}

template <int K8>
static void launch_einsum_forward_direct(const DevTables& t, int first, int count, int kout, const float* params, float* A,
                                         double* Off, float* amax, const Dims& d, hipStream_t s) {
    const int nchunks = (d.B + 127) / 128;
    hipLaunchKernelGGL(k_einsum_forward_direct<K8>, dim3(count * nchunks * ((kout + 3) / 4)), dim3(256), 0, s,
                       t.ein_rec + (size_t)first * EIN_REC_INTS, params, A, Off, amax, first, nchunks, d.B, d.K, kout);
}

template <int KQ>
static void launch_einsum_forward_compact(const DevTables& t, int first, int count, const float* params, float* A, double* Off,
                                          float* amax, const Dims& d, hipStream_t s) {
    // chunks of an item share its weights as long as eight workgroups per compute unit remain
    const int nchunks = (d.B + 63) / 64, want = (8 * EINET_NUM_CUS + count - 1) / count;
    const int cpg = (nchunks + want - 1) / want, ngrp = (nchunks + cpg - 1) / cpg;
    // few items: the groups of four outputs of an item side by side
    int nsplit = EINET_NUM_CUS / (count * ngrp);
    nsplit = nsplit < 1 ? 1 : nsplit > KQ ? KQ : nsplit;
    const int32_t* rec = t.ein_rec + (size_t)first * EIN_REC_INTS;
    if (KQ > 4 || d.K == 4 * KQ)
        hipLaunchKernelGGL((k_einsum_forward_compact<KQ, true>), dim3(count * ngrp * nsplit), dim3(256), 0, s, rec, params, A,
                           Off, amax, first, ngrp, cpg, nsplit, d.B, d.K);
    else if constexpr (KQ <= 4)                           // (17 to 19 entries take other kernels)
        hipLaunchKernelGGL((k_einsum_forward_compact<KQ, false>), dim3(count * ngrp * nsplit), dim3(256), 0, s, rec, params, A,
                           Off, amax, first, ngrp, cpg, nsplit, d.B, d.K);
}

static void launch_einsum_forward_small(const DevTables& t, int first, int count, int kout, const float* params, float* A,
                                        double* Off, float* amax, const Dims& d, hipStream_t s) {
    // chunks of an item share its weights as long as four workgroups per compute unit remain
    const int nchunks = (d.B + 127) / 128, want = (4 * EINET_NUM_CUS + count - 1) / count;
    const int cpg = (nchunks + want - 1) / want, ngrp = (nchunks + cpg - 1) / cpg;
    // few items: the groups of four outputs of an item side by side
    const int groups = (kout + 3) / 4;
    int nsplit = 2 * EINET_NUM_CUS / (count * ngrp);
    nsplit = nsplit < 1 ? 1 : nsplit > groups ? groups : nsplit;
    hipLaunchKernelGGL(k_einsum_forward_small, dim3(count * ngrp * nsplit), dim3(256), FwdSmallLayout::LDS_BYTES, s,
                       t.ein_rec + (size_t)first * EIN_REC_INTS, params, A, Off, amax, first, ngrp, cpg, nsplit, d.B, d.K, kout);
}

// Which kernel a layer takes.  Microseconds of a log-density of a tree of depth 2 (leaf layer, one layer of `count` items,
// root: about 8 us besides the layer for few items, 2 to 3 times the layer's for many), measured for K 8 to 48, 2 to 1280
// items, 1 to 1000 samples.  PLAIN: the float32 kernel with a workgroup per (item, four outputs), which has no operands to
// split and walks the chunks of 128 samples one after the other.  WAVES: the float32 kernel with specialised waves.  COMPACT:
// the short float32 kernel for whole items.
enum FwdKernel { FWD_PLAIN, FWD_WAVES, FWD_COMPACT, FWD_SMALL, FWD_DIRECT, FWD_X };
static FwdKernel einsum_forward_kernel(int count, int kout, const Dims& d) {
    const int K = d.K, B = d.B;
    const bool quads = (K & 3) == 0;                  // rows of 16-byte groups
    const int64_t units = (int64_t)count * ((B + 127) / 128) * ((kout + 3) / 4);
    // (one output per item would leave three of four rows of COMPACT's tiles empty; only items below the root have one)
    // from 13 entries on and with many workgroups the split operands pay: log-density of a tree of 512 items, K = 13, 1000 samples:
    // 112 with COMPACT, 90 with SMALL; K = 16, 103 and 95, 300 samples 57 and 59; K = 10: 84 and 85
    // (rows that are not whole pieces: beyond 64 samples for smaller launches too.  K = 14, 300 samples, 112 / 496 items: 43 and 40, 59
    // and 55)
    if (K > 12 && K <= 16 && kout == K && units >= (quads ? 8192 : B > 64 ? 256 : 1024)) return FWD_SMALL;
    // K = 20 (log-density, 1 / 100 / 1000 samples; COMPACT and the choice below): 194 items 48 / 54 / 109 and 52 / 57 / 129, 512 items
    // 38 / 49 / 148 and 42 / 54 / 190.  Rows of 17 to 19 entries are not whole pieces: 194 items, 18 entries, 200 samples 68 and 63
    // (24 and 28 entries are whole pieces too; their weights take 48 and 63 KB of LDS instead of 33, and they were not measured)
    if (K <= 16 || K == 20) return kout == K ? FWD_COMPACT : FWD_PLAIN;
    // K = 48, 2 items, 1000 samples: plain 63, waves 19; 320 items, 16 samples: 171, 148; 64 samples: 155, 157
    if (K == 48 && kout == K) return B > 32 && B <= 64 ? FWD_PLAIN : FWD_WAVES;
    if (K > 40) return FWD_PLAIN;
    if (K <= 20) {
        // three octets for 17 to 19 entries: the split pays for few items only.  K = 18, 20 items, 16 samples: plain 18.3, direct
        // 16.0; 500 samples 27.6, 23.1; 80 items, 1000 samples: 63.4, persistent 60.5; 1280 items, 1000 samples: 637, 723
        if (units <= 1024 && (count < 64 || B <= 16)) return FWD_DIRECT;
        return count <= 128 && B > 512 ? FWD_X : FWD_PLAIN;
    }
    // K = 24, 20 items: 16 samples plain 15.5, direct 15.3, persistent 15.4, waves 15.0; 64 samples 15.6, 16.7, 16.2, 15.8;
    // 256 samples 21.4, 20.1, 19.2, 18.7; 320 items: 64 samples 79.1, 87.3, 80.4, 81.8; 256 samples 101, 105, 90, 92
    if (K == 24 && B <= 128) return count < 64 && B <= 16 ? FWD_DIRECT : B <= 64 || count <= 128 ? FWD_PLAIN : FWD_X;
    if (K == 24 && count < 64 && kout == K) return FWD_WAVES;
    // K = 28, 80 items: 16 samples plain 25.2, direct 26.4; 48 samples 29.8, 29.5; 320 items, 16 samples: 83.8, 82.8
    if ((K == 28 || K == 32) && B <= 32 && count >= 64 && count <= 160) return FWD_PLAIN;
    // K = 36, 20 items: 16 samples plain 19.6, persistent 18.9; 64 samples 18.5, 19.8; 80 items: 34.4, 38.2; 96 samples 42.9,
    // 41.9
    if (K == 36 && (count < 64 ? B > 16 && B <= 128 : count <= 160 && B <= 64)) return FWD_PLAIN;
    // K = 30, 80 items, 100 samples (640 units): direct 36.1, persistent 37.4; 320 items, 500 samples (10240): 165, 167;
    // K = 21, 320 items, 1000 samples: 205, 190.  With K a multiple of 8 or above 32 the persistent one is always faster.
    return K <= 32 && (K & 7) != 0 && units <= 4 * EINET_NUM_CUS ? FWD_DIRECT : FWD_X;
}

void launch_einsum_forward(const DevTables& t, int first, int count, bool full_k, const float* params, float* A,
                           double* Off, float* amax, float* logp, const Dims& d, hipStream_t s) {
    const int kout = full_k ? d.K : 1, K8 = (d.K + 7) / 8;
    // (only the plain kernel writes logp: an item that writes the root's own node is the root's only partition, which
    // k_root_forward takes)
    switch (einsum_forward_kernel(count, kout, d)) {
    case FWD_SMALL: launch_einsum_forward_small(t, first, count, kout, params, A, Off, amax, d, s); return;
    case FWD_COMPACT:
#define EINET_CASE(J) case J: launch_einsum_forward_compact<J>(t, first, count, params, A, Off, amax, d, s); return;
        switch ((d.K + 3) / 4) { EINET_CASE(1) EINET_CASE(2) EINET_CASE(3) EINET_CASE(4) EINET_CASE(5) }
        return;
#undef EINET_CASE
#define EINET_CASE(J, F) case J: F<J>(t, first, count, kout, params, A, Off, amax, d, s); return;
    case FWD_DIRECT:
        switch (K8) { EINET_CASE(3, launch_einsum_forward_direct) EINET_CASE(4, launch_einsum_forward_direct) }
        return;
    case FWD_X:
        switch (K8) {
            EINET_CASE(3, launch_einsum_forward_x) EINET_CASE(4, launch_einsum_forward_x) EINET_CASE(5, launch_einsum_forward_x)
        }
        return;
#undef EINET_CASE
    case FWD_WAVES:
#define EINET_CASE(J) case J: launch_einsum_forward_s<J>(t, first, count, params, A, Off, amax, d, s); return;
        switch (K8) { EINET_CASE(3) EINET_CASE(6) }
        return;
#undef EINET_CASE
    case FWD_PLAIN:
        break;
    }
    switch ((d.K + 3) / 4) {
#define EINET_CASE(J) \
    case J: launch_einsum_forward_kq<J>(t, first, count, params, A, Off, amax, logp, d, s); break;
        EINET_CASE(1) EINET_CASE(2) EINET_CASE(3) EINET_CASE(4) EINET_CASE(5) EINET_CASE(6) EINET_CASE(7) EINET_CASE(8)
        EINET_CASE(9) EINET_CASE(11) EINET_CASE(12) EINET_CASE(13) EINET_CASE(14) EINET_CASE(15) EINET_CASE(16)
#undef EINET_CASE
    }
}

void launch_mixing_forward(const DevTables& t, int first, int count, int max_children, const float* params, float* A,
                           double* Off, float* logp, const Dims& d, hipStream_t s) {
    if (count == 0) return;
    if (max_children >= 8) {                         // a wave per output element, children over the lanes
        dim3 grid(count, (d.B * d.K + 3) / 4);
        hipLaunchKernelGGL(k_mixing_forward_many, grid, dim3(256), 0, s, t.mix_node + first, t.mix_kout + first,
                           t.mix_cptr + first, t.mix_child, t.mix_voff + first, params, A, Off, logp, d.B, d.K);
        return;
    }
    dim3 grid(count, (d.B * d.K + 255) / 256);
    hipLaunchKernelGGL(k_mixing_forward, grid, dim3(256), 0, s, t.mix_rec + (size_t)first * MIX_REC_INTS, params, A,
                       Off, logp, d.B, d.K);
}

}  // namespace einet_impl
