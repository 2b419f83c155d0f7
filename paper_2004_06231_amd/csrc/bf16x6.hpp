// Products of float32 matrices on the bfloat16 matrix pipe at float32 precision.
//
// A float32 number is the exact sum of three bfloat16 numbers (split_bf16x3: 8 + 8 + 8 mantissa bits), so a product a b is
// the sum of nine products of bfloat16 numbers, each exact in float32.  The three smallest (mid lo, lo mid, lo lo) are left
// out: mid is at most 2^-8 of its number and lo 2^-17, so they are at most 2^-24 of the product, what one float32 product
// is rounded by, and 2^-27.5 in the root mean square over random pairs.  The other six are accumulated in float32 (the
// scheme of Henry, Tang and Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For Higher-Precision
// Computations", 2019).  Weights, exponentials and posteriors are non-negative, so their sums do not cancel and the error of a
// result is the error of its terms plus that of the float32 accumulation, as with float32 operands.  Values of Gaussian leaves
// may be negative; sums of them cancel as they do in float32, from terms that are as accurate.
// (A rest below 2^-133, the smallest bfloat16, is lost: numbers below 2^-109 would keep fewer bits.  Both operands, the
// exponentials and the weights, are therefore multiplied by the power of two X6_SCALE before they are split and the sums by
// X6_UNSCALE at the end: the smallest normal float32 becomes 2^-102, whose last bit is a normal bfloat16.  Sums stay below
// 2^48 for rows of weights that add up to 1.)
// v_mfma_f32_16x16x32_bf16 does 16 times as many multiply-adds per cycle as the float32 shapes: with six products 2.67 times.
//
// One tile: 16 rows x 16 columns (samples), contraction over KP = 8 K8 entries in octets.  An operand register holds one
// octet (8 bfloat16 numbers, 16 bytes) per lane, lane group kg = lane / 16 supplying octet kg of the four that the
// instruction contracts.  For every four octets (quad) the registers hi, mid, lo of the rows and of the samples make six
// instructions.  Two octets left over (R2) take three instructions with two products side by side, one octet left over
// (R1) two instructions with four and two products, so that K = 40 needs 8 instructions where 7.5 are the least.
#ifndef EINET_BF16X6_HPP
#define EINET_BF16X6_HPP

#include "device_common.hpp"

namespace einet_impl {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t uint32x4 __attribute__((ext_vector_type(4)));

constexpr float X6_SCALE = 0x1p+24f, X6_UNSCALE = 0x1p-48f;

template <int K8>
struct X6 {
    static constexpr int KP = 8 * K8;
    static constexpr int NQ = K8 / 4, R2 = (K8 >> 1) & 1, R1 = K8 & 1;
    static constexpr int NR = 3 * NQ + 3 * R2 + 2 * R1;   // operand registers (16 bytes per lane) of a tile, and of a sample
    static constexpr int NT = KP / 4;                     // tiles of 16 rows: four outer entries x four of the KP inner ones
    // LDS image of the rows of a tile: octet `oct` of part p (hi, mid, lo) of row m is the 16-byte unit
    // po * 16 + (m ^ (po & 3)), po = p * K8 + oct: a read of 16 rows takes 16 consecutive units in any order, and stores of
    // consecutive octets of a row go to different banks
    static constexpr int UNITS = 3 * K8 * 16;
    static constexpr int BYTES = UNITS * 16;
};

template <int K8>
__device__ __forceinline__ int x6_unit(int p, int oct, int m) {
    const int po = p * K8 + oct;
    return po * 16 + (m ^ (po & 3));
}

// unit that lane (row m = lane % 16, group kg) reads for operand register a of a tile
template <int K8>
__device__ __forceinline__ int x6_row_unit(int a, int kg, int m) {
    using X = X6<K8>;
    if (a < 3 * X::NQ) return x6_unit<K8>(a % 3, 4 * (a / 3) + kg, m);
    if (X::R2 && a < 3 * X::NQ + 3) {
        const int z = a - 3 * X::NQ;
        const int p = z == 0 ? 0 : z == 1 ? (kg < 2 ? 0 : 1) : (kg < 2 ? 1 : 2);
        return x6_unit<K8>(p, 4 * X::NQ + (kg & 1), m);
    }
    const int z = a - 3 * X::NQ - 3 * X::R2;
    const int p = z == 0 ? (kg < 3 ? 0 : 1) : (kg == 0 ? 1 : 2);
    return x6_unit<K8>(p, K8 - 1, m);
}

__device__ __forceinline__ void split_octet(const float* v, uint32x4& hi, uint32x4& mid, uint32x4& lo) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        uint32_t h, m, l;
        split_bf16x3(v[2 * q], v[2 * q + 1], h, m, l);
        hi[q] = h;
        mid[q] = m;
        lo[q] = l;
    }
}

// operand registers of a sample: lane (column, kg); octet(o, v) yields entries 8 o .. 8 o + 7 of the lane's sample
template <int K8, class F>
__device__ __forceinline__ void x6_sample_operand(int kg, F&& octet, uint32x4 (&b)[X6<K8>::NR]) {
    using X = X6<K8>;
#pragma unroll
    for (int q = 0; q < X::NQ; ++q) {
        float v[8];
        octet(4 * q + kg, v);
        split_octet(v, b[3 * q], b[3 * q + 1], b[3 * q + 2]);
    }
    if constexpr (X::R2) {
        float v[8];
        uint32x4 h, m, l;
        octet(4 * X::NQ + (kg & 1), v);
        split_octet(v, h, m, l);
        constexpr int o = 3 * X::NQ;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            b[o][c] = kg < 2 ? h[c] : m[c];
            b[o + 1][c] = kg < 2 ? l[c] : h[c];
            b[o + 2][c] = kg < 2 ? m[c] : h[c];
        }
    }
    if constexpr (X::R1) {
        float v[8];
        uint32x4 h, m, l;
        octet(K8 - 1, v);
        split_octet(v, h, m, l);
        constexpr int o = 3 * X::NQ + 3 * X::R2;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            b[o][c] = kg == 1 ? m[c] : kg == 2 ? l[c] : h[c];
            b[o + 1][c] = kg == 0 ? m[c] : kg == 1 ? h[c] : 0u;
        }
    }
}

__device__ __forceinline__ floatx4 mfma_bf16(uint32x4 a, uint32x4 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// acc[s] += rows x samples for NS sets of 16 samples (their chains of instructions alternate)
template <int K8, int NS>
__device__ __forceinline__ void x6_tile(const uint32x4 (&a)[X6<K8>::NR], const uint32x4 (&b)[NS][X6<K8>::NR], floatx4 (&acc)[NS]) {
    using X = X6<K8>;
    constexpr int PA[6] = {0, 0, 0, 1, 1, 2}, PB[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
    for (int q = 0; q < X::NQ; ++q)
#pragma unroll
        for (int p = 0; p < 6; ++p)
#pragma unroll
            for (int s = 0; s < NS; ++s) acc[s] = mfma_bf16(a[3 * q + PA[p]], b[s][3 * q + PB[p]], acc[s]);
#pragma unroll
    for (int z = 3 * X::NQ; z < X::NR; ++z)
#pragma unroll
        for (int s = 0; s < NS; ++s) acc[s] = mfma_bf16(a[z], b[s][z], acc[s]);
}

}  // namespace einet_impl

#endif
