// Shared by the HIP translation units: the data layout of the arenas and small device helpers.
//
// Activations live in a node-major arena A[node][b][k] (float32, log domain):
// every region and every simple sum owns one dense [B][K] block, so a layer's
// "gather" of left and right inputs (Sec. 3.3) is an index lookup.  A block does
// not hold the log-densities themselves but their residuals against one offset
// per (node, sample), Off[node][b] (float64):
//     log-density[node][b][k] = Off[node][b] + A[node][b][k].
// Leaves take their largest entry as offset; an einsum output takes the offsets of
// its children plus the two shifts of Eq. 4, so that its residual is log S~ in
// [log of the smallest weight, 0]; a mixing output takes the largest offset of its
// children.  Log-densities of large scopes have magnitudes of 1e3..1e5, where a
// float32 resolves 1e-4..1e-2; the residuals stay small, and the posteriors of the
// top-down pass (exponentials of differences) keep full float32 precision.  The
// posterior arena G has the same shape; Gp holds what einsum item e sends down:
// blocks e*nb .. e*nb+nb-1 ([b][k] each, nb = 1 + ceil(K/4)), the first for its
// left child, the others, one per workgroup of the item's top-down launch, shares
// for its right child.  A child sums the blocks of its parents when it is
// processed: no atomics anywhere.
#ifndef EINET_DEVICE_COMMON_HPP
#define EINET_DEVICE_COMMON_HPP

#include "kernels.hpp"

#include <cmath>

namespace einet_impl {

typedef float floatx4 __attribute__((ext_vector_type(4)));
// four consecutive floats at any multiple of four bytes (the hardware's 16-byte loads need no more)
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));

constexpr int EINET_NUM_CUS = 256;        // compute units of an MI355X: workgroups of a one-per-unit launch
constexpr int EINET_MAX_DEVICES = 16;     // per-device once-flags of the launchers

// Raises the dynamic-LDS limit of a kernel.  A refusal is not kept as the thread's last error: the launch
// that needs the memory then fails and reports it, instead of a later, unrelated call.
template <class Kernel>
inline void allow_dynamic_lds(Kernel kernel, size_t bytes) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)bytes) != hipSuccess)
        (void)hipGetLastError();
}

// Workgroups of a launch are handed to the 8 XCDs round-robin by blockIdx.x, and every XCD has an L2 of its own.
// This renumbering gives each XCD a contiguous range of work items, so that neighbouring items (the workgroups
// of one partition, which read the same child rows) meet in one L2.  It is a bijection on [0, gridDim.x).
__device__ __forceinline__ int xcd_contiguous_block() {
    const int n = gridDim.x, x = blockIdx.x & 7, q = n >> 3, r = n & 7;
    return x * q + min(x, r) + (blockIdx.x >> 3);
}

// Four registers of four lane groups transposed: register r of group g becomes register g of group r.
__device__ __forceinline__ void transpose_groups(float (&r)[4]) {
    auto swap32 = [](float& a, float& b) {
        const auto v = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b), false, false);
        const uint32_t v0 = v[0], v1 = v[1];
        a = __builtin_bit_cast(float, v0);
        b = __builtin_bit_cast(float, v1);
    };
    auto swap16 = [](float& a, float& b) {
        const auto v = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b), false, false);
        const uint32_t v0 = v[0], v1 = v[1];
        a = __builtin_bit_cast(float, v0);
        b = __builtin_bit_cast(float, v1);
    };
    swap32(r[0], r[2]);
    swap32(r[1], r[3]);
    swap16(r[0], r[1]);
    swap16(r[2], r[3]);
}

// Entries 4 p .. 4 p + 3 of a row of K entries, p < KQ = ceil(K / 4) (those beyond K hold anything).  QUADS: K is 4 KQ.
// Otherwise a row's last piece starts at K - 4 and is shifted into place (K below 4: entry by entry).
template <int KQ, bool QUADS>
__device__ __forceinline__ void load_piece(const float* row, int p, int K, float (&v)[4]) {
    if constexpr (QUADS) {
        const float4 f = *reinterpret_cast<const float4*>(row + 4 * p);
        v[0] = f.x, v[1] = f.y, v[2] = f.z, v[3] = f.w;
    } else if constexpr (KQ == 1) {
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = row[min(c, K - 1)];
    } else {
        const int start = min(4 * p, K - 4), d = 4 * p - start;
        const floatx4 f = *reinterpret_cast<const floatx4u*>(row + start);
        const float a0 = (d & 2) ? f[2] : f[0], a1 = (d & 2) ? f[3] : f[1], a2 = f[2], a3 = f[3];
        v[0] = (d & 1) ? a1 : a0;
        v[1] = (d & 1) ? a2 : a1;                         // (d = 3 leaves one entry, d = 2 two, d = 1 three)
        v[2] = (d & 1) ? a3 : a2;
        v[3] = a3;
    }
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Two float32 numbers as the exact sums of three bfloat16 numbers each: hi = the number rounded to bfloat16, mid = the
// rest rounded, lo = the rest of the rest (8 + 8 + 8 mantissa bits hold the 24 of a float32; rests below the smallest
// float32 exponents are lost).  The pairs come packed, a in the low half.
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, bf16x2{(__bf16)a, (__bf16)b});
}
__device__ __forceinline__ float bf16_low(uint32_t p) { return __builtin_bit_cast(float, p << 16); }
__device__ __forceinline__ float bf16_high(uint32_t p) { return __builtin_bit_cast(float, p & 0xffff0000u); }
__device__ __forceinline__ void split_bf16x3(float a, float b, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
    // (the packed pair is made opaque: the compiler would convert each half again, alone, to subtract it, and a conversion
    // takes twice as long as a shift or mask)
    hi = pack_bf16(a, b);
    asm("" : "+v"(hi));
    a -= bf16_low(hi);
    b -= bf16_high(hi);
    mid = pack_bf16(a, b);
    asm("" : "+v"(mid));
    a -= bf16_low(mid);
    b -= bf16_high(mid);
    lo = pack_bf16(a, b);
}

}  // namespace einet_impl

#endif
