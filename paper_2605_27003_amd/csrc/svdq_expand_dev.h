// Expansion of 4-bit weights into the operand form of the E3M2 GEMM: shared by the packing kernels and by the quantise
// pass, which does it beside its own work when a layer's weights stay resident in 4 bits.
#pragma once
#include "svdq_dev.h"
#include "svdq_kernels.h"
#include "svdq_lds.h"
#include "svdq_quant_dev.h"

namespace svdq {

// From the canonical form (qw [N][K/2] nibbles, sw [K/64][N] binary32).
// Region 1: bytes 0..15 of the weight fragments, [N/32][K/64][64 lanes][16 B]; region 2: bytes 16..23,
// [N/32][K/64][64 lanes][8 B]: lane (n = lane % 32, kh = lane / 32) holds the E3M2 fields of k = 64 g + 32 kh + 0..31
// of channel n, k ascending from bit 0.  Region 3: n-side operands of the scale-product MFMA,
// [N/32][K/64][32 channels][8 B]: bf16 {w1, w1, w2, w2} with w1 + w2 ~ sw[g][n] (the lanes of k half 0 read the
// entry; those of k half 1 read zeros).
// Runs before every GEMM whose weights stay resident in the canonical form, so it has to keep up with HBM: a lane turns
// 32 nibbles into 32 fields with the hardware conversions (e3m2_of_nibbles; bit arithmetic per field was 480 vector
// instructions and bound the kernel: 18.7 us for 5120 x 5120, 36 MB).  A wave takes four neighbouring groups of 32 channels: 128 bytes
// of every channel's row, all requested before the first conversion.
constexpr int PACK_GROUPS = 4;
inline size_t expand_waves(int N, int K) { return (size_t)(N / 32) * ((K / 64 + PACK_GROUPS - 1) / PACK_GROUPS); }
__device__ __forceinline__ void expand_canonical(const int id, const int lane, const uint8_t* __restrict__ qw, const float* __restrict__ sw,
                                                 const int N, const int K, uint8_t* __restrict__ out) {
    const int ng = K >> 6;
    const int l32 = lane & 31, kh = lane >> 5;
    const int gq = (ng + PACK_GROUPS - 1) / PACK_GROUPS;
    const int nb = id / gq, g0 = (id - nb * gq) * PACK_GROUPS;
    if (nb >= (N >> 5)) return;
    const int n = nb * 32 + l32;
    uint4* o1 = reinterpret_cast<uint4*>(out);
    uint2* o2 = reinterpret_cast<uint2*>(out + packed_e3m2_w0_bytes(N, K));
    uint2* o3 = reinterpret_cast<uint2*>(out + packed_e3m2_w0_bytes(N, K) + packed_e3m2_w1_bytes(N, K));
    uint4 nib[PACK_GROUPS];
    float sc[2];
#pragma unroll
    for (int i = 0; i < PACK_GROUPS; ++i) {
        const int g = min(g0 + i, ng - 1);
        nib[i] = *reinterpret_cast<const uint4*>(qw + (size_t)n * (K >> 1) + g * 32 + kh * 16);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)                       // scale pieces: half the lanes take even, half odd groups
        sc[i] = sw[(size_t)min(g0 + 2 * i + kh, ng - 1) * N + n];
#pragma unroll
    for (int i = 0; i < PACK_GROUPS; ++i) {
        if (g0 + i >= ng) break;
        const LaneCodes<true> c = e3m2_of_nibbles(nib[i]);
        const size_t v = ((size_t)nb * ng + g0 + i) * 64 + lane;
        o1[v] = c.lo;
        o2[v] = c.hi;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int g = g0 + 2 * i + kh;
        if (g >= ng) break;
        const uint32_t p = split_bf16(sc[i]);
        const uint32_t w1 = p & 0xffffu, w2 = p >> 16;
        o3[((size_t)nb * ng + g) * 32 + l32] = uint2{w1 | (w1 << 16), w2 | (w2 << 16)};
    }
}

// The same from the nibble kernel's packed weights (svdq_gemm.hip): its code fragments hold the same bytes per lane and
// its scale operands the same pieces, eight bytes in the lanes of k half 0.
__device__ __forceinline__ void expand_packed(const int id, const int lane, const uint4* __restrict__ frag, const uint2* __restrict__ sfrag,
                                              const int N, const int K, uint8_t* __restrict__ out) {
    const size_t last = (size_t)(N >> 5) * (K >> 6) - 1, f0 = (size_t)id * PACK_GROUPS;
    uint4 nib[PACK_GROUPS];
    uint2 sc[PACK_GROUPS];
#pragma unroll
    for (int i = 0; i < PACK_GROUPS; ++i) {
        const size_t v = (f0 + i < last ? f0 + i : last) * 64 + lane;
        nib[i] = frag[v];
        sc[i] = sfrag[v];
    }
#pragma unroll
    for (int i = 0; i < PACK_GROUPS; ++i) {
        if (f0 + i > last) break;
        const LaneCodes<true> c = e3m2_of_nibbles(nib[i]);
        const size_t v = (f0 + i) * 64 + lane;
        reinterpret_cast<uint4*>(out)[v] = c.lo;
        reinterpret_cast<uint2*>(out + packed_e3m2_w0_bytes(N, K))[v] = c.hi;
        if (lane < 32) reinterpret_cast<uint2*>(out + packed_e3m2_w0_bytes(N, K) + packed_e3m2_w1_bytes(N, K))[(f0 + i) * 32 + lane] = sc[i];
    }
}

__device__ __forceinline__ void expand_weights(const ExpandJob& e, const int id, const int lane, const int K) {
    if (e.canonical) expand_canonical(id, lane, (const uint8_t*)e.codes, (const float*)e.scales, e.N, K, e.out);
    else expand_packed(id, lane, (const uint4*)e.codes, (const uint2*)e.scales, e.N, K, e.out);
}

}  // namespace svdq
