// The layer's GEMM (b)+(c) for few tokens.
//
// The tile kernels stage 128 or 256 tokens by 128 or 256 channels through LDS and walk all of K in one block: with few
// tokens that leaves most CUs without a tile and the others with one wave per SIMD waiting for every stage (M = 512,
// N = K = 5120, E3M2: 160 blocks, 31 us; MXFP4: 40 blocks, 39 us).  Here a block of eight waves owns a small tile (32 or
// 64 channels by 32 or 64 tokens) and its waves split K: every wave runs its share of the groups straight from global
// memory to registers, with no LDS and no barrier in the loop, and the eight partial tiles meet in LDS at the end.
//
// A wave's K share also decides which part of the low-rank branch it adds: the quantise pass of this path leaves one
// partial h per slice of K (h = sum of the slices), and h L2 is linear in h, so wave w adds (h of slice w) L2 and
// nothing waits for the slices to be added up.  The caller's h gets their sum from one more row of blocks.  (One more
// block per token tile instead moved a channel tile's blocks to other XCDs, whose L2s then held the weights again:
// M = 803, K = 1920, N = 2304 took 25.2 us against 24.2 with a row and 24.0 with h left in slices.)
//
// Operand sources.  E3M2 activations against the canonical 4-bit weights (expanded in registers: with few tokens the
// weights are what is read, and expanding them to 6 bits in memory first would move them three times), against the
// expanded ones, nibble activations against the nibble kernel's packed weights (both turned into E3M2 fields in
// registers; same integer group sums), and MXFP4.
#include <type_traits>

#include "svdq_act.h"
#include "svdq_dev.h"
#include "svdq_epilogue.h"
#include "svdq_kernels.h"
#include "svdq_lds.h"
#include "svdq_quant_dev.h"

namespace svdq {

namespace {

typedef int int8v __attribute__((ext_vector_type(8)));

constexpr int WV = SMALL_SLICES;

// A launch with more than 112 bytes of arguments takes the host 0.4 us longer (3.2 against 2.8), with the grid's size among them
// (256 bytes more that the compiler asks for) 0.6: few tokens wait for the host, so both kernels' arguments are packed below that.
struct SmallArgs {
    const uint8_t* codes;
    const void* scales;
    const uint8_t *w0, *w1;      // w1: the scales of canonical weights; packed ones hold theirs behind the codes
    const float* h;              // hs partial h's, [M, r] each
    float* hsum;                 // out: h, the sum of the partial ones in slice order (null: not wanted)
    const uint16_t* L2;
    const float* bias;
    uint16_t* y;
    int64_t ldy;
    uint32_t M, begin;           // tokens [begin, M)
    int N, K;
    uint8_t hs, r;
};
static_assert(sizeof(SmallArgs) <= 112, "arguments of a cheap launch");

// Loads are buffer loads: a descriptor and a wave-uniform offset in scalar registers plus a per-lane 32-bit offset that is
// fixed for the kernel.  (With 64-bit addresses per lane, two registers for every load in flight, the compiler spills.)
// small_reach keeps every tensor of this path below 4 GB.
struct Buffers {
    __amdgpu_buffer_rsrc_t codes, scales, w0, w1, w2;
};
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const void* p) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, 0xffffffffu, 0x00027000);
}
template <class T>
__device__ __forceinline__ T at(__amdgpu_buffer_rsrc_t b, const uint32_t uniform, const uint32_t lane_off) {
    if constexpr (sizeof(T) == 16) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b128(b, lane_off, uniform, 0));
    else if constexpr (sizeof(T) == 8) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(b, lane_off, uniform, 0));
    else if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(b, lane_off, uniform, 0));
    else return __builtin_amdgcn_raw_buffer_load_b16(b, lane_off, uniform, 0);
}
// the planes of packed weights behind the codes (svdq_kernels.h)
template <int SRC>
__device__ __forceinline__ Buffers buffers_of(const void* codes, const void* scales, const uint8_t* w0, const uint8_t* w1, const int N, const int K) {
    const uint8_t* p1 = SRC == SMALL_E3M2_CANONICAL ? w1 : w0 + (SRC == SMALL_E3M2_PACKED ? packed_e3m2_w0_bytes(N, K) : (size_t)N * (K / 2));
    const uint8_t* p2 = SRC == SMALL_E3M2_PACKED ? p1 + packed_e3m2_w1_bytes(N, K) : nullptr;
    return Buffers{buffer(codes), buffer(scales), buffer(w0), buffer(p1), buffer(p2)};
}
template <int MT>
struct LaneOffsets {
    uint32_t row[MT];            // token (clamped to M - 1)
    uint32_t kh, l32, lane, n;   // k half, lane % 32, lane, first channel + lane % 32
};

// What a lane loads for one step (a 64-group; MXFP4: two) of its tokens and of its channels, and how the two become
// matrix instructions on y.
template <int N> using Vec4 = std::conditional_t<(N > 1), u32x4, uint4>;
template <int N> using Vec2 = std::conditional_t<(N > 1), u32x2, uint2>;
template <int SRC, int MT>
struct Tokens {
    Vec4<MT> x[MT];
    Vec2<MT> xh[MT];
    uint32_t sx[MT];
    __device__ __forceinline__ void load(const SmallArgs& a, const Buffers& B, const int g, const LaneOffsets<MT>& o) {
        const uint32_t M = (uint32_t)a.M;
        if constexpr (SRC == SMALL_NIBBLE) {
#pragma unroll
            for (int mi = 0; mi < MT; ++mi) {
                x[mi] = at<Vec4<MT>>(B.codes, (uint32_t)g * M * 32, o.row[mi] * 32 + o.kh * 16);
                sx[mi] = at<uint32_t>(B.scales, (uint32_t)g * M * 4, o.row[mi] * 4);
            }
        } else {
            const uint32_t Mp = (M + 3) & ~3u;
            const uint32_t blk = (uint32_t)g * Mp * E3M2_ROW_BYTES;
#pragma unroll
            for (int mi = 0; mi < MT; ++mi) {
                x[mi] = at<Vec4<MT>>(B.codes, blk, o.row[mi] * 32 + o.kh * 16);
                xh[mi] = at<Vec2<MT>>(B.codes, blk + Mp * 32, (o.kh * Mp + o.row[mi]) * 8);
                sx[mi] = at<uint32_t>(B.codes, blk + Mp * 48, o.row[mi] * 8);
            }
        }
    }
};
template <int SRC, int NI>
struct Channels {
    Vec4<NI> w[NI];
    Vec2<NI> wh[NI], sf[NI];
    uint32_t sw[NI];
    template <int MT>
    __device__ __forceinline__ void load(const SmallArgs& a, const Buffers& B, const int g, const int nb, const LaneOffsets<MT>& o) {
        const int ng = a.K >> 6;
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
            const uint32_t fr = (uint32_t)(nb + ni) * ng + g;
            if constexpr (SRC == SMALL_E3M2_CANONICAL) {
                w[ni] = at<Vec4<NI>>(B.w0, (uint32_t)g * 32 + (uint32_t)ni * 16 * a.K, o.n * (uint32_t)(a.K >> 1) + o.kh * 16);
                sw[ni] = at<uint32_t>(B.w1, ((uint32_t)g * a.N + ni * 32) * 4, o.n * 4);
            } else if constexpr (SRC == SMALL_E3M2_PACKED) {
                w[ni] = at<Vec4<NI>>(B.w0, fr * 1024, o.lane * 16);
                wh[ni] = at<Vec2<NI>>(B.w1, fr * 512, o.lane * 8);
                sf[ni] = at<Vec2<NI>>(B.w2, fr * 256, o.l32 * 8);
            } else {
                w[ni] = at<Vec4<NI>>(B.w0, fr * 1024, o.lane * 16);
                sf[ni] = at<Vec2<NI>>(B.w1, fr * 512, o.l32 * 8);
            }
        }
    }
};
// y += one group of an n-block times one of a token block: the weights as loaded, the tokens as fields (b) and scale pieces (sp,
// zeros in the lanes of k half 1: the scale product uses those of half 0 only).
template <int SRC, class W4, class W2>
__device__ __forceinline__ LaneCodes<true> weight_fields(const W4& w, const W2& wh) {
    if constexpr (SRC == SMALL_E3M2_PACKED) return LaneCodes<true>{uint4{w.x, w.y, w.z, w.w}, uint2{wh.x, wh.y}};
    else return e3m2_of_nibbles(uint4{w.x, w.y, w.z, w.w});
}
template <int SRC, class W2>
__device__ __forceinline__ uint2 weight_scales(const W2& sf, const uint32_t sw, const int kh) {
    uint2 s = {sf.x, sf.y};
    if constexpr (SRC == SMALL_E3M2_CANONICAL) {
        const uint32_t p = split_bf16(bits_f(sw)), w1 = p & 0xffffu, w2 = p >> 16;
        s = uint2{w1 | (w1 << 16), w2 | (w2 << 16)};
    }
    return uint2{kh ? 0u : s.x, kh ? 0u : s.y};
}
__device__ __forceinline__ void fold(const LaneCodes<true>& w, const uint2& s, const LaneCodes<true>& x, const uint2& sp, float16v& y) {
    const int8v av = {(int)w.lo.x, (int)w.lo.y, (int)w.lo.z, (int)w.lo.w, (int)w.hi.x, (int)w.hi.y, 0, 0};
    const int8v bv = {(int)x.lo.x, (int)x.lo.y, (int)x.lo.z, (int)x.lo.w, (int)x.hi.x, (int)x.hi.y, 0, 0};
    float16v zero;
#pragma unroll
    for (int i = 0; i < 16; ++i) zero[i] = 0.0f;
    const float16v P = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, zero, 3, 3, 0, 0x7f, 0, 0x7f);
    const float16v S = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(__builtin_bit_cast(short4v, s), __builtin_bit_cast(short4v, sp), zero, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 16; ++i) y[i] = __builtin_fmaf(P[i], S[i], y[i]);
}
template <int SRC, int NI, int MT>
__device__ __forceinline__ void multiply(const Tokens<SRC, MT>& t, const Channels<SRC, NI>& c, float16v (&y)[NI][MT], const int kh) {
    LaneCodes<true> xf[MT];
    uint2 sp[MT];
#pragma unroll
    for (int mi = 0; mi < MT; ++mi) {
        if constexpr (SRC == SMALL_NIBBLE) xf[mi] = e3m2_of_nibbles(uint4{t.x[mi].x, t.x[mi].y, t.x[mi].z, t.x[mi].w});
        else xf[mi] = LaneCodes<true>{uint4{t.x[mi].x, t.x[mi].y, t.x[mi].z, t.x[mi].w}, uint2{t.xh[mi].x, t.xh[mi].y}};
        uint32_t p = (SRC == SMALL_NIBBLE) ? split_bf16(bits_f(t.sx[mi])) : t.sx[mi];
        p = kh ? 0u : p;
        sp[mi] = uint2{p, p};
    }
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
        const LaneCodes<true> wf = weight_fields<SRC>(c.w[ni], c.wh[ni]);
        const uint2 s = weight_scales<SRC>(c.sf[ni], c.sw[ni], kh);
#pragma unroll
        for (int mi = 0; mi < MT; ++mi) fold(wf, s, xf[mi], sp[mi], y[ni][mi]);
    }
}

template <int MT>
struct Tokens<SMALL_MXFP4, MT> {
    uint4 x[2][MT];
    uint32_t sx[MT];
    __device__ __forceinline__ void load(const SmallArgs& a, const Buffers& B, const int st, const LaneOffsets<MT>& o) {
        const int ng = a.K >> 6;
        const uint32_t M = (uint32_t)a.M;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int g = (2 * st + j < ng) ? 2 * st + j : ng - 1;      // a group past K: its scale bytes are zero
#pragma unroll
            for (int mi = 0; mi < MT; ++mi) x[j][mi] = at<uint4>(B.codes, (uint32_t)g * M * 32, o.row[mi] * 32 + o.kh * 16);
        }
#pragma unroll
        for (int mi = 0; mi < MT; ++mi) sx[mi] = at<uint16_t>(B.scales, (uint32_t)st * M * 4, o.row[mi] * 4 + o.kh * 2);
    }
};
template <int NI>
struct Channels<SMALL_MXFP4, NI> {
    uint4 w[2][NI];
    uint32_t sw[NI];
    template <int MT>
    __device__ __forceinline__ void load(const SmallArgs& a, const Buffers& B, const int st, const int nb, const LaneOffsets<MT>& o) {
        const int ng = a.K >> 6, nst = (ng + 1) >> 1;
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
                w[j][ni] = at<uint4>(B.w0, ((uint32_t)(nb + ni) * ng + ((2 * st + j < ng) ? 2 * st + j : ng - 1)) * 1024, o.lane * 16);
            sw[ni] = at<uint16_t>(B.w1, ((uint32_t)(nb + ni) * nst + st) * 128, o.lane * 2);
        }
    }
};
template <int NI, int MT, int J>
__device__ __forceinline__ void multiply_group(const Tokens<SMALL_MXFP4, MT>& t, const Channels<SMALL_MXFP4, NI>& c, float16v (&y)[NI][MT]) {
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
        const int8v av = {(int)c.w[J][ni].x, (int)c.w[J][ni].y, (int)c.w[J][ni].z, (int)c.w[J][ni].w, 0, 0, 0, 0};
#pragma unroll
        for (int mi = 0; mi < MT; ++mi) {
            const int8v bv = {(int)t.x[J][mi].x, (int)t.x[J][mi].y, (int)t.x[J][mi].z, (int)t.x[J][mi].w, 0, 0, 0, 0};
            y[ni][mi] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, y[ni][mi], 4, 4, J, (int)c.sw[ni], J, (int)t.sx[mi]);
        }
    }
}
template <int NI, int MT>
__device__ __forceinline__ void multiply(const Tokens<SMALL_MXFP4, MT>& t, const Channels<SMALL_MXFP4, NI>& c, float16v (&y)[NI][MT], const int) {
    multiply_group<NI, MT, 0>(t, c, y);
    multiply_group<NI, MT, 1>(t, c, y);
}

// h = sum of its slices, in slice order: four elements, number v of them (n is a multiple of 16)
__device__ __forceinline__ void sum_slices(const float* __restrict__ part, const int slices, const int64_t n, float* __restrict__ h, const int64_t v) {
    const int64_t i = v * 4;
    if (i >= n) return;
    *reinterpret_cast<float4*>(h + i) = sum_of_slices(part, slices, n, i);
}

// f(IC<0>), f(IC<1>), ..: a loop whose index is a constant from the first.  In a 64 x 64 tile, with Tokens and Channels of language vectors,
// it keeps all of them in registers: packed E3M2 fields were in scratch in part, nibbles spilled (M = 44, K = 3264, N = 9728 18.3 -> 17.2 us).
template <int COUNT, class F>
__device__ __forceinline__ void steps_of(F f) {
    if constexpr (COUNT > 0) {
        steps_of<COUNT - 1>(f);
        f(IC<COUNT - 1>{});
    }
}

template <int SRC, int NI, int MT>
__global__ __launch_bounds__(64 * WV, NI * MT >= 4 ? 2 : 4)
void small_gemm_kernel(const SmallArgs a) {
    constexpr int Q = NI * MT * 4;                        // quads of accumulator registers (four neighbouring channels)
    __shared__ float4 part[WV / 2][Q][64];
    const int lane = threadIdx.x & 63, l32 = lane & 31, kh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n0 = (int)blockIdx.x * 32 * NI;
    const int64_t M = a.M, m0 = a.begin + (int64_t)blockIdx.y * 32 * MT;
    if (m0 >= M) {                                        // the blocks behind the token tiles
        for (int b = (int)blockIdx.x; b < (M * a.r + 4 * 64 * WV - 1) / (4 * 64 * WV); b += a.N / (32 * NI))
            sum_slices(a.h, a.hs, M * a.r, a.hsum, (int64_t)b * (64 * WV) + threadIdx.x);
        return;
    }
    const Buffers B = buffers_of<SRC>(a.codes, a.scales, a.w0, a.w1, a.N, a.K);
    LaneOffsets<MT> off{{}, (uint32_t)kh, (uint32_t)l32, (uint32_t)lane, (uint32_t)(n0 + l32)};
#pragma unroll
    for (int mi = 0; mi < MT; ++mi) {
        const int64_t m = m0 + 32 * mi + l32;
        off.row[mi] = (uint32_t)(m < M ? m : M - 1);  // rows beyond M: results never stored
    }
    float16v y[NI][MT];
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int mi = 0; mi < MT; ++mi)
#pragma unroll
            for (int i = 0; i < 16; ++i) y[ni][mi][i] = 0.0f;

    // this wave's share of K: steps wave, wave + WV, ... (the lines of a canonical weight row hold four groups: taken by
    // neighbouring waves at about the same time they are fetched once)
    constexpr int GROUPS = (SRC == SMALL_MXFP4) ? 2 : 1;
    const int steps = ((a.K >> 6) + GROUPS - 1) / GROUPS;
    const int s1 = (steps - wave + WV - 1) / WV;
    // What bounds a wave is the latency of its loads, above all of the weights, which come from HBM (one step ahead of
    // their use, a step of 32 x 64 codes took 1.4 us at M = 1): their next DW - 1 steps are in flight, of the tokens
    // (in L2) the next one.  Loads past the share re-read its last step: with a condition around every load and step the
    // compiler no longer overlaps them.  As many as the registers hold: nibble operands on both sides spill at 4 in a
    // 32 x 32 tile (M = 1 .. 100, K = 576 .. 10624: 3 to 9 % slower than at 3).
    constexpr int DW = (SRC == SMALL_E3M2_PACKED) ? 2 : ((SRC == SMALL_MXFP4 && NI * MT > 1) || (SRC == SMALL_NIBBLE && NI * MT == 1)) ? 3 : 4;
    Tokens<SRC, MT> xt[2];
    Channels<SRC, NI> wc[DW];
    auto clamp = [&](const int s) { return wave + WV * ((s < s1) ? s : s1 - 1); };
    if (s1 > 0) {
        xt[0].load(a, B, clamp(0), off);
#pragma unroll
        for (int d = 0; d < DW - 1; ++d) wc[d].load(a, B, clamp(d), n0 >> 5, off);
    }
    constexpr int U = (DW % 2) ? 2 * DW : DW;             // both rings return to their first slot
    int s = 0;
    auto step = [&](const int d) __attribute__((always_inline)) {
        wc[(d + DW - 1) % DW].load(a, B, clamp(s + d + DW - 1), n0 >> 5, off);
        xt[(d + 1) & 1].load(a, B, clamp(s + d + 1), off);
        if constexpr (SRC == SMALL_E3M2_PACKED && NI * MT == 1) __builtin_amdgcn_sched_barrier(0);   // left to itself the compiler requests them behind the products
        multiply(xt[d & 1], wc[d % DW], y, kh);
        __builtin_amdgcn_sched_barrier(0);                // steps interleaved would need registers for several
    };
    auto last_step = [&](const int d) __attribute__((always_inline)) {
        if (s + d >= s1) return;
        if (d + DW - 1 < U - 1) wc[(d + DW - 1) % DW].load(a, B, clamp(s + d + DW - 1), n0 >> 5, off);
        xt[(d + 1) & 1].load(a, B, clamp(s + d + 1), off);
        multiply(xt[d & 1], wc[d % DW], y, kh);
    };
    if constexpr (NI * MT > 2) {
        for (; s + U <= s1; s += U) steps_of<U>([&](auto D) { step(decltype(D)::value); });
        steps_of<U - 1>([&](auto D) { last_step(decltype(D)::value); });
    } else {                                              // (with constants 3 % longer)
        for (; s + U <= s1; s += U)
#pragma unroll
            for (int d = 0; d < U; ++d) step(d);
#pragma unroll
        for (int d = 0; d < U - 1; ++d) last_step(d);
    }

    if (wave == 0 || (a.r > 0 && wave < a.hs))
        add_lowrank_bias<NI, MT>(y, a.h + (size_t)wave * M * a.r, a.L2, wave == 0 ? a.bias : nullptr, m0, n0, M, a.N, a.r, lane);

    // sum of the eight partial tiles: waves 4..7 hand theirs to waves 0..3, then every wave finishes Q / 8 quads of four
    auto quad = [&](const int q) {
        const float16v& t = y[(q >> 2) / MT][(q >> 2) % MT];
        return float4{t[4 * (q & 3)], t[4 * (q & 3) + 1], t[4 * (q & 3) + 2], t[4 * (q & 3) + 3]};
    };
    if (wave >= WV / 2) {
#pragma unroll
        for (int q = 0; q < Q; ++q) part[wave - WV / 2][q][lane] = quad(q);
    }
    __syncthreads();
    if (wave < WV / 2) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const float4 o = part[wave][q][lane], v = quad(q);
            part[wave][q][lane] = float4{v.x + o.x, v.y + o.y, v.z + o.z, v.w + o.w};
        }
    }
    __syncthreads();
    for (int q = wave; q < Q; q += WV) {
        const float4 p0 = part[0][q][lane], p1 = part[1][q][lane], p2 = part[2][q][lane], p3 = part[3][q][lane];
        const float v[4] = {(p0.x + p1.x) + (p2.x + p3.x), (p0.y + p1.y) + (p2.y + p3.y), (p0.z + p1.z) + (p2.z + p3.z),
                            (p0.w + p1.w) + (p2.w + p3.w)};
        const int t = q >> 2;
        const int64_t m = m0 + 32 * (t % MT) + l32;
        const int n = n0 + 32 * (t / MT) + 8 * (q & 3) + 4 * kh;
        if (m < M) *reinterpret_cast<uint2*>(a.y + m * a.ldy + n) = uint2{f2_bf16_rne(v[0], v[1]), f2_bf16_rne(v[2], v[3])};
    }
}

template <int SRC>
hipError_t launch_src(const SmallArgs& a, hipStream_t stream) {
    auto go = [&](auto kern, int ni, int mt) {
        hipLaunchKernelGGL(kern, dim3((unsigned)(a.N / (32 * ni)), (a.M - a.begin + 32 * mt - 1) / (32 * mt) + (a.hsum ? 1u : 0u)), dim3(64 * WV), 0, stream, a);
    };
    if (small_shape(a.M - a.begin, a.N, a.K, SRC == SMALL_MXFP4) == 1) go(small_gemm_kernel<SRC, 1, 1>, 1, 1);
    else if constexpr (SRC == SMALL_MXFP4) go(small_gemm_kernel<SRC, 1, 2>, 1, 2);
    else go(small_gemm_kernel<SRC, 2, 2>, 2, 2);
    return hipGetLastError();
}

// ---- The whole layer in one launch, for few tokens and a short K.
//
// There a layer is what its two launches cost: M = 256, K = N = 512, 4.9 us of quantise pass and 4.2 of GEMM on the GPU, most of it
// starts, ends and first loads, and 3.4 us of host time for each.  Here every block quantises the tokens of its tile itself,
// through the quantise pass's own chain, and multiplies them by its channels' weights; only the partial tiles, and those of h,
// meet in LDS.  The blocks of the first channel tile leave codes, scales and h in the layer's buffers.  Wave w has the 64-groups
// w, w + 8, ..
// The price is that the tokens are quantised and projected once per channel tile: 128 bytes of L1 fragments and some 6 vector
// instructions per token for each of K, which is why K is short (small_fused).  M = 256, K = N = 512: 10.6 -> 6.6 us a call, of which
// the kernel's 6.6 (one launch of 3.4 us and the caller's own host work take about as long); MXFP4 9.9 -> 6.9, the kernel 5.8.
// SPREAD = false: 32 tokens.  A wave's lanes hold a group's codes just as the matrix instruction wants them.
// SPREAD: 1 << rs tokens, at most 16.  The chain takes 32 blocks of 32 values per half wave, whatever tokens and groups they are of,
// and the codes go through LDS.
struct FusedArgs {
    const uint16_t* x;
    const float* inv_lambda;
    const uint4* l1p;
    uint8_t* codes;              // out, as the format's quantise pass writes them
    void* scales;                // out; E3M2 fields have none: the scales of canonical weights
    float* h;
    const uint8_t* w0;
    const uint16_t* L2;
    const float* bias;
    uint16_t* y;
    int64_t ldx, ldy;
    uint32_t M;
    float rho;
    uint16_t K, nblocks;         // nblocks: N / 32
    uint8_t r, rs, gelu;
};
static_assert(sizeof(FusedArgs) <= 112, "arguments of a cheap launch");
// wait for this wave's LDS traffic, then for the other waves: loads from global memory stay in flight
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int SRC, int NI, bool SPREAD>
__global__ __launch_bounds__(64 * WV, 2)
void fused_layer_kernel(const FusedArgs a) {
    constexpr bool MX = SRC == SMALL_MXFP4;
    constexpr int Q = NI * 4;                              // quads of the tile
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    float4 (*const part)[Q][64] = reinterpret_cast<float4 (*)[Q][64]>(smem);
    const int rs = SPREAD ? a.rs : 5, rmask = (1 << rs) - 1;
    const FusedLds lds = fused_lds(NI, a.K, a.r > 0, SPREAD, rs);
    // the planes, each formed from the one ahead of it and what is constant written as such (M = 16, K = N = 512 5.92 us, otherwise 5.97)
    constexpr uint32_t TILES = fused_lds(NI, 64, true, SPREAD, 0).tiles;
    float* const hpart = reinterpret_cast<float*>(smem + TILES);                     // [WV][32][32]
    float* const hsum = hpart + FUSED_HPART;                                         // [32][FUSED_H_ROW]
    float* const il_s = a.r ? hsum + FUSED_H : hpart;
    const int N = a.nblocks * 32, K = a.K;
    const int64_t M = a.M;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, kh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n0 = (int)blockIdx.x * 32 * NI, ng = K >> 6;
    const int trow = l32 & rmask;                          // this lane's token of the tile
    const int64_t m0 = (int64_t)blockIdx.y << rs, row = m0 + trow;
    uint8_t* const clo = reinterpret_cast<uint8_t*>(il_s) + lds.il;                // SPREAD: [2 g + kh][token] x 16, x 8, x 4 bytes
    uint8_t* const chi = clo + lds.lo;
    uint8_t* const csc = chi + lds.hi;
    // its piece s at place s ^ (token / 4) % 4: the 16 tokens of a read stand in different banks
    uint8_t* const cxv = csc + lds.scale;
    auto x_place = [&](const int g, const int s) { return reinterpret_cast<uint4*>(cxv + (((2 * g + kh) << rs) + trow) * 64) + (s ^ ((trow >> 2) & 3)); };
    const bool first = blockIdx.x == 0;
    const Buffers B = buffers_of<SRC>(nullptr, nullptr, a.w0, (const uint8_t*)a.scales, N, K);
    const uint16_t* const xrow = a.x + (row < M ? row : M - 1) * a.ldx + kh * 32;
    auto load_x = [&](uint4 (&x)[4], const int g) {
#pragma unroll
        for (int s = 0; s < 4; ++s) x[s] = reinterpret_cast<const uint4*>(xrow + g * 64)[s];
    };

    for (int i = tid * 4; i < K; i += 256 * WV) *reinterpret_cast<float4*>(il_s + (i >> 5) * FUSED_IL_ROW + (i & 31)) = *reinterpret_cast<const float4*>(a.inv_lambda + i);
    // quantise this lane's 32 values of group g into fields (MXFP4: nibbles) and scale, and into the layer's buffers
    struct Coded {
        LaneCodes<true> c;
        uint32_t s;                                        // scale pieces; MXFP4: the E8M0 byte
    };
    auto quantise = [&](const uint4 (&x)[4], const int g, const bool writes) {
        const float* il = il_s + (2 * g + kh) * FUSED_IL_ROW;
        Coded o;
        if constexpr (MX) {
            quantize_block_mx(x, il, a.rho, o.c.lo, o.s);
            if (writes) {
                *reinterpret_cast<uint4*>(a.codes + ((size_t)g * M + row) * 32 + kh * 16) = o.c.lo;
                uint8_t* se = (uint8_t*)a.scales + (((size_t)(g >> 1) * M + row) * 2 + kh) * 2;
                se[g & 1] = (uint8_t)o.s;
                if (g == ng - 1 && (ng & 1)) se[1] = 0;                  // a group past K counts as empty
            }
        } else {
            float s;
            uint4 nib;
            quantize_rows<true, SRC == SMALL_NIBBLE>(x, il, a.rho, o.c, s, &nib);
            o.s = split_bf16(s);
            if (writes) {
                if constexpr (SRC == SMALL_NIBBLE) {
                    *reinterpret_cast<uint4*>(a.codes + ((size_t)g * M + row) * 32 + kh * 16) = nib;
                    if (kh == 0) ((float*)a.scales)[(size_t)g * M + row] = s;
                } else {
                    const size_t Mp = (size_t)((M + 3) & ~(int64_t)3);
                    uint8_t* blk = a.codes + (size_t)g * Mp * E3M2_ROW_BYTES;
                    *reinterpret_cast<uint4*>(blk + (size_t)row * 32 + kh * 16) = o.c.lo;
                    *reinterpret_cast<uint2*>(blk + Mp * 32 + ((size_t)kh * Mp + row) * 8) = o.c.hi;
                    if (kh == 0) *reinterpret_cast<uint2*>(blk + Mp * 48 + (size_t)row * 8) = uint2{o.s, o.s};
                }
            }
        }
        return o;
    };
    uint4 xt[4];                                           // SPREAD: the wave's first share of the chain
    const int per_wave = 32 >> rs, tg = wave * per_wave + (l32 >> rs);
    if (SPREAD && tg < ng) load_x(xt, tg);

    struct Group {
        uint4 x[4], l1[4][2], w[NI];
        uint2 wh[NI], sf[NI];
        uint32_t sw[NI];
    };
    auto load = [&](Group& o, const int g) {
        if (!SPREAD) load_x(o.x, g);
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
            const uint32_t fr = (uint32_t)((n0 >> 5) + ni) * ng + g;
            if constexpr (SRC == SMALL_E3M2_CANONICAL) {
                o.w[ni] = at<uint4>(B.w0, (uint32_t)g * 32 + (uint32_t)ni * 16 * K, (uint32_t)(n0 + l32) * (uint32_t)(K >> 1) + kh * 16);
                o.sw[ni] = at<uint32_t>(B.w1, ((uint32_t)g * N + ni * 32) * 4, (uint32_t)(n0 + l32) * 4);
            } else {
                o.w[ni] = at<uint4>(B.w0, fr * 1024, lane * 16);
                if constexpr (SRC == SMALL_E3M2_PACKED) {
                    o.wh[ni] = at<uint2>(B.w1, fr * 512, lane * 8);
                    o.sf[ni] = at<uint2>(B.w2, fr * 256, l32 * 8);
                } else if constexpr (SRC == SMALL_NIBBLE) {
                    o.sf[ni] = at<uint2>(B.w1, fr * 512, l32 * 8);
                } else {
                    o.sw[ni] = at<uint16_t>(B.w1, (((uint32_t)((n0 >> 5) + ni) * ((ng + 1) >> 1)) + (g >> 1)) * 128, lane * 2);
                }
            }
        }
        if (a.r > 0) {
            const uint4* pb = a.l1p + (size_t)g * (4 * 2 * 64) + lane;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                o.l1[s][0] = pb[(s * 2 + 0) * 64];
                o.l1[s][1] = pb[(s * 2 + 1) * 64];
            }
        }
    };
    Group cur, nxt;
    if (wave < ng) load(cur, wave);
    if (SPREAD && wave + WV < ng) load(nxt, wave + WV);
    // what the end needs, requested now: this wave finishes quad fq of channel block fni
    const int fni = (NI == 1) ? 0 : wave >> 2, fq = wave & 3;
    const bool finishes = wave < Q;
    uint32_t l2w[2][4] = {};
    float4 bv{0.f, 0.f, 0.f, 0.f};
    if (finishes) {
        if (a.r > 0) {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (16 * ks < a.r) {
                        const uint16_t* p = a.L2 + (int64_t)(16 * ks + 8 * kh + 2 * e) * N + n0 + 32 * fni + l32;
                        l2w[ks][e] = (uint32_t)p[0] | ((uint32_t)p[N] << 16);
                    }
        }
        if (a.bias) bv = *reinterpret_cast<const float4*>(a.bias + n0 + 32 * fni + 8 * fq + 4 * kh);
    }
    float16v y[NI], hacc, zero;
#pragma unroll
    for (int i = 0; i < 16; ++i) zero[i] = 0.0f;
    hacc = zero;
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) y[ni] = zero;
    lds_barrier();
    if constexpr (SPREAD) {
        for (int g = tg; g < ng; g += WV * per_wave) {
            if (a.gelu) gelu_tanh_rows(xt);
            const Coded o = quantise(xt, g, first && row < M);
            const int at = ((2 * g + kh) << rs) + trow;
            *reinterpret_cast<uint4*>(clo + at * 16) = o.c.lo;
            if (!MX) *reinterpret_cast<uint2*>(chi + at * 8) = o.c.hi;
            *reinterpret_cast<uint32_t*>(csc + at * 4) = o.s;
            if (a.r > 0) {
#pragma unroll
                for (int s = 0; s < 4; ++s) *x_place(g, s) = xt[s];
            }
            if (g + WV * per_wave < ng) load_x(xt, g + WV * per_wave);
        }
        lds_barrier();
    }

    for (int g = wave; g < ng; g += WV) {
        if (!SPREAD && g + WV < ng) load(nxt, g + WV);
        if (!SPREAD && a.gelu) gelu_tanh_rows(cur.x);
        if (a.r > 0) {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const bf16x8 av = __builtin_bit_cast(bf16x8, SPREAD ? *x_place(g, s) : cur.x[s]);
                hacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, __builtin_bit_cast(bf16x8, cur.l1[s][0]), hacc, 0, 0, 0);
                hacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, __builtin_bit_cast(bf16x8, cur.l1[s][1]), hacc, 0, 0, 0);
            }
        }
        Coded o;
        if constexpr (SPREAD) {
            const int at = ((2 * g + kh) << rs) + trow;
            o.c.lo = *reinterpret_cast<const uint4*>(clo + at * 16);
            if (!MX) o.c.hi = *reinterpret_cast<const uint2*>(chi + at * 8);
            o.s = *reinterpret_cast<const uint32_t*>(csc + at * 4);
        } else {
            o = quantise(cur.x, g, first && row < M);
        }
        if constexpr (MX) {
            const int8v bvx = {(int)o.c.lo.x, (int)o.c.lo.y, (int)o.c.lo.z, (int)o.c.lo.w, 0, 0, 0, 0};
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                const int8v av = {(int)cur.w[ni].x, (int)cur.w[ni].y, (int)cur.w[ni].z, (int)cur.w[ni].w, 0, 0, 0, 0};
                y[ni] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bvx, y[ni], 4, 4, 0, (int)(cur.sw[ni] >> (8 * (g & 1))), 0, (int)o.s);
            }
        } else {
            const uint32_t p = kh ? 0u : o.s;
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
                fold(weight_fields<SRC>(cur.w[ni], cur.wh[ni]), weight_scales<SRC>(cur.sf[ni], cur.sw[ni], kh), o.c, uint2{p, p}, y[ni]);
        }
        cur = nxt;
        if (SPREAD && g + 2 * WV < ng) load(nxt, g + 2 * WV);
    }

#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const float16v& t = y[q >> 2];
        part[wave][q][lane] = float4{t[4 * (q & 3)], t[4 * (q & 3) + 1], t[4 * (q & 3) + 2], t[4 * (q & 3) + 3]};
    }
    if (a.r > 0) {
#pragma unroll
        for (int i = 0; i < 16; ++i) hpart[wave * 1024 + (8 * (i >> 2) + 4 * kh + (i & 3)) * 32 + l32] = hacc[i];
    }
    lds_barrier();
    if (a.r > 0) {
        const int hr = tid >> 4, hj = (tid & 15) * 2;
        auto piece = [&](const int w) { return *reinterpret_cast<const float2*>(hpart + w * 1024 + hr * 32 + hj); };
        auto sum4 = [&](const int w) {
            const float2 p0 = piece(w), p1 = piece(w + 1), p2 = piece(w + 2), p3 = piece(w + 3);
            return float2{(p0.x + p1.x) + (p2.x + p3.x), (p0.y + p1.y) + (p2.y + p3.y)};
        };
        const float2 s0 = sum4(0), s1 = sum4(4), t{s0.x + s1.x, s0.y + s1.y};
        *reinterpret_cast<float2*>(hsum + hr * FUSED_H_ROW + hj) = t;
        if (first && hr <= rmask && hj < a.r && m0 + hr < M) *reinterpret_cast<float2*>(a.h + (m0 + hr) * a.r + hj) = t;
        lds_barrier();
    }
    if (!finishes) return;
    float16v lr = zero;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
        if (16 * ks < a.r) {
            const float* hp = hsum + l32 * FUSED_H_ROW + 16 * ks + 8 * kh;
            uint32_t hi[4], lo[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float2 v = *reinterpret_cast<const float2*>(hp + 2 * e);
                hi[e] = f2_bf16_rne(v.x, v.y);
                lo[e] = f2_bf16_rne(v.x - bf16lo_f(hi[e]), v.y - bf16hi_f(hi[e]));
            }
            const bf16x8 lf = __builtin_bit_cast(bf16x8, uint4{l2w[ks][0], l2w[ks][1], l2w[ks][2], l2w[ks][3]});
            lr = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lf, __builtin_bit_cast(bf16x8, uint4{hi[0], hi[1], hi[2], hi[3]}), lr, 0, 0, 0);
            lr = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lf, __builtin_bit_cast(bf16x8, uint4{lo[0], lo[1], lo[2], lo[3]}), lr, 0, 0, 0);
        }
    float4 p[WV];
#pragma unroll
    for (int w = 0; w < WV; ++w) p[w] = part[w][wave][lane];
    auto sum = [&](auto c, const float l, const float b) {
        return (((c(p[0]) + c(p[4])) + (c(p[1]) + c(p[5]))) + ((c(p[2]) + c(p[6])) + (c(p[3]) + c(p[7])))) + (l + b);
    };
    auto low = [&](const int j) { return fq == 0 ? lr[j] : fq == 1 ? lr[4 + j] : fq == 2 ? lr[8 + j] : lr[12 + j]; };
    const float v0 = sum([](const float4& f) { return f.x; }, low(0), bv.x), v1 = sum([](const float4& f) { return f.y; }, low(1), bv.y);
    const float v2 = sum([](const float4& f) { return f.z; }, low(2), bv.z), v3 = sum([](const float4& f) { return f.w; }, low(3), bv.w);
    if (l32 <= rmask && row < M)
        *reinterpret_cast<uint2*>(a.y + row * a.ldy + n0 + 32 * fni + 8 * fq + 4 * kh) = uint2{f2_bf16_rne(v0, v1), f2_bf16_rne(v2, v3)};
}

template <int SRC>
hipError_t launch_fused_src(FusedArgs a, hipStream_t stream) {
    const unsigned M = a.M;
    auto go = [&](auto kern, unsigned ni, bool spread, int rs) {
        a.rs = (uint8_t)rs;
        hipLaunchKernelGGL(kern, dim3(a.nblocks / ni, (M + (1u << rs) - 1) >> rs), dim3(64 * WV), fused_lds((int)ni, a.K, a.r != 0, spread, rs).end(), stream, a);
    };
    if (small_fused(M, a.nblocks * 32, a.K, a.r, SRC == SMALL_MXFP4) == FUSED_SPREAD) {
        go(fused_layer_kernel<SRC, 1, true>, 1, true, fused_spread(M));
    } else if ((M + 31) / 32 * a.nblocks <= 256) {
        go(fused_layer_kernel<SRC, 1, false>, 1, false, 5);
    } else {
        go(fused_layer_kernel<SRC, 2, false>, 2, false, 5);
    }
    return hipGetLastError();
}

__global__ __launch_bounds__(256)
void sum_slices_kernel(const float* __restrict__ part, int slices, int64_t n, float* __restrict__ h) {
    sum_slices(part, slices, n, h, (int64_t)blockIdx.x * 256 + threadIdx.x);
}

}  // namespace

hipError_t launch_sum_slices(const float* part, int slices, int64_t M, int r, float* h, hipStream_t stream) {
    const int64_t n = M * r;
    hipLaunchKernelGGL(sum_slices_kernel, dim3((unsigned)((n + 1023) / 1024)), dim3(256), 0, stream, part, slices, n, h);
    return hipGetLastError();
}

hipError_t launch_small_gemm(int source, const uint8_t* codes, const void* scales, const void* w0, const void* w1,
                             const float* h, int slices, float* hsum, const void* L2, const float* bias, int64_t M, int64_t begin, int N, int K, int r,
                             void* y, int64_t ldy, hipStream_t stream) {
    const SmallArgs a{codes, scales, (const uint8_t*)w0, (const uint8_t*)w1, h, hsum, (const uint16_t*)L2, bias, (uint16_t*)y, ldy,
                      (uint32_t)M, (uint32_t)begin, N, K, (uint8_t)slices, (uint8_t)r};
    switch (source) {
        case SMALL_E3M2_CANONICAL: return launch_src<SMALL_E3M2_CANONICAL>(a, stream);
        case SMALL_E3M2_PACKED: return launch_src<SMALL_E3M2_PACKED>(a, stream);
        case SMALL_NIBBLE: return launch_src<SMALL_NIBBLE>(a, stream);
        default: return launch_src<SMALL_MXFP4>(a, stream);
    }
}

hipError_t launch_fused_layer(int source, const void* x, int64_t ldx, const float* inv_lambda, float rho, bool gelu, const void* l1p,
                              uint8_t* codes, void* scales, float* h, const void* w0, const void* w1,
                              const void* L2, const float* bias, int64_t M, int N, int K, int r, void* y, int64_t ldy, hipStream_t stream) {
    const FusedArgs a{(const uint16_t*)x, inv_lambda, (const uint4*)l1p, codes, source == SMALL_E3M2_CANONICAL ? const_cast<void*>(w1) : scales, h,
                      (const uint8_t*)w0, (const uint16_t*)L2, bias, (uint16_t*)y, ldx, ldy, (uint32_t)M, rho, (uint16_t)K, (uint16_t)(N / 32),
                      (uint8_t)r, 0, (uint8_t)gelu};
    switch (source) {
        case SMALL_E3M2_CANONICAL: return launch_fused_src<SMALL_E3M2_CANONICAL>(a, stream);
        case SMALL_E3M2_PACKED: return launch_fused_src<SMALL_E3M2_PACKED>(a, stream);
        case SMALL_NIBBLE: return launch_fused_src<SMALL_NIBBLE>(a, stream);
        default: return launch_fused_src<SMALL_MXFP4>(a, stream);
    }
}

}  // namespace svdq
