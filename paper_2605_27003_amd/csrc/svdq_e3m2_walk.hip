// The E3M2 GEMM (svdq_gemm_e3m2.hip: operands, arithmetic and their order) for many tokens: 256 x 256 tiles, eight
// waves of 128 tokens x 64 channels, one block per CU that walks its tiles.  Same bits as the 128 x 128 kernel.
//
// Why: the transfers from L2 into LDS were a fifth of the 128 x 128 kernel (timing only, K = 5120 .. 10240, no transfers in
// its loop: 61 -> 48 ns per 32 x 32 tile, group and SIMD; no LDS reads: 58), and every tile began with 5.6 us for the
// low-rank term, of 50.  A tile of twice the side moves half the bytes per output.  Its accumulators (128 registers) leave
// room for one set of operands, refilled in place, and for three of the four result registers that the smaller kernel
// alternates; a register-only loop of this order runs as fast as with four (46.5 ns, 91 clocks).  A block that is alone on
// its CU shows the start and end of every tile, so the ring of operands never drains: its last stages take the next
// tile's low-rank operands and first groups, and nothing in the kernel loads from global memory to registers.
// Measured, M = 32760, K = N = 5120: 871 us (128 x 128: 945); per tile 80 us loop (113 clocks per 32 x 32 tile and group at
// the 1.85 GHz that the power limit leaves), 0.6 wait, 2.8 low-rank term and bias, 1.4 store.  What is left in the loop:
// transfers 12 clocks, LDS reads 6 (timing only).  Fewer clocks are not always less time: transfers placed elsewhere in a
// step, or waves 4..7 half a step behind, change the clocks by 5 to 14 and the frequency the other way.
#include "svdq_dev.h"
#include "svdq_epilogue.h"
#include "svdq_kernels.h"
#include "svdq_lds.h"
#include "svdq_tiles.h"

namespace svdq {

namespace {

constexpr int BM = 256, BN = 256, NSLOTS = 5;

// A ring slot as one 64-group of the tile (byte offsets).  Fragment planes are in lane order: every LDS read is a wave's
// base plus lane x 16 (or x 8).
constexpr uint32_t OFF_X0 = 0;         // activation codes, bytes 0..15:  [32-token block][half][token] x 16 B
constexpr uint32_t OFF_W0 = 8192;      // weight codes, bytes 0..15:      [n-block][lane] x 16 B
constexpr uint32_t OFF_X1 = 16384;     // activation codes, bytes 16..23: [32-token block][half][token] x 8 B
constexpr uint32_t OFF_W1 = 20480;     // weight codes, bytes 16..23:     [n-block][lane] x 8 B
constexpr uint32_t OFF_SX = 24576;     // token-scale pieces:   [token] x 8 B
constexpr uint32_t OFF_SF = 26624;     // channel-scale pieces: [n-block][channel] x 8 B
constexpr uint32_t STAGE = 28672;
// ... and as 16 columns of the low-rank term
constexpr uint32_t OFF_H = 0;          // h: [32-token block][4 columns][token] x 16 B
constexpr uint32_t OFF_L2 = 16384;     // L2: [row] x 512 B, 16-byte piece c of row k at place c ^ 4 (k % 4)
constexpr uint32_t OFF_B = 24576;      // bias: [channel] x 4 B

constexpr uint32_t OFF_STORE = NSLOTS * STAGE, OFF_ZERO = OFF_STORE + 8 * WALK_STORE_BYTES;
constexpr uint32_t LDS_BYTES = OFF_ZERO + 1024;    // 1 KB of zeros: the scale-product operands of k half 1
static_assert(LDS_BYTES <= 160 * 1024, "LDS of a CU");

typedef int int8v __attribute__((ext_vector_type(8)));

// dma16 by the lower 32 lanes: 512 bytes
__device__ __forceinline__ void dma16_half(const void* sbase, uint32_t voff, uint32_t lds_off) {
    const uint64_t a = (uint64_t)(uintptr_t)sbase;
    const uint64_t sa = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32)) << 32) |
                        (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    lds_off = __builtin_amdgcn_readfirstlane(lds_off);
    asm volatile("s_mov_b32 m0, %2\n\ts_mov_b32 exec_hi, 0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1\n\ts_mov_b32 exec_hi, -1"
                 ::"v"(voff), "s"(sa), "s"(lds_off) : "memory");
}

__global__ __launch_bounds__(512, 1)
void gemm_e3m2_walk_kernel(const uint8_t* __restrict__ act, const uint8_t* __restrict__ w0, const uint8_t* __restrict__ w1,
                           const uint8_t* __restrict__ sfr, const float* __restrict__ h, const uint16_t* __restrict__ L2,
                           const float* __restrict__ bias, int64_t M, int N, int K, int r, int has_bias,
                           uint16_t* __restrict__ yout, int64_t ldy, const WalkGrid tg) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[LDS_BYTES];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;                      // this wave: tokens 128 wm .., channels 64 wn ..
    const int ng = K >> 6;                                        // >= NSLOTS (the launcher sees to it)
    const int64_t Mp = (M + 3) & ~(int64_t)3;
    const uint32_t ring0 = (uint32_t)(uintptr_t)(lds_byte*)lds;
    const uint32_t store0 = ring0 + OFF_STORE + wave * WALK_STORE_BYTES;
    if (tid < 64) *reinterpret_cast<uint4*>(lds + OFF_ZERO + tid * 16) = uint4{0u, 0u, 0u, 0u};     // read behind two barriers

    struct Tile {
        int64_t m0;
        int n0;
    };
    auto exists = [&](const int id) { return (id >> 3) < tg.chunk && (id & 7) * tg.chunk + (id >> 3) < tg.mtiles * tg.ntiles; };
    auto tile_at = [&](const int id) {
        int mt, nt;
        walk_tile(tg, id, mt, nt);
        return Tile{(int64_t)mt * BM, nt * BN};
    };

    // ---- operand transfers, four per wave and group: 1 KB of activation codes (32 tokens), 1 KB of weight codes (an
    // n-block), 1 KB of the 8-byte planes and 512 bytes of scale pieces (activations on waves 0..3, weights on 4..7).
    const size_t gstride = (size_t)Mp * E3M2_ROW_BYTES;
    const size_t stride2 = wave < 4 ? gstride : 512, stride3 = wave < 4 ? gstride : 256;
    const uint32_t lds2 = wave < 4 ? OFF_X1 + wave * 1024 : OFF_W1 + (wave - 4) * 1024;
    const uint32_t lds3 = wave < 4 ? OFF_SX + wave * 512 : OFF_SF + (wave - 4) * 512;
    const uint8_t* sp[4];
    uint32_t sv[4];
    auto set_streams = [&](const Tile& t) {
        int ln = lane;
        asm volatile("" : "+v"(ln));                              // per tile, not kept across the K loop
        const int nb = t.n0 >> 5, v = wave & 3;
        int64_t row = t.m0 + wave * 32 + (ln & 31);
        sv[0] = (uint32_t)((row < M ? row : M - 1) * 32 + (ln >> 5) * 16);
        sp[0] = act;
        sv[1] = (uint32_t)ln * 16;
        sp[1] = w0 + (size_t)(nb + wave) * ng * 1024;
        if (wave < 4) {
            row = t.m0 + v * 64 + (ln >> 5) * 32 + 2 * (ln & 15);
            sv[2] = (uint32_t)((((ln >> 4) & 1) * Mp + (row < Mp - 2 ? row : Mp - 2)) * 8);
            sp[2] = act + (size_t)Mp * 32;
            row = t.m0 + v * 64 + 2 * (ln & 31);
            sv[3] = (uint32_t)((row < Mp - 2 ? row : Mp - 2) * 8);
            sp[3] = act + (size_t)Mp * 48;
        } else {
            sv[2] = (uint32_t)((ln >> 5) * ng * 512 + (ln & 31) * 16);
            sp[2] = w1 + (size_t)(nb + 2 * v) * ng * 512;
            sv[3] = (uint32_t)(((ln >> 4) & 1) * ng * 256 + (ln & 15) * 16);
            sp[3] = sfr + (size_t)(nb + 2 * v) * ng * 256;
        }
    };
    auto group_request = [&](const uint32_t slot, const int i) {
        const uint32_t s = ring0 + slot;
        if (i == 0) { dma16(sp[0], sv[0], s + OFF_X0 + wave * 1024); sp[0] += gstride; }
        if (i == 1) { dma16(sp[1], sv[1], s + OFF_W0 + wave * 1024); sp[1] += 1024; }
        if (i == 2) { dma16(sp[2], sv[2], s + lds2); sp[2] += stride2; }
        if (i == 3) { dma16_half(sp[3], sv[3], s + lds3); sp[3] += stride3; }
    };
    // columns 16 ks .. 16 ks + 15 of the tile's low-rank term: h in two transfers, two rows of L2, the bias
    auto lowrank_request = [&](const Tile& t, const int ks, const uint32_t slot, const int i) {
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const uint32_t s = ring0 + slot;
        const int c0 = 16 * ks < r ? 16 * ks : 0;
        if (i < 2) {
            const int64_t left = M - 1 - t.m0;
            int row = wave * 32 + (ln & 31);
            row = row < left ? row : (int)left;
            dma16(h + t.m0 * r + c0, (uint32_t)(row * r * 4 + (2 * i + (ln >> 5)) * 16), s + OFF_H + wave * 2048 + i * 1024);
        }
        if (i == 2) {
            const int k = 2 * wave + (ln >> 5), c = l2_piece(k, ln & 31);
            const int64_t on = r ? 1 : 0;                         // r = 0: the launcher passes something readable
            dma16(L2 + on * ((int64_t)c0 * N + t.n0), (uint32_t)(k * (int)on * N * 2 + c * 16), s + OFF_L2 + wave * 1024);
        }
        if (i == 3) dma16(bias + (has_bias ? t.n0 : 0), (uint32_t)ln * 16, s + OFF_B);
    };

    // ---- operands of one group; refilled in place as the group's last tile that uses them has been issued
    struct {
        uint4 lo;
        uint2 hi, s;
    } ox[4], ow[2];
    uint32_t rd_x0, rd_x1, rd_w0, rd_w1, rd_sx, rd_sf;            // this lane's operands in the slot that is read next
    const uint32_t smask = lane < 32 ? ~0u : 0u;
    auto point_at = [&](const uint32_t slot) {
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const uint32_t s = ring0 + slot;
        rd_x0 = s + OFF_X0 + wm * 4096 + ln * 16;
        rd_w0 = s + OFF_W0 + wn * 2048 + ln * 16;
        rd_x1 = s + OFF_X1 + wm * 2048 + ln * 8;
        rd_w1 = s + OFF_W1 + wn * 1024 + ln * 8;
        // k half 1 of the scale product multiplies zeros by zeros, which switch nothing
        rd_sx = ln < 32 ? s + OFF_SX + (wm * 128 + ln) * 8 : ring0 + OFF_ZERO;
        rd_sf = ln < 32 ? s + OFF_SF + (wn * 64 + ln) * 8 : ring0 + OFF_ZERO;
    };
    auto advance = [&](const uint32_t slot) {                     // from `slot` to the one behind it
        const uint32_t d = slot == (NSLOTS - 1) * STAGE ? 0u - (NSLOTS - 1) * STAGE : STAGE, dm = d & smask;
        rd_x0 += d; rd_x1 += d; rd_w0 += d; rd_w1 += d; rd_sx += dm; rd_sf += dm;
    };
    auto fetch_x = [&](const int mi) {
        ox[mi].lo = lds_read16_pinned(rd_x0 + mi * 1024);
        ox[mi].hi = lds_read8_pinned(rd_x1 + mi * 512);
        ox[mi].s = lds_read8_pinned(rd_sx + mi * 256);
    };
    auto fetch_w = [&](const int ni) {
        ow[ni].lo = lds_read16_pinned(rd_w0 + ni * 1024);
        ow[ni].hi = lds_read8_pinned(rd_w1 + ni * 512);
        ow[ni].s = lds_read8_pinned(rd_sf + ni * 256);
    };
    float16v y[2][4], P[2], S, zero16;
#pragma unroll
    for (int i = 0; i < 16; ++i) zero16[i] = 0.0f;
    auto pmma = [&](const int t) -> float16v {
        const auto &w = ow[(t >> 2) & 1], &x = ox[t & 3];
        const int8v a = {(int)w.lo.x, (int)w.lo.y, (int)w.lo.z, (int)w.lo.w, (int)w.hi.x, (int)w.hi.y, 0, 0};
        const int8v b = {(int)x.lo.x, (int)x.lo.y, (int)x.lo.z, (int)x.lo.w, (int)x.hi.x, (int)x.hi.y, 0, 0};
        return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, zero16, 3, 3, 0, 0x7f, 0, 0x7f);
    };
    auto smma = [&](const int t) -> float16v {
        return __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(__builtin_bit_cast(short4v, ow[t >> 2].s),
                                                        __builtin_bit_cast(short4v, ox[t & 3].s), zero16, 0, 0, 0);
    };
    auto next_slot = [&](const uint32_t s) { return s == (NSLOTS - 1) * STAGE ? 0u : s + STAGE; };

    int id = blockIdx.x;
    if (!exists(id)) return;
    Tile T = tile_at(id);
    uint32_t cur = 0;                                             // slot of the tile's first low-rank stage
    int stores_counted = 0;                                       // the previous tile's 16 stores stand behind its transfers
    {
        uint32_t s = 0;
        for (int ks = 0; ks < 2; ++ks, s = next_slot(s))
#pragma unroll
            for (int i = 0; i < 4; ++i) lowrank_request(T, ks, s, i);
        set_streams(T);
        for (int g = 0; g < 3; ++g, s = next_slot(s))
#pragma unroll
            for (int i = 0; i < 4; ++i) group_request(s, i);
    }

    while (true) {
        const int nid = id + (int)gridDim.x;
        const bool more = exists(nid);                            // the last tile prefetches its own beginning again: nobody reads it
        const Tile T1 = tile_at(more ? nid : id);

        // ---- y starts as the low-rank term plus the bias
        const uint32_t slot_l1 = next_slot(cur);
        wait_left<12>(stores_counted);
        __syncthreads();
        {
            int ln = lane;
            asm volatile("" : "+v"(ln));
            const uint32_t rd_h = ring0 + OFF_H + wm * 8192 + (ln >> 5) * 1024 + (ln & 31) * 16;
            const uint32_t rd_b = ring0 + OFF_B + cur + (wn * 64 + 4 * (ln >> 5)) * 4;
            bf16x8 l2[2][2];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int ni = 0; ni < 2; ++ni) l2[ks][ni] = l2_fragment(ring0 + OFF_L2 + (ks ? slot_l1 : cur), wn * 64 + ni * 32, ln);
            lowrank_bias_of<4>(y, l2,
                               [&](const int mi, const int ks, const int half) { return lds_read16(rd_h + (ks ? slot_l1 : cur) + mi * 2048 + half * 512); },
                               [&](const int ni, const int q) { return lds_read16(rd_b + ni * 128 + q * 32); }, r, has_bias);
        }
        // group 0 is here; the low-rank stages' slots take groups 3 and 4
        wait_left<8>(stores_counted);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) group_request(cur, i);
#pragma unroll
        for (int i = 0; i < 4; ++i) group_request(slot_l1, i);
        cur = next_slot(slot_l1);
        point_at(cur);
        fetch_w(0);
#pragma unroll
        for (int mi = 0; mi < 4; ++mi) fetch_x(mi);
        P[0] = pmma(0);

        // ---- one group, in slot c.  Step t folds tile t (channel block t / 4, token block t % 4): its scale products are
        // issued, then the next tile's integer sums, and the fold runs beside the latter.  After the barrier of step 3 the
        // next group is visible to all waves and all reads of this one's slot are done: it takes a new stage.
        // KIND: 0 the tile's group g + NSLOTS, 1 the next tile's low-rank stage ks, 2 as 0 in the tile's last group.
        auto group = [&](const uint32_t c, auto KINDC, const int ks) {
            constexpr int KIND = decltype(KINDC)::value;
            auto step = [&](auto TC) {
                constexpr int t = decltype(TC)::value;
                float16v& yt = y[t >> 2][t & 3];
                S = smma(t);
                asm volatile("" : "+v"(yt) : "v"(S));
                if (t < 7 || KIND != 2) {
                    P[(t + 1) & 1] = pmma((t + 1) & 7);
                    asm volatile("" : "+v"(yt) : "v"(P[(t + 1) & 1]));
                }
                if (t == 0) fetch_w(1);
                if (t == 3) {
                    if (KIND != 2) asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
                    __syncthreads();
                    if (KIND != 2) {
                        advance(c);
                        fetch_w(0);
                    }
                }
                if (t >= 4) {
                    if (KIND != 2) fetch_x(t - 4);
                    if (KIND == 1) lowrank_request(T1, ks, c, t - 4);
                    else group_request(c, t - 4);
                }
#pragma unroll
                for (int i = 0; i < 16; ++i) yt[i] = __builtin_fmaf(P[t & 1][i], S[i], yt[i]);
                asm volatile("" : "+v"(yt));
                __builtin_amdgcn_sched_barrier(0);
            };
            step(IC<0>{}); step(IC<1>{}); step(IC<2>{}); step(IC<3>{});
            step(IC<4>{}); step(IC<5>{}); step(IC<6>{}); step(IC<7>{});
        };
        for (int g = NSLOTS; g < ng; ++g) {
            group(cur, IC<0>{}, 0);
            cur = next_slot(cur);
        }
        for (int ks = 0; ks < 2; ++ks) {
            group(cur, IC<1>{}, ks);
            cur = next_slot(cur);
        }
        set_streams(T1);
        for (int g = 0; g < 2; ++g) {
            group(cur, IC<0>{}, 0);
            cur = next_slot(cur);
        }
        group(cur, IC<2>{}, 0);
        cur = next_slot(cur);                                     // the next tile's first low-rank stage

        {
            int ln = lane;
            asm volatile("" : "+v"(ln));                          // the store's address arithmetic stays behind the K loop
            const int64_t mw = T.m0 + wm * 128;
            stores_counted = store_walked_bf16<4>(y, store0, ln, yout + mw * ldy + T.n0 + wn * 64, ldy, M - mw);
        }
        if (!more) break;
        id = nid;
        T = T1;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // nothing may still be writing this block's LDS when it ends
}

}  // namespace

// tokens [0, rows) of M, rows a multiple of 256 or M
hipError_t launch_e3m2_walk(const uint8_t* act, const void* w_packed, const float* h, const void* L2, const float* bias,
                            int64_t M, int64_t rows, int N, int K, int r, void* y, int64_t ldy, hipStream_t stream) {
    const uint8_t* base = (const uint8_t*)w_packed;
    const uint8_t* w1 = base + packed_e3m2_w0_bytes(N, K);
    // transfers have no branch: without a low-rank term or a bias they read the codes
    const float* hr = r ? h : (const float*)act;
    const uint16_t* l2 = r ? (const uint16_t*)L2 : (const uint16_t*)act;
    hipLaunchKernelGGL(gemm_e3m2_walk_kernel, dim3((unsigned)walking_blocks()), dim3(512), 0, stream,
                       act, base, w1, w1 + packed_e3m2_w1_bytes(N, K), hr, l2, bias ? bias : (const float*)act,
                       M, N, K, r, bias != nullptr, (uint16_t*)y, ldy, make_walk_grid((int)((rows + BM - 1) / BM), N / BN));
    return hipGetLastError();
}

}  // namespace svdq
