// The E3M2 GEMM (svdq_gemm_e3m2.hip: operands, arithmetic) for middling numbers of tokens: tiles that leave no CU idle and no
// CU a round behind the others.
//
// Why: with 128 x 128 or 256 x 256 tiles M = 512, N = 5120 is 160 tiles and M = 2048 640 of them, 2.5 for every CU: a third of
// the chip waits for the rest.  Here a wave has 64 tokens x 96 channels (six 32 x 32 tiles: 96 accumulators beside three result
// registers and one set of operands, refilled in place as in svdq_e3m2_walk.hip), a block eight waves, two per SIMD, as
// WM (tokens) x WN (channels) x WK: WK teams, each with a ring of its own, split K.  N = 5120 then makes 216 tiles of M = 512 as
// 128 x 96 in quarters of K, of M = 1024 as 128 x 192 in halves and of M = 2048 as 256 x 192.
// Measured, GEMMs of K = N = 5120, us, 128 x 128 tiles and here: M = 1024 43.6 -> 39.6, M = 2048 73.1 -> 65.9.  What bounds it, timing
// only, M = 2048: no LDS reads in the loop 50 us, no transfers 58, neither 46 (44 ns per 32 x 32 tile, group and SIMD, what the
// instructions alone take): five operands of 2 KB are read for six tiles.  With four teams the transfers weigh more than the reads
// (12.5 KB for twelve tiles of a CU), and a tile's start and end, 8 us, are a third of M = 512.  Counters, one, two, four and eight teams
// (K = 5120; M = 2048 and 1024, N = 5120; M = 2048, N = 1024; M = 384, N = 3072): matrix pipe 37, 31, 19, 13 % busy, vector issue 31, 27,
// 23, 16 % of wave-time, waits 55, 59, 60, 70 %, HBM 2.8, 4.3, 1.8, 1.5 TB/s.
// A last tile may stand over the end of N: it re-reads the last 32 channels and stores nothing of them.
// The group counts of the teams differ by one at most: a team with fewer multiplies the group before its own by zero scales.
#include "svdq_dev.h"
#include "svdq_e3m2_plan.h"
#include "svdq_epilogue.h"
#include "svdq_kernels.h"
#include "svdq_lds.h"
#include "svdq_tiles.h"

namespace svdq {

namespace {

typedef int int8v __attribute__((ext_vector_type(8)));

template <int WM, int WN, int WK>
struct MidGeom {
    static constexpr int TW = WM * WN;                            // waves of a team
    static constexpr int BM = 64 * WM, NB = 3 * WN, BN = 32 * NB;
    // a ring slot of a team, one 64-group (byte offsets); planes in lane order as in svdq_e3m2_walk.hip
    static constexpr uint32_t OFF_X0 = 0;                         // [32-token block][half][token] x 16 B
    static constexpr uint32_t OFF_X1 = OFF_X0 + 2048 * WM;        // [32-token block][half][token] x 8 B
    static constexpr uint32_t OFF_SX = OFF_X1 + 1024 * WM;        // [token] x 8 B
    static constexpr uint32_t OFF_W0 = OFF_SX + 512 * WM;         // [n-block][lane] x 16 B
    static constexpr uint32_t OFF_W1 = OFF_W0 + 1024 * NB;        // [n-block][lane] x 8 B
    static constexpr uint32_t OFF_SF = OFF_W1 + 512 * NB;         // [n-block][channel] x 8 B
    static constexpr uint32_t STAGE = OFF_SF + 256 * NB, SLOT = WK * STAGE;
    // transfers of up to 1 KB per group and team: the planes in the order above
    static constexpr int J1 = 2 * WM, J2 = J1 + WM, J3 = J2 + (WM + 1) / 2, J4 = J3 + NB, J5 = J4 + (NB + 1) / 2, JOBS = J5 + (NB + 3) / 4;
    static constexpr int NDMA = (JOBS + TW - 1) / TW;             // per wave
    static constexpr int NS = E3M2_MID[WK == 1 ? 0 : WK == 2 ? 1 : WK == 4 ? 2 : 3].slots;
    // the last slot holds h of the tile first, [4 columns][token] x 16 B per 32 tokens
    static constexpr uint32_t LAST = SLOT > BM * 128u ? SLOT : BM * 128u;
    static constexpr uint32_t OFF_ZERO = (NS - 1) * SLOT + LAST;  // 1 KB of zeros: the scale-product operands of k half 1
    static constexpr uint32_t OFF_NONE = OFF_ZERO + 1024;         // where the transfers go that fill up a wave's count
    static constexpr uint32_t LDS = OFF_NONE + 1024;
    static_assert(LDS <= 160 * 1024, "LDS of a CU");
};

// dma16 by the lanes of a mask
__device__ __forceinline__ void dma16_masked(const void* sbase, uint32_t voff, uint32_t lds_off, uint64_t lanes) {
    const uint64_t a = (uint64_t)(uintptr_t)sbase;
    const uint64_t sa = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32)) << 32) |
                        (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    lds_off = __builtin_amdgcn_readfirstlane(lds_off);
    lanes = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(lanes >> 32)) << 32) |
            (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)lanes);
    asm volatile("s_mov_b32 m0, %2\n\ts_mov_b64 exec, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1\n\ts_mov_b64 exec, -1"
                 ::"v"(voff), "s"(sa), "s"(lds_off), "s"(lanes) : "memory");
}

template <int WM, int WN, int WK>
__global__ __launch_bounds__(512, 1)
void gemm_e3m2_mid_kernel(const uint8_t* __restrict__ act, const uint8_t* __restrict__ w0, const uint8_t* __restrict__ w1,
                          const uint8_t* __restrict__ sfr, const float* __restrict__ h, const int slices, float* __restrict__ hsum,
                          const uint16_t* __restrict__ L2, const float* __restrict__ bias,
                          int64_t M, int N, int K, int r, uint16_t* __restrict__ yout, int64_t ldy, const TileGrid tg) {
    using G = MidGeom<WM, WN, WK>;
    constexpr int TW = G::TW, NS = G::NS, NDMA = G::NDMA, MT = 2, NI = 3, NT = MT * NI;
    __shared__ __attribute__((aligned(16))) uint8_t lds[G::LDS];
    int mt, nt;
    if (!tile_of(tg, blockIdx.x, mt, nt)) return;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, kh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), team = wave / TW, tw = wave % TW, wm = tw % WM, wn = tw / WM;
    const int64_t Mp = (M + 3) & ~(int64_t)3, m0 = (int64_t)mt * G::BM;
    const int n0 = nt * G::BN, nb = n0 >> 5, nb_last = (N >> 5) - 1, ngk = K >> 6;
    // this team's groups: [first, first + ng), of which the leading `pad` (0 or 1) are the team's before it
    const int ng = (ngk + WK - 1) / WK, rem = ngk % WK, pad = rem && team >= rem ? 1 : 0;
    const int first = team * ng - (rem && team > rem ? team - rem : 0) - pad;
    const uint32_t ring0 = (uint32_t)(uintptr_t)(lds_byte*)lds, mine = ring0 + team * G::STAGE;
    if (tid < 64) *reinterpret_cast<uint4*>(lds + G::OFF_ZERO + tid * 16) = uint4{0u, 0u, 0u, 0u};

    // ---- operand transfers
    const size_t gstride = (size_t)Mp * E3M2_ROW_BYTES;
    const uint8_t* sp[NDMA];
    uint32_t sv[NDMA], sd[NDMA];
    size_t ss[NDMA];
    uint64_t sl[NDMA];
#pragma unroll
    for (int i = 0; i < NDMA; ++i) {
        const int j = tw + TW * i;
        auto at_most = [](int64_t v, int64_t m) { return v < m ? v : m; };
        auto nblock = [&](const int b) { return (uint32_t)(at_most(nb + b, nb_last) - nb); };
        sl[i] = ~0ull;
        ss[i] = gstride;
        if (j < G::J1) {
            sp[i] = act;
            sv[i] = (uint32_t)(at_most(m0 + j * 32 + l32, M - 1) * 32 + kh * 16);
            sd[i] = G::OFF_X0 + j * 1024;
        } else if (j < G::J2) {
            sp[i] = act + (size_t)Mp * 32;
            sv[i] = (uint32_t)((((lane >> 4) & 1) * Mp + at_most(m0 + (j - G::J1) * 64 + kh * 32 + 2 * (lane & 15), Mp - 2)) * 8);
            sd[i] = G::OFF_X1 + (j - G::J1) * 1024;
        } else if (j < G::J3) {
            sp[i] = act + (size_t)Mp * 48;
            sv[i] = (uint32_t)(at_most(m0 + (j - G::J2) * 128 + 2 * (WM == 1 ? l32 : lane), Mp - 2) * 8);
            sd[i] = G::OFF_SX + (j - G::J2) * 1024;
            if (WM == 1) sl[i] = 0xffffffffull;
        } else if (j < G::J4) {
            sp[i] = w0 + (size_t)(nb + (int)nblock(j - G::J3)) * ngk * 1024;
            sv[i] = (uint32_t)lane * 16;
            sd[i] = G::OFF_W0 + (j - G::J3) * 1024;
            ss[i] = 1024;
        } else if (j < G::J5) {
            const int b = 2 * (j - G::J4);
            sp[i] = w1 + (size_t)nb * ngk * 512;
            sv[i] = nblock(b + kh) * (uint32_t)ngk * 512 + l32 * 16;
            sd[i] = G::OFF_W1 + b * 512;
            ss[i] = 512;
            if (b + 1 >= G::NB) sl[i] = 0xffffffffull;
        } else if (j < G::JOBS) {
            const int b = 4 * (j - G::J5);
            sp[i] = sfr + (size_t)nb * ngk * 256;
            sv[i] = nblock(b + (lane >> 4)) * (uint32_t)ngk * 256 + (lane & 15) * 16;
            sd[i] = G::OFF_SF + b * 256;
            ss[i] = 256;
            if (b + 4 > G::NB) sl[i] = (1ull << (16 * (G::NB % 4))) - 1;
        } else {
            sp[i] = act;
            sv[i] = 0;
            sd[i] = G::OFF_NONE;
            ss[i] = 0;
            sl[i] = 1;
        }
        sp[i] += (size_t)first * ss[i];
    }
    auto request = [&](const uint32_t slot, const int i) {
        const uint32_t to = (tw + TW * i >= G::JOBS) ? ring0 + G::OFF_NONE : slot + sd[i];
        dma16_masked(sp[i], sv[i], to, sl[i]);
        sp[i] += ss[i];
    };
    // h of the tile's tokens is asked for first: loads return in order
    constexpr int HP = G::BM * 8 / 512;                           // pieces of 16 bytes per thread, r = 32
    const int sh = r > 16 ? 3 : 2;                                // a row of h is 1 << sh pieces
    float4 hp[HP];
    if (r > 0 && slices <= 1) {
#pragma unroll
        for (int j = 0; j < HP; ++j) {
            const int v = j * 512 + tid, t = v >> sh < G::BM ? v >> sh : G::BM - 1, q = v & ((1 << sh) - 1);
            hp[j] = *reinterpret_cast<const float4*>(h + (m0 + t < M ? m0 + t : M - 1) * r + 4 * q);
        }
    } else if (r > 0) {
#pragma unroll
        for (int j = 0; j < HP; ++j) {
            const int v = j * 512 + tid, t = v >> sh < G::BM ? v >> sh : G::BM - 1, q = v & ((1 << sh) - 1);
            hp[j] = sum_of_slices(h, slices, M * r, (m0 + t < M ? m0 + t : M - 1) * r + 4 * q);
        }
    }
    for (int g = 0; g < NS - 1; ++g)
#pragma unroll
        for (int i = 0; i < NDMA; ++i) request(mine + g * G::SLOT, i);

    // ---- y starts as the low-rank term plus the bias, in the first team; h, the sum of its slices, through the last slot
    float16v y[NI][MT], P[2], S, zero16;
#pragma unroll
    for (int i = 0; i < 16; ++i) zero16[i] = 0.0f;
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int mi = 0; mi < MT; ++mi) y[ni][mi] = zero16;
    uint8_t* const hbuf = lds + (NS - 1) * G::SLOT;
    if (r > 0) {
#pragma unroll
        for (int j = 0; j < HP; ++j) {
            const int v = j * 512 + tid, t = v >> sh, q = v & ((1 << sh) - 1);
            if (t < G::BM) {
                *reinterpret_cast<float4*>(hbuf + (t >> 5) * 4096 + q * 512 + (t & 31) * 16) = hp[j];
                if (slices > 1 && nt == 0 && m0 + t < M) *reinterpret_cast<float4*>(hsum + (m0 + t) * r + 4 * q) = hp[j];
            }
        }
    }
    __syncthreads();
    if (team == 0) {
        const int nw = n0 + wn * 96;
        add_lowrank_bias_from<NI, MT, true>(y, [&](const int mi, const int k) {
            return *reinterpret_cast<const float4*>(hbuf + (wm * 2 + mi) * 4096 + (k >> 2) * 512 + l32 * 16);
        }, L2, bias, nw, N, r, lane, N - 32);
    }
    auto wait_groups = [&](const int k) {                         // until at most k groups of this wave's transfers are outstanding
        if (k <= 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        else if (k == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NDMA) : "memory");
        else if (k == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NDMA) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * NDMA) : "memory");
    };
    wait_groups(NS - 2);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NDMA; ++i) request(mine + (NS - 1) * G::SLOT, i);

    // ---- operands of one group; refilled in place
    struct {
        uint4 lo;
        uint2 hi, s;
    } ox[MT], ow[NI];
    uint32_t rd_x0 = mine + G::OFF_X0 + wm * 2048 + lane * 16, rd_x1 = mine + G::OFF_X1 + wm * 1024 + lane * 8;
    uint32_t rd_w0 = mine + G::OFF_W0 + wn * 3072 + lane * 16, rd_w1 = mine + G::OFF_W1 + wn * 1536 + lane * 8;
    // k half 1 of the scale product multiplies zeros by zeros, which switch nothing
    uint32_t rd_sx = kh ? ring0 + G::OFF_ZERO : mine + G::OFF_SX + (wm * 64 + l32) * 8;
    uint32_t rd_sf = kh ? ring0 + G::OFF_ZERO : mine + G::OFF_SF + (wn * 96 + l32) * 8;
    const uint32_t smask = kh ? 0u : ~0u;
    auto advance = [&](const uint32_t slot) {                     // from `slot` to the one behind it
        const uint32_t d = slot == (NS - 1) * G::SLOT ? 0u - (NS - 1) * G::SLOT : G::SLOT, dm = d & smask;
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
    auto pmma = [&](const int t) -> float16v {
        const auto &w = ow[t >> 1], &x = ox[t & 1];
        const int8v a = {(int)w.lo.x, (int)w.lo.y, (int)w.lo.z, (int)w.lo.w, (int)w.hi.x, (int)w.hi.y, 0, 0};
        const int8v b = {(int)x.lo.x, (int)x.lo.y, (int)x.lo.z, (int)x.lo.w, (int)x.hi.x, (int)x.hi.y, 0, 0};
        return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, zero16, 3, 3, 0, 0x7f, 0, 0x7f);
    };
    auto smma = [&](const int t) -> float16v {
        return __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(__builtin_bit_cast(short4v, ow[t >> 1].s),
                                                        __builtin_bit_cast(short4v, ox[t & 1].s), zero16, 0, 0, 0);
    };
    fetch_w(0);
    fetch_x(0);
    fetch_x(1);
    fetch_w(1);
    if (pad) ox[0].s = ox[1].s = uint2{0u, 0u};                   // the group before this team's: nothing of it
    P[0] = pmma(0);

    // One group, in slot c.  Step t folds tile t (channel block t / 2, token block t % 2): its scale products are issued, then
    // the next tile's integer sums, and the fold runs beside the latter.  Behind the barrier of step 2 the next group is visible to
    // the team and this one's slot is free: it takes group g + NS.  KIND: 0 that one exists, 1 the next group does, 2 the last one.
    auto group = [&](const uint32_t c, const int left, auto KINDC) {
        constexpr int KIND = decltype(KINDC)::value;
        auto step = [&](auto TC) {
            constexpr int t = decltype(TC)::value;
            float16v& yt = y[t >> 1][t & 1];
            S = smma(t);
            asm volatile("" : "+v"(yt) : "v"(S));
            if (t < NT - 1 || KIND != 2) {
                P[(t + 1) & 1] = pmma((t + 1) % NT);
                asm volatile("" : "+v"(yt) : "v"(P[(t + 1) & 1]));
            }
            if (t == 0) fetch_w(2);
            if (t == 2 && KIND != 2) {
                if (KIND == 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 2) * NDMA) : "memory");
                else wait_groups(left);
                __syncthreads();
                advance(c);
                fetch_w(0);
            }
            if (KIND != 2) {
                if (t == 3) fetch_w(1);
                if (t >= 4) fetch_x(t - 4);
            }
            if (KIND == 0 && t >= 2) {
                constexpr int PER = (NDMA + 3) / 4;
#pragma unroll
                for (int i = (t - 2) * PER; i < (t - 1) * PER && i < NDMA; ++i) request(mine + c, i);
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) yt[i] = __builtin_fmaf(P[t & 1][i], S[i], yt[i]);
            asm volatile("" : "+v"(yt));
            __builtin_amdgcn_sched_barrier(0);
        };
        step(IC<0>{}); step(IC<1>{}); step(IC<2>{}); step(IC<3>{}); step(IC<4>{}); step(IC<5>{});
    };
    auto next_slot = [&](const uint32_t s) { return s == (NS - 1) * G::SLOT ? 0u : s + G::SLOT; };
    uint32_t cur = 0;
    int g = 0;
    for (; g + NS < ng; ++g, cur = next_slot(cur)) group(cur, 0, IC<0>{});
    for (; g + 1 < ng; ++g, cur = next_slot(cur)) group(cur, ng - 2 - g, IC<1>{});
    group(cur, 0, IC<2>{});

    // ---- the teams' tiles meet in LDS, in halves: [wave of the half][quad of registers][lane] x 16 B
    auto quad = [&](const int q) -> float4 {
        const float16v& t = y[q >> 3][(q >> 2) & 1];
        return float4{t[4 * (q & 3)], t[4 * (q & 3) + 1], t[4 * (q & 3) + 2], t[4 * (q & 3) + 3]};
    };
#pragma unroll
    for (int half = WK / 2; half >= 1; half >>= 1) {
        __syncthreads();                                          // operands, or the sums before, have been read
        float4* const part = reinterpret_cast<float4*>(lds) + (size_t)((team % half) * TW + tw) * (24 * 64) + lane;
        if (team >= half && team < 2 * half) {
#pragma unroll
            for (int q = 0; q < 24; ++q) part[q * 64] = quad(q);
        }
        __syncthreads();
        if (team < half) {
#pragma unroll
            for (int q = 0; q < 24; ++q) {
                const float4 v = part[q * 64];
                float16v& t = y[q >> 3][(q >> 2) & 1];
                t[4 * (q & 3)] += v.x;
                t[4 * (q & 3) + 1] += v.y;
                t[4 * (q & 3) + 2] += v.z;
                t[4 * (q & 3) + 3] += v.w;
            }
        }
    }
    if (WK == 1) __syncthreads();
    if (team != 0) return;
    // ---- store: 32 tokens x 96 channels at a time through a region of the wave's own (rows of 192 bytes and 16 of padding),
    // then 16 bytes per lane, twelve lanes a token.  (The regions lie over what a smaller team handed over; only its readers write here.)
    constexpr uint32_t ROW = 208;
    static_assert(TW * 32 * ROW <= G::LDS, "the waves' regions");
    if (WK > 1) {                                                 // the first team's waves read each other's regions' place
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    const uint32_t region = ring0 + (WK > 1 ? tw * (24 * 64 * 16) : tw * (32 * ROW));
    const int nw = n0 + wn * 96;
#pragma unroll
    for (int mi = 0; mi < MT; ++mi) {
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float16v& t = y[ni][mi];
                lds_write8_pinned(region + l32 * ROW + (ni * 32 + 8 * q + 4 * kh) * 2,
                                  uint2{f2_bf16_rne(t[4 * q], t[4 * q + 1]), f2_bf16_rne(t[4 * q + 2], t[4 * q + 3])});
            }
        const int64_t mw = m0 + wm * 64 + mi * 32;
#pragma unroll
        for (int it = 0; it < 6; ++it) {
            const int v = it * 64 + lane, row = v / 12, c = v - row * 12;
            const uint4 o = lds_read16_pinned(region + row * ROW + c * 16);
            if (mw + row < M && nw + c * 8 < N) *reinterpret_cast<uint4*>(yout + (mw + row) * ldy + nw + c * 8) = o;
        }
    }
}

}  // namespace

hipError_t launch_e3m2_mid(int shape, const uint8_t* act, const void* w_packed, const float* h, int slices, float* hsum, const void* L2, const float* bias,
                           int64_t M, int N, int K, int r, void* y, int64_t ldy, hipStream_t stream) {
    const uint8_t* base = (const uint8_t*)w_packed;
    const uint8_t* w1 = base + packed_e3m2_w0_bytes(N, K);
    auto go = [&](auto kern, const E3m2Mid& m) {
        const TileGrid tg = make_tile_grid((int)((M + m.bm - 1) / m.bm), (N + m.bn - 1) / m.bn);
        hipLaunchKernelGGL(kern, dim3((unsigned)tile_ids(tg)), dim3(512), 0, stream, act, base, w1, w1 + packed_e3m2_w1_bytes(N, K),
                           h, slices, hsum, (const uint16_t*)L2, bias, M, N, K, r, (uint16_t*)y, ldy, tg);
    };
    switch (shape) {
        case 0: go(gemm_e3m2_mid_kernel<4, 2, 1>, E3M2_MID[0]); break;
        case 1: go(gemm_e3m2_mid_kernel<2, 2, 2>, E3M2_MID[1]); break;
        case 2: go(gemm_e3m2_mid_kernel<2, 1, 4>, E3M2_MID[2]); break;
        default: go(gemm_e3m2_mid_kernel<1, 1, 8>, E3M2_MID[3]); break;
    }
    return hipGetLastError();
}

}  // namespace svdq
