// Host-callable launchers of the gfx950 kernels (internal to the library).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace svdq {

// svdq_quantize.hip.  slices > 1: K is split between that many blocks per row block, and h receives as many partial
// h's ([slices][M, r]; their sum is h)
hipError_t launch_quantize(const void* x, int64_t ldx, const float* inv_lambda, float rho,
                           const void* l1p, int64_t M, int K, int r,
                           uint8_t* qx, float* sx, float* h, bool gelu, hipStream_t stream, int slices = 1);
hipError_t launch_gelu(const void* x, int64_t n, void* out, hipStream_t stream);
hipError_t launch_pack_l1(const void* L1, const float* inv_lambda, int K, int r, void* out, hipStream_t stream);
hipError_t launch_scale_chain(const float* a, float rho, int64_t n, float* s, float* inv, hipStream_t stream);
inline size_t packed_l1_bytes(int K) { return (size_t)(K / 64) * 4 * 2 * 64 * 16; }

// svdq_gemm.hip
size_t packed_weight_bytes(int N, int K);
size_t packed_weight_codes_bytes(int N, int K);          // the code fragments; the scale pieces follow
hipError_t launch_pack_weight(const uint8_t* qw, const float* sw, int N, int K, void* out, hipStream_t stream);
hipError_t launch_linear(const uint8_t* qx, const float* sx, const void* w_packed,
                         const float* h, const void* L2, const float* bias,
                         int64_t M, int N, int K, int r, void* y, int64_t ldy, int out_f32,
                         hipStream_t stream);
hipError_t launch_group_acc(const uint8_t* qx, const void* w_packed, int64_t M, int N, int K,
                            int64_t m0, int mt, int32_t* acc, hipStream_t stream);

// E3M2-container variant of the int4 path (svdq_quantize.hip, svdq_gemm_e3m2.hip).  The activation operand
// buffer holds, per 64-group, Mp = round_up(M, 4) rows of 56 bytes in three planes (see quantize_kernel).
constexpr int E3M2_ROW_BYTES = 56;
inline size_t act_e3m2_bytes(int64_t M, int K) { return (size_t)(K / 64) * (size_t)((M + 3) & ~(int64_t)3) * E3M2_ROW_BYTES; }
// 4-bit weights to be expanded into `out` (packed_weight_e3m2_bytes): canonical qw, sw or the nibble kernel's packed form
struct ExpandJob {
    const void *codes, *scales;
    uint8_t* out;
    int N;
    bool canonical;
};
ExpandJob expand_canonical_job(const void* qw, const void* sw, int N, void* out);
ExpandJob expand_packed_job(const void* w_packed_nibble, int N, int K, void* out);
hipError_t launch_expand(const ExpandJob& e, int K, hipStream_t stream);
// nib: the codes as nibbles too, [K/64][M][32 B] (null: not wanted).  expand: weights [N, K] that blocks of the same launch
// expand beside the pass (out null: none)
hipError_t launch_quantize_e3m2(const void* x, int64_t ldx, const float* inv_lambda, float rho,
                                const void* l1p, int64_t M, int K, int r,
                                uint8_t* act, uint8_t* nib, float* sx, float* h, bool gelu, hipStream_t stream, int slices = 1,
                                const ExpandJob& expand = ExpandJob{});
size_t packed_weight_e3m2_bytes(int N, int K);
__host__ __device__ inline size_t packed_e3m2_w0_bytes(int N, int K) { return (size_t)N * (K / 64) * 32; }     // planes of the packed weights
__host__ __device__ inline size_t packed_e3m2_w1_bytes(int N, int K) { return (size_t)N * (K / 64) * 16; }
hipError_t launch_linear_e3m2(const uint8_t* act, const void* w_packed,
                              const float* h, const void* L2, const float* bias,
                              int64_t M, int N, int K, int r, void* y, int64_t ldy, int out_f32,
                              hipStream_t stream);
// svdq_e3m2_walk.hip: tokens [0, rows) of M, rows a multiple of 256 or M; N a multiple of 256, K >= 320, bf16 y
hipError_t launch_e3m2_walk(const uint8_t* act, const void* w_packed, const float* h, const void* L2, const float* bias,
                            int64_t M, int64_t rows, int N, int K, int r, void* y, int64_t ldy, hipStream_t stream);
// svdq_e3m2_mid.hip: tiles of E3M2_MID[shape] (svdq_e3m2_plan.h), bf16 y.  slices > 1: h is as many partial h's, whose sum goes to hsum
hipError_t launch_e3m2_mid(int shape, const uint8_t* act, const void* w_packed, const float* h, int slices, float* hsum, const void* L2, const float* bias,
                           int64_t M, int N, int K, int r, void* y, int64_t ldy, hipStream_t stream);
// slices > 1: h is as many partial h's, whose sum goes to hsum; only where layer_e3m2_takes_slices says so
hipError_t launch_layer_e3m2(const uint8_t* act, const void* w_packed, const float* h, const void* L2, const float* bias,
                             int64_t M, int N, int K, int r, void* y, int64_t ldy, hipStream_t stream, int slices, float* hsum);
bool layer_e3m2_takes_slices(int64_t M, int N, int K);
hipError_t launch_linear_e3m2_next(const uint8_t* act, const void* w_packed,
                                   const float* h, const void* L2, const float* bias,
                                   int64_t M, int N, int K, int r, bool gelu,
                                   const float* next_inv_lambda, float next_rho, const void* next_l1p, int next_r,
                                   uint8_t* next_act, float* next_sx, float* next_h, hipStream_t stream);
hipError_t launch_group_acc_e3m2(const uint8_t* act, const void* w_packed, int64_t M, int N, int K,
                                 int64_t m0, int mt, int32_t* acc, hipStream_t stream);
hipError_t launch_unpack_act_e3m2(const uint8_t* act, int64_t M, int K, uint8_t* qx, hipStream_t stream);

// svdq_small.hip: the layer for few tokens
enum { SMALL_E3M2_CANONICAL = 0, SMALL_E3M2_PACKED = 1, SMALL_NIBBLE = 2, SMALL_MXFP4 = 3 };   // operand sources
constexpr int SMALL_SLICES = 8;                  // waves of a block = most partial h's the GEMM takes
// Which tile of the few-token GEMM a layer takes: 1: 32 channels x 32 tokens; 2: 64 x 64 (MXFP4: 32 x 64); 0: none, the
// tile kernels.  Measured on whole layers, K = 512 .. 13824, N = 512 .. 13824, us against the tile path (whose weights are
// expanded beside the quantise pass and whose GEMM splits K between two teams).  32 x 32 wins up to two blocks per CU
// (MXFP4, which waits for loads only: one).  64 x 64 then wins while it is one block per CU (E3M2, K = 5120: N = 512,
// M = 1536, 27 against 36; M = 2304, 288 blocks, 45 against 40), and up to two where few tokens meet many weights, which the
// tile path has to expand first (N = 13824, M = 85, 432 blocks: K = 2048 23 against 26, K = 13824 73 against 114; N = 5120,
// M = 307, even; but K = 512 16 against 15, and N = 2048, M = 960, 42 against 38).  MXFP4 expands nothing and wins up to 320
// blocks (K = 5120: N = 512, M = 2304, 30 against 35; N = 5120, M = 230, 24 against 26; M = 307, 400 blocks, 29 against 27),
// with few channels and a long K up to 384 (K = 5120, N = 1024, M = 1536, 27 against 31; K = 512 even).
// fields: the tiles find E3M2 fields with nothing to expand ahead of them, or with the layer's staging for it (packed E3M2 weights;
// svdq_layer_forward of the others).  Where a row of tiles is 48 at most they then win from 161 tokens on with more than one block per CU
// (packed, K = 11840, N = 6144, M = 178, 50 against 42; K = 7040, N = 4736, M = 205, 35 against 27; K = 3968, N = 4096, M = 384, even;
// nibbles, K = 6336, N = 5248, M = 200, 46 against 36; canonical, K = 4736, N = 6016, M = 185, 36 against 31; K = 2240, N = 4224, M = 354, even).  With more channels or fewer tokens the limit is as without them:
// nibbles lose there as often as they gain (N = 13824, M = 66, K = 2944, 28 against 32; N = 9088, M = 77, K = 5120, 36
// against 30), packed weights would gain (N = 10112, M = 123, K = 11648, 58 against 44).
inline int small_shape(int64_t M, int N, int K, bool mxfp4 = true, bool fields = false) {
    const int64_t b32 = ((M + 31) / 32) * (N / 32), b64 = ((M + 63) / 64) * ((N + 63) / 64);
    if (b32 <= (mxfp4 ? 256 : 512)) return 1;
    const int limit = mxfp4 ? (N <= 2048 && K >= 4096 ? 384 : 320) : (N >= 4096 && K >= 2048 && !(fields && M > 160 && N <= 6144)) ? 480 : 256;
    return b64 <= limit ? 2 : 0;
}
// The few-token GEMM addresses codes and weights with 32-bit byte offsets (its tokens may be the last of many).
inline bool small_reach(int64_t M, int64_t N, int64_t K) { return (M > N ? M : N) * K < (int64_t)1 << 32; }
// tokens [begin, M), M up to SVDQ_MAX_M.  w1: the scales of canonical weights (packed ones hold theirs).  hsum: receives the sum of the partial h's (null: not wanted)
hipError_t launch_small_gemm(int source, const uint8_t* codes, const void* scales, const void* w0, const void* w1,
                             const float* h, int slices, float* hsum, const void* L2, const float* bias, int64_t M, int64_t begin, int N, int K, int r,
                             void* y, int64_t ldy, hipStream_t stream);
// The whole layer in one launch (fused_layer_kernel), or FUSED_NONE: a quantise pass and a GEMM.  Every block quantises its own
// tokens, so what it takes grows with K, and sooner with a low-rank term, whose L1 fragments every block reads too; the two launches
// cost 9 to 10 us (6 of them on the host) as long as K is short.  Measured on whole layers, N = 512 .. 4096, us against the two launches:
//   up to 8 tokens, K = 2048: E3M2 6.7 against 9.8 (with a term 10.1, 9.8), MXFP4 6.5 against 9.3 (8.6, 9.4);
//   up to a 16-token tile per CU, K = 1536: M = 32 7.2 against 9.8 (10.4, 10.2), MXFP4 6.6 against 9.4 (9.1, 10.5);
//   32-token tiles, M = 256, N = 2048: K = 1024 8.0 against 9.9 (10.8, 11.4), 2048 12.3 against 11.8; MXFP4 1024 6.6 against 9.4
//   (8.8, 10.6), 2048 9.3 against 9.5 (12.7, 11.7).
// N up to 16384 with few tokens: 0.68 to 0.98 of the two launches.  More than 16 tokens with K <= 512 take as long either way (6.4 to
// 6.9 us, what the launch takes the host): 32-token tiles, whose codes need not go through LDS.
enum { FUSED_NONE = 0, FUSED_SPREAD = 1, FUSED_TILES = 2 };
// LDS of a block, bytes of its planes, one behind the other: partial tiles; with a low-rank term partial h's and h, rows FUSED_H_ROW floats
// apart; smoothing factors, halves of groups FUSED_IL_ROW floats apart; SPREAD (1 << rs tokens), per token and half group, 16 + 8 + 4 bytes
// of codes and scale and with a term the values as they are projected, 64 bytes.  The scales' plane is rounded up to 16 bytes: with one token and an
// odd number of 64-groups it is 8 K / 64, and the values behind it are read 16 bytes at a time.
constexpr int FUSED_IL_ROW = 36, FUSED_H_ROW = 36, FUSED_HPART = SMALL_SLICES * 32 * 32, FUSED_H = 32 * FUSED_H_ROW;
constexpr uint32_t LDS_OF_A_CU = 160 * 1024;
struct FusedLds {
    uint32_t tiles, hpart, h, il, lo, hi, scale, x;
    __host__ __device__ constexpr uint32_t end() const { return tiles + hpart + h + il + lo + hi + scale + x; }
};
__host__ __device__ constexpr FusedLds fused_lds(int ni, int K, bool lowrank, bool spread, int rs) {
    const uint32_t halves = (uint32_t)K / 32;
    FusedLds a{};
    a.tiles = SMALL_SLICES * ni * 4096;
    if (lowrank) a.hpart = FUSED_HPART * 4, a.h = FUSED_H * 4;
    a.il = halves * FUSED_IL_ROW * 4;
    if (spread) {
        a.lo = (halves * 16) << rs, a.hi = (halves * 8) << rs, a.scale = (((halves * 4) << rs) + 15) & ~15u;
        if (lowrank) a.x = (halves * 64) << rs;
    }
    return a;
}
inline int fused_spread(int64_t M) { return M <= 1 ? 0 : M <= 2 ? 1 : M <= 4 ? 2 : M <= 8 ? 3 : 4; }     // rs
inline int small_fused(int64_t M, int N, int K, int r, bool mxfp4) {
    const int64_t b16 = ((M + 15) / 16) * (N / 32), b32 = ((M + 31) / 32) * (N / 32);
    const bool few = M <= 8;
    // (MXFP4 with a term, 16 tokens and K = 1792: 160 640 bytes of LDS)
    if (b16 <= 256 && K <= (few ? (r ? (mxfp4 ? 2304 : 1792) : (mxfp4 ? 4352 : 3328)) : (r ? (mxfp4 ? 1792 : 1408) : (mxfp4 ? 3328 : 2560))) &&
        (few || M <= 16 || K > 512) && fused_lds(1, K, r != 0, true, fused_spread(M)).end() <= LDS_OF_A_CU)
        return FUSED_SPREAD;
    // MXFP4 without a term: from K = 2048 on the quantise pass has four slices and catches up with more tokens (M = 200, N = 2048 10.4
    // against 9.5 here, M = 500, N = 1024 9.8 against 9.9, M = 1000, N = 512 9.7 against 11.4)
    return b32 <= 512 && K <= (r ? (mxfp4 ? 1664 : 1216) : mxfp4 ? (M <= 448 ? 2048 : 1984) : 1664) ? FUSED_TILES : FUSED_NONE;
}
hipError_t launch_fused_layer(int source, const void* x, int64_t ldx, const float* inv_lambda, float rho, bool gelu, const void* l1p,
                              uint8_t* codes, void* scales, float* h, const void* w0, const void* w1,
                              const void* L2, const float* bias, int64_t M, int N, int K, int r, void* y, int64_t ldy, hipStream_t stream);
hipError_t launch_sum_slices(const float* part, int slices, int64_t M, int r, float* h, hipStream_t stream);

// svdq_mxfp4.hip
int walking_blocks();                            // blocks of a kernel that walks its tiles: one per CU, a multiple of 8
size_t packed_weight_mx_bytes(int N, int K);
inline size_t packed_mx_codes_bytes(int N, int K) { return (size_t)N * (K / 2); }
hipError_t launch_pack_weight_mx(const uint8_t* qw, const uint8_t* sw, int N, int K, void* out, hipStream_t stream);
hipError_t launch_quantize_mx(const void* x, int64_t ldx, const float* inv_lambda, float rho,
                              const void* l1p, int64_t M, int K, int r,
                              uint8_t* qx, uint8_t* sxe, float* h, bool gelu, hipStream_t stream, int slices = 1);
// tokens [0, rows) of M, rows a multiple of 256 or M
hipError_t launch_linear_mx(const uint8_t* qx, const uint8_t* sxe, const void* w_packed,
                            const float* h, const void* L2, const float* bias,
                            int64_t M, int64_t rows, int N, int K, int r, void* y, int64_t ldy, int out_f32, hipStream_t stream);
int64_t mx_main_rows(int64_t M, int N, int K, int r);   // tokens that are best left to the tile kernels; the few-token kernel takes the rest
hipError_t launch_linear_mx_next(const uint8_t* qx, const uint8_t* sxe, const void* w_packed,
                                 const float* h, const void* L2, const float* bias,
                                 int64_t M, int N, int K, int r, bool gelu,
                                 const float* next_inv_lambda, float next_rho, const void* next_l1p, int next_r,
                                 uint8_t* next_qx, uint8_t* next_sxe, float* next_h, hipStream_t stream);

// svdq_search.hip
constexpr int SQ_ERROR_PARTIALS = 1024;
hipError_t launch_sq_error(const void* yref, int64_t ldr, const void* y, int64_t ldy, int64_t M, int N,
                           double* workspace, double* out, bool add, hipStream_t stream);
hipError_t launch_sq_error_static(const void* yref, int64_t ldr, const void* y, int64_t ldy, int64_t M, int N,
                                  double* out, hipStream_t stream);
hipError_t launch_argmin_rows(const double* table, int nrows, int ncols, int32_t* idx, hipStream_t stream);

// svdq_gptq.hip (offline calibration)
size_t gptq_workspace_bytes(int N, int K);
hipError_t launch_gptq_hessian(const void* x, int64_t ldx, const float* inv_lambda, int64_t M, int K, double* H,
                               hipStream_t stream);
hipError_t launch_gptq_quantize(const float* R, const double* H, double damp, int N, int K, void* workspace,
                                uint8_t* qw, float* sw, hipStream_t stream);

// svdq_lowrank.hip
hipError_t launch_lowrank_down(const void* x, int64_t ldx, const float* inv_lambda, const void* L1,
                               int64_t M, int K, int r, float* h, hipStream_t stream);
hipError_t launch_lowrank_up(const float* h, const void* L2, int64_t M, int N, int r,
                             void* y, int64_t ldy, hipStream_t stream);

}  // namespace svdq
