// GPTQ on the residual weights (Sec. III-B: the residual branch of the SVDQuant split is quantised with GPTQ
// instead of round-to-nearest).  Offline calibration, not part of the per-step path.
//
// The algorithm in its column-sequential form: weights are visited in the order k = 0..K-1; a visited weight is
// rounded to the int4 grid of its (channel, 64-group) scale and its rounding error is spread over the not yet
// visited weights of the same channel in proportion to row k of the inverse Hessian of the layer-wise objective
// ||X^ (R - R^)||^2 (H = X^T X^ plus damping), from which index k is then eliminated.  Everything runs in
// binary64; every update is one fused multiply-subtract per element and pivot, in pivot order, which is the definition
// that a CPU reference repeats bit for bit (one that rounds the products as well agrees on ordinary Hessians, but at
// condition numbers of 1e13 scales differ and at 1e15 codes), and there are no reductions other than max and one
// sequential sum.  The published implementation factors H^-1 once (Cholesky) and reads the same numbers off the
// factor; this form trades that for elementwise kernels: K^3 updates for the inverse, K^3 / 3 of H^-1 and K^2 N / 2
// of the weights during the visit, taken in panels of 64 pivots (below), two to four at a time, so that the matrices cross
// HBM once per 128 to 256 pivots.
#include <climits>
#include <type_traits>

#include "svdq_dev.h"
#include "svdq_kernels.h"
#include "svdq_lds.h"

namespace svdq {

namespace {

typedef double double4v __attribute__((ext_vector_type(4)));

// The matrix instruction both parts of this file lean on: D = A B + C of 16 x 4 by 4 x 16 in binary64, lane l holding
// A[l % 16][l / 16], B[l / 16][l % 16] and, in register i, C[4 i + l / 16][l % 16].  It forms each element as a chain of
// four fused multiply-adds in k order, rounding after each (2000 random products, exponents 2^-10 .. 2^10, no
// difference from that chain): a sequence of these instructions IS the scalar sequence of updates.
__device__ __forceinline__ double4v mfma_f64(double a, double b, double4v c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// ---- H += X^T X^, X^ = x * inv_lambda in binary32 (eq. 5), products and sums in binary64.
// H's contribution is symmetric, so only tiles on and above the diagonal are formed and each is added twice.  A block
// owns one tile of 16 T x 16 T and its WV waves split the tokens (four per step, one per 16 lanes); the waves' sums meet
// in LDS in a fixed order.  The operands come straight from global memory: lane (j, kq) = (l % 16, l / 16) takes the T
// neighbouring channels T j .. T j + T - 1 of token 4 step + kq, which are row (or column) j of T different matrix
// tiles, so a load feeds T^2 instructions and there is nothing to stage or wait for together.  Bound by the matrix
// instruction (64 clocks each, 78.6 TFLOP/s; the vector unit has the same rate, but not the registers to feed itself
// without LDS traffic).  T = 4 with four waves (two per SIMD); T = 2 with sixteen waves where that leaves CUs idle.
// K = 5120, 8192 tokens: 19.6 ms for the full square on the vector unit.
template <int T, bool ALIGNED>
struct XLoad {
    uint32_t w[T / 2];
    __device__ __forceinline__ void load(const uint16_t* p) {
        if constexpr (ALIGNED && T == 4) {
            const uint2 v = *reinterpret_cast<const uint2*>(p);
            w[0] = v.x;
            w[1] = v.y;
        } else if constexpr (ALIGNED) {
            w[0] = *reinterpret_cast<const uint32_t*>(p);
        } else {
#pragma unroll
            for (int i = 0; i < T / 2; ++i) w[i] = (uint32_t)p[2 * i] | ((uint32_t)p[2 * i + 1] << 16);
        }
    }
    __device__ __forceinline__ void values(const float (&il)[T], double (&v)[T]) const {
#pragma unroll
        for (int i = 0; i < T / 2; ++i) {
            v[2 * i] = (double)__fmul_rn(bf16lo_f(w[i]), il[2 * i]);
            v[2 * i + 1] = (double)__fmul_rn(bf16hi_f(w[i]), il[2 * i + 1]);
        }
    }
};

template <int T, int WV, bool ALIGNED>
__global__ __launch_bounds__(64 * WV, T == 4 ? 2 : 1)
void hessian_kernel(const uint16_t* __restrict__ x, int64_t ldx, const float* __restrict__ inv_lambda,
                    int64_t M, int K, double* __restrict__ H) {
    constexpr int BT = 16 * T;
    __shared__ double tile[BT][BT + 1];
    int tb = (int)((sqrtf(8.0f * (float)blockIdx.x + 1.0f) - 1.0f) * 0.5f);      // column of tiles; ta <= tb
    while (tb * (tb + 1) / 2 > (int)blockIdx.x) --tb;
    while ((tb + 1) * (tb + 2) / 2 <= (int)blockIdx.x) ++tb;
    const int ta = (int)blockIdx.x - tb * (tb + 1) / 2;
    const int a0 = ta * BT, b0 = tb * BT;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j = lane & 15, kq = lane >> 4;
    float ila[T], ilb[T];
#pragma unroll
    for (int i = 0; i < T; ++i) {
        ila[i] = inv_lambda[a0 + T * j + i];
        ilb[i] = inv_lambda[b0 + T * j + i];
    }
    double4v acc[T][T];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int k = 0; k < T; ++k) acc[i][k] = double4v{0.0, 0.0, 0.0, 0.0};
    const int64_t steps = (M + 3) / 4;                      // a step is four tokens; wave w takes steps w, w + WV, ...
    const uint16_t* pa = x + a0 + T * j;
    const uint16_t* pb = x + b0 + T * j;
    constexpr int U = 4;                                    // steps requested together, one batch ahead of their use
    XLoad<T, ALIGNED> xa[2][U], xb[2][U];
    auto request = [&](const int64_t s0, const int buf) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            int64_t m = 4 * (s0 + u * WV) + kq;
            if (m >= M) m = M - 1;                          // the values are replaced by zeros when they are used
            xa[buf][u].load(pa + m * ldx);
            xb[buf][u].load(pb + m * ldx);
        }
    };
    auto multiply = [&](const int64_t s0, const int buf) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            double va[T], vb[T];
            xa[buf][u].values(ila, va);
            xb[buf][u].values(ilb, vb);
            if (4 * (s0 + u * WV) + 4 > M) {
                const bool in = 4 * (s0 + u * WV) + kq < M;
#pragma unroll
                for (int i = 0; i < T; ++i) {
                    va[i] = in ? va[i] : 0.0;
                    vb[i] = in ? vb[i] : 0.0;
                }
            }
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int k = 0; k < T; ++k) acc[i][k] = mfma_f64(va[i], vb[k], acc[i][k]);
        }
    };
    request(wave, 0);
    for (int64_t s = wave; s < steps; s += 2 * U * WV) {
        request(s + U * WV, 1);
        multiply(s, 0);
        request(s + 2 * U * WV, 0);
        multiply(s + U * WV, 1);
    }
    for (int w = 0; w < WV; ++w) {
        if (wave == w) {
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int k = 0; k < T; ++k)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        double& t = tile[T * (4 * e + kq) + i][T * j + k];
                        t = (w == 0) ? acc[i][k][e] : t + acc[i][k][e];
                    }
        }
        __syncthreads();
    }
    for (int e = threadIdx.x; e < BT * BT; e += 64 * WV) {
        const int r = e / BT, c = e % BT;
        H[(size_t)(a0 + r) * K + b0 + c] += tile[r][c];
        if (ta != tb) H[(size_t)(b0 + r) * K + a0 + c] += tile[c][r];
    }
}

// ---- preparation: binary64 copies, dead channels, damping with the diagonal summed in index order
constexpr int DIAG_CHUNK = 4096;
__global__ __launch_bounds__(256)
void diag_sum_kernel(const double* __restrict__ H, double damp, int K, double* __restrict__ add) {
    __shared__ double dg[DIAG_CHUNK];
    double s = 0.0;
    for (int k0 = 0; k0 < K; k0 += DIAG_CHUNK) {
        const int n = min(DIAG_CHUNK, K - k0);
        for (int k = threadIdx.x; k < n; k += 256) {
            const double d = H[(size_t)(k0 + k) * K + k0 + k];
            dg[k] = d == 0.0 ? 1.0 : d;
        }
        __syncthreads();
        if (threadIdx.x == 0)
#pragma unroll 16
            for (int k = 0; k < n; ++k) s = __dadd_rn(s, dg[k]);       // one chain of additions: the definition's order
        __syncthreads();
    }
    if (threadIdx.x == 0) *add = __dmul_rn(damp, __ddiv_rn(s, (double)K));
}
__global__ __launch_bounds__(256)
void prepare_kernel(const float* __restrict__ R, const double* __restrict__ H, const double* __restrict__ add, int N, int K,
                    double* __restrict__ A, double* __restrict__ W) {
    const int k = blockIdx.x;                                          // one row of H and of R
    const double d = H[(size_t)k * K + k], dd = __dadd_rn(d == 0.0 ? 1.0 : d, *add);
    for (int j = threadIdx.x; j < K; j += 256) A[(size_t)k * K + j] = (j == k) ? dd : H[(size_t)k * K + j];
    for (int n = threadIdx.x; n < N; n += 256) W[(size_t)k * N + n] = (d == 0.0) ? 0.0 : (double)R[(size_t)k * N + n];
}

// ---- Panel-blocked form of both eliminations.  Every element of H^-1 (and of W) must receive, in the order of the
// pivots, one fused multiply-subtract per pivot: that sequence per element is the definition, and it does not say WHEN
// an element is touched.  Pivots are taken in panels of PB = 64, two launches per panel:
//   panel kernel   brings the panel's own rows and columns (2 x 64 x K elements, for the weights 64 x N) through all 64
//                  pivots.  A row outside the panel only needs the panel's 64 x 64 diagonal block as it stood at each
//                  pivot (the tables below), and a column likewise, so the rows and columns are independent of each
//                  other.  The pivots' columns and scaled rows, as they stood when taken, are saved.
//   rank update    everything else receives its updates from the saved columns and rows, in pivot order, on the
//                  binary64 matrix instruction.  Block 0 meanwhile brings the NEXT panel's diagonal block up to date, takes
//                  it through its own 64 dependent steps and leaves the next panel's tables: a serial chain of about
//                  30 us (32 with the launch's start and end), which no launch is shorter than.
// Only the strips (rows and columns) of the next panel have to be up to date when a launch ends.  The rest of the matrices
// receives the updates of a whole batch of two to four panels in one pass over memory, and its blocks are dealt over the
// launches of the next batch in whole rounds of one block per CU, beside the strips and the chain.  So at any time the
// rest lacks up to two batches, which is what the rings of saved rows and columns hold, and a strip is brought up from
// where the rest stands.  The diagonal block after the next one is brought up a panel early by a block of its own, so that
// the chain begins with 64 updates instead of 512.
// Same result as the pivot-by-pivot form bit for bit.  K = N = 5120: with a launch per pivot and step (25 600 of them)
// 112 ms; updates of the rest behind every panel 19.56 ms, behind every second one (two passes of 155 us over the
// inverse per 256 pivots, the others of 49 us waiting for the chain) 18.88, behind every fourth one, in rounds, 16.07:
// 78 us each of the inverse's 80 launches, 44 to 162 the visit's.  (K = N = 512: 1.07 -> 1.05, 2048: 4.65 -> 4.20, 4096:
// 11.85 -> 10.78; with panels, chains and batches as they are now 0.72, 2.96, 9.08, and 14.94 for 5120.)  What bounds it: the matrix unit, 246e9 fused
// multiply-subtracts (8.2 ms at the 60 TFLOP/s that a loop of these instructions reaches), and the serial path of a panel:
// its kernel (9 us with a block per CU at most, 18 at K = 5120) and the chain (30 us).
constexpr int PB = 64;
constexpr int MAX_BATCH = 4;                     // panels whose updates of the rest are put off and done together, at most
constexpr int RING_PANELS = 2 * MAX_BATCH;       // whose saved rows and columns are kept; a power of two

// ---- A vector of 64 elements (one row or column of the panel) lives in 16 lanes (a DPP row), four elements each.
// Pivot 4 it + k is always element k of the row's lane 0: after every four pivots the vectors turn by one lane, so the
// loop body needs no lane index of its own.  sl = (lane + it) % 16 is the place of a lane's four elements.
template <int CTRL>
__device__ __forceinline__ double dpp64(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
}
__device__ __forceinline__ double row_first(double v) { return dpp64<0x150>(v); }             // row_newbcast:0
__device__ __forceinline__ double row_turn(double v) { return dpp64<0x120 + 15>(v); }         // row_ror:15: from lane + 1

// a / d, correctly rounded, from y = RN(1 / d): two corrections of a y.  The first makes the quotient faithful, and
// from a faithful quotient and a correctly rounded reciprocal the second gives the rounded quotient (Markstein's
// theorem), as long as nothing leaves the exponent range; `far` collects whether anything may have (far_out), and the callers
// then repeat the whole panel with SLOW, the division itself.  (A branch at every division would cost more than the
// division: it ends the overlap of one vector's chain with the next one's.)  d and y: reciprocal_of below.
template <bool SLOW>
__device__ __forceinline__ double divide_by(double a, double d, double y, uint32_t& far) {
    if (SLOW) return __ddiv_rn(a, d);
    double q = a * y;
    q = __builtin_fma(__builtin_fma(-d, q, a), y, q);
    q = __builtin_fma(__builtin_fma(-d, q, a), y, q);
    // twice the quotient's upper word from that of 2^-600 on: up to that of 2^600 further, or 0 / d (the callers look at y)
    const uint32_t above = ((uint32_t)(__builtin_bit_cast(uint64_t, q) >> 32) << 1) - (423u << 21), t = a == 0.0 ? 0u : above;
    far = t > far ? t : far;
    return q;
}
__device__ __forceinline__ bool far_out(uint32_t far) { return far >= (1201u << 21); }
// RN(1 / d), or NaN where d is too large or small for divide_by
__device__ __forceinline__ double reciprocal_of(double d) {
    const double y = __ddiv_rn(1.0, d);
    return (fabs(d) >= 0x1p-200 && fabs(d) <= 0x1p200) ? y : __builtin_nan("");
}
// wait for this wave's LDS traffic, then for the other waves: stores to global memory stay in flight
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// What a panel kernel needs of its diagonal block D (K-major q = pivot inside the panel)
struct PanelTables {
    double R[PB][PB];      // R[q][t] = D[q][t] / d_q when pivot q was taken
    double C[PB][PB];      // C[q][t] = D[t][q] then
    double D[PB][PB];      // the block after its 64 pivots
    double d[PB], y[PB];   // pivots and their reciprocals
};

// The diagonal block through its 64 pivots, 512 threads: lane group g = tid / 16 holds rows 2 g and 2 g + 1, so pivots
// 4 it + 2 p and 4 it + 2 p + 1 are the rows of group 2 it + p.  INV: in-place Gauss-Jordan inverse (see below); otherwise only the
// rows and columns behind the pivot are updated (row q of D is then the row as it stood at pivot q).  Rt: PB x PB in LDS, ds: 2 in LDS.
// A group takes its own rows through its own two pivots, which need nothing of the others; these take both behind one barrier.
// What bounds it is the number of instructions of the wave that has the pivots: with four rows a group (256 threads) and
// a barrier per pivot the block takes 37 us alone, with one per four pivots 34, and so 28.
template <bool INV, bool SLOW>
__device__ __forceinline__ bool diagonal_pass(double (&x)[2][4], double (*Rt)[PB], double (*ds)[2], PanelTables* __restrict__ out) {
    const int grp = threadIdx.x >> 4, pos = threadIdx.x & 15;
    uint32_t far = 0;
#pragma unroll 1
    for (int it = 0; it < 16; ++it) {
        const int sl = (pos + it) & 15;
        // pivot q = 4 it + k, its scaled row r, on this group's rows; OWN: it is the group's row k % 2
        auto eliminate = [&](auto OWNC, const int k, const double c0, const double c1, const double d, const double y, const double (&r)[4]) {
            constexpr bool OWN = decltype(OWNC)::value;
            const int q = 4 * it + k;
            if (pos == 0) *reinterpret_cast<double2*>(&out->C[q][2 * grp]) = double2{c0, c1};
            if (INV) {
                // the two rows' new elements of column q, in the even lanes and in the odd ones; the pivot's own is 1 / d
                const double e = divide_by<SLOW>(OWN && (pos & 1) == (k & 1) ? 1.0 : -(pos & 1 ? c1 : c0), d, y, far);
#pragma unroll
                for (int v = 0; v < 2; ++v)
#pragma unroll
                    for (int j = 0; j < 4; ++j) x[v][j] = OWN && v == (k & 1) ? r[j] : __builtin_fma(v ? -c1 : -c0, r[j], x[v][j]);
                const double e1 = dpp64<0x151>(e);                           // row_newbcast:1
                x[0][k] = pos == 0 ? e : x[0][k];
                x[1][k] = pos == 0 ? e1 : x[1][k];
            } else if (OWN || 2 * grp > q) {
#pragma unroll
                for (int v = OWN ? (k & 1) + 1 : 0; v < 2; ++v)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const double u = __builtin_fma(v ? -c1 : -c0, r[j], x[v][j]);
                        x[v][j] = (4 * sl + j > q) ? u : x[v][j];
                    }
            }
        };
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            if (grp == 2 * it + p) {
#pragma unroll
                for (int k = 2 * p; k < 2 * p + 2; ++k) {
                    double r[4];
                    const double c0 = row_first(x[0][k]), c1 = row_first(x[1][k]);
                    const double d = k & 1 ? c1 : c0, y = reciprocal_of(d);
                    far = y == y ? far : ~0u;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        r[j] = divide_by<SLOW>(x[k & 1][j], d, y, far);
                        Rt[4 * it + k][4 * sl + j] = r[j];
                    }
                    if (pos == 0) {
                        ds[4 * it + k][0] = d;
                        ds[4 * it + k][1] = y;
                    }
                    eliminate(std::true_type{}, k, c0, c1, d, y, r);
                }
            }
            lds_barrier();
            if (grp != 2 * it + p) {
#pragma unroll
                for (int k = 2 * p; k < 2 * p + 2; ++k) {
                    double r[4];
                    const double d = ds[4 * it + k][0], y = ds[4 * it + k][1];
#pragma unroll
                    for (int j = 0; j < 4; ++j) r[j] = Rt[4 * it + k][4 * sl + j];
                    const double c0 = row_first(x[0][k]), c1 = row_first(x[1][k]);
                    eliminate(std::false_type{}, k, c0, c1, d, y, r);
                }
            }
        }
#pragma unroll
        for (int v = 0; v < 2; ++v)
#pragma unroll
            for (int j = 0; j < 4; ++j) x[v][j] = row_turn(x[v][j]);
    }
    return far_out(far);
}
template <bool INV>
__device__ __forceinline__ void diagonal_block(double (&x)[2][4], double (*Rt)[PB], double (*ds)[2], int* redo, PanelTables* __restrict__ out) {
    const int grp = threadIdx.x >> 4, pos = threadIdx.x & 15;
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int j = 0; j < 4; ++j) out->D[2 * grp + v][4 * pos + j] = x[v][j];       // kept for a second pass
    if (threadIdx.x == 0) *redo = 0;                                  // ahead of the pass's barriers
    if (diagonal_pass<INV, false>(x, Rt, ds, out)) *redo = 1;
    __syncthreads();
    if (*redo) {
#pragma unroll
        for (int v = 0; v < 2; ++v)
#pragma unroll
            for (int j = 0; j < 4; ++j) x[v][j] = out->D[2 * grp + v][4 * pos + j];
        __syncthreads();
        diagonal_pass<INV, true>(x, Rt, ds, out);
        __syncthreads();
    }
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            out->D[2 * grp + v][4 * pos + j] = x[v][j];
            out->R[2 * grp + v][4 * pos + j] = Rt[2 * grp + v][4 * pos + j];
        }
    if (threadIdx.x < PB) {
        out->d[threadIdx.x] = ds[threadIdx.x][0];
        out->y[threadIdx.x] = ds[threadIdx.x][1];
    }
}

// The panel's first tables: nothing precedes them that could carry them along.
template <bool INV>
__global__ __launch_bounds__(512)
void first_tables_kernel(const double* __restrict__ D, size_t ld, PanelTables* __restrict__ out) {
    __shared__ __attribute__((aligned(16))) double Rt[PB][PB], ds[PB][2];
    __shared__ int redo;
    const int grp = threadIdx.x >> 4, pos = threadIdx.x & 15;
    double x[2][4];
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int j = 0; j < 4; ++j) x[v][j] = D[(size_t)(2 * grp + v) * ld + 4 * pos + j];
    diagonal_block<INV>(x, Rt, ds, &redo, out);
}

// Panel kernels: a vector for each of a block's 16 lane groups.  What bounds them is the chain of a vector's 64 pivots (a broadcast,
// five operations of a division, an update) and the instructions beside it on a wave that has its SIMD for itself: the
// table is read an iteration of four pivots ahead of its use and holds the NEGATED values, what is to be saved stays in
// registers (lane `it` keeps iteration it's) and nothing branches.  Two vectors to a group halve the reads of the table, but take
// longer than two blocks on a CU; K = N = 512, 2048, 5120 0.92, 3.74, 15.34 ms with two, 0.84, 3.46, 15.09 with one (three: 0.99, 4.04,
// 15.8; two, read where they are used, masked and saved pivot by pivot: 1.04, 4.18, 16.05, a panel of 15 to 25 us).
constexpr int PVECS = 16;
__device__ __forceinline__ void load_table(double (*to)[PB], const double (*from)[PB]) {
    for (int e = threadIdx.x * 2; e < PB * PB; e += 512) {
        const double2 v = *reinterpret_cast<const double2*>(&from[0][0] + e);
        *reinterpret_cast<double2*>(&to[0][0] + e) = double2{-v.x, -v.y};
    }
}
// (d, y) of the panel's pivots; whether any of them has no reciprocal that divide_by can use.  A barrier.
__device__ __forceinline__ bool load_pivots(double (*ds)[2], const PanelTables* __restrict__ tb) {
    int odd = 0;
    if (threadIdx.x < PB) {
        const double y = tb->y[threadIdx.x];
        ds[threadIdx.x][0] = tb->d[threadIdx.x];
        ds[threadIdx.x][1] = y;
        odd = y != y;
    }
    return __syncthreads_or(odd) != 0;
}
struct TableRows {                               // four pivots' rows at a lane's four places, and (d, y)
    double t[4][4], d[4], y[4];
    __device__ __forceinline__ void load(const double (*tab)[PB], const double (*ds)[2], const int it, const int sl) {
        auto pair = [](const double* p, double& a, double& b) {
            const u32x4 v = *reinterpret_cast<const volatile __attribute__((address_space(3))) u32x4*>((const lds_byte*)p);
            a = __builtin_bit_cast(double, (uint64_t)v.x | ((uint64_t)v.y << 32));
            b = __builtin_bit_cast(double, (uint64_t)v.z | ((uint64_t)v.w << 32));
        };
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            pair(ds[4 * it + k], d[k], y[k]);
            pair(&tab[4 * it + k][4 * sl], t[k][0], t[k][1]);
            pair(&tab[4 * it + k][4 * sl + 2], t[k][2], t[k][3]);
        }
    }
};
// body(it, rows) for the 16 iterations, the vector x turned behind each
template <class Body>
__device__ __forceinline__ void panel_iterations(const double (*tab)[PB], const double (*ds)[2], double (&x)[4], Body body) {
    const int pos = threadIdx.x & 15;
    TableRows rows[2];
    rows[0].load(tab, ds, 0, pos);
    auto one = [&](const int it, const TableRows& now, TableRows& next) {
        next.load(tab, ds, (it + 1) & 15, (pos + it + 1) & 15);
        body(it, now);
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = row_turn(x[j]);
    };
#pragma unroll 1
    for (int it = 0; it < 16; it += 2) {
        one(it, rows[0], rows[1]);
        one(it + 1, rows[1], rows[0]);
    }
}

// ---- in-place Gauss-Jordan inverse without pivoting.  Step p: d = A[p][p], col = A[:, p], row = A[p, :] / d;
// A[a][j] -= col[a] row[j] elsewhere, A[p][j] = row[j], A[a][p] = -col[a] / d, A[p][p] = 1 / d.
// Blocks 0 .. nb - 1: PVECS rows outside the panel; nb .. 2 nb - 1: columns outside it.
// Saves LT[q][a] = column of pivot p0 + q, Rr[q][j] = its scaled row.
__global__ __launch_bounds__(256)
void gj_panel_kernel(double* __restrict__ A, int K, int p0, const PanelTables* __restrict__ tb,
                     double* __restrict__ LT, double* __restrict__ Rr) {
    __shared__ __attribute__((aligned(16))) double tab[PB][PB], ds[PB][2];
    const int nb = (K - PB) / PVECS;
    const int grp = threadIdx.x >> 4, pos = threadIdx.x & 15;
    const bool rows = (int)blockIdx.x < nb;
    double x[4];
    int idx = ((int)blockIdx.x - (rows ? 0 : nb)) * PVECS + grp;
    if (idx >= p0) idx += PB;
    auto load = [&]() {
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = rows ? A[(size_t)idx * K + p0 + 4 * pos + j] : A[(size_t)(p0 + 4 * pos + j) * K + idx];
    };
    load();
    load_table(tab, rows ? tb->R : tb->C);
    const bool slow = load_pivots(ds, tb);
    double keep[4] = {};
    auto pass = [&](auto ROWS, auto SLOWC) {
        constexpr bool R = decltype(ROWS)::value;
        uint32_t far = 0;
        panel_iterations(tab, ds, x, [&](const int it, const TableRows& tr) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const double c = row_first(x[k]);
                const double e = divide_by<decltype(SLOWC)::value>(R ? -c : c, tr.d[k], tr.y[k], far), f = R ? c : e;
#pragma unroll
                for (int j = 0; j < 4; ++j) x[j] = __builtin_fma(f, tr.t[k][j], x[j]);
                x[k] = (pos == 0) ? e : x[k];
                keep[k] = (pos == it) ? f : keep[k];
            }
        });
        return far_out(far);
    };
    auto run = [&](auto ROWS) {
        if (__any(pass(ROWS, std::false_type{}) || slow)) {
            load();
            pass(ROWS, std::true_type{});
        }
    };
    if (rows) run(std::true_type{});
    else run(std::false_type{});
    double* const save = rows ? LT : Rr;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        save[(size_t)(4 * pos + j) * K + idx] = keep[j];
        if (rows) A[(size_t)idx * K + p0 + 4 * pos + j] = x[j];
        else A[(size_t)(p0 + 4 * pos + j) * K + idx] = x[j];
    }
}

// ---- one panel of the visit: indices i0 .. i0 + 63 = one 64-group.  For each index i: code and error of every
// channel, the error spread over the panel's later weights, index i eliminated from H^-1 (A[a][b] -= A[a][i] (A[i][b] / d)
// for a, b > i).  Blocks 0 .. nr - 1: PVECS rows of A behind the panel; nr .. 2 nr - 1: columns; the rest: channels
// of W.  Saves, per pivot q, what the rank updates need: HcT[q][a] = A[a][i], HrT[q][b] = A[i][b],
// T[q][b] = A[i][b] / d, Err[q][n].  The panel's own rows and columns of A and W are not read again, and what a pivot leaves in
// places up to its own is of no use: a vector is updated as a whole.
__global__ __launch_bounds__(256)
void visit_panel_kernel(const double* __restrict__ A, const double* __restrict__ W, int N, int K, int i0,
                        const PanelTables* __restrict__ tb,
                        double* __restrict__ HcT, double* __restrict__ HrT, double* __restrict__ T, double* __restrict__ Err,
                        uint8_t* __restrict__ qw, float* __restrict__ sw) {
    __shared__ __attribute__((aligned(16))) double tab[PB][PB], ds[PB][2];
    const int i1 = i0 + PB, nr = (K - i1) / PVECS;
    const int grp = threadIdx.x >> 4, pos = threadIdx.x & 15;
    const int role = ((int)blockIdx.x < nr) ? 0 : ((int)blockIdx.x < 2 * nr) ? 1 : 2;      // rows, columns, channels
    double x[4];
    int idx = (role < 2 ? i1 : 0) + ((int)blockIdx.x - role * nr) * PVECS + grp;
    const bool live = role < 2 || idx < N;
    if (!live) idx = N - 1;                               // taken along, not stored
    auto load = [&]() {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            x[j] = role == 0 ? A[(size_t)idx * K + i0 + 4 * pos + j] : role == 1 ? A[(size_t)(i0 + 4 * pos + j) * K + idx]
                                                                                 : W[(size_t)(i0 + 4 * pos + j) * N + idx];
    };
    load();
    load_table(tab, role == 0 ? tb->R : role == 1 ? tb->C : tb->D);
    const bool slow = load_pivots(ds, tb);
    if (role == 2) {
        double a = fmax(fmax(fabs(x[0]), fabs(x[1])), fmax(fabs(x[2]), fabs(x[3])));
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) a = fmax(a, __shfl_xor(a, o));
        const float s = __fdiv_rn((float)a, 7.0f), ys = s > 0.0f ? __fdiv_rn(1.0f, s) : 0.0f;
        const bool odd = s != 0.0f && !(s >= 0x1p-60f && s <= 0x1p60f);      // not for the quotients below
        if (pos == 0 && live) sw[(size_t)(i0 >> 6) * N + idx] = s;
        double keep[4] = {};
        uint32_t codes = 0;
        auto pass = [&](auto SLOWC) {
            constexpr bool SLOW = decltype(SLOWC)::value;
            uint32_t far = 0;
            bool large = false;
            panel_iterations(tab, ds, x, [&](const int it, const TableRows& tr) {
                uint32_t cd = 0;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const double w = row_first(x[k]);
                    const float wf = (float)w;
                    float c;
                    if (SLOW) {
                        c = fminf(fmaxf(rintf(__fdiv_rn(wf, s)), -8.0f), 7.0f);
                        c = (s > 0.0f) ? c : 0.0f;
                    } else {
                        // wf / s as in divide_by, in binary32 (a scale of 0 has ys = 0: code 0).  One below 2^-40, where the corrections may not
                        // be exact, is rounded to 0 all the same; a large or not finite wf is left to SLOW.
                        float q = wf * ys;
                        q = __builtin_fmaf(__builtin_fmaf(-s, q, wf), ys, q);
                        q = __builtin_fmaf(__builtin_fmaf(-s, q, wf), ys, q);
                        large |= !(fabsf(wf) < 0x1p60f);
                        c = fminf(fmaxf(rintf(q), -8.0f), 7.0f);
                    }
                    cd |= ((uint32_t)(int)c & 15u) << (4 * k);
                    const double e = divide_by<SLOW>(__builtin_fma(-(double)c, (double)s, w), tr.d[k], tr.y[k], far);   // code x scale is exact
#pragma unroll
                    for (int j = 0; j < 4; ++j) x[j] = __builtin_fma(tr.t[k][j], e, x[j]);
                    keep[k] = (pos == it) ? e : keep[k];
                }
                codes = (pos == it) ? cd : codes;
            });
            return far_out(far) || large;
        };
        if (__any(pass(std::false_type{}) || odd || slow)) {
            load();
            pass(std::true_type{});
        }
        if (!live) return;
#pragma unroll
        for (int k = 0; k < 4; ++k) Err[(size_t)(4 * pos + k) * N + idx] = keep[k];
        // four codes: two bytes, low nibble = even index
        *reinterpret_cast<uint16_t*>(qw + (size_t)idx * (K >> 1) + (i0 >> 1) + 2 * pos) = (uint16_t)codes;
        return;
    }
    double keep_c[4] = {}, keep_f[4] = {};
    auto pass = [&](auto COLS, auto SLOWC) {
        constexpr bool C = decltype(COLS)::value;
        uint32_t far = 0;
        panel_iterations(tab, ds, x, [&](const int it, const TableRows& tr) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const double c = row_first(x[k]);
                const double f = C ? divide_by<decltype(SLOWC)::value>(c, tr.d[k], tr.y[k], far) : c;
#pragma unroll
                for (int j = 0; j < 4; ++j) x[j] = __builtin_fma(f, tr.t[k][j], x[j]);
                keep_c[k] = (pos == it) ? c : keep_c[k];
                if (C) keep_f[k] = (pos == it) ? f : keep_f[k];
            }
        });
        return far_out(far);
    };
    if (role == 0) {
        pass(std::false_type{}, std::false_type{});
    } else if (__any(pass(std::true_type{}, std::false_type{}) || slow)) {
        load();
        pass(std::true_type{}, std::true_type{});
    }
    double* const save = role == 0 ? HcT : HrT;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        save[(size_t)(4 * pos + k) * K + idx] = keep_c[k];
        if (role == 1) T[(size_t)(4 * pos + k) * K + idx] = keep_f[k];
    }
}

// ---- X[a][b] <- (..(X[a][b] - L[q][a] R[q][b]) - L[q + 1][a] R[q + 1][b]).. over the pivots q of panels [base, to) that an
// element has not had yet, in order, for rows a0 + [0, rows) and columns b0 + [0, cols), leaving out the nskip indices from
// skip_a (rows) and skip_b (columns) on (rows and cols count what is left) and the 64 x 64 block at (hole, hole).  L and R are
// rings of RING_PANELS panels' pivots, [64 RING_PANELS][ld].  own (the inverse): an element whose row or column belongs to
// panel p of [base, to) stands as the panel kernel of p left it: it is to have the panels behind p.
struct RankUpdate {
    double* X;
    const double *L, *R;
    size_t ldx, ldl, ldr;
    int a0, rows, b0, cols, skip_a, skip_b, nskip, hole;
    int base, to;
    int own;
    int shape;                   // what a block of eight waves takes: 0: 128 x 256, 64 x 64 a wave; 1: 64 rows x 256, 32 x 64 a wave;
                                 // 2: 256 rows x 64; 3: 64 x 64, 16 x 64 a wave on four waves; 4, 5: half of 1, 2, 16 x 64 a wave;
                                 // 6: half of 0, 32 x 64 a wave
    int tiles_a, tiles_b, tiles; // blocks along a and b, and of this launch (shapes 0 and 6: ids, a multiple of 8)
    int first, count;            // this launch's blocks (shapes 0 and 6)
};
constexpr int MAX_UPDATES = 6;
struct RankUpdates {
    RankUpdate u[MAX_UPDATES];
};
__device__ __forceinline__ int first_pending(int base, int to, int own, int pa, int pb) {
    int from = base;
    if (own && pa >= base && pa < to) from = pa + 1;
    if (own && pb >= from && pb < to) from = pb + 1;
    return from;
}
// The next panel's diagonal block (panel s of A), for the first block of a rank update: brought up to panel `to` from L
// and R (nothing to bring: it is `prev`'s), then through its own pivots (mode 1: inverse, 2: visit) into `next`.  Also puts the
// finished diagonal block `prev` of the current panel (at p0) in place; null: nothing to put.
struct Lookahead {
    double* A;
    const double *L, *R;
    const PanelTables* prev;
    PanelTables* next;
    int from, to, K, p0, s0, mode;
};

// acc[i][k]: a wave's 16 NI x 64 elements through the pivots of panels [from, to); lane (j, kq) = (l % 16, l / 16) holds in acc[i][k][e]
// row 16 i + 4 e + kq, column wave_col(j, k): two neighbouring columns per lane, so that a row's accesses are 256
// contiguous bytes of 16 bytes a lane.  Operands straight from global memory (L2): 64 x 64 elements per wave and 4
// pivots are 16 matrix instructions (1024 clocks) on 6 loads, the next four pivots' requested while they run.
__device__ __forceinline__ int wave_col(int j, int k) { return 32 * (k >> 1) + 2 * j + (k & 1); }
// the two values at p[0], p[1] (second: p + d1, for a matrix whose rows are not 16-byte aligned)
template <bool PAIR>
__device__ __forceinline__ double2 load2(const double* p, int d1) {
    if constexpr (PAIR) return *reinterpret_cast<const double2*>(p);
    return double2{p[0], p[d1]};
}
template <int NI, bool PAIR>
__device__ __forceinline__ void update_chain(const int from, const int to, double4v (&acc)[NI][4], const double* __restrict__ L, size_t ldl,
                                             const double* __restrict__ R, size_t ldr, int lane, const int (&col)[2], const int (&d1)[2]) {
    const int j = lane & 15, kq = lane >> 4;
    double a[2][NI];
    double2 b[2][2];
    const int steps = (to - from) * (PB / 4);
    auto request = [&](const int s, const int buf) {
        const int q = ((from * PB + 4 * s) & (RING_PANELS * PB - 1)) + kq;
#pragma unroll
        for (int i = 0; i < NI; ++i) a[buf][i] = -L[(size_t)q * ldl + 16 * i + j];
#pragma unroll
        for (int i = 0; i < 2; ++i) b[buf][i] = load2<PAIR>(R + (size_t)q * ldr + col[i], d1[i]);
    };
    auto multiply = [&](const int buf) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[i][k] = mfma_f64(a[buf][i], (k & 1) ? b[buf][k >> 1].y : b[buf][k >> 1].x, acc[i][k]);
    };
    request(0, 0);
    for (int s = 0; s < steps; s += 2) {
        request(s + 1, 1);
        multiply(0);
        if (s + 2 < steps) request(s + 2, 0);
        multiply(1);
    }
}

__device__ __forceinline__ void look_ahead(const Lookahead& la, double (*Rt)[PB], double (*ds)[2], int* redo) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, j = lane & 15, kq = lane >> 4;
    if (la.prev)
        for (int e = tid; e < PB * PB; e += 512) la.A[(size_t)(la.p0 + e / PB) * la.K + la.p0 + e % PB] = la.prev->D[e / PB][e % PB];
    if (la.mode == 0) return;
    const int grp = tid >> 4, pos = tid & 15;
    double x[2][4];
    if (la.from < la.to) {
        if (wave < 4) {                                     // 16 rows each
            double4v acc[1][4];
            const double* X = la.A + (size_t)(la.s0 + 16 * wave) * la.K + la.s0;
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[0][k][e] = X[(size_t)(4 * e + kq) * la.K + wave_col(j, k)];
            const int col[2] = {2 * j, 32 + 2 * j}, d1[2] = {1, 1};
            update_chain<1, true>(la.from, la.to, acc, la.L + la.s0 + 16 * wave, (size_t)la.K, la.R + la.s0, (size_t)la.K, lane, col, d1);
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int e = 0; e < 4; ++e) Rt[16 * wave + 4 * e + kq][wave_col(j, k)] = acc[0][k][e];
        }
        __syncthreads();
#pragma unroll
        for (int v = 0; v < 2; ++v)
#pragma unroll
            for (int i = 0; i < 4; ++i) x[v][i] = Rt[2 * grp + v][4 * pos + i];
        __syncthreads();
    } else {
#pragma unroll
        for (int v = 0; v < 2; ++v)
#pragma unroll
            for (int i = 0; i < 4; ++i) x[v][i] = la.prev->D[2 * grp + v][4 * pos + i];
    }
    if (la.mode == 1) diagonal_block<true>(x, Rt, ds, redo, la.next);
    else diagonal_block<false>(x, Rt, ds, redo, la.next);
}

// a wave's 16 NI x 64 elements at row ia, column ib of what u leaves in
template <int NI, bool PAIR>
__device__ __forceinline__ void rank_update_wave(const RankUpdate& u, const int ia, const int ib, const int lane) {
    const int j = lane & 15, kq = lane >> 4;
    if (ia >= u.rows || ib >= u.cols) return;
    int ga = u.a0 + ia, gb = u.b0 + ib;                     // a wave's rows and columns do not straddle what is left out
    if (ga >= u.skip_a) ga += u.nskip;
    if (gb >= u.skip_b) gb += u.nskip;
    if ((ga & ~(PB - 1)) == u.hole && gb == u.hole) return;
    const int from = first_pending(u.base, u.to, u.own, ga / PB, gb / PB);
    if (from >= u.to) return;
    double* X = u.X + (size_t)ga * u.ldx;
    double4v acc[NI][4];
    int col[2], d1[2];                                      // a column beyond the matrix re-reads one that exists
    bool in[2][2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int c = ib + 32 * k + 2 * j;
        in[k][0] = c < u.cols;
        in[k][1] = c + 1 < u.cols;
        col[k] = in[k][0] ? gb + 32 * k + 2 * j : gb;
        d1[k] = in[k][1] ? 1 : 0;
    }
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const double2 v = load2<PAIR>(X + (size_t)(16 * i + 4 * e + kq) * u.ldx + col[k], d1[k]);
                acc[i][2 * k][e] = v.x;
                acc[i][2 * k + 1][e] = v.y;
            }
    update_chain<NI, PAIR>(from, u.to, acc, u.L + ga, u.ldl, u.R, u.ldr, lane, col, d1);
    // the stores' addresses are formed again here; kept from the loads they would spill
#pragma unroll
    for (int k = 0; k < 2; ++k) asm volatile("" : "+v"(col[k]));
#pragma unroll
    for (int k = 0; k < 2; ++k)
        if (in[k][0]) {
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    double* to = X + (size_t)(16 * i + 4 * e + kq) * u.ldx + col[k];
                    if constexpr (PAIR) {
                        *reinterpret_cast<double2*>(to) = double2{acc[i][2 * k][e], acc[i][2 * k + 1][e]};
                    } else {
                        to[0] = acc[i][2 * k][e];
                        if (in[k][1]) to[1] = acc[i][2 * k + 1][e];
                    }
                }
        }
}

// Block 0 looks ahead; the others take blocks of the matrices of `us`, in turn.  Every element of the rest is read and
// written once per batch of panels, 16 bytes: the matrix unit bounds it (K = 5120, four panels, 256 updates: 220 us a batch at its
// rate, and 420 MB, 70 us at the rate of a copy).  A round of 128 x 256 blocks takes 19 us for 64 updates, 76 for 256.
template <bool PAIR>
__global__ __launch_bounds__(512, 1)
void rank_update_kernel(const RankUpdates us, const Lookahead la) {
    __shared__ __attribute__((aligned(16))) double Rt[PB][PB], ds[PB][2];
    __shared__ int redo;
    if (blockIdx.x == 0) {
        look_ahead(la, Rt, ds, &redo);
        return;
    }
    int t = (int)blockIdx.x - 1, which = 0;
    while (which < MAX_UPDATES - 1 && t >= us.u[which].tiles) t -= us.u[which++].tiles;
    const RankUpdate u = us.u[which];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (u.shape == 0 || u.shape == 6) {
        // consecutive block ids go to the 8 XCDs in turn: an XCD takes a run of consecutive blocks, numbered in groups of
        // eight along a, about 8 x 3 blocks whose L and R (256 and 512 KB a block) stay in its L2
        const int chunk = u.tiles >> 3, n = (int)(blockIdx.x & 7) * chunk + (t >> 3);
        if (n >= u.count) return;
        const int m = u.first + n, sm = m / (8 * u.tiles_b), rem = m - sm * (8 * u.tiles_b);
        const int width = u.tiles_a - 8 * sm < 8 ? u.tiles_a - 8 * sm : 8, tb = rem / width, ta = 8 * sm + rem - tb * width;
        if (u.shape == 0) rank_update_wave<4, PAIR>(u, ta * 128 + (wave >> 2) * 64, tb * 256 + (wave & 3) * 64, lane);
        else rank_update_wave<2, PAIR>(u, ta * 64 + (wave >> 2) * 32, tb * 256 + (wave & 3) * 64, lane);
    } else if (u.shape >= 3) {
        const bool flat = u.shape == 4;
        rank_update_wave<1, PAIR>(u, flat ? (wave >> 1) * 16 : t * 128 + wave * 16, flat ? t * 128 + (wave & 1) * 64 : 0, lane);
    } else {
        const bool flat = u.shape == 1;
        rank_update_wave<2, PAIR>(u, flat ? (wave >> 2) * 32 : t * 256 + wave * 32, flat ? t * 256 + (wave & 3) * 64 : 0, lane);
    }
}

// an update's blocks, all of them
RankUpdate whole(RankUpdate u) {
    const int over_b[] = {256, 256, 64, 64, 128, 64, 256}, over_a[] = {128, 64, 256, 64, 64, 128, 64};
    u.tiles_b = (u.cols + over_b[u.shape] - 1) / over_b[u.shape];
    u.tiles_a = (u.rows + over_a[u.shape] - 1) / over_a[u.shape];
    u.count = (u.rows > 0 && u.cols > 0 && u.base < u.to) ? u.tiles_b * u.tiles_a : 0;
    u.tiles = u.shape == 0 || u.shape == 6 ? (u.count + 7) / 8 * 8 : u.count;
    return u;
}
// `count` of them, behind the first `done` (or ahead of the last `done`)
RankUpdate part_of(RankUpdate u, int done, int count, bool backwards) {
    u = whole(u);
    u.first = backwards ? u.count - done - count : done;
    u.count = count;
    u.tiles = (count + 7) / 8 * 8;
    return u;
}
// How many of the `pending` blocks of a batch the next of `launches` launches takes, each of which has `fixed` blocks besides:
// what fills whole rounds of `cus` blocks, as few of them as the batch needs (with room for the looking-ahead block and for
// the ids that part_of adds: an XCD is given every eighth id, and one more than it has CUs is another round).
int quota(int pending, int launches, int fixed, int cus) {
    fixed += 16;
    const int64_t all = pending + (int64_t)launches * fixed, slots = (int64_t)launches * cus;
    const int take = (int)((all + slots - 1) / slots) * cus - fixed;
    return launches <= 1 || take > pending ? pending : take < 0 ? 0 : take;
}

// One block per CU (with the kernel's own 33 KB more than half of its LDS), so that the block that looks ahead has its CU
// for itself: beside another its dependent steps take twice as long, as both want the binary64 unit (100 us instead of 50 when they
// stood on fewer waves; 30 alone by now).
constexpr unsigned RANK_UPDATE_LDS = 52 * 1024;

void launch_rank_updates(const RankUpdates& us, const Lookahead& la, hipStream_t stream) {
    bool pair = true;                                  // rows aligned to 16 bytes: two columns per access
    int blocks = 1;
    for (const RankUpdate& u : us.u) {
        blocks += u.tiles;
        if (u.tiles) pair = pair && u.ldx % 2 == 0 && u.ldr % 2 == 0;
    }
    auto kern = pair ? rank_update_kernel<true> : rank_update_kernel<false>;
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(512), RANK_UPDATE_LDS, stream, us, la);
}

// Panels in a batch.  A long one passes over memory less often and fills its rounds better, but a launch waits for the
// strips, which lack up to two batches: with four panels 38 us where one that waits for the chain takes 32 to 33.  A launch of the inverse
// takes, us, those 33, or its share of the batch's rounds of 128 x 256 blocks (19 per 64 pivots), or half of that where blocks of half the size fit it;
// where the lengths are even the longest is taken.  K = N, batches of 2, 3 and 4 of the inverse, ms: 2048 3.18, 3.15, 3.32, 3072 5.55,
// 5.46, 5.71, 3584 6.97, 7.38, 7.14, 4096 9.77, 9.31, 9.82, 4480 11.6, 11.2, 12.1, 5120 15.9, 15.3, 15.0.
// What is left of the visit shrinks from panel to panel: 2, 3, 4: K = N = 2048 3.11, 3.12, 3.32, 4096 9.79, 9.59, 9.82, 5120 15.34, 14.92, 15.02.
// From some 6000 indices on the passes over memory weigh most, and both take four.  N = 5120, inverse and visit 3 and 3, 4 and 3, 4 and 4:
// 6144 22.4, 23.1, 23.0, 6656 27.7, 27.1, 26.9, 8192 46.2, 44.7, 44.0, 9344 65.8, 63.3, 62.6, 13824 177, 170, 167.
constexpr int LONG_K = 6144;
inline int visit_batch(int K) { return K > LONG_K ? MAX_BATCH : 3; }
int inverse_batch(int K, int cus) {
    if (K > LONG_K) return MAX_BATCH;
    int best = 2;
    double least = 1e30;
    for (int n = 2; n <= MAX_BATCH; ++n) {
        const int rows = K - (n + 1) * PB > 0 ? K - (n + 1) * PB : 0, blocks = (rows + 127) / 128 * ((rows + 255) / 256);
        const int rounds = (blocks + n * (K / 128 + 17) + cus - 1) / cus;
        double c = 2 * blocks / n + K / 64 + 20 <= cus ? 9.5 * n + 2.0 : 19.0 * (rounds > n ? rounds : n);
        if (c < 33.0) c = 33.0;
        if (c <= least) {
            least = c;
            best = n;
        }
    }
    return best;
}

inline size_t up256(size_t v) { return (v + 255) & ~(size_t)255; }

}  // namespace

size_t gptq_workspace_bytes(int N, int K) {
    return up256((size_t)K * K * 8) + up256((size_t)K * N * 8) + 3 * up256((size_t)K * RING_PANELS * PB * 8) +
           up256((size_t)RING_PANELS * PB * N * 8) + 2 * up256(sizeof(PanelTables)) + 256;
}

hipError_t launch_gptq_hessian(const void* x, int64_t ldx, const float* inv_lambda, int64_t M, int K, double* H,
                               hipStream_t stream) {
    const bool aligned = (reinterpret_cast<uintptr_t>(x) & 7) == 0 && ldx % 4 == 0;
    const int n64 = K / 64, n32 = K / 32;
    const unsigned tiles64 = (unsigned)(n64 * (n64 + 1) / 2), tiles32 = (unsigned)(n32 * (n32 + 1) / 2);
    const bool large = tiles64 >= 512;                      // two 64 x 64 tiles for every compute unit
    auto go = [&](auto kern, unsigned blocks, unsigned threads) {
        hipLaunchKernelGGL(kern, dim3(blocks), dim3(threads), 0, stream, (const uint16_t*)x, ldx, inv_lambda, M, K, H);
    };
    if (large && aligned) go(hessian_kernel<4, 4, true>, tiles64, 256);
    else if (large) go(hessian_kernel<4, 4, false>, tiles64, 256);
    else if (aligned) go(hessian_kernel<2, 16, true>, tiles32, 1024);
    else go(hessian_kernel<2, 16, false>, tiles32, 1024);
    return hipGetLastError();
}

hipError_t launch_gptq_quantize(const float* R, const double* H, double damp, int N, int K, void* workspace,
                                uint8_t* qw, float* sw, hipStream_t stream) {
    uint8_t* p = (uint8_t*)workspace;
    double* A = (double*)p;        p += up256((size_t)K * K * 8);
    double* W = (double*)p;        p += up256((size_t)K * N * 8);
    // saved by the panels, in a ring of two batches
    constexpr size_t RING = (size_t)RING_PANELS * PB;
    double* Lc = (double*)p;       p += up256((size_t)K * RING * 8);       // pivot columns         [RING][K]
    double* Rr = (double*)p;       p += up256((size_t)K * RING * 8);       // scaled pivot rows     [RING][K]
    double* Hr = (double*)p;       p += up256((size_t)K * RING * 8);       // rows of H^-1          [RING][K]
    double* Err = (double*)p;      p += up256(RING * N * 8);               // errors of the panels  [RING][N]
    PanelTables* tabs[2];                                              // this panel's and the next one's
    for (auto& t : tabs) {
        t = (PanelTables*)p;
        p += up256(sizeof(PanelTables));
    }
    double* add = (double*)p;                                          // the damping term
    hipLaunchKernelGGL(diag_sum_kernel, dim3(1), dim3(256), 0, stream, H, damp, K, add);
    hipLaunchKernelGGL(prepare_kernel, dim3(K), dim3(256), 0, stream, R, H, add, N, K, A, W);
    const size_t ldk = (size_t)K, ldn = (size_t)N;
    int span = inverse_batch(K, walking_blocks());
    constexpr int ALL = INT_MAX;                       // nothing left out
    const int np = K / PB;
    auto slot = [](int panel) { return (size_t)(panel % RING_PANELS) * PB; };
    // rows [a0, a0 + rows) x columns [b0, b0 + cols) of what is left of the inverse (own), the visited inverse or the weights
    auto update = [&](double* X, const double* L, const double* R, size_t ldx, bool own, int shape, int base, int to,
                      int a0, int rows, int skip_a, int b0, int cols, int skip_b, int nskip, int hole) {
        return RankUpdate{X, L, R, ldx, ldk, ldx, a0, rows, b0, cols, skip_a, skip_b, nskip, hole, base < 0 ? 0 : base, to, own, shape, 1, 1, 0, 0, 0};
    };
    const RankUpdate none = update(A, Lc, Rr, ldk, false, 0, 0, 0, 0, 0, ALL, 0, 0, ALL, 0, -1);
    const int cus = walking_blocks();
    // what panel t's strips have had when it is their turn; its diagonal block, a panel earlier (the one that a batch of
    // updates of the rest would otherwise touch meanwhile is left out of that, as the batch's `hole`)
    auto strip_base = [&](int t) { return t % span ? (t / span - 1) * span : t - 2 * span; };
    auto diag_base = [&](int t) { return (t - 1) % span == 0 ? t - 1 - 2 * span : strip_base(t); };
    // panel t's diagonal block up to panel t - 1, so that only that one's pivots stand ahead of its own
    auto early = [&](int t) { return whole(update(A, Lc, Rr, ldk, false, 3, diag_base(t), t - 1, t * PB, PB, ALL, t * PB, PB, ALL, 0, -1)); };
    // The strips have up to two batches ahead of them, 512 updates, 76 us, at most where a wave has 32 rows of them, 38 where it has 16 (the
    // looking ahead takes 30): in twice the blocks (shape + 3), where those open no round of their own
    auto thin_strips = [&](int others, int length) { return others + length / 128 + 20 <= cus ? 3 : 0; };
    // The same of the rest, for a batch that is less than a round of blocks per launch: 38 us instead of 76.  (With batches of four, without the two
    // rules K = N = 1536 takes 3.57 ms, with the first 3.37, with both 3.15; without batches 3.32.)
    auto rest_shape = [&](int blocks, int launches, int length) { return 2 * blocks / launches + length / 128 + 20 <= cus ? 6 : 0; };
    int cur = 0;                                       // tabs[cur]: the current panel's
    int done_a = 0, done_w = 0;                        // blocks of the batch's updates that its launches have had
    hipLaunchKernelGGL(first_tables_kernel<true>, dim3(1), dim3(512), 0, stream, A, ldk, tabs[cur]);
    for (int b = 0; b < np; ++b) {                     // the inverse, one panel of pivots at a time
        const int p0 = b * PB, t = b + 1, batch = b / span * span;
        const bool back = batch / span & 1;
        if (np > 1)
            hipLaunchKernelGGL(gj_panel_kernel, dim3(2 * (K - PB) / PVECS), dim3(256), 0, stream, A, K, p0, tabs[cur],
                               Lc + slot(b) * ldk, Rr + slot(b) * ldk);
        RankUpdates us{{none, none, none, none, none, none}};
        Lookahead la{A, Lc, Rr, tabs[cur], tabs[cur ^ 1], b, t, K, p0, t * PB, 1};
        if (t < np) {
            const int s0 = t * PB, base = strip_base(t);
            const int left = batch * PB, nleft = K - left < (span + 1) * PB ? K - left : (span + 1) * PB;
            const int launches = (batch + span < np ? span : np - 1 - batch) - (b - batch);   // the last launch of all is below
            RankUpdate rest = update(A, Lc, Rr, ldk, true, 0, batch - span, batch, 0, K - nleft, left, 0, K - nleft, left, nleft,
                                     (batch + span + 1) * PB);
            rest.shape = rest_shape(whole(rest).count, launches + (b - batch), 2 * (K - PB));
            if (b == batch) done_a = 0;
            const int na = whole(rest).count - done_a, thin = thin_strips(na / launches, 2 * (K - PB));
            us.u[0] = whole(update(A, Lc, Rr, ldk, true, 1 + thin, base, t, s0, PB, ALL, 0, K - PB, s0, PB, -1));
            us.u[1] = whole(update(A, Lc, Rr, ldk, true, 2 + thin, base, t, 0, K - PB, s0, s0, PB, ALL, PB, -1));
            if (t + 1 < np) us.u[2] = early(t + 1);
            const int n = quota(na, launches, us.u[0].tiles + us.u[1].tiles + us.u[2].tiles, cus);
            us.u[3] = part_of(rest, done_a, n, back);
            done_a += n;
        } else {
            // everything that is pending; the first diagonal block of the visit is looked ahead for
            const int base = batch + 1 < np ? batch : batch - span;                 // a last batch of one panel had no launch before
            us.u[0] = whole(update(A, Lc, Rr, ldk, true, 0, base, t, 0, K, ALL, 0, K, ALL, 0, 0));
            la.from = base > 0 ? base : 1;                                           // panel 0 is behind its own pivots
            la.s0 = 0;
            la.mode = 2;
        }
        launch_rank_updates(us, la, stream);
        cur ^= 1;
    }
    span = visit_batch(K);
    for (int b = 0; b < np; ++b) {                     // the weights, one panel (= one 64-group) at a time
        const int i0 = b * PB, t = b + 1, i1 = i0 + PB, rest = K - i1, batch = b / span * span;
        hipLaunchKernelGGL(visit_panel_kernel, dim3(2 * (rest / PVECS) + (N + PVECS - 1) / PVECS), dim3(256), 0, stream,
                           A, W, N, K, i0, tabs[cur], Lc + slot(b) * ldk, Hr + slot(b) * ldk, Rr + slot(b) * ldk, Err + slot(b) * ldn, qw, sw);
        if (rest > 0) {                                // the deferred updates of what is behind the panel
            const int base = strip_base(t), behind = (batch + span + 1) * PB, far = K - behind;
            const bool back = batch / span & 1;
            RankUpdate of_w = update(W, Hr, Err, ldn, false, 0, batch - span, batch, behind, far, ALL, 0, N, ALL, 0, -1);
            RankUpdate of_a = update(A, Lc, Rr, ldk, false, 0, batch - span, batch, behind, far, ALL, behind, far, ALL, 0, behind);
            of_w.shape = of_a.shape = rest_shape(whole(of_w).count + whole(of_a).count, span, 2 * (K - batch * PB) + N);
            if (b == batch) done_a = done_w = 0;
            const int nw = whole(of_w).count - done_w, na = whole(of_a).count - done_a, launches = span - (b - batch);
            const int thin = thin_strips((nw + na) / launches, 2 * rest + N);
            RankUpdates us{{
                whole(update(W, Hr, Err, ldn, false, 1 + thin, base, t, i1, PB, ALL, 0, N, ALL, 0, -1)),
                whole(update(A, Lc, Rr, ldk, false, 1 + thin, base, t, i1, PB, ALL, i1 + PB, rest - PB, ALL, 0, -1)),
                whole(update(A, Lc, Rr, ldk, false, 2 + thin, base, t, i1 + PB, rest - PB, ALL, i1, PB, ALL, 0, -1)),
                t + 1 < np ? early(t + 1) : none, none, none}};
            const int n = quota(nw + na, launches, us.u[0].tiles + us.u[1].tiles + us.u[2].tiles + us.u[3].tiles, cus);
            us.u[4] = part_of(of_w, done_w, n < nw ? n : nw, back);
            us.u[5] = part_of(of_a, done_a, n < nw ? 0 : n - nw, back);
            done_w += us.u[4].count;
            done_a += us.u[5].count;
            launch_rank_updates(us, Lookahead{A, Lc, Rr, nullptr, tabs[cur ^ 1], b, t, K, 0, i1, 2}, stream);
        }
        cur ^= 1;
    }
    return hipGetLastError();
}

}  // namespace svdq
