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
// of the weights during the visit, taken in panels of 64 pivots (below), two at a time, so that the matrices cross HBM
// once per 128 pivots.
#include <climits>
#include <type_traits>

#include "svdq_dev.h"
#include "svdq_kernels.h"

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
//                  binary64 matrix instruction.  Behind the first panel of a pair only the second panel's rows and
//                  columns do; behind the second the rest takes both panels' 128 in one pass over memory.  One
//                  block meanwhile does the same for the NEXT panel's diagonal block, takes that through its own 64
//                  dependent steps and leaves the next panel's tables: a serial chain of about 40 us, which is what
//                  the launch behind a pair's first panel takes.
// Same result as the pivot-by-pivot form bit for bit.  K = N = 5120: with a launch per pivot and step (25 600 of them)
// 112 ms, of which the rank updates on the vector unit were 31.
// Pairs: 19.56 -> 18.88 ms (the inverse's launches, us: 49 and 155 in turn).
constexpr int PB = 64;

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
// theorem), as long as nothing leaves the exponent range; `bad` collects whether anything may have, and the callers
// then repeat the whole panel with SLOW, the division itself.  (A branch at every division would cost more than the
// division: it ends the overlap of one vector's chain with the next one's.)  d and y: reciprocal_of below.
template <bool SLOW>
__device__ __forceinline__ double divide_by(double a, double d, double y, bool& bad) {
    if (SLOW) return __ddiv_rn(a, d);
    double q = a * y;
    q = __builtin_fma(__builtin_fma(-d, q, a), y, q);
    q = __builtin_fma(__builtin_fma(-d, q, a), y, q);
    const uint32_t ex = (uint32_t)(__builtin_bit_cast(uint64_t, q) >> 52) & 0x7ffu;     // 2^-600 .. 2^600, or 0 / d
    bad |= (ex - 423u > 1200u) && !(q == 0.0 && a == 0.0);
    return q;
}
// RN(1 / d), or NaN (which every quotient then is: bad) where d is too large or small for divide_by
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

// The diagonal block through its 64 pivots, 256 threads: lane group g = tid / 16 holds rows 4 g .. 4 g + 3, so pivot
// 4 it + k is row k of group it.  INV: in-place Gauss-Jordan inverse (see below); otherwise only the rows and columns
// behind the pivot are updated (row q of D is then the row as it stood at pivot q).  Rt: PB x PB in LDS, ds: 2 in LDS.
template <bool INV, bool SLOW>
__device__ __forceinline__ bool diagonal_pass(double (&x)[4][4], double (*Rt)[PB], double (*ds)[2], PanelTables* __restrict__ out) {
    const int grp = threadIdx.x >> 4, pos = threadIdx.x & 15;
    bool bad = false;
    for (int it = 0; it < 16; ++it) {
        const int sl = (pos + it) & 15;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int q = 4 * it + k;
            double c[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) c[v] = row_first(x[v][k]);
            if (grp == it) {                              // this group's row k is the pivot's
                const double d = c[k], y = reciprocal_of(d);
#pragma unroll
                for (int j = 0; j < 4; ++j) Rt[q][4 * sl + j] = divide_by<SLOW>(x[k][j], d, y, bad);
                if (pos == 0) {
                    ds[q][0] = d;
                    ds[q][1] = y;
                }
            }
            if (pos == 0) {
#pragma unroll
                for (int v = 0; v < 4; ++v) out->C[q][4 * grp + v] = c[v];
            }
            lds_barrier();
            const double d = ds[q][0], y = ds[q][1];
            double r[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) r[j] = Rt[q][4 * sl + j];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (INV) {
                    const bool isq = v == k && grp == it;
                    const double e = divide_by<SLOW>(isq ? 1.0 : -c[v], d, y, bad);
#pragma unroll
                    for (int j = 0; j < 4; ++j) x[v][j] = isq ? r[j] : __builtin_fma(-c[v], r[j], x[v][j]);
                    x[v][k] = (pos == 0) ? e : x[v][k];
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const double u = __builtin_fma(-c[v], r[j], x[v][j]);
                        x[v][j] = (4 * grp + v > q && 4 * sl + j > q) ? u : x[v][j];
                    }
                }
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int j = 0; j < 4; ++j) x[v][j] = row_turn(x[v][j]);
    }
    return bad;
}
template <bool INV>
__device__ __forceinline__ void diagonal_block(double (&x)[4][4], double (*Rt)[PB], double (*ds)[2], PanelTables* __restrict__ out) {
    const int grp = threadIdx.x >> 4, pos = threadIdx.x & 15;
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int j = 0; j < 4; ++j) out->D[4 * grp + v][4 * pos + j] = x[v][j];       // kept for a second pass
    if (__syncthreads_or(diagonal_pass<INV, false>(x, Rt, ds, out))) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int j = 0; j < 4; ++j) x[v][j] = out->D[4 * grp + v][4 * pos + j];
        __syncthreads();
        diagonal_pass<INV, true>(x, Rt, ds, out);
        __syncthreads();
    }
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            out->D[4 * grp + v][4 * pos + j] = x[v][j];
            out->R[4 * grp + v][4 * pos + j] = Rt[4 * grp + v][4 * pos + j];
        }
    if (threadIdx.x < PB) {
        out->d[threadIdx.x] = ds[threadIdx.x][0];
        out->y[threadIdx.x] = ds[threadIdx.x][1];
    }
}

// The panel's first tables: nothing precedes them that could carry them along.
template <bool INV>
__global__ __launch_bounds__(256)
void first_tables_kernel(const double* __restrict__ D, size_t ld, PanelTables* __restrict__ out) {
    __shared__ __attribute__((aligned(16))) double Rt[PB][PB], ds[PB][2];
    const int grp = threadIdx.x >> 4, pos = threadIdx.x & 15;
    double x[4][4];
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int j = 0; j < 4; ++j) x[v][j] = D[(size_t)(4 * grp + v) * ld + 4 * pos + j];
    diagonal_block<INV>(x, Rt, ds, out);
}

// Vectors per block of the panel kernels: 16 lane groups of two vectors.  Two vectors per group halve the LDS reads of
// the table (four values per lane and pivot), and 32 per block spread K = 5120 over every CU.
constexpr int PV = 2, PVECS = 16 * PV;
__device__ __forceinline__ void load_table(double (*to)[PB], const double (*from)[PB]) {
    for (int e = threadIdx.x * 2; e < PB * PB; e += 512)
        *reinterpret_cast<double2*>(&to[0][0] + e) = *reinterpret_cast<const double2*>(&from[0][0] + e);
}

// ---- in-place Gauss-Jordan inverse without pivoting.  Step p: d = A[p][p], col = A[:, p], row = A[p, :] / d;
// A[a][j] -= col[a] row[j] elsewhere, A[p][j] = row[j], A[a][p] = -col[a] / d, A[p][p] = 1 / d.
// Blocks 0 .. nb - 1: PVECS rows outside the panel; nb .. 2 nb - 1: PVECS columns outside it.
// Saves LT[q][a] = column of pivot p0 + q, Rr[q][j] = its scaled row.
__global__ __launch_bounds__(256)
void gj_panel_kernel(double* __restrict__ A, int K, int p0, const PanelTables* __restrict__ tb,
                     double* __restrict__ LT, double* __restrict__ Rr) {
    __shared__ __attribute__((aligned(16))) double tab[PB][PB], ds[PB][2];
    const int nb = (K - PB) / PVECS;
    const int grp = threadIdx.x >> 4, pos = threadIdx.x & 15;
    const bool rows = (int)blockIdx.x < nb;
    double x[PV][4];
    int idx[PV];
#pragma unroll
    for (int v = 0; v < PV; ++v) {
        idx[v] = ((int)blockIdx.x - (rows ? 0 : nb)) * PVECS + (grp >> 2) * 4 * PV + v * 4 + (grp & 3);
        if (idx[v] >= p0) idx[v] += PB;
    }
    auto load = [&]() {
#pragma unroll
        for (int v = 0; v < PV; ++v)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                x[v][j] = rows ? A[(size_t)idx[v] * K + p0 + 4 * pos + j] : A[(size_t)(p0 + 4 * pos + j) * K + idx[v]];
    };
    load();
    load_table(tab, rows ? tb->R : tb->C);
    if (threadIdx.x < PB) {
        ds[threadIdx.x][0] = tb->d[threadIdx.x];
        ds[threadIdx.x][1] = tb->y[threadIdx.x];
    }
    __syncthreads();
    double* const save = rows ? LT : Rr;
    auto pass = [&](auto ROWS, auto SLOWC) {
        constexpr bool R = decltype(ROWS)::value;
        bool bad = false;
        for (int it = 0; it < 16; ++it) {
            const int sl = (pos + it) & 15;
            double f[4][PV];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int q = 4 * it + k;
                const double d = ds[q][0], y = ds[q][1];
                double t[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) t[j] = tab[q][4 * sl + j];
#pragma unroll
                for (int v = 0; v < PV; ++v) {
                    const double c = row_first(x[v][k]);
                    const double e = divide_by<decltype(SLOWC)::value>(R ? -c : c, d, y, bad);
                    f[k][v] = R ? c : e;
#pragma unroll
                    for (int j = 0; j < 4; ++j) x[v][j] = __builtin_fma(-f[k][v], t[j], x[v][j]);
                    x[v][k] = (pos == 0) ? e : x[v][k];
                }
            }
            if (pos == 0) {
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int v = 0; v < PV; ++v) save[(size_t)(4 * it + k) * K + idx[v]] = f[k][v];
            }
#pragma unroll
            for (int v = 0; v < PV; ++v)
#pragma unroll
                for (int j = 0; j < 4; ++j) x[v][j] = row_turn(x[v][j]);
        }
        return bad;
    };
    auto run = [&](auto ROWS) {
        if (__any(pass(ROWS, std::false_type{}))) {
            load();
            pass(ROWS, std::true_type{});
        }
    };
    if (rows) run(std::true_type{});
    else run(std::false_type{});
#pragma unroll
    for (int v = 0; v < PV; ++v)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (rows) A[(size_t)idx[v] * K + p0 + 4 * pos + j] = x[v][j];
            else A[(size_t)(p0 + 4 * pos + j) * K + idx[v]] = x[v][j];
        }
}

// ---- one panel of the visit: indices i0 .. i0 + 63 = one 64-group.  For each index i: code and error of every
// channel, the error spread over the panel's later weights, index i eliminated from H^-1 (A[a][b] -= A[a][i] (A[i][b] / d)
// for a, b > i).  Blocks 0 .. nr - 1: PVECS rows of A behind the panel; nr .. 2 nr - 1: columns; the rest: channels
// of W.  Saves, per pivot q, what the rank updates need: HcT[q][a] = A[a][i], HrT[q][b] = A[i][b],
// T[q][b] = A[i][b] / d, Err[q][n].  The panel's own rows and columns of A and W are not read again.
__global__ __launch_bounds__(256)
void visit_panel_kernel(const double* __restrict__ A, const double* __restrict__ W, int N, int K, int i0,
                        const PanelTables* __restrict__ tb,
                        double* __restrict__ HcT, double* __restrict__ HrT, double* __restrict__ T, double* __restrict__ Err,
                        uint8_t* __restrict__ qw, float* __restrict__ sw) {
    __shared__ __attribute__((aligned(16))) double tab[PB][PB], ds[PB][2];
    const int i1 = i0 + PB, nr = (K - i1) / PVECS;
    const int grp = threadIdx.x >> 4, pos = threadIdx.x & 15;
    const int role = ((int)blockIdx.x < nr) ? 0 : ((int)blockIdx.x < 2 * nr) ? 1 : 2;      // rows, columns, channels
    double x[PV][4];
    int idx[PV];
    bool live[PV];
#pragma unroll
    for (int v = 0; v < PV; ++v) {
        idx[v] = (role < 2 ? i1 : 0) + ((int)blockIdx.x - role * nr) * PVECS + (grp >> 2) * 4 * PV + v * 4 + (grp & 3);
        live[v] = role < 2 || idx[v] < N;
    }
    auto load = [&]() {
#pragma unroll
        for (int v = 0; v < PV; ++v)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                x[v][j] = 0.0;
                if (role == 0) x[v][j] = A[(size_t)idx[v] * K + i0 + 4 * pos + j];
                if (role == 1) x[v][j] = A[(size_t)(i0 + 4 * pos + j) * K + idx[v]];
                if (role == 2 && live[v]) x[v][j] = W[(size_t)(i0 + 4 * pos + j) * N + idx[v]];
            }
    };
    load();
    load_table(tab, role == 0 ? tb->R : role == 1 ? tb->C : tb->D);
    if (threadIdx.x < PB) {
        ds[threadIdx.x][0] = tb->d[threadIdx.x];
        ds[threadIdx.x][1] = tb->y[threadIdx.x];
    }
    __syncthreads();
    if (role == 2) {
        float s[PV];
#pragma unroll
        for (int v = 0; v < PV; ++v) {
            double a = fmax(fmax(fabs(x[v][0]), fabs(x[v][1])), fmax(fabs(x[v][2]), fabs(x[v][3])));
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) a = fmax(a, __shfl_xor(a, o));
            s[v] = __fdiv_rn((float)a, 7.0f);
            if (pos == 0 && live[v]) sw[(size_t)(i0 >> 6) * N + idx[v]] = s[v];
        }
        auto pass = [&](auto SLOWC) {
            bool bad = false;
            for (int it = 0; it < 16; ++it) {
                const int sl = (pos + it) & 15;
                uint32_t codes[PV] = {};
                double e[4][PV];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int q = 4 * it + k;
                    const double d = ds[q][0], y = ds[q][1];
                    double t[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) t[j] = tab[q][4 * sl + j];
#pragma unroll
                    for (int v = 0; v < PV; ++v) {
                        const double w = row_first(x[v][k]);
                        float c = fminf(fmaxf(rintf(__fdiv_rn((float)w, s[v])), -8.0f), 7.0f);
                        c = (s[v] > 0.0f) ? c : 0.0f;
                        codes[v] |= ((uint32_t)(int)c & 15u) << (4 * k);
                        e[k][v] = divide_by<decltype(SLOWC)::value>(__builtin_fma(-(double)c, (double)s[v], w), d, y, bad);   // code x scale is exact
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const double u = __builtin_fma(-t[j], e[k][v], x[v][j]);
                            x[v][j] = (4 * sl + j > q) ? u : x[v][j];
                        }
                    }
                }
#pragma unroll
                for (int v = 0; v < PV; ++v) {
                    if (pos == 0 && live[v]) {
#pragma unroll
                        for (int k = 0; k < 4; ++k) Err[(size_t)(4 * it + k) * N + idx[v]] = e[k][v];
                        // four codes: two bytes, low nibble = even index
                        *reinterpret_cast<uint16_t*>(qw + (size_t)idx[v] * (K >> 1) + (i0 >> 1) + 2 * it) = (uint16_t)codes[v];
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j) x[v][j] = row_turn(x[v][j]);
                }
            }
            return bad;
        };
        if (__any(pass(std::false_type{}))) {
            load();
            pass(std::true_type{});
        }
        return;
    }
    double* const save = role == 0 ? HcT : HrT;
    auto pass = [&](auto COLS, auto SLOWC) {
        constexpr bool C = decltype(COLS)::value;
        bool bad = false;
        for (int it = 0; it < 16; ++it) {
            const int sl = (pos + it) & 15;
            double c[4][PV], f[4][PV];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int q = 4 * it + k;
                double t[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) t[j] = tab[q][4 * sl + j];
#pragma unroll
                for (int v = 0; v < PV; ++v) {
                    c[k][v] = row_first(x[v][k]);
                    f[k][v] = C ? divide_by<decltype(SLOWC)::value>(c[k][v], ds[q][0], ds[q][1], bad) : c[k][v];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const double u = __builtin_fma(-f[k][v], t[j], x[v][j]);
                        x[v][j] = (4 * sl + j > q) ? u : x[v][j];
                    }
                }
            }
            if (pos == 0) {
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int v = 0; v < PV; ++v) {
                        save[(size_t)(4 * it + k) * K + idx[v]] = c[k][v];
                        if (C) T[(size_t)(4 * it + k) * K + idx[v]] = f[k][v];
                    }
            }
#pragma unroll
            for (int v = 0; v < PV; ++v)
#pragma unroll
                for (int j = 0; j < 4; ++j) x[v][j] = row_turn(x[v][j]);
        }
        return bad;
    };
    if (role == 0) {
        pass(std::false_type{}, std::false_type{});
    } else if (__any(pass(std::true_type{}, std::false_type{}))) {
        load();
        pass(std::true_type{}, std::true_type{});
    }
}

// ---- X[a][b] <- (..((X[a][b] - L[0][a] R[0][b]) - L[1][a] R[1][b]).. - L[depth - 1][a] R[depth - 1][b]) over rows
// a0 + [0, rows) and columns b0 + [0, cols), leaving out the nskip indices from skip_a (rows) and skip_b (columns) on (rows
// and cols count what is left) and the 64 x 64 block at (hole, hole).  L and R are [depth][ld].  rows % 64 == 0.
struct RankUpdate {
    double* X;
    const double *L, *R;
    size_t ldx, ldl, ldr;
    int depth, a0, rows, b0, cols, skip_a, skip_b, nskip, hole;
    int tiles_b, tiles;          // 128 x 128 tiles along b, and in all
    bool backwards;              // every other update walks its tiles backwards, first through what is still in the caches
};
// The next panel's diagonal block (at index s0 of A), for the first block of a rank update: brought up to date with L
// and R (none: it is already, as D), then through its own pivots (mode 1: inverse, 2: visit) into `next`.  Also puts the
// finished diagonal block `prev` of the current panel (at p0) in place; null: nothing to put.
struct Lookahead {
    double* A;
    const double *L, *R;
    const PanelTables* prev;
    PanelTables* next;
    int depth, K, p0, s0, mode;
};

// acc[i][k]: a wave's 16 NI x 64 elements through `depth` pivots (a multiple of 8); lane (j, kq) = (l % 16, l / 16) holds in acc[i][k][e]
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
__device__ __forceinline__ void update_chain(const int depth, double4v (&acc)[NI][4], const double* __restrict__ L, size_t ldl,
                                             const double* __restrict__ R, size_t ldr, int lane, const int (&col)[2], const int (&d1)[2]) {
    const int j = lane & 15, kq = lane >> 4;
    double a[2][NI];
    double2 b[2][2];
    auto request = [&](const int s, const int buf) {
#pragma unroll
        for (int i = 0; i < NI; ++i) a[buf][i] = -L[(size_t)(4 * s + kq) * ldl + 16 * i + j];
#pragma unroll
        for (int i = 0; i < 2; ++i) b[buf][i] = load2<PAIR>(R + (size_t)(4 * s + kq) * ldr + col[i], d1[i]);
    };
    auto multiply = [&](const int buf) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[i][k] = mfma_f64(a[buf][i], (k & 1) ? b[buf][k >> 1].y : b[buf][k >> 1].x, acc[i][k]);
    };
    request(0, 0);
    for (int s = 0; s < depth / 4; s += 2) {
        request(s + 1, 1);
        multiply(0);
        if (s + 2 < depth / 4) request(s + 2, 0);
        multiply(1);
    }
}

__device__ __forceinline__ void look_ahead(const Lookahead& la, double (*Rt)[PB], double (*ds)[2]) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, j = lane & 15, kq = lane >> 4;
    if (la.prev)
        for (int e = tid; e < PB * PB; e += 256) la.A[(size_t)(la.p0 + e / PB) * la.K + la.p0 + e % PB] = la.prev->D[e / PB][e % PB];
    if (la.mode == 0) return;
    const int grp = tid >> 4, pos = tid & 15;
    double x[4][4];
    if (la.L) {
        double4v acc[1][4];
        const double* X = la.A + (size_t)(la.s0 + 16 * wave) * la.K + la.s0;
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[0][k][e] = X[(size_t)(4 * e + kq) * la.K + wave_col(j, k)];
        const int col[2] = {2 * j, 32 + 2 * j}, d1[2] = {1, 1};
        update_chain<1, true>(la.depth, acc, la.L + la.s0 + 16 * wave, (size_t)la.K, la.R + la.s0, (size_t)la.K, lane, col, d1);
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e) Rt[16 * wave + 4 * e + kq][wave_col(j, k)] = acc[0][k][e];
        __syncthreads();
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int i = 0; i < 4; ++i) x[v][i] = Rt[4 * grp + v][4 * pos + i];
        __syncthreads();
    } else {
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int i = 0; i < 4; ++i) x[v][i] = la.prev->D[4 * grp + v][4 * pos + i];
    }
    if (la.mode == 1) diagonal_block<true>(x, Rt, ds, la.next);
    else diagonal_block<false>(x, Rt, ds, la.next);
}

// Block 0 looks ahead; the others take 128 x 128 elements of the matrix of u0, u1 or u2, 64 x 64 per wave.  Every element
// is read and written once per `depth` updates, 16 bytes: with 64 HBM bounds the large matrices (K = 5120: 420 MB, 85 us
// at the rate of a copy, and the matrix unit needs half of that), with 128 both take about as long.
template <bool PAIR>
__global__ __launch_bounds__(256, 2)
void rank_update_kernel(const RankUpdate u0, const RankUpdate u1, const RankUpdate u2, const Lookahead la) {
    __shared__ __attribute__((aligned(16))) double Rt[PB][PB], ds[PB][2];
    if (blockIdx.x == 0) {
        look_ahead(la, Rt, ds);
        return;
    }
    int t = (int)blockIdx.x - 1;
    const bool first = t < u0.tiles, second = !first && t < u0.tiles + u1.tiles;
    const RankUpdate u = first ? u0 : second ? u1 : u2;
    t -= first ? 0 : second ? u0.tiles : u0.tiles + u1.tiles;
    if (u.backwards) t = u.tiles - 1 - t;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j = lane & 15, kq = lane >> 4;
    const int ia = (t / u.tiles_b) * 128 + (wave >> 1) * 64, ib = (t % u.tiles_b) * 128 + (wave & 1) * 64;
    if (ia >= u.rows || ib >= u.cols) return;
    int ga = u.a0 + ia, gb = u.b0 + ib;                     // 64-blocks do not straddle what is left out
    if (ga >= u.skip_a) ga += u.nskip;
    if (gb >= u.skip_b) gb += u.nskip;
    if (ga == u.hole && gb == u.hole) return;
    double* X = u.X + (size_t)ga * u.ldx;
    double4v acc[4][4];
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
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const double2 v = load2<PAIR>(X + (size_t)(16 * i + 4 * e + kq) * u.ldx + col[k], d1[k]);
                acc[i][2 * k][e] = v.x;
                acc[i][2 * k + 1][e] = v.y;
            }
    update_chain<4, PAIR>(u.depth, acc, u.L + ga, u.ldl, u.R, u.ldr, lane, col, d1);
    // the stores' addresses are formed again here; kept from the loads they would spill
#pragma unroll
    for (int k = 0; k < 2; ++k) asm volatile("" : "+v"(col[k]));
#pragma unroll
    for (int k = 0; k < 2; ++k)
        if (in[k][0]) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
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

void launch_rank_updates(RankUpdate u0, RankUpdate u1, RankUpdate u2, const Lookahead& la, bool backwards, hipStream_t stream) {
    bool pair = true;
    for (RankUpdate* u : {&u0, &u1, &u2}) {
        u->tiles_b = (u->cols + 127) / 128;
        u->tiles = (u->rows > 0 && u->cols > 0) ? u->tiles_b * ((u->rows + 127) / 128) : 0;
        u->backwards = backwards;
        pair = pair && u->ldx % 2 == 0 && u->ldr % 2 == 0;
    }
    auto kern = pair ? rank_update_kernel<true> : rank_update_kernel<false>;
    hipLaunchKernelGGL(kern, dim3(1 + u0.tiles + u1.tiles + u2.tiles), dim3(256), 0, stream, u0, u1, u2, la);
}

inline size_t up256(size_t v) { return (v + 255) & ~(size_t)255; }

}  // namespace

size_t gptq_workspace_bytes(int N, int K) {
    return up256((size_t)K * K * 8) + up256((size_t)K * N * 8) + 3 * up256((size_t)K * 2 * PB * 8) + up256((size_t)2 * PB * N * 8) +
           2 * up256(sizeof(PanelTables)) + 256;
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
    // saved by the two panels of a pair, one behind the other
    double* Lc = (double*)p;       p += up256((size_t)K * 2 * PB * 8);     // pivot columns         [2 PB][K]
    double* Rr = (double*)p;       p += up256((size_t)K * 2 * PB * 8);     // scaled pivot rows     [2 PB][K]
    double* Hr = (double*)p;       p += up256((size_t)K * 2 * PB * 8);     // rows of H^-1          [2 PB][K]
    double* Err = (double*)p;      p += up256((size_t)2 * PB * N * 8);     // errors of the panel   [2 PB][N]
    PanelTables* tabs[2];                                              // this panel's and the next one's
    for (auto& t : tabs) {
        t = (PanelTables*)p;
        p += up256(sizeof(PanelTables));
    }
    double* add = (double*)p;                                          // the damping term
    hipLaunchKernelGGL(diag_sum_kernel, dim3(1), dim3(256), 0, stream, H, damp, K, add);
    hipLaunchKernelGGL(prepare_kernel, dim3(K), dim3(256), 0, stream, R, H, add, N, K, A, W);
    const size_t ldk = (size_t)K, ldn = (size_t)N;
    constexpr int ALL = INT_MAX;                       // nothing left out
    const RankUpdate none{A, nullptr, nullptr, ldk, ldk, ldk, PB, 0, 0, 0, 0, ALL, ALL, 0, -1, 1, 0, false};
    // `depth` updates of A or W saved from row `from` of the pair's buffers on
    auto of_inverse = [&](int from, int depth, int a0, int rows, int b0, int cols, int skip_a, int skip_b, int nskip, int hole) {
        return RankUpdate{A, Lc + from * ldk, Rr + from * ldk, ldk, ldk, ldk, depth, a0, rows, b0, cols, skip_a, skip_b, nskip, hole, 1, 0, false};
    };
    auto of_weights = [&](int depth, int a0, int rows) {
        return RankUpdate{W, Hr, Err, ldn, ldk, ldn, depth, a0, rows, 0, N, ALL, ALL, 0, -1, 1, 0, false};
    };
    const int np = K / PB;
    int cur = 0;                                       // tabs[cur]: the current panel's
    hipLaunchKernelGGL(first_tables_kernel<true>, dim3(1), dim3(256), 0, stream, A, ldk, tabs[cur]);
    for (int b = 0; b < np; ++b) {                     // the inverse, one panel of pivots at a time
        const int p0 = b * PB, half = (b & 1) * PB;    // half: this panel's place in the pair's buffers
        if (np > 1)
            hipLaunchKernelGGL(gj_panel_kernel, dim3(2 * (K - PB) / PVECS), dim3(256), 0, stream, A, K, p0, tabs[cur],
                               Lc + half * ldk, Rr + half * ldk);
        // next: the following panel, and after the last one the first panel of the visit
        const int s0 = (b + 1 < np) ? p0 + PB : 0;
        const bool same = s0 == p0;                    // a single panel: its own finished block is what is visited
        // What the next diagonal block has not had yet: both panels of a pair, but the second's only where it lies in
        // the first (two panels: the visit starts there).
        const int from = (half && s0 == p0 - PB) ? PB : 0, depth = half + PB - from;
        const Lookahead la{A, same ? nullptr : Lc + from * ldk, Rr + from * ldk, tabs[cur], tabs[cur ^ 1],
                           depth, K, p0, s0, (b + 1 < np) ? 1 : 2};
        if (half) {
            // everything outside both panels; then the first panel's rows and columns, which only the second's pivots are left for
            const int q0 = p0 - PB;
            launch_rank_updates(of_inverse(0, 2 * PB, 0, K - 2 * PB, 0, K - 2 * PB, q0, q0, 2 * PB, s0),
                                of_inverse(PB, PB, q0, PB, 0, K - PB, ALL, p0, PB, s0),
                                of_inverse(PB, PB, 0, K - 2 * PB, q0, PB, q0, ALL, 2 * PB, s0), la, b & 2, stream);
        } else if (b + 1 < np) {                       // the second panel's rows, and its columns in the rows of neither
            launch_rank_updates(of_inverse(0, PB, s0, PB, 0, K - PB, ALL, p0, PB, s0),
                                of_inverse(0, PB, 0, K - 2 * PB, s0, PB, p0, ALL, 2 * PB, s0), none, la, false, stream);
        } else {                                       // a last panel without a second
            launch_rank_updates(of_inverse(0, PB, 0, K - PB, 0, K - PB, p0, p0, PB, same ? -1 : s0), none, none, la, b & 2, stream);
        }
        cur ^= 1;
    }
    for (int b = 0; b < np; ++b) {                     // the weights, one panel (= one 64-group) at a time
        const int i0 = b * PB, i1 = i0 + PB, rest = K - i1, half = (b & 1) * PB;
        hipLaunchKernelGGL(visit_panel_kernel, dim3(2 * (rest / PVECS) + (N + PVECS - 1) / PVECS), dim3(256), 0, stream,
                           A, W, N, K, i0, tabs[cur], Lc + half * ldk, Hr + half * ldk, Rr + half * ldk, Err + half * ldn, qw, sw);
        if (rest > 0) {                                // the deferred updates of what is behind the panel
            const Lookahead la{A, Lc, Rr, nullptr, tabs[cur ^ 1], half + PB, K, 0, i1, 2};
            if (half)
                launch_rank_updates(of_weights(2 * PB, i1, rest), of_inverse(0, 2 * PB, i1, rest, i1, rest, ALL, ALL, 0, i1), none,
                                    la, b & 2, stream);
            else                                       // of the second panel's rows and columns only
                launch_rank_updates(of_weights(PB, i1, PB), of_inverse(0, PB, i1, PB, i1, rest, ALL, ALL, 0, i1),
                                    of_inverse(0, PB, i1 + PB, rest - PB, i1, PB, ALL, ALL, 0, -1), la, false, stream);
        }
        cur ^= 1;
    }
    return hipGetLastError();
}

}  // namespace svdq
