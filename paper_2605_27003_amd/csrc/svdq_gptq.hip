// GPTQ on the residual weights (Sec. III-B: the residual branch of the SVDQuant split is quantised with GPTQ
// instead of round-to-nearest).  Offline calibration, not part of the per-step path: clarity over speed.
//
// The algorithm in its column-sequential form: weights are visited in the order k = 0..K-1; a visited weight is
// rounded to the int4 grid of its (channel, 64-group) scale and its rounding error is spread over the not yet
// visited weights of the same channel in proportion to row k of the inverse Hessian of the layer-wise objective
// ||X^ (R - R^)||^2 (H = X^T X^ plus damping), from which index k is then eliminated.  Everything runs in
// binary64 with one explicitly rounded operation per arithmetic step and no reductions other than max and one
// sequential sum, so that a CPU reference repeats every bit.  The published implementation factors H^-1 once
// (Cholesky) and reads the same numbers off the factor; this form trades that for elementwise kernels:
// K^3 updates for the inverse, K^3 / 3 of H^-1 and K^2 N / 2 of the weights during the visit, taken in panels of 64
// pivots (below) so that the matrices cross HBM once per panel.
#include "svdq_dev.h"
#include "svdq_kernels.h"

namespace svdq {

namespace {

// ---- H += X^T X^, X^ = x * inv_lambda in binary32 (eq. 5), products and sums in binary64
constexpr int HT = 64;   // tile of H per block
__global__ __launch_bounds__(256)
void hessian_kernel(const uint16_t* __restrict__ x, int64_t ldx, const float* __restrict__ inv_lambda,
                    int64_t M, int K, double* __restrict__ H) {
    __shared__ double xa[16][HT + 1], xb[16][HT + 1];
    const int a0 = blockIdx.y * HT, b0 = blockIdx.x * HT;
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    double acc[4][4] = {};
    for (int64_t m0 = 0; m0 < M; m0 += 16) {
        for (int e = threadIdx.x; e < 16 * HT; e += 256) {
            const int mr = e / HT, c = e - mr * HT;
            const int64_t m = m0 + mr;
            double va = 0.0, vb = 0.0;
            if (m < M) {
                if (a0 + c < K) va = (double)__fmul_rn(bits_f((uint32_t)x[m * ldx + a0 + c] << 16), inv_lambda[a0 + c]);
                if (b0 + c < K) vb = (double)__fmul_rn(bits_f((uint32_t)x[m * ldx + b0 + c] << 16), inv_lambda[b0 + c]);
            }
            xa[mr][c] = va;
            xb[mr][c] = vb;
        }
        __syncthreads();
#pragma unroll
        for (int mr = 0; mr < 16; ++mr)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = __fma_rn(xa[mr][ty * 4 + i], xb[mr][tx * 4 + j], acc[i][j]);
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int a = a0 + ty * 4 + i, b = b0 + tx * 4 + j;
            if (a < K && b < K) H[(size_t)a * K + b] += acc[i][j];
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
// pivots, one rounded product and one rounded subtraction per pivot: that sequence per element is the definition, and
// it does not say WHEN an element is touched.  Pivots are taken in panels of PB = 64, two launches per panel:
//   panel kernel   brings the panel's own rows and columns (2 x 64 x K elements, for the weights 64 x N) through all 64
//                  pivots.  A row outside the panel only needs the panel's diagonal block as it stood at each pivot,
//                  and a column likewise, so rows and columns are independent of each other: a block takes 64 of them
//                  and first runs the 64 x 64 diagonal block itself (every block repeats that; it is a chain of 64
//                  dependent steps, and a launch of its own would cost as much again).  The pivot's column and scaled
//                  row, as they stood when the pivot was taken, are saved.
//   rank update    everything else receives its 64 updates in one pass from the saved columns and rows, in pivot
//                  order, with the same two rounded operations per update.
// Bit-identical to the pivot-by-pivot form.  K = N = 5120: one launch per pivot and step (25 600 launches) took 112 ms,
// of which the rank updates were 31.
constexpr int PB = 64;
constexpr int PTHREADS = 1024;           // 64 vectors x 16 lanes

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

struct PanelTables {
    double (*R)[PB];       // [q][t]: row q of the diagonal block divided by its pivot, when pivot q was taken
    double (*C)[PB];       // [q][t]: column q
    double* d;             // [q]: pivot
};

// The diagonal block through its 64 pivots (all 1024 threads: row t = tid / 16).  INV: in-place Gauss-Jordan inverse
// (see below); otherwise elimination of the rows and columns behind the pivot only.  Leaves the tables; the block's
// final values are in x.
template <bool INV>
__device__ __forceinline__ void panel_diagonal(double (&x)[4], const PanelTables& tb) {
    const int t = threadIdx.x >> 4, pos = threadIdx.x & 15;
    for (int it = 0; it < 16; ++it) {
        const int sl = (pos + it) & 15;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int q = 4 * it + k;
            const double c = row_first(x[k]);
            double r[4];
            if (t == q) {                                 // c is the pivot
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    r[j] = __ddiv_rn(x[j], c);
                    tb.R[q][4 * sl + j] = r[j];
                }
                if (pos == 0) tb.d[q] = c;
            }
            if (pos == 0) tb.C[q][t] = c;
            __syncthreads();
            const double d = tb.d[q];
            const bool own = pos == 0;                    // element k of this lane is column q
            if (INV) {
                const double e = __ddiv_rn(t == q ? 1.0 : -c, d);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const double rj = tb.R[q][4 * sl + j];
                    const double v = (t == q) ? rj : __dsub_rn(x[j], __dmul_rn(c, rj));
                    x[j] = (own && j == k) ? e : v;
                }
            } else if (t > q) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const double v = __dsub_rn(x[j], __dmul_rn(c, tb.R[q][4 * sl + j]));
                    x[j] = (4 * sl + j > q) ? v : x[j];
                }
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = row_turn(x[j]);
    }
    __syncthreads();
}

// Where panel index b (64-blocks outside the panel's own) lies.
__device__ __forceinline__ int outside_block(int b, int pb) { return b < pb ? b : b + 1; }

// ---- in-place Gauss-Jordan inverse without pivoting.  Step p: d = A[p][p], col = A[:, p], row = A[p, :] / d;
// A[a][j] -= col[a] row[j] elsewhere, A[p][j] = row[j], A[a][p] = -col[a] / d, A[p][p] = 1 / d.
// Blocks 0 .. nb - 1: 64 rows outside the panel; nb .. 2 nb - 1: 64 columns outside it; the last block only runs the
// diagonal block and writes it to Dnew (the other blocks read it from A meanwhile; the rank update puts it in place).
// Saves LT[q][a] = column of pivot p0 + q, Rr[q][j] = its scaled row.
__global__ __launch_bounds__(PTHREADS)
void gj_panel_kernel(double* __restrict__ A, int K, int p0, double* __restrict__ LT, double* __restrict__ Rr,
                     double* __restrict__ Dnew) {
    __shared__ __attribute__((aligned(16))) double Rt[PB][PB], Ct[PB][PB], dt[PB];
    const PanelTables tb{Rt, Ct, dt};
    const int nb = K / PB - 1, pb = p0 / PB;
    const int v = threadIdx.x >> 4, pos = threadIdx.x & 15;
    const int role = ((int)blockIdx.x < nb) ? 0 : ((int)blockIdx.x < 2 * nb) ? 1 : 2;
    const int idx = outside_block((int)blockIdx.x - role * nb, pb) * PB + v;     // this vector's row or column
    double x[4], dg[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        dg[j] = A[(size_t)(p0 + v) * K + p0 + 4 * pos + j];
        x[j] = 0.0;
        if (role == 0) x[j] = A[(size_t)idx * K + p0 + 4 * pos + j];
        if (role == 1) x[j] = A[(size_t)(p0 + 4 * pos + j) * K + idx];
    }
    panel_diagonal<true>(dg, tb);
    if (role == 2) {
#pragma unroll
        for (int j = 0; j < 4; ++j) Dnew[v * PB + 4 * pos + j] = dg[j];
        return;
    }
    for (int it = 0; it < 16; ++it) {
        const int sl = (pos + it) & 15;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int q = 4 * it + k;
            const double c = row_first(x[k]), d = dt[q];
            const double e = __ddiv_rn(role == 0 ? -c : c, d);
            if (role == 0) {
                if (pos == 0) LT[(size_t)q * K + idx] = c;
#pragma unroll
                for (int j = 0; j < 4; ++j) x[j] = __dsub_rn(x[j], __dmul_rn(c, Rt[q][4 * sl + j]));
            } else {
                if (pos == 0) Rr[(size_t)q * K + idx] = e;
#pragma unroll
                for (int j = 0; j < 4; ++j) x[j] = __dsub_rn(x[j], __dmul_rn(Ct[q][4 * sl + j], e));
            }
            x[k] = (pos == 0) ? e : x[k];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = row_turn(x[j]);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (role == 0) A[(size_t)idx * K + p0 + 4 * pos + j] = x[j];
        else A[(size_t)(p0 + 4 * pos + j) * K + idx] = x[j];
    }
}

// ---- one panel of the visit: indices i0 .. i0 + 63 = one 64-group.  For each index i: code and error of every
// channel, the error spread over the panel's later weights, index i eliminated from H^-1 (A[a][b] -= A[a][i] (A[i][b] / d)
// for a, b > i).  Blocks 0 .. nr - 1: 64 rows of A behind the panel; nr .. 2 nr - 1: 64 columns; the rest: 64 channels
// of W each.  Saves, per pivot q, what the rank updates need: HcT[q][a] = A[a][i], HrT[q][b] = A[i][b],
// T[q][b] = A[i][b] / d, Err[q][n].  The panel's own rows and columns of A and W are not read again.
__global__ __launch_bounds__(PTHREADS)
void visit_panel_kernel(const double* __restrict__ A, const double* __restrict__ W, int N, int K, int i0,
                        double* __restrict__ HcT, double* __restrict__ HrT, double* __restrict__ T, double* __restrict__ Err,
                        uint8_t* __restrict__ qw, float* __restrict__ sw) {
    __shared__ __attribute__((aligned(16))) double Rt[PB][PB], Ct[PB][PB], dt[PB];
    const PanelTables tb{Rt, Ct, dt};
    const int i1 = i0 + PB, nr = (K - i1) / PB;
    const int v = threadIdx.x >> 4, pos = threadIdx.x & 15;
    const int role = ((int)blockIdx.x < nr) ? 0 : ((int)blockIdx.x < 2 * nr) ? 1 : 2;
    const int idx = (role < 2 ? i1 : 0) + ((int)blockIdx.x - role * nr) * PB + v;      // row, column or channel
    const bool live = role < 2 || idx < N;
    double x[4], dg[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        dg[j] = A[(size_t)(i0 + v) * K + i0 + 4 * pos + j];
        x[j] = 0.0;
        if (role == 0) x[j] = A[(size_t)idx * K + i0 + 4 * pos + j];
        if (role == 1) x[j] = A[(size_t)(i0 + 4 * pos + j) * K + idx];
        if (role == 2 && live) x[j] = W[(size_t)(i0 + 4 * pos + j) * N + idx];
    }
    panel_diagonal<false>(dg, tb);
    if (role == 2) {
        // rows of H^-1 as they stood when their index was visited: the diagonal block's final values right of the diagonal
#pragma unroll
        for (int j = 0; j < 4; ++j) Ct[v][4 * pos + j] = dg[j];
        __syncthreads();
        double a = fmax(fmax(fabs(x[0]), fabs(x[1])), fmax(fabs(x[2]), fabs(x[3])));
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) a = fmax(a, __shfl_xor(a, o));
        const float s = __fdiv_rn((float)a, 7.0f);
        if (pos == 0 && live) sw[(size_t)(i0 >> 6) * N + idx] = s;
        for (int it = 0; it < 16; ++it) {
            const int sl = (pos + it) & 15;
            uint32_t codes = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int q = 4 * it + k;
                const double w = row_first(x[k]);
                float c = 0.0f;
                if (s > 0.0f) c = fminf(fmaxf(rintf(__fdiv_rn((float)w, s)), -8.0f), 7.0f);
                codes |= ((uint32_t)(int)c & 15u) << (4 * k);
                const double e = __ddiv_rn(__dsub_rn(w, __dmul_rn((double)c, (double)s)), dt[q]);
                if (pos == 0 && live) Err[(size_t)q * N + idx] = e;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const double u = __dsub_rn(x[j], __dmul_rn(Ct[q][4 * sl + j], e));
                    x[j] = (4 * sl + j > q) ? u : x[j];
                }
            }
            if (pos == 0 && live)                          // four codes: two bytes, low nibble = even index
                *reinterpret_cast<uint16_t*>(qw + (size_t)idx * (K >> 1) + (i0 >> 1) + 2 * it) = (uint16_t)codes;
#pragma unroll
            for (int j = 0; j < 4; ++j) x[j] = row_turn(x[j]);
        }
        return;
    }
    for (int it = 0; it < 16; ++it) {
        const int sl = (pos + it) & 15;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int q = 4 * it + k;
            const double c = row_first(x[k]);
            double e = c;
            if (role == 0) {
                if (pos == 0) HcT[(size_t)q * K + idx] = c;
            } else {
                e = __ddiv_rn(c, dt[q]);
                if (pos == 0) {
                    HrT[(size_t)q * K + idx] = c;
                    T[(size_t)q * K + idx] = e;
                }
            }
            const double* tab = (role == 0) ? Rt[q] : Ct[q];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const double u = __dsub_rn(x[j], __dmul_rn(tab[4 * sl + j], e));
                x[j] = (4 * sl + j > q) ? u : x[j];
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = row_turn(x[j]);
    }
}

// ---- X[a][b] <- (..((X[a][b] - L[0][a] R[0][b]) - L[1][a] R[1][b]).. - L[63][a] R[63][b]) over rows a0 + [0, rows)
// and columns b0 + [0, cols), leaving out the 64 indices from `skip` on in both directions (skip < 0: none; rows and
// cols count what is left).  L and R are [PB][ld].
struct RankUpdate {
    double* X;
    const double *L, *R;
    size_t ldx, ldl, ldr;
    int a0, rows, b0, cols, skip;
    int tiles_b;                 // tiles along b
    int tiles;                   // tiles in all
};

// A block takes a tile of 16 TT x 16 TT elements, TT x TT per thread: two binary64 operations per element and pivot are
// the floor (4 clocks per wave each: 64 K^2 elements and pivots are 83 us at K = 5120), and TT = 8 needs 16 LDS values
// for 64 updates, half of what LDS delivers meanwhile; TT = 4 needs all of it and is for matrices with too few tiles.
// Two problems share a launch (blocks of u0 first), and with Dnew one more block puts the panel's diagonal block back.
template <int TT>
__global__ __launch_bounds__(256, 2)
void rank_update_kernel(const RankUpdate u0, const RankUpdate u1, const double* __restrict__ Dnew, int K, int p0) {
    constexpr int BT = 16 * TT, QC = 32;
    __shared__ __attribute__((aligned(16))) double Ls[QC][BT], Rs[QC][BT];
    int bid = blockIdx.x;
    if (bid >= u0.tiles + u1.tiles) {                       // u0.X is the matrix of the inverse here
        for (int e = threadIdx.x; e < PB * PB; e += 256) u0.X[(size_t)(p0 + e / PB) * K + p0 + e % PB] = Dnew[e];
        return;
    }
    const bool first = bid < u0.tiles;
    const RankUpdate& u = first ? u0 : u1;
    if (!first) bid -= u0.tiles;
    const int ta = (bid / u.tiles_b) * BT, tb = (bid % u.tiles_b) * BT;
    auto place = [&](const int base, const int i) {         // i-th index that is not left out
        const int g = base + i;
        return (u.skip >= 0 && g >= u.skip) ? g + PB : g;
    };
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    double x[TT][TT];
    size_t row[TT];
    int col[TT];
#pragma unroll
    for (int i = 0; i < TT; ++i) {
        row[i] = (size_t)place(u.a0, ta + ty * TT + i) * u.ldx;
        col[i] = place(u.b0, tb + tx + 16 * i);
    }
#pragma unroll
    for (int i = 0; i < TT; ++i)
#pragma unroll
        for (int j = 0; j < TT; ++j)
            x[i][j] = (ta + ty * TT + i < u.rows && tb + tx + 16 * j < u.cols) ? u.X[row[i] + col[j]] : 0.0;
    const int lc = threadIdx.x % BT, lq = threadIdx.x / BT;
    const bool lin = ta + lc < u.rows, rin = tb + lc < u.cols;
    const double* lp = u.L + (lin ? place(u.a0, ta + lc) : 0);
    const double* rp = u.R + (rin ? place(u.b0, tb + lc) : 0);
    for (int q0 = 0; q0 < PB; q0 += QC) {
        if (q0) __syncthreads();
#pragma unroll
        for (int q = 0; q < QC; q += 256 / BT) {
            Ls[q + lq][lc] = lin ? lp[(size_t)(q0 + q + lq) * u.ldl] : 0.0;
            Rs[q + lq][lc] = rin ? rp[(size_t)(q0 + q + lq) * u.ldr] : 0.0;
        }
        __syncthreads();
        for (int q = 0; q < QC; ++q) {
            double l[TT], r[TT];
#pragma unroll
            for (int i = 0; i < TT; ++i) l[i] = Ls[q][ty * TT + i];
#pragma unroll
            for (int j = 0; j < TT; ++j) r[j] = Rs[q][tx + 16 * j];
#pragma unroll
            for (int i = 0; i < TT; ++i)
#pragma unroll
                for (int j = 0; j < TT; ++j) x[i][j] = __dsub_rn(x[i][j], __dmul_rn(l[i], r[j]));
        }
    }
#pragma unroll
    for (int i = 0; i < TT; ++i)
#pragma unroll
        for (int j = 0; j < TT; ++j)
            if (ta + ty * TT + i < u.rows && tb + tx + 16 * j < u.cols) u.X[row[i] + col[j]] = x[i][j];
}

void launch_rank_updates(RankUpdate u0, RankUpdate u1, const double* Dnew, int K, int p0, hipStream_t stream) {
    auto set = [](RankUpdate& u, int bt) {
        u.tiles_b = (u.cols + bt - 1) / bt;
        u.tiles = (u.rows > 0 && u.cols > 0) ? u.tiles_b * ((u.rows + bt - 1) / bt) : 0;
    };
    set(u0, 128);
    set(u1, 128);
    const int extra = Dnew ? 1 : 0;
    if (u0.tiles + u1.tiles >= 256) {                       // at least one large tile for every compute unit
        hipLaunchKernelGGL(rank_update_kernel<8>, dim3(u0.tiles + u1.tiles + extra), dim3(256), 0, stream, u0, u1, Dnew, K, p0);
        return;
    }
    set(u0, 64);
    set(u1, 64);
    if (u0.tiles + u1.tiles + extra)
        hipLaunchKernelGGL(rank_update_kernel<4>, dim3(u0.tiles + u1.tiles + extra), dim3(256), 0, stream, u0, u1, Dnew, K, p0);
}

inline size_t up256(size_t v) { return (v + 255) & ~(size_t)255; }

}  // namespace

size_t gptq_workspace_bytes(int N, int K) {
    return up256((size_t)K * K * 8) + up256((size_t)K * N * 8) + 3 * up256((size_t)K * PB * 8) + up256((size_t)PB * N * 8) +
           up256((size_t)(PB * PB + 1) * 8);
}

hipError_t launch_gptq_hessian(const void* x, int64_t ldx, const float* inv_lambda, int64_t M, int K, double* H,
                               hipStream_t stream) {
    const unsigned t = (unsigned)((K + HT - 1) / HT);
    hipLaunchKernelGGL(hessian_kernel, dim3(t, t), dim3(256), 0, stream, (const uint16_t*)x, ldx, inv_lambda, M, K, H);
    return hipGetLastError();
}

hipError_t launch_gptq_quantize(const float* R, const double* H, double damp, int N, int K, void* workspace,
                                uint8_t* qw, float* sw, hipStream_t stream) {
    uint8_t* p = (uint8_t*)workspace;
    double* A = (double*)p;        p += up256((size_t)K * K * 8);
    double* W = (double*)p;        p += up256((size_t)K * N * 8);
    double* Lc = (double*)p;       p += up256((size_t)K * PB * 8);     // saved pivot columns         [PB][K]
    double* Rr = (double*)p;       p += up256((size_t)K * PB * 8);     // saved scaled pivot rows     [PB][K]
    double* Hr = (double*)p;       p += up256((size_t)K * PB * 8);     // saved rows of H^-1          [PB][K]
    double* Err = (double*)p;      p += up256((size_t)PB * N * 8);     // errors of the panel         [PB][N]
    double* Dnew = (double*)p;                                         // diagonal block of the panel [PB][PB], damping
    double* add = Dnew + PB * PB;
    hipLaunchKernelGGL(diag_sum_kernel, dim3(1), dim3(256), 0, stream, H, damp, K, add);
    hipLaunchKernelGGL(prepare_kernel, dim3(K), dim3(256), 0, stream, R, H, add, N, K, A, W);
    const size_t ldk = (size_t)K, ldn = (size_t)N;
    const RankUpdate none{A, nullptr, nullptr, ldk, ldk, ldk, 0, 0, 0, 0, -1, 1, 0};
    const int np = K / PB;
    for (int p0 = 0; p0 < K; p0 += PB) {               // the inverse, one panel of pivots at a time
        hipLaunchKernelGGL(gj_panel_kernel, dim3(2 * (np - 1) + 1), dim3(PTHREADS), 0, stream, A, K, p0, Lc, Rr, Dnew);
        launch_rank_updates(RankUpdate{A, Lc, Rr, ldk, ldk, ldk, 0, K - PB, 0, K - PB, p0, 1, 0}, none, Dnew, K, p0, stream);
    }
    for (int i0 = 0; i0 < K; i0 += PB) {               // the weights, one panel (= one 64-group) at a time
        const int i1 = i0 + PB, rest = K - i1;
        hipLaunchKernelGGL(visit_panel_kernel, dim3(2 * (rest / PB) + (N + PB - 1) / PB), dim3(PTHREADS), 0, stream,
                           A, W, N, K, i0, Lc, Hr, Rr, Err, qw, sw);
        if (rest > 0)                                   // the deferred updates of everything behind the panel
            launch_rank_updates(RankUpdate{W, Hr, Err, ldn, ldk, ldn, i1, rest, 0, N, -1, 1, 0},
                                RankUpdate{A, Lc, Rr, ldk, ldk, ldk, i1, rest, i1, rest, -1, 1, 0}, nullptr, K, i0, stream);
    }
    return hipGetLastError();
}

}  // namespace svdq
