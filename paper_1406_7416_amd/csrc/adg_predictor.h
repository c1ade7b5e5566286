// Local space-time predictor (a point-owner / line-owner LDS design, see below).
#pragma once
#include <type_traits>

#include "adg_physics.h"

namespace adg {

// ------------------------------------------------------------- space-time predictor
// Eq. (pde.nc.dg2) in nodal form (spatial weights divided out, K1^{-1} L = 1):
//   q^{r+1}(a,s) = u(a) - sum_t Kw[s][t] S(a,t),
//   S(a,t) = sum_k (dt/h_k) sum_b D[a_k][b] F_k(q^r(a|b, t))
// Thread mapping: a "point owner" thread holds one spatial node of one cell with its
// whole time pencil (NV x n values) in registers.  It evaluates the fluxes of the pencil
// and stores them in LDS; "line owner" threads do the length-n spatial contractions
// (n loads -> n outputs each, in place); the point owner accumulates S over the d axes
// and applies the time contraction in registers: d + 1 contractions per sweep.
// What bounds it: vector instructions, the matrix unit and LDS take about a third of the time each
// (2D N = 9, FP32: 36 %, 34 %, 42 %), one after the other between the barriers of a workgroup, with
// four waves per SIMD to overlap them.  So FP32 has its contractions on the matrix unit, 8-byte LDS
// accesses without bank conflicts (33 % of the LDS time before) and no barrier between a point's
// last read and its owner's next store; traces and volume term take one line / node per thread.
// Measured against contractions on the vector unit, 4-byte accesses and items spread over the
// threads (FP32): 2D N = 5, 400 x 100 cells 246 -> 192 us; N = 4, 131 x 75 41.9 -> 31.2 us; N = 3,
// 48 problems 474 -> 302 us; N = 9, 64 x 64 240 -> 232 us; 3D N = 3, 128^3 17.9 -> 12.7 ms.  FP64
// (traces, volume term and barriers only): 3D N = 3, 64^3 4.63 -> 4.05 ms.  FP64 then spent most of
// its LDS time on operator entries broadcast to the lanes (2D N = 9: 1650 of 2290 cycles per wave and
// sweep); from the scalar cache they cost none: vortex N = 9, 32 x 32 cells, Osher flux, 5 steps
// 941 -> 751 us; 12 problems N = 3..5, 5 steps 4.29 -> 4.08 ms.
template <int DIM, int N, typename R = double, int TB = Tune<DIM, N, sizeof(R) == 4>::pred_tb>
struct PredShape;

// 1/x: correctly rounded division in FP64; the hardware reciprocal (within 1 ulp) in
// the FP32 working precision of the mixed form.
__device__ __forceinline__ double recip(double x) { return 1.0 / x; }
__device__ __forceinline__ float recip(float x) { return __builtin_amdgcn_rcpf(x); }

// x / d with ir = recip(d): the division itself in FP64; in FP32 the product corrected by its
// residual, which rounds like the division while d, 1 / d and the quotient are normal numbers.
__device__ __forceinline__ double quotient(double x, double d, double) { return x / d; }
__device__ __forceinline__ float quotient(float x, float d, float ir) {
    const float y = x * ir;
    return fmaf(fmaf(-y, d, x), ir, y);
}

// TB: thread budget of a workgroup (cells per block = TB / n^d)
template <int DIM, int N, typename R, int TB>
struct PredShape {
    static constexpr int n = N + 1;
    static constexpr int NV = DIM + 2;
    static constexpr int NN = cpow(n, DIM);
    static constexpr int NST = NN * n;
    static constexpr int NFN = cpow(n, DIM - 1);
    static constexpr int CPB = NN <= TB ? TB / NN : 1;
    static constexpr int ACT = CPB * NN;                           // active point owners
    static constexpr int BS = ((ACT + 63) / 64) * 64;
    // pencil and flux sums exceed the 128 registers that a workgroup of more than 512 threads leaves a lane
    static constexpr bool TIGHT = BS > 512 && 2 * NV * n * (int)sizeof(R) / 4 > 128;
    // variables per LDS chunk: all where they fit 80 KB, half of a CU's LDS (a second chunk makes the
    // pencils indexed arrays, which live in scratch: 2D N = 8 FP64, 70 KB, in chunks of three of its
    // four variables 4.11 ms on 128 x 128 cells, in one 0.93 ms); else as many as 64 KB hold
    static constexpr int VB = CPB * NST * (int)sizeof(R);   // LDS of one variable
    static constexpr int VC = NV * VB <= 81920 ? NV : (VB <= 65536 ? 65536 / VB : 1);
};

// ---- FP32 contractions on the matrix unit (4x4x1, 16 blocks).  Lane l of a wave is column l % 4
// of block l / 4: its B operand is one value of the pencil or line it owns and the four
// registers of the accumulator are four consecutive outputs of that line, so a lane's data stay
// in its own registers.  The A operand is broadcast from one block (lane group) to all sixteen:
// block b of one register holds column b of four operator rows, so a whole operator of n <= 10
// nodes takes one register per four rows and no operand is read in the loops.
typedef float mvec __attribute__((ext_vector_type(4)));
template <int B>
__device__ __forceinline__ mvec mat4(float a, float x, mvec acc) {
    return __builtin_amdgcn_mfma_f32_4x4x1f32(a, x, acc, 4, B, 0);
}
// acc[g] += (rows 4g .. 4g + 3, columns B .. B + C - 1 of the operator in a) x[0 .. C - 1]
template <int B, int C, int G>
__device__ __forceinline__ void mat_cols(const float *a, const float *x, mvec *acc) {
    if constexpr (C > 0) {
#pragma unroll
        for (int g = 0; g < G; g++) acc[g] = mat4<B>(a[g], x[0], acc[g]);
        mat_cols<B + 1, C - 1, G>(a, x + 1, acc);
    }
}
template <int N>
struct MatOps {
    static constexpr int n = N + 1, h = n / 2, hu = n - h;
    static constexpr bool EO = n >= 6;          // even / odd form of the derivative
    static constexpr int G = (n + 3) / 4;       // row groups of an n x n operator
    static constexpr int GE = (h + 3) / 4, GO = (hu + 3) / 4, GD = EO ? GO : G;
    static constexpr int OB = 8;                // first block of the odd part (columns of the even part: hu <= 5)
    float kw[G];                                // time operator
    float d[GD];                                // derivative: E in blocks 0 .., O in blocks OB ..
};
// Layout of the predictor's LDS array: every cell holds VC variables at n^d nodes and n time
// levels.  FP64 and n < 4: one plane per variable.  Matrix-unit form: variables in pairs (8-byte
// accesses; a last odd variable alone) and an odd number of nodes per time level, so that with
// the line order of LineMap the 16 lanes of an 8-byte access start in 16 different bank pairs.
template <int DIM, int N, int VC, typename R>
struct PredLds {
    static constexpr int n = N + 1;
    static constexpr bool MAT = sizeof(R) == 4 && n >= 4;
    static constexpr int SS = MAT ? cpow(n, DIM) | 1 : cpow(n, DIM);   // time level
    static constexpr int PTS = SS * n;                        // points of one variable
    static constexpr int CELL = MAT ? (VC * PTS + 1) / 2 * 2 : VC * PTS;
    static constexpr bool paired(int v) { return MAT && (v | 1) < VC; }
    static constexpr int at(int v) { return paired(v) ? v / 2 * 2 * PTS + (v & 1) : v * PTS; }
    static constexpr int es(int v) { return paired(v) ? 2 : 1; }
    static constexpr int stride(int k) { return k == 0 ? 1 : (k == 1 ? n : n * n); }   // along axis k
    // first point of line j = a_perp + n^(d-1) s along axis k
    static constexpr int line(int k, int j) {
        const int nf = cpow(n, DIM - 1), st = stride(k), ap = j % nf;
        return SS * (j / nf) + ap % st + ap / st * st * n;
    }
};
// The line that thread i contracts along axis k (cell * n^d + j), one per thread.  Matrix-unit
// form: ordered so that every 16 threads take lines of different bank pairs as far as there are
// any left (neighbouring lines along x are n nodes apart, 2 to 8 of 16 in the same bank pair).  3D
// N = 9 holds one variable at a time, in 4-byte accesses that this order is not made for.
template <int DIM, int N, int CPB, int VC, typename R>
struct LineMap {
    static constexpr int NN = cpow(N + 1, DIM), ACT = CPB * NN;
    uint16_t line[DIM][ACT];
    constexpr LineMap() : line{} {
        using L = PredLds<DIM, N, VC, R>;
        for (int k = 0; k < DIM; k++) {
            if (!L::MAT) {
                for (int i = 0; i < ACT; i++) line[k][i] = (uint16_t)i;
                continue;
            }
            // lines by bank pair: first[b] .. in order, next[i] the following one
            int head[16] = {}, left[16] = {};
            uint16_t next[ACT] = {};
            for (int b = 0; b < 16; b++) head[b] = -1;
            for (int i = ACT - 1; i >= 0; i--) {
                const int b = (i / NN * (L::CELL / 2) + L::line(k, i % NN)) % 16;
                next[i] = (uint16_t)(head[b] + 1);
                head[b] = i;
                left[b]++;
            }
            for (int i = 0; i < ACT;) {
                // one line of each of the bank pairs with most lines left, largest first
                bool used[16] = {};
                int m = 0;
                for (; m < 16 && i < ACT; m++) {
                    int best = -1;
                    for (int b = 0; b < 16; b++)
                        if (!used[b] && left[b] && (best < 0 || left[b] > left[best])) best = b;
                    if (best < 0) {
                        for (int b = 0; b < 16; b++) used[b] = false;
                        m--;
                        continue;
                    }
                    used[best] = true;
                    line[k][i++] = (uint16_t)head[best];
                    head[best] = (int)next[head[best]] - 1;
                    left[best]--;
                }
            }
        }
    }
};
template <int DIM, int N, int CPB, int VC, typename R>
static __device__ const LineMap<DIM, N, CPB, VC, R> line_map{};
template <typename R> struct PairOf;
template <> struct PairOf<float> { typedef float type __attribute__((ext_vector_type(2))); };
template <> struct PairOf<double> { typedef double type __attribute__((ext_vector_type(2))); };
// f(v, x) of every variable v < VC of the point (one or two per access)
template <typename L, int VC, typename R, typename F>
__device__ __forceinline__ void lds_get(const R *X, int pt, F f) {
#pragma unroll
    for (int v = 0; v < VC; v += 2) {
        if (L::paired(v)) {
            const auto x = *reinterpret_cast<const typename PairOf<R>::type *>(X + L::at(v) + 2 * pt);
            f(v, x[0]);
            f(v + 1, x[1]);
        } else {
            f(v, X[L::at(v) + pt]);
            if (v + 1 < VC) f(v + 1, X[L::at(v + 1) + pt]);
        }
    }
}
// the point's variables v < VC set to f(v)
template <typename L, int VC, typename R, typename F>
__device__ __forceinline__ void lds_put(R *X, int pt, F f) {
#pragma unroll
    for (int v = 0; v < VC; v += 2) {
        if (L::paired(v)) {
            typename PairOf<R>::type x;
            x[0] = f(v);
            x[1] = f(v + 1);
            *reinterpret_cast<typename PairOf<R>::type *>(X + L::at(v) + 2 * pt) = x;
        } else {
            X[L::at(v) + pt] = f(v);
            if (v + 1 < VC) X[L::at(v + 1) + pt] = f(v + 1);
        }
    }
}
// y = D x of one line in a lane's registers
template <int N>
__device__ __forceinline__ void mat_line(const MatOps<N> &M, const float *x, float *y) {
    using O = MatOps<N>;
    constexpr int n = O::n, h = O::h;
    if constexpr (O::EO) {
        float e[O::hu], o[h];
#pragma unroll
        for (int b = 0; b < h; b++) {
            e[b] = x[b] + x[n - 1 - b];
            o[b] = x[b] - x[n - 1 - b];
        }
        if constexpr (n % 2) e[h] = x[h];
        mvec pe[O::GE] = {}, po[O::GO] = {};
        mat_cols<0, O::hu, O::GE>(M.d, e, pe);
        mat_cols<O::OB, h, O::GO>(M.d, o, po);
#pragma unroll
        for (int i = 0; i < h; i++) {
            y[i] = po[i / 4][i % 4] + pe[i / 4][i % 4];
            y[n - 1 - i] = po[i / 4][i % 4] - pe[i / 4][i % 4];
        }
        if constexpr (n % 2) y[h] = po[h / 4][h % 4];
    } else {
        mvec acc[O::G] = {};
        mat_cols<0, n, O::G>(M.d, x, acc);
#pragma unroll
        for (int i = 0; i < n; i++) y[i] = acc[i / 4][i % 4];
    }
}
// Contraction with the derivative matrix along axis k of the line that starts at point pt, of
// every variable, in place.  The matrix unit ignores the execution mask, so a wave enters as a
// whole; lanes that have no line of their own read one and store nothing.
template <int DIM, int N, int VC>
__device__ __forceinline__ void mat_lines(float *X, int k, int pt, bool store, const MatOps<N> &M) {
    using L = PredLds<DIM, N, VC, float>;
    constexpr int n = N + 1;
    typedef PairOf<float>::type pair;
    const int st = L::stride(k);
#pragma unroll
    for (int v = 0; v < VC; v += 2) {
        // compiler barrier: one pair's line in registers at a time
        __asm__ volatile("" ::: "memory");
        float x[2][n], y[2][n];
        if (L::paired(v)) {
            pair *line = reinterpret_cast<pair *>(X + L::at(v)) + pt;
#pragma unroll
            for (int b = 0; b < n; b++) {
                const pair p = line[b * st];
                x[0][b] = p[0];
                x[1][b] = p[1];
            }
            mat_line<N>(M, x[0], y[0]);
            mat_line<N>(M, x[1], y[1]);
            if (store) {
#pragma unroll
                for (int b = 0; b < n; b++) line[b * st] = pair{y[0][b], y[1][b]};
            }
        } else {
            float *line = X + L::at(v) + pt;
#pragma unroll
            for (int b = 0; b < n; b++) x[0][b] = line[b * st];
            mat_line<N>(M, x[0], y[0]);
            if (store) {
#pragma unroll
                for (int b = 0; b < n; b++) line[b * st] = y[0][b];
            }
        }
    }
}

// Operator entries of the vector-unit form, the same for every lane: read through the scalar cache.
// The pointer is made uniform, and opaque at every use, so that a row is loaded where it is used
// instead of all rows being held (and spilled) across the sweeps.
template <typename R> using OpPtr = const R __attribute__((address_space(4))) *;
template <typename R>
__device__ __forceinline__ OpPtr<R> op_ptr(const R *p) {
    const uint64_t b = (uint64_t)p;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
    return (OpPtr<R>)((uint64_t)hi << 32 | lo);
}
template <typename R>
__device__ __forceinline__ OpPtr<R> here(OpPtr<R> p) {
    __asm__ volatile("" : "+s"(p));
    return p;
}

// Contraction along axis k of every line held in LDS: line[i] <- sum_b M[i][b] line[b].
// One work item handles the same line of LV variables (independent FMA chains sharing each
// operator entry; one variable for long lines, to bound register use).
// EO: M is the derivative matrix on symmetric nodes, applied through its even / odd parts
// E, O (half-size products on x_b +- x_{n-1-b}: n^2/2 + 2n operations instead of n^2).
template <int DIM, int N, int CPB, int VC, int BS, typename R, bool EO>
__device__ __forceinline__ void lds_lines(R *X, int k, int nlines_per_var, int lstride_s, OpPtr<R> M, int tid,
                                          int nvalid, OpPtr<R> E, OpPtr<R> O) {
    constexpr int n = N + 1, NN = cpow(n, DIM), NST = NN * n;
    constexpr int LV = (n >= 8) ? 1 : VC;
    constexpr int NG = (VC + LV - 1) / LV;   // variable groups per line
    const int st = (k == 0) ? 1 : (k == 1 ? n : n * n);
    const int nitems = CPB * NG * nlines_per_var;
    for (int it = tid; it < nitems; it += BS) {
        // compiler barrier: keeps the operator rows from being hoisted into registers
        __asm__ volatile("" ::: "memory");
        const int lcl = it / (NG * nlines_per_var);
        const int grp = (it / nlines_per_var) % NG;
        const int j = it % nlines_per_var;          // (a_perp, s) flattened, a_perp fastest
        const int s = j / (NN / n), ap = j % (NN / n);
        int base = 0, rem = ap, mul = 1;
#pragma unroll
        for (int jj = 0; jj < DIM; jj++) {
            if (jj == k) { mul *= n; continue; }
            base += (rem % n) * mul;
            rem /= n;
            mul *= n;
        }
        const int v0 = grp * LV;
        R *line0 = &X[(lcl * VC + v0) * NST + lstride_s * s + base];
        R xb[LV][n];
#pragma unroll
        for (int vv = 0; vv < LV; vv++)
#pragma unroll
            for (int b = 0; b < n; b++) xb[vv][b] = (v0 + vv < nvalid) ? line0[vv * NST + b * st] : R(0);
        if constexpr (EO) {
            constexpr int h = n / 2;
            R e[LV][h], o[LV][h];
#pragma unroll
            for (int vv = 0; vv < LV; vv++)
#pragma unroll
                for (int b = 0; b < h; b++) {
                    e[vv][b] = xb[vv][b] + xb[vv][n - 1 - b];
                    o[vv][b] = xb[vv][b] - xb[vv][n - 1 - b];
                }
#pragma unroll
            for (int i = 0; i < h; i++) {
                E = here(E);
                O = here(O);
                R pe[LV], po[LV];
#pragma unroll
                for (int vv = 0; vv < LV; vv++) pe[vv] = po[vv] = 0;
#pragma unroll
                for (int b = 0; b < h; b++) {
                    const R me = E[i * (MAXN / 2 + 1) + b], mo = O[i * (MAXN / 2) + b];
#pragma unroll
                    for (int vv = 0; vv < LV; vv++) {
                        pe[vv] += me * e[vv][b];
                        po[vv] += mo * o[vv][b];
                    }
                }
                if constexpr (n % 2) {
                    const R mm = E[i * (MAXN / 2 + 1) + h];
#pragma unroll
                    for (int vv = 0; vv < LV; vv++) pe[vv] += mm * xb[vv][h];
                }
#pragma unroll
                for (int vv = 0; vv < LV; vv++)
                    if (v0 + vv < nvalid) {
                        const R yi = po[vv] + pe[vv], yr = po[vv] - pe[vv];
                        line0[vv * NST + i * st] = yi;
                        line0[vv * NST + (n - 1 - i) * st] = yr;
                    }
            }
            if constexpr (n % 2) {
                R acc[LV];
#pragma unroll
                for (int vv = 0; vv < LV; vv++) acc[vv] = 0;
#pragma unroll
                for (int b = 0; b < h; b++) {
                    const R mo = O[h * (MAXN / 2) + b];
#pragma unroll
                    for (int vv = 0; vv < LV; vv++) acc[vv] += mo * o[vv][b];
                }
#pragma unroll
                for (int vv = 0; vv < LV; vv++)
                    if (v0 + vv < nvalid) line0[vv * NST + h * st] = acc[vv];
            }
        } else {
#pragma unroll
            for (int i = 0; i < n; i++) {
                R acc[LV];
#pragma unroll
                for (int vv = 0; vv < LV; vv++) acc[vv] = 0;
#pragma unroll
                for (int b = 0; b < n; b++) {
                    const R m = M[i * MAXN + b];
#pragma unroll
                    for (int vv = 0; vv < LV; vv++) acc[vv] += m * xb[vv][b];
                }
#pragma unroll
                for (int vv = 0; vv < LV; vv++)
                    if (v0 + vv < nvalid) line0[vv * NST + i * st] = acc[vv];
            }
        }
    }
}

// Blocks vb = vb0, vb0 + vbs, ... of CPB cells each, out of ncell cells.
// DEV (FP32 working precision only): the pencils carry the deviation dq = q - c from the cell's
// reference state c (its first nodal value rounded to FP32) and the fluxes are evaluated as
// F(c + dq) - F(c) in the expanded form of dev_flux; the derivative matrix annihilates the
// constant F(c), so the Picard iteration, the volume term and the traces are those of the
// deviations, and FP32 rounding is relative to the deviation instead of the state.
template <int DIM, int N, bool VOL, typename R, bool DEV = false, int TB = Tune<DIM, N, sizeof(R) == 4>::pred_tb>
__device__ __forceinline__ void pred_cells(const PredArgs<R> &A, double gamma_d, int64_t ncell, int64_t vb0, int64_t vbs) {
    static_assert(!DEV || sizeof(R) == 4, "the deviation form is an FP32 form");
    using S = PredShape<DIM, N, R, TB>;
    const R gamma = (R)gamma_d;
    constexpr int n = S::n, NV = S::NV, NN = S::NN, NFN = S::NFN, CPB = S::CPB, VC = S::VC;
    using L = PredLds<DIM, N, VC, R>;
    constexpr bool MAT = L::MAT;
    __shared__ __align__(16) R X[CPB * L::CELL];
    __shared__ R Dvs[n][MAXN], ws[MAXN], Bs[2][MAXN];
    // the spatial contractions use the even / odd form where it saves work (n >= 6)
    constexpr bool EO = n >= 6;

    const int tid = threadIdx.x;
    const int lc = tid / NN, a = tid % NN;
    const double dt = *A.dt;
    for (int i = tid; i < n * n; i += S::BS) {
        const int r = i / n, cc = i % n;
        Dvs[r][cc] = VOL ? A.Dvol[r * MAXN + cc] : R(0);
    }
    if (tid < n) {
        ws[tid] = VOL ? A.w[tid] : R(0);
        Bs[0][tid] = A.Lb[tid];
        Bs[1][tid] = A.Rb[tid];
    }
    __syncthreads();
    const OpPtr<R> D = op_ptr(A.D), Kw = op_ptr(A.Kw), DE = op_ptr(A.DE), DO = op_ptr(A.DO);
    const R(*Dvol)[MAXN] = Dvs;
    MatOps<N> M;
    if constexpr (MAT) {
        const int row = tid & 3, col = (tid & 63) >> 2;
#pragma unroll
        for (int g = 0; g < MatOps<N>::G; g++) {
            const int r = 4 * g + row;
            M.kw[g] = (r < n && col < n) ? A.Kw[r * MAXN + col] : R(0);
        }
#pragma unroll
        for (int g = 0; g < MatOps<N>::GD; g++) {
            const int r = 4 * g + row, oc = col - MatOps<N>::OB;
            if constexpr (EO) {
                M.d[g] = (r < n / 2 && col < n - n / 2) ? A.DE[r * (MAXN / 2 + 1) + col]
                         : (r < n - n / 2 && oc >= 0 && oc < n / 2) ? A.DO[r * (MAXN / 2) + oc] : R(0);
            } else {
                M.d[g] = (r < n && col < n) ? A.D[r * MAXN + col] : R(0);
            }
        }
    }
    // this thread's point (slice 0), and the line of each axis that it contracts (threads past the
    // last cell: the last ones, and store nothing)
    const bool act = tid < S::ACT;
    const int ia = act ? tid : S::ACT - 1, la = ia % NN;
    R *Xc = X + ia / NN * L::CELL;
    int lcell[DIM], lj[DIM], lpt[DIM];   // its cell, its number in the cell and its first point
#pragma unroll
    for (int k = 0; k < DIM; k++) {
        const int i = MAT ? line_map<DIM, N, CPB, VC, R>.line[k][ia] : ia;
        lcell[k] = i / NN;
        lj[k] = i % NN;
        lpt[k] = L::line(k, lj[k]);
    }
    // persistent over blocks of CPB cells (uniform per block: barriers stay legal)
    for (int64_t vb = vb0; vb * CPB < ncell; vb += vbs) {
    const int64_t c = vb * CPB + lc;
    const bool owner = act && (c < ncell);

    R u0[NV], q[NV][n], Sacc[NV][n];
    DevRef<DIM, R> cref;
    if (owner) {
        if constexpr (DEV) {
            double c64[NV];
#pragma unroll
            for (int v = 0; v < NV; v++) c64[v] = A.in[c * A.in_cstride + v * A.in_vstride];
            cref = make_devref<DIM, R>(c64, gamma_d);
#pragma unroll
            for (int v = 0; v < NV; v++) u0[v] = (R)(A.in[c * A.in_cstride + v * A.in_vstride + a] - (double)cref.q[v]);
        } else {
#pragma unroll
            for (int v = 0; v < NV; v++) u0[v] = (R)A.in[c * A.in_cstride + v * A.in_vstride + a];
        }
    } else {
        // idle lanes carry a valid constant state so that they never produce NaN
#pragma unroll
        for (int v = 0; v < NV; v++) u0[v] = (v == 0 && !DEV) ? R(1) : R(0);
        if constexpr (!DEV) u0[NV - 1] = R(2.5);
        if constexpr (DEV) {
            double c64[NV];
#pragma unroll
            for (int v = 0; v < NV; v++) c64[v] = (v == 0) ? 1.0 : 0.0;
            c64[NV - 1] = 2.5;
            cref = make_devref<DIM, R>(c64, gamma_d);
        }
    }
#pragma unroll
    for (int v = 0; v < NV; v++)
#pragma unroll
        for (int s = 0; s < n; s++) q[v][s] = u0[v];

    // One Picard sweep.  In the first the iterate is u^n at every time node, so every time slice
    // of the fluxes and of their spatial derivatives is the same: only slice 0 is computed and
    // it stands for all of them (equal to the full sweep in exact arithmetic; the compiled code
    // may round differently, by a few units in the last place).
    auto sweep = [&](auto first_c) __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(first_c)::value;
        constexpr int NT = FIRST ? 1 : n;   // time slices computed
        // (opaque per sweep: the LDS addresses are formed where they are used instead of being
        // held, and spilled, across the sweeps)
        int pt = la;
        __asm__ volatile("" : "+v"(pt));
        // 1/rho of every node of the pencil, shared by the fluxes of all axes (for long FP64 pencils
        // recomputed per axis instead, to stay within 256 registers, and for long pencils of the
        // deviation form to stay within 128: vortex N = 9, 64 x 64 cells, 10 steps 3.41 -> 3.19 ms)
        constexpr bool CACHE_IRHO = n < 8 || (sizeof(R) == 4 && !(DEV && n >= 8));
        R irho[CACHE_IRHO ? n : 1], pr[CACHE_IRHO ? n : 1];
        if constexpr (CACHE_IRHO) {
#pragma unroll
            for (int t = 0; t < NT; t++) {
                if constexpr (DEV) {
                    // deviation form: 1/rho of the full state and the pressure's deviation
                    R dq[NV];
#pragma unroll
                    for (int v = 0; v < NV; v++) dq[v] = q[v][t];
                    irho[t] = recip(cref.q[0] + dq[0]);
                    pr[t] = dev_pressure<DIM, R>(cref, dq, irho[t], gamma);
                } else {
                    irho[t] = recip(q[0][t]);
                    R ke = 0;
#pragma unroll
                    for (int j = 0; j < DIM; j++) ke += q[1 + j][t] * q[1 + j][t];
                    pr[t] = (gamma - R(1)) * (q[NV - 1][t] - R(0.5) * ke * irho[t]);
                }
            }
        }
#pragma unroll
        for (int k = 0; k < DIM; k++) {
            const R ck = (R)(dt * A.dth[k]);
            for (int v0 = 0; v0 < NV; v0 += VC) {
                // point phase: fluxes of the time pencil straight into LDS
                if (tid < S::ACT) {
#pragma unroll
                    for (int t = 0; t < NT; t++) {
                        R ir;
                        if constexpr (CACHE_IRHO) ir = irho[t];
                        else ir = recip(DEV ? cref.q[0] + q[0][t] : q[0][t]);
                        const R un = q[1 + k][t] * ir;
                        R prt;
                        if constexpr (CACHE_IRHO) prt = pr[t];
                        else if constexpr (DEV) {
                            R dq[NV];
#pragma unroll
                            for (int v = 0; v < NV; v++) dq[v] = q[v][t];
                            prt = dev_pressure<DIM, R>(cref, dq, ir, gamma);
                        } else {
                            R ke = 0;
#pragma unroll
                            for (int j = 0; j < DIM; j++) ke += q[1 + j][t] * q[1 + j][t];
                            prt = (gamma - R(1)) * (q[NV - 1][t] - R(0.5) * ke * ir);
                        }
                        R F[NV];
                        if constexpr (DEV) {
                            R dq[NV];
#pragma unroll
                            for (int v = 0; v < NV; v++) dq[v] = q[v][t];
                            dev_flux<DIM, R>(k, cref, dq, ir, prt, F);
                        } else {
                            F[0] = q[1 + k][t];
#pragma unroll
                            for (int j = 0; j < DIM; j++) F[1 + j] = q[1 + j][t] * un + (j == k ? prt : R(0));
                            F[NV - 1] = un * (q[NV - 1][t] + prt);
                        }
                        lds_put<L, VC>(Xc, pt + L::SS * t, [&](int vv) __attribute__((always_inline)) {
                            return v0 + vv < NV ? F[v0 + vv] : R(0);
                        });
                    }
                }
                __syncthreads();
                if constexpr (MAT) {
                    constexpr int NIT = FIRST ? CPB * (NN / n) : S::ACT;   // lines
                    int cell = lcell[k], lp = lpt[k];
                    if constexpr (FIRST) {
                        const int it = tid < NIT ? tid : NIT - 1;
                        cell = it / (NN / n);
                        lp = L::line(k, it % (NN / n));
                    }
                    if (__builtin_amdgcn_readfirstlane(tid) < NIT)
                        mat_lines<DIM, N, VC>(X + cell * L::CELL, k, lp, tid < NIT, M);
                } else {
                    lds_lines<DIM, N, CPB, VC, S::BS, R, EO>(X, k, FIRST ? NN / n : NN, FIRST ? 0 : NN, here(D), tid,
                                                             NV - v0 < VC ? NV - v0 : VC, here(DE), here(DO));
                }
                __syncthreads();
                // S = sum_k (dt/h_k) D_k F_k, the factor applied while accumulating
                // (the next fluxes go to the points that this thread alone has just read: no barrier)
                if (act) {
#pragma unroll
                    for (int t = 0; t < n; t++) {
                        // one time node after the other: read ahead, the contracted values of the longest
                        // deviation pencil push its flux sums into scratch (2D N = 9: 57 -> 48 registers
                        // spilled, 18 fewer in a sweep; vortex, 128 x 128 cells, steps of 1066 -> 1037 us;
                        // N = 8 gains 1 % there and loses 2 % on 17 x 17 cells, N = 7 loses 1 %)
                        if constexpr (DEV && DIM == 2 && n >= 10 && !FIRST) __builtin_amdgcn_sched_barrier(0);
                        lds_get<L, VC>(Xc, pt + L::SS * (FIRST ? 0 : t), [&](int vv, R xk) __attribute__((always_inline)) {
                            if (v0 + vv < NV)
                                Sacc[v0 + vv][t] = (k == 0) ? ck * xk : Sacc[v0 + vv][t] + ck * xk;
                        });
                    }
                } else if (k == 0) {
#pragma unroll
                    for (int vv = 0; vv < VC; vv++)
                        if (v0 + vv < NV)
#pragma unroll
                            for (int t = 0; t < n; t++) Sacc[v0 + vv][t] = 0;
                }
                __asm__ volatile("" ::: "memory");
            }
        }
        // time contraction in registers: on the matrix unit, or with row s of Kw from the scalar cache,
        // shared by the variables.  Where pencil and flux sums exceed a lane's registers (TIGHT) the sums
        // come from scratch: one variable's at a time, against the rows two by two.  Left to itself the
        // compiler keeps the whole operator in scalar registers instead, whose spills cost 1750 lane
        // reads per sweep (24^3 cells of degree 9 in FP64: 87.6 -> 84.2 ms).  The first sweep's sums are
        // the same at every time node and stay in registers, so there the rows go one after the other.
        if constexpr (MAT) {
#pragma unroll
            for (int v = 0; v < NV; v++) {
                mvec acc[MatOps<N>::G] = {};
                mat_cols<0, n, MatOps<N>::G>(M.kw, Sacc[v], acc);
#pragma unroll
                for (int s = 0; s < n; s++) q[v][s] = u0[v] - acc[s / 4][s % 4];
            }
        } else if constexpr (S::TIGHT && !FIRST) {
#pragma unroll
            for (int v = 0; v < NV; v++) {
                R acc[n];
#pragma unroll
                for (int s = 0; s < n; s++) {
                    if (s % 2 == 0) __builtin_amdgcn_sched_barrier(0);
                    const OpPtr<R> row = here(Kw) + s * MAXN;
                    acc[s] = 0;
#pragma unroll
                    for (int t = 0; t < n; t++) acc[s] += row[t] * Sacc[v][t];
                }
#pragma unroll
                for (int s = 0; s < n; s++) q[v][s] = u0[v] - acc[s];
            }
        } else {
#pragma unroll
            for (int s = 0; s < n; s++) {
                if constexpr (S::TIGHT) __builtin_amdgcn_sched_barrier(0);
                const OpPtr<R> row = here(Kw) + s * MAXN;
                R acc[NV];
#pragma unroll
                for (int v = 0; v < NV; v++) acc[v] = 0;
#pragma unroll
                for (int t = 0; t < n; t++) {
                    const R kst = row[t];
#pragma unroll
                    for (int v = 0; v < NV; v++) acc[v] += kst * Sacc[v][t];
                }
#pragma unroll
                for (int v = 0; v < NV; v++) q[v][s] = u0[v] - acc[v];
            }
        }
    };
    if (A.iters > 0) sweep(std::true_type{});
    for (int r = 1; r < A.iters; r++) sweep(std::false_type{});

    // ---- volume term of eq. (pde.nc.gw2), divided by the diagonal mass:
    //   (dt/h_k) sum_b [w_b D[b][a_k] / w_{a_k}] sum_s w_s F_k(q(a|b, s))
    R Fi[VOL ? DIM : 1][NV];   // sum_s w_s F_k(q(a, s))
    if constexpr (VOL) {
#pragma unroll
        for (int v = 0; v < NV; v++)
#pragma unroll
            for (int k = 0; k < DIM; k++) Fi[k][v] = 0;
#pragma unroll
        for (int t = 0; t < n; t++) {
            __builtin_amdgcn_sched_barrier(0);
            R qt[NV], F[NV];
#pragma unroll
            for (int v = 0; v < NV; v++) qt[v] = q[v][t];
            const R ir = recip(DEV ? cref.q[0] + qt[0] : qt[0]);
            R pt_;
            if constexpr (DEV) pt_ = dev_pressure<DIM, R>(cref, qt, ir, gamma);
            else {
                R ke = 0;
#pragma unroll
                for (int j = 0; j < DIM; j++) ke += qt[1 + j] * qt[1 + j];
                pt_ = (gamma - R(1)) * (qt[NV - 1] - quotient(R(0.5) * ke, qt[0], ir));
            }
#pragma unroll
            for (int k = 0; k < DIM; k++) {
                if constexpr (DEV) {
                    dev_flux<DIM, R>(k, cref, qt, ir, pt_, F);
                } else {
                    const R un = quotient(qt[1 + k], qt[0], ir);
                    F[0] = qt[1 + k];
#pragma unroll
                    for (int j = 0; j < DIM; j++) F[1 + j] = qt[1 + j] * un + (j == k ? pt_ : R(0));
                    F[NV - 1] = un * (qt[NV - 1] + pt_);
                }
#pragma unroll
                for (int v = 0; v < NV; v++) Fi[k][v] += ws[t] * F[v];
            }
        }
        if constexpr (sizeof(R) == 4 && !DEV) {
            // An infinite, zero or subnormal density, or a quotient out of range: the residual is NaN
            // or the reciprocal has no bits.  Again by divisions.  (One test per node costs 0 to 0.7 % of
            // a step, most at 2D N = 4; at every quotient 0.5 to 1.3 %.)
            R all = 0, least = INFINITY;
#pragma unroll
            for (int t = 0; t < n; t++) least = fmin(least, fabs(recip(q[0][t])));
#pragma unroll
            for (int k = 0; k < DIM; k++)
#pragma unroll
                for (int v = 0; v < NV; v++) all += Fi[k][v];
            if (!(fabs(all) < R(INFINITY)) || least == R(0)) {
#pragma unroll
                for (int k = 0; k < DIM; k++) {
#pragma unroll
                    for (int v = 0; v < NV; v++) Fi[k][v] = 0;
#pragma unroll
                    for (int t = 0; t < n; t++) {
                        R qt[NV], F[NV];
#pragma unroll
                        for (int v = 0; v < NV; v++) qt[v] = q[v][t];
                        euler_flux<DIM, R>(k, qt, F, gamma);
#pragma unroll
                        for (int v = 0; v < NV; v++) Fi[k][v] += ws[t] * F[v];
                    }
                }
            }
        }
        // formed here, not where they are used: the pencils end with the traces
#pragma unroll
        for (int k = 0; k < DIM; k++)
#pragma unroll
            for (int v = 0; v < NV; v++) __asm__ volatile("" : "+v"(Fi[k][v]));
    }

    // ---- face traces: q at xi_k = 0 / 1 per tangential node and time node; every thread takes
    // the line of each axis that it contracts in the sweeps
    for (int v0 = 0; v0 < NV; v0 += VC) {
        int pt = la;
        __asm__ volatile("" : "+v"(pt));
        if (act) {
#pragma unroll
            for (int s = 0; s < n; s++)
                lds_put<L, VC>(Xc, pt + L::SS * s, [&](int vv) __attribute__((always_inline)) {
                    return v0 + vv < NV ? q[v0 + vv][s] : R(0);
                });
        }
        __syncthreads();
        if (act) {
#pragma unroll
            for (int k = 0; k < DIM; k++) {
                const int64_t cc = vb * CPB + lcell[k];
                const R *Xl = X + lcell[k] * L::CELL;
                R tr[2][VC];
#pragma unroll
                for (int vv = 0; vv < VC; vv++) tr[0][vv] = tr[1][vv] = 0;
#pragma unroll
                for (int b = 0; b < n; b++) {
                    if (b % 4 == 0) __asm__ volatile("" ::: "memory");
                    lds_get<L, VC>(Xl, lpt[k] + b * L::stride(k), [&](int vv, R x) __attribute__((always_inline)) {
                        tr[0][vv] += Bs[0][b] * x;
                        tr[1][vv] += Bs[1][b] * x;
                    });
                }
#pragma unroll
                for (int side = 0; side < 2; side++)
#pragma unroll
                    for (int vv = 0; vv < VC; vv++)
                        if (v0 + vv < NV && cc < ncell)
                            A.trace[((cc * 2 * DIM + 2 * k + side) * NV + v0 + vv) * (NFN * n) + lj[k]] = tr[side][vv];
            }
        }
        __syncthreads();
    }
    // ---- volume term: the contraction of the time-integrated fluxes (after the traces, when the
    // pencils' registers are free)
    if constexpr (VOL) {
        int pt = la;
        __asm__ volatile("" : "+v"(pt));
        R vol[NV];
#pragma unroll
        for (int v = 0; v < NV; v++) vol[v] = 0;
        // every thread contracts for its own node; a slice of X per axis and chunk of variables,
        // used again only after a barrier
        constexpr int NCH = (NV + VC - 1) / VC;
#pragma unroll
        for (int k = 0; k < DIM; k++) {
            const R ck = (R)(dt * A.dth[k]);
            const int ak = (k == 0 ? la : (k == 1 ? la / n : la / (n * n))) % n, l0 = pt - ak * L::stride(k);
#pragma unroll
            for (int ch = 0; ch < NCH; ch++) {
                const int i = k * NCH + ch, v0 = ch * VC, sl = L::SS * (i % n);
                if (act)
                    lds_put<L, VC>(Xc, pt + sl, [&](int vv) __attribute__((always_inline)) {
                        return v0 + vv < NV ? Fi[k][v0 + vv] : R(0);
                    });
                __syncthreads();
                R acc[VC];
#pragma unroll
                for (int vv = 0; vv < VC; vv++) acc[vv] = 0;
#pragma unroll
                for (int b = 0; b < n; b++) {
                    if (b % 4 == 0) __asm__ volatile("" ::: "memory");
                    const R d = Dvol[ak][b];
                    lds_get<L, VC>(Xc, l0 + sl + b * L::stride(k),
                                   [&](int vv, R x) __attribute__((always_inline)) { acc[vv] += d * x; });
                }
#pragma unroll
                for (int vv = 0; vv < VC; vv++)
                    if (v0 + vv < NV) {
                        vol[v0 + vv] += ck * acc[vv];
                        // summed here, not in the owner's branch below: the compiler sinks the sums there
                        // and keeps all their operands instead, 2 n of them per axis and chunk (24^3 cells
                        // of degree 9: FP64 99.4 -> 87.6 ms, FP32 21.5 -> 17.4, deviation form 38.8 -> 35.9;
                        // a cell in one chunk has few enough of them that the order makes no difference)
                        if constexpr (VC < NV) __asm__ volatile("" : "+v"(vol[v0 + vv]));
                    }
                if ((i + 1) % n == 0 || i + 1 == DIM * NCH) __syncthreads();
            }
        }
        if (owner) {
            // u^n is read again here rather than held in registers through the sweeps
#pragma unroll
            for (int v = 0; v < NV; v++)
                A.vol_out[(A.cell0 + c) * NN + (int64_t)v * A.in_vstride + a] =
                    A.in[c * A.in_cstride + v * A.in_vstride + a] + (double)vol[v];
        }
    }
    }  // persistent loop
}

template <int DIM, int N, bool VOL, typename R, bool DEV = false>
// the register budget held to Tune's waves per SIMD (FP32: four, FP64: two by default)
__global__ __launch_bounds__((PredShape<DIM, N, R>::BS), (Tune<DIM, N, sizeof(R) == 4>::pred_wps)) void k_predictor(PredArgs<R> A,
                                                                                                   double gamma_d) {
    pred_cells<DIM, N, VOL, R, DEV>(A, gamma_d, A.ncell, blockIdx.x, gridDim.x);
}

}  // namespace adg
