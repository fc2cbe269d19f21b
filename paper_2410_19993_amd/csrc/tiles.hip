// Batched small crossbars: the output currents of many crossbars of one shape
// (n <= 64 columns), one workgroup per crossbar, the whole solve in one launch.
//
// Per crossbar the method is the one of the large path (Sec. II.A-II.C):
// eliminate each row's word-line nodes (E_i = Q_i - Gam_i T_i^-1 Gam_i, source
// coupling c_i = g_src Gam_i T_i^-1 e_0), then a block LU over the rows.  Here
// the rows are taken top-down in one chain, S_i = E_i - g_bl^2 H_{i-1},
// H_i = S_i^-1, with the forward substitution z_i = H_i (V_i c_i + g_bl z_{i-1})
// run alongside.  The bottom row's forward result is already its solution (the
// back substitution leaves the last row unchanged), so the output currents
// g_sense z_{m-1} need no back substitution and no row block is stored.
//
// Workgroup layout (eight waves, four for NP = 16; blocks padded with identity to NP
// in {16, 32, 64}):
//  * the word-line chains of 32 rows are walked together, a lane per row (the rows'
//    chains are independent; one row at a time left a lone lane walking a 64-step chain
//    of reciprocals per row), and T_i^-1 is filled from them as products of ratios, a
//    wave per eight rows (a thread walking a whole column took 10000 cycles a row);
//  * S_i^-1 is found by third-order Newton-Schulz rounds on the float64 matrix cores from
//    the row before's inverse (X_0 below), each wave owning one or two 16 x 16 tiles:
//        Q = I - X_0 S,  Y = Q X_0,  X = X_0 + Y + Q Y,  I - X S = Q^3.
//    X_0 is H_{i-1} corrected to first order in S_i - S_{i-1} with the diagonal of S_{i-1}
//    for its inverse, and on the diagonal by the change of 1 / S_jj.  A round is the last
//    once every |Q| entry is <= 2.5e-7 (||I - X S|| <= 4.1e-15): one round a row for
//    devices of 1 to 100 uS on 1.5 ohm wires, two for devices of 2 mS and in the last
//    row.  The first row, and a row whose rounds miss the tolerance, is eliminated, and so
//    is every row from conductances so large that rounding may cost S_i its definiteness
//    (round_limit): the rounds find the inverse of an indefinite block as readily as any,
//    while an elimination meets its pivots;
//  * the product H_i Y runs on the matrix cores too: a wave owns every eighth (fourth)
//    group of 16 input vectors, and keeps their forward results in the accumulator
//    layout (item v of lane l = 16 q + c is row q + 4v of a 16-row tile, vector c of a
//    group).  That is also the B-operand layout of the next row's product, so the
//    forward results never move.  The A operand, H_i, is read from LDS along rows (H_i
//    is symmetric).
// Two LDS blocks alternate: T_i^-1, S_i, Q, then H_i, in one, while H_{i-1}, X_0, then Y
// sit in the other.  A tile with a conductance that is not finite and positive, or an
// eliminated pivot that is not positive, gets NaN currents.  float64 throughout.
//
// Bound: the chain of rows; at NP = 64 and 256 vectors a row is 12 us of matrix
// instructions on one CU (7 of them the forward products).  Measured with 256 vectors, 32
// crossbars of 128 x 64: 2.60 ms (20 us a row; every row eliminated: 5.44); 1000 of 64 x 64:
// 5.5 ms (10.8); 48 of 32 x 32: 0.23 ms (0.54); 400 of 16 x 16: 0.116 ms (0.17).  A crossbar
// of a single row has nothing to gain: 1 x 64 57 us, 50 by the eliminating kernel.
#include <climits>
#include <cmath>
#include <cstdint>

#include "common.h"
#include "tiles.h"

namespace {

using xbk::lds_barrier;

constexpr int kMaxVectors = 256;

typedef double dv4 __attribute__((ext_vector_type(4)));

// 1 / x for the positive normal pivots here: the hardware reciprocal estimate
// refined by two Newton-Raphson steps r <- r + r (1 - x r), each of which squares
// the relative error (full double precision after the second)
__device__ inline double recip(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}

// A crossbar's B input vectors may be split over gridDim.y workgroups (Bp each, the
// last one fewer): each redoes the crossbar's factorization and forward-substitutes its
// own vectors, trading repeated elimination for more workgroups in flight.
struct TileArgs {
    int m, n, B, Bp;
    int unit;           // 1: input vector b is the unit vector e_b (V is not read)
    double g_wl, g_bl, g_src, g_sense;
    double g_rounds;    // rows are inverted by rounds up to this conductance (round_limit)
    const double* G;    // [T][m][n]
    const double* V;    // [T][B][m]
    double* I;          // [T][B][n]
};

constexpr double kBlockNsDone = 2.5e-7;  // largest |Q| entry of a row's last round
constexpr int kBlockRounds = 3;          // rounds before a row is eliminated: ||Q|| <= 1/4 cubes to 4e-6 in two

// Largest conductance for which S_i, as computed, is strictly diagonally dominant with a
// positive diagonal, so that its pivots are positive; rows past it are eliminated, which
// checks them.  Without rounding S_i 1 >= below, the conductance under the row: the word
// line's term G - G T^-1 G 1 is not negative, and g_bl H_{i-1} 1 <= 1.  Rounding changes
// the row sums by at most 2e-12 G (products of up to 64 ratios, 3e-14 each) and
// 1e-14 (2 G + 4 g_bl) (H_{i-1}, whose condition is at most (2 G + 4 g_bl) / g_bl): a tenth
// of `below` where G + g_bl <= 1e10 below.  The elimination also takes pivots past 1e300
// for bad.
double round_limit(double g_bl, double g_sense)
{
    if (!(g_bl <= 1e299 && g_sense <= 1e299)) return -1.0;
    return std::fmin(1e10 * std::fmin(g_bl, g_sense) - g_bl, 1e299);
}

__device__ __forceinline__ double nanmax(double a, double b)
{
    return (a > b || a != a) ? a : b;    // a NaN is kept
}

// Waves of a workgroup: with eight, two a SIMD, one's products hide the other's loads
// (128 x 64 with 256 vectors: 3.4 ms with four, 2.9 with eight); a block of 16 is a
// single tile and has nothing for more than four.
template <int NP> constexpr int tile_waves = NP == 16 ? 4 : 8;

typedef __attribute__((address_space(3))) double lds_double;

// Inverse of the n x n block in T (LDS, padded with the identity to NP) over itself, by
// Gauss-Jordan elimination without pivoting on the threads' register blocks, four
// pivots K = {k .. k+3} per step: the 4 x 4 pivot block P = S[K][K] is inverted in
// registers by every thread, and
//   S[K][c] <- P^-1 S'[K][c],  S[r][c] <- S'[r][c] - S[r][K] P^-1 S'[K][c]  (r not in K)
// where S' is S with S[.][K] replaced by the identity columns.  The padding is the
// identity, so blocks that reach past n stay exact.  work: 16 NP doubles of LDS.  False
// if a pivot is not positive and finite.  A function of its own: inlined, its registers
// made the rounds of every row spill.
template <int NP>
__device__ __attribute__((noinline)) bool eliminate(lds_double* T, lds_double* work, int n)
{
    constexpr int LD = NP + 2, CB = 64 * tile_waves<NP> / 16, BR = NP / 16, BC = NP / CB;
    const int tid = threadIdx.x, br = tid / CB, bc = tid % CB;
    bool good = true;
    lds_double (*rowb)[4][NP] = reinterpret_cast<lds_double (*)[4][NP]>(work);            // [buffer][pivot][index]
    lds_double (*colb)[4][NP] = reinterpret_cast<lds_double (*)[4][NP]>(work + 8 * NP);
    double s[BR][BC];
#pragma unroll
    for (int ii = 0; ii < BR; ++ii)
#pragma unroll
        for (int jj = 0; jj < BC; ++jj) s[ii][jj] = T[(BR * br + ii) * LD + BC * bc + jj];
    for (int k = 0, step = 0; k < n; k += 4, ++step) {
        const int kb = step & 1;
#pragma unroll
        for (int ii = 0; ii < BR; ++ii) {
            const int r = BR * br + ii;
            if (r >= k && r < k + 4) {
#pragma unroll
                for (int jj = 0; jj < BC; ++jj) rowb[kb][r - k][BC * bc + jj] = s[ii][jj];
            }
        }
#pragma unroll
        for (int jj = 0; jj < BC; ++jj) {
            const int c = BC * bc + jj;
            if (c >= k && c < k + 4) {
#pragma unroll
                for (int ii = 0; ii < BR; ++ii) colb[kb][c - k][BR * br + ii] = s[ii][jj];
            }
        }
        lds_barrier();
        double P[4][4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) P[u][v] = rowb[kb][u][k + v];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const double pv = P[t][t];
            good &= pv > 0.0 && pv <= 1e300;
            const double rp = recip(pv);
            double row[4], col[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                row[v] = (v == t ? 1.0 : P[t][v]) * rp;
                col[v] = P[v][t];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) P[u][v] = (u == t) ? row[v] : ((v == t ? 0.0 : P[u][v]) - col[u] * row[v]);
        }
        double f[4][BR], nn[4][BC], keep[BC];
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int ii = 0; ii < BR; ++ii) f[t][ii] = colb[kb][t][BR * br + ii];
#pragma unroll
        for (int jj = 0; jj < BC; ++jj) {
            const int c = BC * bc + jj, ck = c - k;
            const bool inK = ck >= 0 && ck < 4;
            double u[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) u[t] = inK ? (ck == t ? 1.0 : 0.0) : rowb[kb][t][c];
#pragma unroll
            for (int t = 0; t < 4; ++t) nn[t][jj] = P[t][0] * u[0] + P[t][1] * u[1] + P[t][2] * u[2] + P[t][3] * u[3];
            keep[jj] = inK ? 0.0 : 1.0;
        }
#pragma unroll
        for (int ii = 0; ii < BR; ++ii) {
            const int rk = BR * br + ii - k;
            const bool inK = rk >= 0 && rk < 4;
#pragma unroll
            for (int jj = 0; jj < BC; ++jj) {
                double own = nn[0][jj];
#pragma unroll
                for (int t = 1; t < 4; ++t) own = (rk == t) ? nn[t][jj] : own;
                const double upd = s[ii][jj] * keep[jj] - f[0][ii] * nn[0][jj] - f[1][ii] * nn[1][jj] -
                                   f[2][ii] * nn[2][jj] - f[3][ii] * nn[3][jj];
                s[ii][jj] = inK ? own : upd;
            }
        }
    }
    lds_barrier();
#pragma unroll
    for (int ii = 0; ii < BR; ++ii)
#pragma unroll
        for (int jj = 0; jj < BC; ++jj) T[(BR * br + ii) * LD + BC * bc + jj] = s[ii][jj];
    return good;
}

constexpr int kChainRows = 32;           // rows whose word-line chains are walked together

// Per row: conductances, r_j, the diagonal of T^-1, and by segments of eight columns the
// products of the r before a column of the segment and of all of them.
template <int NP>
struct Chains {
    double g[kChainRows][NP + 1], r[kChainRows][NP + 1], d[kChainRows][NP + 1];
    double pre[kChainRows][NP], seg[kChainRows][NP / 8];
};
template <int NP> using lds_chains = __attribute__((address_space(3))) Chains<NP>;
typedef __attribute__((address_space(3))) int lds_int;

// The word-line chains of `rows` rows, a lane per row (excess form, no subtraction):
//   e_0 = G_0 + g_src, e_j = G_j + g_wl e_{j-1} / p_{j-1}, p_j = e_j + g_wl [j < n-1];
// then r_j = g_wl / p_j and, from the far end, the diagonal of T^-1:
//   d_k = (1 + g_wl r_k d_{k+1}) / p_k.
// Eight columns of a row pass through registers at a time: column by column, a lane waits
// for what it has just stored (5000 crossbars of 8 x 8 318 us, 310 so).  *beyond becomes
// infinite at a conductance past g_rounds.  A function of its own, like eliminate: inlined,
// 1024 crossbars of 64 x 64 with 256 vectors took 5.82 ms, 5.54 so.  Ends with a barrier.
template <int NP>
__device__ __attribute__((noinline)) void walk_chains(lds_chains<NP>* c, lds_int* bad, lds_double* beyond,
                                                      const double* __restrict__ G, int rows, int n, double gw,
                                                      double g_src, double g_rounds)
{
    const int tid = threadIdx.x;
    for (int e = tid; e < rows * n; e += 64 * tile_waves<NP>) {
        const double g = G[e];
        c->g[e / n][e % n] = g;
        if (!(g > 0.0 && g <= 1e300)) *bad = 1;
        if (!(g <= g_rounds)) *beyond = HUGE_VAL;
    }
    lds_barrier();
    if (tid < rows) {
        lds_double *gr = c->g[tid], *rp = c->r[tid], *d = c->d[tid];
        double e = gr[0] + g_src;
        double rc = recip(e + (n > 1 ? gw : 0.0));
        d[0] = rc;
        for (int j0 = 0; j0 < n; j0 += 8) {
            double g[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) g[u] = gr[j0 + u];        // columns past n: unused
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int j = j0 + u;
                if (j == 0 || j >= n) continue;
                e = g[u] + gw * e * rc;
                rc = recip(e + (j < n - 1 ? gw : 0.0));
                d[j] = rc;
            }
        }
        double x = rc;
        for (int k0 = (n - 1) & ~7; k0 >= 0; k0 -= 8) {
            double p[8], r[8], f = 1.0;
#pragma unroll
            for (int u = 0; u < 8; ++u) p[u] = d[k0 + u];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                r[u] = gw * p[u];
                if (k0 + u < n) c->pre[tid][k0 + u] = f;
                f *= r[u];
            }
            if (k0 + 7 < n - 1) c->seg[tid][k0 >> 3] = f;
#pragma unroll
            for (int u = 7; u >= 0; --u) {
                const int k = k0 + u;
                if (k >= n - 1) continue;
                rp[k] = r[u];
                x = p[u] * fma(gw * r[u], x, 1.0);
                d[k] = x;
            }
        }
    }
    lds_barrier();
}

template <int NP>
__global__ __launch_bounds__(64 * tile_waves<NP>) void tile_currents_kernel(TileArgs a)
{
    constexpr int LD = NP + 2;                         // row stride of the LDS blocks
    constexpr int W = tile_waves<NP>;
    constexpr int NT = NP / 16;                        // 16-row tiles of the product
    constexpr int NG = 16 / W;                         // groups of 16 vectors of a wave
    constexpr int CT = NP == 64 ? 2 : 1;               // tiles of a round that a wave owns
    constexpr int R = kChainRows;
    __shared__ __align__(16) double blk[2][NP * LD];
    __shared__ __align__(16) Chains<NP> chains;
    __shared__ double cr[NP], rdiag[2][NP], wmx[W];
    __shared__ double beyond;                          // 0, or infinite from a conductance past g_rounds on
    __shared__ int bad;

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int q = lane >> 4, l16 = lane & 15;
    const int m = a.m, n = a.n;
    const int64_t t = blockIdx.x;
    const int b0 = (int)blockIdx.y * a.Bp;                 // first vector of this workgroup
    const int B = min(a.Bp, a.B - b0);                      // vectors of this workgroup
    const double* G = a.G + t * m * n;
    const double* V = a.V + (t * a.B + b0) * m;
    double* I = a.I + (t * a.B + b0) * n;
    const double gw = a.g_wl, gb = a.g_bl;
    if (tid == 0) {
        bad = 0;
        beyond = 0.0;
    }
    lds_barrier();
    // the wave's tiles of S_i and H_i: row tile wr, column tiles wc .. wc + CT - 1
    const int wr = NP == 64 ? w >> 1 : NP == 32 ? (w & 3) >> 1 : 0, wc = NP > 16 ? CT * (w & 1) : 0;
    const bool owner = w < NT * NT / CT;
    auto row_of = [&](int v) { return 16 * wr + q + 4 * v; };
    auto col_of = [&](int C) { return 16 * (wc + C) + l16; };
    // acc += (rows 16 wr .. of A) * B, both blocks in LDS
    auto product = [&](dv4 (&acc)[CT], const double* A, const double* Bm) {
        if (!owner) return;
        constexpr int D = 4;                           // steps requested ahead
        const double* ap = A + (16 * wr + l16) * LD + q;
        const double* bp = Bm + q * LD + 16 * wc + l16;
        double x[D], y[D][CT];
#pragma unroll
        for (int k = 0; k < D; ++k) {
            x[k] = ap[4 * k];
#pragma unroll
            for (int C = 0; C < CT; ++C) y[k][C] = bp[4 * k * LD + 16 * C];
        }
#pragma unroll
        for (int k = 0; k < NP / 4; ++k) {
            const double xk = x[k % D];
            double yk[CT];
#pragma unroll
            for (int C = 0; C < CT; ++C) yk[C] = y[k % D][C];
            if (k + D < NP / 4) {
                x[k % D] = ap[4 * (k + D)];
#pragma unroll
                for (int C = 0; C < CT; ++C) y[k % D][C] = bp[4 * (k + D) * LD + 16 * C];
            }
#pragma unroll
            for (int C = 0; C < CT; ++C) acc[C] = __builtin_amdgcn_mfma_f64_16x16x4f64(xk, yk[C], acc[C], 0, 0, 0);
        }
    };
    auto put = [&](double* M, const dv4 (&x)[CT]) {
        if (!owner) return;
#pragma unroll
        for (int C = 0; C < CT; ++C)
#pragma unroll
            for (int v = 0; v < 4; ++v) M[row_of(v) * LD + col_of(C)] = x[C][v];
    };

    // forward results of vectors 16 (NG w + g) + l16: z[tile][g] item v = row 16 tile + q + 4 v
    dv4 z[NT][NG];
#pragma unroll
    for (int tt = 0; tt < NT; ++tt)
#pragma unroll
        for (int g = 0; g < NG; ++g) z[tt][g] = dv4{0.0, 0.0, 0.0, 0.0};
    dv4 prev[CT];                                      // the row's S, then the row before's
#pragma unroll
    for (int C = 0; C < CT; ++C) prev[C] = dv4{0.0, 0.0, 0.0, 0.0};

    for (int i = 0; i < m; ++i) {
        double* Tb = blk[i & 1];                       // T_i^-1, then S_i, Q, H_i
        double* Hp = blk[(i & 1) ^ 1];                 // H_{i-1}, then X_0, Y
        const int ir = i % R;
        // this row's inputs, used after the inverse
        double vi[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const int b = 16 * (W * g + w) + l16;
            vi[g] = (b < B) ? (a.unit ? (b0 + b == i ? 1.0 : 0.0) : V[(int64_t)b * m + i]) : 0.0;
        }
        if (ir == 0)
            walk_chains<NP>((lds_chains<NP>*)&chains, (lds_int*)&bad, (lds_double*)&beyond, G + (int64_t)i * n,
                            min(R, m - i), n, gw, a.g_src, a.g_rounds);
        const double* gr = chains.g[ir];
        // ---- T_i^-1[j][k] = r_j ... r_{k-1} d_k = T_i^-1[k][j], j <= k: wave w stores the rows of
        // segment w, lane k those of column k
        if (w < NP / 8 && lane < n && 8 * w <= lane) {
            const double* rp = chains.r[ir];
            const int k = lane, sk = k >> 3;
            double x = chains.d[ir][k] * (w < sk ? chains.pre[ir][k] : 1.0), f[8], y[NP / 8];
#pragma unroll
            for (int u = 0; u < 8; ++u) f[u] = rp[8 * w + u];
#pragma unroll
            for (int u = 1; u < NP / 8; ++u) y[u] = chains.seg[ir][u];
#pragma unroll
            for (int u = 1; u < NP / 8; ++u) x *= u > w && u < sk ? y[u] : 1.0;
#pragma unroll
            for (int u = 7; u >= 0; --u) {
                const int j = 8 * w + u;
                x *= j < k ? f[u] : 1.0;
                if (j <= k) Tb[j * LD + k] = Tb[k * LD + j] = x;
            }
        }
        lds_barrier();
        // ---- S_i = diag(q_i) - Gam T^-1 Gam - g_bl^2 H_{i-1} (identity on the padding) and,
        // from the row before, X_0; c_i = g_src Gam T^-1 e_0 (zero on the padding).  Every
        // load is issued before the first use; what lies outside the block, or before the
        // first row, is selected away.
        dv4 p[CT], x[CT];
        {
            const double below = (i < m - 1) ? gb : a.g_sense;
            const double above = (i > 0) ? gb : 0.0;
            const double g2 = gb * gb;
            const double* rd = rdiag[(i & 1) ^ 1];
            double grr[4], rdr[4], grc[CT], rdc[CT], tv[CT][4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                grr[v] = gr[row_of(v)];
                rdr[v] = rd[row_of(v)];
            }
#pragma unroll
            for (int C = 0; C < CT; ++C) {
                grc[C] = gr[col_of(C)];
                rdc[C] = rd[col_of(C)];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int r = row_of(v), c = col_of(C);
                    tv[C][v] = Tb[r * LD + c];
                    x[C][v] = Hp[r * LD + c];
                }
            }
            double pd = 1.0;                           // this lane's diagonal element, if it has one
#pragma unroll
            for (int C = 0; C < CT; ++C)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int r = row_of(v), c = col_of(C);
                    double s = -grr[v] * tv[C][v] * grc[C];
                    s = r == c ? s + (grr[v] + above + below) : s;
                    s = i > 0 ? s - g2 * x[C][v] : s;
                    s = r < n && c < n ? s : r == c ? 1.0 : 0.0;
                    pd = r == c ? s : pd;
                    p[C][v] = s;
                }
            const double rnew = recip(pd);
#pragma unroll
            for (int C = 0; C < CT; ++C)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int r = row_of(v), c = col_of(C);
                    if (r == c && owner) rdiag[i & 1][r] = rnew;
                    x[C][v] += r == c ? rnew - rdr[v] : -(p[C][v] - prev[C][v]) * (rdr[v] * rdc[C]);
                }
            if (tid < NP) cr[tid] = (tid < n) ? a.g_src * gr[tid] * Tb[tid] : 0.0;
        }
        lds_barrier();                                 // T^-1 and H_{i-1} read
        put(Tb, p);
        bool found = false;
        if (i > 0) {
            // ---- H_i by third-order Newton-Schulz rounds from X_0
            put(Hp, x);
            for (int round = 0; round < kBlockRounds; ++round) {
                lds_barrier();
                const double past = beyond;            // infinite: no round is the last
                dv4 qv[CT], y[CT];
#pragma unroll
                for (int C = 0; C < CT; ++C) qv[C] = y[C] = dv4{0.0, 0.0, 0.0, 0.0};
                product(qv, Hp, Tb);                   // X_0 S
                double mx = past;
#pragma unroll
                for (int C = 0; C < CT; ++C)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        qv[C][v] = (row_of(v) == col_of(C) ? 1.0 : 0.0) - qv[C][v];
                        mx = nanmax(fabs(qv[C][v]), mx);
                    }
                for (int off = 32; off > 0; off >>= 1) mx = nanmax(mx, __shfl_xor(mx, off));
                if (lane == 0) wmx[w] = owner ? mx : 0.0;
                lds_barrier();                         // X_0 and S read; wmx written
                double nu = wmx[0];
#pragma unroll
                for (int k = 1; k < W; ++k) nu = nanmax(nu, wmx[k]);
                found = nu <= kBlockNsDone;            // the same answer in every wave
                if (!found && (round == kBlockRounds - 1 || !(nu * NP <= 0.25))) break;
                put(Tb, qv);
                lds_barrier();
                product(y, Tb, Hp);                    // Y = Q X_0
                lds_barrier();
                put(Hp, y);
#pragma unroll
                for (int C = 0; C < CT; ++C) x[C] += y[C];
                lds_barrier();
                product(x, Tb, Hp);                    // X = X_0 + Y + Q Y
                lds_barrier();
                if (found) {
                    put(Tb, x);
                    break;
                }
                put(Tb, p);
                put(Hp, x);
            }
        }
        lds_barrier();
        if (!found) {
            if (!eliminate<NP>((lds_double*)Tb, (lds_double*)Hp, n)) bad = 1;
            lds_barrier();
        }
#pragma unroll
        for (int C = 0; C < CT; ++C) prev[C] = p[C];
        // ---- z <- H_i (V_i c_i + g_bl z) on the matrix cores, a group of 16 vectors at a time
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            if (16 * (W * g + w) >= B) break;
            dv4 y[NT];
#pragma unroll
            for (int kc = 0; kc < NT; ++kc)
#pragma unroll
                for (int tq = 0; tq < 4; ++tq) y[kc][tq] = vi[g] * cr[16 * kc + q + 4 * tq] + gb * z[kc][g][tq];
#pragma unroll
            for (int tt = 0; tt < NT; ++tt) z[tt][g] = dv4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int kc = 0; kc < NT; ++kc) {
#pragma unroll
                for (int tq = 0; tq < 4; ++tq)
#pragma unroll
                    for (int tt = 0; tt < NT; ++tt) {
                        // A operand H[16 tt + l16][16 kc + q + 4 tq], read as its mirror H[k][a]
                        const double h = Tb[(16 * kc + q + 4 * tq) * LD + 16 * tt + l16];
                        z[tt][g] = __builtin_amdgcn_mfma_f64_16x16x4f64(h, y[kc][tq], z[tt][g], 0, 0, 0);
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // No barrier: the next row first writes the block that this product does not read,
        // and cr after a barrier.
    }
    lds_barrier();
    const bool fail = bad != 0;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const int b = 16 * (W * g + w) + l16;
        if (b >= B) continue;
#pragma unroll
        for (int tt = 0; tt < NT; ++tt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int j = 16 * tt + q + 4 * v;
                if (j < n) I[(int64_t)b * n + j] = fail ? NAN : a.g_sense * z[tt][g][v];
            }
    }
}

}  // namespace

hipError_t xbk_launch_tile_currents(int T, int m, int n, int B, double g_wl, double g_bl, double g_src,
                                    double g_sense, const double* G, const double* V, double* I, hipStream_t s,
                                    int block, int split, bool unit)
{
    if (T < 1 || m < 1 || n < 1 || n > 64 || B < 1 || B > kMaxVectors || !G || (!V && !unit) || !I)
        return hipErrorInvalidValue;
    if (block == 0) block = n <= 16 ? 16 : n <= 32 ? 32 : 64;
    if ((block != 16 && block != 32 && block != 64) || block < n || split < 1 || split > 4) return hipErrorInvalidValue;
    const int Bp = (B + split - 1) / split;
    const int parts = (B + Bp - 1) / Bp;
    TileArgs a{m, n, B, Bp, unit ? 1 : 0, g_wl, g_bl, g_src, g_sense, round_limit(g_bl, g_sense), G, V, I};
    const dim3 grid((unsigned)T, (unsigned)parts);
    if (block == 16)
        hipLaunchKernelGGL(tile_currents_kernel<16>, grid, dim3(64 * tile_waves<16>), 0, s, a);
    else if (block == 32)
        hipLaunchKernelGGL(tile_currents_kernel<32>, grid, dim3(64 * tile_waves<32>), 0, s, a);
    else
        hipLaunchKernelGGL(tile_currents_kernel<64>, grid, dim3(64 * tile_waves<64>), 0, s, a);
    return hipGetLastError();
}
