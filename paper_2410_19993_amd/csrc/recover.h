// Word-line recovery of the float64 sweeps: the tridiagonal blocks T_i solved for the
// 16 input vectors of a slab, and the row's node voltages written in the paper's order.
// Shared by the sweep that recovers a row while the next product runs (sweep.hip) and
// by the kernel that recovers all rows at once (sweep_rows.hip), so that both give the
// same bits.
#pragma once

#include "common.h"

namespace xbk {

// k position inside a CPR row (16-chunk permuted)
template <typename T>
__device__ __host__ inline int pos(int k) { return (k & ~15) + Frag<T>::slot(k & 15); }

// ---------------------------------------------------------------------------
// Tridiagonal solves T_i w = d split over LANES lanes per vector.
// Lane s owns the contiguous segment [s << lg, (s+1) << lg); element j lives at
// LDS index j + (j >> lg) (one pad slot per segment), so the lanes of a
// segmented pass fall on distinct banks.  Each pass is a scan of affine maps:
//   d'_0 = d_0, d'_j = d_j + fr_j d'_{j-1};  w_{n-1} = ip_{n-1} d'_{n-1},
//   w_j = ip_j (d'_j + g_wl w_{j+1}).
__host__ __device__ inline int seg_lg(int n, int lanes)
{
    int lg = 0;
    while ((lanes << lg) < n) ++lg;
    return lg;
}
__device__ __forceinline__ int padj(int j, int lg) { return j + (j >> lg); }
__host__ __device__ inline int padded_len(int n, int lanes) { return n + (n >> seg_lg(n, lanes)) + 1; }
// smallest power of two >= x
constexpr int seg_cap(int x) { return x <= 1 ? 1 : 2 * seg_cap((x + 1) / 2); }

__device__ __forceinline__ void affine_compose(double& P, double& Q, double Pp, double Qp)
{
    Q = P * Qp + Q;          // x -> P (Pp x + Qp) + Q
    P = P * Pp;
}

// Order this wave's LDS writes before later LDS reads of other lanes of the
// same wave (no workgroup barrier needed: the data is private to the wave).
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Word lines and node voltages of row i for the vectors of wave h (of kHelpers): 16 lanes
// per vector, each a contiguous segment of the row, from the row's bit lines in ybuf
// ([16][ldy], CPR) and the staged coefficients fr, ip, G in coef ([3][PL]).  vb: this
// lane's vector's input voltage.  Loops run to compile-time bounds with masked lanes.
constexpr int kHelpers = 4;      // waves of a row's recovery (the float64 sweep's helpers, one per SIMD)
template <typename T, int NT>
struct RowRecover {
    static constexpr int n_p = 64 * NT;
    static constexpr int ldy = n_p + 4;
    static constexpr int LR = 16;             // lanes per input vector
    static constexpr int VPW = 64 / LR;       // input vectors per wave
    static constexpr int KJ = (n_p + LR - 1) / LR;          // j's per lane in the first pass
    static constexpr int SEG = seg_cap(KJ);                  // longest lane segment
    static __device__ __forceinline__ void run(const SweepArgs& a, int slab, int i, double vb, const T* ybuf,
                                               double* wv, const double* coef, int h, int l, int lg, int PL)
    {
        const int n = a.n, v = l / LR, s = l % LR, cc = h * VPW + v;
        const int bb = 16 * slab + cc;
        const double* fr = coef;                              // padded like d
        const double* ip = fr + PL;
        const double* Gi = fr + 2 * PL;
        double* d = wv + cc * PL;
        const int spare = PL - 1;                              // never a padded index of j < n
#pragma unroll 8
        for (int k = 0; k < KJ; ++k) {
            const int j = s + LR * k;
            const bool ok = j < n;
            const int pj = padj(ok ? j : n - 1, lg);
            const double val = Gi[pj] * (double)ybuf[cc * ldy + pos<T>(ok ? j : n - 1)] +
                               (j == 0 ? a.g_src * vb : 0.0);
            d[ok ? pj : spare] = val;
        }
        wave_lds_fence();
        // T_i w = d by forward and backward affine scans over the LR lanes of a vector
        const int j0 = s << lg, len = max(0, min(n - j0, 1 << lg)), base = j0 + s;
        const double gw = a.g_wl;
        double P = 1.0, Q = 0.0;
#pragma unroll 8
        for (int e = 0; e < SEG; ++e) {
            const bool ok = e < len;
            const int p = ok ? base + e : spare;
            const double f = ok ? fr[p] : 0.0;               // fr at j = 0 is zero
            const double Qn = d[p] + f * Q, Pn = f * P;
            Q = ok ? Qn : Q;
            P = ok ? Pn : P;
        }
        for (int off = 1; off < LR; off <<= 1) {
            const double Pp = __shfl_up(P, off, LR), Qp = __shfl_up(Q, off, LR);
            if (s >= off) affine_compose(P, Q, Pp, Qp);
        }
        double x = __shfl_up(Q, 1, LR);
        if (s == 0) x = 0.0;
#pragma unroll 8
        for (int e = 0; e < SEG; ++e) {
            const bool ok = e < len;
            const int p = ok ? base + e : spare;
            const double f = ok ? fr[p] : 0.0;
            const double xn = d[p] + f * x;
            x = ok ? xn : x;
            d[p] = x;
        }
        P = 1.0;
        Q = 0.0;
#pragma unroll 8
        for (int e = SEG - 1; e >= 0; --e) {
            const bool ok = e < len;
            const int p = ok ? base + e : spare;
            const double ipj = ok ? ip[p] : 0.0;
            const double f = (j0 + e >= n - 1) ? 0.0 : ipj * gw;
            const double Qn = ipj * d[p] + f * Q, Pn = f * P;
            Q = ok ? Qn : Q;
            P = ok ? Pn : P;
        }
        for (int off = 1; off < LR; off <<= 1) {
            const double Pp = __shfl_down(P, off, LR), Qp = __shfl_down(Q, off, LR);
            if (s + off < LR) affine_compose(P, Q, Pp, Qp);
        }
        x = __shfl_down(Q, 1, LR);
        if (s == LR - 1) x = 0.0;
#pragma unroll 8
        for (int e = SEG - 1; e >= 0; --e) {
            const bool ok = e < len;
            const int p = ok ? base + e : spare;
            const double ipj = ok ? ip[p] : 0.0;
            const double f = (j0 + e >= n - 1) ? 0.0 : ipj * gw;
            const double xn = ipj * d[p] + f * x;
            x = ok ? xn : x;
            d[p] = x;
        }
        wave_lds_fence();
        // node voltages (w_j, u_j) of the wave's vectors, 1 KB per store instruction
        typedef double d2v __attribute__((ext_vector_type(2)));
        for (int vv = 0; vv < VPW; ++vv) {
            const int c2 = h * VPW + vv, b2 = 16 * slab + c2;
            if (b2 >= a.B) break;
            double* out = a.node_v + ((int64_t)b2 * a.m + i) * 2 * n;
#pragma unroll 4
            for (int k = 0; k < NT; ++k) {
                const int j = 64 * k + l;
                if (j < n)
                    __builtin_nontemporal_store(d2v{wv[c2 * PL + padj(j, lg)], (double)ybuf[c2 * ldy + pos<T>(j)]},
                                                reinterpret_cast<d2v*>(out + 2 * j));
            }
        }
    }
};

}  // namespace xbk
