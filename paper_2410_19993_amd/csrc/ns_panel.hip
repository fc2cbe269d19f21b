// Newton-Schulz factor at n_p = 128 (65 to 128 columns): one launch per row of each chain.
//
// The method, its starting iterates, rounds and tolerances are those of the slot
// schedule (ns.hip), but a round is formed column panel by column panel,
//     U = I - P X,   X'' = X (I + U + U^2),
// so that a workgroup owning the columns C of the row's inverse needs no other workgroup:
//     u = I_C - P X_C,   u2 = u - P (X u),   X''_C = X_C + X u + X u2,
// four products of the whole P or X with a 16-column panel.  (U is the transpose of the
// slot schedule's Q; float32 rows take the single step X' = X_C + X u.)  Eight workgroups
// of eight waves per chain; a wave keeps its 16-row tiles of P and X in registers, and the
// panel passes through LDS.  Each tile of the result is stored transposed, where it is
// contiguous in the fragment-tiled layout: the iterates are symmetric up to rounding.
//
// Whether a round met the tolerance is known only when all its workgroups have ended.  A
// launch therefore forms the next row's pivot block and first iterate in any case, into
// the other of two buffers, and the following launch looks at the round's flags: it goes
// on to the next row, or repeats the row from the iterate just found.
//
// Bound: the chain of launches, four products of 8 x 32 matrix instructions each (6.8 us
// in float64 on one CU's matrix cores) behind a launch's start and operand loads.  The
// slot schedule takes three launches of a quarter of that work.  Measured at 128 x 128:
// 11.5 us a row of both chains in float64 (20.0 before), 6 us in float32 (12.0).
#include "common.h"

namespace xbk {

namespace {

constexpr int kP = 128, kPT = kP / 16;                 // block edge, tiles a side

template <typename T> struct P4;
template <> struct P4<double> { using type = d4_t; };
template <> struct P4<float> { using type = f4_t; };

template <typename T>
__device__ __forceinline__ typename P4<T>::type tile_load(const T* __restrict__ t, int l)
{
    if constexpr (sizeof(T) == 8) {
        typedef double d2v __attribute__((ext_vector_type(2)));
        const d2v lo = *reinterpret_cast<const d2v*>(t + 2 * l);
        const d2v hi = *reinterpret_cast<const d2v*>(t + 128 + 2 * l);
        return d4_t{lo[0], lo[1], hi[0], hi[1]};
    } else {
        return *reinterpret_cast<const f4_t*>(t + 4 * l);
    }
}
template <typename T>
__device__ __forceinline__ void tile_store(T* t, int l, typename P4<T>::type v)
{
    if constexpr (sizeof(T) == 8) {
        typedef double d2v __attribute__((ext_vector_type(2)));
        *reinterpret_cast<d2v*>(t + 2 * l) = d2v{v[0], v[1]};
        *reinterpret_cast<d2v*>(t + 128 + 2 * l) = d2v{v[2], v[3]};
    } else {
        *reinterpret_cast<f4_t*>(t + 4 * l) = v;
    }
}
template <typename T>
__device__ __forceinline__ typename P4<T>::type panel_get(const T* p)
{
    if constexpr (sizeof(T) == 8) {
        typedef double d2v __attribute__((ext_vector_type(2)));
        const d2v lo = *reinterpret_cast<const d2v*>(p), hi = *reinterpret_cast<const d2v*>(p + 2);
        return d4_t{lo[0], lo[1], hi[0], hi[1]};
    } else {
        return *reinterpret_cast<const f4_t*>(p);
    }
}
template <typename T>
__device__ __forceinline__ void panel_put(T* p, typename P4<T>::type v)
{
    if constexpr (sizeof(T) == 8) {
        typedef double d2v __attribute__((ext_vector_type(2)));
        *reinterpret_cast<d2v*>(p) = d2v{v[0], v[1]};
        *reinterpret_cast<d2v*>(p + 2) = d2v{v[2], v[3]};
    } else {
        *reinterpret_cast<f4_t*>(p) = v;
    }
}

// Rows of a schedule: chain 0 the top chain (0 .. kt-1), 1 the bottom chain (m-1 .. kt+1),
// 2 the twist row (with chain 0's buffers, once both chains have finished).
struct Chain {
    int start, dir, rows;
    __device__ Chain(int m, int chain)
        : start(chain == 0 ? 0 : chain == 1 ? m - 1 : m / 2), dir(chain == 1 ? -1 : 1),
          rows(chain == 0 ? m / 2 : chain == 1 ? m - 1 - m / 2 : 1) {}
    __device__ int index(int row) const { return (row - start) * dir; }
};

}  // namespace

// What a launch did (NSState of its parity): kNsForm formed `row`'s pivot block and cold
// start into buffers xb; kNsResid ran the round `it` of `row` from buffers xb.
template <typename T>
__global__ __launch_bounds__(64 * kPT) void ns_panel_kernel(NSPanelArgs pa, int chain0, int slot)
{
    using v4 = typename P4<T>::type;
    using acc_t = typename Frag<T>::acc_t;
    constexpr bool rounds = sizeof(T) == 8;
    constexpr double done = rounds ? 6.4e-5 / kP : 1e-4;
    constexpr int ldy = kP + 4, steps = rounds ? 2 : 1;
    __shared__ __align__(16) T pan[2][16 * ldy];
    __shared__ int pass[kPT];
    const NSArgs& a = pa.a;
    const int chain = chain0 < 0 ? (int)blockIdx.y : chain0, C = blockIdx.x;
    const int l = threadIdx.x & 63, q = l >> 4, c = l & 15;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n = a.n;
    const Chain ch(a.m, chain);
    const int bc = chain == 1 ? 1 : 0;
    const int64_t blk = (int64_t)kP * kP, own = ((int64_t)C * kPT + w) * 256;   // tile (C, w)
    T* const H = reinterpret_cast<T*>(a.H);
    const NSState prev = a.state[3 * (slot & 1) + chain];
    NSState* const nxt = a.state + 3 * ((slot + 1) & 1) + chain;
    double* const flag_in = a.part + ((slot & 1) * 2 + bc) * kPT;
    double* const flag_out = a.part + (((slot + 1) & 1) * 2 + bc) * kPT;
    const bool first_thread = C == 0 && threadIdx.x == 0;
    if (prev.phase == kNsFinished) {
        if (first_thread) *nxt = prev;
        return;
    }
    // this lane's elements of its tile: rows 16 w + drow(q, v), column 16 C + c
    const int col = 16 * C + c;
    auto rowi = [&](int v) { return 16 * w + Frag<T>::drow(q, v); };
    if (slot == 0) {
        // form: P = E_row - g^2 (H_a + H_b), X_0 = diag(P)^-1, identity on the padding
        const int row = ch.start, kt = a.m / 2;
        v4 s = tile_load<T>(H + row * blk + own, l), x;
        if (chain == 2) {
            const v4 none{0, 0, 0, 0};
            const v4 ha = kt > 0 ? tile_load<T>(H + (kt - 1) * blk + own, l) : none;
            const v4 hb = kt + 1 < a.m ? tile_load<T>(H + (kt + 1) * blk + own, l) : none;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (kt > 0) s[v] -= (T)a.g2 * ha[v];
                if (kt + 1 < a.m) s[v] -= (T)a.g2 * hb[v];
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const bool diag = rowi(v) == col;
            if (rowi(v) >= n || col >= n) s[v] = diag ? (T)1 : (T)0;
            x[v] = diag ? (T)1 / s[v] : (T)0;
            if (diag) a.ch[bc].dprev[(row & 1) * kP + col] = (double)s[v];
        }
        tile_store<T>(reinterpret_cast<T*>(pa.S[bc][0]) + own, l, s);
        tile_store<T>(reinterpret_cast<T*>(pa.X[bc][0]) + own, l, x);
        if (first_thread) *nxt = NSState{row, kNsForm, 0, 0, 0};
        return;
    }
    // which row and iterate
    int row = prev.row, it = 0, xb = prev.xb;
    const T* Xs = reinterpret_cast<const T*>(pa.X[bc][xb]);
    if (prev.phase == kNsResid) {
        const bool warm = chain != 2 && ch.index(row) > 0;
        const double f = l < kPT ? flag_in[l] : 0.0;
        const bool met = __ballot(f != 0.0) == 0ull;
        const bool last = prev.it + steps >= (warm ? a.max_iter : a.max_iter + 4);
        if (met || last) {
            if (!met && first_thread) atomicOr(a.flags + kNsFail, 1);
            if (ch.index(row) + 1 >= ch.rows) {
                if (first_thread) *nxt = NSState{-1, kNsFinished, 0, 0, slot + 1};
                return;
            }
            row += ch.dir;
            xb ^= 1;
            Xs = reinterpret_cast<const T*>(pa.X[bc][xb]);
        } else {
            it = prev.it + steps;
            Xs = reinterpret_cast<const T*>(pa.Y[bc][(slot - 1) & 1]);
        }
    }
    const T* const Ps = reinterpret_cast<const T*>(pa.S[bc][xb]);
    v4 P[kPT], X[kPT];
    const v4 xc = tile_load<T>(Xs + own, l);               // X_C: tile (w, C), read transposed
#pragma unroll
    for (int k = 0; k < kPT; ++k) P[k] = tile_load<T>(Ps + ((int64_t)w * kPT + k) * 256, l);
#pragma unroll
    for (int k = 0; k < kPT; ++k) X[k] = tile_load<T>(Xs + ((int64_t)w * kPT + k) * 256, l);
    // the next row's E and this row's pivot block and its diagonal, used after the products
    const int next = ch.index(row) + 1 < ch.rows ? row + ch.dir : row;
    const v4 e = tile_load<T>(H + next * blk + own, l), sold = tile_load<T>(Ps + own, l);
    const double* const dp = a.ch[bc].dprev + (row & 1) * kP;
    const double dc = dp[col];
    double dr[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) dr[v] = dp[rowi(v)];
    if (it == 0 && C == w) {
        // the row's pivots: the diagonal of its block
        double dmin = __builtin_inf();
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (rowi(v) == col && col < n) dmin = (double)sold[v];
        record_min_pivot(dmin, a.diag, a.flags);
    }
    const int at = c * ldy + 16 * w + 4 * q, from = c * ldy + 4 * q;
    auto product = [&](const v4 (&M)[kPT], const T* p) {
        acc_t acc{0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < kPT; ++k) {
            const v4 y = panel_get<T>(p + from + 16 * k);
#pragma unroll
            for (int t = 0; t < 4; ++t) acc = Frag<T>::mma(M[k][t], y[t], acc);
        }
        return acc;
    };
    panel_put<T>(pan[0] + at, xc);
    lds_barrier();
    v4 u = product(P, pan[0]);
    bool ok = true;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        u[v] = (T)(rowi(v) == col ? 1 : 0) - u[v];
        ok = ok && fabs((double)u[v]) <= done;             // false for NaN
    }
    panel_put<T>(pan[1] + at, u);
    const int all_ok = __ballot(ok) == ~0ull ? 1 : 0;
    if (l == 0) pass[w] = all_ok;
    lds_barrier();
    if (threadIdx.x == 0) {
        int met = 1;
#pragma unroll
        for (int k = 0; k < kPT; ++k) met &= pass[k];
        flag_out[C] = met ? 0.0 : 1.0;
    }
    v4 h = product(X, pan[1]);                             // X u
    if constexpr (rounds) {
        panel_put<T>(pan[0] + at, h);
        lds_barrier();
        v4 u2 = product(P, pan[0]);
#pragma unroll
        for (int v = 0; v < 4; ++v) u2[v] = u[v] - u2[v];
        panel_put<T>(pan[1] + at, u2);
        lds_barrier();
        const v4 z = product(X, pan[1]);                   // X u2
#pragma unroll
        for (int v = 0; v < 4; ++v) h[v] = (xc[v] + h[v]) + z[v];
    } else {
#pragma unroll
        for (int v = 0; v < 4; ++v) h[v] += xc[v];
    }
    tile_store<T>(reinterpret_cast<T*>(pa.Y[bc][slot & 1]) + own, l, h);
    if (next != row) {
        // the next row's pivot block and first iterate, in case this round is the last
        v4 s, x;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const bool diag = rowi(v) == col;
            if (rowi(v) >= n || col >= n) {
                s[v] = x[v] = diag ? (T)1 : (T)0;
                if (diag) a.ch[bc].dprev[(next & 1) * kP + col] = 1.0;
                continue;
            }
            s[v] = e[v] - (T)a.g2 * h[v];
            if (diag) {
                x[v] = h[v] + ((T)1 / s[v] - (T)(1.0 / dc));
                a.ch[bc].dprev[(next & 1) * kP + col] = (double)s[v];
            } else {
                x[v] = h[v] - (T)((double)(s[v] - sold[v]) / (dr[v] * dc));
            }
        }
        tile_store<T>(reinterpret_cast<T*>(pa.S[bc][xb ^ 1]) + own, l, s);
        tile_store<T>(reinterpret_cast<T*>(pa.X[bc][xb ^ 1]) + own, l, x);
    }
    tile_store<T>(H + row * blk + own, l, h);
    if (first_thread) *nxt = NSState{row, kNsResid, it, xb, 0};
}

}  // namespace xbk

hipError_t xbk_launch_ns_panels(const xbk::NSPanelArgs& a, bool fp32, int chain, int slot, hipStream_t s)
{
    if (a.a.n_p != xbk::kP || chain < -1 || chain > 2) return hipErrorInvalidValue;
    const dim3 grid(xbk::kPT, chain < 0 ? 2 : 1), block(64 * xbk::kPT);
    if (fp32)
        hipLaunchKernelGGL(xbk::ns_panel_kernel<float>, grid, block, 0, s, a, chain, slot);
    else
        hipLaunchKernelGGL(xbk::ns_panel_kernel<double>, grid, block, 0, s, a, chain, slot);
    return hipGetLastError();
}
