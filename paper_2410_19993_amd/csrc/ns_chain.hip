// Newton-Schulz factor of crossbars with at most 64 columns: a whole chain of row
// blocks in one workgroup, one launch for both chains and one for the twist row.
//
// The method, its starting iterates, rounds and tolerances are those of the slot
// schedule (ns.hip); here a row block fits one workgroup's LDS, so a row costs three
// workgroup barriers instead of three launches, and nothing is padded past the last
// live 16 x 16 tile (LT = ceil(n / 16) tiles a side, one wave per output tile; the
// rest of the 64-wide block is decoupled padding that no product reads).
//
// Bound: the dependent chain.  A row is three LT x LT x LT tile products back to back
// on one CU's matrix cores (LT = 4: 4096 cycles for Q and 3072 each for Y and X'', which
// are formed on and above the diagonal: 4.3 us at the CU's float64 rate) plus an LDS round trip and a barrier each; the next row's E block is requested a
// row ahead, and the tolerance is a ballot per wave instead of a reduction of the
// largest entry.  Measured: 6.1 us a row at 50 columns (6.7 with whole products), 1.9 us
// at 32, about 1 us at 16, both chains at once (32 x 700 as its reciprocal: 0.70 ms for the factor, against
// 5.7 ms).  The slot schedule was bound by its launches instead, about 2.8 us of host
// time each, six per pair of rows at any size.
#include "common.h"

namespace xbk {

namespace {

template <typename T> struct CV4;
template <> struct CV4<double> { using type = d4_t; };
template <> struct CV4<float> { using type = f4_t; };

// Four values of lane l in an FRG tile (LDS or global memory), 16 bytes per access.
template <typename T>
__device__ __forceinline__ typename CV4<T>::type tile_get(const T* t, int l)
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
__device__ __forceinline__ void tile_put(T* t, int l, typename CV4<T>::type v)
{
    if constexpr (sizeof(T) == 8) {
        typedef double d2v __attribute__((ext_vector_type(2)));
        *reinterpret_cast<d2v*>(t + 2 * l) = d2v{v[0], v[1]};
        *reinterpret_cast<d2v*>(t + 128 + 2 * l) = d2v{v[2], v[3]};
    } else {
        *reinterpret_cast<f4_t*>(t + 4 * l) = v;
    }
}

// Output tile (tr, tc) of A B^T for LT x LT tiles in LDS.
template <typename T, int LT>
__device__ __forceinline__ typename Frag<T>::acc_t tile_product(const T* A, const T* B, int tr, int tc, int l)
{
    typename Frag<T>::acc_t acc{0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < LT; ++k) {
        const auto av = tile_get<T>(A + (tr * LT + k) * 256, l);
        const auto bv = tile_get<T>(B + (tc * LT + k) * 256, l);
#pragma unroll
        for (int t = 0; t < 4; ++t) acc = Frag<T>::mma(bv[t], av[t], acc);
    }
    return acc;
}

// What tile_put(t, l, v) would store, transposed.
template <typename T>
__device__ __forceinline__ void tile_put_across(T* t, int l, typename CV4<T>::type v)
{
#pragma unroll
    for (int k = 0; k < 4; ++k) t[frg<T>(Frag<T>::kidx(l >> 4, k), l & 15, 16)] = v[k];
}

// Tile of wave w: the tiles on and above the diagonal first, so that their waves are
// spread evenly over the SIMDs (wave w on SIMD w % 4).
template <int LT>
__device__ __forceinline__ void chain_tile(int w, int& tr, int& tc)
{
    for (tr = 0; tr < LT; ++tr) {
        if (w < LT - tr) {
            tc = tr + w;
            return;
        }
        w -= LT - tr;
    }
    for (tr = 1; w >= tr; ++tr) w -= tr;
    tc = w;
}

// Chains first, first + 1, ... (one per workgroup): 0 the top chain (rows 0..kt-1),
// 1 the bottom chain (rows m-1..kt+1), 2 the twist row, whose launch follows the
// chains' and, with `report` set, turns a missed tolerance into kErrConv.
template <typename T, int LT>
__global__ __launch_bounds__(64 * LT * LT) void ns_chain_kernel(NSArgs a, int first, int report)
{
    constexpr int NW = LT * LT, SZ = LT * LT * 256;
    constexpr bool rounds = sizeof(T) == 8;       // third-order rounds; float32: single steps
    constexpr double done = rounds ? 6.4e-5 / 64.0 : 1e-4;
    // Y and X'' are symmetric: their products on and above the diagonal only, where that
    // saves a SIMD a tile (LT >= 3: 2 of 3, 3 of 4)
    constexpr bool triangle = rounds && LT >= 3;
    using v4 = typename CV4<T>::type;
    __shared__ __align__(16) T sP[SZ], sQ[SZ], sX[2][SZ];
    __shared__ double rdg[2][16 * LT];       // reciprocals of the pivot block's diagonal
    __shared__ int pass[NW];
    const int l = threadIdx.x & 63, q = l >> 4;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int tr, tc;
    chain_tile<LT>(w, tr, tc);
    const int own = (tr * LT + tc) * 256, across = (tc * LT + tr) * 256;
    const int n = a.n, m = a.m, kt = m / 2, chain = first + (int)blockIdx.x;
    const int rows = chain == 0 ? kt : chain == 1 ? m - 1 - kt : 1;
    if (rows <= 0) return;
    const int start = chain == 0 ? 0 : chain == 1 ? m - 1 : kt, dir = chain == 1 ? -1 : 1;
    const int64_t blk = (int64_t)a.n_p * a.n_p;
    // this wave's tile within a 64 x 64 block, and this lane's row and columns in it
    T* const H = reinterpret_cast<T*>(a.H) + ((int64_t)tr * (a.n_p >> 4) + tc) * 256;
    const int row = 16 * tr + (l & 15);
    auto col = [&](int v) { return 16 * tc + Frag<T>::kidx(q, v); };

    v4 s = tile_get<T>(H + start * blk, l), x;
    if (chain == 2) {
        const v4 none{0, 0, 0, 0};
        const v4 ha = kt > 0 ? tile_get<T>(H + (kt - 1) * blk, l) : none;
        const v4 hb = kt + 1 < m ? tile_get<T>(H + (kt + 1) * blk, l) : none;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if (kt > 0) s[v] -= (T)a.g2 * ha[v];
            if (kt + 1 < m) s[v] -= (T)a.g2 * hb[v];
        }
    }
    double dmin = __builtin_inf();
    // cold start: the inverse of the pivot block's diagonal (identity on the padding)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const bool diag = row == col(v);
        if (row >= n || col(v) >= n) s[v] = diag ? (T)1 : (T)0;
        x[v] = diag ? (T)1 / s[v] : (T)0;
        if (diag && row < n) {
            rdg[0][row] = 1.0 / (double)s[v];
            dmin = ((double)s[v] < dmin || s[v] != s[v]) ? (double)s[v] : dmin;
        }
    }
    tile_put<T>(sP + own, l, s);
    tile_put<T>(sX[0] + own, l, x);
    int xb = 0;
    bool fail = false;
    lds_barrier();
    for (int k = 0; k < rows; ++k) {
        const int i = start + dir * k;
        const bool next = k + 1 < rows;
        v4 e{0, 0, 0, 0};
        if (next) e = tile_get<T>(H + (i + dir) * blk, l);
        // rows after a chain's first start warm
        const int maxit = (k > 0 && chain != 2) ? a.max_iter : a.max_iter + 4;
        v4 h;
        for (int it = 0;; it += rounds ? 2 : 1) {
            // Q = I - X P; a wave's tile passes when every entry is within the tolerance
            // (a NaN never is)
            v4 qv = tile_product<T, LT>(sX[xb], sP, tr, tc, l);
            bool ok = true;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                qv[v] = (T)(row == col(v) ? 1 : 0) - qv[v];
                ok = ok && fabs((double)qv[v]) <= done;
            }
            tile_put<T>(sQ + own, l, qv);
            const int all_ok = __ballot(ok) == ~0ull ? 1 : 0;
            if (l == 0) pass[w] = all_ok;
            lds_barrier();
            const bool fin = __ballot(l >= NW || pass[l] != 0) == ~0ull;
            const bool last = it + (rounds ? 2 : 1) >= maxit;
            if constexpr (triangle) {
                // Y = Q X, then X'' = X + Y + Q Y (into X's buffer below the diagonal)
                v4 y{0, 0, 0, 0};
                if (tr <= tc) {
                    y = tile_product<T, LT>(sQ, sX[0], tr, tc, l);
                    tile_put<T>(sX[1] + own, l, y);
                    if (tr < tc) tile_put_across<T>(sX[1] + across, l, y);
                }
                lds_barrier();
                if (tr <= tc) {
                    const v4 z = tile_product<T, LT>(sQ, sX[1], tr, tc, l);
#pragma unroll
                    for (int v = 0; v < 4; ++v) h[v] = (x[v] + y[v]) + z[v];
                    if (tr < tc) tile_put_across<T>(sX[0] + across, l, h);
                }
                lds_barrier();
                if (tr > tc) h = tile_get<T>(sX[0] + own, l);
            } else if constexpr (rounds) {
                // Y = Q X, then X'' = X + Y + Q Y
                const v4 y = tile_product<T, LT>(sQ, sX[0], tr, tc, l);
                tile_put<T>(sX[1] + own, l, y);
                lds_barrier();
                const v4 z = tile_product<T, LT>(sQ, sX[1], tr, tc, l);
#pragma unroll
                for (int v = 0; v < 4; ++v) h[v] = (x[v] + y[v]) + z[v];
            } else {
                // X' = X + Q X, into the other buffer
                const v4 y = tile_product<T, LT>(sQ, sX[xb], tr, tc, l);
#pragma unroll
                for (int v = 0; v < 4; ++v) h[v] = x[v] + y[v];
                xb ^= 1;
            }
            if (fin || last) {
                fail |= !fin;
                break;
            }
            x = h;
            tile_put<T>(sX[xb] + own, l, x);
            lds_barrier();
        }
        tile_put<T>(H + i * blk, l, h);
        if (!next) break;
        // the next row's pivot block E - g^2 H and its first iterate: H corrected to first
        // order in the change of the pivot block, with H taken as its diagonal there
        const double* rd = rdg[k & 1];
        const double rdr = row < n ? rd[row] : 1.0;
        v4 sv;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int c = col(v);
            sv[v] = e[v] - (T)a.g2 * h[v];
            x[v] = h[v] - (T)((double)(sv[v] - s[v]) * (rdr * (c < n ? rd[c] : 1.0)));
            if (row >= n || c >= n) sv[v] = x[v] = (T)0;
        }
        if (tr == tc) {
            // a diagonal tile: a quarter of its lanes hold one diagonal entry each
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (row != col(v)) continue;
                if (row >= n) {
                    sv[v] = x[v] = (T)1;
                    continue;
                }
                const double r = 1.0 / (double)sv[v];
                x[v] = h[v] + (T)(r - rdr);
                rdg[(k + 1) & 1][row] = r;
                dmin = ((double)sv[v] < dmin || sv[v] != sv[v]) ? (double)sv[v] : dmin;
            }
        }
        s = sv;
        tile_put<T>(sP + own, l, s);
        tile_put<T>(sX[xb] + own, l, x);
        lds_barrier();
    }
    if (tr == tc) record_min_pivot(dmin, a.diag, a.flags);
    if (threadIdx.x == 0) {
        if (fail) atomicOr(a.flags + kNsFail, 1);
        // the chains' launches have ended before the twist's begins
        if (report && chain == 2 && (fail || a.flags[kNsFail])) a.flags[kErrConv] = 1;
    }
}

template <typename T, int LT>
hipError_t launch_chain(const NSArgs& a, bool report, hipStream_t s)
{
    if (a.m > 1) {
        hipLaunchKernelGGL((ns_chain_kernel<T, LT>), dim3(2), dim3(64 * LT * LT), 0, s, a, 0, 0);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((ns_chain_kernel<T, LT>), dim3(1), dim3(64 * LT * LT), 0, s, a, 2, report ? 1 : 0);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_chain_t(const NSArgs& a, bool report, hipStream_t s)
{
    switch ((a.n + 15) / 16) {
        case 1: return launch_chain<T, 1>(a, report, s);
        case 2: return launch_chain<T, 2>(a, report, s);
        case 3: return launch_chain<T, 3>(a, report, s);
        case 4: return launch_chain<T, 4>(a, report, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

}  // namespace xbk

hipError_t xbk_launch_ns_chains(const xbk::NSArgs& a, bool fp32, bool report, hipStream_t s)
{
    if (a.n_p != 64 || a.n < 1 || a.n > 64 || a.m < 1) return hipErrorInvalidValue;
    return fp32 ? xbk::launch_chain_t<float>(a, report, s) : xbk::launch_chain_t<double>(a, report, s);
}
