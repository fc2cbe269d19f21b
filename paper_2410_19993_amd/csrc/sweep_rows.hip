// Forward and back substitution of a plan's batch where the slab sweep (sweep.hip: one
// workgroup walks all the row blocks for 16 input vectors) leaves the GPU waiting:
//
//  * sweep_small_kernel, n <= 64: both chains of the twisted order in one workgroup, or
//    a workgroup each.
//    A row block is at most 4 x 4 tiles, so a step is a short dependent chain (LDS
//    read, 4 LT matrix instructions, LDS write, barrier); the chains' steps run side by
//    side and nothing is computed past the last live 16 x 16 tile.
//  * sweep_step_kernel, larger n and batches that leave most CUs idle: one launch per
//    step of the two chains, a row block's product spread over the GPU (a few row tiles
//    and slabs per workgroup).
//  * recover_rows_kernel: the word lines and node voltages of every row at once, from
//    the solution the sweep left in the workspace.
//
// Panels of these kernels in memory (right-hand sides, forward results, solutions) are
// 16 x n_p blocks in the fragment-tiled layout of H, so that a wave's access is contiguous;
// the slab sweep's are [16][n_p] rows.
//
// The products, the order of their sums and the recovery are those of the slab sweep, so
// an input vector's results have the same bits whichever kernel ran and whatever shares
// its batch.
#include <algorithm>

#include "recover.h"

namespace xbk {

namespace {

typedef double d2v __attribute__((ext_vector_type(2)));
template <typename T> struct R4;
template <> struct R4<double> { using type = d4_t; };
template <> struct R4<float> { using type = f4_t; };

// A-operand fragment of an FRG tile.
template <typename T>
__device__ __forceinline__ typename R4<T>::type frag_load(const T* __restrict__ tile, int l)
{
    if constexpr (sizeof(T) == 8) {
        const d2v lo = *reinterpret_cast<const d2v*>(tile + 2 * l);
        const d2v hi = *reinterpret_cast<const d2v*>(tile + 128 + 2 * l);
        return d4_t{lo[0], lo[1], hi[0], hi[1]};
    } else {
        return *reinterpret_cast<const f4_t*>(tile + 4 * l);
    }
}
__device__ __forceinline__ void frag_store(double* tile, int l, d4_t v)
{
    *reinterpret_cast<d2v*>(tile + 2 * l) = d2v{v[0], v[1]};
    *reinterpret_cast<d2v*>(tile + 128 + 2 * l) = d2v{v[2], v[3]};
}
__device__ __forceinline__ void frag_store(float* tile, int l, f4_t v) { *reinterpret_cast<f4_t*>(tile + 4 * l) = v; }
__device__ __forceinline__ d4_t load4(const double* p)
{
    const d2v lo = *reinterpret_cast<const d2v*>(p), hi = *reinterpret_cast<const d2v*>(p + 2);
    return d4_t{lo[0], lo[1], hi[0], hi[1]};
}
__device__ __forceinline__ f4_t load4(const float* p) { return *reinterpret_cast<const f4_t*>(p); }
__device__ __forceinline__ void store4(double* p, d4_t v)
{
    *reinterpret_cast<d2v*>(p) = d2v{v[0], v[1]};
    *reinterpret_cast<d2v*>(p + 2) = d2v{v[2], v[3]};
}
__device__ __forceinline__ void store4(float* p, f4_t v) { *reinterpret_cast<f4_t*>(p) = v; }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// ---------------------------------------------------------------------------
// n <= 64 (n_p = 64), m >= 3.  Waves c LT + t: row tile t of chain c (0: rows from the
// top, 1: from the bottom).  Forward step p < F = kt is row p and row m - 1 - (p - late):
// the bottom chain is one row shorter when m is even, and then starts one step late
// (from a zero panel, whose product adds nothing).  Both chains form the twist row's
// product, each for the panel it continues from.  Back step s is row kt - s and row
// kt + s (the late chain repeats u_kt in step 1), or without node voltages (UP = false)
// the bottom chain alone: the output currents depend on u_{m-1} only.
//
// A step's panel goes to the other of two LDS buffers: one barrier a step.  H,
// right-hand sides and forward results are requested D steps ahead, and every load is
// unconditional (clamped rows), so that no step waits for a load it does not use: with
// the loads behind branches and one step ahead, a step of 32 columns took 1.14 us.
//
// Bound: the latency of a step, 4 LT dependent matrix instructions of each chain between
// an LDS write, a barrier and an LDS read, and at LT = 4 the 64 KB of H that a step
// brings through one CU's L1.  Measured: 0.64 us a step at 32 columns (700 rows, 16
// vectors: 448 us; the slab sweep 3932 us, whose one matrix-core wave walks both chains
// in turn on padded blocks), 10 us for 16 x 16 (99 us); at 50 columns 1.0 us with a
// workgroup per chain (1.7 with both in one).
template <int V> struct Slot { static constexpr int value = V; };

//
// PART: kBoth, or for more than 32 columns a workgroup per chain (blockIdx.y) and two
// launches, kForward and kTwistBack, with the chains' last forward results handed over in
// a.ysteps ([slab][chain], since a back chain overwrites its own in Z): half of H per
// CU.
enum : int { kBoth, kForward, kTwistBack };

template <int LT, bool UP, int PART>
__global__ __launch_bounds__((PART == kBoth ? 128 : 64) * LT) void sweep_small_kernel(SweepArgs a)
{
    constexpr int n_p = 64, ldy = 16 * LT + 4, D = 4;
    __shared__ __align__(16) double pan[PART == kBoth ? 2 : 1][2][16 * ldy];   // [chain][buffer][vector][CPR position]
    const int l = threadIdx.x & 63, q = l >> 4, col = l & 15;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // without the upward back chain the second launch is the bottom chain's alone
    const int c = PART == kBoth ? w / LT : PART == kTwistBack && !UP ? 1 : (int)blockIdx.y, t = w % LT;
    const int pc = PART == kBoth ? c : 0;                      // the chain's panels in LDS
    const int n = a.n, m = a.m, kt = m / 2, F = kt, late = kt - (m - 1 - kt);
    const int last = F + (UP ? kt : m - 1 - kt), late_back = UP ? late : 0;
    const int slab = blockIdx.x, b = 16 * slab + col;
    const bool bval = b < a.B;
    const double g = a.g_bl;
    const double* const H = reinterpret_cast<const double*>(a.H) + (int64_t)t * (n_p >> 4) * 256;
    double* const Z = reinterpret_cast<double*>(a.Z) + (int64_t)slab * m * 16 * n_p + t * 256;
    const double* const C = a.c + 16 * t + q;                  // zero on the padding
    // input voltage of this lane's vector; reciprocal ordering: none (the terminations'
    // right-hand side of the last row is set apart)
    const bool src = bval && !a.term;
    const double* const Vb = a.V + (src ? (int64_t)b * m : 0);
    const int64_t blk = n_p * n_p, zrow = 16 * n_p;
    const int at = col * ldy + 16 * t + 4 * q;                 // this lane's rows in a panel
    double* const hand = reinterpret_cast<double*>(a.ysteps) + (int64_t)slab * 2 * zrow + t * 256;

    auto row_of = [&](int p) {
        p = min(p, last);
        if (c == 0) return p <= F ? p : (UP ? kt - (p - F) : kt);
        return p < F ? m - 1 - max(p - late, 0) : kt + max(p - F - late_back, 0);
    };
    // of step p, in slot p % D: the H tiles, and (rq, vq) the source coupling and input
    // voltage of its row (forward) or its forward result (back)
    d4_t ring[D][LT], rq[D];
    double vq[D];
    auto load_h = [&](int p, d4_t (&h)[LT]) {
        const double* Hi = H + row_of(p) * blk;
#pragma unroll
        for (int k = 0; k < LT; ++k) h[k] = frag_load(Hi + k * 256, l);
    };
    // right-hand side V_i c_i of step p <= F, multiplied where it is used
    auto load_rhs = [&](int p, d4_t& r, double& v) {
        const int i = row_of(min(p, F));
        v = Vb[src ? i : 0];
        const double* ci = C + (int64_t)i * n_p;
        r = d4_t{ci[0], ci[4], ci[8], ci[12]};
    };
    auto rhs = [&](const d4_t& r, double v) { return r * (src ? v : 0.0); };
    auto load_z = [&](int p, d4_t& r) { r = frag_load<double>(Z + row_of(p) * zrow, l); };
    auto product = [&](const d4_t (&h)[LT], const double* y) {
        d4_t acc{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < LT; ++k) {
            const d4_t yv = load4(y + col * ldy + 16 * k + 4 * q);
#pragma unroll
            for (int s = 0; s < 4; ++s) acc = Frag<double>::mma(h[k][s], yv[s], acc);
        }
        return acc;
    };
    auto axpy = [&](d4_t x, d4_t y) {                          // g x + y
#pragma unroll
        for (int v = 0; v < 4; ++v) x[v] = __builtin_fma(g, x[v], y[v]);
        return x;
    };
    auto rotate = [&]() {                                       // slot 0 becomes the next step's
#pragma unroll
        for (int k = 0; k < LT; ++k) {
            const d4_t r0 = ring[0][k];
#pragma unroll
            for (int d = 0; d + 1 < D; ++d) ring[d][k] = ring[d + 1][k];
            ring[D - 1][k] = r0;
        }
        const d4_t r0 = rq[0];
        const double v0 = vq[0];
#pragma unroll
        for (int d = 0; d + 1 < D; ++d) {
            rq[d] = rq[d + 1];
            vq[d] = vq[d + 1];
        }
        rq[D - 1] = r0;
        vq[D - 1] = v0;
    };

    const int first = PART == kTwistBack ? F : 0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        load_rhs(first + d, rq[d], vq[d]);
        load_h(first + d, ring[d]);
    }
    const bool idle = c == 1 && late == 1;
    int cur = 0;
    d4_t f0{0.0, 0.0, 0.0, 0.0};
    if constexpr (PART != kTwistBack) {
        // the first row's right-hand side: the first panel, or, for a chain that starts late,
        // what step 0 adds to its zero product
        f0 = rhs(rq[0], vq[0]);
        if (a.term && c == 1) {
            const double* Vt = a.V + (int64_t)(bval ? b : 0) * n + (n - 1);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int k = 16 * t + Frag<double>::drow(q, v);
                const double x = Vt[-min(k, n - 1)];
                f0[v] = (bval && k < n) ? a.g_sense * x : 0.0;
            }
        }
        store4(&pan[pc][0][at], idle ? d4_t{0.0, 0.0, 0.0, 0.0} : f0);
        lds_barrier();
    }

    // forward, step p in ring slot d
    auto forward = [&](int p, auto slot) {
        constexpr int d = decltype(slot)::value;
        const d4_t z = product(ring[d], pan[pc][cur]);
        frag_store(Z + row_of(p) * zrow, l, z);
        d4_t f = rhs(rq[(d + 1) % D], vq[(d + 1) % D]);
        if (p == 0 && idle) f = f0;
        // the next row's panel, or the forward result itself for the twist
        const d4_t y = axpy(z, f);
        store4(&pan[pc][cur ^ 1][at], p + 1 < F ? y : z);
        load_h(p + D, ring[d]);
        load_rhs(p + D, rq[d], vq[d]);
        cur ^= 1;
        lds_barrier();
    };
    int p = first;
    for (; p + D <= F; p += D) {
        forward(p, Slot<0>{});
        forward(p + 1, Slot<1>{});
        forward(p + 2, Slot<2>{});
        forward(p + 3, Slot<3>{});
    }
    for (; p < F; ++p) {
        forward(p, Slot<0>{});
        rotate();
    }
    if constexpr (PART == kForward) {
        frag_store(hand + c * zrow, l, load4(&pan[pc][cur][at]));   // this lane's own entries
        return;
    }
    // twist row
    const d4_t ft = rhs(rq[0], vq[0]);
#pragma unroll
    for (int d = 0; d < D; ++d) load_z(F + max(d, 1), rq[d]);
    d4_t zt, zb;
    if constexpr (PART == kTwistBack) {
        zt = frag_load<double>(hand, l);
        zb = frag_load<double>(hand + zrow, l);
    } else {
        zt = load4(&pan[0][cur][at]);
        zb = load4(&pan[1][cur][at]);
    }
    const d4_t yt = axpy(zb, axpy(zt, ft));
    store4(&pan[pc][cur ^ 1][at], yt);
    cur ^= 1;
    lds_barrier();
    const d4_t ut = product(ring[0], pan[pc][cur]);
    if (UP && c == 0) frag_store(Z + kt * zrow, l, ut);
    store4(&pan[pc][cur ^ 1][at], ut);
    load_h(F + D, ring[0]);
    load_z(F + D, rq[0]);
    cur ^= 1;
    lds_barrier();
    rotate();
    if (PART == kBoth && !UP && c == 0) {
        for (p = F + 1; p <= last; ++p) lds_barrier();
        return;
    }
    // back, step p in ring slot d
    d4_t u = ut;
    auto back = [&](int p, auto slot) {
        constexpr int d = decltype(slot)::value;
        u = axpy(product(ring[d], pan[pc][cur]), rq[d]);
        if (UP) {
            if (idle && p == F + 1) u = ut;
            frag_store(Z + row_of(p) * zrow, l, u);
        }
        store4(&pan[pc][cur ^ 1][at], u);
        load_h(p + D, ring[d]);
        load_z(p + D, rq[d]);
        cur ^= 1;
        lds_barrier();
    };
    p = F + 1;
    for (; p + D <= last + 1; p += D) {
        back(p, Slot<0>{});
        back(p + 1, Slot<1>{});
        back(p + 2, Slot<2>{});
        back(p + 3, Slot<3>{});
    }
    for (; p <= last; ++p) {
        back(p, Slot<0>{});
        rotate();
    }
    if (c == 1 && bval) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int k = 16 * t + Frag<double>::drow(q, v);
            if (k < n) a.Iout[(int64_t)b * n + k] = a.g_sense * u[v];
        }
    }
}

// ---------------------------------------------------------------------------
// Word lines and node voltages of row i for the vectors of a slab, one workgroup each:
// blockIdx.x = slab m + i, kHelpers waves of four vectors.  Bound: HBM (u read, 2 x
// node voltages written) once enough rows are in flight; one row alone is the latency
// of its segmented scans (5.2 us for 16 x 16 with 8 vectors, 9.6 us for 700 x 32 with 16).
template <int NT>
__global__ __launch_bounds__(64 * kHelpers) void recover_rows_kernel(SweepArgs a)
{
    using R = RowRecover<double, NT>;
    constexpr int n_p = R::n_p, ldy = R::ldy;
    extern __shared__ __align__(16) double lds[];
    const int n = a.n, m = a.m;
    const int slab = blockIdx.x / m, i = blockIdx.x % m;
    const int lg = seg_lg(n, R::LR), PL = padded_len(n, R::LR);
    double* ybuf = lds;                       // [16][ldy]
    double* wv = ybuf + 16 * ldy;             // [16][PL]
    double* coef = wv + 16 * PL;              // [3][PL] fr, ip, G of the row
    const double* U = reinterpret_cast<const double*>(a.Z) + ((int64_t)slab * m + i) * 16 * n_p;
    const int l = threadIdx.x & 63, h = threadIdx.x >> 6;
    const int vecs = min(16, a.B - 16 * slab);
    for (int e = threadIdx.x; e < 8 * ((n + 15) & ~15); e += 64 * kHelpers) {
        const int le = e & 63, ce = le & 15;                 // 16 bytes of lane le of a tile
        if (ce < vecs)
            *reinterpret_cast<d2v*>(ybuf + ce * ldy + 16 * (e >> 7) + 4 * (le >> 4) + 2 * ((e >> 6) & 1)) =
                *reinterpret_cast<const d2v*>(U + 2 * e);
    }
    for (int j = threadIdx.x; j < n; j += 64 * kHelpers) {
        const int pj = padj(j, lg);
        const int64_t o = (int64_t)i * n + j;
        coef[pj] = a.fr[o];
        coef[PL + pj] = a.ip[o];
        coef[2 * PL + pj] = a.Gc[o];
    }
    const int bb = 16 * slab + h * R::VPW + l / R::LR;
    const double vb = (bb < a.B && !a.term) ? a.V[(int64_t)bb * m + i] : 0.0;
    __syncthreads();
    if (h * R::VPW < vecs) R::run(a, slab, i, vb, ybuf, wv, coef, h, l, lg, PL);
}

template <int NT>
hipError_t launch_recover_rows(const SweepArgs& a, hipStream_t s)
{
    using R = RowRecover<double, NT>;
    const int64_t blocks = (int64_t)a.m * a.nslab;
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    const size_t lds = (16 * (size_t)R::ldy + 19 * (size_t)padded_len(a.n, R::LR)) * sizeof(double);
    hipLaunchKernelGGL((recover_rows_kernel<NT>), dim3((unsigned)blocks), dim3(64 * kHelpers), lds, s, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// One step of both chains as a launch: H_row (its row tiles over the GPU) times the
// panels of every slab.  Forward: z = H y, stored, and the next row's right-hand side
// panel y' = f + g z.  Twist and back: u = H y, u = z + g H u', stored over z.
//
// Bound: few vectors, the start of a launch and one wave's chain of n_p / 4 dependent
// matrix instructions (K is not split: the sums keep the slab sweep's order); more, the
// L2-to-L1 rate.  Measured a step (two rows) with one vector: 5.0 us at n_p = 256, 5.7 at
// 320, 8.0 at 512, against 21, 35 and 70 us on one workgroup; 512 vectors at 512: 17
// against 72 us (24 with panels in rows, whose loads touch twice the cache lines).
// Slabs up to which the steps are launches over the GPU (n_p > 128), and up to which each
// chain has workgroups of its own.  Microseconds a step with node voltages, as launches /
// chain per workgroup / slab per workgroup: 1024 vectors n = 512 28 / 37 / 72, 320 18.7 /
// 18.4 / 36, 256 12.5 / 11.7 / 22, 192 9.1 / 9.3 / 18; 1536 vectors 40 / 38, 22 / 18.5,
// 16.5 / 12.3.  (The line is one for all sizes: at 64 slabs it costs 256 and 320 columns up
// to 7%.)  At n_p = 128 a step is too short to be a launch (4.6 / 3.7 / 7.4 with one
// vector).  Refinement sweeps (float32, with their residual) as launches / slab per
// workgroup: 2048 vectors 36 / 44 at 512, 31 / 38 at 448, 24 / 28 at 384, 12.4 / 13.5 at 192;
// 1536 vectors 21 / 27 at 320, 17 / 20 at 256.
constexpr int kStepSlabs = 64, kPartSlabs = 128;

template <typename T>
struct StepJob {
    int row = -1;          // row whose product this is (-1: none)
    int next = -1;         // forward: row whose right-hand side panel follows (-1: none)
    const T* pan = nullptr;        // panel of slab 0 (16 x n_p, FRG)
    T* ynext = nullptr;            // forward: next panel of slab 0
};
template <typename T>
struct StepArgs {
    SweepArgs a;
    StepJob<T> job[2];
    int64_t pan_stride;    // elements between the panels of consecutive slabs
    int back;              // 0: forward or twist (u = H y), 1: u = z + g H u'
};

// Panels of the first rows (ra = rb = -1) or of the twist row, y = f + g z_ra + g z_rb, with
// f = V c, or in refinement sweeps past the first the residual.
template <typename T>
__global__ void step_form_kernel(SweepArgs a, int row0, T* y0, int row1, T* y1, int ra, int rb)
{
    const int n_p = a.n_p, m = a.m, n = a.n;
    const int64_t panel = (int64_t)16 * n_p, total = panel * a.nslab;
    const int i = blockIdx.y == 0 ? row0 : row1;
    T* y = blockIdx.y == 0 ? y0 : y1;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t slab = e / panel, o = e - slab * panel;
        int col, k;
        frg_rc<T>(o, n_p, col, k);
        const int b = (int)(16 * slab) + col;
        const bool bval = b < a.B;
        T f = 0;
        if (sizeof(T) == 4 && a.iter > 0) {
            if (k < n) f = reinterpret_cast<const T*>(a.R)[slab * m * panel + i * panel + cpr<T>(col, k, n_p)];
        } else if (a.term) {
            if (i == m - 1 && bval && k < n) f = (T)(a.g_sense * a.V[(int64_t)b * n + (n - 1 - k)]);
        } else if (bval) {
            f = (T)(a.c[(int64_t)i * n_p + k] * a.V[(int64_t)b * m + i]);
        }
        const T* Zs = reinterpret_cast<const T*>(a.Z) + slab * m * panel + o;
        const T g = (T)a.g_bl;
        if (ra >= 0) f = fma_t(g, Zs[ra * panel], f);
        if (rb >= 0) f = fma_t(g, Zs[rb * panel], f);
        y[e] = f;
    }
}

// One wave a workgroup: row tile idx % KC, S slabs.  Workgroup b runs on XCD b % 8: with
// two jobs each chain has four XCDs, and consecutive workgroups of an XCD group take
// consecutive row tiles, so an XCD's L2 holds a quarter of each H block.
//
// float: the sweeps of the refinement.  A solution row is then the correction d; it is
// added to the float64 solution at once, and the largest |d| and |u| of each vector go
// to a.norms as bit patterns (their order is that of the non-negative numbers, a NaN
// above all), for step_decide_kernel.
template <typename T, int NT, int S>
__global__ __launch_bounds__(64) void sweep_step_kernel(StepArgs<T> sa)
{
    using v4 = typename R4<T>::type;
    constexpr bool IR = sizeof(T) == 4;
    constexpr int n_p = 64 * NT, KC = 4 * NT;
    constexpr int PF = S == 1 ? 12 : 6;                    // chunks in flight
    const SweepArgs& a = sa.a;
    const bool two = sa.job[1].row >= 0 && sa.job[0].row >= 0;
    const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
    const int c = two ? xcd >> 2 : (sa.job[0].row >= 0 ? 0 : 1);
    const int idx = two ? local * 4 + (xcd & 3) : blockIdx.x;
    const int t = idx % KC, slab0 = (idx / KC) * S;
    if (slab0 >= a.nslab) return;
    const int last = a.nslab - 1;                          // slabs past the last repeat it, unstored
    bool live[S];
    bool any = false;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        live[s] = slab0 + s <= last && !(IR && a.iter > 0 && a.slab_done[min(slab0 + s, last)]);
        any |= live[s];
    }
    if (!any) return;
    const int row = c == 0 ? sa.job[0].row : sa.job[1].row;
    const int next = c == 0 ? sa.job[0].next : sa.job[1].next;
    const T* const pan = c == 0 ? sa.job[0].pan : sa.job[1].pan;
    T* const ynext = c == 0 ? sa.job[0].ynext : sa.job[1].ynext;
    const int l = threadIdx.x & 63, q = l >> 4, col = l & 15;
    const int m = a.m, n = a.n;
    const T* const H = reinterpret_cast<const T*>(a.H) + (int64_t)row * n_p * n_p + (int64_t)t * KC * 256;
    const T* y[S];
#pragma unroll
    for (int s = 0; s < S; ++s)
        y[s] = pan + min(slab0 + s, last) * sa.pan_stride;
    v4 hr[PF], yr[PF][S], acc[S];
#pragma unroll
    for (int k = 0; k < PF; ++k) {
        hr[k] = frag_load(H + k * 256, l);
#pragma unroll
        for (int s = 0; s < S; ++s) yr[k][s] = frag_load(y[s] + 256 * k, l);
    }
    // requested before the product, used after it: the forward result (back), or the next
    // row's right-hand side
    const int o = col * n_p + 16 * t + 4 * q;              // in the refinement's CPR panels
    const int64_t rowo = (int64_t)row * 16 * n_p + o, zslab = (int64_t)m * 16 * n_p;
    T* const Z = reinterpret_cast<T*>(a.Z) + (int64_t)row * 16 * n_p + 256 * t;
    const bool fwd = next >= 0, resid = IR && a.iter > 0;
    v4 e[S];
    d4_t cn{0.0, 0.0, 0.0, 0.0}, up[IR ? S : 1];
    double vn[S];
    if (sa.back) {
#pragma unroll
        for (int s = 0; s < S; ++s) e[s] = frag_load<T>(Z + min(slab0 + s, last) * zslab, l);
    } else if (resid) {
        const T* R = reinterpret_cast<const T*>(a.R) + (int64_t)(fwd ? next : 0) * 16 * n_p + o;
#pragma unroll
        for (int s = 0; s < S; ++s) e[s] = load4(R + min(slab0 + s, last) * zslab);
    } else {
        const double* ci = a.c + (int64_t)(fwd ? next : 0) * n_p + 16 * t;
#pragma unroll
        for (int v = 0; v < 4; ++v) cn[v] = ci[Frag<T>::drow(q, v)];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int b = 16 * (slab0 + s) + col;
            const bool src = fwd && b < a.B && !a.term;
            const double v = a.V[src ? (int64_t)b * m + next : 0];
            vn[s] = src ? v : 0.0;
        }
    }
    if (IR && !fwd) {
        // a solution row (forward rows without a next one are loaded in vain)
#pragma unroll
        for (int s = 0; s < S; ++s)
            up[IR ? s : 0] = a.iter > 0 ? load4(a.Uin + rowo + min(slab0 + s, last) * zslab) : d4_t{0.0, 0.0, 0.0, 0.0};
    }
#pragma unroll
    for (int s = 0; s < S; ++s) acc[s] = v4{0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < KC; ++k) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int s = 0; s < S; ++s) acc[s] = Frag<T>::mma(hr[k % PF][j], yr[k % PF][s][j], acc[s]);
        if (k + PF < KC) {
            hr[k % PF] = frag_load(H + (k + PF) * 256, l);
#pragma unroll
            for (int s = 0; s < S; ++s) yr[k % PF][s] = frag_load(y[s] + 256 * (k + PF), l);
        }
    }
    const T g = (T)a.g_bl;
    const bool solution = sa.back || row == m / 2;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        if (!live[s]) continue;
        const int slab = slab0 + s, b = 16 * slab + col;
        v4 u = acc[s];
        if (sa.back) {
#pragma unroll
            for (int v = 0; v < 4; ++v) u[v] = fma_t(g, u[v], e[s][v]);
        }
        frag_store(Z + slab * zslab, l, u);
        if (fwd) {
            v4 yn;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const T f = resid ? (16 * t + Frag<T>::drow(q, v) < n ? e[s][v] : (T)0) : (T)(cn[v] * vn[s]);
                yn[v] = fma_t(g, u[v], f);
            }
            frag_store(ynext + (int64_t)slab * 16 * n_p + 256 * t, l, yn);
        }
        if (!solution) continue;
        d4_t x;
#pragma unroll
        for (int v = 0; v < 4; ++v) x[v] = (double)u[v];
        if constexpr (IR) {
            double dm = 0.0, um = 0.0;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const double d = x[v];
                x[v] = up[s][v] + d;
                dm = nan_max(dm, fabs(d));
                um = nan_max(um, fabs(x[v]));
            }
            store4(a.Uout + rowo + slab * zslab, x);
            if (a.tol >= 0.0) {
                for (int off = 16; off < 64; off <<= 1) {
                    dm = nan_max(dm, __shfl_xor(dm, off));
                    um = nan_max(um, __shfl_xor(um, off));
                }
                if (q == 0) {
                    unsigned long long* key = a.norms + 2 * (int64_t)b;
                    atomicMax(key, __builtin_bit_cast(unsigned long long, fabs(dm)));
                    atomicMax(key + 1, __builtin_bit_cast(unsigned long long, fabs(um)));
                }
            }
        }
        if (row == m - 1) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int k = 16 * t + Frag<T>::drow(q, v);
                if (b < a.B && k < n) a.Iout[(int64_t)b * n + k] = a.g_sense * x[v];
            }
        }
    }
}

// Refinement bookkeeping of every slab after a sweep by steps (the slab sweep's own rule:
// SweepCtx::decide); clears the norms for the next sweep.
__global__ __launch_bounds__(64) void step_decide_kernel(SweepArgs a)
{
    const int slab = blockIdx.x * 4 + (threadIdx.x >> 4), c = threadIdx.x & 15;
    const bool open = slab < a.nslab && !(a.iter > 0 && a.slab_done[slab]);
    bool ok = true;
    if (open) {
        unsigned long long* key = a.norms + 2 * (16 * (int64_t)slab + c);
        const double D = __builtin_bit_cast(double, key[0]), U = __builtin_bit_cast(double, key[1]);
        key[0] = key[1] = 0ull;
        double* dprev = a.dnorm + (int64_t)slab * 16 + c;
        const double est = (a.iter > 0 && *dprev > 0.0) ? D * fmin(1.0, D / *dprev) : D;
        ok = (D == 0.0) || (a.iter > 0 && est <= a.tol * U);
        *dprev = D;
    }
    const unsigned long long bad = __ballot(!ok) >> (threadIdx.x & 48) & 0xffffull;
    if (open && c == 0) {
        const bool all = bad == 0, last = a.iter + 1 >= a.max_iter;
        if (all || last) {
            a.slab_done[slab] = 1;
            a.slab_final[slab] = (a.iter + 1) & 1;
            atomicMax(a.flags + kIrIters, a.iter + 1);
            if (!all) atomicOr(a.flags + kErrConv, 1);
        }
    }
}

template <typename T, int NT, int S>
hipError_t launch_step(const StepArgs<T>& sa, hipStream_t s)
{
    const int work = 4 * NT * ((sa.a.nslab + S - 1) / S);
    const bool two = sa.job[0].row >= 0 && sa.job[1].row >= 0;
    hipLaunchKernelGGL((sweep_step_kernel<T, NT, S>), dim3(two ? 8 * ((work + 3) / 4) : work), dim3(64), 0, s, sa);
    return hipGetLastError();
}

template <typename T, int NT, int S>
hipError_t run_steps(const SweepArgs& a, hipStream_t s)
{
    const int m = a.m, kt = m / 2;
    const int64_t row = (int64_t)16 * a.n_p, panel = row * a.nslab;
    T* const Y = reinterpret_cast<T*>(a.ysteps);           // [2 chains][2][nslab][16][n_p]
    T* const Z = reinterpret_cast<T*>(a.Z);
    const unsigned blocks = (unsigned)std::min<int64_t>((panel + 255) / 256, 2048);
    const bool bottom = kt + 1 < m, up = a.node_v != nullptr || sizeof(T) == 4;
    StepArgs<T> sa;
    sa.a = a;
    hipError_t e = hipSuccess;
    if (kt > 0) {
        hipLaunchKernelGGL(step_form_kernel<T>, dim3(blocks, bottom ? 2 : 1), dim3(256), 0, s, a, 0, Y, m - 1,
                           Y + 2 * panel, -1, -1);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    sa.pan_stride = row;
    sa.back = 0;
    for (int p = 0; p < kt; ++p) {
        const int rows[2] = {p, m - 1 - p > kt ? m - 1 - p : -1};
        const int next[2] = {p + 1 < kt ? p + 1 : -1, m - 2 - p > kt ? m - 2 - p : -1};
        for (int c = 0; c < 2; ++c)
            sa.job[c] = StepJob<T>{rows[c], next[c], Y + (2 * c + (p & 1)) * panel, Y + (2 * c + ((p + 1) & 1)) * panel};
        if ((e = launch_step<T, NT, S>(sa, s)) != hipSuccess) return e;
    }
    hipLaunchKernelGGL(step_form_kernel<T>, dim3(blocks), dim3(256), 0, s, a, kt, Y, 0, (T*)nullptr,
                       kt > 0 ? kt - 1 : -1, bottom ? kt + 1 : -1);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    sa.job[0] = StepJob<T>{kt, -1, Y, nullptr};
    sa.job[1] = StepJob<T>{};
    if ((e = launch_step<T, NT, S>(sa, s)) != hipSuccess) return e;
    sa.pan_stride = m * row;
    sa.back = 1;
    for (int p = 1; p <= kt; ++p) {
        // without node voltages only the rows below the twist (the currents' row is the last)
        sa.job[0] = up ? StepJob<T>{kt - p, -1, Z + (kt - p + 1) * row, nullptr} : StepJob<T>{};
        sa.job[1] = kt + p < m ? StepJob<T>{kt + p, -1, Z + (kt + p - 1) * row, nullptr} : StepJob<T>{};
        if (sa.job[0].row < 0 && sa.job[1].row < 0) break;
        if ((e = launch_step<T, NT, S>(sa, s)) != hipSuccess) return e;
    }
    return hipSuccess;
}

// A workgroup per chain pays where a step is bound by its loads and the chains are longer
// than a launch: microseconds a batch with node voltages, chain per workgroup / both in
// one: 64 x 64 83 / 127, with 2048 vectors 126 / 170; 300 x 48 232 / 327; 3 x 40 25 / 24.
// At 32 columns the chains gain 0.04 us a step (700 rows 385 / 413, 64 rows 56 / 56, 89 / 85
// with 2048 vectors; 3 rows 24 / 22), and keep one workgroup.
constexpr int kSplitRows = 8;

template <int LT, bool UP>
hipError_t run_small_up(const SweepArgs& a, hipStream_t s)
{
    if (LT > 2 && a.m >= kSplitRows) {
        hipLaunchKernelGGL((sweep_small_kernel<LT, UP, kForward>), dim3(a.nslab, 2), dim3(64 * LT), 0, s, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((sweep_small_kernel<LT, UP, kTwistBack>), dim3(a.nslab, UP ? 2 : 1), dim3(64 * LT), 0, s, a);
    } else {
        hipLaunchKernelGGL((sweep_small_kernel<LT, UP, kBoth>), dim3(a.nslab), dim3(128 * LT), 0, s, a);
    }
    return hipGetLastError();
}

template <int LT>
hipError_t launch_small(const SweepArgs& a, hipStream_t s)
{
    return a.node_v ? run_small_up<LT, true>(a, s) : run_small_up<LT, false>(a, s);
}

// One slab a wave up to a wave per SIMD, two (on each H tile it loads) past that: with
// 1024 vectors at n = 512 27.8 against 32.4 us a step, with 16 vectors 10.7 against 8.0.
// (Four slabs a wave, or four row tiles a workgroup to share panels in its L1, were
// slower or equal everywhere.)
template <int NT>
hipError_t run_steps_nt(const SweepArgs& a, hipStream_t s)
{
    const int waves = 2 * (4 * NT) * a.nslab;
    const hipError_t e = waves <= 1024 ? run_steps<double, NT, 1>(a, s) : run_steps<double, NT, 2>(a, s);
    if (e != hipSuccess || !a.node_v) return e;
    return launch_recover_rows<NT>(a, s);
}

// (float32 products are half as long: one slab a wave up to four waves per SIMD, 18.3
// against 21.0 us a step with 512 vectors at n = 512, 26.6 against 25.9 with 1024)
template <int NT>
hipError_t run_ir_steps_nt(const SweepArgs& a, hipStream_t s)
{
    const int waves = 2 * (4 * NT) * a.nslab;
    const hipError_t e = waves < 4096 ? run_steps<float, NT, 1>(a, s) : run_steps<float, NT, 2>(a, s);
    if (e != hipSuccess || a.tol < 0.0) return e;
    hipLaunchKernelGGL(step_decide_kernel, dim3((a.nslab + 3) / 4), dim3(64), 0, s, a);
    return hipGetLastError();
}

}  // namespace

}  // namespace xbk

int xbk_step_slabs(int n_p, bool fp32)
{
    return n_p <= 128 ? 0 : fp32 ? xbk::kPartSlabs : xbk::kStepSlabs;
}

// A refinement queues every sweep that it may need.  One that finds its slabs finished is
// one launch in the slab sweep, but m + 3 by steps, 1.8 to 3.5 us each; so by steps go the
// sweeps expected, and past them as many as those gain, six at most (a float32 factor takes
// 3 to 5 to the default tolerance, 2 to a loose one).  A sweep's microseconds per row, slab
// sweep (and 0.023 a slab) against steps (and `per` a slab), measured at 256 and 512 rows
// with 1, 32 and 128 slabs; 3 rows of 192 columns, 16 vectors to 1e-3: 122 us by slab sweeps,
// 182 with six by steps, 136 with three.
int xbk_step_sweeps(int m, int n_p, int nslab, int expected)
{
    constexpr int most = 6;
    static constexpr double slab[] = {10.4, 13.2, 20.4, 25.0, 35.0, 41.0};     // n_p = 192 .. 512
    static constexpr double step[] = {4.3, 5.3, 6.2, 7.0, 7.8, 9.0};
    static constexpr double per[] = {0.063, 0.073, 0.1, 0.131, 0.181, 0.2};
    const int k = n_p / 64 - 3;
    if (k < 0 || k > 5) return 0;
    const double gain = m * (slab[k] + 0.023 * nslab - step[k] - per[k] * nslab), idle = 3.5 * (m + 3);
    return std::min(most, expected + (gain > 0.0 ? (int)(expected * gain / idle) : 0));
}

hipError_t xbk_launch_sweep_plan(const xbk::SweepArgs& a, hipStream_t s)
{
    if (a.batch > 1 || a.unit) return hipErrorInvalidValue;
    // one or two rows have no chains to run side by side
    if (a.m < 3 || (int64_t)a.m * a.nslab > INT32_MAX) return xbk_launch_sweep(a, s);
    if (a.n_p == 64) {
        hipError_t e = hipErrorInvalidValue;
        switch ((a.n + 15) / 16) {
            case 1: e = xbk::launch_small<1>(a, s); break;
            case 2: e = xbk::launch_small<2>(a, s); break;
            case 3: e = xbk::launch_small<3>(a, s); break;
            case 4: e = xbk::launch_small<4>(a, s); break;
        }
        if (e != hipSuccess || !a.node_v) return e;
        return xbk::launch_recover_rows<1>(a, s);
    }
    if (a.nslab > xbk::kPartSlabs) return xbk_launch_sweep(a, s);
    if (a.ysteps == nullptr || a.nslab > xbk_step_slabs(a.n_p, false)) return xbk_launch_sweep_parts(a, s);
    switch (a.n_p / 64) {
        case 3: return xbk::run_steps_nt<3>(a, s);
        case 4: return xbk::run_steps_nt<4>(a, s);
        case 5: return xbk::run_steps_nt<5>(a, s);
        case 6: return xbk::run_steps_nt<6>(a, s);
        case 7: return xbk::run_steps_nt<7>(a, s);
        case 8: return xbk::run_steps_nt<8>(a, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t xbk_launch_sweep_ir_plan(const xbk::SweepArgs& a, int step_sweeps, hipStream_t s)
{
    if (a.m < 3 || a.ysteps == nullptr || a.nslab > xbk_step_slabs(a.n_p, true) || a.iter >= step_sweeps)
        return xbk_launch_sweep_ir(a, s);
    switch (a.n_p / 64) {
        case 3: return xbk::run_ir_steps_nt<3>(a, s);
        case 4: return xbk::run_ir_steps_nt<4>(a, s);
        case 5: return xbk::run_ir_steps_nt<5>(a, s);
        case 6: return xbk::run_ir_steps_nt<6>(a, s);
        case 7: return xbk::run_ir_steps_nt<7>(a, s);
        case 8: return xbk::run_ir_steps_nt<8>(a, s);
        default: return hipErrorInvalidValue;
    }
}
