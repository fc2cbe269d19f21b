// Inference of the learned surrogate in one pass over the maps: all layers of the
// bfloat16 network on a tile of crosspoints, from the features to the column readouts,
// with the activations between the layers kept in LDS.
//
// The layer-by-layer path writes and reads every activation map in float32 (128 x 128,
// 32 channels: 2 MiB a sample and layer), which is what bounds it.  A layer's activations
// are rounded to bfloat16 when the next layer reads them, so here they are rounded when
// they are produced and held as bfloat16 in LDS only; products, their order and the
// float32 accumulation are those of sg_conv_mfma_kernel, so the last map has the same bits.
//
//  * infer_prep_kernel: per sample the line totals, the ideal currents and the rounded
//    log-conductance plane; infer_pack_kernel: the weights as matrix-core fragments.
//  * infer_tile_kernel<CP, L, TH>: a TH x 32 tile of one sample per workgroup of eight
//    waves.  Layer k computes the tile widened by L - k crosspoints on every side (zero
//    outside the map, as the convolutions pad), positions in strips of 16 in row order; a
//    wave takes every eighth strip, the weights come as fragments from L1, and the two
//    LDS buffers alternate ([position][channel], 16-byte reads of eight channels of a
//    tap).  The weights are the A operand, so that a lane ends with four consecutive
//    channels of one position.  The last layer's two channels are summed over the tile's
//    rows.
//  * infer_readout_kernel: the tiles' sums to currents and error estimates.
//
// Tile choice: the widened tiles cost (per output crosspoint, L = 4) 1.52 times the
// layers' products at 8 x 32 and 1.32 at 16 x 32; 8 x 32 keeps two workgroups on a CU.
// Bound: the LDS reads of the position fragments (1 KB per strip and 32-deep step, at
// 128 bytes a cycle) about level with the matrix cores.  Measured, 256 samples of 128 x 128,
// 32 channels, 4 layers: 407 us a call (prep 27, readout 7, pack 5), 1071 us layer by layer;
// 16 x 32 tiles and 4 or 16 waves measured within 10% of this.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "surrogate_infer.h"

typedef __bf16 ib8_t __attribute__((ext_vector_type(8)));
typedef __bf16 ib4_t __attribute__((ext_vector_type(4)));
typedef float if4_t __attribute__((ext_vector_type(4)));

namespace {

constexpr int kIW = 32;                    // tile columns
constexpr int kIWaves = 8;
constexpr int kIMaxDepth = 5;
constexpr int kIParts = 8;                 // workgroups of a sample's preparation

struct InferArgs {
    int B, m, n, C, L;
    const double* G;
    const double* V;
    const double* r;
    const float* params;
    // workspace
    __bf16* logg;        // [B][m][n]
    float* rowt;         // [B][m] row totals
    float* colt;         // [B][n] column totals
    double* ideal;       // [B][n] G^T V
    __bf16* pack;        // fragments of every layer
    double* part;        // [B][tile rows][2][n]
    double* I;
    double* est;
};

__host__ __device__ inline int steps_of(int cin)      // matrix-core steps of a layer
{
    return (9 * ((cin + 7) / 8) + 3) / 4;
}
__host__ __device__ inline int nt_of(int cout) { return cout > 16 ? 2 : 1; }
// fragments (of 512 bfloat16) before layer k (0-based)
__host__ __device__ inline int frags_before(int k, int C, int L)
{
    int f = 0;
    for (int i = 0; i < k; ++i) f += steps_of(i == 0 ? XBAR_SG_FEATURES : C) * nt_of(i == L - 1 ? 2 : C);
    return f;
}
// floats of parameters before layer k
__host__ __device__ inline int params_before(int k, int C, int L)
{
    int f = 0;
    for (int i = 0; i < k; ++i) {
        const int ci = i == 0 ? XBAR_SG_FEATURES : C, co = i == L - 1 ? 2 : C;
        f += co * ci * 9 + co;
    }
    return f;
}

// A float32 feature as the convolutions stage it.  The value passes through a float32
// register on purpose: folded into one conversion, float64 to bfloat16 would round once
// instead of twice.
__device__ __forceinline__ __bf16 staged(float x)
{
    asm volatile("" : "+v"(x));
    return (__bf16)x;
}

__device__ __forceinline__ double wave_total(double x)
{
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
    return x;
}

// The sums, their order and the roundings of sg_features_kernel and sg_predict_kernel.
__global__ __launch_bounds__(256) void infer_prep_kernel(InferArgs a)
{
    __shared__ double part[2][4][64];
    const int m = a.m, n = a.n, b = blockIdx.x, l = threadIdx.x & 63, w = threadIdx.x >> 6;
    const double* gb = a.G + (int64_t)b * m * n;
    const double* vb = a.V + (int64_t)b * m;
    const int per = (m + (int)gridDim.y - 1) / (int)gridDim.y;
    const int i0 = blockIdx.y * per, i1 = min(m, i0 + per);
    __bf16* lg = a.logg + (int64_t)b * m * n;
    for (int i = i0 + w; i < i1; i += 4) {
        double s = 0.0;
        for (int j = l; j < n; j += 64) {
            const double g = gb[(int64_t)i * n + j];
            s += g;
            lg[(int64_t)i * n + j] = staged((float)(log10(g) + 5.0));
        }
        s = wave_total(s);
        if (l == 0) a.rowt[(int64_t)b * m + i] = (float)(1e4 * s / n);
    }
    // the columns, 64 at a time, shared among the sample's workgroups
    constexpr int R = 8;
    for (int j0 = 64 * blockIdx.y; j0 < n; j0 += 64 * gridDim.y) {
        const int j = min(j0 + l, n - 1);
        double s = 0.0, i00 = 0.0;
        for (int i = w; i < m; i += 4 * R) {
            double g[R], v[R];
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const int ii = min(i + 4 * k, m - 1);
                g[k] = gb[(int64_t)ii * n + j];
                v[k] = vb[ii];
            }
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const bool ok = i + 4 * k < m;
                s += ok ? g[k] * 2.0 * v[k] : 0.0;
                i00 += ok ? g[k] * v[k] : 0.0;
            }
        }
        part[0][w][l] = s;
        part[1][w][l] = i00;
        __syncthreads();
        if (w == 0 && j0 + l < n) {
            a.colt[(int64_t)b * n + j] =
                (float)(1e4 * (((part[0][0][l] + part[0][1][l]) + part[0][2][l]) + part[0][3][l]) / m);
            a.ideal[(int64_t)b * n + j] = ((part[1][0][l] + part[1][1][l]) + part[1][2][l]) + part[1][3][l];
        }
        __syncthreads();
    }
}

// Layer blockIdx.y's weights as A fragments: [step][output tile][lane][8], lane l holding
// output channel 16 nt + l % 16 and the eight input channels of pair 4 s + l / 16.
__global__ __launch_bounds__(64) void infer_pack_kernel(InferArgs a)
{
    const int k = blockIdx.y, ci = k == 0 ? XBAR_SG_FEATURES : a.C, co = k == a.L - 1 ? 2 : a.C;
    const int S = steps_of(ci), NT = nt_of(co), nch = (ci + 7) / 8;
    if ((int)blockIdx.x >= S * NT) return;
    const int s = blockIdx.x / NT, nt = blockIdx.x % NT, l = threadIdx.x;
    const int oc = 16 * nt + (l & 15), j = 4 * s + (l >> 4), t = j / nch, cc = j % nch;
    const float* w = a.params + params_before(k, a.C, a.L);
    ib8_t f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int ic = 8 * cc + i;
        const bool ok = j < 9 * nch && oc < co && ic < ci;
        f[i] = (__bf16)(ok ? w[((int64_t)oc * ci + ic) * 9 + t] : 0.0f);
    }
    *reinterpret_cast<ib8_t*>(a.pack + ((int64_t)(frags_before(k, a.C, a.L) + blockIdx.x) * 64 + l) * 8) = f;
}

// One layer on a widened tile: input region IH x IW positions of PSI elements (CI channels
// used), output (IH - 2) x (IW - 2) positions.  emit(pos, row, col, nt, values) receives four
// consecutive output channels (16 nt + 4 (lane / 16) ..) of one position.
template <int CI, int PSI, int NT, int IH, int IW, typename Emit>
__device__ __forceinline__ void infer_layer(const __bf16* __restrict__ in, const __bf16* __restrict__ pack, int wv,
                                            int l, const Emit& emit)
{
    constexpr int OW = IW - 2, POS = (IH - 2) * OW, STRIPS = (POS + 15) / 16;
    constexpr int MS = (STRIPS + kIWaves - 1) / kIWaves;
    constexpr int NCH = CI / 8, P = 9 * NCH, S = (P + 3) / 4;
    const int g = l >> 4, c16 = l & 15;
    int base[MS];
#pragma unroll
    for (int st = 0; st < MS; ++st) {
        const int pos = min(16 * (wv + kIWaves * st) + c16, POS - 1);
        base[st] = ((pos / OW) * IW + pos % OW) * PSI;
    }
    if4_t acc[MS][NT];
#pragma unroll
    for (int st = 0; st < MS; ++st)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[st][nt] = if4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const int j = 4 * s + g, jj = j < P ? j : P - 1;
        const int t = jj / NCH, cc = jj % NCH;
        const int off = ((t / 3) * IW + t % 3) * PSI + 8 * cc;
        ib8_t wf[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            wf[nt] = *reinterpret_cast<const ib8_t*>(pack + ((s * NT + nt) * 64 + l) * 8);
#pragma unroll
        for (int st = 0; st < MS; ++st) {
            ib8_t x = *reinterpret_cast<const ib8_t*>(in + base[st] + off);
            if constexpr (P % 4 != 0) {
                if (s == S - 1 && j >= P)
#pragma unroll
                    for (int i = 0; i < 8; ++i) x[i] = (__bf16)0.0f;
            }
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                acc[st][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[nt], x, acc[st][nt], 0, 0, 0);
        }
    }
#pragma unroll
    for (int st = 0; st < MS; ++st) {
        const int pos = 16 * (wv + kIWaves * st) + c16;
        if (pos >= POS) continue;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) emit(pos, pos / OW, pos % OW, nt, acc[st][nt]);
    }
}

// CP = hidden channels rounded up to 8.
template <int CP, int L, int TH>
struct InferTile {
    static constexpr int PS = CP + 8;                              // padded: conflict-free 16-byte reads
    static constexpr int NT = CP > 16 ? 2 : 1;
    static constexpr int rows(int k) { return TH + 2 * (L - k); }  // region of layer k's output (0: features)
    static constexpr int cols(int k) { return kIW + 2 * (L - k); }
    static constexpr int pos(int k) { return rows(k) * cols(k); }
    static constexpr int size_a() { return pos(1) * PS; }          // outputs of odd layers
    static constexpr int size_b() { return L > 2 && pos(2) * PS > pos(0) * 8 ? pos(2) * PS : pos(0) * 8; }
    static constexpr size_t bytes() { return sizeof(__bf16) * (size_t)(size_a() + size_b()); }
};

// Hidden layers K .. L - 1 (K >= 2): input in `in`, output to `out`, then swapped.
template <int CP, int L, int TH, int K, typename Hidden>
__device__ __forceinline__ const __bf16* infer_hidden(__bf16* in, __bf16* out, const Hidden& layer)
{
    if constexpr (K < L) {
        layer(std::integral_constant<int, K>{}, in, out);
        __syncthreads();
        return infer_hidden<CP, L, TH, K + 1>(out, in, layer);
    } else {
        return in;
    }
}

template <int CP, int L, int TH>
__global__ __launch_bounds__(64 * kIWaves) void infer_tile_kernel(InferArgs a)
{
    using Tl = InferTile<CP, L, TH>;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ float last[2][TH][kIW];
    __bf16* const bufa = reinterpret_cast<__bf16*>(smem);
    __bf16* const bufb = bufa + Tl::size_a();
    const int m = a.m, n = a.n, l = threadIdx.x & 63, wv = threadIdx.x >> 6, g = l >> 4;
    const int th = (m + TH - 1) / TH, tw = (n + kIW - 1) / kIW;
    const int b = blockIdx.x / (th * tw), rest = blockIdx.x % (th * tw);
    const int p0 = (rest / tw) * TH, q0 = (rest % tw) * kIW;
    // features of the widened tile, eight channels (the last zero) a position
    {
        constexpr int W0 = Tl::cols(0), N0 = Tl::pos(0), IT = (N0 + 64 * kIWaves - 1) / (64 * kIWaves);
        const __bf16* lg = a.logg + (int64_t)b * m * n;
        const float rr = (float)((a.r[b] - 3.0) * 0.5);
        __bf16 lv[IT];
        float vv[IT], rv[IT], cv[IT];
#pragma unroll
        for (int k = 0; k < IT; ++k) {
            const int e = min((int)threadIdx.x + k * 64 * kIWaves, N0 - 1);
            const int i = min(max(p0 - L + e / W0, 0), m - 1), j = min(max(q0 - L + e % W0, 0), n - 1);
            lv[k] = lg[(int64_t)i * n + j];
            vv[k] = (float)(2.0 * a.V[(int64_t)b * m + i]);
            rv[k] = a.rowt[(int64_t)b * m + i];
            cv[k] = a.colt[(int64_t)b * n + j];
        }
#pragma unroll
        for (int k = 0; k < IT; ++k) {
            const int e = threadIdx.x + k * 64 * kIWaves;
            if (e >= N0) break;
            const int i = p0 - L + e / W0, j = q0 - L + e % W0;
            ib8_t f;
#pragma unroll
            for (int c = 0; c < 8; ++c) f[c] = (__bf16)0.0f;
            if (i >= 0 && i < m && j >= 0 && j < n) {
                f[0] = lv[k];
                f[1] = staged(vv[k]);
                f[2] = staged(rr);
                f[3] = staged(n > 1 ? (float)(2.0 * j / (n - 1) - 1.0) : 0.0f);
                f[4] = staged(m > 1 ? (float)(2.0 * i / (m - 1) - 1.0) : 0.0f);
                f[5] = staged(rv[k]);
                f[6] = staged(cv[k]);
            }
            *reinterpret_cast<ib8_t*>(bufb + e * 8) = f;
        }
    }
    __syncthreads();
    // layer k (1-based): bias, ReLU, zero outside the map, rounded for the next layer
    auto hidden = [&](auto kk, const __bf16* in, __bf16* out) {
        constexpr int K = decltype(kk)::value;
        const float* bias = a.params + params_before(K - 1, a.C, L) + a.C * (K == 1 ? XBAR_SG_FEATURES : a.C) * 9;
        const __bf16* pack = a.pack + (int64_t)frags_before(K - 1, a.C, L) * 512;
        if4_t bo[Tl::NT];
#pragma unroll
        for (int nt = 0; nt < Tl::NT; ++nt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int oc = 16 * nt + 4 * g + v;
                const float x = bias[oc < a.C ? oc : 0];
                bo[nt][v] = oc < a.C ? x : 0.0f;
            }
        auto emit = [&](int pos, int pr, int pc, int nt, if4_t y) {
            if (16 * nt + 4 * g >= CP) return;
            const int i = p0 - (L - K) + pr, j = q0 - (L - K) + pc;
            const bool ok = i >= 0 && i < m && j >= 0 && j < n;
            ib4_t o;
#pragma unroll
            for (int v = 0; v < 4; ++v) o[v] = (__bf16)(ok ? fmaxf(y[v] + bo[nt][v], 0.0f) : 0.0f);
            *reinterpret_cast<ib4_t*>(out + pos * Tl::PS + 16 * nt + 4 * g) = o;
        };
        if constexpr (K == 1)
            infer_layer<8, 8, Tl::NT, Tl::rows(0), Tl::cols(0)>(in, pack, wv, l, emit);
        else
            infer_layer<CP, Tl::PS, Tl::NT, Tl::rows(K - 1), Tl::cols(K - 1)>(in, pack, wv, l, emit);
    };
    hidden(std::integral_constant<int, 1>{}, bufb, bufa);
    __syncthreads();
    const __bf16* lin = infer_hidden<CP, L, TH, 2>(bufa, bufb, hidden);
    {
        const float* bias = a.params + params_before(L - 1, a.C, L) + 2 * a.C * 9;
        const float b0 = bias[0], b1 = bias[1];
        auto emit = [&](int, int pr, int pc, int, if4_t y) {
            if (g != 0) return;
            const bool ok = p0 + pr < m;
            last[0][pr][pc] = ok ? y[0] + b0 : 0.0f;
            last[1][pr][pc] = ok ? y[1] + b1 : 0.0f;
        };
        infer_layer<CP, Tl::PS, 1, Tl::rows(L - 1), Tl::cols(L - 1)>(
            lin, a.pack + (int64_t)frags_before(L - 1, a.C, L) * 512, wv, l, emit);
    }
    __syncthreads();
    if (threadIdx.x < 2 * kIW) {
        const int c = threadIdx.x / kIW, j = threadIdx.x % kIW;
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < TH; ++i) s += last[c][i][j];
        if (q0 + j < n) a.part[(((int64_t)b * th + rest / tw) * 2 + c) * n + q0 + j] = s;
    }
}

__global__ __launch_bounds__(64) void infer_readout_kernel(InferArgs a, int th)
{
    const int j = blockIdx.x * 64 + threadIdx.x, b = blockIdx.y, n = a.n;
    if (j >= n) return;
    double s0 = 0.0, s1 = 0.0;
    for (int t = 0; t < th; ++t) {
        s0 += a.part[(((int64_t)b * th + t) * 2) * n + j];
        s1 += a.part[(((int64_t)b * th + t) * 2 + 1) * n + j];
    }
    a.I[(int64_t)b * n + j] = a.ideal[(int64_t)b * n + j] * (1.0 + s0 / a.m);
    if (a.est)
        a.est[(int64_t)b * n + j] =
            exp(0.5 * (XBAR_SG_EST_SIGMA * s1 / a.m + XBAR_SG_EST_MU)) / fabs(1.0 + s0 / a.m);
}

constexpr int kITH = 8;

int64_t align16(int64_t x) { return (x + 15) & ~(int64_t)15; }

// Byte offsets of the workspace's arrays; returns its size.
int64_t layout(int B, int m, int n, int C, int L, int64_t (&off)[6])
{
    const int th = (m + kITH - 1) / kITH;
    const int64_t size[6] = {(int64_t)B * m * n * 2,     (int64_t)B * m * 4, (int64_t)B * n * 4,
                             (int64_t)B * n * 8,         (int64_t)frags_before(L, C, L) * 1024,
                             (int64_t)B * th * 2 * n * 8};
    int64_t at = 0;
    for (int k = 0; k < 6; ++k) {
        off[k] = at;
        at += align16(size[k]);
    }
    return at;
}

template <int CP, int L>
hipError_t launch_tiles(const InferArgs& a, hipStream_t s)
{
    using Tl = InferTile<CP, L, kITH>;
    const int64_t tiles = (int64_t)a.B * ((a.m + kITH - 1) / kITH) * ((a.n + kIW - 1) / kIW);
    hipLaunchKernelGGL((infer_tile_kernel<CP, L, kITH>), dim3((unsigned)tiles), dim3(64 * kIWaves), Tl::bytes(), s, a);
    return hipGetLastError();
}

template <int CP>
hipError_t launch_depth(const InferArgs& a, hipStream_t s)
{
    switch (a.L) {
        case 2: return launch_tiles<CP, 2>(a, s);
        case 3: return launch_tiles<CP, 3>(a, s);
        case 4: return launch_tiles<CP, 4>(a, s);
        case 5: return launch_tiles<CP, 5>(a, s);
        default: return hipErrorInvalidValue;
    }
}

bool infer_shape_ok(int32_t B, int32_t m, int32_t n, int32_t C, int32_t L)
{
    if (B < 1 || B > 65535 || m < 1 || n < 1 || m > XBAR_SG_MAX_LINE || n > XBAR_SG_MAX_LINE || C < 1 ||
        C > XBAR_SG_MAX_CHANNELS || L < 2 || L > kIMaxDepth)
        return false;
    const int64_t tiles = (int64_t)B * ((m + kITH - 1) / kITH) * ((n + kIW - 1) / kIW);
    return tiles <= INT32_MAX;
}

bool meets(const void* a, int64_t na, const void* b, int64_t nb)
{
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return x < y + (uintptr_t)nb && y < x + (uintptr_t)na;
}

}  // namespace

extern "C" {

int64_t xbar_sg_infer_workspace_bytes(int32_t B, int32_t m, int32_t n, int32_t C, int32_t depth)
{
    int64_t off[6];
    return infer_shape_ok(B, m, n, C, depth) ? layout(B, m, n, C, depth, off) : -1;
}

xbar_status xbar_sg_infer_bf16(int32_t B, int32_t m, int32_t n, int32_t C, int32_t depth, const double* G,
                               const double* V, const double* r, const float* params, void* work,
                               int64_t work_bytes, double* I, double* est, void* stream)
{
    if (!infer_shape_ok(B, m, n, C, depth) || !G || !V || !r || !params || !work || !I) return XBAR_ERR_ARG;
    int64_t off[6];
    const int64_t need = layout(B, m, n, C, depth, off), ni = (int64_t)B * n * 8;
    if (work_bytes < need || (reinterpret_cast<uintptr_t>(work) & 15)) return XBAR_ERR_ARG;
    const void* ins[4] = {G, V, r, params};
    const int64_t sizes[4] = {(int64_t)B * m * n * 8, (int64_t)B * m * 8, (int64_t)B * 8,
                              (int64_t)params_before(depth, C, depth) * 4};
    for (int k = 0; k < 4; ++k)
        if (meets(work, need, ins[k], sizes[k])) return XBAR_ERR_ARG;
    // as xbar_sg_predict: I may not lie on G or V.  (Outputs on the other inputs are sound:
    // the last kernel alone writes them, and it reads the workspace only.)
    for (int k = 0; k < 2; ++k)
        if (meets(I, ni, ins[k], sizes[k])) return XBAR_ERR_ARG;
    if (meets(work, need, I, ni) || (est && (meets(work, need, est, ni) || meets(est, ni, I, ni)))) return XBAR_ERR_ARG;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    char* w = static_cast<char*>(work);
    InferArgs a{};
    a.B = B;
    a.m = m;
    a.n = n;
    a.C = C;
    a.L = depth;
    a.G = G;
    a.V = V;
    a.r = r;
    a.params = params;
    a.logg = reinterpret_cast<__bf16*>(w + off[0]);
    a.rowt = reinterpret_cast<float*>(w + off[1]);
    a.colt = reinterpret_cast<float*>(w + off[2]);
    a.ideal = reinterpret_cast<double*>(w + off[3]);
    a.pack = reinterpret_cast<__bf16*>(w + off[4]);
    a.part = reinterpret_cast<double*>(w + off[5]);
    a.I = I;
    a.est = est;
    const int parts = std::max(1, std::min(kIParts, 1024 / B));
    hipLaunchKernelGGL(infer_prep_kernel, dim3(B, parts), dim3(256), 0, s, a);
    if (hipGetLastError() != hipSuccess) return XBAR_ERR_DEVICE;
    const int frags = std::max(steps_of(C) * nt_of(C), steps_of(XBAR_SG_FEATURES) * nt_of(C));
    hipLaunchKernelGGL(infer_pack_kernel, dim3(frags, depth), dim3(64), 0, s, a);
    if (hipGetLastError() != hipSuccess) return XBAR_ERR_DEVICE;
    hipError_t e;
    switch ((C + 7) / 8) {
        case 1: e = launch_depth<8>(a, s); break;
        case 2: e = launch_depth<16>(a, s); break;
        case 3: e = launch_depth<24>(a, s); break;
        default: e = launch_depth<32>(a, s); break;
    }
    if (e != hipSuccess) return XBAR_ERR_DEVICE;
    hipLaunchKernelGGL(infer_readout_kernel, dim3((n + 63) / 64, B), dim3(64), 0, s, a, (m + kITH - 1) / kITH);
    return hipGetLastError() == hipSuccess ? XBAR_OK : XBAR_ERR_DEVICE;
}

}  // extern "C"
