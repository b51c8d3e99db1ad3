// Block-sparse convolution, channels-first fp32 (the small-channel path).
//
// A workgroup computes one active output block for a tile of CT output channels (a
// multiple of four). For each chunk of input channels it stages the block's halo tile
// [ci][(bh-1)*s + kh][(bw-1)*s + kw] (zeros outside the image) and the weights, as
// [ci][tap][CT], in LDS; all of a thread's loads are requested before the first is
// stored. The block's pixels are taken in groups of 64, one pixel per lane, and a wave
// accumulates four output channels of a group (an item), so that one LDS read of the
// input serves four FMAs and the four weights are one 16-byte read at an address that
// the whole wave shares. Every sum runs in the fixed order ci -> i -> j with fp32 FMAs.
// The epilogue adds bias and residual in fp32, applies ReLU and writes straight to the
// block's position of the persistent output; elements outside active blocks are never
// touched.
//
// What bounds it: latency (a small layer is the index's round trip, one of loads, 16 x 9
// taps of two LDS reads and four FMAs per lane, one of stores). 3x3 16 -> 16 on 64x128
// with 32 active 8x8 blocks: 36.3 -> 10.2 us (before: up to eight scattered outputs per
// thread, two LDS reads per FMA, divisions by run-time sizes in every loop).
#include "bc_internal.h"

namespace bc {
namespace {

constexpr int kThreads = 256;
constexpr int kMaxPerThread = 8;             // outputs a workgroup's thread held in the limits below
constexpr int kLdsBudget = 48 * 1024;
constexpr int kCo = 4;                       // output channels per item

// n / d for a per-launch constant d: umulhi(n, ceil(2^32 / d)), exact while n * d < 2^32
// (LDS indices: n < 2^16, d < 2^15); d = 1 is stored as 0.
struct Div {
    uint32_t m;
    int d;
};

__device__ __forceinline__ int fdiv(int n, Div f) { return f.m ? (int)__umulhi((uint32_t)n, f.m) : n; }

Div make_div(int d)
{
    return Div{d == 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + (uint64_t)d - 1) / (uint64_t)d), d};
}

struct F32Args {
    const float *x, *w, *bias, *res;
    float *y;
    LayerGeom g;
    int th, tw, ct, ci_t, n_co_tiles, npg;   // halo tile, channel tile and chunk, pixel groups
    int relu;
    Div f_tile, f_tw, f_bw, f_row;           // th * tw, tw, bw, ci_t * taps
};

// KS > 0: a KS x KS kernel known at compile time; KS = 0: any kernel. NI items per wave.
template <int KS, int NI>
__global__ __launch_bounds__(kThreads) void k_conv_nchw_f32(F32Args a)
{
    extern __shared__ __align__(16) float lds[];
    const LayerGeom &g = a.g;
    const int k = blockIdx.x / a.n_co_tiles;
    const int cot = blockIdx.x - k * a.n_co_tiles;
    // the block id with the active count, one round trip (k < total_blocks: a valid read)
    const int bid = g.idx ? g.idx[k] : k;
    const int cnt = g.count ? *g.count : g.total_blocks;
    if (k >= cnt) return;
    const int img = bid / (g.gh * g.gw);
    const int rem = bid - img * g.gh * g.gw;
    const int gy = rem / g.gw, gx = rem - (rem / g.gw) * g.gw;
    const int npx = g.bh * g.bw;
    const int co0 = cot * a.ct;
    const int kh = KS ? KS : g.kh, kw = KS ? KS : g.kw;
    const int taps = kh * kw;
    const int y0 = gy * g.bh * g.stride - g.pad, x0 = gx * g.bw * g.stride - g.pad;
    const int tile = a.th * a.tw;
    float *ws = lds;                                     // [ci_t][taps][ct]
    float *xs = lds + (size_t)a.ci_t * taps * a.ct;      // [ci_t][th][tw]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

    int base[NI], cg[NI];                                // input offset and channel group per item
    bool live[NI];
#pragma unroll
    for (int u = 0; u < NI; ++u) {
        const int item = wave + 4 * u;
        cg[u] = item / a.npg;
        const int p = (item - cg[u] * a.npg) * 64 + lane;
        live[u] = cg[u] * kCo < a.ct && p < npx;
        const int pc = min(p, npx - 1);
        const int py = fdiv(pc, a.f_bw), px = pc - py * g.bw;
        base[u] = py * g.stride * a.tw + px * g.stride;
        cg[u] = min(cg[u], a.ct / kCo - 1);
    }
    float acc[NI][kCo];
#pragma unroll
    for (int u = 0; u < NI; ++u)
#pragma unroll
        for (int c = 0; c < kCo; ++c) acc[u][c] = 0.f;

    for (int c0 = 0; c0 < g.cin; c0 += a.ci_t) {
        const int cn = min(a.ci_t, g.cin - c0);
        const int nx = cn * tile, row = cn * taps;
        constexpr int B = 10;                            // loads in flight per thread and round
        auto load_x = [&](int e) {
            const int ci = fdiv(e, a.f_tile);
            const int r = e - ci * tile;
            const int ty = fdiv(r, a.f_tw), tx = r - ty * a.tw;
            const int iy = y0 + ty, ix = x0 + tx;
            const bool in = e < nx && iy >= 0 && iy < g.hin && ix >= 0 && ix < g.win;
            const size_t o = in ? (((size_t)img * g.cin + c0 + ci) * g.hin + iy) * (size_t)g.win + ix : 0;
            const float v = a.x[o];                      // a valid address either way
            return in ? v : 0.f;
        };
        // rows of ci_t * taps values (the last chunk uses the first `row` of each)
        auto load_w = [&](int e, int &dst) {
            const int co = fdiv(e, a.f_row);
            const int r = e - co * a.f_row.d;
            const bool in = e < a.ct * a.f_row.d && r < row && co0 + co < g.cout;
            dst = e < a.ct * a.f_row.d && r < row ? r * a.ct + co : -1;
            const float v = a.w[in ? ((size_t)(co0 + co) * g.cin + c0) * taps + r : 0];
            return in ? v : 0.f;
        };
        if (c0) __syncthreads();                         // the previous chunk is done with
        float vx[B], vw[B];
        int dw[B];
        for (int e0 = 0; e0 < max(nx, a.ct * a.f_row.d); e0 += B * kThreads) {
#pragma unroll
            for (int u = 0; u < B; ++u) vx[u] = load_x(e0 + u * kThreads + tid);
#pragma unroll
            for (int u = 0; u < B; ++u) vw[u] = load_w(e0 + u * kThreads + tid, dw[u]);
#pragma unroll
            for (int u = 0; u < B; ++u)
                if (e0 + u * kThreads + tid < nx) xs[e0 + u * kThreads + tid] = vx[u];
#pragma unroll
            for (int u = 0; u < B; ++u)
                if (dw[u] >= 0) ws[dw[u]] = vw[u];
        }
        __syncthreads();
        for (int ci = 0; ci < cn; ++ci) {
            const float *xc = xs + ci * tile;
            const float *wc = ws + ci * taps * a.ct;
            if constexpr (KS > 0) {
#pragma unroll
                for (int t = 0; t < KS * KS; ++t) {
#pragma unroll
                    for (int u = 0; u < NI; ++u) {
                        const float v = xc[base[u] + (t / KS) * a.tw + t % KS];
                        const float4 w = *(const float4 *)(wc + t * a.ct + cg[u] * kCo);
                        acc[u][0] = fmaf(w.x, v, acc[u][0]);
                        acc[u][1] = fmaf(w.y, v, acc[u][1]);
                        acc[u][2] = fmaf(w.z, v, acc[u][2]);
                        acc[u][3] = fmaf(w.w, v, acc[u][3]);
                    }
                }
            } else {
                for (int i = 0; i < kh; ++i)
                    for (int j = 0; j < kw; ++j)
#pragma unroll
                        for (int u = 0; u < NI; ++u) {
                            const float v = xc[base[u] + i * a.tw + j];
                            const float4 w = *(const float4 *)(wc + (i * kw + j) * a.ct + cg[u] * kCo);
                            acc[u][0] = fmaf(w.x, v, acc[u][0]);
                            acc[u][1] = fmaf(w.y, v, acc[u][1]);
                            acc[u][2] = fmaf(w.z, v, acc[u][2]);
                            acc[u][3] = fmaf(w.w, v, acc[u][3]);
                        }
            }
        }
    }
#pragma unroll
    for (int u = 0; u < NI; ++u) {
        if (!live[u]) continue;
        const int item = wave + 4 * u;
        const int p = (item - cg[u] * a.npg) * 64 + lane;
        const int py = fdiv(p, a.f_bw), px = p - py * g.bw;
#pragma unroll
        for (int c = 0; c < kCo; ++c) {
            const int co = co0 + cg[u] * kCo + c;
            if (co >= g.cout) continue;
            const size_t o = (((size_t)img * g.cout + co) * g.hout + gy * g.bh + py) * g.wout + gx * g.bw + px;
            float z = acc[u][c];
            if (a.bias) z += a.bias[co];
            if (a.res) z += a.res[o];
            if (a.relu) z = (z > 0.f || z != z) ? z : 0.f;
            a.y[o] = z;
        }
    }
}

template <int KS>
hipError_t launch_items(const F32Args &a, int ni, dim3 grid, size_t lds, hipStream_t s)
{
    auto go = [&](auto kern) {
        if (lds > 60 * 1024) {
            const hipError_t e = hipFuncSetAttribute((const void *)kern,
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kern, grid, dim3(kThreads), lds, s, a);
        return hipGetLastError();
    };
    if (ni <= 1) return go(k_conv_nchw_f32<KS, 1>);
    if (ni <= 2) return go(k_conv_nchw_f32<KS, 2>);
    if (ni <= 4) return go(k_conv_nchw_f32<KS, 4>);
    return go(k_conv_nchw_f32<KS, 8>);
}

}  // namespace

hipError_t launch_conv_nchw_f32(const float *x, const float *w, const float *bias,
                                const float *res, float *y, int relu, const LayerGeom &g,
                                hipStream_t s, const char **why)
{
    F32Args a;
    a.x = x; a.w = w; a.bias = bias; a.res = res; a.y = y; a.g = g; a.relu = relu;
    a.th = (g.bh - 1) * g.stride + g.kh;
    a.tw = (g.bw - 1) * g.stride + g.kw;
    const int npx = g.bh * g.bw, taps = g.kh * g.kw;
    // the accepted sizes: 2048 pixels per block, and one input channel with the weights of
    // as many output channels as 2048 outputs hold in 48 KB
    const int co_t = g.cout < (kThreads * kMaxPerThread) / npx ? g.cout : (kThreads * kMaxPerThread) / npx;
    if (co_t < 1) {
        *why = "fp32 path: output block larger than 2048 pixels";
        return hipErrorInvalidValue;
    }
    if ((a.th * a.tw + co_t * taps) * (int)sizeof(float) > kLdsBudget) {
        *why = "fp32 path: one channel of the halo tile does not fit in LDS";
        return hipErrorInvalidValue;
    }
    // one item per wave where that covers the block's pixel groups (16 output channels at
    // most, then more workgroups share a block): a small layer is latency, so its work is
    // spread over as many waves as there are. Up to 8 items per wave (2048 pixels).
    a.npg = (npx + 63) / 64;
    const int fit = a.npg >= 4 ? 1 : 4 / a.npg;          // channel groups of one item per wave
    const int groups = (g.cout + kCo - 1) / kCo;
    a.ct = kCo * (groups < fit ? groups : fit);
    const int ni = (a.npg * (a.ct / kCo) + 3) / 4;
    const int per_ci = (a.th * a.tw + a.ct * taps) * (int)sizeof(float);
    a.ci_t = kLdsBudget / per_ci;
    if (a.ci_t < 1) a.ci_t = 1;                          // four channels of a very large kernel
    if (a.ci_t > g.cin) a.ci_t = g.cin;
    a.n_co_tiles = (g.cout + a.ct - 1) / a.ct;
    a.f_tile = make_div(a.th * a.tw);
    a.f_tw = make_div(a.tw);
    a.f_bw = make_div(g.bw);
    a.f_row = make_div(a.ci_t * taps);
    const size_t lds = (size_t)a.ci_t * per_ci;
    const dim3 grid((unsigned)g.total_blocks * a.n_co_tiles);
    if (g.kh == 3 && g.kw == 3) return launch_items<3>(a, ni, grid, lds, s);
    if (g.kh == 1 && g.kw == 1) return launch_items<1>(a, ni, grid, lds, s);
    return launch_items<0>(a, ni, grid, lds, s);
}

}  // namespace bc
