// Block-sparse convolution, channels-first fp32 (the small-channel path).
//
// A workgroup computes one active output block, or 256 consecutive pixels of a larger one,
// for a tile of CT output channels (a multiple of four). For each chunk of input channels
// it stages the halo tile of the pixels' R rows [ci][(R-1)*s + kh][(bw-1)*s + kw] (zeros
// outside the image) and the weights, as [ci][tap][CT], in LDS; up to twenty of a thread's
// loads are requested before the first is stored. A thread accumulates four output channels
// of one pixel, so that one LDS read of the input serves four FMAs and the four weights are
// one 16-byte read.
// Threads take (channel group, pixel) pairs in order: with 64 pixels or more a wave shares
// its weights' address; smaller blocks fill the workgroup with more channel groups.
// Every sum runs in the fixed order ci -> i -> j with fp32 FMAs. The epilogue adds bias and
// residual in fp32, applies ReLU and writes straight to the block's position of the
// persistent output; elements outside active blocks are never touched.
//
// What bounds it: latency (a small layer is the index's round trip, one of loads, 16 x 9
// taps of two LDS reads and four FMAs per lane, one of stores). 3x3 16 -> 16 on 64x128
// with 32 active 8x8 blocks: 36.7 -> 9.5 us (before: up to eight scattered outputs per
// thread, two LDS reads per FMA, divisions by run-time sizes in every loop).
#include <algorithm>
#include <type_traits>

#include "bc_internal.h"

namespace bc {
namespace {

constexpr int kThreads = 256;
constexpr int kMaxOutputs = 2048;            // outputs per workgroup in the accepted sizes below
constexpr int kLdsBudget = 48 * 1024;
constexpr int kCo = 4;                       // output channels per thread

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
    int npx, parts;                          // pixels per part, parts per block
    int th, tw, ct, wp, ci_t, n_co_tiles;    // halo tile, channel tile, its LDS pitch, chunk
    int relu;
    Div f_tile, f_tw, f_bw, f_npx, f_row;    // th * tw, tw, bw, npx, ci_t * taps
};

// KS > 0: a KS x KS kernel known at compile time; KS = 0: any kernel.
template <int KS>
__global__ __launch_bounds__(kThreads) void k_conv_nchw_f32(F32Args a)
{
    extern __shared__ __align__(16) float lds[];
    const LayerGeom &g = a.g;
    int k = blockIdx.x / a.n_co_tiles, p0 = 0, r0 = 0;   // block, first pixel and its row
    const int cot = blockIdx.x - k * a.n_co_tiles;
    if (a.parts > 1) {
        const int kp = k / a.parts;
        p0 = (k - kp * a.parts) * kThreads;
        r0 = p0 / g.bw;
        k = kp;
    }
    // the block id with the active count, one round trip (k < total_blocks: a valid read)
    const int bid = g.idx ? g.idx[k] : k;
    const int cnt = g.count ? *g.count : g.total_blocks;
    if (k >= cnt) return;
    const int img = bid / (g.gh * g.gw);
    const int rem = bid - img * g.gh * g.gw;
    const int gy = rem / g.gw, gx = rem - (rem / g.gw) * g.gw;
    const int co0 = cot * a.ct;
    const int kh = KS ? KS : g.kh, kw = KS ? KS : g.kw;
    const int taps = kh * kw;
    const int oy0 = gy * g.bh, ox0 = gx * g.bw;
    const int y0 = (oy0 + r0) * g.stride - g.pad, x0 = ox0 * g.stride - g.pad;
    const int tile = a.th * a.tw;
    float *ws = lds;                                     // [ci_t][taps][wp]
    float *xs = lds + (size_t)a.ci_t * taps * a.wp;      // [ci_t][th][tw]
    const int tid = threadIdx.x;

    // this thread's channel group and pixel (threads past the last pair: its group, dead)
    const int grp = fdiv(tid, a.f_npx), p = p0 + tid - grp * a.npx;
    const int py = fdiv(p, a.f_bw), px = p - py * g.bw;
    const bool live = grp * kCo < a.ct && py < g.bh;
    const int base = live ? (py - r0) * g.stride * a.tw + px * g.stride : 0;
    const int cg = min(grp, a.ct / kCo - 1);
    const bool busy = __any(live);                       // a wave without a pair only loads
    float acc[kCo] = {0.f, 0.f, 0.f, 0.f};
    for (int c0 = 0; c0 < g.cin; c0 += a.ci_t) {
        const int cn = min(a.ci_t, g.cin - c0);
        const int nx = cn * tile, row = cn * taps;
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
            dst = e < a.ct * a.f_row.d && r < row ? r * a.wp + co : -1;
            const float v = a.w[in ? ((size_t)(co0 + co) * g.cin + c0) * taps + r : 0];
            return in ? v : 0.f;
        };
        if (c0) __syncthreads();                         // the previous chunk is done with
        const int nw = a.ct * a.f_row.d;
        // NX and NW loads in flight per thread, from element e0 of x and of the weights
        auto stage = [&](auto x_c, auto w_c, int e0) {
            constexpr int NX = decltype(x_c)::value, NW = decltype(w_c)::value;
            float vx[NX + 1], vw[NW];
            int dw[NW];
#pragma unroll
            for (int u = 0; u < NX; ++u) vx[u] = load_x(e0 + u * kThreads + tid);
#pragma unroll
            for (int u = 0; u < NW; ++u) vw[u] = load_w(e0 + u * kThreads + tid, dw[u]);
#pragma unroll
            for (int u = 0; u < NX; ++u)
                if (e0 + u * kThreads + tid < nx) xs[e0 + u * kThreads + tid] = vx[u];
#pragma unroll
            for (int u = 0; u < NW; ++u)
                if (dw[u] >= 0) ws[dw[u]] = vw[u];
        };
        using std::integral_constant;
        if (max(nx, nw) <= 2 * kThreads) {
            stage(integral_constant<int, 2>{}, integral_constant<int, 2>{}, 0);
        } else {
            for (int e0 = 0; e0 < max(nx, nw);) {
                if (e0 < nx) {
                    stage(integral_constant<int, 10>{}, integral_constant<int, 10>{}, e0);
                    e0 += 10 * kThreads;
                } else {
                    stage(integral_constant<int, 0>{}, integral_constant<int, 16>{}, e0);
                    e0 += 16 * kThreads;
                }
            }
        }
        __syncthreads();
        if (!busy) continue;
        // N taps (or channels, of a 1x1 kernel) are read before the first one's FMAs: left to
        // itself the compiler waits tap by tap (10 -> 12 us in the case above)
        constexpr int N = KS == 1 ? 8 : KS == 3 ? 9 : KS ? KS : 1;
        float v[N];
        float4 w[N];
        auto fmas = [&](int n) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < N; ++t) {
                if (t >= n) break;
                acc[0] = fmaf(w[t].x, v[t], acc[0]);
                acc[1] = fmaf(w[t].y, v[t], acc[1]);
                acc[2] = fmaf(w[t].z, v[t], acc[2]);
                acc[3] = fmaf(w[t].w, v[t], acc[3]);
            }
        };
        const float *xc = xs + base, *wc = ws + cg * kCo;
        if constexpr (KS == 1) {
            for (int ci = 0; ci < cn; ci += N) {
                const int n = min(N, cn - ci);
#pragma unroll
                for (int t = 0; t < N; ++t) {            // past the chunk: the last channel again, not used
                    const int c = min(ci + t, cn - 1);
                    v[t] = xc[c * tile];
                    w[t] = *(const float4 *)(wc + c * a.wp);
                }
                fmas(n);
            }
        } else if constexpr (KS > 0) {
            for (int ci = 0; ci < cn; ++ci) {
#pragma unroll
                for (int t0 = 0; t0 < KS * KS; t0 += N) {
#pragma unroll
                    for (int t = 0; t < N; ++t) {
                        v[t] = xc[(t0 + t) / KS * a.tw + (t0 + t) % KS];
                        w[t] = *(const float4 *)(wc + (t0 + t) * a.wp);
                    }
                    fmas(N);
                }
                xc += tile;
                wc += taps * a.wp;
            }
        } else {
            for (int ci = 0; ci < cn; ++ci) {
                for (int i = 0; i < kh; ++i)
                    for (int j = 0; j < kw; ++j) {
                        v[0] = xc[i * a.tw + j];
                        w[0] = *(const float4 *)(wc + (i * kw + j) * a.wp);
                        fmas(1);
                    }
                xc += tile;
                wc += taps * a.wp;
            }
        }
    }
    if (!live) return;
#pragma unroll
    for (int c = 0; c < kCo; ++c) {
        const int co = co0 + cg * kCo + c;
        if (co >= g.cout) continue;
        const size_t o = (((size_t)img * g.cout + co) * g.hout + oy0 + py) * g.wout + ox0 + px;
        float z = acc[c];
        if (a.bias) z += a.bias[co];
        if (a.res) z += a.res[o];
        if (a.relu) z = (z > 0.f || z != z) ? z : 0.f;
        a.y[o] = z;
    }
}

template <int KS>
hipError_t launch_ks(const F32Args &a, unsigned grid, size_t lds, hipStream_t s)
{
    auto kern = k_conv_nchw_f32<KS>;
    const hipError_t e = allow_lds((const void *)kern, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kThreads), lds, s, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_conv_nchw_f32(const float *x, const float *w, const float *bias,
                                const float *res, float *y, int relu, const LayerGeom &g,
                                hipStream_t s, const char **why)
{
    F32Args a;
    a.x = x; a.w = w; a.bias = bias; a.res = res; a.y = y; a.g = g; a.relu = relu;
    const int npx = g.bh * g.bw, taps = g.kh * g.kw;
    // the accepted sizes: 2048 pixels per block, and one input channel of its halo tile with
    // the weights of as many output channels as 2048 outputs hold in 48 KB
    const int co_t = g.cout < kMaxOutputs / npx ? g.cout : kMaxOutputs / npx;
    if (co_t < 1) {
        *why = "fp32 path: output block larger than 2048 pixels";
        return hipErrorInvalidValue;
    }
    const int block_tile = ((g.bh - 1) * g.stride + g.kh) * ((g.bw - 1) * g.stride + g.kw);
    if ((block_tile + co_t * taps) * (int)sizeof(float) > kLdsBudget) {
        *why = "fp32 path: one channel of the halo tile does not fit in LDS";
        return hipErrorInvalidValue;
    }
    // One pixel and four channels per thread: a small layer is latency, so its work is
    // spread over as many waves as there are (four 40x40 blocks, 16 -> 16: 87 us with seven
    // outputs per thread, 102 with seven pixels of four channels, 14 in parts of 256).
    // Blocks below 256 pixels take channel groups until the threads are used up (128x128
    // blocks of one pixel, 1x1 16 -> 128: 115 us with scattered outputs, 768 with 16 channels
    // per workgroup and one pixel in 64 lanes, 73 so) ...
    a.npx = std::min(npx, kThreads);
    a.parts = (npx + kThreads - 1) / kThreads;
    int rows = g.bh;                                     // that 256 pixels can touch
    if (a.parts > 1) rows = kThreads % g.bw ? (kThreads + g.bw - 2) / g.bw + 1 : kThreads / g.bw;
    a.th = (std::min(rows, g.bh) - 1) * g.stride + g.kh;
    a.tw = (g.bw - 1) * g.stride + g.kw;
    const int fit = kThreads / a.npx, groups = (g.cout + kCo - 1) / kCo;
    // ... but at most 16 channels where a thread would stage more than 20 of their weights
    // (16x16 blocks of 4x4, 64 active, 3x3 64 -> 64: 22 us, 76 with all channels), unless
    // blocks below 16 pixels are many (64x64 blocks of 2x2, 64 -> 64: 311 us with all
    // channels, 440 with 16), and at most 16 where blocks are few
    int most = fit;
    if (npx >= 16 || g.total_blocks < 2048)
        most = std::max(4, (int)(20 * kThreads / ((long long)g.cin * taps * kCo)));
    if (g.total_blocks < 512) most = 4;
    // ... and as many as it takes to stay below the 2^32 threads of a launch, past which the
    // runtime launches nothing and reports no error. All groups do, for the 4e9 output
    // elements and 2^20 blocks that a call can have.
    auto workgroups = [&](int n) { return (size_t)g.total_blocks * a.parts * ((groups + n - 1) / n); };
    most = std::min({groups, fit, most});
    if (workgroups(most) >= (size_t)1 << 24) most = std::min(groups, fit);
    a.ct = kCo * most;
    // an odd number of 16-byte units per row of weights: consecutive rows, which consecutive
    // threads write, start in other banks; not if that costs another chunk
    auto chunk = [&](int wp) {
        const int n = kLdsBudget / ((a.th * a.tw + wp * taps) * (int)sizeof(float));
        return n < 1 ? 1 : n > g.cin ? g.cin : n;        // at least one: four channels of a large kernel
    };
    a.wp = a.ct % 8 ? a.ct : a.ct + kCo;
    if ((g.cin - 1) / chunk(a.wp) > (g.cin - 1) / chunk(a.ct)) a.wp = a.ct;
    a.ci_t = chunk(a.wp);
    const int per_ci = (a.th * a.tw + a.wp * taps) * (int)sizeof(float);
    a.n_co_tiles = (g.cout + a.ct - 1) / a.ct;
    a.f_tile = make_div(a.th * a.tw);
    a.f_tw = make_div(a.tw);
    a.f_bw = make_div(g.bw);
    a.f_npx = make_div(a.npx);
    a.f_row = make_div(a.ci_t * taps);
    const size_t lds = (size_t)a.ci_t * per_ci;
    const unsigned grid = (unsigned)workgroups(most);
    if (g.kh != g.kw) return launch_ks<0>(a, grid, lds, s);
    switch (g.kh) {
    case 1: return launch_ks<1>(a, grid, lds, s);
    case 3: return launch_ks<3>(a, grid, lds, s);
    case 5: return launch_ks<5>(a, grid, lds, s);
    case 7: return launch_ks<7>(a, grid, lds, s);
    default: return launch_ks<0>(a, grid, lds, s);
    }
}

}  // namespace bc
