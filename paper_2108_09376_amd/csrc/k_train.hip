// The policy network's online update (Section 4 configuration: RMSprop every 4 frames
// on the REINFORCE loss of Section 3.5). Channels-last 16-bit activations and
// gradients, fp32 weight gradients and optimiser state.
//
//  * logit gradient: dL/dz_b = -R_b (a_b - p_b), written to channel 0 of the head's
//    [n][gh][gw][c] gradient map (other channels 0);
//  * gradient combine: out = (a + b) * [y > 0]: the ReLU's backward pass (b absent),
//    a residual's gradient added to another (y absent), or both;
//  * input gradient of a convolution (the transposed convolution) runs on the forward
//    matrix-core conv: weights flipped and transposed ([cout][kh][kw][cin] ->
//    [cin][kh][kw][cout], taps reversed), and for stride 2 the output gradient spread
//    onto the even pixels of a map of the input's size (zeros between), then a
//    stride-1 convolution with padding k/2 (these two kernels are here);
//  * weight gradient: dW[co][i][j][ci] += sum_p G[p][co] X[p*s - pad + (i, j)][ci], an
//    implicit GEMM whose reduction runs over pixels (maps that divide into 8 x 8 tiles:
//    k_wgrad_row16; the rest, here:). A workgroup owns a 64 x 64
//    (co, ci) tile of one tap and a range of 1024 pixels; per 128-pixel chunk it loads
//    G and the tap-shifted X rows with 16-byte requests (eight channels of one pixel),
//    transposes them in registers and stores them in LDS as [channel][pixel], so that
//    matrix-core fragments (eight consecutive pixels of one channel per lane) are
//    contiguous 16-byte LDS reads; the next two chunks' loads are in flight during the
//    current chunk's 16 MFMAs per wave (registers plus an LDS double buffer); the tile
//    is added to dW with fp32 atomics at the end (the order of those additions varies
//    between runs);
//  * bias gradient: db[co] += sum_p G[p][co], summed from the same G registers by the
//    workgroups of tap 0 (and the first ci tile), reduced across lanes, one atomic per
//    channel and workgroup;
//  * RMSprop (PyTorch's definition, no momentum): g' = g + wd w; v = alpha v +
//    (1 - alpha) g'^2; w -= lr g' / (sqrt(v) + eps); the gradient is reset to 0 and the
//    16-bit copy of w rewritten (round to nearest even); for one tensor, or for up to
//    kMaxParams tensors in one launch (their pointers and sizes in the kernel arguments).
#include <algorithm>
#include <cmath>
#include <mutex>
#include <type_traits>

#include "bc_internal.h"
#include "lds_dma.h"

namespace bc {
namespace {

constexpr int kThreads = 256;

typedef short short8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <bool BF16>
__device__ __forceinline__ float h16_to_f32(uint32_t h)
{
    if constexpr (BF16) return __uint_as_float(h << 16);
    else return (float)__builtin_bit_cast(_Float16, (uint16_t)h);
}

template <bool BF16>
__device__ __forceinline__ uint32_t f32_to_h16(float z)
{
    if constexpr (BF16) {
        const uint32_t u = __float_as_uint(z);
        if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (u >> 16) | 0x40u;
        return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
    } else {
        return __builtin_bit_cast(uint16_t, (_Float16)z);
    }
}

template <bool BF16>
__device__ __forceinline__ f32x4 mfma(short8 a, short8 b, f32x4 c)
{
    if constexpr (BF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a),
                                                      __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// ---------------------------------------------------------------- elementwise

template <bool BF16>
__global__ __launch_bounds__(kThreads) void k_logit_grad16(const float *__restrict__ reward,
                                                           const uint8_t *__restrict__ mask,
                                                           const float *__restrict__ prob,
                                                           uint4 *__restrict__ grad, int blocks,
                                                           int vpb)
{
    const int t = blockIdx.x * kThreads + threadIdx.x;
    if (t >= blocks * vpb) return;
    const int b = t / vpb, v = t - b * vpb;
    uint4 o = make_uint4(0u, 0u, 0u, 0u);
    if (v == 0) {
        const float a = mask[b] ? 1.f : 0.f;
        o.x = f32_to_h16<BF16>(-reward[b] * (a - prob[b]));
    }
    grad[t] = o;
}

template <bool BF16>
__global__ __launch_bounds__(kThreads) void k_grad_combine16(const uint4 *__restrict__ a,
                                                             const uint4 *__restrict__ b,
                                                             const uint4 *__restrict__ y,
                                                             uint4 *__restrict__ out, long long nvec)
{
    const long long t = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (t >= nvec) return;
    const uint4 va = a[t];
    const uint4 vb = b ? b[t] : make_uint4(0u, 0u, 0u, 0u);
    const uint4 vy = y ? y[t] : make_uint4(0u, 0u, 0u, 0u);
    const uint32_t aa[4] = {va.x, va.y, va.z, va.w}, bb[4] = {vb.x, vb.y, vb.z, vb.w};
    const uint32_t yy[4] = {vy.x, vy.y, vy.z, vy.w};
    uint32_t o[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        uint32_t r = 0;
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            const int sh = 16 * hh;
            float z = h16_to_f32<BF16>((aa[q] >> sh) & 0xFFFFu);
            if (b) z += h16_to_f32<BF16>((bb[q] >> sh) & 0xFFFFu);
            if (y && !(h16_to_f32<BF16>((yy[q] >> sh) & 0xFFFFu) > 0.f)) z = 0.f;
            r |= f32_to_h16<BF16>(z) << sh;
        }
        o[q] = r;
    }
    out[t] = make_uint4(o[0], o[1], o[2], o[3]);
}

// W [co][kh][kw][ci] -> W' [ci][kh][kw][co], taps reversed
// W' [ci][i][j][co] = W[co][k-1-i][k-1-j][ci]: the weights of the transposed convolution
__device__ __forceinline__ void flip_transpose_at(const uint16_t *__restrict__ w,
                                                  uint16_t *__restrict__ wt, int cout, int k,
                                                  int cin, int t)
{
    if (t >= cout * k * k * cin) return;
    const int co = t % cout;
    int r = t / cout;
    const int j = r % k;
    r /= k;
    const int i = r % k;
    const int ci = r / k;
    wt[t] = w[((co * k + (k - 1 - i)) * k + (k - 1 - j)) * cin + ci];
}

// Z [n][2h][2w][C]: Z[2y][2x] = G[y][x], zero elsewhere (16-byte vectors, C % 8 == 0)
__device__ __forceinline__ void zero_insert_at(const uint4 *__restrict__ g, uint4 *__restrict__ z,
                                               int n, int h, int w, int vpp, long long t)
{
    if (t >= (long long)n * 4 * h * w * vpp) return;
    const int v = (int)(t % vpp);
    long long r = t / vpp;
    const int x = (int)(r % (2 * w));
    r /= 2 * w;
    const int y = (int)(r % (2 * h));
    const int img = (int)(r / (2 * h));
    uint4 o = make_uint4(0u, 0u, 0u, 0u);
    if (!(x & 1) && !(y & 1)) o = g[(((long long)img * h + (y >> 1)) * w + (x >> 1)) * vpp + v];
    z[t] = o;
}

// Both inputs of the transposed convolution in one launch: workgroups below wblocks
// flip the weights, the rest (none at stride 1) spread the output gradient.
__global__ __launch_bounds__(kThreads) void k_input_grad_prep16(
    const uint16_t *__restrict__ w, uint16_t *__restrict__ wt, int cout, int k, int cin,
    unsigned wblocks, const uint4 *__restrict__ g, uint4 *__restrict__ z, int n, int h, int wd,
    int vpp)
{
    if (blockIdx.x < wblocks)
        flip_transpose_at(w, wt, cout, k, cin, (int)(blockIdx.x * kThreads + threadIdx.x));
    else
        zero_insert_at(g, z, n, h, wd, vpp,
                       (long long)(blockIdx.x - wblocks) * kThreads + threadIdx.x);
}

// ---------------------------------------------------------------- weight gradient

constexpr int kPx = 128;                      // pixels per chunk (four MFMA k steps)
constexpr int kRow = kPx * 2 + 16;            // LDS bytes per channel row (+16 pad)
constexpr int kWgPx = 1024;                   // pixels per workgroup (8 chunks)

struct WgradGeom {
    int n, hin, win, cin, hout, wout, cout, k, stride, pad;
    int npix;                                 // n * hout * wout
    int splits;                               // pixel ranges per (tile, tap)
    int x_bytes, g_bytes;
};

// LDS per chunk: G and X transposed, [channel][pixel], 64 rows of kRow bytes each. A
// thread holds eight channels (vector cv) of four consecutive pixels (quad pq) of each
// tensor and writes each channel's four pixels as one 8-byte word. With pq the fast
// index over a wave's lanes and a row pitch of 68 dwords, those writes and the MFMA
// fragment reads (16 rows at one column) are both free of bank conflicts.
template <bool BF16>
__global__ __launch_bounds__(kThreads) void k_wgrad16(const uint16_t *__restrict__ x,
                                                      const uint16_t *__restrict__ g,
                                                      float *__restrict__ dw, float *__restrict__ db,
                                                      WgradGeom G)
{
    __shared__ __align__(16) uint8_t lds[2][2][64 * kRow];   // [buffer][G, X][channel][pixel]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    // blockIdx.x = ((co tile * ci tiles + ci tile) * taps + tap) * splits + split
    const int ci_tiles = (G.cin + 63) / 64, taps = G.k * G.k;
    int r = blockIdx.x;
    const int split = r % G.splits;
    r /= G.splits;
    const int tap = r % taps;
    r /= taps;
    const int cit = r % ci_tiles, cot = r / ci_tiles;
    const int co0 = cot * 64, ci0 = cit * 64;
    const int ti = tap / G.k, tj = tap - ti * G.k;
    const int p_lo = split * kWgPx, p_hi = min(G.npix, p_lo + kWgPx);
    const int nch = (p_hi - p_lo + kPx - 1) / kPx;
    // the bias gradient comes from the first ci tile's tap-0 workgroups
    const bool bias = db != nullptr && cit == 0 && tap == 0;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
        (void *)x, (short)0, G.x_bytes, kBufferFlags);
    const __amdgpu_buffer_rsrc_t rg = __builtin_amdgcn_make_buffer_rsrc(
        (void *)g, (short)0, G.g_bytes, kBufferFlags);
    const int pq = tid & 31, cv = tid >> 5;
    const int hw = G.hout * G.wout;
    const bool ci_ok = ci0 + cv * 8 < G.cin;
    auto load = [&](int c, i32x4 (&vg)[4], i32x4 (&vx)[4]) {
        const int p0 = p_lo + c * kPx + 4 * pq;
        int img = 0, oy = 0, ox = 0;
        if (p0 < p_hi) {
            img = p0 / hw;
            const int rem = p0 - img * hw;
            oy = rem / G.wout;
            ox = rem - oy * G.wout;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int p = p0 + j;
            int og = kOutOfRange, oi = kOutOfRange;
            if (p < p_hi) {
                og = (p * G.cout + co0 + cv * 8) * 2;
                const int iy = oy * G.stride - G.pad + ti, ix = ox * G.stride - G.pad + tj;
                if (iy >= 0 && iy < G.hin && ix >= 0 && ix < G.win && ci_ok)
                    oi = (((img * G.hin + iy) * G.win + ix) * G.cin + ci0 + cv * 8) * 2;
            }
            asm volatile("" : "+v"(og), "+v"(oi));
            vg[j] = __builtin_amdgcn_raw_buffer_load_b128(rg, og, 0, 0);
            vx[j] = __builtin_amdgcn_raw_buffer_load_b128(rx, oi, 0, 0);
            if (++ox == G.wout) {
                ox = 0;
                if (++oy == G.hout) {
                    oy = 0;
                    ++img;
                }
            }
        }
    };
    float bsum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // channel e of the four pixels: halves e&1 of dword e>>1, pixels 0..3 -> one 8-byte word
    auto pack = [](const i32x4 (&v)[4], int e) {
        const int w = e >> 1;
        uint2 o;
        if (e & 1) {
            o.x = ((uint32_t)v[0][w] >> 16) | ((uint32_t)v[1][w] & 0xFFFF0000u);
            o.y = ((uint32_t)v[2][w] >> 16) | ((uint32_t)v[3][w] & 0xFFFF0000u);
        } else {
            o.x = ((uint32_t)v[0][w] & 0xFFFFu) | ((uint32_t)v[1][w] << 16);
            o.y = ((uint32_t)v[2][w] & 0xFFFFu) | ((uint32_t)v[3][w] << 16);
        }
        return o;
    };
    auto store = [&](int buf, const i32x4 (&vg)[4], const i32x4 (&vx)[4]) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int off = (cv * 8 + e) * kRow + pq * 8;
            *(uint2 *)(lds[buf][0] + off) = pack(vg, e);
            *(uint2 *)(lds[buf][1] + off) = pack(vx, e);
        }
        if (bias) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    bsum[e] += h16_to_f32<BF16>(((uint32_t)vg[j][e >> 1] >> (16 * (e & 1))) & 0xFFFFu);
        }
    };
    f32x4 acc[2][2];
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) acc[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto compute = [&](int buf) {
#pragma unroll
        for (int ks = 0; ks < kPx / 32; ++ks) {
            const int foff = ks * 64 + (lane >> 4) * 16;   // this lane's 8 pixels
            short8 af[2], bf[2];
#pragma unroll
            for (int mi = 0; mi < 2; ++mi)
                af[mi] = *(const short8 *)(lds[buf][0] + (wm * 32 + mi * 16 + (lane & 15)) * kRow + foff);
#pragma unroll
            for (int ni = 0; ni < 2; ++ni)
                bf[ni] = *(const short8 *)(lds[buf][1] + (wn * 32 + ni * 16 + (lane & 15)) * kRow + foff);
#pragma unroll
            for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                for (int ni = 0; ni < 2; ++ni) acc[mi][ni] = mfma<BF16>(af[mi], bf[ni], acc[mi][ni]);
        }
    };
    // two chunks in flight: register slot d holds chunk c (d = c & 1) until its store,
    // then receives chunk c + 2; LDS buffer d is rewritten two chunks after it was
    // read, and every thread passes the barrier in between
    i32x4 vg[2][4], vx[2][4];
    load(0, vg[0], vx[0]);
    load(1, vg[1], vx[1]);
    auto step = [&](auto dc, int cc) {
        constexpr int d = decltype(dc)::value;
        store(d, vg[d], vx[d]);
        __syncthreads();
        load(cc + 2, vg[d], vx[d]);              // past the range: zeros, never used
        compute(d);
    };
    // whole pairs of chunks in the loop (no exit inside it), then the odd last chunk
    int c = 0;
    for (; c + 2 <= nch; c += 2) {
        step(std::integral_constant<int, 0>{}, c);
        step(std::integral_constant<int, 1>{}, c + 1);
    }
    if (c < nch) step(std::integral_constant<int, 0>{}, c);
    // acc[mi][ni][i]: co = wm*32 + mi*16 + (lane>>4)*4 + i, ci = wn*32 + ni*16 + (lane&15)
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) {
            const int ci = ci0 + wn * 32 + ni * 16 + (lane & 15);
            if (ci >= G.cin) continue;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int co = co0 + wm * 32 + mi * 16 + (lane >> 4) * 4 + i;
                unsafeAtomicAdd(&dw[((size_t)co * taps + tap) * G.cin + ci], acc[mi][ni][i]);
            }
        }
    if (bias) {
        // the 32 lanes of one channel vector (one half of the wave) hold its pixel quads
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int m = 1; m < 32; m <<= 1) bsum[e] += __shfl_xor(bsum[e], m, 64);
        if (pq == 0)
#pragma unroll
            for (int e = 0; e < 8; ++e) unsafeAtomicAdd(&db[co0 + cv * 8 + e], bsum[e]);
    }
}

// ---------------------------------------------------------------- weight gradient, one kernel row
//
// Maps whose output divides into 8 x 8 pixel tiles. The general form above loads both
// operands once per tap and transposes them in registers; here a workgroup owns a 64 x 64
// (co, ci) tile of a whole kernel row (KW taps) and a run of pixel tiles:
//  * a tile's 64 output-gradient pixels and the input pixels under them for this kernel
//    row (8 rows of XC columns; zeros outside the image) go straight from memory to LDS,
//    128 bytes (64 channels) per pixel, NB tiles deep, one barrier per tile;
//  * matrix-core fragments want eight pixels of one channel per lane: ds_read_b64_tr_b16
//    transposes on the way out (16 lanes read 4 pixels x 16 channels and each gets four
//    pixels of one channel), so a tap is a shift of the row address and nothing is copied.
//    The order of the pixels within a product is the same for both operands;
//  * the 32-byte channel pairs of a row are stored at pair ^ f(row), f running over every
//    second row a read touches: 32 lanes then cover all 64 banks (no conflicts counted);
//  * two groups of four waves take one half of a tile's pixels each (32 x 32 quadrants),
//    and read the next tile's fragments while the current one's products run: one wave per
//    SIMD that waits for its own reads took 0.77 us per tile. The groups exchange halves
//    through LDS at the end;
//  * products of at most kFold tiles are added up by the matrix cores, whose running sums
//    round less well than fp32 additions do; then they join the run's totals;
//  * dW is added with fp32 atomics (one per element and workgroup);
//  * the bias gradient has workgroups of its own at the end of the grid (bias_run).
typedef short s16x4 __attribute__((ext_vector_type(4)));

// Eight pixels of one channel: two transposed reads of four pixels each.
__device__ __forceinline__ short8 read_tr(const uint8_t *lo, const uint8_t *hi)
{
    typedef __attribute__((address_space(3))) s16x4 *lds_p;
    const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(__attribute__((address_space(3))) uint8_t *)lo);
    const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(__attribute__((address_space(3))) uint8_t *)hi);
    return short8{a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
}

struct WgradRow {
    int hin, win, cin, hout, wout, cout, pad;
    int tw, tpi, tiles;                       // pixel tiles per row, per image, in all
    int ci_tiles, splits, run;                // runs of `run` tiles
    int npix, wgs;                            // output pixels; workgroups of dW (db's follow)
    int bias_px, bias_runs;                   // pixels per workgroup of db, workgroups per co tile
    int x_bytes, g_bytes;
};

constexpr int kRowThreads = 512;
constexpr int kFold = 16;

// Adds the gradients of 64 output channels (from co0) over the pixels [p_lo, p_hi) to db.
// Of every kBiasPx pixels a thread sums sixteen (requested together) for eight channels;
// the 64 threads of a channel then meet in a tree through LDS (18 KB), one atomic each.
constexpr int kBiasPx = 1024;

template <bool BF16>
__device__ __forceinline__ void bias_run(const __amdgpu_buffer_rsrc_t &rg, float *db, int cout, int co0, int p_lo,
                                         int p_hi, float *part)
{
    constexpr int N = kBiasPx / 64;
    const int tid = threadIdx.x, cv = tid & 7, pq = tid >> 3;
    float tot[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int p0 = p_lo + pq; p0 - pq < p_hi; p0 += kBiasPx) {
        i32x4 v[N];
#pragma unroll
        for (int i = 0; i < N; ++i)
            v[i] = __builtin_amdgcn_raw_buffer_load_b128(
                rg, p0 + 64 * i < p_hi ? ((p0 + 64 * i) * cout + co0 + cv * 8) * 2 : kOutOfRange, 0, 0);
        float sum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                sum[e] += h16_to_f32<BF16>(((uint32_t)v[i][e >> 1] >> (16 * (e & 1))) & 0xFFFFu);
#pragma unroll
        for (int e = 0; e < 8; ++e) tot[e] += sum[e];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) part[pq * 64 + cv * 8 + e] = tot[e];
    __syncthreads();
    auto eight = [](const float *p) {
        return ((p[0] + p[64]) + (p[128] + p[192])) + ((p[256] + p[320]) + (p[384] + p[448]));
    };
    const int ch = tid & 63;
    float *joined = part + 64 * 64;
    joined[(tid >> 6) * 64 + ch] = eight(part + (tid >> 6) * 512 + ch);
    __syncthreads();
    if (tid < 64) unsafeAtomicAdd(&db[co0 + ch], eight(joined + ch));
}

template <int KW, int S>
struct WgradShape {
    static constexpr int ST = KW == 1 ? 1 : S;            // slots between adjacent output pixels
    static constexpr int XC = 7 * ST + KW;                // staged input columns
    static constexpr int XI = (8 * XC + 63) / 64;         // input requests per wave (8 rows each)
    static constexpr int DW = 1 + XI;                     // requests per wave and tile
    static constexpr int BUF = 8192 + XI * 8192;          // LDS bytes per tile
    static constexpr int NB = 4;
    static_assert(NB * BUF <= 128 * 1024 && NB * DW <= 63, "LDS and vmcnt");
};

template <bool BF16, int KW, int S>
__global__ __launch_bounds__(kRowThreads, 1) void k_wgrad_row16(const uint16_t *__restrict__ x,
                                                                const uint16_t *__restrict__ g,
                                                                float *__restrict__ dw, float *__restrict__ db,
                                                                WgradRow G)
{
    using W = WgradShape<KW, S>;
    extern __shared__ __align__(16) uint8_t smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1;
    if ((int)blockIdx.x >= G.wgs) {                      // db (uniform)
        const int b = blockIdx.x - G.wgs, cot = b / G.bias_runs;
        const int p_lo = (b - cot * G.bias_runs) * G.bias_px;
        const __amdgpu_buffer_rsrc_t rg = __builtin_amdgcn_make_buffer_rsrc((void *)g, (short)0, G.g_bytes,
                                                                            kBufferFlags);
        bias_run<BF16>(rg, db, G.cout, cot * 64, p_lo, min(G.npix, p_lo + G.bias_px), (float *)smem);
        return;
    }
    // blockIdx.x = ((co tile * ci tiles + ci tile) * KW + kernel row) * splits + run
    int r = blockIdx.x;
    const int split = r % G.splits;
    r /= G.splits;
    const int ki = r % KW;
    r /= KW;
    const int cit = r % G.ci_tiles, cot = r / G.ci_tiles;
    const int co0 = cot * 64, ci0 = cit * 64;
    const int t_lo = split * G.run, t_hi = min(G.tiles, t_lo + G.run);
    const i32x4 xd = raw_desc(x, G.x_bytes), gd = raw_desc(g, G.g_bytes);
    const uint32_t lbase = __builtin_amdgcn_readfirstlane(lds_addr(smem));
    // this lane's part of a request of 8 rows: row lane >> 3, 16-byte unit lane & 7 of LDS;
    // f of its row (8 (wave + 8 v) + (lane >> 3)) does not depend on v
    const int row8 = 8 * wave + (lane >> 3);
    const int gu = (lane & 7) ^ (((row8 >> 1) & 3) * 2);
    const int xu = (lane & 7) ^ (((W::ST == 2 ? row8 >> 2 : row8 >> 1) & 3) * 2);
    const bool ci_ok = ci0 + xu * 8 < G.cin;
    // per request: this lane's row and column of the input tile (rows past it: never in the
    // image) and its byte offset from the tile's first input pixel
    int xdy[W::XI], xdx[W::XI], xoff[W::XI];
#pragma unroll
    for (int v = 0; v < W::XI; ++v) {
        const int slot = row8 + 64 * v;
        const int hy = slot / W::XC, hx = slot - hy * W::XC;
        xdy[v] = ci_ok && hy < 8 ? hy * S : -(1 << 28);
        xdx[v] = hx * (KW == 1 ? S : 1);
        xoff[v] = ((hy * S * G.win + xdx[v]) * G.cin + ci0 + xu * 8) * 2;
    }
    const int goff = ((wave * G.wout + (lane >> 3)) * G.cout + co0 + gu * 8) * 2;
    int img = t_lo / G.tpi, ty = (t_lo - img * G.tpi) / G.tw, tx = t_lo - img * G.tpi - ty * G.tw;
    int left = t_hi - t_lo;                              // tiles not yet requested
    auto issue = [&](int buf) {                          // past the run: zeros, never used
        const int gb = ((img * G.hout + ty * 8) * G.wout + tx * 8) * G.cout * 2;
        dma16(gd, lbase + buf * W::BUF + wave * 1024, left > 0 ? gb + goff : kOutOfRange);
        const int iy0 = ty * 8 * S - G.pad + ki, ix0 = tx * 8 * S - G.pad;
        const int xb = ((img * G.hin + iy0) * G.win + ix0) * G.cin * 2;
#pragma unroll
        for (int v = 0; v < W::XI; ++v) {
            const bool ok = left > 0 && (unsigned)(iy0 + xdy[v]) < (unsigned)G.hin &&
                            (unsigned)(ix0 + xdx[v]) < (unsigned)G.win;
            dma16(xd, lbase + buf * W::BUF + 8192 + (wave + 8 * v) * 1024, ok ? xb + xoff[v] : kOutOfRange);
        }
        --left;
        if (++tx == G.tw) {
            tx = 0;
            if ((++ty) * G.tw == G.tpi) {
                ty = 0;
                ++img;
            }
        }
    };
    // fragment addresses: lane = 16 gq + 4 j + a reads pixel 4 gq + j (of 16), channels 4 a ..;
    // this group's 32 pixels are tile rows 4 grp .. 4 grp + 3, two halves of 16
    const int gq = lane >> 4, j = (lane >> 2) & 3, ac = lane & 3;
    int ga[2], xa[KW][2];                                // [half], [tap][half]: channel pairs 2 wm, 2 wn
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int p = grp * 32 + h * 16 + 4 * gq + j;
        ga[h] = p * 128 + ((wm * 2) ^ ((p >> 1) & 3)) * 32 + ac * 8;
#pragma unroll
        for (int kj = 0; kj < KW; ++kj) {
            const int slot = (p >> 3) * W::XC + (p & 7) * W::ST + kj;
            const int f = (W::ST == 2 ? slot >> 2 : slot >> 1) & 3;
            xa[kj][h] = 8192 + slot * 128 + ((wn * 2) ^ f) * 32 + ac * 8;
        }
    }
    auto read_g = [&](const uint8_t *b, int mi) { return read_tr(b + (ga[0] ^ (mi * 32)), b + (ga[1] ^ (mi * 32))); };
    auto read_x = [&](const uint8_t *b, int kj, int ni) {
        return read_tr(b + (xa[kj][0] ^ (ni * 32)), b + (xa[kj][1] ^ (ni * 32)));
    };
    f32x4 acc[KW][2][2], tot[KW][2][2];                  // tot: of the batches before, if any
#pragma unroll
    for (int kj = 0; kj < KW; ++kj)
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int ni = 0; ni < 2; ++ni) acc[kj][mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Tile t + 1 has arrived for this wave and its reads of tile t are done; past the
    // barrier both hold for every wave, so tile t's buffer takes tile t + NB.
    auto arrived = [&](auto n) {
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(decltype(n)::value) : "memory");
    };
#pragma unroll
    for (int d = 0; d < W::NB; ++d) issue(d);
    arrived(std::integral_constant<int, (W::NB - 1) * W::DW>{});
    short8 af[2], bf[KW][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) af[i] = read_g(smem, i);
#pragma unroll
    for (int kj = 0; kj < KW; ++kj)
#pragma unroll
        for (int i = 0; i < 2; ++i) bf[kj][i] = read_x(smem, kj, i);
    int buf = 0;
    bool folded = false;
    for (int t = t_lo;;) {
        const int t_fold = min(t_hi, t + kFold);
        for (; t < t_fold; ++t) {
            arrived(std::integral_constant<int, (W::NB - 2) * W::DW>{});
            const int next = buf + 1 == W::NB ? 0 : buf + 1;
            const uint8_t *b = smem + next * W::BUF;     // past the run: the zeros requested there
            short8 an[2], bn[KW][2];
#pragma unroll
            for (int i = 0; i < 2; ++i) an[i] = read_g(b, i);
#pragma unroll
            for (int kj = 0; kj < KW; ++kj) {
#pragma unroll
                for (int i = 0; i < 2; ++i) bn[kj][i] = read_x(b, kj, i);
#pragma unroll
                for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                    for (int ni = 0; ni < 2; ++ni) acc[kj][mi][ni] = mfma<BF16>(af[mi], bf[kj][ni], acc[kj][mi][ni]);
                __builtin_amdgcn_sched_barrier(0);
            }
            issue(buf);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                af[i] = an[i];
#pragma unroll
                for (int kj = 0; kj < KW; ++kj) bf[kj][i] = bn[kj][i];
            }
            buf = next;
        }
        if (t == t_hi) break;
#pragma unroll
        for (int kj = 0; kj < KW; ++kj)
#pragma unroll
            for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                for (int ni = 0; ni < 2; ++ni) {
                    tot[kj][mi][ni] = folded ? tot[kj][mi][ni] + acc[kj][mi][ni] : acc[kj][mi][ni];
                    acc[kj][mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
        folded = true;
    }
    if (folded) {
#pragma unroll
        for (int kj = 0; kj < KW; ++kj)
#pragma unroll
            for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                for (int ni = 0; ni < 2; ++ni) acc[kj][mi][ni] = tot[kj][mi][ni] + acc[kj][mi][ni];
    }
    // every request must be done before LDS is used for the exchange (and given back)
    arrived(std::integral_constant<int, 0>{});
    // The tile [tap][co][ci] in LDS: the second group's sums, then the first's added
    // (first half of the pixels + second half, per element).
    // acc[kj][mi][ni][i]: co = wm*32 + mi*16 + (lane>>4)*4 + i, ci = wn*32 + ni*16 + (lane&15)
    float *out = (float *)smem;
    const int oo = (wm * 32 + (lane >> 4) * 4) * 64 + wn * 32 + (lane & 15);
    if (grp == 1) {
#pragma unroll
        for (int kj = 0; kj < KW; ++kj)
#pragma unroll
            for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                for (int ni = 0; ni < 2; ++ni)
#pragma unroll
                    for (int i = 0; i < 4; ++i) out[oo + (kj * 64 + mi * 16 + i) * 64 + ni * 16] = acc[kj][mi][ni][i];
    }
    __syncthreads();
    if (grp == 0) {
#pragma unroll
        for (int kj = 0; kj < KW; ++kj)
#pragma unroll
            for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                for (int ni = 0; ni < 2; ++ni)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        float *o = &out[oo + (kj * 64 + mi * 16 + i) * 64 + ni * 16];
                        *o = acc[kj][mi][ni][i] + *o;
                    }
    }
    __syncthreads();
    // One add covers 64 consecutive ci of a (tap, co) row; every run starts at another row,
    // so that runs which end together do not queue at the same addresses.
    const int rowb = KW * KW * G.cin * 4;
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(dw + ((size_t)co0 * KW + ki) * KW * G.cin + ci0), (short)0, kOutOfRange, kBufferFlags);
    const int lo = ci0 + lane < G.cin ? lane * 4 : kOutOfRange;
#pragma unroll 8
    for (int it = 0; it < KW * 8; ++it) {
        const int row = (it * 8 + wave + split * 24) % (KW * 64);      // uniform
        __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_f32(out[row * 64 + lane], rw, lo,
                                                        (row & 63) * rowb + (row >> 6) * G.cin * 4, 0);
    }
}

template <bool BF16, int KW, int S>
hipError_t launch_wgrad_row(const uint16_t *x, const uint16_t *g, float *dw, float *db, const WgradRow &G,
                            unsigned grid, hipStream_t s)
{
    constexpr int lds = WgradShape<KW, S>::NB * WgradShape<KW, S>::BUF;
    auto kern = k_wgrad_row16<BF16, KW, S>;
    const hipError_t e = allow_lds((const void *)kern, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kRowThreads), lds, s, x, g, dw, db, G);
    return hipGetLastError();
}

// ---------------------------------------------------------------- RMSprop

template <bool BF16>
__global__ __launch_bounds__(kThreads) void k_rmsprop(float *__restrict__ w, float *__restrict__ v,
                                                      float *__restrict__ grad, long long count,
                                                      float lr, float alpha, float eps, float wd,
                                                      uint16_t *__restrict__ w16)
{
    const long long t = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (t >= count) return;
    const float wi = w[t];
    const float gi = grad[t] + wd * wi;
    const float vi = alpha * v[t] + (1.f - alpha) * gi * gi;
    const float wn = wi - lr * gi / (sqrtf(vi) + eps);
    v[t] = vi;
    w[t] = wn;
    grad[t] = 0.f;
    if (w16) w16[t] = (uint16_t)f32_to_h16<BF16>(wn);
}

// Several tensors in one launch: workgroup b belongs to the tensor t with
// first[t] <= b < first[t + 1] (a uniform scan over at most kMaxParams entries of the
// kernel arguments), elements [(b - first[t]) * kThreads * U, ...) of that tensor, U per
// thread and all requested before the first is used (1.4 M parameters in 22 tensors: 12.8
// us with U = 1, 8.2 with U = 4).
template <bool BF16, int U>
__global__ __launch_bounds__(kThreads) void k_rmsprop_many(RmspropMany m, float lr, float alpha,
                                                           float eps, float wd)
{
    const int b = blockIdx.x;
    int t = 0;
    while (t + 1 < m.n && m.first[t + 1] <= b) ++t;
    const long long i0 = (long long)(b - m.first[t]) * (kThreads * U) + threadIdx.x;
    float *w = m.w[t], *v = m.v[t], *grad = m.grad[t];
    const long long count = m.count[t];
    if (i0 >= count) return;
    float wi[U], vo[U], go[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const long long i = i0 + u * kThreads < count ? i0 + u * kThreads : i0;
        wi[u] = w[i];
        vo[u] = v[i];
        go[u] = grad[i];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const long long i = i0 + u * kThreads;
        if (i >= count) continue;
        const float gi = go[u] + wd * wi[u];
        const float vi = alpha * vo[u] + (1.f - alpha) * gi * gi;
        const float wn = wi[u] - lr * gi / (sqrtf(vi) + eps);
        v[i] = vi;
        w[i] = wn;
        grad[i] = 0.f;
        if (m.w16[t]) m.w16[t][i] = (uint16_t)f32_to_h16<BF16>(wn);
    }
}

// ---------------------------------------------------------------- workspace

// Library-owned workspace of the input gradients, one per device. It grows by allocating
// a larger buffer; the old one is kept (never freed), so a graph that captured a call
// keeps a valid pointer. hipMalloc is not allowed during capture: a capturing call that
// would grow it is refused.
std::mutex g_tw_mu;
void *g_tw_ptr[64];
size_t g_tw_bytes[64];

hipError_t train_workspace(size_t bytes, hipStream_t s, void **out, const char **why)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_tw_mu);
    if (g_tw_bytes[dev] < bytes) {
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        e = hipStreamIsCapturing(s, &cs);
        if (e != hipSuccess) return e;
        if (cs != hipStreamCaptureStatusNone) {
            *why = "the input-gradient workspace must grow and the stream is capturing (no "
                   "allocation during capture): make one uncaptured call at the largest size first";
            return hipErrorStreamCaptureUnsupported;
        }
        size_t want = 2 * g_tw_bytes[dev];
        if (want < bytes) want = bytes;
        if (want < ((size_t)16 << 20)) want = (size_t)16 << 20;
        void *p = nullptr;
        e = hipMalloc(&p, want);
        if (e != hipSuccess) return e;
        g_tw_ptr[dev] = p;          // the previous buffer stays allocated (see above)
        g_tw_bytes[dev] = want;
    }
    *out = g_tw_ptr[dev];
    return hipSuccess;
}

unsigned blocks_for(long long n) { return (unsigned)((n + kThreads - 1) / kThreads); }

}  // namespace

hipError_t launch_logit_grad(const float *reward, const uint8_t *mask, const float *prob,
                             void *grad, int blocks, int c, bool bf16, hipStream_t s)
{
    const int vpb = c / 8;
    if (bf16)
        hipLaunchKernelGGL(k_logit_grad16<true>, dim3(blocks_for((long long)blocks * vpb)), dim3(kThreads), 0, s,
                           reward, mask, prob, (uint4 *)grad, blocks, vpb);
    else
        hipLaunchKernelGGL(k_logit_grad16<false>, dim3(blocks_for((long long)blocks * vpb)), dim3(kThreads), 0, s,
                           reward, mask, prob, (uint4 *)grad, blocks, vpb);
    return hipGetLastError();
}

hipError_t launch_grad_combine(const void *a, const void *b, const void *y, void *out,
                               long long elems, bool bf16, hipStream_t s)
{
    const long long nvec = elems / 8;
    if (bf16)
        hipLaunchKernelGGL(k_grad_combine16<true>, dim3(blocks_for(nvec)), dim3(kThreads), 0, s,
                           (const uint4 *)a, (const uint4 *)b, (const uint4 *)y, (uint4 *)out, nvec);
    else
        hipLaunchKernelGGL(k_grad_combine16<false>, dim3(blocks_for(nvec)), dim3(kThreads), 0, s,
                           (const uint4 *)a, (const uint4 *)b, (const uint4 *)y, (uint4 *)out, nvec);
    return hipGetLastError();
}

hipError_t launch_conv_input_grad(const uint16_t *grad_out, const uint16_t *w, const uint16_t *accum,
                                  uint16_t *grad_in, const LayerGeom &fwd, Half16 fmt,
                                  hipStream_t s, const char **why)
{
    // workspace: flipped weights, then (stride 2) the spread output gradient
    const size_t wbytes = ((size_t)fwd.cout * fwd.kh * fwd.kw * fwd.cin * 2 + 255) & ~(size_t)255;
    const size_t zbytes = fwd.stride == 2 ? (size_t)fwd.n * fwd.hin * fwd.win * fwd.cout * 2 : 0;
    void *ws = nullptr;
    hipError_t e = train_workspace(wbytes + zbytes, s, &ws, why);
    if (e != hipSuccess) return e;
    uint16_t *wt = (uint16_t *)ws;
    const unsigned wblocks = blocks_for((long long)fwd.cout * fwd.kh * fwd.kw * fwd.cin);
    const uint16_t *src = grad_out;
    uint16_t *z = nullptr;
    unsigned zblocks = 0;
    if (fwd.stride == 2) {
        z = (uint16_t *)((uint8_t *)ws + wbytes);
        zblocks = blocks_for((long long)fwd.n * fwd.hin * fwd.win * (fwd.cout / 8));
        src = z;
    }
    hipLaunchKernelGGL(k_input_grad_prep16, dim3(wblocks + zblocks), dim3(kThreads), 0, s, w, wt,
                       fwd.cout, fwd.kh, fwd.cin, wblocks, (const uint4 *)grad_out, (uint4 *)z,
                       fwd.n, fwd.hout, fwd.wout, fwd.cout / 8);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    // stride-1 convolution of the (spread) output gradient with the flipped weights,
    // every block of the input-sized map (blocks of at most 8 x 8 pixels)
    LayerGeom L;
    L.n = fwd.n;
    L.cin = fwd.cout; L.hin = fwd.hin; L.win = fwd.win;
    L.cout = fwd.cin; L.hout = fwd.hin; L.wout = fwd.win;
    L.kh = fwd.kh; L.kw = fwd.kw; L.stride = 1; L.pad = fwd.kh / 2;
    L.bh = fwd.hin < 8 ? fwd.hin : 8;
    L.bw = fwd.win < 8 ? fwd.win : 8;
    L.gh = fwd.hin / L.bh; L.gw = fwd.win / L.bw;
    L.total_blocks = L.n * L.gh * L.gw;
    L.idx = nullptr;
    L.count = nullptr;
    return launch_conv_nhwc_mfma(src, wt, nullptr, accum, grad_in, 0, fmt, L, s, why);
}

hipError_t launch_conv_weight_grad(const uint16_t *x, const uint16_t *g, float *dw, float *db,
                                   const LayerGeom &fwd, bool bf16, hipStream_t s)
{
    // One kernel row per workgroup where the output divides into 8 x 8 tiles (us per launch,
    // before -> with it: 3x3 64 -> 64 at 128 x 256 24.1 -> 17.3, 128 -> 128 at 64 x 128 20.2
    // -> 15.9, 32 -> 64 stride 2 21.2 -> 16.3; 1x1 64 -> 64 at 64 x 128 14.3 -> 6.5), not for
    // 3x3 layers below 1024 output pixels (8 x 16 pixels 4.8 -> 6.1), nor where the uniform
    // offsets of a 64-row tile could pass 2 GiB, nor for maps not aligned to 16 bytes, which
    // the requests to LDS need.
    const bool aligned = (((uintptr_t)x | (uintptr_t)g) & 15) == 0;
    if (aligned && fwd.hout % 8 == 0 && fwd.wout % 8 == 0 && fwd.cin <= (1 << 18) &&
        (fwd.kh == 1 || fwd.n * fwd.hout * fwd.wout >= 1024)) {
        WgradRow R;
        R.hin = fwd.hin; R.win = fwd.win; R.cin = fwd.cin;
        R.hout = fwd.hout; R.wout = fwd.wout; R.cout = fwd.cout; R.pad = fwd.pad;
        R.tw = fwd.wout / 8;
        R.tpi = (fwd.hout / 8) * R.tw;
        R.tiles = fwd.n * R.tpi;
        R.npix = fwd.n * fwd.hout * fwd.wout;
        R.ci_tiles = (fwd.cin + 63) / 64;
        const int base = (fwd.cout / 64) * R.ci_tiles * fwd.kh;
        // Splits of the tiles. More splits shorten a workgroup's run (a tile's time is that of
        // its loads, 2 to 4 KB per wave) and add to dW more often. Over 60 shapes the time is
        // least near sqrt(6 KB * tiles / base), and up to 48 workgroups cost nothing. Not more
        // workgroups, db's among them, than run at once (a second round: 3x3 256 -> 256 at
        // 128 x 256, 79 us with 5 splits, 118 with 6; CUs with two of them and CUs with one,
        // which 1x1 layers' LDS allows: 256 -> 256 at 256 x 256, 44 us with 400, 33 with 240),
        // nor more additions per address than 16 + one per 2048 pixels: each rounds the whole
        // sum (1x1 64 -> 64 at 64 x 128, values of one sign: error 7.2e-8 with the general
        // form, 6.4e-8 with 20 additions, 8.1e-8 with 32, 1.5e-7 with 128).
        const int kb = fwd.kh == 1 ? 2 : 2 + fwd.stride;
        const float best = sqrtf(6.f * kb * R.tiles / base);
        const int slots = fwd.kh == 1 && best * base >= 512.f ? 512 : 256;
        const int cot = fwd.cout / 64;
        const int fit = (int)((slots / cot - 1) / (R.ci_tiles * fwd.kh + 0.5f));
        int splits = std::max((int)(best + 0.5f), 48 / base);
        splits = std::min({splits, fit, R.tiles, 16 + R.npix / 2048});
        if (splits < 1) splits = 1;
        R.run = (R.tiles + splits - 1) / splits;
        R.splits = (R.tiles + R.run - 1) / R.run;
        R.x_bytes = (int)((size_t)fwd.n * fwd.hin * fwd.win * fwd.cin * 2);
        R.g_bytes = (int)((size_t)fwd.n * fwd.hout * fwd.wout * fwd.cout * 2);
        R.wgs = base * R.splits;
        // db: about twice the pixels of a run per workgroup, less than its time
        R.bias_px = kBiasPx * ((R.run + 7) / 8);
        R.bias_runs = (R.npix + R.bias_px - 1) / R.bias_px;
        const unsigned grid = (unsigned)(R.wgs + (db ? (fwd.cout / 64) * R.bias_runs : 0));
        auto go = [&](auto kw, auto st) {
            constexpr int KW = decltype(kw)::value, S = decltype(st)::value;
            return bf16 ? launch_wgrad_row<true, KW, S>(x, g, dw, db, R, grid, s)
                        : launch_wgrad_row<false, KW, S>(x, g, dw, db, R, grid, s);
        };
        using one = std::integral_constant<int, 1>;
        using two = std::integral_constant<int, 2>;
        using three = std::integral_constant<int, 3>;
        if (fwd.kh == 1) return fwd.stride == 1 ? go(one{}, one{}) : go(one{}, two{});
        return fwd.stride == 1 ? go(three{}, one{}) : go(three{}, two{});
    }
    WgradGeom G;
    G.n = fwd.n; G.hin = fwd.hin; G.win = fwd.win; G.cin = fwd.cin;
    G.hout = fwd.hout; G.wout = fwd.wout; G.cout = fwd.cout;
    G.k = fwd.kh; G.stride = fwd.stride; G.pad = fwd.pad;
    G.npix = fwd.n * fwd.hout * fwd.wout;
    G.splits = (G.npix + kWgPx - 1) / kWgPx;
    G.x_bytes = (int)((size_t)fwd.n * fwd.hin * fwd.win * fwd.cin * 2);
    G.g_bytes = (int)((size_t)G.npix * fwd.cout * 2);
    const unsigned grid = (unsigned)((fwd.cout / 64) * ((fwd.cin + 63) / 64) * G.k * G.k * G.splits);
    if (bf16) hipLaunchKernelGGL(k_wgrad16<true>, dim3(grid), dim3(kThreads), 0, s, x, g, dw, db, G);
    else hipLaunchKernelGGL(k_wgrad16<false>, dim3(grid), dim3(kThreads), 0, s, x, g, dw, db, G);
    return hipGetLastError();
}

hipError_t launch_rmsprop_many(const RmspropMany &m, float lr, float alpha, float eps, float wd,
                               bool bf16, hipStream_t s)
{
    static_assert(kThreads == kRmspropThreads, "workgroups counted by the caller");
    const dim3 grid((unsigned)m.first[m.n]), block(kThreads);
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, block, 0, s, m, lr, alpha, eps, wd); };
    if (m.per == 4) bf16 ? go(k_rmsprop_many<true, 4>) : go(k_rmsprop_many<false, 4>);
    else bf16 ? go(k_rmsprop_many<true, 1>) : go(k_rmsprop_many<false, 1>);
    return hipGetLastError();
}

hipError_t launch_rmsprop(float *w, float *v, float *grad, long long count, float lr, float alpha,
                          float eps, float wd, void *w16, bool bf16, hipStream_t s)
{
    if (bf16)
        hipLaunchKernelGGL(k_rmsprop<true>, dim3(blocks_for(count)), dim3(kThreads), 0, s, w, v, grad,
                           count, lr, alpha, eps, wd, (uint16_t *)w16);
    else
        hipLaunchKernelGGL(k_rmsprop<false>, dim3(blocks_for(count)), dim3(kThreads), 0, s, w, v, grad,
                           count, lr, alpha, eps, wd, (uint16_t *)w16);
    return hipGetLastError();
}

}  // namespace bc
