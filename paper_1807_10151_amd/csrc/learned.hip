// Learned SPD preconditioner M = C^T diag(softplus(d)) C (used in Algorithm 2,
// step 2, in place of the Fourier preconditioner of Section 3.2).
//
// C is a stack of L linear 3x3 cross-correlations without bias with zero
// "same" padding: 1 -> 16 channels, then 16 -> 16.  C^T applies, in reverse
// layer order, each layer's adjoint: the correlation with the spatially
// flipped kernel and swapped channel roles.  d has one entry per channel.
//
// Layout: activations are channels-last float32 [B][H][W][16]; images are
// [B][H][W].  Parameters theta (float32) = W_1 [16][1][3][3], W_2..W_L
// [16][16][3][3], d [16]; tap t = 3 ky + kx reads the input at offset
// (ky - 1, kx - 1).
//
// The layers run as implicit GEMM on MFMA (v_mfma_f32_16x16x4f32).  16 -> 16: a
// wave walks strips of 16 columns down the rows, a tile of 16 pixels of a row by
// the 16 output channels at a time (A = 16 pixels x 4 input channels of one
// tap, B = 4 input channels x 16 output channels), 9 taps x 4 channel groups =
// 36 MFMAs per tile.  MFMA cg takes input channel 4 kq + cg from lane group kq,
// so each lane reads its 4 channels of a pixel as one 16-byte load, and a row's
// three shifted tiles stay in registers for the three rows that need them.  The
// 1 -> 16 layer takes the taps as the contracted index, its adjoint the
// channels.  The weight gradients are MFMA products over the pixels of a tile;
// the loss and Adam are plain VALU kernels.
#include "sp_internal.h"
#include "sp_reduce.h"

#include <algorithm>

namespace sp {

typedef float f4v __attribute__((ext_vector_type(4)));

constexpr int LF = 16;   // channels

__device__ __forceinline__ bool in_img(int h, int w, int H, int W) {
    return h >= 0 && h < H && w >= 0 && w < W;
}

// Quotient of a wave-uniform index; 32-bit arithmetic where the index allows it.
__device__ __forceinline__ unsigned long udiv(unsigned long n, unsigned d) {
    return n >> 32 ? n / d : (unsigned long)((unsigned)n / d);
}

// Buffer resource over n pixels of activations from p (reads past either end give
// 0, writes are dropped).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t act_pixels(const float* p, int n) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), (short)0, n * LF * 4, 0x00020000);
}

__device__ __forceinline__ float softplus(float d) {
    const double x = d;
    return (float)(x > 20.0 ? x : log1p(exp(x)));
}

// ---- 16 -> 16 correlation on MFMA --------------------------------------------
// out[b,h,w,j] = sum_{t, ci} in[b, h+dy_t, w+dx_t, ci] * K[j][ci][t], with
// K = W (TRANS = false) or K[j][ci][t] = W[ci][j][8 - t] (TRANS: the adjoint).
// If d != nullptr, out2 = softplus(d[j]) * out as well (formed here, not in a
// launch of its own: an apply at 512^2 107.5 -> 105.8 us).
//
// Bound: the MFMAs (36 of 32 cycles per tile of 16 pixels: 7.7 us at 512^2, 31 at
// 256 x 64^2) and the activations' traffic (27 us there at the copy rate); at
// 512^2 as much again goes into the launch, the weights' way to the lanes and
// the last stores.  What stood in between: 64-bit divisions for each tile (now
// one per strip, uniform), nine loads per tile (three, the next row's under
// way during a row's MFMAs), a wave's 36 weight loads of 64 cache lines each (now
// through LDS), rows shared across XCDs.  512^2: 25 -> 17 us; 256 x 64^2: 84 -> 48.
template <bool TRANS>
__global__ __launch_bounds__(256) void k_lp_conv_mid(int B, int H, int W, int S,
                                                     const float* __restrict__ in,
                                                     float* __restrict__ out,
                                                     const float* __restrict__ Wl,
                                                     const float* __restrict__ d,
                                                     float* __restrict__ out2,
                                                     const int* __restrict__ halt,
                                                     const int* __restrict__ run) {
    if (halt && *halt) return;
    if (run && !*run) return;
    const int lane = threadIdx.x & 63;
    const int i = lane & 15;     // A row (pixel) / B column (out channel)
    const int kq = lane >> 4;    // A column / B row within a group of 4 input channels
    const int wtiles = (W + 15) >> 4, hs = (H + S - 1) / S, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long ntasks = (long)B * hs * wtiles, nwaves = (long)gridDim.x * 4;
    // neighbouring strips on one XCD, whose L2 then serves the rows they share
    long task = ((long)(blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3)) * 4 + wave;
    // a task: columns tw .. of rows y0 .. y1 - 1 of an image; all uniform
    int tw, y0, y1, voff;
    size_t img;   // element of the image's first pixel
    f4v a[4][3];  // rows y - 1, y, y + 1 and, on its way, y + 2
    // the three shifted tiles of row y: channels 4 kq .. 4 kq + 3 of the pixel in one
    // 16-byte load each
    auto load = [&](int y, f4v (&v)[3]) {
        const int x0 = max(tw - 1, 0);
        const __amdgpu_buffer_rsrc_t row =
            act_pixels(in + img + ((ptrdiff_t)y * W + x0) * LF, y >= 0 && y < H ? min(W - x0, 18) : 0);
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
            v[dx] = __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(row, voff + (dx - 1) * LF * 4, 0, 0));
    };
    auto begin = [&] {
        const long br = (long)udiv((unsigned long)task, wtiles), b = (long)udiv((unsigned long)br, hs);
        tw = (int)(task - br * wtiles) * 16;
        y0 = (int)(br - b * hs) * S;
        y1 = min(H, y0 + S);
        img = (size_t)b * H * W * LF;
        voff = (((tw > 0 ? 1 : 0) + i) * LF + 4 * kq) * 4;   // from pixel max(tw - 1, 0)
        load(y0 - 1, a[0]);
        load(y0, a[1]);
        load(y0 + 1, a[2]);
    };
    if (task < ntasks) begin();   // on its way while the weights are staged
    // ws[t][lane][cg]: lane's weight of MFMA (t, cg), whose input channel is 4 kq + cg
    __shared__ float ws[9 * 64 * 4];
    for (int e = threadIdx.x; e < LF * LF * 9; e += 256) {
        const int t = e % 9, c1 = e / 9 % LF, c0 = e / (9 * LF);   // Wl[c0][c1][t]
        const int ci = TRANS ? c0 : c1, co = TRANS ? c1 : c0, tt = TRANS ? 8 - t : t;
        ws[(tt * 64 + (ci >> 2) * 16 + co) * 4 + (ci & 3)] = Wl[e];
    }
    __syncthreads();
    f4v wr[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) wr[t] = *reinterpret_cast<const f4v*>(&ws[(t * 64 + lane) * 4]);
    const float sc = d ? softplus(d[i]) : 0.0f;
    while (task < ntasks) {
        for (int y = y0; y < y1; y += 4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (y + u >= y1) break;
                if (y + u + 1 < y1) load(y + u + 2, a[(u + 3) & 3]);
                f4v acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int t = 0; t < 9; ++t) {
#pragma unroll
                    for (int cg = 0; cg < 4; ++cg)
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[(u + t / 3) & 3][t % 3][cg], wr[t][cg], acc, 0, 0, 0);
                }
                // lane holds D[4*(lane>>4) + r][lane & 15]: pixel tw + 4*kq + r, channel i
                const int off = (4 * kq * LF + i) * 4;
                auto put = [&](float* dst, float f) {
                    const __amdgpu_buffer_rsrc_t row = act_pixels(dst + img + ((size_t)(y + u) * W + tw) * LF, min(W - tw, 16));
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, acc[r] * f), row, off + r * LF * 4, 0, 0);
                };
                if (out) put(out, 1.0f);
                if (out2) put(out2, sc);
            }
        }
        task += nwaves;
        if (task < ntasks) begin();
    }
}

// ---- 1 -> 16 (first layer) and its adjoint 16 -> 1 ------------------------------
// out[b,h,w,co] = sum_t W1[co][t] * in[src(b), h+dy, w+dx]; src(b) = idx[b] if idx.
// On MFMA as well: 16 pixels x taps (three groups of four, the last three of them
// zero) by taps x 16 channels, so a pixel costs a lane three loads and the
// result leaves in whole cache lines.  Bound: the activations written (512^2,
// 17 MB: 17 us with a pixel per thread before, now 13; 256 x 64^2, 67 MB: 22, 17).
__global__ __launch_bounds__(256) void k_lp_conv_in(int B, int H, int W, int S, const float* __restrict__ in,
                                                    const int32_t* __restrict__ idx, int nsrc,
                                                    float* __restrict__ out,
                                                    const float* __restrict__ W1,
                                                    const int* __restrict__ halt,
                                                    const int* __restrict__ run) {
    if (halt && *halt) return;
    if (run && !*run) return;
    const int lane = threadIdx.x & 63, i = lane & 15, kq = lane >> 4;
    float wr[3];
    int dy[3], dx[3];
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        const int t = 4 * s + kq;   // (t >= 9: no tap)
        wr[s] = t < 9 ? W1[i * 9 + t] : 0.0f;
        dy[s] = t < 9 ? t / 3 - 1 : -(1 << 30);   // outside any image
        dx[s] = t % 3 - 1;
    }
    const int wtiles = (W + 15) >> 4, hs = (H + S - 1) / S, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long ntasks = (long)B * hs * wtiles;
    const long blk = (long)(blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);   // as k_lp_conv_mid
    for (long task = blk * 4 + wave; task < ntasks; task += (long)gridDim.x * 4) {
        const long br = (long)udiv((unsigned long)task, wtiles), b = (long)udiv((unsigned long)br, hs);
        const int tw = (int)(task - br * wtiles) * 16, y0 = (int)(br - b * hs) * S, y1 = min(H, y0 + S);
        const int src = idx ? min(max(idx[b], 0), nsrc - 1) : (int)b;
        const float* img = in + (size_t)src * H * W;
        for (int y = y0; y < y1; y += 4) {   // four rows' loads in flight
            float v[4][3];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
#pragma unroll
                for (int s = 0; s < 3; ++s) {
                    const bool ok = in_img(y + u + dy[s], tw + i + dx[s], H, W);
                    const float x = img[ok ? (y + u + dy[s]) * W + tw + i + dx[s] : 0];
                    v[u][s] = ok ? x : 0.0f;
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (y + u >= y1) break;
                f4v acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int s = 0; s < 3; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(v[u][s], wr[s], acc, 0, 0, 0);
                // lane holds pixel tw + 4 kq + r, channel i
                const __amdgpu_buffer_rsrc_t row = act_pixels(out + (((size_t)b * H + y + u) * W + tw) * LF, min(W - tw, 16));
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float f = acc[r];   // (a bit cast of the element itself takes element 0)
                    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, f), row,
                                                          ((4 * kq + r) * LF + i) * 4, 0, 0);
                }
            }
        }
    }
}

// out[b,h,w] = sum_co sum_t W1[co][t] * in[b, h-dy, w-dx, co]   (adjoint of
// k_lp_conv_in).  A workgroup makes 16 x 16 pixels: each of the 18 x 18 pixels
// around them is read once and multiplied by all taps on MFMA (16 pixels x 16
// channels by 16 channels x 9 taps), and the taps are summed through LDS.
// Bound: the activations read (a thread per pixel gathered each of its 9
// neighbours' 64 bytes through the vector L1: 512^2 13 -> 6 us, 256 x 64^2
// 25 -> 15).
constexpr int LP_OUT = 16, LP_OUTH = LP_OUT + 2;

__global__ __launch_bounds__(256) void k_lp_conv_out(unsigned ntile, int H, int W, const float* __restrict__ in,
                                                     float* __restrict__ out,
                                                     const float* __restrict__ W1,
                                                     const int* __restrict__ halt,
                                                     const int* __restrict__ run) {
    if (halt && *halt) return;
    if (run && !*run) return;
    constexpr int NP = LP_OUTH * LP_OUTH, NT = (NP + 15) / 16;
    __shared__ float s[NT * 16][9];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 15, kq = lane >> 4;
    const int tx = (W + LP_OUT - 1) / LP_OUT, ty = (H + LP_OUT - 1) / LP_OUT;
    f4v wr;   // channel 4 kq + cg, tap i
#pragma unroll
    for (int cg = 0; cg < 4; ++cg) wr[cg] = i < 9 ? W1[(4 * kq + cg) * 9 + i] : 0.0f;
    for (unsigned t0 = blockIdx.x; t0 < ntile; t0 += gridDim.x) {
        const unsigned b = t0 / (unsigned)(tx * ty), rem = t0 - b * (unsigned)(tx * ty);
        const int y0 = (int)(rem / (unsigned)tx) * LP_OUT, x0 = (int)(rem % (unsigned)tx) * LP_OUT;
        const float* img = in + (size_t)b * H * W * LF;
        constexpr int PW = (NT + 3) / 4;   // tiles per wave
        f4v a[PW];
#pragma unroll
        for (int q = 0; q < PW; ++q) {
            const int p = (4 * q + wave) * 16 + i;   // pixel of the 18 x 18
            const int y = y0 - 1 + p / LP_OUTH, x = x0 - 1 + p % LP_OUTH;
            const bool ok = p < NP && in_img(y, x, H, W);
            const f4v v = *reinterpret_cast<const f4v*>(img + (ok ? ((size_t)y * W + x) * LF : 0) + 4 * kq);
            a[q] = ok ? v : f4v{0.0f, 0.0f, 0.0f, 0.0f};
        }
        if (t0 != blockIdx.x) __syncthreads();   // the previous sums are done
#pragma unroll
        for (int q = 0; q < PW; ++q) {
            const int tile = 4 * q + wave;
            if (tile >= NT) break;
            f4v acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int cg = 0; cg < 4; ++cg) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[q][cg], wr[cg], acc, 0, 0, 0);
            // lane holds pixel 4 kq + r of the tile, tap i
            if (i < 9) {
#pragma unroll
                for (int r = 0; r < 4; ++r) s[tile * 16 + 4 * kq + r][i] = acc[r];
            }
        }
        __syncthreads();
        const int py = threadIdx.x / LP_OUT, px = threadIdx.x % LP_OUT;
        float sum = 0.0f;
#pragma unroll
        for (int t = 0; t < 9; ++t) sum += s[(py + 2 - t / 3) * LP_OUTH + px + 2 - t % 3][t];
        if (y0 + py < H && x0 + px < W) out[(size_t)b * H * W + (size_t)(y0 + py) * W + x0 + px] = sum;
    }
}

// out = scale[c] * in, channels-last
__global__ __launch_bounds__(256) void k_lp_scale(long n16, const float* __restrict__ in,
                                                  const float* __restrict__ scale,
                                                  float* __restrict__ out) {
    const long q = (long)blockIdx.x * 256 + threadIdx.x;
    if (q < n16) out[q] = in[q] * scale[q & (LF - 1)];
}

// softplus(d) and sigmoid(d) into sc[0..15], sg[0..15]
__global__ void k_lp_softplus(const float* __restrict__ d, float* __restrict__ sp_out,
                              float* __restrict__ sg_out) {
    const int c = threadIdx.x;
    if (c < LF) {
        sp_out[c] = softplus(d[c]);
        if (sg_out) sg_out[c] = (float)(1.0 / (1.0 + exp(-(double)d[c])));
    }
}

// ---- loss ---------------------------------------------------------------------
// One workgroup per sample b: nv = ||v||^2, lb = ||z - v||^2 / nv,
// e0 = (2 / B) (z - v) / nv; loss partial lb / B.
// Per sample b: loss over the pixels at least `margin` from every edge,
// e0 = d loss / dz (zero on the margin).
__global__ __launch_bounds__(256) void k_lp_loss(int B, int H, int W, int margin,
                                                 const float* __restrict__ z,
                                                 const float* __restrict__ v,
                                                 const int32_t* __restrict__ idx, int nsrc,
                                                 float* __restrict__ e0,
                                                 double* __restrict__ lpart) {
    __shared__ double red[4];
    const int b = blockIdx.x;
    const int HW = H * W;
    const float* vb = v + (size_t)(idx ? min(max(idx[b], 0), nsrc - 1) : b) * HW;
    const float* zb = z + (size_t)b * HW;
    auto inside = [&](int q) {
        const int y = q / W, x = q - (q / W) * W;
        return y >= margin && y < H - margin && x >= margin && x < W - margin;
    };
    double nv = 0.0;
    for (int q = threadIdx.x; q < HW; q += 256)
        if (inside(q)) nv += (double)vb[q] * (double)vb[q];
    nv = block_sum(nv, red);
    const double sc = nv > 0.0 ? 2.0 / ((double)B * nv) : 0.0;
    double r2 = 0.0;
    for (int q = threadIdx.x; q < HW; q += 256) {
        const double r = inside(q) ? (double)zb[q] - (double)vb[q] : 0.0;
        r2 += r * r;
        e0[(size_t)b * HW + q] = (float)(sc * r);
    }
    r2 = block_sum(r2, red);
    if (threadIdx.x == 0) lpart[b] = nv > 0.0 ? r2 / nv / (double)B : 0.0;
}

// ---- weight gradients ----------------------------------------------------------
// partial[blk][o][ci][t] = sum over the block's tiles' pixels p of G[p][o] *
// X[p + t][ci] (X zero outside the image).  G: [B][H][W][16]; X: [B][H][W][FI].
// A tile is 16 x 16 pixels of one image, staged in LDS; per tap t its share of
// dW_t is a [16 x 256] x [256 x FI] MFMA product over its pixels (FI = 1: one
// product with the taps as columns).  Wave w takes pixel columns 4 w .. 4 w + 3,
// the four pixels of an MFMA, down the 16 rows for all nine taps: a row's G and
// three shifted X are read from LDS once and serve nine MFMAs, the next two rows'
// taps included.  The sums of a wave's 64 pixels are float32 MFMA accumulators,
// those over tiles and waves float64.  Blocks go on to further tiles, the next
// one's loads under way during a tile's MFMAs.
// Bound: the MFMAs (31 us at 256 x 64^2) and the activations' traffic (27 us).
// Nine waves, one per tap, on one tile per block took 144 us: one wave of nine
// left its SIMD's share uneven, single floats were staged one load after
// another, and 4096 blocks' partials went to memory (now at most 512); 256 x 64^2,
// partial sums included: 180 -> 69 us; first layer 61 -> 26.
constexpr int WG_T = 16, WG_H = WG_T + 2;
constexpr int LP_WG_BLOCKS = 512;   // two per CU

template <int FI>
__global__ __launch_bounds__(256, 2) void k_lp_wgrad(int B, int H, int W, const float* __restrict__ G,
                                                     const float* __restrict__ X,
                                                     double* __restrict__ partial) {
    constexpr int NG = WG_T * WG_T * LF / 4, NX = WG_H * WG_H * FI, XV = FI == 1 ? 1 : 4;   // XV: floats per load of X
    constexpr int NTAP = FI == 1 ? 1 : 9;
    constexpr int PG = NG / 256, PX = (NX / XV + 255) / 256;   // loads per thread
    __shared__ __attribute__((aligned(16))) float lds[WG_T * WG_T * LF + NX];
    float* gs = lds;
    float* xs = lds + WG_T * WG_T * LF;
    const int lane = threadIdx.x & 63, i = lane & 15, kq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tx = (W + WG_T - 1) / WG_T, ty = (H + WG_T - 1) / WG_T;
    const unsigned ntile = (unsigned)B * tx * ty;
    f4v rg[PG], rx[FI == 1 ? 1 : PX];
    float rx1[FI == 1 ? PX : 1];
    // a tile and its X with a halo of one pixel to registers, zero outside the image
    auto fetch = [&](unsigned tile) {
        const unsigned b = tile / (unsigned)(tx * ty), rem = tile - b * (unsigned)(tx * ty);
        const int y0 = (int)(rem / (unsigned)tx) * WG_T, x0 = (int)(rem % (unsigned)tx) * WG_T;
        const float* gb = G + (size_t)b * H * W * LF;
        const float* xb = X + (size_t)b * H * W * FI;
#pragma unroll
        for (int q = 0; q < PG; ++q) {
            const int e = threadIdx.x + 256 * q, y = y0 + e / (WG_T * 4), x = x0 + e / 4 % WG_T;
            const bool ok = y < H && x < W;
            const f4v v = *reinterpret_cast<const f4v*>(gb + (ok ? ((size_t)y * W + x) * LF : 0) + 4 * (e & 3));
            rg[q] = ok ? v : f4v{0.0f, 0.0f, 0.0f, 0.0f};
        }
#pragma unroll
        for (int q = 0; q < PX; ++q) {
            const int e = threadIdx.x + 256 * q, px = e * XV / FI, y = y0 - 1 + px / WG_H, x = x0 - 1 + px % WG_H;
            const bool ok = px < WG_H * WG_H && in_img(y, x, H, W);
            if constexpr (FI == 1) {
                const float v = xb[ok ? (size_t)y * W + x : 0];
                rx1[q] = ok ? v : 0.0f;
            } else {
                const f4v v = *reinterpret_cast<const f4v*>(xb + (ok ? ((size_t)y * W + x) * FI : 0) + 4 * (e & 3));
                rx[q] = ok ? v : f4v{0.0f, 0.0f, 0.0f, 0.0f};
            }
        }
    };
    double sum[NTAP][4];
#pragma unroll
    for (int t = 0; t < NTAP; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) sum[t][r] = 0.0;
    unsigned tile = blockIdx.x;
    if (tile < ntile) fetch(tile);
    for (; tile < ntile; tile += gridDim.x) {
        __syncthreads();   // the previous tile's reads are done
#pragma unroll
        for (int q = 0; q < PG; ++q) *reinterpret_cast<f4v*>(gs + 4 * (threadIdx.x + 256 * q)) = rg[q];
#pragma unroll
        for (int q = 0; q < PX; ++q) {
            const int e = threadIdx.x + 256 * q;
            if (e * XV >= NX) break;
            if constexpr (FI == 1) xs[e] = rx1[q];
            else *reinterpret_cast<f4v*>(xs + 4 * e) = rx[q];
        }
        __syncthreads();
        if (tile + gridDim.x < ntile) fetch(tile + gridDim.x);
        f4v acc[NTAP];
#pragma unroll
        for (int t = 0; t < NTAP; ++t) acc[t] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
        const float* ga = gs + (4 * wave + kq) * LF + i;   // this lane's pixel of row 0: A[o = i][k = kq]
        if constexpr (FI == 1) {
            const int t = min(i, 8);
            const float* xa = xs + t / 3 * WG_H + 4 * wave + kq + t % 3;   // B[k = kq][tap = i]
#pragma unroll
            for (int y = 0; y < WG_T; ++y) {
                const float bv = i < 9 ? xa[y * WG_H] : 0.0f;
                acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(ga[y * WG_T * LF], bv, acc[0], 0, 0, 0);
            }
        } else {
            const float* xa = xs + (4 * wave + kq) * FI + i;   // B[k = kq][ci = i] of tap 0
            float bv[3][3];   // rows y .. y + 2 of the halo, three columns
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
                for (int dx = 0; dx < 3; ++dx) bv[y][dx] = xa[(y * WG_H + dx) * FI];
#pragma unroll
            for (int y = 0; y < WG_T; ++y) {
#pragma unroll
                for (int dx = 0; dx < 3; ++dx) bv[(y + 2) % 3][dx] = xa[((y + 2) * WG_H + dx) * FI];
                const float av = ga[y * WG_T * LF];
#pragma unroll
                for (int t = 0; t < 9; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv[(y + t / 3) % 3][t % 3], acc[t], 0, 0, 0);
            }
        }
#pragma unroll
        for (int t = 0; t < NTAP; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) sum[t][r] += (double)acc[t][r];
    }
    // the four waves' sums in wave order; a lane holds D[o = 4 kq + r][i]
    constexpr int NOUT = LF * FI * 9;
    double* red = reinterpret_cast<double*>(lds);
    static_assert(NOUT * 2 <= WG_T * WG_T * LF + NX, "LDS");
    for (int w = 0; w < 4; ++w) {
        __syncthreads();
        if (wave != w) continue;
#pragma unroll
        for (int t = 0; t < NTAP; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int o = 4 * kq + r, e = FI == 1 ? o * 9 + min(i, 8) : (o * LF + i) * 9 + t;
                if (FI != 1 || i < 9) red[e] = w ? red[e] + sum[t][r] : sum[t][r];
            }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < NOUT; e += 256) partial[(size_t)blockIdx.x * NOUT + e] = red[e];
}

// out[q] (+)= sum over the blocks' partials, float64 in a fixed order: 16 outputs
// per workgroup, 16 groups of threads over every 16th block each, then the groups.
__global__ __launch_bounds__(256) void k_lp_reduce(int nblk, int nout, const double* __restrict__ pa,
                                                   int accumulate, float* __restrict__ out) {
    __shared__ double red[256];
    const int c = threadIdx.x & 15, grp = threadIdx.x >> 4, q = blockIdx.x * 16 + c;
    double s = 0.0;
#pragma unroll 8
    for (int k = grp; k < nblk; k += 16) s += pa[(size_t)k * nout + q];
    red[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x >= 16) return;
    double t = 0.0;
    for (int g = 0; g < 16; ++g) t += red[g * 16 + c];
    out[q] = (float)(accumulate ? (double)out[q] + t : t);
}

// gd partials: part[blk][c] = sum over the block's pixels of E[p][c] * A[p][c]
__global__ __launch_bounds__(256) void k_lp_gd_part(long npix, const float* __restrict__ E,
                                                    const float* __restrict__ A,
                                                    double* __restrict__ part) {
    __shared__ double red[256];
    const int c = threadIdx.x & (LF - 1);
    const int lane_pix = threadIdx.x >> 4;   // 16 pixels per pass
    double s = 0.0;
    for (long p = (long)blockIdx.x * 16 + lane_pix; p < npix; p += (long)gridDim.x * 16)
        s += (double)E[p * LF + c] * (double)A[p * LF + c];
    red[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x < LF) {
        double t = 0.0;
        for (int k = 0; k < 16; ++k) t += red[k * LF + threadIdx.x];
        part[(size_t)blockIdx.x * LF + threadIdx.x] = t;
    }
}

// 64 groups of threads per channel sum strided blocks, then the groups are added
// in order.
__global__ __launch_bounds__(1024) void k_lp_gd_final(int nblk, const double* __restrict__ part,
                                                      const float* __restrict__ sg,
                                                      float* __restrict__ gd) {
    __shared__ double red[1024];
    const int c = threadIdx.x & (LF - 1), grp = threadIdx.x >> 4;
    double s = 0.0;
#pragma unroll 8
    for (int k = grp; k < nblk; k += 64) s += part[(size_t)k * LF + c];
    red[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x < LF) {
        double t = 0.0;
        for (int g = 0; g < 64; ++g) t += red[g * LF + threadIdx.x];
        gd[threadIdx.x] = (float)(t * (double)sg[threadIdx.x]);
    }
}

__global__ __launch_bounds__(256) void k_lp_adam(int n, float* __restrict__ theta,
                                                 float* __restrict__ m, float* __restrict__ v,
                                                 const float* __restrict__ g, double lr, double b1,
                                                 double b2, double eps, double c1, double c2) {
    const int q = blockIdx.x * 256 + threadIdx.x;
    if (q >= n) return;
    const double gq = g[q];
    const double mq = b1 * (double)m[q] + (1.0 - b1) * gq;
    const double vq = b2 * (double)v[q] + (1.0 - b2) * gq * gq;
    m[q] = (float)mq;
    v[q] = (float)vq;
    theta[q] = (float)((double)theta[q] - lr * (mq / c1) / (sqrt(vq / c2) + eps));
}

// ---- launchers ------------------------------------------------------------------
static inline unsigned nblk(long n, int per) { return (unsigned)((n + per - 1) / per); }

// Strips of S rows by 16 columns (k_lp_conv_mid), a wave each in turn: as many
// rows, up to 16, as leave two strips per SIMD (256 x 64^2 with 4, 8, 16, 32 rows:
// 58, 58, 48, 48 us; 512^2 with 2, 4, 8, 16: 22, 18, 17, 18).
struct ConvGrid {
    int S;
    unsigned grid;
};
static ConvGrid conv_grid(int B, int H, int W) {
    const long wt = (W + 15) / 16;
    const int S = (int)std::min<long>(16, std::max<long>(1, (long)B * H * wt / 2048));
    const long tasks = (long)B * ((H + S - 1) / S) * wt;
    return {S, (std::min(nblk(tasks, 4), 2048u) + 7) / 8 * 8};
}

void lp_conv_mid(hipStream_t st, bool trans, int B, int H, int W, const float* in, float* out,
                 const float* Wl, const float* d, float* out2, const int* halt, const int* run) {
    const ConvGrid cg = conv_grid(B, H, W);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(cg.grid), dim3(256), 0, st, B, H, W, cg.S, in, out, Wl, d, out2, halt, run);
    };
    if (trans) go(k_lp_conv_mid<true>);
    else go(k_lp_conv_mid<false>);
}

void lp_conv_in(hipStream_t st, int B, int H, int W, const float* in, const int32_t* idx, int nsrc,
                float* out, const float* W1, const int* halt, const int* run) {
    const ConvGrid cg = conv_grid(B, H, W);
    hipLaunchKernelGGL(k_lp_conv_in, dim3(cg.grid), dim3(256), 0, st, B, H, W, cg.S, in, idx, nsrc, out, W1, halt,
                       run);
}

__global__ __launch_bounds__(256) void k_lp_gather(int B, int HW, const float* __restrict__ src,
                                                   const int32_t* __restrict__ idx, int nsrc,
                                                   float* __restrict__ dst) {
    const long q = (long)blockIdx.x * 256 + threadIdx.x;
    if (q >= (long)B * HW) return;
    const int b = (int)(q / HW);
    const int s = min(max(idx[b], 0), nsrc - 1);
    dst[q] = src[(size_t)s * HW + (q - (long)b * HW)];
}

void lp_gather(hipStream_t st, int B, int HW, const float* src, const int32_t* idx, int nsrc, float* dst) {
    hipLaunchKernelGGL(k_lp_gather, dim3(nblk((long)B * HW, 256)), dim3(256), 0, st, B, HW, src, idx,
                       nsrc, dst);
}

void lp_conv_out(hipStream_t st, int B, int H, int W, const float* in, float* out, const float* W1,
                 const int* halt, const int* run) {
    // (a launch holds fewer than 2^32 threads: images of less than a tile take several
    // tiles per workgroup beyond 2^22 of them)
    const unsigned g = (unsigned)((long)B * ((H + LP_OUT - 1) / LP_OUT) * ((W + LP_OUT - 1) / LP_OUT));
    hipLaunchKernelGGL(k_lp_conv_out, dim3(std::min(g, 1u << 22)), dim3(256), 0, st, g, H, W, in, out, W1, halt, run);
}

void lp_scale(hipStream_t st, long npix, const float* in, const float* scale, float* out) {
    hipLaunchKernelGGL(k_lp_scale, dim3(nblk(npix * LF, 256)), dim3(256), 0, st, npix * LF, in, scale, out);
}

void lp_softplus(hipStream_t st, const float* d, float* sp_out, float* sg_out) {
    hipLaunchKernelGGL(k_lp_softplus, dim3(1), dim3(64), 0, st, d, sp_out, sg_out);
}

void lp_loss(hipStream_t st, int B, int H, int W, int margin, const float* z, const float* v,
             const int32_t* idx, int nsrc, float* e0, double* lpart) {
    hipLaunchKernelGGL(k_lp_loss, dim3(B), dim3(256), 0, st, B, H, W, margin, z, v, idx, nsrc, e0,
                       lpart);
}

int lp_wgrad_blocks(int B, int H, int W) {
    return (int)std::min<long>(LP_WG_BLOCKS, (long)B * ((H + WG_T - 1) / WG_T) * ((W + WG_T - 1) / WG_T));
}

void lp_wgrad(hipStream_t st, int fi, int B, int H, int W, const float* G, const float* X, double* partial) {
    const unsigned g = (unsigned)lp_wgrad_blocks(B, H, W);
    if (fi == LF) hipLaunchKernelGGL(k_lp_wgrad<LF>, dim3(g), dim3(256), 0, st, B, H, W, G, X, partial);
    else hipLaunchKernelGGL(k_lp_wgrad<1>, dim3(g), dim3(256), 0, st, B, H, W, G, X, partial);
}

void lp_reduce(hipStream_t st, int nb, int nout, const double* pa, bool accumulate, float* out) {
    hipLaunchKernelGGL(k_lp_reduce, dim3(nout / 16), dim3(256), 0, st, nb, nout, pa, accumulate ? 1 : 0, out);
}

int lp_gd_blocks() { return 2048; }

void lp_gd(hipStream_t st, long npix, const float* E, const float* A, double* part, const float* sg,
           float* gd) {
    hipLaunchKernelGGL(k_lp_gd_part, dim3(lp_gd_blocks()), dim3(256), 0, st, npix, E, A, part);
    hipLaunchKernelGGL(k_lp_gd_final, dim3(1), dim3(1024), 0, st, lp_gd_blocks(), part, sg, gd);
}

void lp_adam(hipStream_t st, int n, float* theta, float* m, float* v, const float* g, double lr,
             double b1, double b2, double eps, int step) {
    const double c1 = 1.0 - pow(b1, step), c2 = 1.0 - pow(b2, step);
    hipLaunchKernelGGL(k_lp_adam, dim3(nblk(n, 256)), dim3(256), 0, st, n, theta, m, v, g, lr, b1, b2,
                       eps, c1, c2);
}

}  // namespace sp
