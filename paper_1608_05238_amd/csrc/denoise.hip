// denoise.hip -- BF16 matrix-core kernels of the learned denoiser: 3x3
// convolution (stride 1, zero padding 1) as an implicit GEMM on the gfx950
// MFMA units with FP32 accumulation, its weight gradient and the gradient of
// the bias.  The input gradient is the forward kernel applied to the flipped,
// transposed weights.
//
// Layouts (channels last, so that the GEMM's reduction index -- the input
// channel -- is contiguous): BF16 activations [n][h][w][c] (raw 16-bit
// patterns) with c a multiple of 8; packed weights [co][3][3][ci] BF16; outputs
// FP32 [n][h][w][co].  FP32 activations may have any strides.
//
// The layers are narrow (24-160 channels), so at full resolution they are
// bound by memory, and everything is arranged to read an activation once, as
// the program holds it, and write the result once: FP32 operands are rounded
// to BF16 on their way into LDS (one pass less over memory than a conversion
// before), the BF16 copy the backward pass keeps is written beside, and the
// bias gradient is summed from the same loads as the weight gradient.
//
// MFMA lane layout of v_mfma_f32_16x16x32_bf16 (checked on the device):
// A[m][k] with m = lane % 16, k = 8 (lane / 16) + i, i = 0..7; B[k][n] with
// n = lane % 16, k = 8 (lane / 16) + i; D[m][n] with n = lane % 16,
// m = 4 (lane / 16) + i, i = 0..3.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "mcrad.h"
#include "denoise.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kCiC = 32;                   // input channels per chunk (the MFMA K)
constexpr int kTCo = 64;                   // output channels per workgroup
constexpr int kTY = 8, kTX = 8;            // output pixels per workgroup
constexpr int kHY = kTY + 2, kHX = kTX + 2;
constexpr int kXVec = kHY * kHX * (kCiC / 8);      // 16-byte vectors of a halo tile chunk (400)
constexpr int kThreads = 256;
constexpr int kXPer = (kXVec + kThreads - 1) / kThreads;   // 2

__device__ __forceinline__ u32x4 load16(const uint16_t *p) {
    return *reinterpret_cast<const u32x4 *>(p);
}

// BF16 element q (0..7) of a 16-byte vector
__device__ __forceinline__ uint16_t half_of(const u32x4 v, int q) {
    return (uint16_t)(v[q >> 1] >> (16 * (q & 1)));
}

__device__ __forceinline__ uint16_t to_bf16(float v) { return __builtin_bit_cast(uint16_t, (__bf16)v); }

__device__ __forceinline__ u32x4 pack8(const float (&v)[8]) {
    u32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        r[i] = (uint32_t)to_bf16(v[2 * i]) | ((uint32_t)to_bf16(v[2 * i + 1]) << 16);
    return r;
}

// ---- forward
// GEMM: D[co][p] = sum_{tap, ci} W[co][tap][ci] X[p + off(tap)][ci] for the
// pixels p of a TS x TS block of one image and 16 MB output channels.  A chunk
// of U units of 8 input channels (all of them, if they are few) is staged in
// LDS: the block's halo tile and the weights.  The sums run over groups of 32
// channels (four units, one MFMA; units past the last read a unit of zeros)
// and, within a group, over the nine taps.
// A workgroup of four waves takes block after block; the next block's (or
// chunk's) activations are in flight in registers while it multiplies, and the
// weights stay in LDS if there is one chunk.  LDS rows are an odd number of
// 16-byte units, so the 16 lanes of a read fall into different banks.
// 16 x 256^2 pixels, 48 -> 48 channels, with the BF16 copy: 125 us = 4.1 TB/s
// of what it must read and write; a conversion pass (26 us) and a kernel that
// staged 32-channel chunks of 8 x 8 blocks without overlap took 366 us.
// FP32 channels last, 16-byte rows; FP32, any strides; BF16; or FP32 channels
// last put together on the way in: the 2 x 2 maxima of a map twice the size, or
// a map of half the size repeated, and the channels of a second map after it
enum : int { X_F32 = 0, X_STRIDED = 1, X_BF16 = 2, X_MIX = 3 };

struct ConvArgs {
    const void *x;
    long long sn, sc, sh, sw;   // element strides (X_STRIDED)
    const uint16_t *w;          // [co][9][cip]
    const float *bias;
    float *y;
    uint16_t *xb;               // BF16 copy of x, [n][h][w][cip], or NULL
    int ci, cip, co, h, wd;
    int tiles_x, tiles_y, n_tiles;
    int units, nchunk;          // units of 8 channels a chunk; chunks
    // X_MIX: x is [n][hs][ws][ca]; x2 [n][h][w][ci - ca] or NULL (maxima)
    const float *x2;
    int hs, ws, ca, vec;        // vec: whole units of each map's channels
};

constexpr int kUnitsMax = 6;    // units a chunk may have
constexpr int kUnetLevels = 8, kUnetLayers = 4 * kUnetLevels - 2;   // of a network in one call
constexpr int kUnetOutMax = 512;                                    // its first width (LDS of k_unet_out)

constexpr int halo_units(int ts) { return ((ts + 2) * (ts + 2) * kUnitsMax + kThreads - 1) / kThreads; }

size_t conv_lds(int ts, int mb, int units) {
    return ((size_t)(ts + 2) * (ts + 2) * (units | 1) + (size_t)16 * mb * ((9 * units) | 1) + 1) * 16;
}

// The larger, NaN if either is (as a maximum pool)
__device__ __forceinline__ float max_nan(float a, float b) { return a > b || a != a ? a : b; }

// Eight channels from ch on of a pixel of X_MIX.
__device__ __forceinline__ void mixed8(const ConvArgs &A, int img, int yy, int xx, int ch, float (&v)[8]) {
    const float *x = (const float *)A.x;
    if (!A.x2) {
        const int y = 2 * yy, c = 2 * xx;
        const float *p = x + (((size_t)img * A.hs + y) * A.ws + c) * A.ca + ch;
        const size_t right = c + 1 < A.ws ? A.ca : 0, down = y + 1 < A.hs ? (size_t)A.ws * A.ca : 0;
        if (A.vec) {
#pragma unroll
            for (int i = 0; i < 8; i += 4) {
                const f32x4 a = *(const f32x4 *)(p + i), b = *(const f32x4 *)(p + right + i);
                const f32x4 e = *(const f32x4 *)(p + down + i), g = *(const f32x4 *)(p + down + right + i);
#pragma unroll
                for (int k = 0; k < 4; ++k) v[i + k] = max_nan(max_nan(a[k], b[k]), max_nan(e[k], g[k]));
            }
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (ch + i < A.ci) v[i] = max_nan(max_nan(p[i], p[right + i]), max_nan(p[down + i], p[down + right + i]));
        }
        return;
    }
    const float *p = x + (((size_t)img * A.hs + (yy >> 1)) * A.ws + (xx >> 1)) * A.ca + ch;
    const float *q = A.x2 + (((size_t)img * A.h + yy) * A.wd + xx) * (A.ci - A.ca) + (ch - A.ca);
    if (A.vec) {
        const f32x4 *r = (const f32x4 *)(ch < A.ca ? p : q);
        const f32x4 a = r[0], b = r[1];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[i] = a[i];
            v[4 + i] = b[i];
        }
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (ch + i < A.ci) v[i] = ch + i < A.ca ? p[i] : q[i];
    }
}

template <int TS, int MB, int KIND, bool RELU>
__global__ void __launch_bounds__(kThreads, 2) k_conv3x3(ConvArgs A) {
    constexpr int HS = TS + 2, NPX = HS * HS, NB = TS * TS / 64;   // halo side and pixels; 16-pixel blocks a wave
    constexpr int NJ = halo_units(TS);                             // activation units a thread stages
    extern __shared__ u32x4 lds[];
    const int U = A.units, pu = U | 1, pw = (9 * U) | 1;
    // several chunks (of 4 units) of 8 x 8 blocks: weights are prefetched too, these units a thread
    // (16 x 16 blocks have no registers left for them)
    constexpr int WJ = TS == 8 ? (16 * MB * 37 + kThreads - 1) / kThreads : 1;
    u32x4 *xs = lds;                       // [NPX][pu]
    u32x4 *ws = lds + NPX * pu;            // [16 MB][pw]
    u32x4 *zero = ws + 16 * MB * pw;        // a unit of zeros
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, kg = lane >> 4, l16 = lane & 15;
    const int co0 = blockIdx.y * 16 * MB;
    const u32x4 none = {0u, 0u, 0u, 0u};
    if (tid == 0) *zero = none;

    // the staged units of this thread: pixel of the halo and channel group
    int upix[NJ];   // pixel << 8 | group; -1: none
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int v = tid + j * kThreads;
        const int pix = KIND == X_STRIDED ? v % NPX : v / U, part = KIND == X_STRIDED ? v / NPX : v - (v / U) * U;
        upix[j] = v < NPX * U ? pix << 8 | part : -1;
    }
    float rf[KIND == X_BF16 ? 1 : NJ][8];
    u32x4 rb[KIND == X_BF16 ? NJ : 1];
    auto fetch = [&](int t, int c) {        // block t, chunk c
        const int per = A.tiles_x * A.tiles_y, img = t / per, tt = t - img * per;
        const int ty = (tt / A.tiles_x) * TS - 1, tx = (tt % A.tiles_x) * TS - 1;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int pix = upix[j] >> 8, ch = (c * U + (upix[j] & 255)) * 8;
            const int hy = pix / HS, yy = ty + hy, xx = tx + pix - hy * HS;
            const bool in = upix[j] >= 0 && (unsigned)yy < (unsigned)A.h && (unsigned)xx < (unsigned)A.wd;
            if constexpr (KIND == X_BF16) {
                rb[j] = none;
                if (in && ch < A.cip)
                    rb[j] = load16((const uint16_t *)A.x + (((size_t)img * A.h + yy) * A.wd + xx) * A.cip + ch);
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) rf[j][i] = 0.f;
                if constexpr (KIND == X_MIX) {
                    if (in && ch < A.ci) mixed8(A, img, yy, xx, ch, rf[j]);
                } else if (KIND == X_F32) {
                    if (in && ch < A.ci) {
                        const f32x4 *p = (const f32x4 *)((const float *)A.x + (((size_t)img * A.h + yy) * A.wd + xx) * A.ci + ch);
                        const f32x4 a = p[0], b = p[1];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            rf[j][i] = a[i];
                            rf[j][4 + i] = b[i];
                        }
                    }
                } else if (in) {
                    const float *p = (const float *)A.x + img * A.sn + yy * A.sh + xx * A.sw + ch * A.sc;
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        if (ch + i < A.ci) rf[j][i] = p[i * A.sc];
                }
            }
        }
    };
    auto stash = [&](int t, int c) {        // what fetch(t, c) loaded
        const int per = A.tiles_x * A.tiles_y, img = t / per, tt = t - img * per;
        const int ty = (tt / A.tiles_x) * TS - 1, tx = (tt % A.tiles_x) * TS - 1;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            if (upix[j] < 0) continue;
            const int pix = upix[j] >> 8, part = upix[j] & 255;
            u32x4 v;
            if constexpr (KIND == X_BF16) v = rb[j];
            else v = pack8(rf[j]);
            xs[pix * pu + part] = v;
            if (KIND != X_BF16 && A.xb && blockIdx.y == 0) {
                const int hy = pix / HS, hx = pix - hy * HS, ch = (c * U + part) * 8;
                if (hy >= 1 && hy <= TS && hx >= 1 && hx <= TS && ty + hy < A.h && tx + hx < A.wd && ch < A.cip)
                    *(u32x4 *)(A.xb + (((size_t)img * A.h + ty + hy) * A.wd + tx + hx) * A.cip + ch) = v;
            }
        }
    };
    auto weight = [&](int v, int c) {       // unit v of chunk c's weights in LDS
        const int row = v / pw, g = v - row * pw, tap = g / U, ch = (c * U + g - tap * U) * 8;
        return co0 + row < A.co && tap < 9 && ch < A.cip ? load16(A.w + ((size_t)(co0 + row) * 9 + tap) * A.cip + ch) : none;
    };
    const int wunits = 16 * MB * pw;
    auto weights = [&](int c) {
#pragma unroll 4
        for (int v = tid; v < wunits; v += kThreads) ws[v] = weight(v, c);
    };
    u32x4 rw[WJ];
    auto fetch_w = [&](int c) {
#pragma unroll
        for (int j = 0; j < WJ; ++j) rw[j] = weight(std::min(tid + j * kThreads, wunits - 1), c);
    };
    auto stash_w = [&] {
#pragma unroll
        for (int j = 0; j < WJ; ++j)
            if (tid + j * kThreads < wunits) ws[tid + j * kThreads] = rw[j];
    };
    // first pixel of each of this lane's 16-pixel blocks in the halo tile
    int base[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int p = (wave * NB + b) * 16 + l16;
        base[b] = ((p / TS) * HS + p % TS) * pu;
    }
    f32x4 acc[MB][NB];
    int t = blockIdx.x, c = 0;
    if (t >= A.n_tiles) return;
    fetch(t, 0);
    weights(0);
    stash(t, 0);
    __syncthreads();
    for (;;) {
        int t1 = t, c1 = c + 1;             // what comes next
        if (c1 == A.nchunk) {
            c1 = 0;
            t1 = t + gridDim.x;
        }
        if (t1 < A.n_tiles) {
            fetch(t1, c1);
            if (TS == 8 && A.nchunk > 1) fetch_w(c1);
        }
        if (c == 0) {
#pragma unroll
            for (int a = 0; a < MB; ++a)
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        for (int q = 0; 4 * q < U; ++q) {   // a group of 32 channels: this lane's unit is 4 q + kg
            const int u = 4 * q + kg;
            const bool in = u < U;
            const u32x4 *wr = in ? ws + l16 * pw + u : zero;
            const int wrow = in ? 16 * pw : 0, wtap = in ? U : 0, xcol = in ? pu : 0;
            const u32x4 *xr[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) xr[b] = in ? xs + base[b] + u : zero;
#pragma unroll
            for (int tap = 0; tap < 9; ++tap) {
                bf16x8 fa[MB], fb[NB];
#pragma unroll
                for (int a = 0; a < MB; ++a) fa[a] = __builtin_bit_cast(bf16x8, wr[a * wrow + tap * wtap]);
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    fb[b] = __builtin_bit_cast(bf16x8, xr[b][(tap / 3 * HS + tap % 3) * xcol]);
#pragma unroll
                for (int a = 0; a < MB; ++a)
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[a], fb[b], acc[a][b], 0, 0, 0);
            }
        }
        __syncthreads();
        if (c1 == 0) {                      // the block is done: D[m][n], m = 4 kg + i (channel), n = l16 (pixel)
            const int per = A.tiles_x * A.tiles_y, img = t / per, tt = t - img * per;
            const int ty = (tt / A.tiles_x) * TS, tx = (tt % A.tiles_x) * TS;
            const bool vec = (A.co & 3) == 0;
#pragma unroll
            for (int a = 0; a < MB; ++a) {
                const int co = co0 + 16 * a + 4 * kg;
                f32x4 bias = {0.f, 0.f, 0.f, 0.f};
                if (A.bias)
#pragma unroll
                    for (int i = 0; i < 4; ++i) bias[i] = co + i < A.co ? A.bias[co + i] : 0.f;
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const int p = (wave * NB + b) * 16 + l16, gy = ty + p / TS, gx = tx + p % TS;
                    if (gy >= A.h || gx >= A.wd || co >= A.co) continue;
                    float *dst = A.y + (((size_t)img * A.h + gy) * A.wd + gx) * A.co + co;
                    f32x4 v = acc[a][b] + bias;
                    if constexpr (RELU)
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] = v[i] <= 0.f ? 0.f : v[i];   // (NaN stays)
                    if (vec) {
                        *(f32x4 *)dst = v;
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (co + i < A.co) dst[i] = v[i];
                    }
                }
            }
        }
        if (t1 >= A.n_tiles) break;
        stash(t1, c1);
        if (A.nchunk > 1) {
            if (TS == 8) stash_w();
            else weights(c1);
        }
        __syncthreads();
        t = t1;
        c = c1;
    }
}

// Weights [co][ci][3][3] FP32 as the forward kernel reads them: BF16
// [co][9][cip] (zeros past ci), or with `flip` those of the input gradient,
// [ci][9][cop], both spatial directions reversed.
__device__ __forceinline__ void pack_weights(const float *w, uint16_t *out, int co, int ci, int inner, int flip) {
    const int rows = flip ? ci : co, cols = flip ? co : ci;
    const size_t total = (size_t)rows * 9 * inner;
    for (size_t v = blockIdx.x * (size_t)blockDim.x + threadIdx.x; v < total; v += (size_t)gridDim.x * blockDim.x) {
        const int line = (int)(total >> 32 ? v / (size_t)inner : (uint32_t)v / (uint32_t)inner);
        const int col = (int)(v - (size_t)line * inner);
        const int row = line / 9, tap = line - row * 9;
        float x = 0.f;
        if (col < cols) x = flip ? w[((size_t)col * ci + row) * 9 + 8 - tap] : w[((size_t)row * ci + col) * 9 + tap];
        out[v] = to_bf16(x);
    }
}

__global__ void k_pack_weights(const float *w, uint16_t *out, int co, int ci, int inner, int flip) {
    pack_weights(w, out, co, ci, inner, flip);
}

// All layers of a network in one launch (blockIdx.y: the layer).
struct PackList {
    const float *w[kUnetLayers];
    uint16_t *out[kUnetLayers];
    int co[kUnetLayers], ci[kUnetLayers];
};

__global__ void k_pack_layers(PackList P) {
    const int l = blockIdx.y;
    pack_weights(P.w[l], P.out[l], P.co[l], P.ci[l], (P.ci[l] + 7) & ~7, 0);
}

// ---- output layer of the network: y = x + W a + b per pixel
// a: FP32 [pixels][c]; x, y: FP32 of any strides.  A workgroup stages 64 pixels
// of a in LDS, transposed; each of its waves then takes every fourth group of
// four output channels, a pixel a lane.  Bound by memory (one read of a and x,
// one write of y); 3 x 256^2 pixels, 24 -> 33 channels: 30 us, 2.3 TB/s (as a
// matrix product, two sums and a copy: 95 us).
struct Strided {
    long long n, c, h, w;
};

__global__ void __launch_bounds__(kThreads) k_unet_out(const float *a, const float *w, const float *b, const float *x, Strided sx,
                                                       float *y, Strided sy, int c, int channels, int h, int wd, int pixels) {
    extern __shared__ u32x4 lds[];
    float *as = (float *)lds;   // [c][65]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int p0 = blockIdx.x * 64, np = min(64, pixels - p0);
#pragma unroll 4
    for (int e = tid; e < np * c; e += kThreads) {
        const int px = e / c, ch = e - px * c;
        as[ch * 65 + px] = a[(size_t)p0 * c + e];
    }
    __syncthreads();
    const int p = p0 + min(lane, np - 1), img = p / (h * wd), q = p - img * (h * wd), yy = q / wd, xx = q - yy * wd;
    const float *xp = x + img * sx.n + yy * sx.h + xx * sx.w;
    float *yp = y + img * sy.n + yy * sy.h + xx * sy.w;
    for (int o0 = 4 * wave; o0 < channels; o0 += 16) {
        float acc[4] = {0.f, 0.f, 0.f, 0.f}, xv[4];
        int row[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            row[i] = min(o0 + i, channels - 1) * c;
            xv[i] = xp[min(o0 + i, channels - 1) * sx.c];   // on its way during the sums
        }
        auto add = [&](int k) {
            const float v = as[k * 65 + lane];
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] = fmaf(w[row[i] + k], v, acc[i]);
        };
        int k = 0;
        for (; k + 8 <= c; k += 8)   // (the weights come as scalar loads of eight)
#pragma unroll
            for (int j = 0; j < 8; ++j) add(k + j);
        for (; k < c; ++k) add(k);
        if (lane < np)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (o0 + i < channels) yp[(o0 + i) * sy.c] = xv[i] + (acc[i] + b[o0 + i]);
    }
}

// ---- weight gradient from BF16 operands, for C callers that hold those and no
// scratch memory (dn_conv3x3_wgrad); a layer's own is below
// gw[co][tap][ci] = sum_p gy[p][co] x[p + off(tap)][ci].  GEMM per tap with
// M = output channels, N = input channels, K = pixels.  A workgroup holds 64
// output channels x one chunk of 32 input channels x the nine taps and runs
// over a slice of 8 x 8 pixel tiles; per tile it stages gy transposed
// ([co][pixel]) and the input halo transposed into three copies shifted by
// kx ([kx][ci][row][8 pixels]), so that a lane's eight consecutive pixels of
// either operand are one aligned 16-byte LDS read.  Each wave owns 16 output
// channels: per 32-pixel K step its A fragment serves 2 x 9 MFMAs.  Partial
// sums over the pixel slices are added with FP32 atomics.
constexpr int kGP = 64 + 8;                            // LDS pitch (BF16) of a gy^T row: 64 pixels
constexpr int kGVec = kTY * kTX * (kTCo / 8);          // 16-byte vectors of the gy tile (512)
constexpr int kXTRow = kTX;                            // BF16 per [kx][ci][row] run: 8 pixels
constexpr size_t kWgradLds = ((size_t)kTCo * kGP + 3ull * kCiC * kHY * kXTRow) * sizeof(uint16_t);

__global__ void __launch_bounds__(kThreads) k_conv3x3_wgrad(const uint16_t *__restrict__ x,
                                                            const uint16_t *__restrict__ gy, float *__restrict__ gw,
                                                            int Ci, int Co, int H, int W, int tiles_x, int tiles_y,
                                                            int n_tiles, int tiles_per_slice) {
    extern __shared__ uint16_t smem[];
    uint16_t *sg = smem;                      // [64 co][kGP]
    uint16_t *sxT = smem + kTCo * kGP;        // [3 kx][32 ci][kHY rows][8 px]
    const int c0 = blockIdx.x * kCiC, co0 = blockIdx.y * kTCo;
    const int t0 = blockIdx.z * tiles_per_slice, t1 = min(n_tiles, t0 + tiles_per_slice);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int kg = lane >> 4, l16 = lane & 15;
    f32x4 acc[9][2];
#pragma unroll
    for (int tap = 0; tap < 9; ++tap)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[tap][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int t = t0; t < t1; ++t) {
        const int img = t / (tiles_x * tiles_y), tt = t - img * tiles_x * tiles_y;
        const int ty0 = (tt / tiles_x) * kTY, tx0 = (tt % tiles_x) * kTX;
        // gy tile, transposed: 512 vectors of 8 output channels of one pixel
        u32x4 rg[kGVec / kThreads];
#pragma unroll
        for (int j = 0; j < kGVec / kThreads; ++j) {
            const int v = tid + j * kThreads;
            const int p = v >> 3, part = v & 7;
            const int py = p >> 3, px = p & 7;
            const int yy = ty0 + py, xx = tx0 + px, co = co0 + 8 * part;
            u32x4 val = {0u, 0u, 0u, 0u};
            if (yy < H && xx < W && co < Co) val = load16(gy + (((size_t)img * H + yy) * W + xx) * Co + co);
            rg[j] = val;
        }
        // input halo: 400 vectors of 8 input channels of one pixel
        u32x4 rx[kXPer];
#pragma unroll
        for (int j = 0; j < kXPer; ++j) {
            const int v = tid + j * kThreads;
            u32x4 val = {0u, 0u, 0u, 0u};
            if (v < kXVec) {
                const int pix = v >> 2, part = v & 3;
                const int hy = pix / kHX, hx = pix - hy * kHX;
                const int yy = ty0 + hy - 1, xx = tx0 + hx - 1, c = c0 + 8 * part;
                if (yy >= 0 && yy < H && xx >= 0 && xx < W && c < Ci)
                    val = load16(x + (((size_t)img * H + yy) * W + xx) * Ci + c);
            }
            rx[j] = val;
        }
        __syncthreads();   // the previous tile's fragments have been read
#pragma unroll
        for (int j = 0; j < kGVec / kThreads; ++j) {
            const int v = tid + j * kThreads;
            const int p = v >> 3, part = v & 7;
#pragma unroll
            for (int q = 0; q < 8; ++q) sg[(8 * part + q) * kGP + p] = half_of(rg[j], q);
        }
#pragma unroll
        for (int j = 0; j < kXPer; ++j) {
            const int v = tid + j * kThreads;
            if (v >= kXVec) continue;
            const int pix = v >> 2, part = v & 3;
            const int hy = pix / kHX, hx = pix - hy * kHX;
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) {
                const int px = hx - kx;   // this halo column is pixel px of the copy shifted by kx
                if (px < 0 || px >= kTX) continue;
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    sxT[((kx * kCiC + 8 * part + q) * kHY + hy) * kXTRow + px] = half_of(rx[j], q);
            }
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < 2; ++s) {   // K steps: tile rows 4s .. 4s + 3, lane group kg takes row 4s + kg
            const int row = 4 * s + kg;
            const bf16x8 fa = __builtin_bit_cast(bf16x8, load16(sg + (16 * wave + l16) * kGP + 8 * row));
#pragma unroll
            for (int tap = 0; tap < 9; ++tap) {
                const int ky = tap / 3, kx = tap - 3 * ky;
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    const bf16x8 fb = __builtin_bit_cast(
                        bf16x8, load16(sxT + ((kx * kCiC + 16 * b + l16) * kHY + row + ky) * kXTRow));
                    acc[tap][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fb, acc[tap][b], 0, 0, 0);
                }
            }
        }
    }
    // D[m][n]: m = 4 kg + i (output channel within the wave's 16), n = l16 (+16 b) input channel
#pragma unroll
    for (int tap = 0; tap < 9; ++tap)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int ci = c0 + 16 * b + l16;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int co = co0 + 16 * wave + 4 * kg + i;
                if (co < Co && ci < Ci && acc[tap][b][i] != 0.f)
                    atomicAdd(gw + ((size_t)co * 9 + tap) * Ci + ci, acc[tap][b][i]);
            }
        }
}

// ---- weight and bias gradient from what a layer holds
// As above, from the BF16 copy of x and the FP32 upstream gradient itself.
// GEMM per tap with M = output channels, N = input channels, K = pixels.  Both
// operands lie in LDS as they lie in memory, [pixel][channel]; the transpose
// to eight consecutive pixels of a channel per lane is done by the LDS read
// (ds_read_b64_tr_b16: 16 lanes read four pixels x 16 channels and each gets
// its channel's four pixels, checked on the device), so one copy of the halo
// tile serves the nine taps.  A workgroup holds 16 MB output x 16 NB input
// channels x nine taps, the (tap, block of input channels) pairs dealt to its
// four waves, and runs over every gridDim.x-th 16 x 8 pixel block, the next
// one in flight in registers.  The workgroups' parts are written to a scratch
// buffer and added in order by k_wgrad_sum: the result does not depend on
// timing.  16 x 256^2 pixels, 48 x 48 channels: 90 us, the sum 9 us; from a
// converted copy (26 us), with transposing stores to LDS, three shifted copies
// of the halo and atomics 267 us, and 86 us for the bias gradient.
//
// A sum of many FP32 terms in one register loses a rounding a term, so every
// kWFold blocks the sums go into a second set and start again.  48 x 48 channels
// leave no registers for one (248 of 256): there a workgroup takes at most
// kWBlocks blocks.  Relative error against 64 bits, 16 x 256^2 pixels: 224 x 128
// channels (455 blocks a workgroup) 1.5e-6 -> 2.0e-7, the bias 5.5e-7 -> 1.6e-7;
// 96 x 96 channels 5.0e-7 -> 3.3e-7.  896 -> 870 us for the former.
constexpr int kWY = 8, kWX = 16, kWHalo = (kWY + 2) * (kWX + 2);
constexpr int kWFold = 8, kWBlocks = 32;
constexpr bool wgrad_folds(int mb, int nb) { return mb * nb < 9; }

struct WgradArgs {
    const uint16_t *x;     // [n][h][w][cip]
    const float *gy;       // [n][h][w][co]
    float *part;           // [slices][co tiles][ci tiles][9 NB][MB][256]
    float *bpart;          // [slices][co tiles][16 MB]
    int cip, co, h, wd, tiles_x, tiles_y, n_tiles;
};

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ s16x4 read_tr(const uint16_t *p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)p);
}

template <int MB, int NB, bool VEC>
__global__ void __launch_bounds__(kThreads, 2) k_wgrad(WgradArgs A) {
    constexpr int UX = 2 * NB, UG = 2 * MB, PX = UX | 1, PG = UG | 1;   // units of 8 channels, and LDS pitches
    constexpr int GT = kThreads / UG * UG;                              // threads that stage gy: each keeps its channels
    constexpr int XJ = (kWHalo * UX + kThreads - 1) / kThreads, GJ = (kWX * kWY * UG + GT - 1) / GT;
    constexpr int PW = (9 * NB + 3) / 4;                                // (tap, block) pairs of a wave
    constexpr bool FOLD = wgrad_folds(MB, NB);
    __shared__ u32x4 xs[kWHalo * PX], gs[kWX * kWY * PG];
    __shared__ float bs[GT * 8];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c0 = blockIdx.z * 16 * NB, co0 = blockIdx.y * 16 * MB;
    const u32x4 none = {0u, 0u, 0u, 0u};
    const int gpart = tid % UG, gco = co0 + 8 * gpart;
    u32x4 rx[XJ];
    float rg[GJ][8], bsum[8], btot[FOLD ? 8 : 1];
#pragma unroll
    for (int i = 0; i < 8; ++i) bsum[i] = 0.f;
    if constexpr (FOLD)
#pragma unroll
        for (int i = 0; i < 8; ++i) btot[i] = 0.f;
    auto fetch = [&](int t) {
        const int per = A.tiles_x * A.tiles_y, img = t / per, tt = t - img * per;
        const int ty = (tt / A.tiles_x) * kWY, tx = (tt % A.tiles_x) * kWX;
#pragma unroll
        for (int j = 0; j < XJ; ++j) {
            const int v = tid + j * kThreads, pix = v / UX, part = v - pix * UX;
            const int hy = pix / (kWX + 2), yy = ty + hy - 1, xx = tx + pix - hy * (kWX + 2) - 1, ch = c0 + 8 * part;
            rx[j] = none;
            if (v < kWHalo * UX && (unsigned)yy < (unsigned)A.h && (unsigned)xx < (unsigned)A.wd && ch < A.cip)
                rx[j] = load16(A.x + (((size_t)img * A.h + yy) * A.wd + xx) * A.cip + ch);
        }
#pragma unroll
        for (int j = 0; j < GJ; ++j) {
            const int pix = tid / UG + j * (GT / UG), yy = ty + pix / kWX, xx = tx + pix % kWX;
#pragma unroll
            for (int i = 0; i < 8; ++i) rg[j][i] = 0.f;
            if (tid < GT && pix < kWX * kWY && yy < A.h && xx < A.wd && gco < A.co) {
                const float *p = A.gy + (((size_t)img * A.h + yy) * A.wd + xx) * A.co + gco;
                if constexpr (VEC) {
                    const f32x4 a = *(const f32x4 *)p, b = *(const f32x4 *)(p + 4);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        rg[j][i] = a[i];
                        rg[j][4 + i] = b[i];
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        if (gco + i < A.co) rg[j][i] = p[i];
                }
            }
        }
    };
    auto stash = [&]() {
#pragma unroll
        for (int j = 0; j < XJ; ++j) {
            const int v = tid + j * kThreads, pix = v / UX, part = v - pix * UX;
            if (v < kWHalo * UX) xs[pix * PX + part] = rx[j];
        }
        if (tid < GT) {
#pragma unroll
            for (int j = 0; j < GJ; ++j) {
                const int pix = tid / UG + j * (GT / UG);
                if (pix < kWX * kWY) gs[pix * PG + gpart] = pack8(rg[j]);
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {   // (zeros past the block)
                float v = rg[0][i];
#pragma unroll
                for (int j = 1; j < GJ; ++j) v += rg[j][i];
                bsum[i] += v;
            }
        }
    };
    f32x4 acc[PW][MB], tot[FOLD ? PW : 1][FOLD ? MB : 1];
#pragma unroll
    for (int i = 0; i < PW; ++i)
#pragma unroll
        for (int a = 0; a < MB; ++a) {
            acc[i][a] = f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (FOLD) tot[i][a] = acc[i][a];
        }
    auto fold = [&] {
        if constexpr (FOLD) {
#pragma unroll
            for (int i = 0; i < PW; ++i)
#pragma unroll
                for (int a = 0; a < MB; ++a) {
                    tot[i][a] += acc[i][a];
                    acc[i][a] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                btot[i] += bsum[i];
                bsum[i] = 0.f;
            }
        }
    };
    // a read of four pixels x 16 channels per 16 lanes: lane's pixel 4 (lane / 16) + (lane % 16) / 4, channels 4 (lane % 4)
    const int rpix = 4 * (lane >> 4) + ((lane & 15) >> 2), rch = 4 * (lane & 3);
    const uint16_t *gr = (const uint16_t *)gs + rpix * PG * 8 + rch;
    const uint16_t *xr[PW];
#pragma unroll
    for (int i = 0; i < PW; ++i) {
        const int p = min(wave + 4 * i, 9 * NB - 1), tap = p / NB, nb = p - tap * NB;   // (a wave's last pair may repeat)
        xr[i] = (const uint16_t *)xs + ((tap / 3) * (kWX + 2) + tap % 3 + rpix) * PX * 8 + 16 * nb + rch;
    }
    int t = blockIdx.x;
    if (t < A.n_tiles) {
        fetch(t);
        stash();
    }
    __syncthreads();
    for (int k = 1; t < A.n_tiles; t += gridDim.x, ++k) {
        const bool next = t + (int)gridDim.x < A.n_tiles;
        if (next) fetch(t + gridDim.x);
#pragma unroll
        for (int s = 0; s < kWY / 2; ++s) {   // 32 pixels: rows 2 s and 2 s + 1
            s16x8 fa[MB];
#pragma unroll
            for (int a = 0; a < MB; ++a) {
                const uint16_t *q = gr + (2 * s * kWX) * PG * 8 + 16 * a;
                fa[a] = __builtin_shufflevector(read_tr(q), read_tr(q + kWX * PG * 8), 0, 1, 2, 3, 4, 5, 6, 7);
            }
#pragma unroll
            for (int i = 0; i < PW; ++i) {
                const uint16_t *q = xr[i] + (2 * s * (kWX + 2)) * PX * 8;
                const s16x8 fb =
                    __builtin_shufflevector(read_tr(q), read_tr(q + (kWX + 2) * PX * 8), 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
                for (int a = 0; a < MB; ++a)
                    acc[i][a] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fa[a]),
                                                                        __builtin_bit_cast(bf16x8, fb), acc[i][a], 0, 0, 0);
            }
        }
        __syncthreads();
        if (FOLD && k % kWFold == 0) fold();
        if (next) stash();
        __syncthreads();
    }
    if constexpr (FOLD) {
        fold();
#pragma unroll
        for (int i = 0; i < PW; ++i)
#pragma unroll
            for (int a = 0; a < MB; ++a) acc[i][a] = tot[i][a];
#pragma unroll
        for (int i = 0; i < 8; ++i) bsum[i] = btot[i];
    }
    float *out = A.part + (((size_t)blockIdx.x * gridDim.y + blockIdx.y) * gridDim.z + blockIdx.z) * (9 * NB * MB * 256);
#pragma unroll
    for (int i = 0; i < PW; ++i)
        if (wave + 4 * i < 9 * NB)
#pragma unroll
            for (int a = 0; a < MB; ++a) *(f32x4 *)(out + ((wave + 4 * i) * MB + a) * 256 + 4 * lane) = acc[i][a];
    if (blockIdx.z == 0) {
        if (tid < GT)
#pragma unroll
            for (int i = 0; i < 8; ++i) bs[tid * 8 + i] = bsum[i];
        __syncthreads();
        if (tid < 16 * MB) {   // channel tid: unit tid / 8 of the threads that staged it
            double v = 0.;
            for (int k = tid >> 3; k < GT; k += UG) v += bs[k * 8 + (tid & 7)];
            A.bpart[((size_t)blockIdx.x * gridDim.y + blockIdx.y) * (16 * MB) + tid] = (float)v;
        }
    }
}

// gw[co][ci][3][3] and gb[co] from the slices' parts.  A lane takes a value, the
// sixteen waves of a workgroup share its slices (so a load is of 64
// consecutive values), and the first adds their sums in order; the sums over
// slices are FP64 (rounding is then that of the parts: relative error of the
// bias gradient of 16 x 256^2 pixels 3e-8 of values of one sign, 9e-8 of both).  Bound by the parts' bytes and, with
// few values, by latency: 512 slices of 48 x 48 channels, 42 MB, 9 us (24
// with a value's slices in consecutive lanes).
constexpr int kSumWaves = 16;

__global__ void __launch_bounds__(64 * kSumWaves) k_wgrad_sum(const float *part, const float *bpart, float *gw, float *gb,
                                                              int slices, int ty, int tz, int mb, int nb, int co, int ci) {
    __shared__ double s_sum[kSumWaves][64];
    const int frag = 9 * nb * mb * 256, bt = ty * 16 * mb;   // a workgroup's 64 values are of one tile
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long long total = (long long)ty * tz * frag, v = blockIdx.x * 64ll + lane;
    const bool bias = v >= total;
    const size_t step = bias ? (size_t)bt : (size_t)total;
    const float *src = bias ? bpart + (v - total) : part + v;
    double sum = 0.;
    if (v < total + bt)
#pragma unroll 8
        for (int k = wave; k < slices; k += kSumWaves) sum += src[(size_t)k * step];
    s_sum[wave][lane] = sum;
    __syncthreads();
    if (wave != 0 || v >= total + bt) return;
#pragma unroll
    for (int w = 1; w < kSumWaves; ++w) sum += s_sum[w][lane];
    if (!bias) {
        const int tile = blockIdx.x / (frag / 64), e = (int)(v - (long long)tile * frag), pair = e / (mb * 256), a = e / 256 - pair * mb, l = (e & 255) >> 2;
        const int c = (tile / tz) * 16 * mb + 16 * a + 4 * (l >> 4) + (e & 3);
        const int k = (tile % tz) * 16 * nb + 16 * (pair % nb) + (l & 15);
        if (c < co && k < ci) gw[((size_t)c * ci + k) * 9 + pair / nb] = (float)sum;
    } else if (v - total < co && gb) {
        gb[v - total] = (float)sum;
    }
}

__global__ void k_zero_f32(float *p, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0.f;
}

bool dims_ok(int n, int ci, int co, int h, int w) {
    if (n < 1 || ci < 1 || co < 1 || h < 1 || w < 1) return false;
    const long long tiles = (long long)n * ((h + kTY - 1) / kTY) * ((w + kTX - 1) / kTX);
    const long long P = (long long)n * h * w;
    return P <= (1ll << 30) && tiles < (1ll << 31) && ci <= (1 << 16) && co <= (1 << 16);
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

mc_status set_lds(const void *fn, size_t bytes) {
    return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) == hipSuccess
               ? MC_OK
               : MC_ERR_DEVICE;
}

// ---- plans
using ConvFn = void (*)(ConvArgs);
using WgradFn = void (*)(WgradArgs);

template <int TS, int KIND, bool RELU>
ConvFn conv_of(int mb) {
    return mb == 1   ? k_conv3x3<TS, 1, KIND, RELU>
           : mb == 2 ? k_conv3x3<TS, 2, KIND, RELU>
           : mb == 3 ? k_conv3x3<TS, 3, KIND, RELU>
                     : k_conv3x3<TS, 4, KIND, RELU>;
}

template <int TS>
ConvFn conv_fn(int mb, int kind, bool relu) {
    if (kind == X_MIX) return conv_of<TS, X_MIX, true>(mb);
    if (kind == X_BF16) return conv_of<TS, X_BF16, false>(mb);
    if (kind == X_F32) return relu ? conv_of<TS, X_F32, true>(mb) : conv_of<TS, X_F32, false>(mb);
    return relu ? conv_of<TS, X_STRIDED, true>(mb) : conv_of<TS, X_STRIDED, false>(mb);
}

// Blocks of 16 channels per workgroup: the count that pads `c` channels least,
// the largest of those.
int blocks_for(int c, int most) {
    int best = 1, pad = 1 << 30;
    for (int b = 1; b <= most; ++b) {
        const int p = (c + 16 * b - 1) / (16 * b) * b;
        if (p <= pad) {
            pad = p;
            best = b;
        }
    }
    return best;
}

// relu: negative results become zero (kinds X_F32, X_STRIDED, and X_MIX always)
mc_status run_conv(ConvArgs A, int kind, int n, hipStream_t s, bool relu = false) {
    // 16 x 16 pixel blocks and all output channels up to 64 in a workgroup read
    // least (16 x 256^2 pixels, 48 -> 48: 117 us; 8 x 8 blocks 151; 32 channels
    // a workgroup 141).  With less than two workgroups a CU, 32 channels each
    // (16 x 64^2, 64 -> 64: 18 us, with 64 channels 23; 3 x 128^2: 17 and 21).
    // With less than one a CU then, 8 x 8 blocks, and fewer channels until
    // every CU has one (3 x 64^2, 48 -> 48: 8.3 us, 16 x 16 blocks 10.6; 3 x 32^2,
    // 64 -> 64: 6.3 against 12.8, with 64 channels 11.5; 3 x 8^2, 128 -> 128:
    // 8.8 against 20.5, with 64 channels 16.1).
    const int mb0 = blocks_for(A.co, 4);
    int ts = 16, mb = mb0;
    auto groups = [&](int t, int m) {
        return (long long)n * ((A.h + t - 1) / t) * ((A.wd + t - 1) / t) * ((A.co + 16 * m - 1) / (16 * m));
    };
    if (groups(16, mb) < 512) mb = std::min(mb, 2);
    if (groups(16, mb) < 256) {
        ts = 8;
        for (mb = mb0; mb > 1 && groups(8, mb) < 256;) --mb;
    }
    const int most = mb >= 4 ? 4 : kUnitsMax;   // chunks that leave room for two workgroups a CU
    const int total = A.cip / 8;
    A.units = total <= most ? total : 4;        // several chunks: whole groups of 32 channels
    A.nchunk = (total + A.units - 1) / A.units;
    A.tiles_x = (A.wd + ts - 1) / ts;
    A.tiles_y = (A.h + ts - 1) / ts;
    const long long tiles = (long long)n * A.tiles_x * A.tiles_y;
    const int gco = (A.co + 16 * mb - 1) / (16 * mb);
    if (tiles >= (1ll << 31) || gco > 65535) return MC_ERR_UNSUPPORTED;
    A.n_tiles = (int)tiles;
    const size_t lds = conv_lds(ts, mb, A.units);
    const ConvFn fn = ts == 16 ? conv_fn<16>(mb, kind, relu) : conv_fn<8>(mb, kind, relu);
    const mc_status st = set_lds(reinterpret_cast<const void *>(fn), lds);
    if (st != MC_OK) return st;
    // two workgroups a CU, each taking several blocks: the weights are staged
    // once and the next block's loads overlap the products
    const long long most_groups = std::max(1, (ts == 16 ? 2 : 4) * 256 / gco);
    const long long rounds = (tiles + most_groups - 1) / most_groups;
    const unsigned gx = (unsigned)((tiles + rounds - 1) / rounds);
    hipLaunchKernelGGL(fn, dim3(gx, (unsigned)gco), dim3(kThreads), lds, s, A);
    return hipGetLastError() == hipSuccess ? MC_OK : MC_ERR_DEVICE;
}

// Sets the FP32 input of a convolution; returns how it is read.
int f32_input(ConvArgs &A, const float *x, const int64_t *strides, int ci, int h, int w) {
    A.x = x;
    A.sn = strides[0];
    A.sc = strides[1];
    A.sh = strides[2];
    A.sw = strides[3];
    A.ci = ci;
    A.cip = (ci + 7) & ~7;
    A.h = h;
    A.wd = w;
    // whole units of eight channels, rows of 16 bytes: two 16-byte loads a unit
    const bool vec = (ci & 7) == 0 && aligned16(x) && A.sc == 1 && A.sw == ci && A.sh == (int64_t)w * ci &&
                     A.sn == (int64_t)h * w * ci;
    return vec ? X_F32 : X_STRIDED;
}

// A network's layers and where their data lie in the scratch buffer.
struct UnetPlan {
    int levels, layers;
    int h[kUnetLevels], w[kUnetLevels];
    int ci[kUnetLayers], co[kUnetLayers];
    size_t map[kUnetLevels], hidden, packed[kUnetLayers], bytes;
};

bool unet_plan(UnetPlan &P, int channels, int levels, const int32_t *widths, int n, int h, int w) {
    if (channels < 1 || levels < 1 || levels > kUnetLevels || widths[0] > kUnetOutMax) return false;
    P.levels = levels;
    P.layers = 4 * levels - 2;
    size_t off = 0, hidden = 0;
    auto take = [&](size_t b) {
        const size_t at = off;
        off += (b + 255) & ~(size_t)255;
        return at;
    };
    for (int i = 0; i < levels; ++i) {
        P.h[i] = i ? (P.h[i - 1] + 1) / 2 : h;
        P.w[i] = i ? (P.w[i - 1] + 1) / 2 : w;
        if (widths[i] < 1 || !dims_ok(n, i ? widths[i - 1] : channels, widths[i], P.h[i], P.w[i])) return false;
        const size_t b = (size_t)n * P.h[i] * P.w[i] * widths[i] * sizeof(float);
        P.map[i] = take(b);
        hidden = std::max(hidden, b);
        P.ci[2 * i] = i ? widths[i - 1] : channels;
        P.co[2 * i] = P.ci[2 * i + 1] = P.co[2 * i + 1] = widths[i];
    }
    for (int i = levels - 2, l = 2 * levels; i >= 0; --i, l += 2) {
        P.ci[l] = widths[i + 1] + widths[i];
        P.co[l] = P.ci[l + 1] = P.co[l + 1] = widths[i];
        if (!dims_ok(n, P.ci[l], P.co[l], P.h[i], P.w[i])) return false;
    }
    P.hidden = take(hidden);
    for (int l = 0; l < P.layers; ++l) P.packed[l] = take((size_t)P.co[l] * 9 * ((P.ci[l] + 7) & ~7) * sizeof(uint16_t));
    P.bytes = off;
    return true;
}

template <int MB, bool VEC>
WgradFn wgrad_of(int nb) {
    return nb == 1 ? k_wgrad<MB, 1, VEC> : nb == 2 ? k_wgrad<MB, 2, VEC> : k_wgrad<MB, 3, VEC>;
}

WgradFn wgrad_fn(int mb, int nb, bool vec) {
    if (vec) return mb == 1 ? wgrad_of<1, true>(nb) : mb == 2 ? wgrad_of<2, true>(nb) : wgrad_of<3, true>(nb);
    return mb == 1 ? wgrad_of<1, false>(nb) : mb == 2 ? wgrad_of<2, false>(nb) : wgrad_of<3, false>(nb);
}

struct WgradPlan {
    int mb, nb, ty, tz, slices;
    size_t part_floats() const { return (size_t)slices * ty * tz * 9 * nb * mb * 256; }
    size_t bias_floats() const { return (size_t)slices * ty * 16 * mb; }
    long long sum_blocks() const { return ((long long)ty * tz * 9 * nb * mb * 256 + (long long)ty * 16 * mb + 63) / 64; }
};

// Two workgroups a CU over all channel tiles, no more than there are blocks; up
// to 48 x 48 channels each (more would not fit the registers beside the next
// block's loads).  More workgroups where one that cannot fold would take too many
// blocks (96 x 96 channels, 16 x 256^2 pixels: 275 us, 232 with 64 blocks each; 48 x
// 32 channels each, which fold, 351; sums stored between blocks spill, and take
// 268 and, with 48 x 48 channels, 91 for 74).
WgradPlan wgrad_plan(int n, int ci, int co, int h, int w) {
    WgradPlan P;
    P.mb = blocks_for(co, 3);
    P.nb = blocks_for(ci, 3);
    P.ty = (co + 16 * P.mb - 1) / (16 * P.mb);
    P.tz = (ci + 16 * P.nb - 1) / (16 * P.nb);
    const long long tiles = (long long)n * ((w + kWX - 1) / kWX) * ((h + kWY - 1) / kWY);
    const long long most = std::max<long long>(1, 512 / ((long long)P.ty * P.tz));
    long long rounds = (tiles + most - 1) / most;
    if (!wgrad_folds(P.mb, P.nb)) {   // whole multiples of the workgroups that fit at once
        const long long times = (rounds + kWBlocks - 1) / kWBlocks;
        rounds = (rounds + times - 1) / times;
    }
    P.slices = (int)((tiles + rounds - 1) / rounds);
    return P;
}

}  // namespace

extern "C" {

mc_status dn_conv3x3_fwd(const uint16_t *x_d, const uint16_t *w_d, const float *bias_d, float *y_d, int n, int ci,
                         int co, int h, int w, void *stream) {
    if (!x_d || !w_d || !y_d || !dims_ok(n, ci, co, h, w) || (ci & 7) || !aligned16(x_d) || !aligned16(w_d) ||
        ((co & 3) == 0 && !aligned16(y_d)))
        return MC_ERR_INVALID_ARG;
    ConvArgs A{};
    A.x = x_d;
    A.w = w_d;
    A.bias = bias_d;
    A.y = y_d;
    A.ci = A.cip = ci;
    A.co = co;
    A.h = h;
    A.wd = w;
    return run_conv(A, X_BF16, n, reinterpret_cast<hipStream_t>(stream));
}

mc_status dn_conv3x3_f32(const float *x_d, const int64_t *strides, const uint16_t *w_d, const float *bias_d, float *y_d,
                         uint16_t *xb_d, int n, int ci, int co, int h, int w, void *stream) {
    if (!x_d || !strides || !w_d || !y_d || !dims_ok(n, ci, co, h, w) || !aligned16(w_d) ||
        (xb_d && !aligned16(xb_d)) || ((co & 3) == 0 && !aligned16(y_d)))
        return MC_ERR_INVALID_ARG;
    ConvArgs A{};
    const int kind = f32_input(A, x_d, strides, ci, h, w);
    A.w = w_d;
    A.bias = bias_d;
    A.y = y_d;
    A.xb = xb_d;
    A.co = co;
    return run_conv(A, kind, n, reinterpret_cast<hipStream_t>(stream));
}

mc_status dn_pack_weights(const float *w_d, uint16_t *out_d, int co, int ci, int flip, void *stream) {
    if (!w_d || !out_d || co < 1 || ci < 1 || co > (1 << 16) || ci > (1 << 16) || (flip != 0 && flip != 1))
        return MC_ERR_INVALID_ARG;
    const int inner = ((flip ? co : ci) + 7) & ~7;
    const long long total = (long long)(flip ? ci : co) * 9 * inner;
    hipLaunchKernelGGL(k_pack_weights, dim3((unsigned)std::min<long long>((total + 255) / 256, 1024)), dim3(256), 0,
                       reinterpret_cast<hipStream_t>(stream), w_d, out_d, co, ci, inner, flip);
    return hipGetLastError() == hipSuccess ? MC_OK : MC_ERR_DEVICE;
}

size_t dn_unet_bytes(int channels, int levels, const int32_t *widths, int n, int h, int w) {
    UnetPlan P;
    return widths && unet_plan(P, channels, levels, widths, n, h, w) ? P.bytes : 0;
}

// One call and 24 launches for six levels instead of ~110: what is between two
// convolutions (ReLU, maxima, repetition, joining channels) is done where one
// writes or the next reads, and the weights of all layers are packed at once.
// Three 256^2 maps of 33 channels, widths 24 to 128: 990 us (bound by the host's
// launches, ~270 us of it passes over memory) -> 424 us, of which 75 are the
// caller's normalisation; bound now by the small layers' latency (8 - 17 us each
// from 64^2 down) and by memory at 256^2.
mc_status dn_unet_forward(int channels, int levels, const int32_t *widths, const float *const *weights,
                          const float *const *biases, const float *out_w, const float *out_b, const float *x_d,
                          const int64_t *x_strides, float *y_d, const int64_t *y_strides, void *scratch_d,
                          size_t scratch_bytes, int n, int h, int w, void *stream) {
    UnetPlan P;
    if (!widths || !weights || !biases || !out_w || !out_b || !x_d || !x_strides || !y_d || !y_strides)
        return MC_ERR_INVALID_ARG;
    if (!unet_plan(P, channels, levels, widths, n, h, w)) return MC_ERR_UNSUPPORTED;
    if (!scratch_d || scratch_bytes < P.bytes || !aligned16(scratch_d)) return MC_ERR_WORKSPACE;
    for (int l = 0; l < P.layers; ++l)
        if (!weights[l] || !biases[l]) return MC_ERR_INVALID_ARG;
    const hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    char *base = static_cast<char *>(scratch_d);
    PackList pk{};
    for (int l = 0; l < P.layers; ++l) {
        pk.w[l] = weights[l];
        pk.out[l] = reinterpret_cast<uint16_t *>(base + P.packed[l]);
        pk.co[l] = P.co[l];
        pk.ci[l] = P.ci[l];
    }
    hipLaunchKernelGGL(k_pack_layers, dim3(64, (unsigned)P.layers), dim3(256), 0, s, pk);
    auto map = [&](int i) { return reinterpret_cast<float *>(base + P.map[i]); };
    float *hidden = reinterpret_cast<float *>(base + P.hidden);
    // layer l at level i, from A's input
    auto conv = [&](ConvArgs A, int kind, int l, int i, float *y) {
        A.w = pk.out[l];
        A.bias = biases[l];
        A.y = y;
        A.co = P.co[l];
        A.h = P.h[i];
        A.wd = P.w[i];
        A.ci = P.ci[l];
        A.cip = (P.ci[l] + 7) & ~7;
        return run_conv(A, kind, n, s, true);
    };
    auto second = [&](int l, int i) {   // hidden -> the level's map
        ConvArgs A{};
        const int64_t c = P.ci[l], st[4] = {c * P.w[i] * P.h[i], 1, c * P.w[i], c};
        const int kind = f32_input(A, hidden, st, P.ci[l], P.h[i], P.w[i]);
        return conv(A, kind, l, i, map(i));
    };
    for (int i = 0; i < levels; ++i) {
        ConvArgs A{};
        int kind = X_MIX;
        if (i == 0) {
            kind = f32_input(A, x_d, x_strides, channels, h, w);
        } else {
            A.x = map(i - 1);
            A.hs = P.h[i - 1];
            A.ws = P.w[i - 1];
            A.ca = widths[i - 1];
            A.vec = (A.ca & 7) == 0;
        }
        mc_status st = conv(A, kind, 2 * i, i, hidden);
        if (st == MC_OK) st = second(2 * i + 1, i);
        if (st != MC_OK) return st;
    }
    for (int i = levels - 2, l = 2 * levels; i >= 0; --i, l += 2) {
        ConvArgs A{};
        A.x = map(i + 1);
        A.x2 = map(i);
        A.hs = P.h[i + 1];
        A.ws = P.w[i + 1];
        A.ca = widths[i + 1];
        A.vec = (A.ca & 7) == 0 && (widths[i] & 7) == 0;
        mc_status st = conv(A, X_MIX, l, i, hidden);
        if (st == MC_OK) st = second(l + 1, i);   // over the map that was read
        if (st != MC_OK) return st;
    }
    const int pixels = n * h * w;
    const size_t lds = (size_t)widths[0] * 65 * sizeof(float);
    const mc_status st = set_lds(reinterpret_cast<const void *>(k_unet_out), lds);
    if (st != MC_OK) return st;
    const Strided sx{x_strides[0], x_strides[1], x_strides[2], x_strides[3]};
    const Strided sy{y_strides[0], y_strides[1], y_strides[2], y_strides[3]};
    hipLaunchKernelGGL(k_unet_out, dim3((unsigned)((pixels + 63) / 64)), dim3(kThreads), lds, s, map(0), out_w, out_b, x_d, sx,
                       y_d, sy, widths[0], channels, h, w, pixels);
    return hipGetLastError() == hipSuccess ? MC_OK : MC_ERR_DEVICE;
}

size_t dn_conv3x3_grads_bytes(int n, int ci, int co, int h, int w) {
    if (!dims_ok(n, ci, co, h, w)) return 0;
    const WgradPlan P = wgrad_plan(n, ci, co, h, w);
    return P.ty > 65535 || P.tz > 65535 || P.sum_blocks() >= (1ll << 31) ? 0 : P.part_floats() * sizeof(float) + P.bias_floats() * sizeof(float);
}

mc_status dn_conv3x3_grads(const uint16_t *xb_d, const float *gy_d, float *gw_d, float *gb_d, void *scratch_d,
                           size_t scratch_bytes, int n, int ci, int co, int h, int w, void *stream) {
    if (!xb_d || !gy_d || !gw_d || !dims_ok(n, ci, co, h, w) || !aligned16(xb_d) || (reinterpret_cast<uintptr_t>(gy_d) & 3))
        return MC_ERR_INVALID_ARG;
    const size_t need = dn_conv3x3_grads_bytes(n, ci, co, h, w);
    if (!need) return MC_ERR_UNSUPPORTED;
    if (!scratch_d || scratch_bytes < need || !aligned16(scratch_d)) return MC_ERR_WORKSPACE;
    const WgradPlan P = wgrad_plan(n, ci, co, h, w);
    const hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    WgradArgs A{};
    A.x = xb_d;
    A.gy = gy_d;
    A.part = static_cast<float *>(scratch_d);
    A.bpart = A.part + P.part_floats();
    A.cip = (ci + 7) & ~7;
    A.co = co;
    A.h = h;
    A.wd = w;
    A.tiles_x = (w + kWX - 1) / kWX;
    A.tiles_y = (h + kWY - 1) / kWY;
    A.n_tiles = n * A.tiles_x * A.tiles_y;
    const bool vec = (co & 7) == 0 && aligned16(gy_d);
    wgrad_fn(P.mb, P.nb, vec)<<<dim3(P.slices, P.ty, P.tz), dim3(kThreads), 0, s>>>(A);
    hipLaunchKernelGGL(k_wgrad_sum, dim3((unsigned)P.sum_blocks()), dim3(64 * kSumWaves), 0, s, A.part, A.bpart, gw_d, gb_d, P.slices,
                       P.ty, P.tz, P.mb, P.nb, co, ci);
    return hipGetLastError() == hipSuccess ? MC_OK : MC_ERR_DEVICE;
}

mc_status dn_conv3x3_wgrad(const uint16_t *x_d, const uint16_t *gy_d, float *gw_d, int n, int ci, int co, int h, int w,
                           void *stream) {
    if (!x_d || !gy_d || !gw_d || !dims_ok(n, ci, co, h, w) || (ci & 7) || (co & 7) || !aligned16(x_d) ||
        !aligned16(gy_d))
        return MC_ERR_INVALID_ARG;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const size_t nw = (size_t)co * 9 * ci;
    hipLaunchKernelGGL(k_zero_f32, dim3((unsigned)std::min<size_t>((nw + 255) / 256, 4096)), dim3(256), 0, s, gw_d, nw);
    const int tx = (w + kTX - 1) / kTX, ty = (h + kTY - 1) / kTY;
    const long long tiles = (long long)n * tx * ty;
    const unsigned gx = (unsigned)((ci + kCiC - 1) / kCiC), gyd = (unsigned)((co + kTCo - 1) / kTCo);
    if (gyd > 65535) return MC_ERR_UNSUPPORTED;
    // enough pixel slices to give the device ~2048 workgroups
    const long long blocks = (long long)gx * gyd;
    long long slices = std::max<long long>(1, std::min<long long>(tiles, (2048 + blocks - 1) / blocks));
    slices = std::min<long long>(slices, 65535);
    const long long per = (tiles + slices - 1) / slices;
    slices = (tiles + per - 1) / per;
    mc_status st = set_lds(reinterpret_cast<const void *>(k_conv3x3_wgrad), kWgradLds);
    if (st != MC_OK) return st;
    hipLaunchKernelGGL(k_conv3x3_wgrad, dim3(gx, gyd, (unsigned)slices), dim3(kThreads), kWgradLds, s, x_d, gy_d, gw_d,
                       ci, co, h, w, tx, ty, (int)tiles, (int)per);
    return hipGetLastError() == hipSuccess ? MC_OK : MC_ERR_DEVICE;
}

}  // extern "C"
