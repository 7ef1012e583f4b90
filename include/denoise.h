/*
 * denoise.h -- C ABI of the BF16 matrix-core kernels of the learned denoiser
 * (part of librmc.so).  The denoiser maps harmonic coefficient maps from few
 * packets to maps from many packets; its convolutions run here.
 *
 * Conventions as in mcrad.h: pointers ending in _d are caller-owned device
 * memory; calls only enqueue on `stream`; errors are status codes checked on
 * the host before anything is enqueued.  BF16 tensors are raw 16-bit
 * patterns (uint16_t).  Activations are channels last, [n][h][w][c], with c
 * a multiple of 8 and 16-byte aligned rows (pad with zero channels); weights
 * [co][3][3][ci].  Products are exact in FP32 and summed in FP32 on the
 * MFMA units (v_mfma_f32_16x16x32_bf16); the order of the sums differs from
 * a sequential loop.  Invalid shapes or alignment: MC_ERR_INVALID_ARG.
 */
#ifndef DENOISE_H
#define DENOISE_H

#include <stddef.h>
#include <stdint.h>

#include "mcrad.h"

#ifdef __cplusplus
extern "C" {
#endif

/* 3x3 convolution, stride 1, zero padding 1:
 *   y[n][h][w][co] = bias[co] + sum_{ky,kx,ci} w[co][ky][kx][ci] x[n][h+ky-1][w+kx-1][ci]
 * x_d: BF16 [n][h][w][ci], ci % 8 == 0, 16-byte aligned; w_d: BF16
 * [co][3][3][ci], 16-byte aligned; bias_d: FP32 [co] or NULL; y_d: FP32
 * [n][h][w][co] (overwritten; 16-byte aligned when co % 4 == 0).  The
 * gradient with respect to x is this same call on the upstream gradient with
 * the weights flipped in both spatial directions and ci/co swapped. */
mc_status dn_conv3x3_fwd(const uint16_t *x_d, const uint16_t *w_d, const float *bias_d, float *y_d, int n, int ci,
                         int co, int h, int w, void *stream);

/* The same from FP32 activations as a program holds them: x_d is FP32 with
 * element strides strides_h = {n, c, h, w}; the values are rounded to BF16
 * (nearest even) on their way into the product.  w_d: BF16 [co][3][3][cip] as
 * dn_pack_weights writes it, cip = ci rounded up to a multiple of 8.  xb_d: if
 * not NULL, receives the BF16 values, [n][h][w][cip] with zeros past ci, for
 * dn_conv3x3_grads. */
mc_status dn_conv3x3_f32(const float *x_d, const int64_t *strides_h, const uint16_t *w_d, const float *bias_d, float *y_d,
                         uint16_t *xb_d, int n, int ci, int co, int h, int w, void *stream);

/* Weights FP32 [co][ci][3][3] to BF16 [co][3][3][cip] (zeros past ci), or with
 * flip = 1 to those of the gradient with respect to x: [ci][3][3][cop], both
 * spatial directions reversed. */
mc_status dn_pack_weights(const float *w_d, uint16_t *out_d, int co, int ci, int flip, void *stream);

/* The denoiser's network, without gradients: an encoder and decoder over
 * `levels` levels (1 .. 8) of the given widths (host array; widths[0] <= 512).
 * Every level is two 3x3 convolutions with ReLU; a level's map goes to the
 * next by 2 x 2 maxima (odd sizes round up) and comes back repeated 2 x 2 (cut
 * to size) before the channels of the map kept on the way down; last,
 *   y = x + out_w a + out_b
 * with out_w FP32 [channels][widths[0]].  weights (host array of 4 levels - 2
 * device pointers): FP32 [co][ci][3][3], encoder from the top, then decoder
 * from the bottom; biases: FP32 [co].  x_d, y_d: FP32 with element strides
 * {n, c, h, w}; they may not overlap.  The same values as dn_conv3x3_f32 layer
 * by layer.  scratch_d: at least dn_unet_bytes() bytes (0: the network or sizes
 * are not supported), 16-byte aligned. */
size_t dn_unet_bytes(int channels, int levels, const int32_t *widths, int n, int h, int w);
mc_status dn_unet_forward(int channels, int levels, const int32_t *widths, const float *const *weights,
                          const float *const *biases, const float *out_w, const float *out_b, const float *x_d,
                          const int64_t *x_strides, float *y_d, const int64_t *y_strides, void *scratch_d,
                          size_t scratch_bytes, int n, int h, int w, void *stream);

/* Gradients of dn_conv3x3_f32 with respect to the weights, FP32
 * [co][ci][3][3], and (if gb_d is not NULL) the bias, FP32 [co]: xb_d as that
 * call wrote it, gy_d FP32 [n][h][w][co].  The weight gradient's products take
 * gy rounded to BF16, the bias gradient sums gy itself.  scratch_d: at least
 * dn_conv3x3_grads_bytes() bytes (0 on invalid arguments), 16-byte aligned.
 * The sums' order is fixed: the result is the same every time. */
size_t dn_conv3x3_grads_bytes(int n, int ci, int co, int h, int w);
mc_status dn_conv3x3_grads(const uint16_t *xb_d, const float *gy_d, float *gw_d, float *gb_d, void *scratch_d,
                           size_t scratch_bytes, int n, int ci, int co, int h, int w, void *stream);

/* Weight gradient of dn_conv3x3_fwd:
 *   gw[co][ky][kx][ci] = sum_{n,h,w} gy[n][h][w][co] x[n][h+ky-1][w+kx-1][ci]
 * x_d: BF16 [n][h][w][ci]; gy_d: BF16 [n][h][w][co]; ci and co multiples of
 * 8, both 16-byte aligned; gw_d: FP32 [co][3][3][ci] (overwritten; partial
 * sums over pixel slices are added with FP32 atomics, so the last bits
 * depend on their order). */
mc_status dn_conv3x3_wgrad(const uint16_t *x_d, const uint16_t *gy_d, float *gw_d, int n, int ci, int co, int h, int w,
                           void *stream);

#ifdef __cplusplus
}
#endif
#endif /* DENOISE_H */
