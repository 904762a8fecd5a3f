// Host-visible interface of the 2-D kernels (truncated-spectrum pipeline).
#pragma once
#include "common.h"

namespace tfno {

// True when the image kernels exist for N1 x N2 images keeping K1 x K2 modes: N1, N2 in {64, 128, 256},
// K1, K2 in {16, 32, 64}.
bool fused2d_supported(int N1, int N2, int K1, int K2);
// Workspace for Xh[B, C_in, K1, K2] and Yh[B, C_out, K1, K2].
size_t fused2d_workspace_bytes(long long B, int C_in, int C_out, int K1, int K2);
// Enqueues forward transform, mode CGEMM and inverse transform on stream s.
hipError_t fused2d_launch(const c64 *x, const c64 *W, c64 *y, long long B, int C_in, int C_out, int N1, int N2,
                          int K1, int K2, int k1_keep, int k2_keep, c64 *ws, hipStream_t s);
// One of the two image kernels: dir < 0 forward x[images, N1, N2] -> Xh (C = C_in), dir > 0 inverse Yh -> y (C = C_out).
// Only the first k1_keep x k2_keep modes of the kernels' K1 x K2 exist in the spectra (the others are not stored and read
// as zeros): mode m = k1 k2_keep + k2 of batch element b at joint mode b spectrum_stride(k1_keep k2_keep) + m.
// fno: the real-field variants (x, y float32 images; first-axis frequencies -h1 .. K1-h1-1 at positions 0 .. K1-1;
// R2C / C2R along the last axis, the caller's contraction carries the scale 2 / (N1 N2)); h1 is ignored otherwise.
hipError_t fused2d_images(int dir, const c64 *in, c64 *out, long long images, int C, int N1, int N2, int K1, int K2,
                          int k1_keep, int k2_keep, bool fno, int h1, hipStream_t s);
// The two image kernels for one first-axis length (one translation unit each; fused2d_fno_*: the real-field variants).
#define TFNO_DECLARE_IMAGES(name)                                                                                     \
    hipError_t name(int dir, const c64 *in, c64 *out, long long images, int C, int N2, int K1, int K2, int k1_keep, \
                    int k2_keep, int h1, hipStream_t s)
TFNO_DECLARE_IMAGES(fused2d_images_n64);
TFNO_DECLARE_IMAGES(fused2d_images_n128);
TFNO_DECLARE_IMAGES(fused2d_images_n256);
TFNO_DECLARE_IMAGES(fused2d_fno_images_n64);
TFNO_DECLARE_IMAGES(fused2d_fno_images_n128);
TFNO_DECLARE_IMAGES(fused2d_fno_images_n256);
#undef TFNO_DECLARE_IMAGES

// Yh = Xh . (scale W) over `tiles` tiles of 128 modes; both spectra mode-tile major ([tile][channel][128]).  all_products: sums
// over up to 16 channels as precise as FP32 ones, where the direct kernel runs.
hipError_t cgemm_modes_launch(const c64 *Xh, const c64 *W, c64 *Yh, int C_in, int C_out, float scale, long long tiles,
                              hipStream_t s, bool all_products = false);

// Yh[b][o][m] = scale * sum_c Xh[b][c][m] * W[c][o][m], m < Ma, with an own weight matrix per mode: W is [C_in, C_out, Ma],
// the spectra are mode-tile major over the joint mode b Mp + m (Mp >= Ma, a multiple of 8).  Results at m >= Ma: zeros if
// `zeros` is set, which says that Xh holds zeros there, else unspecified.
hipError_t cgemm_permode_launch(const c64 *Xh, const c64 *W, c64 *Yh, int C_in, int C_out, long long B, int Mp, int Ma,
                                bool zeros, float scale, hipStream_t s);

// Modes per batch element in the joint mode index of a spectrum that keeps `modes` of them: 64-byte rows.
inline int spectrum_stride(int modes) { return (modes + 7) & ~7; }

// The same with one W for spectra in rows of whole 32 modes, K <= 128 of them contracted: batch element b, channel c of X at b x_batch + c x_channel.
hipError_t cgemm_rows_launch(const c64 *Xh, const c64 *W, c64 *Yh, int C_in, int C_out, float scale, long long B, int K, long long x_batch, int x_channel,
                             long long y_batch, int y_channel, hipStream_t s);

}  // namespace tfno
