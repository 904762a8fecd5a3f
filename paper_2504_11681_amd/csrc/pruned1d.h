// Host-visible interface of the unfused 1-D variant with pruned transforms (three kernels).
#pragma once
#include "common.h"

namespace tfno {

// N in {64, 128, 256} with K a multiple of 16 such that K/16 divides N/16, N = 1024 with K in {64, 128}, or
// N in {2048, 4096} with K / (N / 256) in {16, 32, 64, 128, 256}.
bool pruned1d_supported(int N, int K);
// The smallest built power of two >= K for pencils of N points; 0: none.
int pruned1d_modes(int N, int K);
// Workspace for the truncated spectra of input and output, padded to whole 128-mode tiles.
size_t pruned1d_workspace_bytes(long long B, int C_in, int C_out, int K);
// K_keep (1 .. K): bins K_keep .. K-1 of the forward transform are dropped, which truncates to K_keep modes.
hipError_t pruned1d_launch(const c64 *x, const c64 *W, c64 *y, long long B, int C_in, int C_out, int N, int K,
                           int K_keep, c64 *ws, hipStream_t s);
// Single stages for the partially fused variants: stages is a mask of PRUNED_FWD (x -> Xh), PRUNED_GEMM
// (Xh -> Yh, scaled by 1/N) and PRUNED_INV (Yh -> y); Xh holds ceil(B Mp / 128) * 128 * C_in elements, Yh the same
// with C_out.
enum { PRUNED_FWD = 1, PRUNED_GEMM = 2, PRUNED_INV = 4 };
size_t pruned1d_spectrum_elems(long long B, int C, int Mp);
// Modes per pencil in the joint mode index of the spectra when K_keep of the kernel's K bins are kept (at most K): the
// bins past it are neither stored nor contracted (N 2048, K 316 of 512: 320; K 500 of 512: 512).
int pruned1d_stride(int N, int K, int K_keep, bool per_mode = false);
// Mp: pruned1d_stride(N, K, K_keep), or K with N <= 1024 for the partially fused kernels, which read and write all K.  With
// Mp = K the forward transform writes zeros to the bins that are not kept and the inverse expects zeros there.
hipError_t pruned1d_stages(int stages, const c64 *x, const c64 *W, c64 *y, c64 *Xh, c64 *Yh, long long B, int C_in,
                           int C_out, int N, int K, int K_keep, int Mp, hipStream_t s);

// Rows of 512 or 1024 points by the long-pencil kernels: dir < 0 [rows, N] -> [rows, stride], K_keep bins in an order of their
// own and zeros; dir > 0 the unscaled zero-padded inverse, which takes all `stride` of them.  stride 0: other lengths.
int pruned1d_row_stride(int N, int K_keep);
hipError_t pruned1d_rows(int dir, const c64 *in, c64 *out, long long rows, int N, int K_keep, hipStream_t s);

// Real pencils (x, y float32; N <= 1024): PRUNED_FWD writes the R2C bins with bin 0 halved, PRUNED_INV stores the real
// part of the zero-padded inverse; the contraction between them (not run here) carries the scale 2 / N.
hipError_t pruned1d_real_stages(int stages, const float *x, float *y, c64 *Xh, c64 *Yh, long long B, int C_in, int C_out,
                                int N, int K, int K_keep, int Mp, hipStream_t s);

// Contraction with own weights per mode (W [C_in, C_out, Ma], times scale) and zero-padded inverse in one kernel: Xh -> y, for
// small layers.  real: y float32, as pruned1d_real_stages.
bool pruned1d_permode_fused(long long B, int C_in, int C_out, int N, int K, int Ma);
hipError_t pruned1d_permode_inverse(bool real, const c64 *Xh, const c64 *W, c64 *y, long long B, int C_in, int C_out, int N, int K, int Ma,
                                    int Mp, float scale, hipStream_t s);

// Layers of N = 1024 with up to 128 modes and few batch elements (shared W; real: x, y float32): three kernels whose spectra are held in y.
bool pruned1d_in_y_supported(bool real, long long B, int C_in, int C_out, int N, int K_keep);
hipError_t pruned1d_in_y(bool real, const void *x, const c64 *W, void *y, long long B, int C_in, int C_out, int N, int K_keep, hipStream_t s);

}  // namespace tfno
