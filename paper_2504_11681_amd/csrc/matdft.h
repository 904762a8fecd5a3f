// Host-visible interface of the matrix transform: pruned DFTs of any length as contractions on the matrix pipe.
#pragma once
#include "common.h"

namespace tfno {

// One transform of P pencils q of N points that keeps K of its N bins:
//   forward  out[q][k] = sum_{n < N} in[q][n] exp(-2 pi i n k / N),  k < K      (output pruned: truncation)
//   inverse  out[q][n] = sum_{k < K} in[q][k] exp(+2 pi i n k / N),  n < N      (input pruned: zero padding; unscaled)
// How a side is laid out:
//   MD_ROWS     element e of pencil q at q * outer + e
//   MD_STRIDED  element e at (q / inner) * outer + q % inner + e * inner: a leading axis of a row-major field, the
//               `inner` pencils of an outer item being adjacent columns
//   MD_SPEC     truncated spectrum, mode-tile major as the contraction kernels read it: with img = q / inner, batch
//               element b = img / C and channel c = img % C, element e is mode m = b M + e * inner + q % inner at
//               ((m / 128) * C + c) * 128 + m % 128
enum MatdftSide { MD_ROWS = 0, MD_STRIDED = 1, MD_SPEC = 2 };
struct MatdftArgs {
    const c64 *in;
    c64 *out;
    int N, K;
    unsigned P;                     // pencils, below 2^31
    unsigned inner;
    long long in_outer, out_outer;  // MD_ROWS and MD_STRIDED sides
    int C;                          // MD_SPEC side
    long long M;
    int groups;                     // filled in by the launcher
};

// Pairs of sides that exist: forward ROWS -> SPEC (1-D), ROWS -> ROWS (contiguous axis of a field), STRIDED -> SPEC (leading
// axis); inverse SPEC -> ROWS, SPEC -> STRIDED, ROWS -> ROWS.
hipError_t matdft_forward(MatdftSide in_side, MatdftSide out_side, MatdftArgs a, hipStream_t s);
hipError_t matdft_inverse(MatdftSide in_side, MatdftSide out_side, MatdftArgs a, hipStream_t s);

// The whole layer on fields N1 x N2 (1-D: N1 = K1 = 1) of any side lengths up to 4096: truncated transforms, the mode
// contraction, zero-padded inverses.  Workspace: matdft_workspace_bytes.
size_t matdft_workspace_bytes(long long B, int C_in, int C_out, int N1, int N2, int K1, int K2);
hipError_t matdft_conv(const c64 *x, const c64 *W, c64 *y, long long B, int C_in, int C_out, int N1, int N2, int K1, int K2,
                       c64 *ws, hipStream_t s);

}  // namespace tfno
