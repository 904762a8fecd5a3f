// Host-visible interface of the matrix transform: pruned DFTs of any length as contractions on the matrix pipe.
#pragma once
#include "common.h"

namespace tfno {

// One transform out[q][j] = sum_{i < I} in[q][i] exp(dir 2 pi i (i j) / N),  j < J, of P pencils q.  I <= N and J <= N
// prune the input (zero padding) and the output (truncation); nothing is scaled.  How a side is laid out:
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
    int N, I, J;
    unsigned P;                     // pencils, below 2^31
    unsigned inner;
    long long in_outer, out_outer;  // MD_ROWS and MD_STRIDED sides
    int C;                          // MD_SPEC side
    long long M;
    int dir;                        // -1 or +1
    int jgroups;                    // filled in by the launcher
};

// Which pairs of sides exist: ROWS -> SPEC, SPEC -> ROWS (1-D), ROWS -> ROWS (contiguous axis of a field),
// STRIDED -> SPEC, SPEC -> STRIDED (leading axis).
hipError_t matdft_launch(MatdftSide in_side, MatdftSide out_side, MatdftArgs a, hipStream_t s);

// The whole layer on fields N1 x N2 (1-D: N1 = K1 = 1) of any side lengths up to 4096: truncated transforms, the mode
// contraction, zero-padded inverses.  Workspace: matdft_workspace_bytes.
size_t matdft_workspace_bytes(long long B, int C_in, int C_out, int N1, int N2, int K1, int K2);
hipError_t matdft_conv(const c64 *x, const c64 *W, c64 *y, long long B, int C_in, int C_out, int N1, int N2, int K1, int K2,
                       c64 *ws, hipStream_t s);

}  // namespace tfno
