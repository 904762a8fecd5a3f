// Host-visible interface of the column transforms: pruned transforms along the leading axis of row-major fields.
#pragma once
#include "common.h"

namespace tfno {

// True when column kernels exist for fields of N1 rows keeping K1 modes of every column (N1 in {64, 128, 256, 512}).
bool colfft_supported(int N1, int K1);
// dir < 0: out[f][k][n2] = sum_n in[f][n][n2] exp(-2 pi i n k / N1), k < K1  (in [fields, N1, N2], out [fields, K1, N2]);
// dir > 0: the unscaled zero-padded inverse (in [fields, K1, N2], out [fields, N1, N2]).  N2 a multiple of 16.
hipError_t colfft_launch(int dir, const c64 *in, c64 *out, long long fields, int N1, int N2, int K1, hipStream_t s);
// The same with the modes in a mode-tile-major spectrum of C channels with M modes per batch element (mode k of column n2 is
// mode k N2 + n2): dir < 0 writes it, dir > 0 reads it.  Any N2.
hipError_t colfft_spec_launch(int dir, const c64 *in, c64 *out, long long fields, int N1, int N2, int K1, int C, long long M,
                              hipStream_t s);

}  // namespace tfno
