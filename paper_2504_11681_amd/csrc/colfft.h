// Host-visible interface of the column transforms: pruned transforms along the leading axis of row-major fields.
#pragma once
#include "common.h"

namespace tfno {

// True when column kernels exist for fields of N1 rows keeping K1 modes of every column (N1 in {64, 128, 256, 512}).
bool colfft_supported(int N1, int K1);
// dir < 0: out[f][k][n2] = sum_n in[f][n][n2] exp(-2 pi i n k / N1), k < K1  (in [fields, N1, N2], out K1 rows of N2 per field);
// dir > 0: the unscaled zero-padded inverse.  N2 a multiple of 16.
// Where the K1 rows of field f begin: dir < 0 (f / channels) outer + (f % channels) inner, dir > 0 f outer (there `in` may be `out`, the rows of a
// field in its own first ones).
struct ColRows { int channels; long long outer, inner; };
hipError_t colfft_launch(int dir, const c64 *in, c64 *out, long long fields, int N1, int N2, int K1, ColRows rows, hipStream_t s);
// The same with the modes in a mode-tile-major spectrum of C channels with M modes per batch element (mode k of column n2 is
// mode k N2 + n2): dir < 0 writes it, dir > 0 reads it.  Any N2.
hipError_t colfft_spec_launch(int dir, const c64 *in, c64 *out, long long fields, int N1, int N2, int K1, int C, long long M,
                              hipStream_t s);

}  // namespace tfno
