// Host-visible interface of the field transforms for sides that are no powers of two: both axes in one kernel.
#pragma once
#include "common.h"

namespace tfno {

struct MatgridArgs {
    const c64 *in;          // forward: fields [images, N1, N2]; inverse: spectrum
    c64 *out;
    int N1, N2, K1, K2, C;  // image = batch element * C + channel; spectrum as in matdft.h with K1 K2 modes per batch element
    int parts, parts2;      // filled in by the launcher
};

// Whether `images` fields are transformed by these kernels (dir < 0: forward).
bool matgrid_supported(int dir, long long images, int N1, int N2, int K1, int K2);
hipError_t matgrid_launch(int dir, const c64 *in, c64 *out, long long images, int C, int N1, int N2, int K1, int K2, hipStream_t s);

}  // namespace tfno
