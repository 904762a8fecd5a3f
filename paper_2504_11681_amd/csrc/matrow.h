// Host-visible interface of the 1-D layer for lengths that are no powers of two: forward transform, then contraction and inverse
// transform in one kernel.
#pragma once
#include "common.h"

namespace tfno {

struct MatrowArgs {
    const c64 *x, *W;
    c64 *Xh, *y;            // Xh: truncated spectrum of the input as in matdft.h (MD_SPEC, K modes per batch element)
    int B, C_in, C_out, N, K;
    float scale;
    int parts, groups;      // filled in by the launcher
};

bool matrow_forward_supported(long long B, int C_in, int N, int K);
hipError_t matrow_forward(const MatrowArgs &a, hipStream_t s);
bool matrow_inverse_supported(long long B, int C_in, int C_out, int N, int K);
hipError_t matrow_inverse(const MatrowArgs &a, hipStream_t s);

}  // namespace tfno
