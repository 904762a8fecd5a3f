// Long-pencil kernels for rows of 512 and 1024 points: the last axis of grids whose other side has odd factors.  (1-D layers and
// the 2-D pipelines of these lengths have fused kernels; N = 1024 with up to 128 modes has the short-pencil kernels.)
#include "pruned1d_long_kernel.h"
#include "pruned1d.h"

namespace tfno {

int pruned1d_row_stride(int N, int K_keep)
{
    if ((N != 512 && N != 1024) || K_keep < 1 || K_keep > N) return 0;
    const int N1 = N / 256;
    return (K_keep + N1 - 1) / N1 * N1;                     // whole columns of the N1 x 256 array
}

template <int N1, int K2>
static hipError_t launch(int dir, const c64 *in, c64 *out, long long rows, int K_keep, int K2k, hipStream_t s)
{
    constexpr int G = CfgLong<N1, K2>::G;
    const long long sweeps = (rows + G - 1) / G;
    // (a few sweeps per workgroup: the next one's loads are in flight; three workgroups per CU at once)
    const unsigned grid = (unsigned)(sweeps < 768 ? sweeps : 768);
    if (dir < 0) hipLaunchKernelGGL((k_fwd1d_long<N1, K2, false>), dim3(grid), dim3(256), 0, s, in, out, 1, rows, K_keep, K2k);
    else hipLaunchKernelGGL((k_inv1d_long<N1, K2, false>), dim3(grid), dim3(256), 0, s, in, out, 1, rows, K2k);
    return hipGetLastError();
}

template <int N1>
static hipError_t launch_n(int dir, const c64 *in, c64 *out, long long rows, int K_keep, hipStream_t s)
{
    const int K2k = (K_keep + N1 - 1) / N1;
    if (K2k <= 16) return launch<N1, 16>(dir, in, out, rows, K_keep, K2k, s);
    if (K2k <= 32) return launch<N1, 32>(dir, in, out, rows, K_keep, K2k, s);
    if (K2k <= 64) return launch<N1, 64>(dir, in, out, rows, K_keep, K2k, s);
    if (K2k <= 128) return launch<N1, 128>(dir, in, out, rows, K_keep, K2k, s);
    return launch<N1, 256>(dir, in, out, rows, K_keep, K2k, s);
}

hipError_t pruned1d_rows(int dir, const c64 *in, c64 *out, long long rows, int N, int K_keep, hipStream_t s)
{
    if (!pruned1d_row_stride(N, K_keep)) return hipErrorInvalidValue;
    if (rows <= 0) return hipSuccess;
    return N == 512 ? launch_n<2>(dir, in, out, rows, K_keep, s) : launch_n<4>(dir, in, out, rows, K_keep, s);
}

}  // namespace tfno
