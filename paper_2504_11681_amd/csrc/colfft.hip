// Instantiations and launcher of the column transforms.
#include "colfft_kernel.h"
#include "colfft.h"

namespace tfno {

namespace {
int stage_a_points(int N1) { return N1 == 64 ? 8 : 16; }

template <int P, int T, int Q>
hipError_t launch_pq(int dir, const c64 *in, c64 *out, long long fields, int N2, int K1, hipStream_t s)
{
    using C = CfgCol<P, T, Q>;
    static LdsLimitOnce limit;
    const hipError_t e = limit.set({reinterpret_cast<const void *>(&k_colfft_fwd<P, T, Q>), reinterpret_cast<const void *>(&k_colfft_inv<P, T, Q>)},
                                   (int)C::LDS);
    if (e != hipSuccess) return e;
    const unsigned groups = (unsigned)(N2 / 16);
    const dim3 grid((unsigned)(fields * groups));
    constexpr int nt = C::NT;
    if (dir < 0) hipLaunchKernelGGL((k_colfft_fwd<P, T, Q>), grid, dim3(nt), C::LDS, s, in, out, N2, K1, groups);
    else hipLaunchKernelGGL((k_colfft_inv<P, T, Q>), grid, dim3(nt), C::LDS, s, in, out, N2, K1, groups);
    return hipGetLastError();
}

template <int P, int T>
hipError_t launch_p(int dir, const c64 *in, c64 *out, long long fields, int N2, int K1, hipStream_t s)
{
    const int q = (K1 + P - 1) / P;
    if (q <= 1) return launch_pq<P, T, 1>(dir, in, out, fields, N2, K1, s);
    if (q <= 2) return launch_pq<P, T, 2>(dir, in, out, fields, N2, K1, s);
    if (q <= 4) return launch_pq<P, T, 4>(dir, in, out, fields, N2, K1, s);
    return launch_pq<P, T, 8>(dir, in, out, fields, N2, K1, s);
}
}  // namespace

bool colfft_supported(int N1, int K1)
{
    return (N1 == 64 || N1 == 128 || N1 == 256 || N1 == 512) && K1 >= 1 && K1 <= 8 * stage_a_points(N1) && K1 <= N1;
}

hipError_t colfft_launch(int dir, const c64 *in, c64 *out, long long fields, int N1, int N2, int K1, hipStream_t s)
{
    if (!colfft_supported(N1, K1) || N2 < 16 || N2 % 16 != 0 || fields * (N2 / 16) > 0x7fffffffLL) return hipErrorInvalidValue;
    if (fields <= 0) return hipSuccess;
    switch (N1) {
    case 64: return launch_p<8, 8>(dir, in, out, fields, N2, K1, s);
    case 128: return launch_p<16, 8>(dir, in, out, fields, N2, K1, s);
    case 256: return launch_p<16, 16>(dir, in, out, fields, N2, K1, s);
    default: return launch_p<16, 32>(dir, in, out, fields, N2, K1, s);
    }
}

}  // namespace tfno
