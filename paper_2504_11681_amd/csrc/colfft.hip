// Instantiations and launcher of the column transforms.
#include "colfft_kernel.h"
#include "colfft.h"

namespace tfno {

namespace {
int stage_a_points(int N1) { return N1 == 64 ? 8 : 16; }

struct Cols { const c64 *in; c64 *out; long long fields; int N2, K1, C; long long M, channel; };

template <int P, int T, int Q, bool SPEC>
hipError_t launch_pq(int dir, const Cols &a, hipStream_t s)
{
    using C = CfgCol<P, T, Q>;
    static LdsLimitOnce limit;
    const hipError_t e = limit.set({reinterpret_cast<const void *>(&k_colfft_fwd<P, T, Q, SPEC>),
                                    reinterpret_cast<const void *>(&k_colfft_inv<P, T, Q, SPEC>)}, (int)C::LDS);
    if (e != hipSuccess) return e;
    const unsigned groups = (unsigned)((a.N2 + 15) / 16);
    const dim3 grid((unsigned)(a.fields * groups));
    constexpr int nt = C::NT;
    // Neighbouring columns per XCD in the forward kernel for fields one and a half times the last-level cache and larger, with rows of
    // 1 KB and more.  Whole layers, every eighth line and neighbouring ones (us), on fields that the program has just written / that no cache
    // holds / pass after pass over the same three: 512 x 512, 268 MB 142 151 / 147 141 / 134 130, 335 MB 181 190 / 194 186 / 175 168, 403 MB
    // 211 209 / 226 216 / 204 196, 470 MB 244 234 / 262 251 / 235 231; 512 x 256, 335 MB 171 176 / 180 175 / 163 157, 403 MB 202 195 / 212 204 / 193 185;
    // 512 x 128, 403 MB 202 198 / 215 208 / 195 186.  Smaller fields lose where they were just written, the usual case.  (In the inverse kernel as
    // well 512 x 512 gains another 1 - 4 % and 512 x 256 and 512 x 128 lose up to 3 %; 512 x 64 in both kernels 111 and 120.)
    // The columns of truncated spectra gain in both kernels (256 x 360, 24 x 24 modes, 8 x 16 fields 79 77 / 83 82 / 65 62; 128 x 300, 24 x 50
    // modes, 32 x 32 fields 304 299 / 308 300 / 277 261; 64 to 256 rows of 200, 16 x 32 modes: equal within 1 %) from a workgroup per CU on, unless
    // they are one group of 16.
    const bool contiguous = SPEC ? groups > 1 && a.fields * groups >= 256 : a.N2 >= 128 && a.fields * C::N1 * a.N2 * (long long)sizeof(c64) >= 384LL << 20;
    if (dir < 0) hipLaunchKernelGGL((k_colfft_fwd<P, T, Q, SPEC>), grid, dim3(nt), C::LDS, s, a.in, a.out, a.N2, a.K1, groups, contiguous, a.C, a.M, a.channel);
    else hipLaunchKernelGGL((k_colfft_inv<P, T, Q, SPEC>), grid, dim3(nt), C::LDS, s, a.in, a.out, a.N2, a.K1, groups, SPEC && contiguous, a.C, a.M);
    return hipGetLastError();
}

template <int P, int T, bool SPEC>
hipError_t launch_p(int dir, const Cols &a, hipStream_t s)
{
    const int q = (a.K1 + P - 1) / P;
    if (q <= 1) return launch_pq<P, T, 1, SPEC>(dir, a, s);
    if (q <= 2) return launch_pq<P, T, 2, SPEC>(dir, a, s);
    if (q <= 4) return launch_pq<P, T, 4, SPEC>(dir, a, s);
    return launch_pq<P, T, 8, SPEC>(dir, a, s);
}

template <bool SPEC>
hipError_t launch(int dir, int N1, const Cols &a, hipStream_t s)
{
    if (!colfft_supported(N1, a.K1) || a.fields * ((a.N2 + 15) / 16) > 0x7fffffffLL) return hipErrorInvalidValue;
    if (a.fields <= 0) return hipSuccess;
    switch (N1) {
    case 64: return launch_p<8, 8, SPEC>(dir, a, s);
    case 128: return launch_p<16, 8, SPEC>(dir, a, s);
    case 256: return launch_p<16, 16, SPEC>(dir, a, s);
    default: return launch_p<16, 32, SPEC>(dir, a, s);
    }
}
}  // namespace

// (1024 rows of 16 columns would take 131 KB of LDS: one workgroup per CU and nothing beside it to cover its load and store
// phases; fewer columns touch parts of lines.  Not built; such columns run the radix-2 transform.)
bool colfft_supported(int N1, int K1)
{
    return (N1 == 64 || N1 == 128 || N1 == 256 || N1 == 512) && K1 >= 1 && K1 <= 8 * stage_a_points(N1) && K1 <= N1;
}

hipError_t colfft_launch(int dir, const c64 *in, c64 *out, long long fields, int N1, int N2, int K1, ColRows rows, hipStream_t s)
{
    if (N2 < 16 || N2 % 16 != 0 || rows.channels < 1 || (dir > 0 && rows.channels != 1)) return hipErrorInvalidValue;
    return launch<false>(dir, N1, Cols{in, out, fields, N2, K1, rows.channels, rows.outer, rows.inner}, s);
}

hipError_t colfft_spec_launch(int dir, const c64 *in, c64 *out, long long fields, int N1, int N2, int K1, int C, long long M, hipStream_t s)
{
    if (N2 < 1 || C < 1) return hipErrorInvalidValue;
    return launch<true>(dir, N1, Cols{in, out, fields, N2, K1, C, M, 0}, s);
}

}  // namespace tfno
