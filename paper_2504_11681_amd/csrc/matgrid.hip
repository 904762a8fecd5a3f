// Launcher of the field transforms for sides that are no powers of two.
#include "matgrid_kernel.h"

namespace tfno {

namespace {
constexpr size_t MOST_LDS = 160 * 1024;
struct Plan { int waves, parts, parts2, RG; size_t lds; };

Plan plan(int dir, long long images, int N1, int N2, int K1, int K2)
{
    Plan p{};
    const int tiles = (N2 + 31) / 32, P = mg_pitch(N2);
    p.parts = 1;
    const size_t tables = MG_ROOT * (size_t)(N1 == N2 ? N1 : N1 + N2);
    if (dir < 0) {
        // few columns: the rows are dealt out to two or four waves per tile
        const int most = images >= 1024 ? MG_WAVES / 2 : MG_WAVES;
        while (2 * p.parts * tiles <= most && 2 * p.parts <= N1 / 32 + 1) p.parts *= 2;
        p.waves = tiles * p.parts;
        p.parts2 = p.waves < 4 ? p.waves : 4;
        if (p.parts2 > N2 / 32 + 1) p.parts2 = N2 / 32 + 1;
        p.lds = tables + sizeof(c64) * ((size_t)p.parts * K1 * P + (size_t)p.parts2 * K1 * K2);
    } else {
        // (with a workgroup for every CU more sets only take registers from one another: 85 x 85, 512 fields 28.9 us the layer, 36.2 with two)
        while (images < 256 && (p.parts + 1) * tiles <= MG_WAVES && 32 * p.parts <= N1 / 2) ++p.parts;
        p.waves = tiles * p.parts;
        p.RG = N2 <= 128 || K1 <= 16 ? 2 : 1;
        p.lds = tables + sizeof(c64) * (32 * (size_t)mg_modes_pitch(K2) + (K1 > 16 ? 32 : 16) * (size_t)P + 16 * (size_t)p.RG * p.parts * N2);
    }
    return p;
}

bool forward_long(int N1, int N2, const Plan &p) { return N1 / 32 + 1 > 3 * p.parts || N2 / 32 + 1 > 3 * p.parts2; }

typedef void (*Kernel)(MatgridArgs);
template <bool LONG>
Kernel pick_fwd(int K1, int K2)
{
    if (K1 <= 16) return K2 <= 16 ? k_matgrid_fwd<1, 1, LONG> : k_matgrid_fwd<1, 2, LONG>;
    return K2 <= 16 ? k_matgrid_fwd<2, 1, LONG> : k_matgrid_fwd<2, 2, LONG>;
}
Kernel pick(int dir, int N1, int N2, int K1, int K2, const Plan &p)
{
    if (dir > 0) {
        if (K1 <= 16) return N2 > 128 ? k_matgrid_inv<2, 1, 4> : k_matgrid_inv<2, 1, 3>;
        return p.RG == 2 ? k_matgrid_inv<2, 2, 3> : k_matgrid_inv<1, 2, 3>;
    }
    return forward_long(N1, N2, p) ? pick_fwd<true>(K1, K2) : pick_fwd<false>(K1, K2);
}
}  // namespace

// Waves of the chosen kernel that a SIMD holds, from its registers.
static int waves_per_simd(int dir, int N1, int N2, int K1, const Plan &p)
{
    if (dir > 0) return K1 <= 16 && N2 > 128 ? 4 : 3;
    const bool LONG = forward_long(N1, N2, p);
    return LONG ? (K1 > 16 ? 2 : 3) : K1 > 16 ? 3 : 4;
}

// Which is faster for a direction, these kernels or a kernel per axis, is a question of rounds and of the longest chain: a field's workgroup takes its blocks of 32 rows
// (forward) or its tiles of 32 output pairs (inverse) in turn, and what a last short round leaves idle is lost, while a kernel per axis spreads each field over
// many workgroups and takes a launch more and what its bytes cost.  In microseconds, fitted to whole layers with both kinds of kernels for either direction (3350 drawn shapes of 30 to
// 512 x 30 to 480 points, 1 to 4500 fields): chosen like this they take 0.837 of the time of kernels per axis (the best of the four combinations 0.833), and 22 of them are more than
// 3 % slower, at most 12 %.  85 x 85, K 12 x 12, 1024 fields each way: forward 25.2 -> 14.5 us, inverse 29.9 -> 18.7; 158 x 131, 594 and 342
// fields: 46.6 -> 34.1, 31.2 -> 19.8; 300 x 300, 8 fields 13.0 against 37 us; whole layers with an inverse by these kernels at 320 fields of 273 x 133, K 28 x 8, two rounds, the second
// a quarter full, 55.1 and 77.3, and a forward transform at 1805 of 77 x 141, K 18 x 10, 66.7 and 93.8.
// More than 256 columns go to a kernel per axis: two column tiles to a wave measured 13 % slower to 25 % faster, without a clear line.
bool matgrid_supported(int dir, long long images, int N1, int N2, int K1, int K2)
{
    if (N1 < 30 || N2 < 30 || N1 > MG_ROWS || N2 > MG_COLUMNS || K1 > MG_MODES || K2 > MG_MODES) return false;
    if (images < 1 || images >= (1LL << 31)) return false;
    const Plan p = plan(dir, images, N1, N2, K1, K2);
    if (p.lds > MOST_LDS) return false;
    // (workgroups of up to four waves fill the SIMDs' places one by one; of a larger one some SIMD holds two waves, always the same: 273 x 133, K 28 x 8, five waves at three to a
    // SIMD, 256, 270, 512 and 530 fields 46.5, 74.1, 74.6 and 101.7 us the layer)
    const int simd = waves_per_simd(dir, N1, N2, K1, p), by_waves = p.waves <= 4 ? 4 * simd / p.waves : simd / ((p.waves + 3) / 4), by_lds = (int)(MOST_LDS / p.lds);
    const long long resident = 256LL * (by_waves < 1 ? 1 : by_waves < by_lds ? by_waves : by_lds);
    const double rounds = (double)((images + resident - 1) / resident);
    const double field_us = (double)images * N1 * N2 * sizeof(c64) / 5e6, half_us = (double)images * N1 * 2 * sizeof(c64) / 5e6;
    const int two1 = K1 > 16 ? 2 : 1, two2 = K2 > 16 ? 2 : 1;
    if (dir < 0) {
        const int columns = (N1 / 32 + p.parts) / p.parts, rows = (N2 / 32 + p.parts2) / p.parts2 * ((two1 * p.parts2 + p.waves - 1) / p.waves);
        // (fewer than 16 kept columns cost a kernel per axis what 16 do, the width of its products: 3250 fields of 54 x 39, K 2 x 2 37.5 and 54.2 us the layer)
        return rounds * (4.0 + 0.45 * columns * (1 + two1) + 0.35 * rows * (1 + two2)) <= 8.5 + 0.9 * field_us + half_us * (K2 > 16 ? K2 : 16);
    }
    const int turns = (N1 / 64 + p.parts) / p.parts;
    return rounds * (2.5 + turns * (2.0 + 0.8 * two1)) <= 6.5 + 0.7 * field_us + 1.2 * half_us * K2;
}

hipError_t matgrid_launch(int dir, const c64 *in, c64 *out, long long images, int C, int N1, int N2, int K1, int K2, hipStream_t s)
{
    if (images == 0) return hipSuccess;
    if (!matgrid_supported(dir, images, N1, N2, K1, K2)) return hipErrorInvalidValue;
    const Kernel kernel = pick(dir, N1, N2, K1, K2, plan(dir, images, N1, N2, K1, K2));
    static LdsLimitOnce limit;
    const hipError_t e = limit.set({reinterpret_cast<const void *>(&k_matgrid_fwd<1, 1, false>), reinterpret_cast<const void *>(&k_matgrid_fwd<1, 2, false>),
                                    reinterpret_cast<const void *>(&k_matgrid_fwd<2, 1, false>), reinterpret_cast<const void *>(&k_matgrid_fwd<2, 2, false>),
                                    reinterpret_cast<const void *>(&k_matgrid_fwd<1, 1, true>), reinterpret_cast<const void *>(&k_matgrid_fwd<1, 2, true>),
                                    reinterpret_cast<const void *>(&k_matgrid_fwd<2, 1, true>), reinterpret_cast<const void *>(&k_matgrid_fwd<2, 2, true>),
                                    reinterpret_cast<const void *>(&k_matgrid_inv<2, 1, 4>), reinterpret_cast<const void *>(&k_matgrid_inv<2, 1, 3>),
                                    reinterpret_cast<const void *>(&k_matgrid_inv<2, 2, 3>), reinterpret_cast<const void *>(&k_matgrid_inv<1, 2, 3>)},
                                   (int)MOST_LDS);
    if (e != hipSuccess) return e;
    const Plan p = plan(dir, images, N1, N2, K1, K2);
    MatgridArgs a{in, out, N1, N2, K1, K2, C, p.parts, p.parts2};
    hipLaunchKernelGGL(kernel, dim3((unsigned)images), dim3(64 * p.waves), p.lds, s, a);
    return hipGetLastError();
}

}  // namespace tfno
