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
    const bool LONG = N1 / 32 + 1 > 3 * p.parts || N2 / 32 + 1 > 3 * p.parts2;
    return LONG ? pick_fwd<true>(K1, K2) : pick_fwd<false>(K1, K2);
}
}  // namespace

// From a workgroup for every CU on the field kernels are ahead of a kernel per axis (85 x 85, K 12 x 12, 1024 fields each way: forward
// 25.2 -> 14.5 us, inverse 29.9 -> 18.7; 158 x 131, 594 and 342 fields: 46.6 -> 34.1, 31.2 -> 19.8; the worst of 47 drawn shapes 71 x 149: inverse
// 20.8 -> 22.9).  Fewer fields are a question of the longest chain: a kernel per axis spreads one field over many workgroups and
// takes about 9 us and what its bytes cost, a field's workgroup takes its blocks of 32 rows (forward) or its tiles of 32
// output pairs (inverse) in turn.  In tenths of a microsecond, from the same measurements: 300 x 300, 8 fields 13.0 against 37 us, 85 x 85,
// 8 fields 9.0 against 7.1, 200 x 120, K 32 x 17, 32 fields 11.6 against 12.2, 126 fields 16.7 against 13.3.
// More than 256 columns go to a kernel per axis: two column tiles to a wave measured 13 % slower to 25 % faster, without a clear line.
bool matgrid_supported(int dir, long long images, int N1, int N2, int K1, int K2)
{
    if (N1 < 30 || N2 < 30 || N1 > MG_ROWS || N2 > MG_COLUMNS || K1 > MG_MODES || K2 > MG_MODES) return false;
    if (images < 1 || images >= (1LL << 31)) return false;
    const Plan p = plan(dir, images, N1, N2, K1, K2);
    if (p.lds > MOST_LDS) return false;
    // Two sixteens of rows take a wave's registers twice: with seven and eight waves to a workgroup one fits a CU (40 x 250, K 20 x 20, 600 fields: forward
    // 19.4 -> 29.2 us, inverse 24.1 -> 28.9; 200 x 200, K 25 x 25, 400 fields: 52.1 -> 40.6, 56.0 -> 49.5), and its inverse stays a question of the
    // chain up to two workgroups for every CU (220 x 56, K 25 x 8, 400 fields: 17.4 -> 21.2; 348 x 82, K 17 x 13, 486 fields: 45 -> 34).
    // Four waves and more and fewer than two fields for every CU only pay with larger fields (132 x 160, K 19 x 20, 300 fields: 24.3 -> 31.0, 30.8 -> 35.0;
    // 600 fields of 132 x 192 50.7 -> 49.0, 54.7 -> 54.0).
    if (K1 > 16 && (N2 > 224 || (N2 > 128 && images < 512 && N1 * N2 < 32768))) return false;
    if (images >= (dir > 0 && K1 > 16 ? 512 : 256)) return true;
    const long long bytes = images * N1 * N2 * (long long)sizeof(c64);
    if (dir < 0) {
        const int turns = (N1 / 32 + p.parts) / p.parts;
        return turns * (K1 > 16 ? 21 : 16) <= 45 + bytes / 260000;
    }
    const int turns = (N1 / 64 + p.parts) / p.parts;
    return 55 + turns * (K1 > 16 ? 48 : 34) <= 90 + bytes / 350000;
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
