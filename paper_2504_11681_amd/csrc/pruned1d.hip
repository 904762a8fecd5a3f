// Instantiations and launcher of the unfused 1-D variant with pruned transforms.
#include "pruned1d_kernel.h"
#include "pruned1d_long_kernel.h"
#include "fused2d.h"          // cgemm_modes_launch
#include "pruned1d.h"

namespace tfno {

bool pruned1d_supported(int N, int K)
{
    if (K < 16 || K % 16 != 0 || K > N) return false;
    const int KH = K / 16;
    if (N == 1024) return KH == 4 || KH == 8;
    if (N == 2048 || N == 4096) {
        // long pencils: N1 = N / 256 rows of 256 points, each keeping K / N1 bins
        const int N1 = N / 256;
        if (K % N1) return false;
        const int K2 = K / N1;
        return K2 == 16 || K2 == 32 || K2 == 64 || K2 == 128 || K2 == 256;
    }
    if (N != 64 && N != 128 && N != 256) return false;
    const int LPR = N / 16;
    return (KH & (KH - 1)) == 0 && KH <= LPR;
}

int pruned1d_modes(int N, int K)
{
    for (int k = 16; k <= N; k <<= 1)
        if (k >= K && pruned1d_supported(N, k)) return k;
    return 0;
}

static long long mode_tiles(long long B, int K) { return (B * K + 127) / 128; }

// Grid of a grid-stride transform kernel: as many workgroups as the chip holds at once (asked of the runtime once per
// kernel), then trimmed so that every workgroup runs the same number of sweeps.  A fixed grid of 1024 ran the N = 1024
// kernels (three workgroups per CU, 768 at once) as one full round plus a round of 256 workgroups on an empty chip.
template <auto Kern>
static unsigned balanced_grid(long long sweeps, int threads)
{
    static std::once_flag once;
    static long long slots = 0;
    std::call_once(once, [&] {
        int per_cu = 0, dev = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, Kern, threads, 0) != hipSuccess || per_cu < 1) per_cu = 2;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
            cus = 256;
        slots = (long long)per_cu * cus;
    });
    if (sweeps <= slots) return (unsigned)sweeps;
    const long long rounds = (sweeps + slots - 1) / slots;
    return (unsigned)((sweeps + rounds - 1) / rounds);
}

size_t pruned1d_workspace_bytes(long long B, int C_in, int C_out, int K)
{
    return sizeof(c64) * (size_t)mode_tiles(B, K) * 128 * ((size_t)C_in + C_out);
}

size_t pruned1d_spectrum_elems(long long B, int C, int Mp) { return (size_t)mode_tiles(B, Mp) * 128 * (size_t)C; }

int pruned1d_stride(int N, int K, int K_keep, bool per_mode)
{
    if (N < 2048) {
        // The kept bins in 64-byte rows, or all of the kernel's where the masks of cut spectra cost more than the shorter
        // spectra save: past 7/8 of them where the contraction weighs most, in kernels that keep all N bins (B 512, 128 channels, 128
        // points: 112 modes 93.4 us cut and 97 in full, 120 modes 100.6 and 96.6) and with own weights per mode up to 256 points (B 64,
        // 28 -> 256 channels, 256 points, 100 modes 28.1 and 29.9); past 3/4 in the others (B 256: 1024 real points, 128 channels,
        // own weights, 100 modes 113 and 106; 256 points, 64 channels, shared weights, 100 modes 35.9 and 32.8).
        const int s = spectrum_stride(K_keep);
        return (K == N || (per_mode && N <= 256) ? 8 * s > 7 * K : 4 * s > 3 * K) ? K : s;
    }
    // Long pencils: whole columns of the N1 x 256 array, and all of the kernel's K2 columns where less than an eighth
    // of them would go: the masks then cost what the shorter spectra save (B 64, 128 x 128 channels, 2048 points: 63 of 64
    // columns 95.8 us masked, 94.8 in full; 34 of 64 columns 88.7 against 92.6; B 32, 4096 points, 57 of 64: 99.0 both).
    const int N1 = N / 256, cols = (K_keep + N1 - 1) / N1;
    int K2 = 16;
    while (K2 < cols) K2 *= 2;
    return (8 * cols > 7 * K2 ? K2 : cols) * N1;
}

template <int N, int K, bool REAL, int FORM>
static hipError_t launch_fwd(const c64 *x, c64 *Xh, int C, long long pencils, int K_keep, int Mp, hipStream_t s)
{
    using Cf = CfgP1<N, K>;
    // a few sweeps per workgroup amortise the twiddle tables and keep a prefetch in flight
    // (measured: the forward kernels gain 2 - 4 % and the real-valued inverse 13 % from the balanced grid; the complex
    // inverse kernels, which write twice the bytes, lose 4 % and keep the fixed grid)
    const unsigned grid = balanced_grid<&k_fwd1d<N, K, REAL, FORM>>((pencils + Cf::PPS - 1) / Cf::PPS, 256);
    hipLaunchKernelGGL((k_fwd1d<N, K, REAL, FORM>), dim3(grid), dim3(256), 0, s, x, Xh, C, pencils, K_keep, Mp, 0LL, 0LL);
    return hipGetLastError();
}

template <int N, int K, bool REAL, int FORM>
static hipError_t launch_inv(const c64 *Yh, c64 *y, int C, long long pencils, int K_keep, int Mp, hipStream_t s)
{
    using Cf = CfgP1<N, K>;
    const long long sweeps = (pencils + Cf::PPS - 1) / Cf::PPS;
    const unsigned grid = REAL ? balanced_grid<&k_inv1d<N, K, REAL, FORM>>(sweeps, 256) : (unsigned)(sweeps < 1024 ? sweeps : 1024);
    hipLaunchKernelGGL((k_inv1d<N, K, REAL, FORM>), dim3(grid), dim3(256), 0, s, Yh, y, C, pencils, K_keep, Mp, 0LL);
    return hipGetLastError();
}

template <int N, int K, bool REAL = false>
static hipError_t launch_nk(int stages, const c64 *x, const c64 *W, c64 *y, c64 *Xh, c64 *Yh, long long B, int C_in,
                            int C_out, int K_keep, int Mp, hipStream_t s)
{
    const long long pin = B * C_in, pout = B * C_out;
    hipError_t e = hipSuccess;
    if (stages & PRUNED_FWD) {
        e = Mp < K ? launch_fwd<N, K, REAL, P1_CUT>(x, Xh, C_in, pin, K_keep, Mp, s)
            : K_keep < K ? launch_fwd<N, K, REAL, P1_FULL>(x, Xh, C_in, pin, K_keep, Mp, s)
                         : launch_fwd<N, K, REAL, P1_ALL>(x, Xh, C_in, pin, K_keep, Mp, s);
        if (e != hipSuccess) return e;
    }
    if (stages & PRUNED_GEMM)
        if ((e = cgemm_modes_launch(Xh, W, Yh, C_in, C_out, 1.0f / (float)N, mode_tiles(B, Mp), s)) != hipSuccess) return e;
    if (stages & PRUNED_INV)
        e = Mp < K ? launch_inv<N, K, REAL, P1_CUT>(Yh, y, C_out, pout, K_keep, Mp, s)
                   : launch_inv<N, K, REAL, P1_ALL>(Yh, y, C_out, pout, K_keep, Mp, s);
    return e;
}

template <int N1, int K2, bool ALL>
static hipError_t launch_long(int stages, const c64 *x, const c64 *W, c64 *y, c64 *Xh, c64 *Yh, long long B, int C_in,
                              int C_out, int K_keep, int Mp, hipStream_t s)
{
    using Cf = CfgLong<N1, K2>;
    const long long tiles = mode_tiles(B, Mp);
    const int K2k = Mp / N1;
    const long long pin = B * C_in, pout = B * C_out;
    const long long sin = (pin + Cf::G - 1) / Cf::G, sout = (pout + Cf::G - 1) / Cf::G;
    const unsigned gin = balanced_grid<&k_fwd1d_long<N1, K2, ALL>>(sin, 256), gout = (unsigned)(sout < 2048 ? sout : 2048);
    hipError_t e = hipSuccess;
    if (stages & PRUNED_FWD) {
        hipLaunchKernelGGL((k_fwd1d_long<N1, K2, ALL>), dim3(gin), dim3(256), 0, s, x, Xh, C_in, pin, K_keep, K2k);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (stages & PRUNED_GEMM)
        if ((e = cgemm_modes_launch(Xh, W, Yh, C_in, C_out, 1.0f / (float)Cf::N, tiles, s)) != hipSuccess) return e;
    if (stages & PRUNED_INV) {
        hipLaunchKernelGGL((k_inv1d_long<N1, K2, ALL>), dim3(gout), dim3(256), 0, s, (const c64 *)Yh, y, C_out, pout, K2k);
        e = hipGetLastError();
    }
    return e;
}

template <int N1, int K2>
static hipError_t launch_long(int stages, const c64 *x, const c64 *W, c64 *y, c64 *Xh, c64 *Yh, long long B, int C_in,
                              int C_out, int K_keep, int Mp, hipStream_t s)
{
    if (Mp == N1 * K2) return launch_long<N1, K2, true>(stages, x, W, y, Xh, Yh, B, C_in, C_out, K_keep, Mp, s);
    return launch_long<N1, K2, false>(stages, x, W, y, Xh, Yh, B, C_in, C_out, K_keep, Mp, s);
}

template <int N1>
static hipError_t launch_long_n(int K2, int stages, const c64 *x, const c64 *W, c64 *y, c64 *Xh, c64 *Yh, long long B,
                                int C_in, int C_out, int K_keep, int Mp, hipStream_t s)
{
    switch (K2) {
    case 16: return launch_long<N1, 16>(stages, x, W, y, Xh, Yh, B, C_in, C_out, K_keep, Mp, s);
    case 32: return launch_long<N1, 32>(stages, x, W, y, Xh, Yh, B, C_in, C_out, K_keep, Mp, s);
    case 64: return launch_long<N1, 64>(stages, x, W, y, Xh, Yh, B, C_in, C_out, K_keep, Mp, s);
    case 128: return launch_long<N1, 128>(stages, x, W, y, Xh, Yh, B, C_in, C_out, K_keep, Mp, s);
    case 256: return launch_long<N1, 256>(stages, x, W, y, Xh, Yh, B, C_in, C_out, K_keep, Mp, s);
    default: return hipErrorInvalidValue;
    }
}

template <int N, bool REAL = false>
static hipError_t launch_n(int K, int stages, const c64 *x, const c64 *W, c64 *y, c64 *Xh, c64 *Yh, long long B,
                           int C_in, int C_out, int K_keep, int Mp, hipStream_t s)
{
    constexpr int LPR = N / 16;
    switch (K) {
    case 16: return launch_nk<N, 16, REAL>(stages, x, W, y, Xh, Yh, B, C_in, C_out, K_keep, Mp, s);
    case 32: if constexpr (LPR >= 2) return launch_nk<N, 32, REAL>(stages, x, W, y, Xh, Yh, B, C_in, C_out, K_keep, Mp, s); break;
    case 64: if constexpr (LPR >= 4) return launch_nk<N, 64, REAL>(stages, x, W, y, Xh, Yh, B, C_in, C_out, K_keep, Mp, s); break;
    case 128: if constexpr (LPR >= 8) return launch_nk<N, 128, REAL>(stages, x, W, y, Xh, Yh, B, C_in, C_out, K_keep, Mp, s); break;
    case 256: if constexpr (LPR >= 16) return launch_nk<N, 256, REAL>(stages, x, W, y, Xh, Yh, B, C_in, C_out, K_keep, Mp, s); break;
    default: break;
    }
    return hipErrorInvalidValue;
}

hipError_t pruned1d_stages(int stages, const c64 *x, const c64 *W, c64 *y, c64 *Xh, c64 *Yh, long long B, int C_in,
                           int C_out, int N, int K, int K_keep, int Mp, hipStream_t s)
{
    if (!pruned1d_supported(N, K) || K_keep < 1 || K_keep > K || Mp > K || Mp < K_keep || (N < 2048 ? Mp % 8 : Mp % (N / 256)) != 0)
        return hipErrorInvalidValue;
    switch (N) {
    case 64: return launch_n<64>(K, stages, x, W, y, Xh, Yh, B, C_in, C_out, K_keep, Mp, s);
    case 128: return launch_n<128>(K, stages, x, W, y, Xh, Yh, B, C_in, C_out, K_keep, Mp, s);
    case 256: return launch_n<256>(K, stages, x, W, y, Xh, Yh, B, C_in, C_out, K_keep, Mp, s);
    case 1024:
        if (K == 64) return launch_nk<1024, 64>(stages, x, W, y, Xh, Yh, B, C_in, C_out, K_keep, Mp, s);
        return launch_nk<1024, 128>(stages, x, W, y, Xh, Yh, B, C_in, C_out, K_keep, Mp, s);
    case 2048: return launch_long_n<8>(K / 8, stages, x, W, y, Xh, Yh, B, C_in, C_out, K_keep, Mp, s);
    case 4096: return launch_long_n<16>(K / 16, stages, x, W, y, Xh, Yh, B, C_in, C_out, K_keep, Mp, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t pruned1d_real_stages(int stages, const float *x, float *y, c64 *Xh, c64 *Yh, long long B, int C_in, int C_out,
                                int N, int K, int K_keep, int Mp, hipStream_t s)
{
    if (!pruned1d_supported(N, K) || N > 1024 || K_keep < 1 || K_keep > K || Mp > K || Mp < K_keep || (stages & PRUNED_GEMM))
        return hipErrorInvalidValue;
    const c64 *xc = reinterpret_cast<const c64 *>(x);
    c64 *yc = reinterpret_cast<c64 *>(y);
    switch (N) {
    case 64: return launch_n<64, true>(K, stages, xc, nullptr, yc, Xh, Yh, B, C_in, C_out, K_keep, Mp, s);
    case 128: return launch_n<128, true>(K, stages, xc, nullptr, yc, Xh, Yh, B, C_in, C_out, K_keep, Mp, s);
    case 256: return launch_n<256, true>(K, stages, xc, nullptr, yc, Xh, Yh, B, C_in, C_out, K_keep, Mp, s);
    case 1024:
        if (K == 64) return launch_nk<1024, 64, true>(stages, xc, nullptr, yc, Xh, Yh, B, C_in, C_out, K_keep, Mp, s);
        return launch_nk<1024, 128, true>(stages, xc, nullptr, yc, Xh, Yh, B, C_in, C_out, K_keep, Mp, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t pruned1d_launch(const c64 *x, const c64 *W, c64 *y, long long B, int C_in, int C_out, int N, int K,
                           int K_keep, c64 *ws, hipStream_t s)
{
    const int Mp = pruned1d_stride(N, K, K_keep);
    return pruned1d_stages(PRUNED_FWD | PRUNED_GEMM | PRUNED_INV, x, W, y, ws, ws + pruned1d_spectrum_elems(B, C_in, Mp),
                           B, C_in, C_out, N, K, K_keep, Mp, s);
}

// Outputs per workgroup: results for at most two lanes' worth of a wave, but workgroups for every CU.
static int permode_outputs(long long B, int C_out, int N, int Ma)
{
    const int pencils = 4096 / N;                           // that 256 lanes transform
    int G = pencils < 16 ? pencils : 16;
    while (G > 1 && (G * Ma > 128 || B * ((C_out + G - 1) / G) < 256)) G /= 2;
    return G;
}

// Every batch element reads the weights again, and every workgroup sets up its twiddles: up to 20 MB of the one and three of the other for every CU the
// launch and the latency that are saved weigh more (whole layers, two kernels after the forward transform against one: B 32, 64 x 64 channels, N 1024, 16
// modes, 16.8 MB, 512 workgroups 13.6 and 10.9 us; B 15, 22 -> 41, N 64, 13 modes 11.6 and 8.7; B 11, 82 -> 72, N 128, 39 modes, 20.3 MB 11.9 and 13.1; B 8,
// 15 -> 98, N 256, 79 modes, 784 workgroups 11.5 and 11.9; B 182, 13 -> 32, N 128, 16 modes, 728 workgroups 11.5 and 8.8; B 54, 62 -> 96, N 256, 45 modes, 116 MB 19.9 and 31.4).
// A wave walks a quarter of the channels, 16 at a time, or 8 with results for two lanes each, where a contraction of its own spreads them over the chip: up to two steps
// of the latter, three of the former, eight where no workgroup waits for a CU (in a graph, two kernels and one: B 3, 186 -> 2, N 256, 90 modes 13.0 and 16.4; B 10, 95 -> 11, N 256,
// 103 modes, 110 workgroups 14.3 and 13.5; B 8, 636 -> 45, N 64, 3 modes, 360 workgroups 19.1 and 26.3; B 9, 373 -> 76, N 128, 7 modes, 342 workgroups 15.5 and 18.7; B 20, 166 -> 10, N 64,
// 15 modes, 200 workgroups 11.9 and 9.9; B 7, 365 -> 31, N 128, 7 modes, 217 workgroups 14.9 and 13.1; 2000 channels up to 2.1 times as slow).
bool pruned1d_permode_fused(long long B, int C_in, int C_out, int N, int K, int Ma)
{
    if (N > 1024 || !pruned1d_supported(N, K) || Ma > 256) return false;
    if (B > 768 || B * C_out > (1LL << 24) || B * C_in * C_out * (long long)Ma * (long long)sizeof(c64) > 20000000) return false;
    const int G = permode_outputs(B, C_out, N, Ma);
    const long long workgroups = B * ((C_out + G - 1) / G);
    return workgroups <= 768 && C_in <= (G * Ma > 64 ? 64 : workgroups > 256 ? 192 : 512);
}

template <int N, int K, bool REAL>
static hipError_t launch_permode(const c64 *Xh, const c64 *W, c64 *y, long long B, int C_in, int C_out, int Ma, int Mp, float scale, hipStream_t s)
{
    const int G = permode_outputs(B, C_out, N, Ma), slabs = (C_out + G - 1) / G;
    hipLaunchKernelGGL((k_inv1d_permode<N, K, REAL>), dim3((unsigned)(B * slabs)), dim3(256), 0, s, Xh, W, y, C_in, C_out, Mp, Ma, G, slabs, scale);
    return hipGetLastError();
}

template <int N, bool REAL>
static hipError_t permode_k(int K, const c64 *Xh, const c64 *W, c64 *y, long long B, int C_in, int C_out, int Ma, int Mp, float scale, hipStream_t s)
{
    switch (K) {
    case 16: if constexpr (N <= 256) return launch_permode<N, 16, REAL>(Xh, W, y, B, C_in, C_out, Ma, Mp, scale, s); break;
    case 32: if constexpr (N <= 256) return launch_permode<N, 32, REAL>(Xh, W, y, B, C_in, C_out, Ma, Mp, scale, s); break;
    case 64: return launch_permode<N, 64, REAL>(Xh, W, y, B, C_in, C_out, Ma, Mp, scale, s);
    case 128: if constexpr (N >= 128) return launch_permode<N, 128, REAL>(Xh, W, y, B, C_in, C_out, Ma, Mp, scale, s); break;
    case 256: if constexpr (N == 256) return launch_permode<N, 256, REAL>(Xh, W, y, B, C_in, C_out, Ma, Mp, scale, s); break;
    default: break;
    }
    return hipErrorInvalidValue;
}

template <bool REAL>
static hipError_t permode_n(const c64 *Xh, const c64 *W, c64 *y, long long B, int C_in, int C_out, int N, int K, int Ma, int Mp, float scale, hipStream_t s)
{
    switch (N) {
    case 64: return permode_k<64, REAL>(K, Xh, W, y, B, C_in, C_out, Ma, Mp, scale, s);
    case 128: return permode_k<128, REAL>(K, Xh, W, y, B, C_in, C_out, Ma, Mp, scale, s);
    case 256: return permode_k<256, REAL>(K, Xh, W, y, B, C_in, C_out, Ma, Mp, scale, s);
    case 1024: return permode_k<1024, REAL>(K, Xh, W, y, B, C_in, C_out, Ma, Mp, scale, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t pruned1d_permode_inverse(bool real, const c64 *Xh, const c64 *W, c64 *y, long long B, int C_in, int C_out, int N, int K, int Ma,
                                    int Mp, float scale, hipStream_t s)
{
    if (Ma < 1 || Ma > K || Mp < Ma || !pruned1d_permode_fused(B, C_in, C_out, N, K, Ma)) return hipErrorInvalidValue;
    return real ? permode_n<true>(Xh, W, y, B, C_in, C_out, N, K, Ma, Mp, scale, s) : permode_n<false>(Xh, W, y, B, C_in, C_out, N, K, Ma, Mp, scale, s);
}

// Input pencils whose bins an output pencil has room for beside its own: rows of 128 bins, two of them for every part.
static int channels_per_pencil(bool real, int C_in, int C_out)
{
    const int pitch = real ? 512 : 1024;                    // complex numbers in an output pencil
    int g = 1;
    while (g * (long long)C_out < C_in) g *= 2;
    return pitch / g >= 256 ? g : 0;
}

// A fused workgroup takes its row's channels 8 at a time, 0.42 us per channel however few rows there are; the three kernels take about as long as their
// bytes at 4 TB/s, and both some 9 us besides (fused and three kernels, us: B 4, C 32, K 64 23 and 12; B 48, C 128 56 and 33; B 48, 200 -> 100 91 and 44; B 100,
// C 32 23 and 20, 16 -> 64 18.7 and 20.9; real rows, C 128, B 90 65 and 41, B 180, on the symmetric kernel, 73 and 83).
// Up to 8 channels are one step of a fused workgroup, and three launches cost more than what its few slabs of outputs wait for (1 -> 1 channels, B 13, K 5, real
// rows 8.8 and 11.6; 8 -> 2, B 5, K 43 10.4 and 11.6; 8 -> 13, B 3, K 5 13.0 and 11.9).
bool pruned1d_in_y_supported(bool real, long long B, int C_in, int C_out, int N, int K_keep)
{
    if (N != 1024 || K_keep < 1 || K_keep > 128 || B >= (1LL << 24) || !channels_per_pencil(real, C_in, C_out)) return false;
    if (C_in <= 8 && C_out <= (real ? 16 : 8)) return false;
    const double bytes = (real ? 4.0 : 8.0) * N * (double)B * ((double)C_in + C_out);
    return bytes <= (real ? 1.2e6 : 1.6e6) * C_in;
}

template <int K, bool REAL>
static hipError_t rows_in_y(const void *x, const c64 *W, void *y, long long B, int C_in, int C_out, int K_keep, hipStream_t s)
{
    constexpr int N = 1024, pitch = REAL ? N / 2 : N;
    using Cf = CfgP1<N, K>;
    const int g = channels_per_pencil(REAL, C_in, C_out), channel = pitch / g;
    const long long batch = (long long)C_out * pitch, pin = B * C_in, pout = B * C_out;
    c64 *Yh = reinterpret_cast<c64 *>(y), *Xh = Yh + 128;
    const unsigned gin = balanced_grid<&k_fwd1d<N, K, REAL, P1_ROWS>>((pin + Cf::PPS - 1) / Cf::PPS, 256);
    const unsigned gout = balanced_grid<&k_inv1d<N, K, REAL, P1_ROWS>>((pout + Cf::PPS - 1) / Cf::PPS, 256);
    hipLaunchKernelGGL((k_fwd1d<N, K, REAL, P1_ROWS>), dim3(gin), dim3(256), 0, s, (const c64 *)x, Xh, C_in, pin, K_keep, K_keep, batch, (long long)channel);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = cgemm_rows_launch(Xh, W, Yh, C_in, C_out, (REAL ? 2.0f : 1.0f) / (float)N, B, K_keep, batch, channel, batch, pitch, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_inv1d<N, K, REAL, P1_ROWS>), dim3(gout), dim3(256), 0, s, (const c64 *)nullptr, Yh, C_out, pout, K_keep, K_keep, (long long)pitch);
    return hipGetLastError();
}

hipError_t pruned1d_in_y(bool real, const void *x, const c64 *W, void *y, long long B, int C_in, int C_out, int N, int K_keep, hipStream_t s)
{
    if (!pruned1d_in_y_supported(real, B, C_in, C_out, N, K_keep)) return hipErrorInvalidValue;
    if (K_keep <= 64) return real ? rows_in_y<64, true>(x, W, y, B, C_in, C_out, K_keep, s) : rows_in_y<64, false>(x, W, y, B, C_in, C_out, K_keep, s);
    return real ? rows_in_y<128, true>(x, W, y, B, C_in, C_out, K_keep, s) : rows_in_y<128, false>(x, W, y, B, C_in, C_out, K_keep, s);
}

}  // namespace tfno
