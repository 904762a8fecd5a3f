// Launcher of the matrix transform and the layer built from it.
#include "matdft_kernel.h"
#include "colfft.h"
#include "fused2d.h"          // cgemm_modes_launch
#include "matgrid.h"
#include "matrow.h"
#include "pruned1d.h"
#include "staged.h"           // launch_axis_fft

namespace tfno {

template <int JT, int WI, int NMAX, int IN, int OUT, bool VEC>
static hipError_t launch_fwd(MatdftArgs a, hipStream_t s)
{
    using Cf = CfgMdF<JT, WI, NMAX>;
    constexpr int nt = Cf::NT;
    constexpr size_t lds = Cf::LDS;
    static LdsLimitOnce limit;
    const hipError_t e = limit.set({reinterpret_cast<const void *>(&k_matdft_fwd<JT, WI, NMAX, IN, OUT, VEC>)}, (int)lds);
    if (e != hipSuccess) return e;
    a.groups = (a.K + 32 * JT - 1) / (32 * JT);
    const unsigned long long items = (unsigned long long)((a.P + 31) / 32) * a.groups;
    const unsigned long long blocks = WI > 1 ? items : (items + 3) / 4;
    if (blocks > 0x7fffffffULL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_matdft_fwd<JT, WI, NMAX, IN, OUT, VEC>), dim3((unsigned)blocks), dim3(nt), lds, s, a);
    return hipGetLastError();
}
// (two sizes of the root table)
template <int JT, int WI, int IN, int OUT, bool VEC>
static hipError_t launch_fwd(const MatdftArgs &a, hipStream_t s)
{
    return a.N <= 1024 ? launch_fwd<JT, WI, 1024, IN, OUT, VEC>(a, s) : launch_fwd<JT, WI, 4096, IN, OUT, VEC>(a, s);
}

template <int IN, int OUT, bool VEC>
static hipError_t pick_fwd(const MatdftArgs &a, hipStream_t s)
{
    const unsigned long long tiles = (a.P + 31) / 32;
    const int kt = (a.K + 31) / 32;
    // Output tiles per wave: the input is fetched, folded and split once per wave, so as many as divide the outputs best --
    // unless that leaves the chip's 1024 SIMDs without a wave; then fewer, and the sum dealt out to 4 or 8 waves.
    int w = 1;
    for (int c = 2; c <= 4; ++c)
        if ((kt + c - 1) / c * c <= (kt + w - 1) / w * w && tiles * ((kt + c - 1) / c) >= 1024) w = c;
    if constexpr (IN == MD_ROWS && !VEC)                    // (fewer than 40 points: one wave to a sum, at most two tiles)
        return w == 2 ? launch_fwd<2, 1, 1024, IN, OUT, VEC>(a, s) : launch_fwd<1, 1, 1024, IN, OUT, VEC>(a, s);
    const unsigned long long waves = tiles * ((kt + w - 1) / w);
    // (64 to 127 points have 3 or 4 blocks of 16 slots to deal out, worth it while most of the chip is idle: 8 fields of 123 x 3
    // points, all modes, whole layer 32.5 -> 28.5 us, 28.5 us with direct sums)
    const int parts = waves >= 1024 || a.N < (waves < 256 ? 64 : 128) ? 1 : waves >= 256 || a.N < 256 ? 4 : 8;
    switch (w) {
    case 4: return launch_fwd<4, 1, IN, OUT, VEC>(a, s);
    case 3: return launch_fwd<3, 1, IN, OUT, VEC>(a, s);
    case 2: return launch_fwd<2, 1, IN, OUT, VEC>(a, s);
    default:
        // (1-D layers with so few pencils and 256 points or more run k_matrow_fwd, but for 1025 to 1632 pencils with more than 128 modes, for which four
        // parts measured level with eight: 11 x 99 pencils, 200 modes, 398 to 2411 points 34.1 against 33.7 to 53.8 against 54.8 us the layer)
        if constexpr (!(IN == MD_ROWS && OUT == MD_SPEC)) {
            if (parts == 8) return launch_fwd<1, 8, IN, OUT, VEC>(a, s);
        }
        return parts >= 4 ? launch_fwd<1, 4, IN, OUT, VEC>(a, s) : launch_fwd<1, 1, IN, OUT, VEC>(a, s);
    }
}

template <int PT, int NMAX, int IN, int OUT, int G = 0>
static hipError_t launch_inv(MatdftArgs a, hipStream_t s)
{
    // (G: the eight pencils that each of the 4 / G groups of waves puts together, N < 128 G points each)
    constexpr size_t most = MdRoots<NMAX>::BYTES + 16 + (G ? sizeof(c64) * 4 / (G ? G : 1) * 8 * (128 * G - 1) : 0);
    static LdsLimitOnce limit;
    const hipError_t e = limit.set({reinterpret_cast<const void *>(&k_matdft_inv<PT, NMAX, IN, OUT, G>)}, (int)most);
    if (e != hipSuccess) return e;
    const size_t lds = MdRoots<NMAX>::BYTES + 16 + (G ? sizeof(c64) * 4 / (G ? G : 1) * 8 * a.N : 0);
    a.groups = G ? G : (a.N / 2 + 32 * PT) / (32 * PT);     // output pairs 0 .. N/2
    const unsigned long long blocks = ((unsigned long long)((a.P + 31) / 32) * a.groups + 3) / 4;
    if (blocks > 0x7fffffffULL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_matdft_inv<PT, NMAX, IN, OUT, G>), dim3((unsigned)blocks), dim3(256), lds, s, a);
    return hipGetLastError();
}

template <int IN, int OUT>
static hipError_t pick_inv(const MatdftArgs &a, hipStream_t s)
{
    const unsigned long long tiles = (a.P + 31) / 32;
    if constexpr (OUT == MD_ROWS) {
        // Whole pencils per workgroup for outputs that the caches do not hold and that fill the chip this way: layers whose
        // buffers change from call to call, outputs of 40, 80, 160 MB: 85 points 40.6 -> 39.8, 74.0 -> 63.9, 122.8 -> 113.4 us,
        // 200 points 40.3 -> 40.2, 72.8 -> 60.7, 120.8 -> 112.5 us, 500 points 41.8 -> 41.3, 71.4 -> 61.2, 134.1 -> 115.1 us.
        // Where more than 3/8 of the pairs that the waves cover are padding, only larger outputs gain (257 points, 16 -> 16
        // channels: 39.7 -> 45.0, 75.0 -> 66.1, 113.6 -> 112.1 us; 4 -> 16: 32.2 -> 38.4, 49.8 -> 50.8, 77.3 -> 72.4 us).  Below 64 points half the pairs would be padding: 48 x 60 points 47 -> 50 us.
        const int G = a.N < 128 ? 1 : a.N < 256 ? 2 : 4;
        const unsigned long long bytes = (unsigned long long)a.P * a.N * sizeof(c64), least = 8 * (a.N / 2 + 1) < 5 * 64 * G ? 64ULL << 20 : 32ULL << 20;
        if (a.N >= 64 && a.N < 512 && a.out_outer == a.N && bytes >= least && tiles * G >= 1024) {
            if (G == 1) return launch_inv<2, 1024, IN, OUT, 1>(a, s);
            return G == 2 ? launch_inv<2, 1024, IN, OUT, 2>(a, s) : launch_inv<2, 1024, IN, OUT, 4>(a, s);
        }
    }
    // two tiles of output pairs per wave where they divide the pairs evenly and leave a wave for every SIMD
    const int nt = (a.N / 2 + 32) / 32;
    const bool two = nt % 2 == 0 && tiles * (nt / 2) >= 1024;
    if (a.N <= 1024) return two ? launch_inv<2, 1024, IN, OUT>(a, s) : launch_inv<1, 1024, IN, OUT>(a, s);
    return two ? launch_inv<2, 4096, IN, OUT>(a, s) : launch_inv<1, 4096, IN, OUT>(a, s);
}

static bool args_ok(const MatdftArgs &a) { return a.N >= 2 && a.N <= 4096 && a.K >= 1 && a.K <= a.N && a.inner >= 1 && a.C >= 1; }

hipError_t matdft_forward(MatdftSide in_side, MatdftSide out_side, MatdftArgs a, hipStream_t s)
{
    if (!args_ok(a)) return hipErrorInvalidValue;
    if (a.P == 0) return hipSuccess;
    const bool vec = a.N >= 40;
    if (in_side == MD_ROWS && out_side == MD_SPEC) return vec ? pick_fwd<MD_ROWS, MD_SPEC, true>(a, s) : pick_fwd<MD_ROWS, MD_SPEC, false>(a, s);
    if (in_side == MD_ROWS && out_side == MD_ROWS) return vec ? pick_fwd<MD_ROWS, MD_ROWS, true>(a, s) : pick_fwd<MD_ROWS, MD_ROWS, false>(a, s);
    if (in_side == MD_STRIDED && out_side == MD_SPEC) return pick_fwd<MD_STRIDED, MD_SPEC, false>(a, s);
    return hipErrorInvalidValue;
}

hipError_t matdft_inverse(MatdftSide in_side, MatdftSide out_side, MatdftArgs a, hipStream_t s)
{
    if (!args_ok(a)) return hipErrorInvalidValue;
    if (a.P == 0) return hipSuccess;
    if (in_side == MD_SPEC && out_side == MD_ROWS) return pick_inv<MD_SPEC, MD_ROWS>(a, s);
    if (in_side == MD_SPEC && out_side == MD_STRIDED) return pick_inv<MD_SPEC, MD_STRIDED>(a, s);
    if (in_side == MD_ROWS && out_side == MD_ROWS) return pick_inv<MD_ROWS, MD_ROWS>(a, s);
    return hipErrorInvalidValue;
}

static long long mode_tiles(long long B, long long M) { return (B * M + 127) / 128; }

static bool is_pow2(int n) { return (n & (n - 1)) == 0; }

// 2-D: columns of the fields transformed along their last axis, K2 or, from the row kernels of powers of two, their
// stride (its bins past K2 are zeros)
static int row_modes(int N2, int K2)
{
    const int K = is_pow2(N2) ? pruned1d_modes(N2, K2) : 0;
    const int rows = K ? 0 : pruned1d_row_stride(N2, K2);
    return K ? pruned1d_stride(N2, K, K2) : rows ? rows : K2;
}

// workspace: Xh, Yh in whole tiles of 128 modes; 2-D: the fields transformed along their last axis, [B, C, N1, cols],
// input and output in turn in the same place
size_t matdft_workspace_bytes(long long B, int C_in, int C_out, int N1, int N2, int K1, int K2)
{
    const int cols = N1 > 1 ? row_modes(N2, K2) : K2;
    const size_t spectra = (size_t)mode_tiles(B, (long long)K1 * cols) * 128 * ((size_t)C_in + C_out);
    const size_t half = N1 > 1 ? (size_t)B * N1 * cols * (size_t)(C_in > C_out ? C_in : C_out) : 0;
    return sizeof(c64) * (spectra + half);
}

// The two axes of a 2-D layer.  A side that is a power of two keeps a butterfly transform: one 32-bit sum per bin has 2 to 6
// times its error (4096 x 3 points, all modes: 1.1e-6 against 2.0e-7 for the whole layer), and its time grows with the
// modes that are kept (same grid: 315 against 74 us).
namespace {
struct Grid { int N1, N2, K1, K2, cols; long long M; hipStream_t s; };

// last axis, `rows` pencils: [rows, N2] <-> [rows, cols]
hipError_t last_axis(int dir, const Grid &g, const c64 *in, c64 *out, long long rows)
{
    if (is_pow2(g.N2)) {
        const int K = pruned1d_modes(g.N2, g.K2);
        // (the spectrum of one channel is [rows, cols])
        if (K && dir < 0) return pruned1d_stages(PRUNED_FWD, in, nullptr, nullptr, out, nullptr, rows, 1, 1, g.N2, K, g.K2, g.cols, g.s);
        if (K) return pruned1d_stages(PRUNED_INV, nullptr, nullptr, out, nullptr, const_cast<c64 *>(in), rows, 1, 1, g.N2, K, g.K2, g.cols, g.s);
        if (pruned1d_row_stride(g.N2, g.K2)) return pruned1d_rows(dir, in, out, rows, g.N2, g.K2, g.s);
        if (dir < 0) return launch_axis_fft(-1, in, out, g.N2, rows, 1, g.N2, g.cols, 1, g.N2, g.K2, 1.f, g.s);
        return launch_axis_fft(+1, in, out, g.N2, rows, 1, g.cols, g.N2, 1, g.K2, g.N2, 1.f, g.s);
    }
    MatdftArgs a{};
    a.in = in; a.out = out; a.N = g.N2; a.K = g.K2; a.P = (unsigned)rows; a.inner = 1; a.C = 1;
    a.in_outer = dir < 0 ? g.N2 : g.cols;
    a.out_outer = dir < 0 ? g.cols : g.N2;
    return dir < 0 ? matdft_forward(MD_ROWS, MD_ROWS, a, g.s) : matdft_inverse(MD_ROWS, MD_ROWS, a, g.s);
}

// first axis, columns of B fields of C channels: [B, C, N1, cols] <-> spectrum
hipError_t first_axis(int dir, const Grid &g, const c64 *in, c64 *out, long long B, int C)
{
    if (is_pow2(g.N1)) {
        if (colfft_supported(g.N1, g.K1)) return colfft_spec_launch(dir, in, out, B * C, g.N1, g.cols, g.K1, C, g.M, g.s);
        return launch_axis_fft_spec(dir, in, out, g.N1, g.K1, B * C, g.cols, C, g.M, g.s);
    }
    MatdftArgs a{};
    a.in = in; a.out = out; a.N = g.N1; a.K = g.K1; a.P = (unsigned)(B * C * g.cols); a.inner = (unsigned)g.cols; a.C = C; a.M = g.M;
    a.in_outer = a.out_outer = (long long)g.N1 * g.cols;
    return dir < 0 ? matdft_forward(MD_STRIDED, MD_SPEC, a, g.s) : matdft_inverse(MD_SPEC, MD_STRIDED, a, g.s);
}
}  // namespace

hipError_t matdft_conv(const c64 *x, const c64 *W, c64 *y, long long B, int C_in, int C_out, int N1, int N2, int K1, int K2,
                       c64 *ws, hipStream_t s)
{
    const int cols = N1 > 1 ? row_modes(N2, K2) : K2;
    const Grid g{N1, N2, K1, K2, cols, (long long)K1 * cols, s};
    const long long tiles = mode_tiles(B, g.M);
    const float scale = 1.0f / ((float)N1 * (float)N2);
    c64 *Xh = ws, *Yh = Xh + (size_t)tiles * 128 * C_in, *T = Yh + (size_t)tiles * 128 * C_out;
    hipError_t e;
    if (N1 == 1) {
        MatdftArgs a{};
        a.in = x; a.out = Xh; a.N = N2; a.K = K2; a.P = (unsigned)(B * C_in); a.inner = 1; a.in_outer = N2; a.C = C_in; a.M = g.M;
        const MatrowArgs r{x, W, Xh, y, (int)B, C_in, C_out, N2, K2, scale, 0, 0};
        e = matrow_forward_supported(B, C_in, N2, K2) ? matrow_forward(r, s) : matdft_forward(MD_ROWS, MD_SPEC, a, s);
        if (e != hipSuccess) return e;
        if (matrow_inverse_supported(B, C_in, C_out, N2, K2)) return matrow_inverse(r, s);
        if ((e = cgemm_modes_launch(Xh, W, Yh, C_in, C_out, scale, tiles, s, true)) != hipSuccess) return e;
        a.in = Yh; a.out = y; a.P = (unsigned)(B * C_out); a.out_outer = N2; a.C = C_out;
        return matdft_inverse(MD_SPEC, MD_ROWS, a, s);
    }
    const bool odd = !is_pow2(N1) && !is_pow2(N2);
    if (odd && matgrid_supported(-1, B * C_in, N1, N2, K1, K2)) {
        if ((e = matgrid_launch(-1, x, Xh, B * C_in, C_in, N1, N2, K1, K2, s)) != hipSuccess) return e;
    } else {
        if ((e = last_axis(-1, g, x, T, B * C_in * N1)) != hipSuccess) return e;
        if ((e = first_axis(-1, g, T, Xh, B, C_in)) != hipSuccess) return e;
    }
    if ((e = cgemm_modes_launch(Xh, W, Yh, C_in, C_out, scale, tiles, s, true)) != hipSuccess) return e;
    if (odd && matgrid_supported(+1, B * C_out, N1, N2, K1, K2)) return matgrid_launch(+1, Yh, y, B * C_out, C_out, N1, N2, K1, K2, s);
    if ((e = first_axis(+1, g, Yh, T, B, C_out)) != hipSuccess) return e;
    return last_axis(+1, g, T, y, B * C_out * N1);
}

}  // namespace tfno
