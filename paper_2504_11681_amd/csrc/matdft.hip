// Launcher of the matrix transform and the layer built from it.
#include "matdft_kernel.h"
#include "fused2d.h"          // cgemm_modes_launch

namespace tfno {

template <int JT, int WI, int IN, int OUT>
static hipError_t launch_md(MatdftArgs a, hipStream_t s)
{
    static LdsLimitOnce limit;
    const hipError_t e = limit.set({reinterpret_cast<const void *>(&k_matdft<JT, WI, IN, OUT>)}, (int)CfgMd<JT, WI>::lds_bytes(4096));
    if (e != hipSuccess) return e;
    a.jgroups = (a.J + 32 * JT - 1) / (32 * JT);
    const unsigned long long items = (unsigned long long)((a.P + 31) / 32) * a.jgroups;
    const unsigned long long blocks = WI > 1 ? items : (items + 3) / 4;
    if (blocks > 0x7fffffffULL) return hipErrorInvalidValue;
    const size_t lds = CfgMd<JT, WI>::lds_bytes(a.N);
    constexpr int nt = CfgMd<JT, WI>::NT;
    hipLaunchKernelGGL((k_matdft<JT, WI, IN, OUT>), dim3((unsigned)blocks), dim3(nt), lds, s, a);
    return hipGetLastError();
}

template <int IN, int OUT>
static hipError_t pick_md(const MatdftArgs &a, hipStream_t s)
{
    const unsigned long long tiles = (a.P + 31) / 32;
    const int jt = (a.J + 31) / 32;
    // Output tiles per wave: the input is fetched and split once per wave, so as many as divide the outputs best -- unless
    // that leaves the chip's 1024 SIMDs without a wave; then fewer, and the sum over the input dealt out to 4 or 8 waves.
    // (three and four tiles between a spectrum and a leading axis spill)
    constexpr int most = IN == MD_SPEC && OUT == MD_STRIDED ? 2 : 4;
    int w = 1;
    for (int c = 2; c <= most; ++c)
        if ((jt + c - 1) / c * c <= (jt + w - 1) / w * w && tiles * ((jt + c - 1) / c) >= 1024) w = c;
    const unsigned long long waves = tiles * ((jt + w - 1) / w);
    const int parts = waves >= 1024 || a.I < 128 ? 1 : waves >= 256 || a.I < 256 ? 4 : 8;
    if constexpr (most == 4) {
        if (w == 4) return launch_md<4, 1, IN, OUT>(a, s);
        if (w == 3) return launch_md<3, 1, IN, OUT>(a, s);
    }
    switch (w) {
    case 2: return launch_md<2, 1, IN, OUT>(a, s);
    default:
        return parts == 8 ? launch_md<1, 8, IN, OUT>(a, s) : parts == 4 ? launch_md<1, 4, IN, OUT>(a, s) : launch_md<1, 1, IN, OUT>(a, s);
    }
}

hipError_t matdft_launch(MatdftSide in_side, MatdftSide out_side, MatdftArgs a, hipStream_t s)
{
    if (a.N < 1 || a.N > 4096 || a.I < 1 || a.I > a.N || a.J < 1 || a.J > a.N || a.inner < 1) return hipErrorInvalidValue;
    if (a.P == 0) return hipSuccess;
    switch (in_side * 4 + out_side) {
    case MD_ROWS * 4 + MD_ROWS: return pick_md<MD_ROWS, MD_ROWS>(a, s);
    case MD_ROWS * 4 + MD_SPEC: return pick_md<MD_ROWS, MD_SPEC>(a, s);
    case MD_SPEC * 4 + MD_ROWS: return pick_md<MD_SPEC, MD_ROWS>(a, s);
    case MD_STRIDED * 4 + MD_SPEC: return pick_md<MD_STRIDED, MD_SPEC>(a, s);
    case MD_SPEC * 4 + MD_STRIDED: return pick_md<MD_SPEC, MD_STRIDED>(a, s);
    default: return hipErrorInvalidValue;
    }
}

static long long mode_tiles(long long B, long long M) { return (B * M + 127) / 128; }

// workspace: Xh, Yh in whole tiles of 128 modes; 2-D: the fields transformed along their last axis, [B, C, N1, K2],
// input and output in turn in the same place
size_t matdft_workspace_bytes(long long B, int C_in, int C_out, int N1, int N2, int K1, int K2)
{
    (void)N2;
    const size_t spectra = (size_t)mode_tiles(B, (long long)K1 * K2) * 128 * ((size_t)C_in + C_out);
    const size_t half = N1 > 1 ? (size_t)B * N1 * K2 * (size_t)(C_in > C_out ? C_in : C_out) : 0;
    return sizeof(c64) * (spectra + half);
}

hipError_t matdft_conv(const c64 *x, const c64 *W, c64 *y, long long B, int C_in, int C_out, int N1, int N2, int K1, int K2,
                       c64 *ws, hipStream_t s)
{
    const long long M = (long long)K1 * K2, tiles = mode_tiles(B, M);
    c64 *Xh = ws, *Yh = Xh + (size_t)tiles * 128 * C_in, *T = Yh + (size_t)tiles * 128 * C_out;
    MatdftArgs f{}, g{};
    hipError_t e;
    // last axis, truncated
    f.in = x; f.N = N2; f.I = N2; f.J = K2; f.inner = 1; f.in_outer = N2; f.dir = -1;
    f.P = (unsigned)(B * C_in * N1); f.C = C_in; f.M = M;
    // leading axis
    g.N = N1; g.inner = (unsigned)K2; g.M = M;
    if (N1 == 1) {
        f.out = Xh;
        e = matdft_launch(MD_ROWS, MD_SPEC, f, s);
    } else {
        f.out = T; f.out_outer = K2;
        e = matdft_launch(MD_ROWS, MD_ROWS, f, s);
        g.in = T; g.in_outer = (long long)N1 * K2; g.out = Xh; g.I = N1; g.J = K1; g.dir = -1;
        g.P = (unsigned)(B * C_in * K2); g.C = C_in;
        if (e == hipSuccess) e = matdft_launch(MD_STRIDED, MD_SPEC, g, s);
    }
    if (e != hipSuccess) return e;
    if ((e = cgemm_modes_launch(Xh, W, Yh, C_in, C_out, 1.0f / ((float)N1 * (float)N2), tiles, s)) != hipSuccess) return e;
    f.dir = +1; f.I = K2; f.J = N2; f.C = C_out; f.P = (unsigned)(B * C_out * N1); f.out = y; f.out_outer = N2;
    if (N1 == 1) {
        f.in = Yh;
        return matdft_launch(MD_SPEC, MD_ROWS, f, s);
    }
    g.in = Yh; g.out = T; g.out_outer = (long long)N1 * K2; g.I = K1; g.J = N1; g.dir = +1;
    g.P = (unsigned)(B * C_out * K2); g.C = C_out;
    if ((e = matdft_launch(MD_SPEC, MD_STRIDED, g, s)) != hipSuccess) return e;
    f.in = T; f.in_outer = K2;
    return matdft_launch(MD_ROWS, MD_ROWS, f, s);
}

}  // namespace tfno
