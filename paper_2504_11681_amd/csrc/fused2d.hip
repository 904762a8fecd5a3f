// Mode CGEMM instantiations and the launcher of the 2-D pipeline (the image kernels live in fused2d_n*.hip).
#include "cgemm_modes_kernel.h"
#include "fused2d.h"
#include "fused1d.h"

namespace tfno {

bool fused2d_supported(int N1, int N2, int K1, int K2)
{
    auto n_ok = [](int n) { return n == 64 || n == 128 || n == 256; };
    auto k_ok = [](int k) { return k == 16 || k == 32 || k == 64; };
    return n_ok(N1) && n_ok(N2) && k_ok(K1) && k_ok(K2);
}

size_t fused2d_workspace_bytes(long long B, int C_in, int C_out, int K1, int K2)
{
    return sizeof(c64) * (size_t)B * K1 * K2 * ((size_t)C_in + C_out);
}

hipError_t cgemm_rows_launch(const c64 *Xh, const c64 *W, c64 *Yh, int C_in, int C_out, float scale, long long B, int K, long long x_batch, int x_channel,
                             long long y_batch, int y_channel, hipStream_t s)
{
    if (B < 1 || B >= (1LL << 24) || K < 1 || K > 128) return hipErrorInvalidValue;
    const dim3 grid((unsigned)B, (unsigned)((C_out + 31) / 32)), block(64 * ((K + 31) / 32));
    const ModeRows rows{x_batch, y_batch, x_channel, y_channel};
    if (C_in <= 16) hipLaunchKernelGGL((k_cgemm_modes_direct<2, 8, true>), grid, block, 0, s, Xh, W, Yh, C_in, C_out, scale, rows);
    else hipLaunchKernelGGL((k_cgemm_modes_direct<4, 6, true>), grid, block, 0, s, Xh, W, Yh, C_in, C_out, scale, rows);
    return hipGetLastError();
}

hipError_t cgemm_modes_launch(const c64 *Xh, const c64 *W, c64 *Yh, int C_in, int C_out, float scale, long long tiles,
                              hipStream_t s, bool all_products)
{
    // The direct kernel up to two workgroups per CU (at 512 of them 13.4 against 15.1 us with 64 channels and 20 against 27 us
    // with 128; at 800 and 1024 it loses, 23 against 18 us and 37 against 29 us), one per CU with more than 128 channels, whose
    // weights every wave splits again (whole layers, 256 points, 128 modes, 384 -> 64 channels, 160 and 280 workgroups: 50.1
    // against 69.9 us and 84.4 against 82.2 us), and for up to 32 outputs, where the others
    // would contract half a slab of padding (1024 tiles, C 64 -> 24: 22 against 25 us; 2048 tiles, C 32: 25 against 31 us).
    // (Up to 32 outputs: measured over 1 to 512 channels and up to 2048 tiles, 1.2 to 1.6 times the others' speed.)
    // A tile is a workgroup there, and a launch has fewer than 2^32 threads.
    if (!contraction_forced_f32() && (C_out <= 32 || tiles * ((C_out + 31) / 32) <= (C_in <= 128 ? 512 : 256)) && tiles < (1LL << 24)) {
        const dim3 gd((unsigned)tiles, (unsigned)((C_out + 31) / 32));
        if (C_in <= 16 && all_products) hipLaunchKernelGGL((k_cgemm_modes_direct<2, 8>), gd, dim3(256), 0, s, Xh, W, Yh, C_in, C_out, scale, ModeRows{});
        else if (C_in <= 16) hipLaunchKernelGGL((k_cgemm_modes_direct<2, 6>), gd, dim3(256), 0, s, Xh, W, Yh, C_in, C_out, scale, ModeRows{});
        else hipLaunchKernelGGL((k_cgemm_modes_direct<4, 6>), gd, dim3(256), 0, s, Xh, W, Yh, C_in, C_out, scale, ModeRows{});
        return hipGetLastError();
    }
    if (!contraction_forced_f32() && C_in <= 64) {
        // one block of W: the straight-line kernel, two mode tiles per workgroup
        const dim3 g2((unsigned)((tiles + 1) / 2), (unsigned)((C_out + 63) / 64));
        if (C_in <= 32)
            hipLaunchKernelGGL(k_cgemm_modes_small<4>, g2, dim3(256), 0, s, Xh, W, Yh, C_in, C_out, scale, tiles);
        else
            hipLaunchKernelGGL(k_cgemm_modes_small<8>, g2, dim3(256), 0, s, Xh, W, Yh, C_in, C_out, scale, tiles);
        return hipGetLastError();
    }
    if (!contraction_forced_f32() && C_in <= 128) {
        // all of W resident in LDS, eight waves, two mode tiles at a time; about one workgroup per CU
        const int c_pad = (C_in + 31) / 32 * 32, lds = c_pad * 3 * 64 * 4;
        static LdsLimitOnce lds_limit;
        const hipError_t e = lds_limit.set({reinterpret_cast<const void *>(&k_cgemm_modes_resident)}, 128 * 3 * 64 * 4);
        if (e != hipSuccess) return e;
        const long long pairs = (tiles + 1) / 2, gy = (C_out + 63) / 64;
        long long ppw = pairs * gy / 256;
        ppw = ppw < 1 ? 1 : ppw > 16 ? 16 : ppw;
        const dim3 gr((unsigned)((pairs + ppw - 1) / ppw), (unsigned)gy);
        hipLaunchKernelGGL(k_cgemm_modes_resident, gr, dim3(512), lds, s, Xh, W, Yh, C_in, C_out, scale, tiles, (int)ppw);
        return hipGetLastError();
    }
    // about two workgroups per CU, each walking several mode tiles
    const int tpw = tiles >= 1024 ? (int)(tiles / 512 > 16 ? 16 : tiles / 512) : 1;
    const dim3 ggrid((unsigned)((tiles + tpw - 1) / tpw), (unsigned)((C_out + 63) / 64));
    if (contraction_forced_f32())
        hipLaunchKernelGGL(k_cgemm_modes_f32, ggrid, dim3(256), 0, s, Xh, W, Yh, C_in, C_out, scale, tiles, tpw);
    else
        hipLaunchKernelGGL(k_cgemm_modes, ggrid, dim3(256), 0, s, Xh, W, Yh, C_in, C_out, scale, tiles, tpw);
    return hipGetLastError();
}

hipError_t fused2d_images(int dir, const c64 *in, c64 *out, long long images, int C, int N1, int N2, int K1, int K2,
                          int k1_keep, int k2_keep, bool fno, int h1, hipStream_t s)
{
    if (!fused2d_supported(N1, N2, K1, K2) || (fno && (h1 < 0 || h1 > K1))) return hipErrorInvalidValue;
    auto run = fno ? (N1 == 64 ? fused2d_fno_images_n64 : N1 == 128 ? fused2d_fno_images_n128 : fused2d_fno_images_n256)
                   : (N1 == 64 ? fused2d_images_n64 : N1 == 128 ? fused2d_images_n128 : fused2d_images_n256);
    return run(dir, in, out, images, C, N2, K1, K2, k1_keep, k2_keep, fno ? h1 : 0, s);
}

hipError_t fused2d_launch(const c64 *x, const c64 *W, c64 *y, long long B, int C_in, int C_out, int N1, int N2,
                          int K1, int K2, int k1_keep, int k2_keep, c64 *ws, hipStream_t s)
{
    // joint modes b Mp + m in whole tiles of 128: at most the K1 x K2 (a multiple of 128) modes per element of the workspace
    const long long tiles = (B * spectrum_stride(k1_keep * k2_keep) + 127) / 128;
    c64 *Xh = ws, *Yh = ws + (size_t)tiles * 128 * C_in;
    hipError_t e = fused2d_images(-1, x, Xh, B * C_in, C_in, N1, N2, K1, K2, k1_keep, k2_keep, false, 0, s);
    if (e != hipSuccess) return e;
    e = cgemm_modes_launch(Xh, W, Yh, C_in, C_out, 1.0f / ((float)N1 * (float)N2), tiles, s);
    if (e != hipSuccess) return e;
    return fused2d_images(+1, Yh, y, B * C_out, C_out, N1, N2, K1, K2, k1_keep, k2_keep, false, 0, s);
}

}  // namespace tfno
