// Launcher of the per-mode-weight contraction.
#include "cgemm_permode_kernel.h"
#include "cgemm_permode_mfma_kernel.h"
#include "fused1d.h"
#include "fused2d.h"

namespace tfno {

template <int BT, int OT, int KS>
static void launch_f32(const c64 *Xh, const c64 *W, c64 *Yh, int C_in, int C_out, long long B, int Mp, int Ma, int Mc, float scale,
                       hipStream_t s)
{
    const unsigned long long threads = (unsigned long long)((B + BT - 1) / BT) * Mc;
    const unsigned slabs = (unsigned)((C_out + OT - 1) / OT);
    constexpr unsigned RESULTS = 256 / KS;
    const dim3 grid((unsigned)((threads + RESULTS - 1) / RESULTS * slabs));
    auto run = Mc > Ma ? &k_cgemm_permode<BT, OT, true, KS> : &k_cgemm_permode<BT, OT, false, KS>;
    hipLaunchKernelGGL(run, grid, dim3(256), 0, s, Xh, W, Yh, C_in, C_out, B, Mp, Ma, Mc, scale, slabs);
}

hipError_t cgemm_permode_launch(const c64 *Xh, const c64 *W, c64 *Yh, int C_in, int C_out, long long B, int Mp, int Ma,
                                bool zeros, float scale, hipStream_t s)
{
    if (B <= 0) return hipSuccess;
    if (Ma < 1 || Mp < Ma || Mp % 8 != 0) return hipErrorInvalidValue;
    // Matrix-pipe kernel from 36 workgroups' worth of results on, 48 below 32 channels (its time hardly falls below that: whole layers of 64 x 64
    // channels, 256 points, with either kernel, FP32 first: 262144 results 22.1 and 22.6 us, 327680 results 29.9 and 24.9 us;
    // 16 modes, B 64: 19.2 and 20.9 us; 18 -> 256 channels, 327680 results: 19.2 and 22.4 us), with enough channels, outputs and batch elements for its 32 x 32 x 8-channel
    // tiles; everything else (and TFNO_CONTRACTION=f32) runs the FP32 kernel.
    const long long gy = (B + 31) / 32, gz = (C_out + 31) / 32;
    if (C_in >= 16 && C_out >= 16 && B >= 16 && B * Ma * C_out >= (C_in < 32 ? 48 : 36) * 8192 && !contraction_forced_f32() && gy <= 65535 && gz <= 65535) {
        const dim3 grid((unsigned)(Mp / 8), (unsigned)gy, (unsigned)gz);
        // without masks where every tile is full and the extents a workgroup addresses with 32-bit offsets (32 batch
        // elements of Xh, all of W) stay below 2^31 bytes
        const bool fits32 = (32LL * Mp + 256) * C_in * 8 < (1LL << 31) && (long long)C_in * C_out * Ma * 8 < (1LL << 31);
        const bool full = B % 32 == 0 && C_out % 32 == 0 && C_in % 8 == 0 && fits32;
        // (eight partial products below 32 channels where they are hidden: with more than 64 modes they take up to 9 %)
        auto run = C_in < 32 && Mp <= 64 ? (full ? &k_cgemm_permode_mfma<true, 8> : &k_cgemm_permode_mfma<false, 8>)
                                         : (full ? &k_cgemm_permode_mfma<true, 6> : &k_cgemm_permode_mfma<false, 6>);
        hipLaunchKernelGGL(run, grid, dim3(512), 0, s, Xh, W, Yh, C_in, C_out, B, Mp, Ma, scale);
        return hipGetLastError();
    }
    const int Mc = zeros ? Mp : Ma;
    // Batch elements x outputs per thread: more reuse of what is loaded where that still gives every SIMD a wave.
    auto waves = [&](int bt, int ot) { return (B + bt - 1) / bt * Ma * ((C_out + ot - 1) / ot) / 64; };
    if (waves(8, 8) >= 1024) launch_f32<8, 8, 1>(Xh, W, Yh, C_in, C_out, B, Mp, Ma, Mc, scale, s);
    else if (waves(4, 4) >= 1024) launch_f32<4, 4, 1>(Xh, W, Yh, C_in, C_out, B, Mp, Ma, Mc, scale, s);
    else if (waves(2, 2) >= 256) {
        if (C_in > 8) launch_f32<2, 2, 4>(Xh, W, Yh, C_in, C_out, B, Mp, Ma, Mc, scale, s);     // more than one block of channels
        else launch_f32<2, 2, 1>(Xh, W, Yh, C_in, C_out, B, Mp, Ma, Mc, scale, s);
    } else {
        if (C_in > 16) launch_f32<1, 1, 4>(Xh, W, Yh, C_in, C_out, B, Mp, Ma, Mc, scale, s);
        else launch_f32<1, 1, 1>(Xh, W, Yh, C_in, C_out, B, Mp, Ma, Mc, scale, s);
    }
    return hipGetLastError();
}

}  // namespace tfno
