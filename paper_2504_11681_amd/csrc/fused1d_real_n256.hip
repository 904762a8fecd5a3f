// Real-valued layer: fused-kernel instantiations for N = 256.
#include "fused1d_kernel.h"

namespace tfno {

// At most a workgroup of 32 (K <= 64: or 64) outputs per CU: eight waves to a workgroup, as for complex rows (B 64, C 64, 64 modes
// 10.5 -> 8.3 us; B 44, 249 -> 48, 96 modes 43.8 -> 31.5; B 128, C 128, 64 modes 22.1 -> 18.9).  Not with so few channels that four waves take them in
// one block, where the larger workgroup only costs its barriers (64 modes: B 14, 2 -> 1 5.5 against 5.9 us, B 2, 16 -> 32 5.7 and 6.1, B 23, 19 -> 7 7.8 and 6.0;
// 128 modes: B 1, 7 -> 2 5.9 and 6.1; 32 modes level).
int fused1d_real_eight_waves(int K, long long rows, int C_in, int C_out)
{
    if (K != 32 && K != 64 && K != 128) return 0;
    if (rows * ((C_out + 31) / 32) <= 256) return C_in > (K == 64 ? 16 : K == 128 ? 8 : 0) ? 1 : 0;
    return K != 128 && rows * ((C_out + 63) / 64) <= 256 ? 2 : 0;
}

template <int K>
static hipError_t launch_few_rows(const Fused1dArgs &a, long long rows, hipStream_t s, bool *done)
{
    const int slabs = fused1d_real_eight_waves(K, rows, a.C_in, a.C_out);
    *done = slabs != 0;
    if (slabs == 1) return launch_fused1d_impl<256, K, 1, true, 0, true, 8, 1, split_steps_over_waves<256, K, 1, 8>()>(a, rows, s);
    if constexpr (K != 128) {
        if (slabs == 2) return launch_fused1d_impl<256, K, 2, true, 0, true, 8, 1, split_steps_over_waves<256, K, 2, 8>()>(a, rows, s);
    }
    return hipSuccess;
}

hipError_t fused1d_real_launch_n256(int K, const Fused1dArgs &a, long long rows, hipStream_t s)
{
    if (!contraction_forced_f32() && !generic_kernels_forced()) {
        bool done = false;
        hipError_t e = hipSuccess;
        switch (K) {
        case 32: e = launch_few_rows<32>(a, rows, s, &done); break;
        case 64: e = launch_few_rows<64>(a, rows, s, &done); break;
        case 128: e = launch_few_rows<128>(a, rows, s, &done); break;
        default: break;
        }
        if (done) return e;
    }
    switch (K) {
    case 16: return launch_fused1d_real<256, 16, 4>(a, rows, s);
    case 32: return launch_fused1d_real<256, 32, 4>(a, rows, s);
    case 64: return launch_fused1d_real<256, 64, 4>(a, rows, s);
    case 128: return launch_fused1d_real<256, 128, 4>(a, rows, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace tfno
