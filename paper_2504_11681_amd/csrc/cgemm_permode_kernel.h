// Contraction over the hidden dimension with an own weight matrix per retained mode (the learned transformation of
// the Fourier layer as the FNO model defines it, Sec. 1 / Sec. 2.1 step 3; Sec. 3.1 treats the case of one shared
// matrix, which the MFMA kernels of cgemm_modes_kernel.h cover):
//
//   Yh[b, o, m] = scale * sum_c Xh[b, c, m] * W[c, o, m],   m < Ma;     0,   Ma <= m < Mc
//
// Spectra are mode-tile major ([tile][channel][128]) over the joint mode b Mp + m, W is [C_in, C_out, Ma]; Mc is
// Ma, or Mp where the surplus modes have to be zeros (ZEROS: the last threads store them).  FP32 kernel
// for products too small for the matrix pipe (cgemm_permode_mfma_kernel.h): a thread owns one mode of BT batch elements
// and OT outputs, so a W value loaded is used BT times and an Xh value OT times; the threads of a wave own consecutive
// modes (coalesced runs of Ma) and, where Ma is short, of consecutive batch groups.  Bound by the latency of the loads:
// U channels are in flight, and BT and OT are chosen small enough to give the chip a wave per SIMD (B 32, 16 modes, 64 x 64
// channels: 51 -> 7 us against 8 x 8 per thread, which made 8 workgroups; one wave for all channels).
// KS: waves that share a result's channels.  With one or four results per thread a wave's chain of U-channel blocks, a memory
// latency each, is the whole time; four waves take every fourth block and the sums meet in LDS.  Whole layers, one wave and four:
// B 32, 16 modes, 64 x 64 channels, 1024 real points 15.6 and 12.8 us; B 16, 16 modes, 128 x 128 channels, 256 points 17.4 and 13.4 us; B 7,
// 27 -> 41 channels, 128 x 256, 32 x 24 modes 37.7 and 35.0 us.  The channels left over take a block of 8, 4, 2 and 1, not one after the other
// (B 25, 12 -> 7 channels, 64 x 64: 16.4 and 14.2 us).
#pragma once
#include "common.h"
#include <type_traits>

namespace tfno {

template <int BT, int OT, bool ZEROS, int KS>
__global__ void __launch_bounds__(256, 2)
k_cgemm_permode(const c64 *__restrict__ Xh, const c64 *__restrict__ W, c64 *__restrict__ Yh, int C_in, int C_out,
                long long B, int Mp, int Ma, int Mc, float scale, unsigned slabs)
{
    constexpr int U = BT + OT <= 2 ? 16 : BT + OT <= 4 ? 8 : BT + OT <= 8 ? 4 : 2;
    constexpr int RESULTS = 256 / KS;                       // threads' worth of results per workgroup
    const int slot = threadIdx.x % RESULTS;
    const int part = KS > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / RESULTS) : 0;
    const unsigned long long f = blockIdx.x / slabs * (unsigned long long)RESULTS + slot;    // (slabs of OT outputs innermost)
    const int o0 = (int)(blockIdx.x % slabs) * OT;
    auto spec = [&](long long b, int m, int C) __attribute__((always_inline)) {   // element (b, channel 0, m)
        const long long j = b * Mp + m;
        return (j >> 7) * C * 128 + (j & 127);
    };
    if constexpr (ZEROS) {                                  // (a branch of their own: in the sums' loops they cost 0.4 us)
        const unsigned long long sums = (unsigned long long)((B + BT - 1) / BT) * (unsigned)Ma;      // threads that have a sum
        if (f >= sums && part == 0) {
            const unsigned extra = (unsigned)(Mc - Ma);
            const long long z0 = (long long)((f - sums) / extra) * BT;
            const int m = Ma + (int)((f - sums) % extra);
            for (long long b = z0; b < z0 + BT && b < B; ++b)
                for (int o = o0; o < o0 + OT && o < C_out; ++o) Yh[spec(b, m, C_out) + (long long)o * 128] = make_float2(0.f, 0.f);
        }
    }
    const long long grp = (long long)(f / (unsigned)Ma);
    const bool mine = grp * BT < B;                         // (with KS > 1 every wave reaches the barrier)
    if (KS == 1 && !mine) return;
    const long long b0 = mine ? grp * BT : 0;
    const int m = (int)(f % (unsigned)Ma);

    const c64 *xp[BT];
#pragma unroll
    for (int bi = 0; bi < BT; ++bi) xp[bi] = Xh + spec(b0 + bi < B ? b0 + bi : B - 1, m, C_in);
    const c64 *wp[OT];
#pragma unroll
    for (int oi = 0; oi < OT; ++oi) wp[oi] = W + (long long)(o0 + oi < C_out ? o0 + oi : C_out - 1) * Ma + m;
    const long long wstep = (long long)C_out * Ma;

    c64 acc[BT][OT];
#pragma unroll
    for (int bi = 0; bi < BT; ++bi)
#pragma unroll
        for (int oi = 0; oi < OT; ++oi) acc[bi][oi] = make_float2(0.f, 0.f);

    auto block = [&](int c0, auto count) __attribute__((always_inline)) {
        constexpr int n = decltype(count)::value;
        c64 xv[n][BT], wv[n][OT];
#pragma unroll
        for (int u = 0; u < n; ++u) {
#pragma unroll
            for (int oi = 0; oi < OT; ++oi) wv[u][oi] = wp[oi][(c0 + u) * wstep];
#pragma unroll
            for (int bi = 0; bi < BT; ++bi) xv[u][bi] = xp[bi][(long long)(c0 + u) * 128];
        }
        __builtin_amdgcn_sched_barrier(0);
        // (a sum per block where there are few results per thread: one chain over all channels rounds more than the matrix
        // pipe's sums do, which this kernel stands in for at small sizes)
        constexpr bool SPLIT = BT * OT <= 4 && n > 1;
        c64 part[BT][OT];
#pragma unroll
        for (int bi = 0; bi < BT; ++bi)
#pragma unroll
            for (int oi = 0; oi < OT; ++oi) part[bi][oi] = SPLIT ? make_float2(0.f, 0.f) : acc[bi][oi];
#pragma unroll
        for (int u = 0; u < n; ++u)
#pragma unroll
            for (int bi = 0; bi < BT; ++bi)
#pragma unroll
                for (int oi = 0; oi < OT; ++oi) part[bi][oi] = cmac(part[bi][oi], xv[u][bi], wv[u][oi]);
#pragma unroll
        for (int bi = 0; bi < BT; ++bi)
#pragma unroll
            for (int oi = 0; oi < OT; ++oi) acc[bi][oi] = SPLIT ? cadd(acc[bi][oi], part[bi][oi]) : part[bi][oi];
    };
    int c = part * U;
    for (; c + U <= C_in; c += KS * U) block(c, std::integral_constant<int, U>{});
    if (c < C_in) {                                         // (KS > 1: of the wave whose next block is the incomplete one)
        if constexpr (U >= 16) { if (c + 8 <= C_in) { block(c, std::integral_constant<int, 8>{}); c += 8; } }
        if constexpr (U >= 8) { if (c + 4 <= C_in) { block(c, std::integral_constant<int, 4>{}); c += 4; } }
        if constexpr (U >= 4) { if (c + 2 <= C_in) { block(c, std::integral_constant<int, 2>{}); c += 2; } }
        if (c < C_in) block(c, std::integral_constant<int, 1>{});
    }

    if constexpr (KS > 1) {
        __shared__ c64 sums[KS - 1][BT * OT][RESULTS];
        if (part > 0) {
#pragma unroll
            for (int i = 0; i < BT * OT; ++i) sums[part - 1][i][slot] = acc[i / OT][i % OT];
        }
        __syncthreads();
        if (part > 0 || !mine) return;
#pragma unroll
        for (int k = 0; k < KS - 1; ++k)
#pragma unroll
            for (int i = 0; i < BT * OT; ++i) acc[i / OT][i % OT] = cadd(acc[i / OT][i % OT], sums[k][i][slot]);
    }
#pragma unroll
    for (int bi = 0; bi < BT; ++bi) {
        if (b0 + bi >= B) continue;
        c64 *yp = Yh + spec(b0 + bi, m, C_out);
#pragma unroll
        for (int oi = 0; oi < OT; ++oi)
            if (o0 + oi < C_out) yp[(long long)(o0 + oi) * 128] = make_float2(acc[bi][oi].x * scale, acc[bi][oi].y * scale);
    }
}

}  // namespace tfno
