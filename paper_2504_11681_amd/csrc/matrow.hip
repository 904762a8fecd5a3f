// Launcher of the 1-D layer's kernels for lengths that are no powers of two.
#include "matrow_kernel.h"

namespace tfno {

namespace {
constexpr size_t MOST_LDS = 160 * 1024;
typedef void (*Kernel)(MatrowArgs);

int forward_parts(int N) { return N / 32 + 1 < MR_WAVES ? N / 32 + 1 : MR_WAVES; }
// sixteens of modes per wave: as few groups of at most four as there can be, of equal size; groups of at most two while most of the chip
// is idle (1 x 4 pencils of 3000 points, 200 modes: 43.4 -> 35.37 us the layer)
int forward_tiles(long long P, int K)
{
    const int all = (K + 15) / 16, most = (P + 15) / 16 * ((all + 1) / 2) <= 128 ? 2 : 4, groups = (all + most - 1) / most;
    return (all + groups - 1) / groups;
}
int forward_groups(long long P, int K) { return ((K + 15) / 16 + forward_tiles(P, K) - 1) / forward_tiles(P, K); }
size_t forward_lds(long long P, int N, int K) { return MG_ROOT * (size_t)N + sizeof(c64) * forward_parts(N) * 256 * forward_tiles(P, K); }

struct Inverse { int waves, parts, groups; size_t lds; };
Inverse inverse_plan(long long B, int C_in, int C_out, int N, int K)
{
    Inverse p{};
    const int tiles = N / 64 + 1, mt = (K + 31) / 32, steps = (C_in + 7) / 8;
    const long long slabs = B * ((C_out + 31) / 32);
    // eight waves, or with two workgroups for every CU and few outputs as many as have a tile of them
    p.waves = slabs < 512 || tiles >= MR_WAVES ? MR_WAVES : tiles > mt ? tiles : mt;
    p.parts = p.waves / mt < steps ? p.waves / mt : steps;
    const int most = (tiles + p.waves - 1) / p.waves;
    p.groups = (int)(slabs * most <= 512 ? most : slabs >= 512 ? 1 : 512 / slabs);
    p.lds = MG_ROOT * (size_t)N + 16 * 64 * 6 * (size_t)mr_steps(K) + sizeof(c64) * p.parts * 32 * mr_pitch(K);
    return p;
}

template <bool LONG>
Kernel pick_fwd(int KT)
{
    switch (KT) {
    case 1: return k_matrow_fwd<1, LONG>;
    case 2: return k_matrow_fwd<2, LONG>;
    case 3: return k_matrow_fwd<3, LONG>;
    default: return k_matrow_fwd<4, LONG>;
    }
}
}  // namespace

bool matrow_forward_supported(long long B, int C_in, int N, int K)
{
    const long long P = B * C_in;
    if (N < 32 || N > 4096 || P < 1 || P > 16383 || forward_lds(P, N, K) > MOST_LDS) return false;
    // (few pencils: with 16384 of them and more the transform of one sum per wave has the chip full, 256 x 64 pencils of 500 points, 60 modes
    // 25 against 30 us; 64 x 128 of 500 points, 64 modes 16.0 -> 15.4, 64 x 40 of 1000, 50 modes 12.7 -> 11.1, 5 x 71 of 162, 9 modes 5.9 -> 4.0)
    // More than 64 modes are several workgroups to a tile of pencils, each of which fetches and folds them again, one to a CU: ahead while all
    // are there at once, or from 512 points on nearly fill a second round (whole layers: 33 x 33 pencils of 398 points, 195 modes, 276 workgroups 29.2 against 33.3;
    // 76 x 166 of 581, 241 modes 88 against 119; 67 x 34 of 977, 152 modes, 429 workgroups 61.3 -> 57.8).
    const long long workgroups = (P + 15) / 16 * forward_groups(P, K);
    if (forward_groups(P, K) > 1) return workgroups <= 256 || (N >= 512 && workgroups > 384 && workgroups <= 512);
    // Short sums, which a wave gets through by itself, lose earlier, with more modes sooner (whole layers: 103 x 43 of 203 points, 35 modes 14.5 against 16.6;
    // 29 x 163 of 130, 55 modes 18.5 and 21.8; 189 x 52 of 304, 50 modes 25.7 and 27.3; 64 x 128 of 50, 12 modes 22.6 -> 11.8).
    if (N < 256) return P <= (K <= 16 ? 8192 : 4096);
    return N >= 512 || K <= 32 || P <= 8192;
}

hipError_t matrow_forward(const MatrowArgs &args, hipStream_t s)
{
    if (!matrow_forward_supported(args.B, args.C_in, args.N, args.K)) return hipErrorInvalidValue;
    static LdsLimitOnce limit;
    const hipError_t e = limit.set({reinterpret_cast<const void *>(&k_matrow_fwd<1, false>), reinterpret_cast<const void *>(&k_matrow_fwd<2, false>),
                                    reinterpret_cast<const void *>(&k_matrow_fwd<3, false>), reinterpret_cast<const void *>(&k_matrow_fwd<4, false>),
                                    reinterpret_cast<const void *>(&k_matrow_fwd<1, true>), reinterpret_cast<const void *>(&k_matrow_fwd<2, true>),
                                    reinterpret_cast<const void *>(&k_matrow_fwd<3, true>), reinterpret_cast<const void *>(&k_matrow_fwd<4, true>)},
                                   (int)MOST_LDS);
    if (e != hipSuccess) return e;
    MatrowArgs a = args;
    a.parts = forward_parts(a.N);
    const int KT = forward_tiles((long long)a.B * a.C_in, a.K);
    const dim3 grid((unsigned)(((long long)a.B * a.C_in + 15) / 16), (unsigned)((a.K + 16 * KT - 1) / (16 * KT)));
    const Kernel kernel = a.N / 32 + 1 > 4 * a.parts ? pick_fwd<true>(KT) : pick_fwd<false>(KT);
    hipLaunchKernelGGL(kernel, grid, dim3(64 * a.parts), forward_lds((long long)a.B * a.C_in, a.N, a.K), s, a);
    return hipGetLastError();
}

bool matrow_inverse_supported(long long B, int C_in, int C_out, int N, int K)
{
    if (N < 32 || N > 4096 || K > 32 * MR_WAVES) return false;
    if ((long long)C_in * C_out >= (1LL << 28) || (long long)C_in * 128 >= (1LL << 28) || B * C_out >= (1LL << 31) / 32) return false;
    const Inverse p = inverse_plan(B, C_in, C_out, N, K);
    if (p.lds > MOST_LDS) return false;
    // A wave's share of the channels is one chain: with many modes, two waves or one to a sum, a contraction for all workgroups is ahead past 128 channels
    // (3 x 257 -> 13 channels, N 551, K 169: 42.3 and 45.6 us the layer).
    const long long slabs = (C_out + 31) / 32, steps = (C_in + 7) / 8;
    if (steps > 16 * p.parts) return false;
    // What is done beside the layer, for every CU.  The slab of a batch element is 32 outputs and whole tiles of 32 modes; separate kernels lay the outputs
    // (modes) of all batch elements side by side, and contract once where here every group of workgroups does.  In tiles of 32 outputs x 64 points x 16 modes (0.16 us)
    // and of 8 channels x 32 modes x 32 outputs (0.1 us), against some 4.5 us for a launch and the pass over the contracted spectrum that go: 617 batch elements, 1 -> 1 channels,
    // N 1713, K 121, 504 tiles beside the layer, 34.8 and 114 us; 282, 3 -> 10, N 1307, K 153 44.0 and 83.6; 547, 224 -> 269, N 77, K 4, 468 sums 71 and 112; 42, 44 -> 1,
    // N 1954, K 74, 24 tiles 30.5 and 26.6.  Several rounds of workgroups cost their latency besides (571, 1 -> 5, N 291, K 2, 9 tiles, two rounds 14.5 and 18.6; 453, 2 -> 17, N 273, K 50,
    // 17 tiles 25.2 and 21.5; 145, 3 -> 244, N 447, K 98, 10 tiles, five rounds 98.6 and 62.5).  Of 2400 drawn layers 21 are more than 3 % slower than with kernels of their own.
    const long long pairs = (long long)(N / 64 + 1) * mr_steps(K), mt = (K + 31) / 32, workgroups = B * slabs * p.groups;
    const double tiles = (double)(B * slabs - (B * C_out + 31) / 32) * pairs / 256, sums = (double)(workgroups * mt - (B * K + 127) / 128 * 4 * slabs) * steps / 256;
    const int by_waves = 12 / p.waves, by_lds = (int)(MOST_LDS / p.lds), resident = 256 * (by_waves < 1 ? 1 : by_waves < by_lds ? by_waves : by_lds);
    const double rounds = (double)((workgroups + resident - 1) / resident);
    const double out_us = (double)B * C_out * N * sizeof(c64) / 5e6, spectrum_us = (double)B * C_out * K * 2 * sizeof(c64) / 5e6;
    return sums <= 80 && (rounds > 1.0 ? 2.0 + rounds : 0.0) + 0.16 * tiles <= 4.5 + 1.5 * spectrum_us + 0.1 * out_us;
}

hipError_t matrow_inverse(const MatrowArgs &args, hipStream_t s)
{
    if (!matrow_inverse_supported(args.B, args.C_in, args.C_out, args.N, args.K)) return hipErrorInvalidValue;
    static LdsLimitOnce limit;
    const hipError_t e = limit.set({reinterpret_cast<const void *>(&k_matrow_inv<6>), reinterpret_cast<const void *>(&k_matrow_inv<8>)}, (int)MOST_LDS);
    if (e != hipSuccess) return e;
    MatrowArgs a = args;
    const Inverse p = inverse_plan(a.B, a.C_in, a.C_out, a.N, a.K);
    a.parts = p.parts;
    a.groups = p.groups;
    const long long blocks = (long long)a.B * ((a.C_out + 31) / 32) * a.groups;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((a.C_in <= 16 ? k_matrow_inv<8> : k_matrow_inv<6>), dim3((unsigned)blocks), dim3(64 * p.waves), p.lds, s, a);
    return hipGetLastError();
}

}  // namespace tfno
