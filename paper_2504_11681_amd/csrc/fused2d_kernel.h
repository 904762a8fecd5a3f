// 2-D spectral convolution for gfx950 as three kernels whose only HBM intermediates are the TRUNCATED
// spectra (K1 x K2 per image instead of the K x N strips of the 2-D pipeline in Sec. 3.2 / 3.3).  Images are
// N1 x N2 (N2 the contiguous axis); the first axis keeps its first K1 bins, the last its first K2; N (K) below
// stands for the length (mode count) of whichever axis a stage transforms.
//
//   k_fwd2d   one workgroup per input image x[b, c]: truncated, output-pruned 2-D forward transform
//             -> Xh[b, c, k1, k2], k1 < K1, k2 < K2                     (reads N1*N2, writes K1*K2)
//             stored mode-tile major, [j / 128][c][j % 128] over the joint mode j = b Mp + k1 K2 + k2 (of the modes
//             that are kept; Mp = their count rounded up to 8), so that the CGEMM streams contiguous [C, 128] blocks
//   k_cgemm_modes   (cgemm_modes_kernel.h) Yh[b, o, m] = sum_c Xh[b, c, m] * W[c, o] / (N1 N2) over the K1*K2
//             retained modes; one W for all modes (Sec. 3.1)
//   k_inv2d   one workgroup per output image: zero-padded, input-pruned 2-D inverse -> y[b, o]
//
// Both transforms are separable (Sec. 3.3).  With RP rows per pass (16 or 32) and S = N/RP the pruned first-axis
// transform is written as
//   X[k1] = sum_{r<S} w_N^(r k1) * F_r[k1 mod RP],   F_r = RP-point DFT of the rows n1 = r + S s, s < RP,
// so an image is processed in S passes of RP rows: the last-axis transform of these rows (truncated to K
// bins, Sec. 3.3) goes into an RP x K LDS tile, the RP-point column transform of that tile is accumulated
// into registers with the pass twiddle, and the full N x K strip never exists anywhere.  The inverse runs
// the transposed network: spectrum in registers, per pass a twiddled RP-point inverse column transform
// into the tile and zero-padded inverse row transforms of its rows.  The passes of an image can run in any
// order; workgroups start at different passes (see r_rot) because the rows of one pass map to few L2 channels.
//
// Row transform (N = 16 * LPR): LPR lanes per row, lane p holds x[p + LPR j], j < 16 (coalesced loads),
// 16-point DFT in registers, twiddle w_N^(p k_lo), transpose through a wave-private XOR-swizzled LDS patch,
// then the LPR-point DFT pruned to the K/16 retained outputs of each column k_lo (bins k_lo + 16 k_hi).
// Column transform: 4 adjacent lanes per tile column, RP/4-point DFT in registers, 4-point DFT across the quad
// with DPP.  All LDS accesses of the handoffs hit distinct banks per 16 lanes (the counterpart of the two
// swizzles of Sec. 4.1 / 4.2 for 8-byte accesses on wave64; checked with an LDS microbenchmark).
#pragma once
#include "common.h"
#include "fft_regs.h"
#include "fused1d_kernel.h"   // wave_sync, floatx16
#include "bf16x3.h"

namespace tfno {

// RP16: 16-row passes with two tile buffers (one barrier per pass) instead of 32-row passes with one buffer
template <int N1, int N2, int K1, int K2, bool RP16, bool FNO = false, bool INV = false>
struct Cfg2d {
    static constexpr int LPR = N2 / 16;                         // lanes per row
    static constexpr int RP = RP16 ? 16 : 32;                   // rows per pass
    static constexpr int RPS = (256 / LPR) < RP ? 256 / LPR : RP; // rows per sweep of the workgroup
    static constexpr int ACTIVE = RPS * LPR;                    // threads that take part in the row stage
    // Workgroup size: the larger of the row stage's threads and the column stage's (four lanes per column k2).  Rows
    // of 64 points keep 128 threads busy in the row stage; with 256 threads per workgroup half of every workgroup's
    // registers belonged to waves that only met the barriers, and half as many images were in flight per CU.
    static constexpr int NT = ACTIVE > 4 * K2 ? ACTIVE : 4 * K2;
    static constexpr int WG_PER_CU = 768 / NT;                  // twelve waves per CU whatever the workgroup size
    static constexpr int S = N1 / RP;                           // passes
    static constexpr int SWEEPS = RP / RPS;
    static constexpr int NSWEEP = S * SWEEPS;
    static constexpr int KH = K2 / 16;                          // retained outputs per column k_lo
    static constexpr int CPL = 16 / LPR;                        // columns k_lo per lane after the transpose
    static constexpr int COLS = FNO ? 9 : 16;                   // columns k_lo of a patch (real rows: 0..8)
    static constexpr int GS = FNO ? 9 * LPR : N2 + (LPR < 16 ? LPR : 0);    // patch stride between the rows of a sweep
    // FNO: the real rows of a wave also pass through its patches as plain floats, 16 bytes at a time on the side of the memory (a
    // row's lanes follow each other) and one by one (p + LPR j) on the side of the transforms; pitch FP puts the latter on 64 banks.
    static constexpr int RPW = 64 / LPR;                        // rows per wave
    static constexpr int FP = N2 + LPR, WREG = RPW * GS;
    static_assert(FP * sizeof(float) <= GS * sizeof(c64), "a row of floats is no longer than its patch");
    static constexpr int PATCHES = RPS * GS;
    static constexpr int TS = K2 + 4;                           // tile row stride (== 4 mod 16)
    static constexpr int RPL = RP / 4;                          // tile rows per lane in the column stage
    static constexpr int MREP = (K1 + RP - 1) / RP;             // k1 = k' + RP m
    // The column stage takes 4 K2 threads.  Where the row stage of the forward kernel keeps twice as many busy, two such groups
    // share it (H = 2), one with the even, one with the odd outputs of the lanes' register transforms (real 64 x 64 fields: the
    // CUs are busy for 147 instead of 152 thousand cycles).  The inverse kernel gains nothing from two groups with a pass each
    // (121 against 112: the second tile costs it two workgroups per CU).
    static constexpr int H = FNO && !INV && NT >= 8 * K2 ? 2 : 1;
    static constexpr int OUTS = INV ? RPL : RPL / H;            // first-axis residues of a lane
    static constexpr int NACC = OUTS * MREP;
    static constexpr int NBUF = RP == 16 ? 2 : 1;               // tile buffers (2: one barrier per pass)
    static constexpr size_t LDS_BYTES = sizeof(c64) * ((size_t)PATCHES + (size_t)NBUF * RP * TS + N1 + COLS * LPR);
    static_assert((N1 == 64 || N1 == 128 || N1 == 256) && (N2 == 64 || N2 == 128 || N2 == 256), "N in {64, 128, 256}");
    static_assert((K1 == 16 || K1 == 32 || K1 == 64) && (K2 == 16 || K2 == 32 || K2 == 64), "K in {16, 32, 64}");
    static_assert(K1 <= N1 && K2 <= N2 && KH <= LPR && LPR % KH == 0, "K must divide N");
    static_assert(LDS_BYTES <= 64 * 1024, "static LDS limit");
    static_assert(!FNO || (ACTIVE % 64 == 0 && WREG % 2 == 0), "whole waves, 16-byte aligned patches");
    static_assert(!FNO || 2 * K2 <= N2, "a real row has N2 / 2 bins of its own");
};

// value of lane (quad position PERM[q]) of the same quad
template <int CTRL>
__device__ __forceinline__ float quad_perm(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
constexpr int QP_XOR1 = 0xB1;   // [1, 0, 3, 2]
constexpr int QP_XOR2 = 0x4E;   // [2, 3, 0, 1]

// 4-point DFT across the four lanes of a quad, forward sign: lane q4 holds input q4 on entry and output
// kb = bitrev2(q4) on exit.
__device__ __forceinline__ c64 quad_dft4_fwd(c64 g, int q4)
{
    const float s2 = (q4 & 2) ? -1.f : 1.f, s1 = (q4 & 1) ? -1.f : 1.f;
    c64 t = make_float2(fmaf(s2, g.x, quad_perm<QP_XOR2>(g.x)), fmaf(s2, g.y, quad_perm<QP_XOR2>(g.y)));
    if (q4 == 3) t = make_float2(t.y, -t.x);                    // * (-i)
    return make_float2(fmaf(s1, t.x, quad_perm<QP_XOR1>(t.x)), fmaf(s1, t.y, quad_perm<QP_XOR1>(t.y)));
}
// transposed network, inverse sign: lane q4 holds input kb = bitrev2(q4) on entry and output q4 on exit.
__device__ __forceinline__ c64 quad_dft4_inv(c64 g, int q4)
{
    const float s2 = (q4 & 2) ? -1.f : 1.f, s1 = (q4 & 1) ? -1.f : 1.f;
    c64 t = make_float2(fmaf(s1, g.x, quad_perm<QP_XOR1>(g.x)), fmaf(s1, g.y, quad_perm<QP_XOR1>(g.y)));
    if (q4 == 3) t = make_float2(-t.y, t.x);                    // * (+i)
    return make_float2(fmaf(s2, t.x, quad_perm<QP_XOR2>(t.x)), fmaf(s2, t.y, quad_perm<QP_XOR2>(t.y)));
}

typedef float tfno_lds4 __attribute__((ext_vector_type(4)));

struct Lds2d {
    c64 *scr;    // [RPS][GS]   transpose patches, one per row of a sweep
    c64 *tile;   // [NBUF][RP][TS]  truncated rows of one pass
    c64 *tw;     // [COLS][LPR]   w_N2^(p k_lo)
    c64 *twn;    // [N1]        w_N1^t
};

template <class C>
__device__ __forceinline__ Lds2d lds_setup(unsigned char *raw)
{
    Lds2d l;
    l.scr = reinterpret_cast<c64 *>(raw);
    l.tile = l.scr + C::PATCHES;
    l.tw = l.tile + C::NBUF * C::RP * C::TS;
    l.twn = l.tw + C::COLS * C::LPR;
    return l;
}

// (the row table from the last thread down: in small workgroups the two tables are then the work of different waves)
template <class C, int N1, int N2>
__device__ __forceinline__ void lds_tables(const Lds2d &l, int tid)
{
    for (int i = C::NT - 1 - tid; i < C::COLS * C::LPR; i += C::NT) l.tw[i] = cis2pi(-(float)((i / C::LPR) * (i % C::LPR)), (float)N2);
    for (int i = tid; i < N1; i += C::NT) l.twn[i] = cis2pi(-(float)i, (float)N1);
}

// ------------------------------------------------------------------------------------------------ forward
// Element offsets of the modes m of one image (channel c of batch element b) in a mode-tile-major spectrum buffer with Mp modes per
// batch element (128 consecutive joint modes b Mp + m make a tile): the first tile and the position of mode 0 in it once per
// workgroup (uniform), so that a mode costs a shift, a mask and a multiply-add (in 64-bit arithmetic of its own, eight modes of a lane
// took 200 instructions).
struct SpecImage {
    long long base;
    int pos;
    unsigned tile;
    __device__ __forceinline__ SpecImage(long long b, int c, int C, int Mp)
        : base((((b * Mp) >> 7) * C + c) * 128), pos((int)((b * Mp) & 127)), tile((unsigned)C * 128u) {}
    __device__ __forceinline__ long long at(int m) const
    {
        const unsigned j = (unsigned)(pos + m);
        return base + (long long)((unsigned long long)(j >> 7) * tile + (j & 127u));
    }
};

// Sixteen-byte accesses to the RPW real rows of a wave (rows first, first + stride, ... of N2 floats at mem), four per lane: a row's
// N2 / 4 pieces belong to lanes that follow each other, so every access covers whole lines.  One by one, the floats p + LPR j of a
// lane's own row are 16-byte pieces of 16 lines for 64-point rows: four times the work for the address units, and partial lines
// cannot bypass the last-level cache, where outputs stay dirty and delay the next call's reads.
template <class C>
struct RowPieces {
    float *lds;
    int row, col;
    __device__ __forceinline__ RowPieces(c64 *scr, int tid)
    {
        const int lane = tid & 63;
        row = lane / (C::LPR * 4);
        col = 4 * (lane % (C::LPR * 4));
        lds = reinterpret_cast<float *>(scr + (tid >> 6) * C::WREG) + row * C::FP + col;
    }
    static constexpr int ROWS = 16 / C::LPR;                    // rows per access
    __device__ __forceinline__ tfno_lds4 *at(int j) const { return reinterpret_cast<tfno_lds4 *>(lds + j * ROWS * C::FP); }
};

// FNO (both kernels): the layer as FNO models apply it to real fields.  x and y are float32 images; the first axis
// keeps the frequencies k1 = -h1 .. K1-h1-1 (both low-frequency blocks; position j = k1 + h1 in the spectrum
// buffers) -- a thread's accumulator slots then stand for other frequencies of the same residue mod RP, which only
// changes the exponents of the pass twiddles --; the last axis is the R2C / C2R pair: the C2R inverse equals twice the real
// part of the zero-padded complex inverse once the k2 = 0 column is halved (done here, at the spectrum store).
// Row stage of a real row: the 16-point transforms of the lanes are real ones, whose bins 0..8 say it all, so only the columns
// k_lo = 0..8 are twiddled and go through the patch; bin k_lo + 16 k_hi, k_hi < 0, of such a column is the conjugate of bin
// -(k_lo + 16 k_hi), one of those that columns 9..15 would have given.  The inverse row stage is the mirror image: a
// column takes its bins of both signs, and the row is a sum of real parts.  Bound by memory, with the vector work close behind:
// 64 x 64 fields, 24 x 12 modes, B 256, 64 -> 64 channels: the three kernels took 181 us with complex rows and pieces of 16 and 32 bytes
// per row and access, 174 us with the networks of real rows, 133 us with whole lines past the caches as well (floor 107).
template <int N1, int N2, int K1, int K2, bool FNO = false>
__global__ void __launch_bounds__((Cfg2d<N1, N2, K1, K2, N2 == 256, FNO>::NT), (Cfg2d<N1, N2, K1, K2, N2 == 256, FNO>::WG_PER_CU))
k_fwd2d(const c64 *__restrict__ x, c64 *__restrict__ Xh, int C_in, int K1_keep, int K2_keep, int Mp, int h1)
{
    using C = Cfg2d<N1, N2, K1, K2, N2 == 256, FNO>;
    constexpr int LPR = C::LPR, RPS = C::RPS, S = C::S, SWEEPS = C::SWEEPS, KH = C::KH, CPL = C::CPL;
    constexpr int GS = C::GS, TS = C::TS, MREP = C::MREP, RP = C::RP, RPL = C::RPL, NBUF = C::NBUF;
    __shared__ __align__(16) unsigned char raw[C::LDS_BYTES];
    const int tid = threadIdx.x;
    const Lds2d L = lds_setup<C>(raw);

    // (workgroup id = image: giving each XCD a contiguous range of images, which helps the 1-D kernels, measured
    // 5-9 % slower here)
    using XT = std::conditional_t<FNO, float, c64>;
    const unsigned image = blockIdx.x;
    const XT *__restrict__ img = reinterpret_cast<const XT *>(x) + (long long)image * N1 * N2;
    // row-stage identity
    const bool row_on = tid < C::ACTIVE;
    const int g = tid / LPR, p = tid % LPR;
    c64 *scr = L.scr + g * GS;
    // column-stage identity
    const int hs = C::H == 2 ? __builtin_amdgcn_readfirstlane(tid / (4 * K2)) : 0;     // group (from H on: none)
    const int k2 = (tid - 4 * K2 * hs) >> 2, q4 = tid & 3, kb = ((q4 & 1) << 1) | (q4 >> 1);
    const bool col_on = C::H == 2 ? hs < 2 : k2 < K2;

    constexpr int OUTS = C::OUTS;
    auto slot_ka = [&](int i) __attribute__((always_inline)) { return C::H == 2 ? 2 * i + hs : i; };
    c64 acc[C::NACC];
#pragma unroll
    for (int i = 0; i < C::NACC; ++i) acc[i] = make_float2(0.f, 0.f);

    // Passes may run in any order (their contributions are summed).  The rows of one pass are N2*S*8 bytes apart
    // in memory, which maps them to a fraction of the L2 channels; workgroups that share an XCD (every 8th
    // workgroup id) therefore start at different passes so that together they use all channels.
    const int r_rot = (int)(blockIdx.x >> 3);
    const RowPieces<C> pieces(L.scr, tid);
    // (real rows with more than 32 modes are loaded by the lanes that transform them: kernel alone, through the patch and so, 128 x 128, 1024
    // images 25.8 and 23.7 us, 64 x 256, 256 images 9.4 and 8.7 us, larger fields equal)
    constexpr bool PIECES = FNO && KH <= 2;
    using VT = std::conditional_t<PIECES, tfno_vf4, std::conditional_t<FNO, float, c64>>;
    constexpr int NV = PIECES ? 4 : 16;
    auto load_rows = [&](VT *v, int sweep) __attribute__((always_inline)) {
        const int r = (sweep / SWEEPS + r_rot) & (S - 1), s = (sweep % SWEEPS) * RPS + g;
        if (row_on) {
            if constexpr (PIECES) {
                // (s: the wave's first row here)
                const XT *src = img + (long long)(r + S * (s - (tid & 63) / LPR + pieces.row)) * N2 + pieces.col;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    v[j] = __builtin_nontemporal_load(reinterpret_cast<const tfno_vf4 *>(src + j * pieces.ROWS * S * N2));
            } else if constexpr (FNO) {
                const XT *src = img + (long long)(r + S * s) * N2 + p;
#pragma unroll
                for (int j = 0; j < 16; ++j) v[j] = LPR >= 16 ? __builtin_nontemporal_load(src + LPR * j) : src[LPR * j];
            } else {
                const XT *src = img + (long long)(r + S * s) * N2 + p;
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    // (quarter-line pieces per row and instruction, LPR = 4, measured 13 % faster through the cache)
                    // (non-temporal where measured to help: 256-point rows, 312 -> 267 us on the 256 x 256 layer)
                    if constexpr (LPR >= 8) v[j] = load_nt(src + LPR * j);
                    else v[j] = src[LPR * j];
                }
            }
        }
    };
    // Row transforms of the sweep held in v.  The first butterfly level consumes v, so the loads of the next
    // sweep are issued right after it and stay in flight while the rest of this sweep is computed.
    auto row_stage = [&](VT *v, int sweep, auto refill, int next_sweep) __attribute__((always_inline)) {
        constexpr bool REFILL = decltype(refill)::value;    // false only for the last sweep of the image
        if (!row_on) return;
        const int s = (sweep % SWEEPS) * RPS + g;
        c64 *tile = L.tile + ((sweep / SWEEPS) % NBUF) * (RP * TS);
        c64 z[C::COLS];
        if constexpr (FNO) {
            float vs[8], vd[8];
            if constexpr (PIECES) {
                const float *flat = reinterpret_cast<const float *>(L.scr + (tid >> 6) * C::WREG) + (tid & 63) / LPR * C::FP;
                float u[16];
                wave_sync();                                // the previous sweep's patch reads are done
#pragma unroll
                for (int j = 0; j < 4; ++j) *pieces.at(j) = v[j];
                wave_sync();
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (REFILL) load_rows(v, next_sweep);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < 16; ++j) u[j] = flat[p + LPR * j];
                real_first_level16(u, vs, vd);
            } else {
                real_first_level16(v, vs, vd);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (REFILL) load_rows(v, next_sweep);
                __builtin_amdgcn_sched_barrier(0);
            }
            real_dft16(vs, vd, z);
        } else {
            c64 ea[8], eb[8], za[8], zo[8];
            dif_first_level<16, -1>(v, ea, eb);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (REFILL) load_rows(v, next_sweep);
            __builtin_amdgcn_sched_barrier(0);
            RegFFT<8, -1, 1>::run(ea, za);
            RegFFT<8, -1, 1>::run(eb, zo);
#pragma unroll
            for (int k = 0; k < 8; ++k) { z[2 * k] = za[k]; z[2 * k + 1] = zo[k]; }
        }
        // the twiddles are read eight at a time before their first use: left alone, the compiler reads, waits and
        // multiplies one at a time (15 exposed LDS round trips per sweep); all 15 at once do not fit the registers
        wave_sync();                                        // the previous sweep's patch reads are done
#pragma unroll
        for (int half = 0; half < (FNO ? 1 : 2); ++half) {
            c64 tw[8];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (half + j != 0) tw[j] = L.tw[(8 * half + j) * LPR + p];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int kl = 8 * half + j;
                const c64 zt = kl == 0 ? z[0] : cmul(z[kl], tw[j]);
                scr[kl * LPR + (p ^ (kl % LPR))] = zt;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (FNO) {                                // column 8: the value is real
            const c64 w = L.tw[8 * LPR + p];
            scr[8 * LPR + (p ^ (8 % LPR))] = make_float2(z[8].x * w.x, z[8].x * w.y);
        }
        wave_sync();
        if constexpr (FNO) {
            c64 *row = tile + s * TS;
            c64 c8[LPR];                                    // column 8, read beside the others by all lanes though one transforms it
            if constexpr (LPR < 16) {
#pragma unroll
                for (int pp = 0; pp < LPR; ++pp) c8[pp] = scr[8 * LPR + pp];
            }
            static_for<0, (LPR < 16 ? 8 / LPR : 1)>([&](auto ic) __attribute__((always_inline)) {
                const int kl = p + LPR * decltype(ic)::value;   // kl % LPR == p
                if (LPR < 16 || kl < 9) {
                    c64 xo[2 * KH];                         // bins kl + 16 kh, kh = -KH..KH-1
                    dft_prune_out_sym<LPR, KH, -1>([&](auto ppc) __attribute__((always_inline)) {
                        constexpr int pp = decltype(ppc)::value;
                        return scr[kl * LPR + (pp ^ p)];
                    }, xo);
#pragma unroll
                    for (int kh = 0; kh < KH; ++kh) row[kl + 16 * kh] = xo[kh];
                    if (kl != 0 && kl != 8) {               // (columns 0 and 8 mirror themselves)
#pragma unroll
                        for (int kh = 1; kh <= KH; ++kh) row[16 * kh - kl] = make_float2(xo[2 * KH - kh].x, -xo[2 * KH - kh].y);
                    }
                }
            });
            if constexpr (LPR < 16) {
                if (p == 0) {                               // column 8
                    c64 xo[KH];
                    dft_prune_out<LPR, KH, -1>([&](auto ppc) __attribute__((always_inline)) {
                        constexpr int pp = decltype(ppc)::value;
                        return c8[pp];
                    }, xo);
#pragma unroll
                    for (int kh = 0; kh < KH; ++kh) row[8 + 16 * kh] = xo[kh];
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < CPL; ++i) {
                const int kl = p + LPR * i;                     // kl % LPR == p
                c64 xo[KH];
                dft_prune_out<LPR, KH, -1>([&](auto ppc) __attribute__((always_inline)) {
                    constexpr int pp = decltype(ppc)::value;
                    return scr[kl * LPR + (pp ^ p)];
                }, xo);
#pragma unroll
                for (int kh = 0; kh < KH; ++kh) tile[s * TS + kl + 16 * kh] = xo[kh];
            }
        }
    };
    // RP-point transform of the tile columns of pass `i` (rows r + S s), accumulated with the pass twiddle
    auto col_stage = [&](int pass) __attribute__((always_inline)) {
        if (!col_on) return;
        const int r = (pass + r_rot) & (S - 1);
        const c64 *tile = L.tile + (pass % NBUF) * (RP * TS);
        c64 u[RPL], G[OUTS];
#pragma unroll
        for (int j = 0; j < RPL; ++j) u[j] = tile[(q4 + 4 * j) * TS + k2];
        if constexpr (C::H == 2) {
            c64 e[OUTS];
            if (hs == 0) {
#pragma unroll
                for (int j = 0; j < OUTS; ++j) e[j] = cadd(u[j], u[j + OUTS]);
            } else {
                static_for<0, OUTS>([&](auto jc) __attribute__((always_inline)) {
                    constexpr int j = decltype(jc)::value;
                    e[j] = mul_tw<RPL, -1, j>(csub(u[j], u[j + OUTS]));
                });
            }
            RegFFT<OUTS, -1, 1>::run(e, G);
        } else {
            RegFFT<RPL, -1, 1>::run(u, G);
        }
#pragma unroll
        for (int i = 0; i < OUTS; ++i) {
            const int ka = slot_ka(i);
            c64 t = C::H == 1 && i == 0 ? G[0] : cmul(G[i], L.twn[(q4 * ka) * (N1 / RP)]);
            t = quad_dft4_fwd(t, q4);                       // F_r[ka + RPL kb]
#pragma unroll
            for (int m = 0; m < MREP; ++m) {
                // frequency of accumulator slot (ka, m); FNO: position jres + RP m of the block, frequency - h1
                const int k1 = FNO ? (ka + RPL * kb + h1) % RP + RP * m - h1 : ka + RPL * kb + RP * m;
                acc[m * OUTS + i] = cmac(acc[m * OUTS + i], t, L.twn[(r * k1) & (N1 - 1)]);
            }
        }
    };

    if constexpr (FNO) {
        static_assert(SWEEPS == 1 && S % 2 == 0, "a pair of passes at a time");
        // Two passes of loads are in flight (64-point rows: the whole image), from before the tables are set up
        VT va[NV], vb[NV];
        load_rows(va, 0);
        load_rows(vb, 1);
        __builtin_amdgcn_sched_barrier(0);
        lds_tables<C, N1, N2>(L, tid);
        __syncthreads();
        auto pass = [&](VT *v, int i, auto refill) __attribute__((always_inline)) {
            row_stage(v, i, refill, i + 2);
            __syncthreads();
            col_stage(i);
        };
        for (int i = 0; i < S - 2; i += 2) {
            pass(va, i, std::true_type{});
            if constexpr (NBUF == 1) __syncthreads();       // with two tile buffers the next pass writes the other one
            pass(vb, i + 1, std::true_type{});
            if constexpr (NBUF == 1) __syncthreads();
        }
        pass(va, S - 2, std::false_type{});
        if constexpr (NBUF == 1) __syncthreads();
        pass(vb, S - 1, std::false_type{});
    } else {
        VT v[NV];
        load_rows(v, 0);
        lds_tables<C, N1, N2>(L, tid);
        __syncthreads();                                    // twiddle tables are ready
        // the last pass is peeled off so that every other sweep refills v unconditionally
        for (int i = 0; i < S - 1; ++i) {
#pragma unroll
            for (int w = 0; w < SWEEPS; ++w) row_stage(v, i * SWEEPS + w, std::true_type{}, i * SWEEPS + w + 1);
            __syncthreads();
            col_stage(i);
            if constexpr (NBUF == 1) __syncthreads();       // with two tile buffers the next pass writes the other one
        }
#pragma unroll
        for (int w = 0; w < SWEEPS; ++w) {
            if (w + 1 < SWEEPS) row_stage(v, (S - 1) * SWEEPS + w, std::true_type{}, (S - 1) * SWEEPS + w + 1);
            else row_stage(v, (S - 1) * SWEEPS + w, std::false_type{}, 0);
        }
        __syncthreads();
        col_stage(S - 1);
    }

    if (col_on) {
        const long long b = image / C_in;
        const SpecImage spec(b, (int)(image % C_in), C_in, Mp);
#pragma unroll
        for (int m = 0; m < MREP; ++m)
#pragma unroll
            for (int i = 0; i < OUTS; ++i) {
                const int ka = slot_ka(i);
                // position in the block of retained first-axis modes (FNO: frequency k1 - h1)
                const int k1 = FNO ? (ka + RPL * kb + h1) % RP + RP * m : ka + RPL * kb + RP * m;
                c64 val = acc[m * OUTS + i];
                if constexpr (FNO) {
                    if (k2 == 0) val = make_float2(0.5f * val.x, 0.5f * val.y);
                }
                // (truncation finer than the kernel's: only the K1_keep x K2_keep block exists in the spectrum)
                if (k1 < K1_keep && k2 < K2_keep) Xh[spec.at(__mul24(k1, K2_keep) + k2)] = val;
            }
    }
}

// ------------------------------------------------------------------------------------------------ inverse
template <int N1, int N2, int K1, int K2, bool FNO = false>
__global__ void __launch_bounds__((Cfg2d<N1, N2, K1, K2, false, FNO, true>::NT), (Cfg2d<N1, N2, K1, K2, false, FNO, true>::WG_PER_CU))
k_inv2d(const c64 *__restrict__ Yh, c64 *__restrict__ y, int C_out, int K1_keep, int K2_keep, int Mp, int h1)
{
    using C = Cfg2d<N1, N2, K1, K2, false, FNO, true>;
    constexpr int LPR = C::LPR, RPS = C::RPS, S = C::S, SWEEPS = C::SWEEPS, KH = C::KH, CPL = C::CPL;
    constexpr int GS = C::GS, TS = C::TS, MREP = C::MREP, RP = C::RP, RPL = C::RPL, NBUF = C::NBUF;
    __shared__ __align__(16) unsigned char raw[C::LDS_BYTES];
    const int tid = threadIdx.x;
    const Lds2d L = lds_setup<C>(raw);

    using XT = std::conditional_t<FNO, float, c64>;
    const unsigned image = blockIdx.x;
    XT *__restrict__ img = reinterpret_cast<XT *>(y) + (long long)image * N1 * N2;
    const bool row_on = tid < C::ACTIVE;
    const int g = tid / LPR, p = tid % LPR;
    c64 *scr = L.scr + g * GS;
    const int k2 = tid >> 2, q4 = tid & 3, kb = ((q4 & 1) << 1) | (q4 >> 1);
    const bool col_on = k2 < K2;

    // the retained spectrum of this image, K1*K2/256 (or fewer) bins per thread, for all passes
    c64 Y[C::NACC];
    {
        const long long b = image / C_out;
        const SpecImage spec(b, (int)(image % C_out), C_out, Mp);
#pragma unroll
        for (int m = 0; m < MREP; ++m)
#pragma unroll
            for (int ka = 0; ka < RPL; ++ka) {
                const int k1 = FNO ? (ka + RPL * kb + h1) % RP + RP * m : ka + RPL * kb + RP * m;   // position in the block
                const bool ok = k2 < K2_keep && k1 < K1_keep;
                c64 v = Yh[spec.at(ok ? __mul24(k1, K2_keep) + k2 : 0)];
                Y[m * RPL + ka] = ok ? v : make_float2(0.f, 0.f);
            }
    }

    const int r_rot = (int)(blockIdx.x >> 3);               // pass order rotated as in the forward kernel
    // twiddled RP-point inverse column transform of pass `i` (rows r + S s) into the tile
    auto col_stage = [&](int i) __attribute__((always_inline)) {
        if (!col_on) return;
        const int r = (i + r_rot) & (S - 1);
        c64 *tile = L.tile + (i % NBUF) * (RP * TS);
        auto pass_twiddle = [&](int ka, int m) __attribute__((always_inline)) {
            const int k1 = FNO ? (ka + RPL * kb + h1) % RP + RP * m - h1 : ka + RPL * kb + RP * m;     // frequency
            return L.twn[(r * k1) & (N1 - 1)];
        };
        // Real fields: all read before their first use.  The kernel's LDS holds four workgroups per CU there, so the compiler saves
        // registers and reads, waits and multiplies one at a time (256 x 256, 64 x 64 modes, 256 images: 30.4 and 26.8 us).
        c64 G[RPL], f[RPL], w1[FNO ? C::NACC : 1];
        if constexpr (FNO) {
#pragma unroll
            for (int ka = 0; ka < RPL; ++ka)
#pragma unroll
                for (int m = 0; m < MREP; ++m) w1[m * RPL + ka] = pass_twiddle(ka, m);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int ka = 0; ka < RPL; ++ka) {
            c64 t = make_float2(0.f, 0.f);
#pragma unroll
            for (int m = 0; m < MREP; ++m) {
                const c64 w = FNO ? w1[FNO ? m * RPL + ka : 0] : pass_twiddle(ka, m);
                t = cmac(t, Y[m * RPL + ka], make_float2(w.x, -w.y));
            }
            t = quad_dft4_inv(t, q4);
            if (ka != 0) {
                const c64 w = L.twn[(q4 * ka) * (N1 / RP)];
                t = cmul(t, make_float2(w.x, -w.y));
            }
            G[ka] = t;
        }
        RegFFT<RPL, +1, 1>::run(G, f);
#pragma unroll
        for (int j = 0; j < RPL; ++j) tile[(q4 + 4 * j) * TS + k2] = f[j];
    };
    // zero-padded inverse row transforms of sweep `sweep`, results left in out[]
    auto row_stage = [&](XT *out, int sweep) __attribute__((always_inline)) {
        if (!row_on) return;
        const int s = (sweep % SWEEPS) * RPS + g;
        const c64 *tile = L.tile + ((sweep / SWEEPS) % NBUF) * (RP * TS);
        wave_sync();                                        // the previous sweep's patch reads are done
        if constexpr (FNO) {
            const c64 *row = tile + s * TS;
            static_for<0, (LPR < 16 ? 8 / LPR : 1)>([&](auto ic) __attribute__((always_inline)) {
                const int kl = p + LPR * decltype(ic)::value;   // kl % LPR == p
                if (LPR < 16 || kl < 9) {
                    c64 yin[2 * KH];                        // bins kl + 16 kh, kh = -KH..KH-1 (columns 0 and 8: from 0 on)
                    const bool mirrored = kl != 0 && kl != 8;
#pragma unroll
                    for (int kh = 0; kh < KH; ++kh) yin[kh] = row[kl + 16 * kh];
#pragma unroll
                    for (int kh = 1; kh <= KH; ++kh) {
                        const c64 t = row[mirrored ? 16 * kh - kl : 0];
                        yin[2 * KH - kh] = mirrored ? make_float2(t.x, -t.y) : make_float2(0.f, 0.f);
                    }
                    dft_prune_in_sym<LPR, KH, +1>(yin, [&](auto ppc, c64 val) __attribute__((always_inline)) {
                        constexpr int pp = decltype(ppc)::value;
                        scr[kl * LPR + (pp ^ p)] = val;
                    });
                }
            });
            if constexpr (LPR < 16) {
                if (p == 0) {                               // column 8
                    c64 yin[KH];
#pragma unroll
                    for (int kh = 0; kh < KH; ++kh) yin[kh] = row[8 + 16 * kh];
                    dft_prune_in<LPR, KH, +1>(yin, [&](auto ppc, c64 val) __attribute__((always_inline)) {
                        constexpr int pp = decltype(ppc)::value;
                        scr[8 * LPR + pp] = val;
                    });
                }
            }
            wave_sync();
            c64 h[8];
#pragma unroll
            for (int kl = 1; kl < 8; ++kl) {
                const c64 w = L.tw[kl * LPR + p];
                h[kl] = cmul(scr[kl * LPR + (p ^ (kl % LPR))], make_float2(w.x, -w.y));
            }
            const c64 t8 = scr[8 * LPR + (p ^ (8 % LPR))], w8 = L.tw[8 * LPR + p];
            hermitian_dft16(scr[p].x, fmaf(t8.x, w8.x, t8.y * w8.y), h, out);
        } else {
#pragma unroll
            for (int i = 0; i < CPL; ++i) {
                const int kl = p + LPR * i;
                c64 yin[KH];
#pragma unroll
                for (int kh = 0; kh < KH; ++kh) yin[kh] = tile[s * TS + kl + 16 * kh];
                dft_prune_in<LPR, KH, +1>(yin, [&](auto ppc, c64 val) __attribute__((always_inline)) {
                    constexpr int pp = decltype(ppc)::value;
                    scr[kl * LPR + (pp ^ p)] = val;
                });
            }
            wave_sync();
            c64 z[16];
#pragma unroll
            for (int kl = 0; kl < 16; ++kl) {
                c64 t = scr[kl * LPR + (p ^ (kl % LPR))];
                if (kl != 0) {
                    const c64 w = L.tw[kl * LPR + p];
                    t = cmul(t, make_float2(w.x, -w.y));
                }
                z[kl] = t;
            }
            RegFFT<16, +1, 1>::run(z, out);
        }
    };
    auto store_rows = [&](const XT *out, int sweep) __attribute__((always_inline)) {
        if (!row_on) return;
        const int r = (sweep / SWEEPS + r_rot) & (S - 1), s = (sweep % SWEEPS) * RPS + g;
        if constexpr (FNO) {
            float *flat = reinterpret_cast<float *>(L.scr + (tid >> 6) * C::WREG) + (tid & 63) / LPR * C::FP;
            wave_sync();                                    // the patch reads are done
#pragma unroll
            for (int j = 0; j < 16; ++j) flat[p + LPR * j] = out[j];
            wave_sync();
            const RowPieces<C> pieces(L.scr, tid);
            XT *dst = img + (long long)(r + S * (s - (tid & 63) / LPR + pieces.row)) * N2 + pieces.col;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const tfno_vf4 q = *pieces.at(j);
                __builtin_nontemporal_store(q, reinterpret_cast<tfno_vf4 *>(dst + j * pieces.ROWS * S * N2));
            }
        } else {
            XT *dst = img + (long long)(r + S * s) * N2 + p;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                // non-temporal only where the LPR lanes of a row write whole 128-byte lines: with narrower rows every
                // store instruction leaves half or quarter lines, which cost up to 40 % of the kernel time when they
                // bypass the cache that would have merged them.  (Lanes that swap halves with their neighbour and
                // write two complex elements each measured no faster for 64- and 128-point rows.)
                if constexpr (LPR >= 16) store_nt(dst + LPR * j, out[j]);
                else dst[LPR * j] = out[j];
            }
        }
    };

    lds_tables<C, N1, N2>(L, tid);
    __syncthreads();                                        // twiddle tables are ready
    for (int i = 0; i < S; ++i) {
        col_stage(i);
        __syncthreads();
#pragma unroll
        for (int w = 0; w < SWEEPS; ++w) {
            XT out[16];
            row_stage(out, i * SWEEPS + w);
            store_rows(out, i * SWEEPS + w);
        }
        if constexpr (NBUF == 1) __syncthreads();           // with two tile buffers the next pass writes the other one
    }
}

}  // namespace tfno
