// Both axes of a field whose sides are no powers of two, in one kernel each way.
//
// The transforms of matdft_kernel.h (contractions with the roots of unity on the matrix pipe, elements n and N - n folded,
// operands split exactly into three BF16 terms), with a workgroup per field and the field transformed along its first axis
// kept in LDS.  As one kernel per axis, the last axis came first: a lane read (or wrote) a contiguous pencil of its own, so that
// every load of a wave touched 64 lines, and the half-transformed fields went through memory.  Here the columns of the field are
// the pencils of the first axis: 16 neighbouring lanes read 256 contiguous bytes of a row, two columns each.
//
//   forward  wave = 32 columns (and a share of the rows): T[k1][n2] = sum_{n1} x[n1][n2] w1^(-n1 k1), n1 folded, into LDS;
//            then the kept rows k1 are 32 pencils of the last axis, whose sum is dealt out to the waves; partial sums meet in LDS
//   inverse  U[k1][n2] = sum_{k2} Y[k1][k2] w2^(k2 n2) by tiles of 32 output pairs, into LDS; then wave = 32 columns,
//            y[n1][n2] = sum_{k1} U[k1][n2] w1^(n1 k1), rows n1 and N1 - n1 together, put together in LDS sixteen or 32 rows at a time
//            and stored as whole lines past the caches (pieces of lines stay dirty in the last-level cache, and the
//            next kernel's reads wait for their write-back)
//
// 85 x 85, K 12 x 12, 1024 fields each way: forward 17.6 + 7.6 -> 14.5 us, inverse 8.3 + 21.6 -> 18.7 us (59 MB each: 4.1 and 3.2 TB/s).  What
// bounds them: vector issue (folds, exact splits, addresses), with the matrix pipe at a
// quarter and memory at two thirds; all fields are resident at once and go through their phases together, so that the phases add up.
// The forward kernel takes tiles of 16 pencils x 16 modes (v_mfma_f32_16x16x32_bf16), half the products of 32 x 32 where 12 modes
// are kept; the inverse has only K1 terms to a sum and 32 x 32 x 16 fits them.
#pragma once
#include "matdft_kernel.h"
#include "matgrid.h"

namespace tfno {

constexpr int MG_ROWS = 512, MG_COLUMNS = 256, MG_MODES = 32, MG_WAVES = 8;
typedef float md_floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned md_u3 __attribute__((ext_vector_type(3)));

// Root table of a side: the three terms (cos | sin << 16) of a root side by side, so that a lane fetches it in one access; exponents are
// kept as byte offsets.
constexpr unsigned MG_ROOT = 16;
// (both sides' tables in one pass over the threads; sides of equal length share one)
__device__ __forceinline__ void mg_tables(unsigned char *tab, int N1, int N2, int tid, int threads)
{
    const int entries = N1 == N2 ? N1 : N1 + N2;
    for (int i = tid; i < entries; i += threads) {
        const int N = i < N1 ? N1 : N2, e = i < N1 ? i : i - N1;
        const c64 w = root_of_unity(e, N, 1.0f / (float)N);
        const Split3 re = split3(w.x), im = split3(w.y);
        *reinterpret_cast<uintx4 *>(tab + MG_ROOT * i) = uintx4{pack_bf16(re.t0, im.t0), pack_bf16(re.t1, im.t1), pack_bf16(re.t2, im.t2), 0u};
    }
}
__device__ __forceinline__ unsigned mg_second(int N1, int N2) { return N1 == N2 ? 0u : MG_ROOT * (unsigned)N1; }
__device__ __forceinline__ md_u3 mg_root(const unsigned char *tab, unsigned off) { return *reinterpret_cast<const md_u3 *>(tab + off); }

// Four pairs of a pencil in the operand form of matdft_kernel.h: (s.re, d.im) and (s.im, -d.re) of u[e] and v[3 - e], negated
// for NEG.
template <bool NEG>
__device__ __forceinline__ void mg_fold(uintx4 (&re)[3], uintx4 (&im)[3], const c64 *u, const c64 *v)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const c64 x = NEG ? make_float2(-u[e].x, -u[e].y) : u[e], y = NEG ? make_float2(-v[3 - e].x, -v[3 - e].y) : v[3 - e];
        const Split3 sr = split3(x.x + y.x), di = split3(x.y - y.y), si = split3(x.y + y.y), dr = split3(y.x - x.x);
        re[0][e] = pack_bf16(sr.t0, di.t0);
        re[1][e] = pack_bf16(sr.t1, di.t1);
        re[2][e] = pack_bf16(sr.t2, di.t2);
        im[0][e] = pack_bf16(si.t0, dr.t0);
        im[1][e] = pack_bf16(si.t1, dr.t1);
        im[2][e] = pack_bf16(si.t2, dr.t2);
    }
}

// What a block holds that does not belong to a pair: slot 0 has no partner, the middle of an even length is its own, slots past H.
__device__ __forceinline__ void mg_mend(c64 *u, c64 *v, int n, int H, int N)
{
    const c64 zero = make_float2(0.f, 0.f);
    if (n == 0) v[3] = zero;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (n + e > H) u[e] = zero;
        if (n + e > H || 2 * (n + e) == N) v[3 - e] = zero;
    }
}

// Sums over the slots of blocks part, part + parts, ... of CT tiles of 16 pencils: 16 KT modes.  A lane owns pencil lane % 16 of each
// tile and the slots 4 (lane / 16) .. + 3 of every 16.  COLQ: the pencils are the columns of the product, and those of odd tiles go
// through with their sign turned round (below).  fetch(u, v, n): raw elements of the slots n .. n + 3, every address valid; begin()
// runs once the first ones are on their way.  ROW: slot 0's partners come one element early.  Modes k0 .. k0 + 16 KT - 1.
template <int CT, int KT>
struct MgSums { md_floatx4 re[CT][KT], im[CT][KT]; };
// LONG: the matrix pipe cuts off what a sum cannot hold, always in one direction, so that the offset grows with the number of
// products added up; every other block the sums go into others by rounded additions (443 x 302 points: 3.7e-7 -> 2.4e-7 of the
// whole layer).
template <int CT, int KT, bool COLQ, bool LONG, bool ROW = false, class Fetch, class Begin>
__device__ __forceinline__ void mg_sum(MgSums<CT, KT> &acc, const unsigned char *tab, int N, int K, int part, int parts, Fetch fetch, Begin begin, int k0 = 0)
{
    const int lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4, H = N / 2, nblk = H / 16 + 1;
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) { acc.re[c][t][r] = 0.f; acc.im[c][t][r] = 0.f; }
    const int last = part + (nblk - 1 - part) / parts * parts;              // (part < nblk)
    MgSums<CT, KT> total = acc;
    int count = 0;
    c64 u[CT][4], v[CT][4];
    fetch(u, v, 16 * part + 4 * g);
    begin();
    const unsigned NB = MG_ROOT * (unsigned)N;
    unsigned idx[KT], step[KT], skip[KT];
#pragma unroll
    for (int t = 0; t < KT; ++t) {
        const unsigned k = k0 + 16 * t + col < K ? (unsigned)(k0 + 16 * t + col) : 0u;     // (past K: not stored)
        idx[t] = MG_ROOT * (k * (unsigned)(16 * part + 4 * g) % (unsigned)N);
        skip[t] = MG_ROOT * (k * (unsigned)(16 * parts - 4) % (unsigned)N);
        step[t] = MG_ROOT * k;
    }
    auto wrap = [&](unsigned e) __attribute__((always_inline)) { return min(e, e - NB); };
    auto roots = [&](uintx4 (*w)[3]) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < KT; ++t) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const md_u3 root = mg_root(tab, idx[t]);
#pragma unroll
                for (int k = 0; k < 3; ++k) w[t][k][e] = root[k];
                idx[t] = wrap(idx[t] + step[t]);
            }
            idx[t] = wrap(idx[t] + skip[t]);
        }
    };
#pragma unroll 1
    for (int blk = part; blk <= last; blk += parts) {
        uintx4 w[KT][3];
        roots(w);
        if (blk == 0 || blk == nblk - 1) {
            if constexpr (ROW) {
                if (blk == 0 && g == 0) v[0][2] = v[0][3];
            }
#pragma unroll
            for (int c = 0; c < CT; ++c) mg_mend(u[c], v[c], 16 * blk + 4 * g, H, N);
        }
        auto products = [&](const uintx4 (&re)[3], const uintx4 (&im)[3], int c) __attribute__((always_inline)) {
#pragma unroll
            for (int p = 0; p < 6; ++p)
#pragma unroll
                for (int t = 0; t < KT; ++t) {
                    const bf16x8 r16 = __builtin_bit_cast(bf16x8, w[t][MD_SB[p]]);
                    const bf16x8 re16 = __builtin_bit_cast(bf16x8, re[MD_SA[p]]), im16 = __builtin_bit_cast(bf16x8, im[MD_SA[p]]);
                    if constexpr (COLQ) {
                        acc.re[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(r16, re16, acc.re[c][t], 0, 0, 0);
                        acc.im[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(r16, im16, acc.im[c][t], 0, 0, 0);
                    } else {
                        acc.re[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(re16, r16, acc.re[c][t], 0, 0, 0);
                        acc.im[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(im16, r16, acc.im[c][t], 0, 0, 0);
                    }
                }
        };
        uintx4 re0[3], im0[3], re1[3], im1[3];
        mg_fold<false>(re0, im0, u[0], v[0]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (CT == 2) {                            // (the products of one tile under the folds of the other)
            products(re0, im0, 0);
            mg_fold<COLQ>(re1, im1, u[1], v[1]);
            __builtin_amdgcn_sched_barrier(0);
        }
        fetch(u, v, 16 * min(blk + parts, last) + 4 * g);   // (the last one is fetched again and dropped)
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (CT == 2) products(re1, im1, 1);
        else products(re0, im0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (LONG && ((++count & 1) == 0 || blk == last)) {
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int t = 0; t < KT; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        total.re[c][t][r] += acc.re[c][t][r];
                        total.im[c][t][r] += acc.im[c][t][r];
                        acc.re[c][t][r] = 0.f;
                        acc.im[c][t][r] = 0.f;
                    }
        }
    }
    if constexpr (LONG) acc = total;
}

// Row pitch of the inverse kernel's spectrum in LDS.
TFNO_HD int mg_modes_pitch(int K2) { return (K2 > 16 ? 32 : 16) + 1; }
// Row pitch in LDS: odd, so that lanes along a column hit different banks.
TFNO_HD int mg_pitch(int N2) { return (N2 + 1) | 1; }

// Place of joint mode m of channel c in the spectrum (matdft.h, MD_SPEC).
__device__ __forceinline__ long long mg_place(long long m, int c, int C) { return ((m >> 7) * C + c) * 128 + (m & 127); }

// LDS: two root tables, T [parts][K1][P], partial sums [parts2][K1][K2].
// A lane loads two neighbouring columns in one access; the even ones are one tile of pencils, the odd ones the other, and the odd
// ones go through with their sign turned round, as every other pencil of the first transform of a field in matdft_kernel.h: the
// matrix pipe rounds downwards, and the last axis would add the offsets of all columns up in its bin 0.
template <int KT1, int KT2, bool LONG>
__global__ void __launch_bounds__(64 * MG_WAVES, KT1 == 2 && LONG ? 2 : 3)
k_matgrid_fwd(MatgridArgs a)
{
    extern __shared__ __align__(16) unsigned char mg_lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, threads = blockDim.x;
    const int col = lane & 15, g = lane >> 4;
    const int N1 = a.N1, N2 = a.N2, K1 = a.K1, K2 = a.K2, P = mg_pitch(N2);
    unsigned char *tab1 = mg_lds, *tab2 = tab1 + mg_second(N1, N2);
    c64 *T = reinterpret_cast<c64 *>(tab2 + MG_ROOT * N2), *red = T + a.parts * K1 * P;

    const unsigned img = blockIdx.x;
    const char *__restrict__ field = reinterpret_cast<const char *>(a.in + (long long)img * N1 * N2);
    const int groups = (threads >> 6) / a.parts, part = wave / groups;     // (a wave of every part for each 32 columns)
    const unsigned pitch = 8u * (unsigned)N2;
    {
        const int n2 = 32 * (wave % groups) + 2 * col, first = min(n2, N2 - 2);          // (an odd last column is the second of its pair)
        const unsigned place = 8u * (unsigned)first;
        MgSums<2, KT1> acc;
        mg_sum<2, KT1, true, LONG>(acc, tab1, N1, K1, part, a.parts, [&](c64 (*u)[4], c64 (*v)[4], int n) __attribute__((always_inline)) {
            // (a field has at most 1 MB: 32-bit offsets from a uniform address.  Slots go up to N1 / 2 + 15, rows of the field from 30
            // points on; only slot 0 has no partner)
            const unsigned lo = __umul24((unsigned)n, pitch) + place, hi = __umul24((unsigned)(N1 - n), pitch) + place;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const md_u4a8 x = *reinterpret_cast<const md_u4a8 *>(field + (lo + e * pitch));
                const md_u4a8 y = *reinterpret_cast<const md_u4a8 *>(field + (e ? hi - e * pitch : n ? hi : hi - pitch));
                u[0][e] = make_float2(__uint_as_float(x[0]), __uint_as_float(x[1]));
                u[1][e] = make_float2(__uint_as_float(x[2]), __uint_as_float(x[3]));
                v[0][3 - e] = make_float2(__uint_as_float(y[0]), __uint_as_float(y[1]));
                v[1][3 - e] = make_float2(__uint_as_float(y[2]), __uint_as_float(y[3]));
            }
        }, [&]() __attribute__((always_inline)) {
            mg_tables(tab1, N1, N2, tid, threads);
            __syncthreads();
        });
#pragma unroll
        for (int t = 0; t < KT1; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int k1 = 16 * t + 4 * g + r;
                c64 *row = T + (part * K1 + k1) * P + first;
                if (k1 < K1 && n2 < N2 - 1) row[0] = make_float2(acc.re[0][t][r], acc.im[0][t][r]);
                if (k1 < K1 && n2 < N2) row[1] = make_float2(-acc.re[1][t][r], -acc.im[1][t][r]);
            }
    }
    __syncthreads();
    if (a.parts > 1) {
        for (int i = tid; i < K1 * P; i += threads) {
            c64 sum = T[i];
            for (int p = 1; p < a.parts; ++p) sum = cadd(sum, T[p * K1 * P + i]);
            T[i] = sum;
        }
        __syncthreads();
    }

    // last axis: KT1 tiles of 16 rows, each sum dealt out to parts2 waves
    const int parts2 = a.parts2;
    for (int item = wave; item < KT1 * parts2; item += threads >> 6) {
        const int t1 = item / parts2, p2 = item - t1 * parts2, k = 16 * t1 + col;
        const c64 *row = T + (k < K1 ? k : 0) * P;
        MgSums<1, KT2> acc;
        mg_sum<1, KT2, false, LONG>(acc, tab2, N2, K2, p2, parts2, [&](c64 (*u)[4], c64 (*v)[4], int n) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                u[0][e] = row[n + e];
                v[0][3 - e] = row[N2 - n - e];              // (slot 0: the pad after the row, or the next one)
            }
        }, [] {});
#pragma unroll
        for (int t = 0; t < KT2; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int k1 = 16 * t1 + 4 * g + r, k2 = 16 * t + col;
                if (k1 < K1 && k2 < K2) red[(p2 * K1 + k1) * K2 + k2] = make_float2(acc.re[0][t][r], acc.im[0][t][r]);
            }
    }
    __syncthreads();
    const int M = K1 * K2, c = (int)(img % (unsigned)a.C);
    const long long m0 = (long long)(img / (unsigned)a.C) * M;
    for (int i = tid; i < M; i += threads) {
        c64 sum = red[i];
        for (int p = 1; p < parts2; ++p) sum = cadd(sum, red[p * M + i]);
        a.out[mg_place(m0 + i, c, a.C)] = sum;
    }
}

// 16 modes of a tile of 32 pencils x 32 output pairs, as in k_matdft_inv: the four real sums cr, ci, sr, si.  u: the modes i0 + 8 h + e
// (zeros past K); idx: exponent of this lane's pair, advanced.
struct MgPairs { md_floatx16 cr, ci, sr, si; };
template <bool COLQ>
__device__ __forceinline__ void mg_pairs(MgPairs &s, const uintx4 (&re)[3], const uintx4 (&im)[3], const uintx4 (&wc)[3], const uintx4 (&ws)[3])
{
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const bf16x8 c16 = __builtin_bit_cast(bf16x8, wc[MD_SB[k]]), s16 = __builtin_bit_cast(bf16x8, ws[MD_SB[k]]);
        const bf16x8 re16 = __builtin_bit_cast(bf16x8, re[MD_SA[k]]), im16 = __builtin_bit_cast(bf16x8, im[MD_SA[k]]);
        if constexpr (COLQ) {
            s.cr = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c16, re16, s.cr, 0, 0, 0);
            s.ci = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c16, im16, s.ci, 0, 0, 0);
            s.sr = __builtin_amdgcn_mfma_f32_32x32x16_bf16(s16, re16, s.sr, 0, 0, 0);
            s.si = __builtin_amdgcn_mfma_f32_32x32x16_bf16(s16, im16, s.si, 0, 0, 0);
        } else {
            s.cr = __builtin_amdgcn_mfma_f32_32x32x16_bf16(re16, c16, s.cr, 0, 0, 0);
            s.ci = __builtin_amdgcn_mfma_f32_32x32x16_bf16(im16, c16, s.ci, 0, 0, 0);
            s.sr = __builtin_amdgcn_mfma_f32_32x32x16_bf16(re16, s16, s.sr, 0, 0, 0);
            s.si = __builtin_amdgcn_mfma_f32_32x32x16_bf16(im16, s16, s.si, 0, 0, 0);
        }
    }
}
__device__ __forceinline__ void mg_clear(MgPairs &s)
{
#pragma unroll
    for (int r = 0; r < 16; ++r) { s.cr[r] = 0.f; s.ci[r] = 0.f; s.sr[r] = 0.f; s.si[r] = 0.f; }
}
// real and imaginary parts of 8 modes, two modes to a dword
__device__ __forceinline__ void mg_split(uintx4 (&re)[3], uintx4 (&im)[3], const c64 *u)
{
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const Split3 r0 = split3(u[2 * d].x), r1 = split3(u[2 * d + 1].x), m0 = split3(u[2 * d].y), m1 = split3(u[2 * d + 1].y);
        re[0][d] = pack_bf16(r0.t0, r1.t0);
        re[1][d] = pack_bf16(r0.t1, r1.t1);
        re[2][d] = pack_bf16(r0.t2, r1.t2);
        im[0][d] = pack_bf16(m0.t0, m1.t0);
        im[1][d] = pack_bf16(m0.t1, m1.t1);
        im[2][d] = pack_bf16(m0.t2, m1.t2);
    }
}
// (cos, cos) and (sin, sin) of the modes i0 + 8 h .. + 7 at output n
__device__ __forceinline__ void mg_roots(uintx4 (&wc)[3], uintx4 (&ws)[3], const unsigned char *tab, int N, int n, int mode)
{
    const unsigned NB = MG_ROOT * (unsigned)N, step = MG_ROOT * (unsigned)n;
    unsigned idx = MG_ROOT * ((unsigned)n * (unsigned)mode % (unsigned)N);
    auto wrap = [&](unsigned e) __attribute__((always_inline)) { return min(e, e - NB); };
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const md_u3 r0 = mg_root(tab, idx);
        idx = wrap(idx + step);
        const md_u3 r1 = mg_root(tab, idx);
        idx = wrap(idx + step);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            wc[k][d] = __builtin_amdgcn_perm(r1[k], r0[k], 0x05040100u);
            ws[k][d] = __builtin_amdgcn_perm(r1[k], r0[k], 0x07060302u);
        }
    }
}

// A run of elements from LDS to memory past the caches: 16 bytes per lane, from the line boundary before it on.
__device__ __forceinline__ void mg_flush(c64 *dst, const c64 *from, int count, int tid, int threads)
{
    typedef float vf4 __attribute__((ext_vector_type(4)));
    const int lead = (int)(((unsigned long long)dst >> 3) & 15);
    for (int i = 2 * tid - lead; i < count - 1; i += 2 * threads)
        if (i >= 0) {
            const c64 p = from[i], q = from[i + 1];
            __builtin_nontemporal_store(vf4{p.x, p.y, q.x, q.y}, reinterpret_cast<vf4 *>(dst + i));
        }
    if (tid == 0 && (lead & 1) && count > 0) store_nt(dst, from[0]);
    if (tid == 0 && ((lead + count) & 1) && count > 0) store_nt(dst + count - 1, from[count - 1]);
}

// KT: sixteens of K1.  The waves are `parts` sets, each of which covers all columns and takes every parts-th tile of 32 output pairs.
// RG: output pairs that a set puts together at a time, in eights.  WAVES: on a SIMD.  More than 128 columns are five waves and more to a
// workgroup, of which two fit a CU with the registers that the compiler would like (158 x 131 points, 342 fields: 27.4 us, with a fourth
// wave 19.5; 85 x 85, 1024 fields: 18.7 and 20.0).
// LDS: two root tables, the spectrum [32][K2P] (K2P: K2 in whole sixteens, one more for the banks; zeros past K1 and K2), U [16 KT][P],
// 16 RG rows of the field for every set.
template <int RG, int KT, int WAVES>
__global__ void __launch_bounds__(64 * MG_WAVES, WAVES)
k_matgrid_inv(MatgridArgs a)
{
    extern __shared__ __align__(16) unsigned char mg_lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, threads = blockDim.x, waves = threads >> 6;
    const int col = lane & 31, h = lane >> 5;
    const int N1 = a.N1, N2 = a.N2, K1 = a.K1, K2 = a.K2, P = mg_pitch(N2), H1 = N1 / 2, H2 = N2 / 2;
    unsigned char *tab1 = mg_lds, *tab2 = tab1 + mg_second(N1, N2);
    const int K2P = mg_modes_pitch(K2);
    c64 *Y = reinterpret_cast<c64 *>(tab2 + MG_ROOT * N2), *U = Y + 32 * K2P, *stages = U + 16 * KT * P;
    const unsigned img = blockIdx.x;
    {
        const int c = (int)(img % (unsigned)a.C);
        const long long m0 = (long long)(img / (unsigned)a.C) * (K1 * K2);
        for (int i = tid; i < 32 * (K2P - 1); i += threads) {
            const int k1 = K2 > 16 ? i >> 5 : i >> 4, k2 = i - k1 * (K2P - 1);
            Y[k1 * K2P + k2] = k1 < K1 && k2 < K2 ? a.in[mg_place(m0 + (k1 * K2 + k2), c, a.C)] : make_float2(0.f, 0.f);
        }
    }
    mg_tables(tab1, N1, N2, tid, threads);
    __syncthreads();

    // ---- last axis: rows k1 are the pencils, tiles of 32 output pairs
    for (int t = wave; 32 * t <= H2; t += waves) {
        const int n = 32 * t + col;
        const c64 *row = Y + col * K2P + 8 * h;
        MgPairs s;
        mg_clear(s);
        for (int i0 = 0; i0 < K2; i0 += 16) {
            c64 u[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) u[e] = row[i0 + e];
            uintx4 re[3], im[3], wc[3], ws[3];
            mg_split(re, im, u);
            mg_roots(wc, ws, tab2, N2, min(n, H2), i0 + 8 * h);
            mg_pairs<false>(s, re, im, wc, ws);
        }
        c64 *dst = U + 4 * h * P + n, *mirror = U + 4 * h * P + N2 - n;
        if (n <= H2) {
#pragma unroll
            for (int r = 0; r < 8 * KT; ++r) dst[(8 * (r / 4) + r % 4) * P] = make_float2(s.cr[r] - s.si[r], s.ci[r] + s.sr[r]);
        }
        if (n <= H2 && n && 2 * n != N2) {
#pragma unroll
            for (int r = 0; r < 8 * KT; ++r) mirror[(8 * (r / 4) + r % 4) * P] = make_float2(s.cr[r] + s.si[r], s.ci[r] - s.sr[r]);
        }
    }
    __syncthreads();

    // ---- first axis: columns are the pencils, rows n and N1 - n together
    c64 *__restrict__ field = a.out + (long long)img * N1 * N2;
    const int own = waves / a.parts, set = __builtin_amdgcn_readfirstlane(wave / own), n2 = 32 * (wave % own) + col;
    const c64 *src = U + 8 * h * P + min(n2, N2 - 1);
    for (int turn = 0; turn <= H1; turn += 32 * a.parts) {
        const int n0 = turn + 32 * set;
        MgPairs s;
        if (n0 <= H1) {
            mg_clear(s);
#pragma unroll 1
            for (int i0 = 0; i0 < 16 * KT; i0 += 16) {
                uintx4 wc[3], ws[3], re[3], im[3];
                mg_roots(wc, ws, tab1, N1, min(n0 + col, H1), i0 + 8 * h);
                c64 u[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) u[e] = src[(i0 + e) * P];
                mg_split(re, im, u);
                mg_pairs<true>(s, re, im, wc, ws);
            }
        }
#pragma unroll
        for (int rg = 0; rg < 4; rg += RG) {                // pairs n0 + 8 rg .. + 8 RG - 1
            if (turn + 8 * rg > H1) break;                  // (none left in any set)
            __syncthreads();                                // (the rows before have been read)
            if (n0 + 8 * rg <= H1 && n2 < N2) {
                c64 *stage = stages + set * (16 * RG * N2) + n2;
#pragma unroll
                for (int r = 4 * rg; r < 4 * rg + 4 * RG; ++r) {
                    const int i = 8 * (r / 4 - rg) + 4 * h + (r % 4);
                    stage[i * N2] = make_float2(s.cr[r] - s.si[r], s.ci[r] + s.sr[r]);
                    stage[(16 * RG - 1 - i) * N2] = make_float2(s.cr[r] + s.si[r], s.ci[r] - s.sr[r]);
                }
            }
            __syncthreads();
            if (n0 + 8 * rg <= H1) {
                // rows base .. of the first half, rows .. N1 - base of the second: row N1 - n lies at stage row 16 RG - 1 - (n - base)
                const int base = n0 + 8 * rg, t = tid - 64 * own * set;
                const c64 *stage = stages + set * (16 * RG * N2);
                const int first = max(N1 - base - 8 * RG + 1, H1 + 1);
                const int count0 = (min(base + 8 * RG - 1, H1) - base + 1) * N2, count1 = (min(N1 - base, N1 - 1) - first + 1) * N2;
                mg_flush(field + base * N2, stage, count0, t, 64 * own);
                mg_flush(field + first * N2, stage + (16 * RG - 1 - (N1 - first - base)) * N2, count1, t, 64 * own);
            }
        }
    }
}

}  // namespace tfno
