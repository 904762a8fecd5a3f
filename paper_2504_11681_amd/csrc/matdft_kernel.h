// Pruned DFTs of any length on the matrix pipe.
//
// A length without factors of two has no butterfly network to prune, but a transform that keeps K of N bins is a
// contraction of the pencils with an N x K matrix of roots of unity w = exp(2 pi i / N), and K is small.  The matrix is never
// stored: its entries are w^((n k) mod N), so a workgroup builds the N roots once in LDS, already split into three BF16 terms
// (bf16x3.h: the split is exact, six products, FP32 accumulation), and a lane fetches the root of its (n, k) from there, the
// exponent advanced by one addition and one wrap.  n and N - n have conjugate roots, which halves the products:
//
//   forward  the elements n and N - n of a pencil are folded first, s = x[n] + x[N-n], d = x[n] - x[N-n]:
//              X[k] = sum_{n <= N/2} (s.re cos + d.im sin) + i (s.im cos - d.re sin)
//            8 folded pairs per v_mfma_f32_32x32x16_bf16: an operand dword is (s.re, d.im) or (s.im, -d.re) against a root
//            (cos, sin)
//   inverse  the outputs n and N - n come from the same four real sums, Cr, Ci = sum_k Y[k] cos and Sr, Si = sum_k Y[k] sin:
//              y[n] = (Cr - Si) + i (Ci + Sr),   y[N-n] = (Cr + Si) + i (Ci - Sr)
//            16 modes per MFMA: an operand dword holds the real (or imaginary) parts of two modes, the roots of two modes
//            are regrouped into (cos, cos) and (sin, sin)
//
// Work split: a wave owns 32 pencils and 32 T outputs (or 32 T output pairs); a lane owns one pencil (lane % 32) and 8 of
// every 16 consecutive slots (lane / 32).  WI = 4, 8 (forward): the waves of a workgroup share a tile and deal the blocks
// of 16 slots out among them, partial sums meet in LDS -- for few pencils and long sums (truncating a batch of 2560 pencils
// fills 80 waves without it).  The pencils are the rows of the product where outputs of one pencil are contiguous in memory,
// and its columns where neighbouring pencils are (COLQ), so a half wave always stores 256 contiguous bytes.
// Root table: one plane of dwords (cos | sin << 16) per BF16 term, exponents kept as byte offsets.
#pragma once
#include "common.h"
#include "bf16x3.h"
#include "matdft.h"

namespace tfno {

typedef float md_floatx16 __attribute__((ext_vector_type(16)));
typedef unsigned md_u4a8 __attribute__((ext_vector_type(4), aligned(8)));

// exp(2 pi i m / N) for 0 <= m < N: the quotient 2 m / N is rounded, so its remainder is put back to first order (without
// it the angle of a length that is no power of two is off by up to 2e-7).
__device__ __forceinline__ c64 root_of_unity(int m, int N, float invN)
{
    if (2 * m > N) m -= N;                                  // -N/2 < m <= N/2: a smaller angle, a smaller rounding error
    const float num = (float)(2 * m);
    const float q = num * invN;
    const float d = 3.14159265358979f * (fmaf(-q, (float)N, num) * invN);
    float s, c;
    sincospif(q, &s, &c);
    return make_float2(fmaf(-s, d, c), fmaf(c, d, s));
}

// The root table: planes of NMAX dwords at a constant distance.
template <int NMAX>
struct MdRoots {
    static constexpr unsigned STEP = NMAX + 1;              // dwords between the planes
    static constexpr size_t BYTES = 4 * (size_t)(3 * STEP);
    static __device__ __forceinline__ void build(unsigned char *lds, int N, int tid, int threads)
    {
        unsigned *tab = reinterpret_cast<unsigned *>(lds);
        const float invN = 1.0f / (float)N;
        for (int e = tid; e < N; e += threads) {
            const c64 w = root_of_unity(e, N, invN);
            const Split3 re = split3(w.x), im = split3(w.y);
            tab[e] = pack_bf16(re.t0, im.t0);
            tab[STEP + e] = pack_bf16(re.t1, im.t1);
            tab[2 * STEP + e] = pack_bf16(re.t2, im.t2);
        }
        __syncthreads();
    }
    // term t of the root at byte offset `off` (4 times the exponent)
    static __device__ __forceinline__ unsigned get(const unsigned char *lds, unsigned off, int t)
    {
        return reinterpret_cast<const unsigned *>(lds + off)[t * STEP];
    }
};

// Orders this wave's LDS traffic (all lanes) without a workgroup barrier.
__device__ __forceinline__ void wave_sync_md()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Position of a pencil on the strided and spectrum sides.
struct MdPencil {
    long long strided;      // offset of element 0, strided side with `outer`
    long long m;            // spectrum side: joint mode of element 0 ...
    int c;                  // ... and channel
};
__device__ __forceinline__ MdPencil md_pencil(const MatdftArgs &a, unsigned q, long long outer)
{
    const unsigned img = a.inner == 1 ? q : q / a.inner, r = a.inner == 1 ? 0 : q - img * a.inner;
    const unsigned b = img / (unsigned)a.C;
    return MdPencil{img * outer + r, b * a.M + r, (int)(img - b * (unsigned)a.C)};
}

constexpr int MD_SA[6] = {2, 0, 1, 1, 0, 0}, MD_SB[6] = {0, 2, 1, 0, 1, 0};      // the six products, smallest first

// ------------------------------------------------------------------------------------------------ forward
template <int JT, int WI, int NMAX>
struct CfgMdF {
    static constexpr int NT = WI > 4 ? 64 * WI : 256;
    static constexpr size_t RED = WI > 1 ? sizeof(c64) * WI * 32 * 32 : 0;         // one 32 x 32 tile of every wave
    static constexpr size_t LDS = MdRoots<NMAX>::BYTES > RED ? MdRoots<NMAX>::BYTES : RED;
};

// VEC: contiguous pencils of at least 40 points, fetched 16 bytes at a time.
//
// ROWS -> ROWS (the first transform of a field): the matrix pipe rounds its sums downwards, not to nearest, so that all bins of
// all rows carry an offset of the same sign.  The other axis adds the rows up, and bin 0 there collects the offsets while the
// data add up like noise: 4096 x 3 points had 4.9e-7 of error in the bins of k1 = 0 against 1e-7 in the others.  Every
// other pencil therefore goes through with its sign turned round, which moves the offsets to the highest frequency.
template <int JT, int WI, int NMAX, int IN, int OUT, bool VEC>
__global__ void __launch_bounds__((CfgMdF<JT, WI, NMAX>::NT), 2)
k_matdft_fwd(MatdftArgs a)
{
    using Cf = CfgMdF<JT, WI, NMAX>;
    using Tab = MdRoots<NMAX>;
    constexpr bool COLQ = IN == MD_STRIDED;
    static_assert(!VEC || IN == MD_ROWS, "vector loads need contiguous pencils");
    extern __shared__ __align__(16) unsigned char md_lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 31, h = lane >> 5;
    const int N = a.N, H = N / 2;                           // slots 0 .. H: the pairs (n, N - n)
    constexpr bool ALT = IN == MD_ROWS && OUT == MD_ROWS;   // (above)
    const unsigned turn = (unsigned)(lane & 1) << 31;
    Tab::build(md_lds, N, tid, Cf::NT);

    const unsigned item = WI > 1 ? blockIdx.x : blockIdx.x * 4 + wave;
    const unsigned q0 = item / (unsigned)a.groups * 32;
    const int part = WI > 1 ? wave : 0, k0 = (int)(item % (unsigned)a.groups) * 32 * JT;
    if (WI == 1 && q0 >= a.P) return;

    // this lane's pencil (past the end: the last one, its results are not stored)
    const unsigned q = q0 + col < a.P ? q0 + col : a.P - 1;
    MdPencil pos{};
    if constexpr (IN == MD_STRIDED || OUT == MD_SPEC) pos = md_pencil(a, q, a.in_outer);
    const c64 *__restrict__ src = IN == MD_ROWS ? a.in + q * a.in_outer : a.in + pos.strided;
    const long long es = IN == MD_STRIDED ? a.inner : 1;

    // Raw elements of the slots n = n0 + 8 h + e: x[n] in u[e], x[N-n] in v[7 - e].  Every address is valid; what does not
    // belong to a pair (slot 0 has no partner, the middle of an even length is its own, slots past H) is put right by
    // `mend`, which only the first and the last block need.
    auto fetch = [&](c64 *u, c64 *v, int n0) __attribute__((always_inline)) {
        const int n = n0 + 8 * h;
        if constexpr (VEC) {
            const c64 *pu = src + n, *pv = src + (n ? N - n - 7 : N - 8);      // (n = 0: one element early)
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const md_u4a8 x = *reinterpret_cast<const md_u4a8 *>(pu + 2 * p), y = *reinterpret_cast<const md_u4a8 *>(pv + 2 * p);
                u[2 * p] = make_float2(__uint_as_float(x[0]), __uint_as_float(x[1]));
                u[2 * p + 1] = make_float2(__uint_as_float(x[2]), __uint_as_float(x[3]));
                v[2 * p] = make_float2(__uint_as_float(y[0]), __uint_as_float(y[1]));
                v[2 * p + 1] = make_float2(__uint_as_float(y[2]), __uint_as_float(y[3]));
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                u[e] = src[min(n + e, N - 1) * es];
                v[7 - e] = src[max(min(N - n - e, N - 1), 0) * es];
            }
        }
    };
    auto mend = [&](c64 *u, c64 *v, int n0) __attribute__((always_inline)) {
        const int n = n0 + 8 * h;
        const c64 zero = make_float2(0.f, 0.f);
        if (n0 == 0) {
            if constexpr (VEC) {
#pragma unroll
                for (int j = 0; j < 7; ++j) v[j] = n ? v[j] : v[j + 1];
            }
            v[7] = n ? v[7] : zero;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if (n + e > H) u[e] = zero;
            if (n + e > H || 2 * (n + e) == N) v[7 - e] = zero;
        }
    };

    // exponents (n k) mod N, times 4, of this lane's output column in each tile; advanced by k per slot, by `skip` from the
    // end of one block of 16 to the next one of this wave (the other half wave's 8 slots, the other waves' blocks)
    unsigned idx[JT], km[JT], skip[JT];
    const unsigned N4 = 4u * (unsigned)N;
#pragma unroll
    for (int t = 0; t < JT; ++t) {
        const unsigned k = k0 + 32 * t + col < a.K ? (unsigned)(k0 + 32 * t + col) : 0u;       // (past K: not stored)
        idx[t] = 4u * (k * (unsigned)(16 * part + 8 * h) % (unsigned)N);
        skip[t] = 4u * (k * (unsigned)(16 * WI - 8) % (unsigned)N);
        km[t] = 4u * k;
    }
    auto wrap = [&](unsigned e) __attribute__((always_inline)) { return min(e, e - N4); };
    // the next four roots of output tile t
    auto roots = [&](uintx4 *w, int t) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
#pragma unroll
            for (int k = 0; k < 3; ++k) w[k][e] = Tab::get(md_lds, idx[t], k);
            idx[t] = wrap(idx[t] + km[t]);
        }
    };

    md_floatx16 acc_re[JT], acc_im[JT];
#pragma unroll
    for (int t = 0; t < JT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) { acc_re[t][r] = 0.f; acc_im[t][r] = 0.f; }

    const int nblk = H / 16 + 1;
    if (part < nblk) {
        const int last = part + (nblk - 1 - part) / WI * WI;
        c64 u[8], v[8];
        uintx4 w[2][3];
        fetch(u, v, 16 * part);
        roots(w[0], 0);
#pragma unroll 1
        for (int blk = part; blk <= last; blk += WI) {
            if (blk == 0 || blk == nblk - 1) mend(u, v, 16 * blk);
            uintx4 re[2][3], im[2][3];                      // (s.re, d.im) and (s.im, -d.re) of the 8 pairs
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                c64 x = u[e], y = v[7 - e];
                if constexpr (ALT) {
                    x = make_float2(__uint_as_float(__float_as_uint(x.x) ^ turn), __uint_as_float(__float_as_uint(x.y) ^ turn));
                    y = make_float2(__uint_as_float(__float_as_uint(y.x) ^ turn), __uint_as_float(__float_as_uint(y.y) ^ turn));
                }
                const Split3 sr = split3(x.x + y.x), di = split3(x.y - y.y), si = split3(x.y + y.y), dr = split3(y.x - x.x);
                re[e / 4][0][e % 4] = pack_bf16(sr.t0, di.t0);
                re[e / 4][1][e % 4] = pack_bf16(sr.t1, di.t1);
                re[e / 4][2][e % 4] = pack_bf16(sr.t2, di.t2);
                im[e / 4][0][e % 4] = pack_bf16(si.t0, dr.t0);
                im[e / 4][1][e % 4] = pack_bf16(si.t1, dr.t1);
                im[e / 4][2][e % 4] = pack_bf16(si.t2, dr.t2);
            }
            __builtin_amdgcn_sched_barrier(0);
            fetch(u, v, 16 * min(blk + WI, last));          // (the last one is fetched again and dropped)
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int t = 0; t < JT; ++t) {
                    const int n = s * JT + t;
                    if (n >= JT) idx[t] = wrap(idx[t] + skip[t]);               // (the roots of both steps have been read)
                    __builtin_amdgcn_sched_barrier(0);
                    roots(w[(n + 1) & 1], (t + 1) % JT);                        // one ahead of the products
#pragma unroll
                    for (int k = 0; k < 6; ++k) {
                        const bf16x8 r16 = __builtin_bit_cast(bf16x8, w[n & 1][MD_SB[k]]);
                        const bf16x8 re16 = __builtin_bit_cast(bf16x8, re[s][MD_SA[k]]), im16 = __builtin_bit_cast(bf16x8, im[s][MD_SA[k]]);
                        if constexpr (COLQ) {
                            acc_re[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(r16, re16, acc_re[t], 0, 0, 0);
                            acc_im[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(r16, im16, acc_im[t], 0, 0, 0);
                        } else {
                            acc_re[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(re16, r16, acc_re[t], 0, 0, 0);
                            acc_im[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(im16, r16, acc_im[t], 0, 0, 0);
                        }
                    }
                }
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    // ---- stores.  (row, col) of a 32 x 32 tile: pencil row and output col, or the other way round (COLQ)
    auto put = [&](int t, int row, c64 val) __attribute__((always_inline)) {
        const int k = k0 + 32 * t + (COLQ ? row : col);
        const bool ok = k < a.K && q0 + (COLQ ? col : row) < a.P;
        if constexpr (OUT == MD_ROWS) {
            if (ALT && (row & 1)) val = make_float2(-val.x, -val.y);
            if (ok) a.out[(long long)(q0 + row) * a.out_outer + k] = val;
        } else {
            long long m = pos.m;
            int c = pos.c;
            if constexpr (!COLQ) {                          // (lane `row` holds that pencil's)
                const unsigned lo = __shfl((unsigned)pos.m, row), hi = __shfl((unsigned)(pos.m >> 32), row);
                m = (long long)(((unsigned long long)hi << 32) | lo);
                c = __shfl(pos.c, row);
            }
            m += (long long)k * a.inner;
            if (ok) a.out[((m >> 7) * a.C + c) * 128 + (m & 127)] = val;
        }
    };
    if constexpr (WI == 1) {
#pragma unroll
        for (int t = 0; t < JT; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                put(t, 8 * (r / 4) + 4 * h + (r % 4), make_float2(acc_re[t][r], acc_im[t][r]));
                __builtin_amdgcn_sched_barrier(0);          // (all addresses at once do not fit the registers)
            }
    } else {
        c64 *red = reinterpret_cast<c64 *>(md_lds);         // [WI][32 rows][32 columns], over the root table
#pragma unroll
        for (int t = 0; t < JT; ++t) {
            __syncthreads();
#pragma unroll
            for (int r = 0; r < 16; ++r)
                red[(part * 32 + 8 * (r / 4) + 4 * h + (r % 4)) * 32 + col] = make_float2(acc_re[t][r], acc_im[t][r]);
            __syncthreads();
#pragma unroll
            for (int r = 0; r < 16 / WI; ++r) {
                const int row = (32 / WI) * part + 2 * r + h;
                c64 sum = red[row * 32 + col];
#pragma unroll
                for (int p = 1; p < WI; ++p) sum = cadd(sum, red[(p * 32 + row) * 32 + col]);
                put(t, row, sum);
            }
        }
    }
}

// ------------------------------------------------------------------------------------------------ inverse
// G (contiguous outputs only): G = 1, 2, 4 waves of the workgroup own whole pencils, N < 128 G.  They put eight of them at a
// time together in LDS and store them as whole 128-byte lines past the caches (for odd N every other boundary between two
// eights splits a line).  A wave that stores its own 256-byte pieces
// leaves partial lines, which only the caches can merge; of a large output these stay in the last-level cache as dirty lines,
// and the next kernel's reads wait for their write-back (32 x 32 fields of 85 x 85: the next forward kernel takes 25 instead
// of 18 us; with non-temporal stores of pieces it is the inverse kernel that doubles).  G = 0: every wave on its own.
template <int PT, int NMAX, int IN, int OUT, int G>
__global__ void __launch_bounds__(256, 2)
k_matdft_inv(MatdftArgs a)
{
    using Tab = MdRoots<NMAX>;
    constexpr bool COLQ = OUT == MD_STRIDED;
    static_assert(G == 0 || (OUT == MD_ROWS && PT == 2), "whole pencils are contiguous ones");
    extern __shared__ __align__(16) unsigned char md_lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 31, h = lane >> 5;
    const int N = a.N, H = N / 2;                           // output pairs 0 .. H
    Tab::build(md_lds, N, tid, 256);

    const unsigned item = blockIdx.x * 4 + wave;            // (G: groups = G)
    const unsigned q0 = item / (unsigned)a.groups * 32;
    const int n0 = (int)(item % (unsigned)a.groups) * 32 * PT;
    if (G == 0 && q0 >= a.P) return;

    const unsigned q = q0 + col < a.P ? q0 + col : a.P - 1;
    MdPencil pos{};
    if constexpr (OUT == MD_STRIDED || IN == MD_SPEC) pos = md_pencil(a, q, a.out_outer);
    const c64 *__restrict__ src = IN == MD_ROWS ? a.in + q * a.in_outer : a.in + ((pos.m >> 7) * a.C + pos.c) * 128;
    const unsigned first = (unsigned)(pos.m & 127);         // place in the tile of element 0

    // modes i0 + 8 h + e of the pencil (past K: a valid address, zeroed by the caller)
    auto fetch = [&](c64 *u, int i0) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const unsigned i = (unsigned)min(i0 + 8 * h + e, a.K - 1);
            if constexpr (IN == MD_ROWS) u[e] = src[i];
            else {
                const unsigned m = first + i * a.inner;
                u[e] = src[(unsigned long long)(m >> 7) * ((unsigned)a.C * 128ULL) + (m & 127)];
            }
        }
    };

    unsigned idx[PT], nm[PT], skip[PT];                     // exponents of this lane's output column, as in the forward kernel
    const unsigned N4 = 4u * (unsigned)N;
#pragma unroll
    for (int t = 0; t < PT; ++t) {
        const unsigned n = n0 + 32 * t + col <= H ? (unsigned)(n0 + 32 * t + col) : 0u;        // (past H: not stored)
        idx[t] = 4u * (n * (unsigned)(8 * h) % (unsigned)N);
        skip[t] = 4u * (n * 8u % (unsigned)N);
        nm[t] = 4u * n;
    }
    auto wrap = [&](unsigned e) __attribute__((always_inline)) { return min(e, e - N4); };

    md_floatx16 cr[PT], ci[PT], sr[PT], si[PT];
#pragma unroll
    for (int t = 0; t < PT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) { cr[t][r] = 0.f; ci[t][r] = 0.f; sr[t][r] = 0.f; si[t][r] = 0.f; }

    c64 u[8];
    fetch(u, 0);
    const int modes = G > 0 && n0 > H ? 0 : a.K;            // (a wave past the last pair only helps to store)
#pragma unroll 1
    for (int i0 = 0; i0 < modes; i0 += 16) {
        if (i0 + 16 > a.K) {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (i0 + 8 * h + e >= a.K) u[e] = make_float2(0.f, 0.f);
        }
        uintx4 re[3], im[3];                                // real and imaginary parts, two modes per dword
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
        __builtin_amdgcn_sched_barrier(0);
        fetch(u, i0 + 16);
#pragma unroll
        for (int t = 0; t < PT; ++t) {
            __builtin_amdgcn_sched_barrier(0);
            uintx4 wc[3], ws[3];                            // (cos, cos) and (sin, sin) of two modes
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                unsigned r0[3], r1[3];
#pragma unroll
                for (int k = 0; k < 3; ++k) r0[k] = Tab::get(md_lds, idx[t], k);
                idx[t] = wrap(idx[t] + nm[t]);
#pragma unroll
                for (int k = 0; k < 3; ++k) r1[k] = Tab::get(md_lds, idx[t], k);
                idx[t] = wrap(idx[t] + nm[t]);
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    wc[k][d] = __builtin_amdgcn_perm(r1[k], r0[k], 0x05040100u);
                    ws[k][d] = __builtin_amdgcn_perm(r1[k], r0[k], 0x07060302u);
                }
            }
            idx[t] = wrap(idx[t] + skip[t]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                const bf16x8 c16 = __builtin_bit_cast(bf16x8, wc[MD_SB[k]]), s16 = __builtin_bit_cast(bf16x8, ws[MD_SB[k]]);
                const bf16x8 re16 = __builtin_bit_cast(bf16x8, re[MD_SA[k]]), im16 = __builtin_bit_cast(bf16x8, im[MD_SA[k]]);
                if constexpr (COLQ) {
                    cr[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c16, re16, cr[t], 0, 0, 0);
                    ci[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c16, im16, ci[t], 0, 0, 0);
                    sr[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(s16, re16, sr[t], 0, 0, 0);
                    si[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(s16, im16, si[t], 0, 0, 0);
                } else {
                    cr[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(re16, c16, cr[t], 0, 0, 0);
                    ci[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(im16, c16, ci[t], 0, 0, 0);
                    sr[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(re16, s16, sr[t], 0, 0, 0);
                    si[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(im16, s16, si[t], 0, 0, 0);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }

    // ---- stores: outputs n and N - n (0 and the middle of an even length have no partner)
    if constexpr (G > 0) {
        constexpr int T = 64 * G;                           // threads that store together
        const int t = tid % T;
        c64 *stage = reinterpret_cast<c64 *>(md_lds + Tab::BYTES / 16 * 16 + 16) + (tid / T) * (8 * N);
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {                    // pencils q0 + 8 rg .. + 7
            if constexpr (G > 1) __syncthreads();
            else wave_sync_md();
#pragma unroll
            for (int tt = 0; tt < PT; ++tt) {
                const int n = n0 + 32 * tt + col;
#pragma unroll
                for (int r = 4 * rg; r < 4 * rg + 4; ++r) {
                    c64 *row = stage + (4 * h + r % 4) * N;
                    if (n <= H) row[n] = make_float2(cr[tt][r] - si[tt][r], ci[tt][r] + sr[tt][r]);
                    if (n <= H && n && 2 * n != N) row[N - n] = make_float2(cr[tt][r] + si[tt][r], ci[tt][r] - sr[tt][r]);
                }
            }
            if constexpr (G > 1) __syncthreads();
            else wave_sync_md();
            const unsigned p0 = q0 + 8 * rg;
            if (p0 < a.P) {
                const int count = (int)(a.P - p0 < 8 ? a.P - p0 : 8) * N;
                c64 *dst = a.out + (long long)p0 * N;
                const int lead = (int)(((unsigned long long)dst >> 3) & 15);       // elements since the last line boundary
                for (int e = t - lead; e < count; e += T)
                    if (e >= 0) store_nt(dst + e, stage[e]);
            }
        }
        return;
    }
    const int out_es = COLQ ? (int)a.inner : 1;
#pragma unroll
    for (int t = 0; t < PT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = 8 * (r / 4) + 4 * h + (r % 4);
            const int n = n0 + 32 * t + (COLQ ? row : col);
            const bool ok = n <= H && q0 + (COLQ ? col : row) < a.P;
            c64 *dst = a.out + (COLQ ? pos.strided : (long long)(q0 + row) * a.out_outer);
            if (ok) dst[(long long)n * out_es] = make_float2(cr[t][r] - si[t][r], ci[t][r] + sr[t][r]);
            if (ok && n && 2 * n != N) dst[(long long)(N - n) * out_es] = make_float2(cr[t][r] + si[t][r], ci[t][r] - sr[t][r]);
            __builtin_amdgcn_sched_barrier(0);
        }
}

}  // namespace tfno
