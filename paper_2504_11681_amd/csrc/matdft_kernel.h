// Pruned DFT of any length on the matrix pipe:  out[q][j] = sum_i in[q][i] w^(i j),  w = exp(dir 2 pi i / N).
//
// A length without factors of two has no butterfly network to prune, but a transform that keeps K of N bins is a
// contraction of the pencils with an N x K matrix of roots of unity, and K is small.  The matrix is never stored: its
// entries are w^((i j) mod N), so a workgroup builds the N roots once in LDS, already split into three BF16 terms
// (bf16x3.h: the split is exact, six products, FP32 accumulation), and a lane fetches the root of its (i, j) with one
// 16-byte LDS read, the exponent advanced by one addition and one wrap.
//
//   wave      = 32 pencils x 32 JT outputs, v_mfma_f32_32x32x16_bf16 over 8 complex inputs per step
//   input     a lane owns one pencil (lane % 32) and 8 of every 16 consecutive elements (lane / 32): 64 contiguous
//             bytes of a contiguous pencil, 256 contiguous bytes per half wave of a strided one; the next 16 elements
//             are in flight while these are contracted
//   WI = 4, 8 the waves of a workgroup share a tile and deal the blocks of 16 elements out among them; partial sums meet
//             in LDS.  For few pencils and long sums (truncating a batch of 2560 pencils fills 80 waves without the split).
//   WI = 1    a wave per tile, for many pencils or short sums
// The pencils are the rows of the product where outputs of one pencil are contiguous in memory, and its columns where
// neighbouring pencils are (COLQ), so a half wave always stores 256 contiguous bytes.
// Root table: entry e at e + e / 16, so that the lanes of a step, whose exponents are multiples of i apart, do not all
// meet in the same four banks when i is a multiple of 16.
#pragma once
#include "common.h"
#include "bf16x3.h"
#include "matdft.h"

namespace tfno {

typedef float md_floatx16 __attribute__((ext_vector_type(16)));
typedef unsigned md_u4a8 __attribute__((ext_vector_type(4), aligned(8)));

// exp(2 pi i m / N) for 0 <= m < N: the quotient 2 m / N is rounded, so its remainder is put back to first order (without
// it the angle of a length that is no power of two is off by up to 2e-7).
__device__ __forceinline__ c64 root_of_unity(int m, int N)
{
    if (2 * m > N) m -= N;                                  // -N/2 < m <= N/2: a smaller angle, a smaller rounding error
    const float n = (float)N, num = (float)(2 * m);
    const float q = num / n;
    const float d = 3.14159265358979f * (fmaf(-q, n, num) / n);
    float s, c;
    sincospif(q, &s, &c);
    return make_float2(fmaf(-s, d, c), fmaf(c, d, s));
}

template <int JT, int WI>
struct CfgMd {
    static constexpr int NT = WI > 4 ? 64 * WI : 256;
    static constexpr size_t RED = WI > 1 ? sizeof(c64) * WI * 32 * 32 : 0;         // one 32 x 32 tile of every wave
    static size_t lds_bytes(int N)
    {
        const size_t tw = 16 * (size_t)(N + N / 16 + 1);
        return tw > RED ? tw : RED;
    }
};

template <int JT, int WI, int IN, int OUT>
__global__ void __launch_bounds__((CfgMd<JT, WI>::NT), 2)
k_matdft(MatdftArgs a)
{
    constexpr bool COLQ = IN == MD_STRIDED || OUT == MD_STRIDED;
    extern __shared__ __align__(16) unsigned char md_lds[];
    uintx4 *tw = reinterpret_cast<uintx4 *>(md_lds);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 31, h = lane >> 5;
    const int N = a.N;

    for (int e = tid; e < N; e += CfgMd<JT, WI>::NT) {
        c64 w = root_of_unity(e, N);
        if (a.dir < 0) w.y = -w.y;
        const Split3 re = split3(w.x), im = split3(w.y);
        tw[e + (e >> 4)] = uintx4{pack_bf16(re.t0, im.t0), pack_bf16(re.t1, im.t1), pack_bf16(re.t2, im.t2), 0u};
    }
    __syncthreads();

    const unsigned item = WI > 1 ? blockIdx.x : blockIdx.x * 4 + wave;
    const unsigned tile = item / (unsigned)a.jgroups, jg = item % (unsigned)a.jgroups;
    const unsigned q0 = tile * 32;                          // (past the end for the last waves of the last workgroup)
    const int part = WI > 1 ? wave : 0;
    if (WI == 1 && q0 >= a.P) return;

    // ---- this lane's pencil on the input side (past the end: the last one, its results are not stored)
    const unsigned q = q0 + col < a.P ? q0 + col : a.P - 1;
    const c64 *src;
    long long sb = 0;                                       // MD_SPEC: mode of element 0
    int sc = 0;                                             // MD_SPEC: channel
    long long ob = 0;                                       // output side: offset of element 0, or its mode
    int oc = 0;
    {
        const unsigned img = a.inner == 1 ? q : q / a.inner, r = a.inner == 1 ? 0 : q - img * a.inner;
        if constexpr (IN == MD_SPEC || OUT == MD_SPEC) {
            const unsigned b = img / (unsigned)a.C;
            const int c = (int)(img - b * (unsigned)a.C);
            const long long m = b * a.M + r;
            if constexpr (IN == MD_SPEC) { sb = m; sc = c; }
            if constexpr (OUT == MD_SPEC) { ob = m; oc = c; }
        }
        if constexpr (IN == MD_ROWS) src = a.in + q * a.in_outer;
        else if constexpr (IN == MD_STRIDED) src = a.in + img * a.in_outer + r;
        else src = a.in;
        if constexpr (OUT == MD_ROWS) ob = q * a.out_outer;
        else if constexpr (OUT == MD_STRIDED) ob = img * a.out_outer + r;
    }
    const long long es = IN == MD_STRIDED ? a.inner : 1;    // input element stride

    auto element = [&](int i) __attribute__((always_inline)) {
        if constexpr (IN == MD_SPEC) {
            const long long m = sb + (long long)i * a.inner;
            return src[((m >> 7) * a.C + sc) * 128 + (m & 127)];
        } else {
            return src[i * es];
        }
    };
    // elements i0 + 8 h .. + 7 of the pencil (a whole block)
    auto fetch = [&](c64 *v, int i0) __attribute__((always_inline)) {
        const int i = i0 + 8 * h;
        if constexpr (IN == MD_ROWS) {
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const md_u4a8 w = *reinterpret_cast<const md_u4a8 *>(src + i + 2 * p);
                v[2 * p] = make_float2(__uint_as_float(w[0]), __uint_as_float(w[1]));
                v[2 * p + 1] = make_float2(__uint_as_float(w[2]), __uint_as_float(w[3]));
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = element(i + e);
        }
    };

    // ---- exponents (i j) mod N of this lane's output column in each tile; advanced by j per element, by `skip` from
    // the end of one block of 16 to the next one of this wave (the other half wave's 8 elements, the other waves' blocks)
    unsigned idx[JT], jm[JT], skip[JT];
    const int j0 = (int)jg * 32 * JT;
#pragma unroll
    for (int t = 0; t < JT; ++t) {
        const int j = j0 + 32 * t + col;
        jm[t] = j < a.J ? (unsigned)j : 0u;                 // (columns past J are not stored)
        idx[t] = jm[t] * (unsigned)(16 * part + 8 * h) % (unsigned)N;
        skip[t] = jm[t] * (unsigned)(16 * WI - 8) % (unsigned)N;
    }
    auto wrap = [&](unsigned e) __attribute__((always_inline)) { return min(e, e - (unsigned)N); };

    md_floatx16 acc_re[JT], acc_im[JT];
#pragma unroll
    for (int t = 0; t < JT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) { acc_re[t][r] = 0.f; acc_im[t][r] = 0.f; }

    // the split of a group of four elements: dword = (re | im << 16) of one term
    auto split4 = [&](const c64 *v, uintx4 *d) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const Split3 re = split3(v[e].x), im = split3(v[e].y);
            d[0][e] = pack_bf16(re.t0, im.t0);
            d[1][e] = pack_bf16(re.t1, im.t1);
            d[2][e] = pack_bf16(re.t2, im.t2);
        }
    };
    // the next four roots of output tile t
    auto roots = [&](uintx4 *w, int t) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uintx4 z = tw[idx[t] + (idx[t] >> 4)];
            w[0][e] = z[0];
            w[1][e] = z[1];
            w[2][e] = z[2];
            idx[t] = wrap(idx[t] + jm[t]);
        }
    };
    // four elements of every lane against four roots: x . (re, -im) is the real part, x . (im, re) the imaginary part
    auto contract = [&](const uintx4 *x_re, const uintx4 *x_im, const uintx4 *w, int t) __attribute__((always_inline)) {
        constexpr int SA[6] = {2, 0, 1, 1, 0, 0}, SB[6] = {0, 2, 1, 0, 1, 0};   // smallest products first
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const bf16x8 r16 = __builtin_bit_cast(bf16x8, w[SB[k]]);
            const bf16x8 re16 = __builtin_bit_cast(bf16x8, x_re[SA[k]]), im16 = __builtin_bit_cast(bf16x8, x_im[SA[k]]);
            if constexpr (COLQ) {
                acc_re[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(r16, re16, acc_re[t], 0, 0, 0);
                acc_im[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(r16, im16, acc_im[t], 0, 0, 0);
            } else {
                acc_re[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(re16, r16, acc_re[t], 0, 0, 0);
                acc_im[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(im16, r16, acc_im[t], 0, 0, 0);
            }
        }
    };
    auto parts = [&](const uintx4 *d, uintx4 *x_re, uintx4 *x_im) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                x_re[k][e] = d[k][e] ^ 0x80000000u;
                x_im[k][e] = __builtin_amdgcn_alignbit(d[k][e], d[k][e], 16);
            }
    };

    // whole blocks of 16 elements, the next D in flight (past the end the last one is fetched again and dropped); the
    // roots of the next (step, tile) are read while this one is contracted
    const int full = a.I / 16, left = a.I - 16 * full;
    if (part < full) {
        constexpr int D = JT <= 2 ? 2 : 1;
        const int last = part + (full - 1 - part) / WI * WI;
        c64 v[D][8];
        uintx4 w[2][3];
#pragma unroll
        for (int e = 0; e < D; ++e) fetch(v[e], 16 * min(part + e * WI, last));
        roots(w[0], 0);
        for (int blk = part; blk <= last; blk += D * WI) {
#pragma unroll
            for (int e = 0; e < D; ++e) {
                if (e && blk + e * WI > last) break;
                uintx4 d[2][3];
                split4(v[e], d[0]);
                split4(v[e] + 4, d[1]);
                __builtin_amdgcn_sched_barrier(0);
                fetch(v[e], 16 * min(blk + (e + D) * WI, last));
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    uintx4 x_re[3], x_im[3];
                    parts(d[s], x_re, x_im);
#pragma unroll
                    for (int t = 0; t < JT; ++t) {
                        const int n = s * JT + t, tn = (t + 1) % JT;
                        if (n >= JT) idx[t] = wrap(idx[t] + skip[t]);       // (the roots of both steps have been read)
                        __builtin_amdgcn_sched_barrier(0);
                        roots(w[(n + 1) & 1], tn);
                        contract(x_re, x_im, w[n & 1], t);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    // the remainder: one step of up to 8 elements (four per half wave), or two
    if (left && part == full % WI) {
        const int per = left > 8 ? 8 : 4, i0 = 16 * full + per * h;
#pragma unroll
        for (int t = 0; t < JT; ++t) idx[t] = jm[t] * (unsigned)i0 % (unsigned)N;
#pragma unroll 1
        for (int s = 0; s < per; s += 4) {
            c64 v[4];
            uintx4 d[3], x_re[3], x_im[3];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool in = i0 + s + e < a.I;
                const c64 u = element(in ? i0 + s + e : 0);
                v[e] = in ? u : make_float2(0.f, 0.f);
            }
            split4(v, d);
            parts(d, x_re, x_im);
#pragma unroll
            for (int t = 0; t < JT; ++t) {
                uintx4 w[3];
                roots(w, t);
                contract(x_re, x_im, w, t);
            }
        }
    }

    // ---- stores.  (row, col) of a 32 x 32 tile: pencil row and output col, or the other way round (COLQ)
    auto put = [&](int t, int row, c64 val) __attribute__((always_inline)) {
        const int j = j0 + 32 * t + (COLQ ? row : col);
        const bool ok = j < a.J && q0 + (COLQ ? col : row) < a.P;
        if constexpr (COLQ) {
            if (!ok) return;
            if constexpr (OUT == MD_SPEC) {
                const long long m = ob + (long long)j * a.inner;
                a.out[((m >> 7) * a.C + oc) * 128 + (m & 127)] = val;
            } else {
                a.out[ob + (long long)j * a.inner] = val;
            }
        } else if constexpr (OUT == MD_ROWS) {
            if (ok) a.out[(long long)(q0 + row) * a.out_outer + j] = val;
        } else {
            // (lane `row` holds the mode of element 0 and the channel of that pencil)
            const unsigned lo = __shfl((unsigned)ob, row), hi = __shfl((unsigned)(ob >> 32), row);
            const int c = __shfl(oc, row);
            const long long m = (long long)(((unsigned long long)hi << 32) | lo) + j;
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

}  // namespace tfno
