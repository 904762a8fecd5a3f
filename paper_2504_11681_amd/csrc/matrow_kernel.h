// 1-D layers of lengths that are no powers of two, few pencils: forward transform; contraction and inverse transform.
//
// The transforms of matdft_kernel.h (contractions with the roots of unity on the matrix pipe, elements n and N - n folded, exact split
// into three BF16 terms).  One kernel per step left each of them a few microseconds of work behind a launch, and a wave with
// most of its time in work that its neighbours did as well.  Here
//   forward  16 pencils per workgroup, whose sums of N / 2 pairs are dealt out to up to eight waves; a wave forms all modes (up to 64), so
//            that a pair is fetched, folded and split once
//   inverse  one batch element x 32 outputs x a share of the output pairs per workgroup: it contracts the channels itself (the
//            spectrum of a batch element is some tens of KB, which the caches hold), splits the 32 contracted pencils once, into LDS in operand
//            form, and every wave forms tiles of 32 output pairs from them
//
// B 64, C 40 -> 56, N 1000, K 50: forward 12.7 -> 11.1 us (160 workgroups on 256 CUs; vector issue of the folds and splits and the matrix pipe in turn,
// two waves per SIMD), contraction 6.4 and inverse 17.5 -> 15.7 us together (all 256 workgroups contract, transform and then store their 29 MB
// at the same time, so that the phases add up); the layer 36.2 -> 26.0.  B 8, C 69 -> 72, N 116, K 12, all latency: 18.1 -> 10.2.
#pragma once
#include "matgrid_kernel.h"
#include "matrow.h"

namespace tfno {

constexpr int MR_WAVES = 8;

// LDS: root table, partial sums [parts][16][16 KT].
template <int KT, bool LONG>
__global__ void __launch_bounds__(64 * MR_WAVES, 2)
k_matrow_fwd(MatrowArgs a)
{
    extern __shared__ __align__(16) unsigned char mr_lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, threads = blockDim.x;
    const int col = lane & 15, g = lane >> 4;
    const int N = a.N, K = a.K, k0 = blockIdx.y * 16 * KT;
    const unsigned P = (unsigned)a.B * (unsigned)a.C_in, q0 = blockIdx.x * 16;
    c64 *red = reinterpret_cast<c64 *>(mr_lds + MG_ROOT * N);
    const c64 *__restrict__ src = a.x + (long long)min(q0 + col, P - 1) * N;     // (past the end: the last one, not stored)

    MgSums<1, KT> acc;
    mg_sum<1, KT, false, LONG, true>(acc, mr_lds, N, K, wave, a.parts, [&](c64 (*u)[4], c64 (*v)[4], int n) __attribute__((always_inline)) {
        // (slots go up to N / 2 + 15, inside the pencil from 32 points on)
        const c64 *lo = src + n, *hi = src + (N - n - 3);
        const md_u4a8 x0 = *reinterpret_cast<const md_u4a8 *>(lo), x1 = *reinterpret_cast<const md_u4a8 *>(lo + 2);
        const md_u4a8 y0 = *reinterpret_cast<const md_u4a8 *>(hi), y1 = *reinterpret_cast<const md_u4a8 *>(n ? hi + 2 : hi + 1);
        u[0][0] = make_float2(__uint_as_float(x0[0]), __uint_as_float(x0[1]));
        u[0][1] = make_float2(__uint_as_float(x0[2]), __uint_as_float(x0[3]));
        u[0][2] = make_float2(__uint_as_float(x1[0]), __uint_as_float(x1[1]));
        u[0][3] = make_float2(__uint_as_float(x1[2]), __uint_as_float(x1[3]));
        v[0][0] = make_float2(__uint_as_float(y0[0]), __uint_as_float(y0[1]));
        v[0][1] = make_float2(__uint_as_float(y0[2]), __uint_as_float(y0[3]));
        v[0][2] = make_float2(__uint_as_float(y1[0]), __uint_as_float(y1[1]));
        v[0][3] = make_float2(__uint_as_float(y1[2]), __uint_as_float(y1[3]));
    }, [&]() __attribute__((always_inline)) {
        mg_tables(mr_lds, N, N, tid, threads);
        __syncthreads();
    }, k0);
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            red[(wave * 16 + 4 * g + r) * (16 * KT) + 16 * t + col] = make_float2(acc.re[0][t][r], acc.im[0][t][r]);
    __syncthreads();
    for (int i = tid; i < 16 * 16 * KT; i += threads) {
        const int row = i / (16 * KT), k = k0 + i % (16 * KT);
        const unsigned q = q0 + row;
        if (k >= K || q >= P) continue;
        c64 sum = red[i];
        for (int p = 1; p < a.parts; ++p) sum = cadd(sum, red[p * (16 * 16 * KT) + i]);
        const unsigned b = q / (unsigned)a.C_in;
        a.Xh[mg_place((long long)b * K + k, (int)(q - b * (unsigned)a.C_in), a.C_in)] = sum;
    }
}

// LDS of the inverse kernel: root table, operands [steps][re, im][3 terms][64 lanes] of 16 bytes, partial sums [parts][32][KP].
TFNO_HD int mr_steps(int K) { return (K + 15) / 16; }
TFNO_HD int mr_pitch(int K) { return 16 * mr_steps(K) + 1; }

// NP: partial products of the contraction, as in k_cgemm_modes_direct.
template <int NP>
__global__ void __launch_bounds__(64 * MR_WAVES, 2)
k_matrow_inv(MatrowArgs a)
{
    extern __shared__ __align__(16) unsigned char mr_lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, waves = blockDim.x >> 6;
    const int col = lane & 31, h = lane >> 5;
    const int N = a.N, K = a.K, H = N / 2, steps = mr_steps(K), KP = mr_pitch(K), C_in = a.C_in;
    uintx4 *ops = reinterpret_cast<uintx4 *>(mr_lds + MG_ROOT * N);
    c64 *Y = reinterpret_cast<c64 *>(ops + steps * 6 * 64);
    const unsigned slabs = (unsigned)(a.C_out + 31) / 32, item = blockIdx.x / (unsigned)a.groups, group = blockIdx.x - item * (unsigned)a.groups;
    const unsigned b = item / slabs;
    const int o0 = 32 * (int)(item - b * slabs);

    // ---- contraction: 32 outputs x 32 modes per wave, the channels dealt out to `parts` waves
    const int mt = (K + 31) / 32, tile = wave % mt, part = wave / mt;
    auto tables = [&]() __attribute__((always_inline)) { mg_tables(mr_lds, N, N, tid, blockDim.x); };
    if (part < a.parts) {
        const int k = 32 * tile + col, o = min(o0 + col, a.C_out - 1);
        const long long m = (long long)b * K + min(k, K - 1);
        const c64 *__restrict__ xsrc = a.Xh + (m >> 7) * C_in * 128 + (m & 127);
        c64 xq[4], wq[4];
        auto load = [&](int c0) __attribute__((always_inline)) {
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int c = c0 + 4 * h + d, cc = c < C_in ? c : 0;       // (channels past C_in meet zero weights)
                wq[d] = a.W[cc * a.C_out + o];
                xq[d] = xsrc[cc * 128];
            }
        };
        md_floatx16 re, im;
#pragma unroll
        for (int r = 0; r < 16; ++r) { re[r] = 0.f; im[r] = 0.f; }
        load(8 * part);
        tables();
#pragma unroll 1
        for (int c0 = 8 * part; c0 < C_in; c0 += 8 * a.parts) {
            uintx4 x[3], wr[3], wi[3];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const Split3 xr = split3(xq[d].x), xi = split3(xq[d].y);
                x[0][d] = pack_bf16(xr.t0, xi.t0);
                x[1][d] = pack_bf16(xr.t1, xi.t1);
                x[2][d] = pack_bf16(xr.t2, xi.t2);
                const float s = c0 + 4 * h + d < C_in ? a.scale : 0.f;
                const Split3 r = split3(wq[d].x * s), i = split3(wq[d].y * s);
                wr[0][d] = pack_bf16(r.t0, i.t0) ^ 0x80000000u;
                wr[1][d] = pack_bf16(r.t1, i.t1) ^ 0x80000000u;
                wr[2][d] = pack_bf16(r.t2, i.t2) ^ 0x80000000u;
                wi[0][d] = pack_bf16(i.t0, r.t0);
                wi[1][d] = pack_bf16(i.t1, r.t1);
                wi[2][d] = pack_bf16(i.t2, r.t2);
            }
            __builtin_amdgcn_sched_barrier(0);
            load(min(c0 + 8 * a.parts, C_in - 1));          // (past the last step: loaded and dropped)
            __builtin_amdgcn_sched_barrier(0);
            constexpr int SA[8] = {2, 1, 2, 0, 1, 1, 0, 0}, SB[8] = {1, 2, 0, 2, 1, 0, 1, 0};
#pragma unroll
            for (int p = 8 - NP; p < 8; ++p) {
                const bf16x8 xx = __builtin_bit_cast(bf16x8, x[SB[p]]);
                re = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wr[SA[p]]), xx, re, 0, 0, 0);
                im = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wi[SA[p]]), xx, im, 0, 0, 0);
            }
        }
        if (k < 16 * steps) {
            c64 *dst = Y + (part * 32 + 4 * h) * KP + k;
#pragma unroll
            for (int r = 0; r < 16; ++r)
                dst[(8 * (r / 4) + r % 4) * KP] = k < K ? make_float2(re[r], im[r]) : make_float2(0.f, 0.f);
        }
    } else
        tables();
    __syncthreads();

    // ---- the 32 pencils in operand form
    for (int s = wave; s < steps; s += waves) {
        const c64 *row = Y + col * KP + 16 * s + 8 * h;
        c64 u[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) u[e] = row[e];
        for (int p = 1; p < a.parts; ++p)
#pragma unroll
            for (int e = 0; e < 8; ++e) u[e] = cadd(u[e], row[p * 32 * KP + e]);
        uintx4 re[3], im[3];
        mg_split(re, im, u);
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            ops[(s * 6 + t) * 64 + lane] = re[t];
            ops[(s * 6 + 3 + t) * 64 + lane] = im[t];
        }
    }
    __syncthreads();

    // ---- inverse transform, 32 output pairs at a time
    const unsigned NB = MG_ROOT * (unsigned)N;
    auto wrap = [&](unsigned e) __attribute__((always_inline)) { return min(e, e - NB); };
    c64 *__restrict__ out = a.y + ((long long)b * a.C_out + o0) * N;
    for (int n0 = 32 * ((int)group * waves + wave); n0 <= H; n0 += 32 * waves * a.groups) {
        const int n = n0 + col, nn = min(n, H);
        const unsigned step = MG_ROOT * (unsigned)nn, skip = MG_ROOT * ((unsigned)nn * 8u % (unsigned)N);
        unsigned idx = h ? skip : 0u;
        MgPairs s;
        mg_clear(s);
#pragma unroll 1
        for (int st = 0; st < steps; ++st) {
            uintx4 wc[3], ws[3], re[3], im[3];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const md_u3 r0 = mg_root(mr_lds, idx);
                idx = wrap(idx + step);
                const md_u3 r1 = mg_root(mr_lds, idx);
                idx = wrap(idx + step);
#pragma unroll
                for (int t = 0; t < 3; ++t) {
                    wc[t][d] = __builtin_amdgcn_perm(r1[t], r0[t], 0x05040100u);
                    ws[t][d] = __builtin_amdgcn_perm(r1[t], r0[t], 0x07060302u);
                }
            }
            idx = wrap(idx + skip);
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                re[t] = ops[(st * 6 + t) * 64 + lane];
                im[t] = ops[(st * 6 + 3 + t) * 64 + lane];
            }
            mg_pairs<false>(s, re, im, wc, ws);
        }
        c64 *lo = out + (unsigned)(4 * h * N + n), *hi = out + (unsigned)(4 * h * N + N - n);
        const int rows = a.C_out - o0 - 4 * h;              // (output row 8 (r / 4) + r % 4 of this half exists below this)
        const bool mirror = n && 2 * n != N;
        if (n <= H) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = 8 * (r / 4) + r % 4;
                if (row < rows) {
                    lo[(unsigned)(row * N)] = make_float2(s.cr[r] - s.si[r], s.ci[r] + s.sr[r]);
                    if (mirror) hi[(unsigned)(row * N)] = make_float2(s.cr[r] + s.si[r], s.ci[r] - s.sr[r]);
                }
            }
        }
    }
}

}  // namespace tfno
