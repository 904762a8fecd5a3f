// Pruned transforms along the leading (strided) axis of row-major fields, the outer two stages of the 2-D strip pipeline
// (Sec. 3.2 / 3.3): N1 = P T points of every column, of which K1 <= P Q modes are kept.
//
//   workgroup = 16 adjacent columns of one field (a 128-byte line of every row), read and written once
//   stage A   thread (column, t) transforms the rows t + T j, j < P, in registers, times w_N1^(t p)
//   stage B   thread (column, p): T-point transform over t, pruned to the Q outputs that are modes p + P q < P Q
// through one LDS tile [p][t][column]; the inverse runs the transposed network with the missing modes as zeros.  Bound:
// HBM (about 30 vector instructions per element); all rows of the 16 columns are in flight at once, two or more
// workgroups per CU (512 rows: 64 KB of LDS).  4 x 32 fields of 512 x 512 (268 MB), 64 modes: forward 59 us, inverse 57 us
// = 5.1 and 5.3 TB/s (a radix-2 transform of the same columns in LDS: 397 and 323 us); 32 modes: 54 us each.  The
// tile's p rows are padded by 16 elements, so that the four p of a wave meet different bank halves.
//
// `contiguous`: the workgroups of an XCD take neighbouring columns and fields (see xcd_contiguous) instead of every eighth line of
// each row; when, and what it measured, stands at the launcher.
//
// SPEC: the modes are the truncated spectrum of grids whose last axis has another transform, mode-tile major as the
// contraction kernels take it (mode k of column n2 of field b C + c is mode b M + k N2 + n2), and N2 is any number of columns.
#pragma once
#include "common.h"
#include "fft_regs.h"

namespace tfno {

template <int P, int T, int Q>
struct CfgCol {
    static constexpr int N1 = P * T, COLS = 16;
    static constexpr int NT = T >= 16 ? 256 : 16 * T;       // threads
    static constexpr int TPT = T * COLS / NT;               // stage-A slices per thread
    static constexpr int IPT = P * COLS / NT;               // stage-B items per thread
    static constexpr int PS = T * COLS + COLS;              // elements between the p rows of the tile
    static constexpr size_t LDS = sizeof(c64) * (P * PS);
    static constexpr int WG_PER_CU = LDS <= 40 * 1024 ? 4 : 2;
    static_assert(TPT >= 1 && IPT >= 1 && TPT * NT == T * COLS && IPT * NT == P * COLS, "work divides evenly");
    static_assert(T % Q == 0, "pruned stage");
};

template <int P, int T, int Q>
__device__ __forceinline__ void col_twiddles(c64 *tw, int tid)
{
    for (int i = tid; i < P * T; i += CfgCol<P, T, Q>::NT) tw[i] = cis2pi(-(float)((i / P) * (i % P)), (float)(P * T));
}

// element `col` of row k of a mode-tile-major spectrum (see above)
__device__ __forceinline__ long long col_spec(unsigned b, unsigned c, int C, long long M, int k, int N2, int col)
{
    const long long m = b * M + (long long)k * N2 + col;
    return ((m >> 7) * C + c) * 128 + (m & 127);
}

template <int P, int T, int Q, bool SPEC>
__global__ void __launch_bounds__((CfgCol<P, T, Q>::NT), (CfgCol<P, T, Q>::WG_PER_CU))
k_colfft_fwd(const c64 *__restrict__ in, c64 *__restrict__ out, int N2, int K1, unsigned groups, bool contiguous, int Cs, long long M, long long channel)
{
    using C = CfgCol<P, T, Q>;
    extern __shared__ __align__(16) unsigned char col_lds[];
    c64 *Z = reinterpret_cast<c64 *>(col_lds);
    __shared__ c64 tw[P * T];                               // w_N1^(t p) at [t][p]
    const int tid = threadIdx.x, col = tid & 15, sub = tid >> 4;
    const unsigned wg = contiguous ? xcd_contiguous(blockIdx.x, gridDim.x) : blockIdx.x, field = wg / groups, g = wg % groups;
    // (SPEC: columns past the last one read it again and are not stored)
    const int n2 = (int)(16 * g) + col, n2_in = SPEC && n2 >= N2 ? N2 - 1 : n2;
    const c64 *__restrict__ src = in + (long long)field * C::N1 * N2 + n2_in;
    const unsigned sb = field / (unsigned)Cs, sc = field - sb * (unsigned)Cs;
    c64 *__restrict__ dst = out + (SPEC ? 0 : (long long)sb * M + (long long)sc * channel) + n2;

    c64 v[C::TPT][P];
#pragma unroll
    for (int i = 0; i < C::TPT; ++i)
#pragma unroll
        for (int j = 0; j < P; ++j) {
            const c64 *row = src + (long long)(sub + (C::NT / 16) * i + T * j) * N2;
            v[i][j] = SPEC ? *row : load_nt(row);
        }
    __builtin_amdgcn_sched_barrier(0);
    col_twiddles<P, T, Q>(tw, tid);                         // while the loads are in flight
    __syncthreads();
#pragma unroll
    for (int i = 0; i < C::TPT; ++i) {
        const int t = sub + (C::NT / 16) * i;
        c64 z[P];
        RegFFT<P, -1, 1>::run(v[i], z);
#pragma unroll
        for (int p = 0; p < P; ++p) Z[p * C::PS + t * 16 + col] = p == 0 ? z[0] : cmul(z[p], tw[t * P + p]);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < C::IPT; ++i) {
        const int p = sub + (C::NT / 16) * i;
        c64 xo[Q];
        dft_prune_out_blocks<T, Q, -1>([&](auto tc) __attribute__((always_inline)) {
            constexpr int t = decltype(tc)::value;
            return Z[p * C::PS + t * 16 + col];
        }, xo);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int k = p + P * q;
            if constexpr (SPEC) {
                if (k < K1 && n2 < N2) out[col_spec(sb, sc, Cs, M, k, N2, n2)] = xo[q];
            } else {
                if (k < K1) dst[(long long)k * N2] = xo[q];
            }
        }
    }
}

template <int P, int T, int Q, bool SPEC>
__global__ void __launch_bounds__((CfgCol<P, T, Q>::NT), (CfgCol<P, T, Q>::WG_PER_CU))
k_colfft_inv(const c64 *in, c64 *out, int N2, int K1, unsigned groups, bool contiguous, int Cs, long long M)
{
    using C = CfgCol<P, T, Q>;
    extern __shared__ __align__(16) unsigned char col_lds[];
    c64 *Z = reinterpret_cast<c64 *>(col_lds);
    __shared__ c64 tw[P * T];
    const int tid = threadIdx.x, col = tid & 15, sub = tid >> 4;
    const unsigned wg = contiguous ? xcd_contiguous(blockIdx.x, gridDim.x) : blockIdx.x, field = wg / groups, g = wg % groups;
    const int n2 = (int)(16 * g) + col, n2_in = SPEC && n2 >= N2 ? N2 - 1 : n2;
    // (the modes of a field may lie in its own rows: a workgroup has read its columns when it first writes to them)
    const c64 *src = in + (SPEC ? 0 : (long long)field * M) + n2;
    c64 *dst = out + (long long)field * C::N1 * N2 + n2;
    const unsigned sb = SPEC ? field / (unsigned)Cs : 0, sc = SPEC ? field % (unsigned)Cs : 0;

    c64 v[C::IPT][Q];
#pragma unroll
    for (int i = 0; i < C::IPT; ++i)
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int k = sub + (C::NT / 16) * i + P * q;
            const c64 w = SPEC ? in[col_spec(sb, sc, Cs, M, k < K1 ? k : 0, N2, n2_in)] : src[(long long)(k < K1 ? k : 0) * N2];
            v[i][q] = k < K1 ? w : make_float2(0.f, 0.f);
        }
    __builtin_amdgcn_sched_barrier(0);
    col_twiddles<P, T, Q>(tw, tid);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < C::IPT; ++i) {
        const int p = sub + (C::NT / 16) * i;
        dft_prune_in<T, Q, +1>(v[i], [&](auto tc, c64 val) __attribute__((always_inline)) {
            constexpr int t = decltype(tc)::value;
            if constexpr (t == 0) Z[p * C::PS + col] = val;
            else {
                const c64 w = tw[t * P + p];
                Z[p * C::PS + t * 16 + col] = cmul(val, make_float2(w.x, -w.y));
            }
        });
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < C::TPT; ++i) {
        const int t = sub + (C::NT / 16) * i;
        c64 z[P], r[P];
#pragma unroll
        for (int p = 0; p < P; ++p) z[p] = Z[p * C::PS + t * 16 + col];
        RegFFT<P, +1, 1>::run(z, r);
#pragma unroll
        for (int j = 0; j < P; ++j) {
            if constexpr (SPEC) {           // (read again by the next kernel)
                if (n2 < N2) dst[(long long)(t + T * j) * N2] = r[j];
            } else {
                store_nt(dst + (long long)(t + T * j) * N2, r[j]);
            }
        }
    }
}

}  // namespace tfno
