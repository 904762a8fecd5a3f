// Register-resident small transforms for the fused kernels: every index and every twiddle is a
// compile-time constant, so a transform is a straight line of VALU instructions on VGPRs.
//
//  RegFFT<L, DIR>        full L-point DFT, L in {1,2,4,8,16,32}, natural order in and out
//  dft_prune_out<T,Q>    first Q outputs of a T-point DFT     (output pruning: the forward transform only
//                        feeds retained modes, Sec. 3.3 "FFT pruning")
//  dft_prune_in<T,Q>     T-point DFT of an input whose bins Q..T-1 are zero (input pruning: the inverse
//                        transform of a zero-padded spectrum, Sec. 3.3)
//  dft_prune_out_sym<T,Q>, dft_prune_in_sym<T,Q>   the same for the 2 Q bins -Q..Q-1
//  real_dft16, hermitian_dft16   16-point DFT of real values (bins 0..8), and its mirror: real results from bins 0..8
// DIR = -1: exp(-2 pi i k n / L) (forward);  DIR = +1: inverse, unscaled.
#pragma once
#include "common.h"
#include <type_traits>

namespace tfno {

template <int I, int E, class F>
TFNO_HD void static_for(F &&f)
{
    if constexpr (I < E) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, E>(f);
    }
}

// cos(2 pi m / 32), built from the first quadrant so that the symmetries are exact.
__host__ __device__ constexpr float cos32(int m)
{
    constexpr float q[9] = {1.0f, 9.807852804e-01f, 9.238795325e-01f, 8.314696123e-01f, 7.071067812e-01f,
                            5.555702330e-01f, 3.826834324e-01f, 1.950903220e-01f, 0.0f};
    m &= 31;
    return m <= 8 ? q[m] : m <= 16 ? -q[16 - m] : m <= 24 ? -q[m - 16] : q[32 - m];
}
__host__ __device__ constexpr float sin32(int m) { return cos32(m + 24); }

// a * exp(DIR * 2 pi i * M / L), with L | 32; trivial factors cost no multiply.
template <int L, int DIR, int M>
TFNO_HD c64 mul_tw(c64 a)
{
    constexpr int m = (((M % L) + L) % L) * (32 / L);   // index into the 32nd roots
    if constexpr (m == 0) return a;
    else if constexpr (m == 16) return make_float2(-a.x, -a.y);
    else if constexpr (m == 8) return DIR > 0 ? make_float2(-a.y, a.x) : make_float2(a.y, -a.x);
    else if constexpr (m == 24) return DIR > 0 ? make_float2(a.y, -a.x) : make_float2(-a.y, a.x);
    else {
        constexpr float c = cos32(m), s = DIR * sin32(m);
        return make_float2(fmaf(a.x, c, -(a.y * s)), fmaf(a.x, s, a.y * c));
    }
}

// acc + a * exp(DIR * 2 pi i * M / L)
template <int L, int DIR, int M>
TFNO_HD c64 mac_tw(c64 acc, c64 a)
{
    constexpr int m = (((M % L) + L) % L) * (32 / L);
    if constexpr (m == 0 || m == 8 || m == 16 || m == 24) return cadd(acc, mul_tw<L, DIR, M>(a));
    else {
        constexpr float c = cos32(m), s = DIR * sin32(m);
        float re = fmaf(a.x, c, acc.x);
        re = fmaf(-a.y, s, re);
        float im = fmaf(a.x, s, acc.y);
        im = fmaf(a.y, c, im);
        return make_float2(re, im);
    }
}

// lo = e + w o, hi = e - w o with w = exp(DIR * 2 pi i * M / L).  For a general twiddle the product is folded into
// the sum (4 FMAs) and hi = 2 e - lo (2 FMAs): 6 instructions instead of 8.
template <int L, int DIR, int M>
TFNO_HD void butterfly_tw(c64 e, c64 o, c64 &lo, c64 &hi)
{
    constexpr int m = (((M % L) + L) % L) * (32 / L);
    if constexpr (m % 8 == 0) {
        const c64 t = mul_tw<L, DIR, M>(o);
        lo = cadd(e, t);
        hi = csub(e, t);
    } else {
        constexpr float c = cos32(m), s = DIR * sin32(m);
        lo.x = fmaf(-o.y, s, fmaf(o.x, c, e.x));
        lo.y = fmaf(o.x, s, fmaf(o.y, c, e.y));
        hi.x = fmaf(2.f, e.x, -lo.x);
        hi.y = fmaf(2.f, e.y, -lo.y);
    }
}

// Recursive radix-2 decimation in time on registers.  in[i * STRIDE], i < L  ->  out[k], k < L.
template <int L, int DIR, int STRIDE = 1>
struct RegFFT {
    TFNO_HD static void run(const c64 *in, c64 *out)
    {
        c64 e[L / 2], o[L / 2];
        RegFFT<L / 2, DIR, 2 * STRIDE>::run(in, e);
        RegFFT<L / 2, DIR, 2 * STRIDE>::run(in + STRIDE, o);
        static_for<0, L / 2>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            butterfly_tw<L, DIR, k>(e[k], o[k], out[k], out[k + L / 2]);
        });
    }
};
template <int DIR, int STRIDE>
struct RegFFT<1, DIR, STRIDE> {
    TFNO_HD static void run(const c64 *in, c64 *out) { out[0] = in[0]; }
};

// First (decimation-in-frequency) level of an L-point transform: after it the input registers are dead, so a
// caller can refill them from memory while the two half-size transforms run.
//   even outputs  X[2k]   = DFT_{L/2}(a)[k],  a[i] = v[i] + v[i + L/2]
//   odd outputs   X[2k+1] = DFT_{L/2}(b)[k],  b[i] = (v[i] - v[i + L/2]) exp(DIR 2 pi i i / L)
template <int L, int DIR>
TFNO_HD void dif_first_level(const c64 *v, c64 *a, c64 *b)
{
    static_for<0, L / 2>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        a[i] = cadd(v[i], v[i + L / 2]);
        b[i] = mul_tw<L, DIR, i>(csub(v[i], v[i + L / 2]));
    });
}

// out[q] = sum_{t<T} in(t) exp(DIR 2 pi i t q / T),  q < Q,  Q | T.     in: callable int -> c64
// t = t1 + S t2 (S = T/Q):  S full Q-point transforms of the decimated input, then a twiddled S-term sum.
// The input is consumed Q values at a time, so a caller that reads it from LDS keeps only one group live.
// One group of the network: g = inputs t1, t1 + S, ..., t1 + (Q-1) S (destroyed); adds its share to out.
template <int T, int Q, int DIR, int T1>
TFNO_HD void dft_prune_out_group(c64 *g, c64 *out)
{
    c64 F[Q];
    RegFFT<Q, DIR, 1>::run(g, F);
    static_for<0, Q>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        if constexpr (T1 == 0) out[q] = F[q];
        else out[q] = mac_tw<T, DIR, T1 * q>(out[q], F[q]);
    });
}

template <int T, int Q, int DIR, class In>
TFNO_HD void dft_prune_out(In &&in, c64 *out)
{
    constexpr int S = T / Q;
    static_for<0, S>([&](auto t1c) {
        constexpr int t1 = decltype(t1c)::value;
        c64 g[Q];
        static_for<0, Q>([&](auto t2c) {
            constexpr int t2 = decltype(t2c)::value;
            g[t2] = in(std::integral_constant<int, t1 + S * t2>{});
        });
        dft_prune_out_group<T, Q, DIR, t1>(g, out);
    });
}

// The same with the S-term sums added up four terms at a time: for few outputs of a long transform (Q much smaller than T) one
// chain of S terms rounds more than a butterfly network would (32 terms: 1.06e-7 against 0.70e-7).
template <int T, int Q, int DIR, class In>
TFNO_HD void dft_prune_out_blocks(In &&in, c64 *out)
{
    constexpr int S = T / Q;
    if constexpr (S <= 4) {
        dft_prune_out<T, Q, DIR>(in, out);
    } else {
        static_for<0, S / 4>([&](auto bc) {
            constexpr int b = decltype(bc)::value;
            c64 part[Q];
            static_for<4 * b, 4 * b + 4>([&](auto t1c) {
                constexpr int t1 = decltype(t1c)::value;
                c64 g[Q], F[Q];
                static_for<0, Q>([&](auto t2c) {
                    constexpr int t2 = decltype(t2c)::value;
                    g[t2] = in(std::integral_constant<int, t1 + S * t2>{});
                });
                RegFFT<Q, DIR, 1>::run(g, F);
                static_for<0, Q>([&](auto qc) {
                    constexpr int q = decltype(qc)::value;
                    if constexpr (t1 == 4 * b) part[q] = mul_tw<T, DIR, t1 * q>(F[q]);
                    else part[q] = mac_tw<T, DIR, t1 * q>(part[q], F[q]);
                });
            });
            static_for<0, Q>([&](auto qc) {
                constexpr int q = decltype(qc)::value;
                out[q] = b == 0 ? part[q] : cadd(out[q], part[q]);
            });
        });
    }
}

// emit(t, sum_{q<Q} in[q] exp(DIR 2 pi i t q / T)),  t < T.   (the transpose of the network above)
// emit: callable (integral_constant t, c64); outputs are produced Q at a time.
template <int T, int Q, int DIR, class Emit>
TFNO_HD void dft_prune_in(const c64 *in, Emit &&emit)
{
    constexpr int S = T / Q;
    static_for<0, S>([&](auto t1c) {
        constexpr int t1 = decltype(t1c)::value;
        c64 g[Q], G[Q];
        static_for<0, Q>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            g[q] = mul_tw<T, DIR, t1 * q>(in[q]);
        });
        RegFFT<Q, DIR, 1>::run(g, G);
        static_for<0, Q>([&](auto t2c) {
            constexpr int t2 = decltype(t2c)::value;
            emit(std::integral_constant<int, t1 + S * t2>{}, G[t2]);
        });
    });
}

// Both pruned networks for the bins q = -Q..Q-1 (2 Q | T), slot r < 2 Q holding bin r or, from Q on, r - 2 Q: with the 2 Q-point
// transforms of the decimated input only the twiddle exponents of the upper slots differ.
template <int T, int Q, int DIR, class In>
TFNO_HD void dft_prune_out_sym(In &&in, c64 *out)
{
    constexpr int M = 2 * Q, S = T / M;
    static_for<0, S>([&](auto t1c) {
        constexpr int t1 = decltype(t1c)::value;
        c64 g[M], F[M];
        static_for<0, M>([&](auto t2c) {
            constexpr int t2 = decltype(t2c)::value;
            g[t2] = in(std::integral_constant<int, t1 + S * t2>{});
        });
        RegFFT<M, DIR, 1>::run(g, F);
        static_for<0, M>([&](auto rc) {
            constexpr int r = decltype(rc)::value, q = r < Q ? r : r - M;
            if constexpr (t1 == 0) out[r] = F[r];
            else out[r] = mac_tw<T, DIR, t1 * q>(out[r], F[r]);
        });
    });
}

template <int T, int Q, int DIR, class Emit>
TFNO_HD void dft_prune_in_sym(const c64 *in, Emit &&emit)
{
    constexpr int M = 2 * Q, S = T / M;
    static_for<0, S>([&](auto t1c) {
        constexpr int t1 = decltype(t1c)::value;
        c64 g[M], G[M];
        static_for<0, M>([&](auto rc) {
            constexpr int r = decltype(rc)::value, q = r < Q ? r : r - M;
            g[r] = mul_tw<T, DIR, t1 * q>(in[r]);
        });
        RegFFT<M, DIR, 1>::run(g, G);
        static_for<0, M>([&](auto t2c) {
            constexpr int t2 = decltype(t2c)::value;
            emit(std::integral_constant<int, t1 + S * t2>{}, G[t2]);
        });
    });
}

// Real decimation in time: a[i * STRIDE], i < L, are real -> bins 0..L/2 (the others are their conjugates; bins 0 and L/2 are
// real).  Its last level has radix 2 over pairs (x[i], x[i + L/2]) of the whole transform, so it starts from the sums and
// differences of those: s[i], d[i], i < LT/2, LT the whole length.
template <int L, int STRIDE>
struct RealFFT {
    TFNO_HD static void run(const float *s, const float *d, c64 *z)
    {
        c64 e[L / 4 + 1], o[L / 4 + 1];
        RealFFT<L / 2, 2 * STRIDE>::run(s, d, e);
        RealFFT<L / 2, 2 * STRIDE>::run(s + STRIDE, d + STRIDE, o);
        z[0] = make_float2(e[0].x + o[0].x, 0.f);
        z[L / 2] = make_float2(e[0].x - o[0].x, 0.f);
        static_for<1, L / 4>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            // (both results as sums of their own: the difference as 2 e - lo, two instructions less, doubles its rounding error)
            constexpr int m = k * (32 / L);
            constexpr float c = cos32(m), s1 = sin32(m);
            z[k] = make_float2(fmaf(o[k].y, s1, fmaf(o[k].x, c, e[k].x)), fmaf(-o[k].x, s1, fmaf(o[k].y, c, e[k].y)));
            z[L / 2 - k] = make_float2(fmaf(-o[k].y, s1, fmaf(-o[k].x, c, e[k].x)), -fmaf(o[k].x, s1, fmaf(-o[k].y, c, e[k].y)));
        });
        z[L / 4] = make_float2(e[L / 4].x, -o[L / 4].x);
    }
};
template <int STRIDE>
struct RealFFT<2, STRIDE> {
    TFNO_HD static void run(const float *s, const float *d, c64 *z)
    {
        z[0] = make_float2(s[0], 0.f);
        z[1] = make_float2(d[0], 0.f);
    }
};
// First level of the real 16-point transform (afterwards v is dead and can be refilled), and the rest of it: 70 additions and
// multiply-adds in all, hermitian_dft16 65, RegFFT<16> of complex values 148.
TFNO_HD void real_first_level16(const float *v, float *s, float *d)
{
    static_for<0, 8>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        s[i] = v[i] + v[i + 8];
        d[i] = v[i] - v[i + 8];
    });
}
TFNO_HD void real_dft16(const float *s, const float *d, c64 *z) { RealFFT<16, 1>::run(s, d, z); }

// Mirror image: out[j] = h0 + (-1)^j hn + Re sum_{0 < c < L/2} h[c] exp(2 pi i c j / L), j < L; out[j * STRIDE].
template <int L, int STRIDE>
struct HermitianFFT {
    TFNO_HD static void run(float h0, float hn, const c64 *h, float *out)
    {
        c64 a[L / 4 + 1], b[L / 4 + 1];
        static_for<1, L / 4>([&](auto cc) {
            constexpr int c = decltype(cc)::value;
            const c64 u = h[c], v = h[L / 2 - c];
            a[c] = make_float2(u.x + v.x, u.y - v.y);
            b[c] = mul_tw<L, +1, c>(make_float2(u.x - v.x, u.y + v.y));
        });
        HermitianFFT<L / 2, 2 * STRIDE>::run(h0 + hn, h[L / 4].x, a, out);
        HermitianFFT<L / 2, 2 * STRIDE>::run(h0 - hn, -h[L / 4].y, b, out + STRIDE);
    }
};
template <int STRIDE>
struct HermitianFFT<2, STRIDE> {
    TFNO_HD static void run(float h0, float hn, const c64 *, float *out)
    {
        out[0] = h0 + hn;
        out[STRIDE] = h0 - hn;
    }
};
TFNO_HD void hermitian_dft16(float h0, float h8, const c64 *h, float *out) { HermitianFFT<16, 1>::run(h0, h8, h, out); }

}  // namespace tfno
