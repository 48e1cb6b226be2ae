// Scalar device helpers of the coefficient, moment and bisection kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

namespace chebdm {

// cos(pi q / (2M)) for the Chebyshev-Gauss angles theta_j = pi (j + 1/2) / M:
// q / (2M) is exact because 2M is a power of two, so every cosine is a
// correctly reduced cospi (q = n (2j+1) mod 4M is formed in integers).
__device__ inline double node_cos(int64_t q, int64_t M) { return cospi((double)q / (double)(2 * M)); }

// 1 / (1 + exp(beta'(x - mu~)))  (eq. "fermifunc" in scaled variables)
__device__ inline double fermi_scaled(double x, double beta_s, double mu_s) {
    return 1.0 / (1.0 + exp(beta_s * (x - mu_s)));
}

// Jackson damping factor g_n of a series of N = order + 1 terms (kernel polynomial method):
// g_n = [(N - n + 1) cos(pi n/(N+1)) + sin(pi n/(N+1)) cot(pi/(N+1))] / (N + 1); 1 if damping == 0.
__device__ inline double damping_factor(int damping, int n, int order) {
    if (damping == 0) return 1.0;
    const double N1 = (double)order + 2.0;   // N + 1
    const double u = (double)n / N1;
    return (((double)order + 2.0 - n) * cospi(u) + sinpi(u) * cospi(1.0 / N1) / sinpi(1.0 / N1)) / N1;
}

// Cosines along an arithmetic sequence of angles: an exactly reduced sincospi every kTurn terms and
// plane rotations between, within kTurn ulp of 1.  A cospi per term bound these transforms
// (M (L + 1) of them).  c_n against long double sums, order 512, M = 16384: at most 2.2e-17 off, 3.9e-18
// rms (with a cospi per term 1.9e-17 and 3.3e-18, with eight terms a turn 2.5e-17 and 4.8e-18 for
// 1 us less).
constexpr int kTurn = 4;

__device__ __forceinline__ void node_sincos(int64_t q, int64_t M, double& s, double& c) {
    sincospi((double)q / (double)(2 * M), &s, &c);
}


// The transforms' shares of one thread of 256 (DCT-II) or one lane of a group of four (DCT-III).
//
// Turned: nodes j and M-1-j are mirror images, cos(n theta_{M-1-j}) = (-1)^n cos(n theta_j).
__device__ inline double dct2_turned(int64_t n, int64_t M, const double* __restrict__ f) {
    const int64_t mod = 4 * M, half = M / 2;
    // q_j = n (2j+1) mod 4M, advanced by 2n*256 per stride without a 64-bit divide
    const int64_t step = (512 * n) % mod, turn = (kTurn * step) % mod;
    int64_t q = (n * (2 * (int64_t)threadIdx.x + 1)) % mod;
    double ds, dc;
    node_sincos(step, M, ds, dc);
    const double sign = n % 2 ? -1.0 : 1.0;
    double acc = 0.0;
    for (int64_t j0 = threadIdx.x; j0 < half; j0 += 256 * kTurn) {
        double g[kTurn], cs, sn;
#pragma unroll
        for (int u = 0; u < kTurn; ++u) {
            const int64_t j = j0 + 256 * u, jc = j < half ? j : half - 1;
            const double v = fma(sign, f[M - 1 - jc], f[jc]);
            g[u] = j < half ? v : 0.0;
        }
        node_sincos(q, M, sn, cs);
#pragma unroll
        for (int u = 0; u < kTurn; ++u) {
            acc = fma(g[u], cs, acc);
            const double t = fma(cs, dc, -sn * ds);
            sn = fma(sn, dc, cs * ds);
            cs = t;
        }
        q += turn;
        if (q >= mod) q -= mod;
    }
    if (M % 2 && threadIdx.x == 0) acc = fma(f[half], node_cos((n * M) % mod, M), acc);   // the node x = 0
    return acc;
}

// A cospi per term, for the reduced forms: their block sums are rounded to float32, where a last-digit
// change of c_n moves entries of D by a float32 ulp, so they keep the sums (and the bits) they had.
// The angles are 32-bit integers (4 M <= 2^28); with M a power of two (the library's rule) q / (2M) is an
// exact product with 1 / (2M), the same number as the quotient.
template <bool POW2>
__device__ __forceinline__ double node_cos32(int q, double two_m) {
    return POW2 ? cospi((double)q * two_m) : cospi((double)q / two_m);
}
template <bool POW2>
__device__ __forceinline__ double dct2_terms_sum(int64_t n, int M, const double* __restrict__ f) {
    const int mod = 4 * M, step = (int)((512 * n) % mod);
    const double two_m = POW2 ? 1.0 / (2.0 * M) : 2.0 * M;
    int q = (int)((n * (2 * (int64_t)threadIdx.x + 1)) % mod);
    double acc = 0.0;
    for (int j = threadIdx.x; j < M; j += 256) {
        acc += f[j] * node_cos32<POW2>(q, two_m);
        q += step;
        if (q >= mod) q -= mod;
    }
    return acc;
}
__device__ inline double dct2_terms(int64_t n, int64_t M, const double* __restrict__ f) {
    return (M & (M - 1)) == 0 ? dct2_terms_sum<true>(n, (int)M, f) : dct2_terms_sum<false>(n, (int)M, f);
}

// DCT-III: kDctSplit neighbouring lanes share a pair of nodes, lane s summing n = s, s + kDctSplit, ...;
// the even n of the mirrored node add up, the odd ones change sign.
constexpr int kDctSplit = 4;
__host__ __device__ inline int dct3_padded(int order) { return (order / (kDctSplit * kTurn) + 1) * kDctSplit * kTurn; }

// The moments into LDS: (2 - delta_{n0}) tau_n, zero up to a whole turn of every lane; tau_n for TERMS.
// With damping, t(mu~) = sum_n g_n c_n(mu~) tau_n: the factors go onto the moments.
template <bool TERMS>
__device__ inline void dct3_stage(const double* __restrict__ tau, int order, int damping, double* st) {
    for (int i = threadIdx.x; i < dct3_padded(order); i += 256) {
        const double v = i <= order ? tau[i] * damping_factor(damping, i, order) : 0.0;
        st[i] = !TERMS && i > 0 ? 2.0 * v : v;
    }
}

// One node's lane sum with a cospi per term.
template <bool POW2>
__device__ __forceinline__ double dct3_terms_sum(const double* st, int order, int s, int64_t q1, int M) {
    const int mod = 4 * M, step = (int)((kDctSplit * q1) % mod);
    const double two_m = POW2 ? 1.0 / (2.0 * M) : 2.0 * M;
    int q = (int)((s * q1) % mod);   // n q1 mod 4M for n = s
    double acc = 0.0;
    for (int nn = s; nn <= order; nn += kDctSplit) {
        acc += nn == 0 ? st[0] : 2.0 * st[nn] * node_cos32<POW2>(q, two_m);
        q += step;
        if (q >= mod) q -= mod;
    }
    return acc;
}

// w and x at the nodes j and M-1-j; every lane of the work-group calls it (shuffles).
template <bool TERMS>
__device__ inline void dct3_pair(const double* st, int order, int64_t M, int64_t j, double* __restrict__ w,
                                 double* __restrict__ x_tab) {
    static_assert(kDctSplit == 4, "two shuffle steps");
    const int s = threadIdx.x % kDctSplit;
    const bool live = j < (M + 1) / 2;
    const int64_t jm = M - 1 - j, q1 = 2 * j + 1;
    if constexpr (TERMS) {   // mirrored cosines are the same numbers with M a power of two
        double a = 0.0, b = 0.0;
        if (live) {
            if ((M & (M - 1)) == 0) {
                a = dct3_terms_sum<true>(st, order, s, q1, (int)M);
                b = s % 2 ? -a : a;
            } else {
                a = dct3_terms_sum<false>(st, order, s, q1, (int)M);
                b = dct3_terms_sum<false>(st, order, s, 2 * jm + 1, (int)M);
            }
        }
        a += __shfl_xor(a, 1, 64);
        b += __shfl_xor(b, 1, 64);
        a += __shfl_xor(a, 2, 64);
        b += __shfl_xor(b, 2, 64);
        if (live && s == 0) {
            w[j] = a;
            x_tab[j] = node_cos(q1, M);
            if (jm != j) {
                w[jm] = b;
                x_tab[jm] = node_cos(2 * jm + 1, M);
            }
        }
    } else {
        const int64_t mod = 4 * M, step = (kDctSplit * q1) % mod, turn = (kTurn * step) % mod;
        double acc = 0.0;
        if (live) {
            double ds, dc;
            node_sincos(step, M, ds, dc);
            int64_t q = (s * q1) % mod;   // n q1 mod 4M for n = s
            for (int nn = s; nn <= order; nn += kDctSplit * kTurn) {
                double cs, sn;
                node_sincos(q, M, sn, cs);
#pragma unroll
                for (int u = 0; u < kTurn; ++u) {
                    acc = fma(st[nn + kDctSplit * u], cs, acc);
                    const double t = fma(cs, dc, -sn * ds);
                    sn = fma(sn, dc, cs * ds);
                    cs = t;
                }
                q += turn;
                if (q >= mod) q -= mod;
            }
        }
        acc += __shfl_xor(acc, 2, 64);                   // lanes 0, 2: the even n; lanes 1, 3: the odd ones
        const double other = __shfl_xor(acc, 1, 64);
        if (live && s == 0) {
            const double xj = node_cos(q1, M);
            w[j] = acc + other;
            x_tab[j] = xj;
            if (jm != j) {
                w[jm] = acc - other;
                x_tab[jm] = -xj;
            }
        }
    }
}

// Distance from |v| to the next larger double (|v| = 0 is taken as 1e-300).
__device__ inline double ulp_spacing(double v) {
    const double a = v != 0.0 ? fabs(v) : 1e-300;
    return nextafter(a, INFINITY) - a;
}

// Quadrature size M = 2^ceil(log2 max(2(L+1), L/2 + 7 beta' + 64)); -1 if above 2^29.
__host__ __device__ inline int64_t quad_rule(int order, double beta_s) {
    const double need = fmax(2.0 * (order + 1), 0.5 * order + 7.0 * beta_s + 64.0);
    int64_t m = 1;
    int lg = 0;
    while ((double)m < need) {
        m <<= 1;
        if (++lg > 29) return -1;
    }
    return m;
}

}  // namespace chebdm
