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

// Angles of the transforms are 32-bit integers (4 M <= 2^28); with M a power of two (the library's rule)
// q / (2M) is an exact product with 1 / (2M), the same number as the quotient.
template <bool POW2>
__device__ __forceinline__ double node_angle(int q, double two_m) {
    return POW2 ? (double)q * two_m : (double)q / two_m;
}
template <bool POW2>
__device__ __forceinline__ double node_two_m(int M) { return POW2 ? 1.0 / (2.0 * M) : 2.0 * M; }

// Turned (float64 forms, M a power of two): cosines along an arithmetic sequence of angles, an exactly
// reduced sincospi every kTurn terms and between them one plane rotation each from there, by an angle that
// is exactly reduced too.  A cospi per term bound these transforms (M (L + 1) of them).  Error of c_n,
// 4 <= n <= 512, M = 8192 and 16384, against long double sums, as a multiple of that of correctly rounded
// cosines: 1.02, a cospi per term on the device 0.98, a chain of rotations instead of single ones 1.13.
// With other M (a caller's n_quad) the angles are rounded, which the rotations would repeat in every term:
// these keep a cospi per term (TERMS, chosen by the launch).
constexpr int kTurn = 4;
__host__ __device__ inline bool turns_exact(int64_t M) { return (M & (M - 1)) == 0; }

// v of lane U of this lane's group of four.
template <int U>
__device__ __forceinline__ double quad_lane(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, U * 0x55, 0xf, 0xf, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), U * 0x55, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// Sine and cosine of u step (mod 4M) for 0 < u < kTurn: each lane of a group of kTurn takes one of them and
// reads the others' (step is the same in the group, whose lanes are live together).
struct Turns {
    double s[kTurn], c[kTurn];
    __device__ __forceinline__ double turn(double cs, double sn, int u) const { return fma(cs, c[u], -sn * s[u]); }
};
__device__ __forceinline__ Turns turns_of(unsigned step, int M) {
    static_assert(kTurn == 4, "groups of four, 4 step < 2^31");
    const unsigned mod = 4u * M;
    unsigned q = threadIdx.x % kTurn * step;
    if (q >= 2 * mod) q -= 2 * mod;
    if (q >= mod) q -= mod;
    double s, c;
    sincospi(node_angle<true>((int)q, node_two_m<true>(M)), &s, &c);
    Turns t;
    t.s[1] = quad_lane<1>(s), t.c[1] = quad_lane<1>(c);
    t.s[2] = quad_lane<2>(s), t.c[2] = quad_lane<2>(c);
    t.s[3] = quad_lane<3>(s), t.c[3] = quad_lane<3>(c);
    return t;
}

// The transforms' shares of one thread of 256 (DCT-II) or one lane of a group of four (DCT-III).
//
// Nodes j and M-1-j are mirror images, cos(n theta_{M-1-j}) = (-1)^n cos(n theta_j).
__device__ inline double dct2_turned(int n, int M, const double* __restrict__ f) {
    const int half = M / 2;
    const unsigned mod = 4u * M;   // n < 2^12: all products below 2^31
    // q_j = n (2j+1) mod 4M, advanced by 2n*256 a node
    const unsigned step = 512u * n % mod, turn = kTurn * step % mod;
    const double two_m = node_two_m<true>(M);
    unsigned q = n * (2u * threadIdx.x + 1u) % mod;
    const Turns d = turns_of(step, M);
    const double sign = n % 2 ? -1.0 : 1.0;
    double acc = 0.0;
    for (int j0 = threadIdx.x; j0 < half; j0 += 256 * kTurn) {
        double lo[kTurn], hi[kTurn], cs, sn;
#pragma unroll
        for (int u = 0; u < kTurn; ++u) {
            const int j = j0 + 256 * u, jc = j < half ? j : half - 1;
            lo[u] = f[jc];
            hi[u] = f[M - 1 - jc];
        }
        __builtin_amdgcn_sched_barrier(0);   // all loads are in flight during the sincospi
        sincospi(node_angle<true>((int)q, two_m), &sn, &cs);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kTurn; ++u) {
            const double g = j0 + 256 * u < half ? fma(sign, hi[u], lo[u]) : 0.0;
            acc = fma(g, u ? d.turn(cs, sn, u) : cs, acc);
        }
        q += turn;
        if (q >= mod) q -= mod;
    }
    if (M == 1 && threadIdx.x == 0) acc = fma(f[0], node_cos(n, 1), acc);   // the node x = 0
    return acc;
}

// A cospi per term, also for the reduced forms: their block sums are rounded to float32, where a last-digit
// change of c_n moves entries of D by a float32 ulp, so they keep the sums (and the bits) they had.
template <bool POW2>
__device__ __forceinline__ double dct2_terms_sum(int64_t n, int M, const double* __restrict__ f) {
    const int mod = 4 * M, step = (int)((512 * n) % mod);
    const double two_m = node_two_m<POW2>(M);
    int q = (int)((n * (2 * (int64_t)threadIdx.x + 1)) % mod);
    double acc = 0.0;
    for (int j = threadIdx.x; j < M; j += 256) {
        acc += f[j] * cospi(node_angle<POW2>(q, two_m));
        q += step;
        if (q >= mod) q -= mod;
    }
    return acc;
}
template <bool TERMS>
__device__ inline double dct2(int64_t n, int64_t M, const double* __restrict__ f) {
    if constexpr (!TERMS) return dct2_turned((int)n, (int)M, f);
    return turns_exact(M) ? dct2_terms_sum<true>(n, (int)M, f) : dct2_terms_sum<false>(n, (int)M, f);
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
    const double two_m = node_two_m<POW2>(M);
    int q = (int)((s * q1) % mod);   // n q1 mod 4M for n = s
    double acc = 0.0;
    for (int nn = s; nn <= order; nn += kDctSplit) {
        acc += nn == 0 ? st[0] : 2.0 * st[nn] * cospi(node_angle<POW2>(q, two_m));
        q += step;
        if (q >= mod) q -= mod;
    }
    return acc;
}

// The same with turned angles; st is zero up to a whole turn.
__device__ __forceinline__ double dct3_turned_sum(const double* st, int order, int s, int64_t q1, int M) {
    static_assert(kDctSplit == kTurn, "a node's lanes share its turns");
    const unsigned mod = 4u * M;   // q1 < 2^27: all products below 2^31
    const unsigned step = kDctSplit * (unsigned)q1 % mod, turn = kTurn * step % mod;
    const double two_m = node_two_m<true>(M);
    const Turns d = turns_of(step, M);
    unsigned q = s * (unsigned)q1 % mod;   // n q1 mod 4M for n = s
    double acc = 0.0;
    for (int nn = s; nn <= order; nn += kDctSplit * kTurn) {
        double cs, sn;
        sincospi(node_angle<true>((int)q, two_m), &sn, &cs);
        acc = fma(st[nn], cs, acc);
#pragma unroll
        for (int u = 1; u < kTurn; ++u) acc = fma(st[nn + kDctSplit * u], d.turn(cs, sn, u), acc);
        q += turn;
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
            if (turns_exact(M)) {
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
        double acc = 0.0;
        if (live) acc = dct3_turned_sum(st, order, s, q1, (int)M);
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
