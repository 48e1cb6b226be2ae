// Tight spectral bounds by a few Lanczos steps (an alternative to Gershgorin's
// discs for the extreme eigenvalues e_a, e_b of Sec. II.B, which the paper
// asks for without naming a method).
//
// Start vector: SplitMix64 (Steele, Lea, Flood 2014) doubles in [-1, 1),
// normalised.  Step j (0-based), with one full reorthogonalisation pass:
//     w = H v_j;  alpha_j = v_j . w;  w -= alpha_j v_j + beta_{j-1} v_{j-1};
//     w -= sum_{i<=j} (v_i . w) v_i;   beta_j = ||w||;   v_{j+1} = w / beta_j.
// The recurrence ends after `steps` steps or when beta_j falls to 1e-12 times
// the Gershgorin scale max(|g_lo|, |g_hi|) (an invariant subspace).  The bounds
// are [theta_min - r, theta_max + r] with theta the extreme eigenvalues of the
// tridiagonal T_k and r = beta_{k-1}, widened by margin * width on each side
// and intersected with the Gershgorin interval already in the scalars (the
// Gershgorin interval alone if the intersection is empty).
//
// Two kernels per step.  k_lz_step: z_j = H v_j (one wavefront per two rows, H read once along rows)
// and partials of alpha_j = v_j . z_j.  k_lz_update: w = z_j - alpha_j v_j - beta_{j-1} v_{j-1}
// - sum_i c_i v_i with the reorthogonalisation coefficients
//     c_i = v_i . (z_j - alpha_j v_j - beta_{j-1} v_{j-1}) = z_i . v_j - alpha_j g_i - beta_{j-1} g'_i
// (v_i . H v_j = z_i . v_j; g_i = v_i . v_j, g' the previous step's), and the partials of ||w||^2,
// v_i . w and z_i . w that the next step's coefficients come from.  The measured g_i, not 0 and 1,
// keep it the stated pass: with one classical Gram-Schmidt pass on z_j itself a loss of
// orthogonality E would grow by about (|alpha| + |beta|) / beta a step.
//
// What bounds a step (N = 2000): two launches of 1.6 us and chains of loads that miss L2 (other
// XCDs wrote the data), and per-CU bandwidth where few work-groups read much, so loads go out
// at the top of a kernel and slices are 64 elements.  40 steps at N = 2000: 1050 us with three
// kernels a step and 1024-element slices, 692 us with its two read-backs now (8.7 + 7.3 a step).  Every reduction is a fixed-order sum of
// per-block partials, so the result does not depend on scheduling.  The tridiagonal extremes come
// from Sturm-sequence multisection (Barth, Martin, Wilkinson 1967) in one work-group.
//
// The same kernels serve one problem and a batch of problems of different n
// (the batched form): blockIdx.y selects the problem, whose workspace, scalars and step count min(steps, n) are its own.
#include <cmath>

#include "internal.h"
#include "reduce.h"

namespace chebdm {

namespace {

constexpr int kNT = 256;
constexpr int kSlice = 64;         // vector elements per work-group of the update: a wavefront's lanes
constexpr int kUpdateNT = 1024;    // wavefront u takes the basis vectors i = u mod 16

constexpr int kRowsPerWave = 2;
constexpr int kRows = (kNT / 64) * kRowsPerWave;   // rows of H of a k_lz_step work-group
constexpr double kBreakdown = 1e-12;

__host__ __device__ inline int64_t blocks_of(int64_t n, int64_t per) { return (n + per - 1) / per; }

// One problem of a run: its matrix, size, scalars, workspace views and step count.
struct LzProblem {
    const double* H;
    int64_t n, ldh;
    DevScalars* s;
    LanczosWork L;
    int k, nbv, nbr;
};

__device__ inline LzProblem problem_of(const LanczosRun& r, int p) {
    LzProblem q;
    if (r.tab) {
        q.H = r.tab[p].H;
        q.ldh = r.tab[p].ldh;
        q.n = r.geo[p].n;
    } else {
        q.H = r.H;
        q.ldh = r.ldh;
        q.n = r.n;
    }
    q.s = r.s + p;
    q.k = (int)(q.n < r.steps ? q.n : r.steps);
    q.L = lanczos_layout(r.base + (int64_t)p * r.stride, q.n, q.k);
    q.nbv = (int)blocks_of(q.n, kSlice);
    q.nbr = (int)blocks_of(q.n, kRows);
    return q;
}

__device__ inline uint64_t splitmix64_at(uint64_t seed, uint64_t i) {
    uint64_t z = seed + (i + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Sum over a wavefront in every lane: DPP rotations inside the rows of 16, then across the rows.
template <int N>
__device__ __forceinline__ double row_ror(double x) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, 0x120 + N, 0xf, 0xf, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), 0x120 + N, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ double row_wave_sum(double x) {
    x += row_ror<8>(x);
    x += row_ror<4>(x);
    x += row_ror<2>(x);
    x += row_ror<1>(x);
    x += __shfl_xor(x, 16, 64);
    return x + __shfl_xor(x, 32, 64);
}

__global__ void __launch_bounds__(kSlice) k_lz_init(const LanczosRun r) {
    const LzProblem q = problem_of(r, blockIdx.y);
    if ((int)blockIdx.x >= q.nbv) return;
    const int64_t e = (int64_t)blockIdx.x * kSlice + threadIdx.x;
    double u = 0.0;
    if (e < q.n) {
        const uint64_t z = splitmix64_at(r.seed, (uint64_t)e);
        u = 2.0 * ((double)(z >> 11) * 0x1.0p-53) - 1.0;
        q.L.w[e] = u;
    }
    const double acc = row_wave_sum(u * u);
    if (threadIdx.x == 0) q.L.pn[blockIdx.x] = acc;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        q.L.state[0] = 0;   // steps done at a breakdown (0: none)
        q.L.state[1] = 0;   // steps done in total
    }
}

// beta_{j-1} = ||w||; v_j = w / beta; z_j = H v_j; partial v_j . z_j of the block's rows.  Whole
// chunks of unconditional loads at clamped addresses: the remainder iterations of an unrolled loop
// are waited for one by one.
__global__ void __launch_bounds__(kNT) k_lz_step(const LanczosRun r, int j) {
    __shared__ double part[kNT / 64];
    const LzProblem q = problem_of(r, blockIdx.y);
    if (j >= q.k || (int)blockIdx.x >= q.nbr) return;
    const int n = (int)q.n;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int r0 = blockIdx.x * kRows + wave * kRowsPerWave;
    const double* __restrict__ w = q.L.w;
    const int row = r0 + lane;
    const double wr = w[row < n ? row : n - 1];
    const double pn = q.L.pn[lane < q.nbv ? lane : 0];
    const int broken = q.L.state[0];
    const double* h0 = q.H + (int64_t)(r0 < n ? r0 : n - 1) * q.ldh;
    const double* h1 = q.H + (int64_t)(r0 + 1 < n ? r0 + 1 : n - 1) * q.ldh;
    double y0 = 0.0, y1 = 0.0;
    constexpr int U = 16;
#pragma unroll 1
    for (int c0 = lane; c0 < n; c0 += 64 * U) {
        double x[U], a[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = c0 + 64 * u, cc = c < n ? c : n - 1;
            x[u] = w[cc];
            a[u] = h0[cc];
            b[u] = h1[cc];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double xu = c0 + 64 * u < n ? x[u] : 0.0;
            y0 = fma(a[u], xu, y0);
            y1 = fma(b[u], xu, y1);
        }
    }
    if (broken) return;
    double acc = lane < q.nbv ? pn : 0.0;
    for (int b = lane + 64; b < q.nbv; b += 64) acc += q.L.pn[b];
    const double bt = sqrt(row_wave_sum(acc));
    if (j > 0) {
        const double scale = fmax(fabs(q.s->emin), fabs(q.s->emax));
        const bool broke = !(bt > kBreakdown * scale);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            q.L.beta[j - 1] = bt;
            if (broke) q.L.state[0] = j;
        }
        if (broke) return;
    }
    y0 = row_wave_sum(y0);
    y1 = row_wave_sum(y1);
    double vz = 0.0;
    if (lane < kRowsPerWave && row < n) {
        const double v = wr / bt, z = (lane == 0 ? y0 : y1) / bt;
        q.L.V[(int64_t)j * n + row] = v;
        q.L.Z[(int64_t)j * n + row] = z;
        vz = v * z;
    }
    vz += __shfl_xor(vz, 1, 64);
    if (lane == 0) part[wave] = vz;
    __syncthreads();
    if (threadIdx.x == 0) q.L.pa[blockIdx.x] = (part[0] + part[1]) + (part[2] + part[3]);
}

// w on a slice, and its partial norm, v_i . w and z_i . w.  Wavefront u holds the elements of v_i and
// z_i for i = u, u + 16, .. (the first PRE of them in registers throughout).
__global__ void __launch_bounds__(kUpdateNT) k_lz_update(const LanczosRun r, int j) {
    constexpr int W = kUpdateNT / 64, PRE = 3;
    __shared__ double p[kMaxLanczosSteps], g[kMaxLanczosSteps];
    __shared__ double sums[W][kSlice];
    __shared__ double alpha;
    const LzProblem q = problem_of(r, blockIdx.y);
    if (j >= q.k || (int)blockIdx.x >= q.nbv) return;
    const int n = (int)q.n, nbv = q.nbv;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int e = blockIdx.x * kSlice + lane, ec = e < n ? e : n - 1;
    const double* pvr = q.L.pv + (int64_t)(~j & 1) * q.k * nbv;
    const double* pzr = q.L.pz + (int64_t)(~j & 1) * q.k * nbv;
    double* pvw = q.L.pv + (int64_t)(j & 1) * q.k * nbv;
    double* pzw = q.L.pz + (int64_t)(j & 1) * q.k * nbv;
    const double* gm = q.L.g + (~j & 1) * q.k;   // g of the step before; this step's go to the other half
    const int broken = q.L.state[0];
    const double bm = j > 0 ? q.L.beta[j - 1] : 1.0;
    double v[PRE], z[PRE], pv[PRE], pz[PRE];
#pragma unroll
    for (int t = 0; t < PRE; ++t) {
        const int i = wave + W * t, ic = i < j ? i : j;
        v[t] = q.L.V[(int64_t)ic * n + ec];
        z[t] = q.L.Z[(int64_t)ic * n + ec];
        pv[t] = pvr[(int64_t)ic * nbv + (lane < nbv ? lane : 0)];
        pz[t] = pzr[(int64_t)ic * nbv + (lane < nbv ? lane : 0)];
    }
    const double zj = q.L.Z[(int64_t)j * n + ec], vj = q.L.V[(int64_t)j * n + ec];
    const double vm = q.L.V[(int64_t)(j > 0 ? j - 1 : 0) * n + ec];
    const double gmi = gm[(int)threadIdx.x < j ? threadIdx.x : 0];
    if (wave == W - 1) {
        double a = 0.0;
#pragma unroll 4
        for (int b = lane; b < q.nbr; b += 64) a += q.L.pa[b];
        a = row_wave_sum(a);
        if (lane == 0) alpha = a;
    }
    if (broken) return;
    // z_i . v_j and v_i . v_j, i < j, from the partials with w = beta v_j
#pragma unroll
    for (int t = 0; t < PRE; ++t) {
        const int i = wave + W * t;
        if (i < j) {
            double a = lane < nbv ? pv[t] : 0.0, b = lane < nbv ? pz[t] : 0.0;
            for (int c = lane + 64; c < nbv; c += 64) {
                a += pvr[(int64_t)i * nbv + c];
                b += pzr[(int64_t)i * nbv + c];
            }
            a = row_wave_sum(a);
            b = row_wave_sum(b);
            if (lane == 0) {
                g[i] = a / bm;
                p[i] = b / bm;
            }
        }
    }
#pragma unroll 1
    for (int i = wave + W * PRE; i < j; i += W) {
        double a = 0.0, b = 0.0;
        for (int c = lane; c < nbv; c += 64) {
            a += pvr[(int64_t)i * nbv + c];
            b += pzr[(int64_t)i * nbv + c];
        }
        a = row_wave_sum(a);
        b = row_wave_sum(b);
        if (lane == 0) {
            g[i] = a / bm;
            p[i] = b / bm;
        }
    }
    __syncthreads();
    const double al = alpha;
    double c = 0.0;
    if ((int)threadIdx.x <= j) {
        const int i = threadIdx.x;
        // v_j . v_j = 1 by beta's definition; v_{j-1} . v_{j-1} likewise
        if (i < j) c = fma(-bm, i == j - 1 ? 1.0 : gmi, fma(-al, g[i], p[i]));
        else if (j > 0) c = -bm * g[j - 1];
        if (blockIdx.x == 0) {
            if (i < j) q.L.g[(j & 1) * q.k + i] = g[i];
            else q.L.alpha[j] = al;
        }
    }
    __syncthreads();
    if ((int)threadIdx.x <= j) p[threadIdx.x] = c;
    __syncthreads();
    double acc = 0.0;
#pragma unroll
    for (int t = 0; t < PRE; ++t) {
        const int i = wave + W * t;
        acc = fma(i <= j ? p[i] : 0.0, v[t], acc);
    }
#pragma unroll 1
    for (int i = wave + W * PRE; i <= j; i += W) acc = fma(p[i], q.L.V[(int64_t)i * n + ec], acc);
    sums[wave][lane] = acc;
    __syncthreads();
    double x = zj - al * vj;
    if (j > 0) x -= bm * vm;
    double corr = 0.0;
#pragma unroll
    for (int u = 0; u < W; ++u) corr += sums[u][lane];
    x -= corr;
    if (e >= n) x = 0.0;
    if (wave == 0) {
        if (e < n) q.L.w[e] = x;
        const double s = row_wave_sum(x * x);
        if (lane == 0) q.L.pn[blockIdx.x] = s;
    }
#pragma unroll
    for (int t = 0; t < PRE; ++t) {
        const int i = wave + W * t;
        if (i <= j) {
            const double a = row_wave_sum(v[t] * x), b = row_wave_sum(z[t] * x);
            if (lane == 0) {
                pvw[(int64_t)i * nbv + blockIdx.x] = a;
                pzw[(int64_t)i * nbv + blockIdx.x] = b;
            }
        }
    }
#pragma unroll 1
    for (int i = wave + W * PRE; i <= j; i += W) {
        const double a = row_wave_sum(q.L.V[(int64_t)i * n + ec] * x), b = row_wave_sum(q.L.Z[(int64_t)i * n + ec] * x);
        if (lane == 0) {
            pvw[(int64_t)i * nbv + blockIdx.x] = a;
            pzw[(int64_t)i * nbv + blockIdx.x] = b;
        }
    }
}

// Number of eigenvalues below x of the tridiagonal with diagonal a and squared off-diagonal b2 (b2[i]
// couples i and i - 1; b2[0] = 0), scaled so that |a|, |x| <= 1 and b2 <= 1: sign changes along
// p_i = (a_i - x) p_{i-1} - b2_i p_{i-2}, a zero counting as the sign opposite to its
// predecessor's.  No division in the serial chain.  Both arrays are padded to a multiple of eight
// with a = 2, b2 = 0, which changes no sign.  A step grows p at most threefold and shrinks it by
// no more than min(b2) >= 1e-24, so rescaling every eight steps keeps it inside the float64 range.
__device__ __forceinline__ int sturm_count(const double* a, const double* b2, int k, double x) {
    int cnt = 0;
    double p0 = 0.0, p1 = 1.0;
#pragma unroll 1
    for (int i = 0; i < k; i += 8) {
        double d[8], o[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            d[u] = a[i + u] - x;
            o[u] = b2[i + u];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            double p2 = fma(d[u], p1, -o[u] * p0);
            if (p2 == 0.0) p2 = p1 < 0.0 ? 1e-290 : -1e-290;
            cnt += (p2 < 0.0) != (p1 < 0.0);
            p0 = p1;
            p1 = p2;
        }
        const int e = -__builtin_amdgcn_frexp_exp(fmax(fabs(p0), fabs(p1)));
        p0 = ldexp(p0, e);
        p1 = ldexp(p1, e);
    }
    return cnt;
}

// The first half of the threads looks for theta_min, the second for theta_max, 257 ways a round
// (257^8 > 2^64).
constexpr int kFinalNT = 512;
constexpr int kWays = kFinalNT / 2 + 1;
constexpr int kRounds = 8;

__global__ void __launch_bounds__(kFinalNT) k_lz_final(const LanczosRun r) {
    __shared__ __attribute__((aligned(16))) double a[kMaxLanczosSteps + 8], b[kMaxLanczosSteps], b2[kMaxLanczosSteps + 8];
    __shared__ double theta[2];
    __shared__ int below[2][kFinalNT / 64];
    __shared__ double r_last;
    const LzProblem q = problem_of(r, blockIdx.y);
    const int done = q.L.state[0];
    const int k = done ? done : q.k;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (wave == 0) {
        double acc = 0.0;
        for (int c = lane; c < q.nbv; c += 64) acc += q.L.pn[c];
        acc = wave_sum(acc);
        if (lane == 0) {
            r_last = done ? q.L.beta[k - 1] : sqrt(acc);
            if (!done) q.L.beta[k - 1] = r_last;
            q.L.state[1] = k;
        }
    }
    for (int i = threadIdx.x; i < k; i += kFinalNT) {
        a[i] = q.L.alpha[i];
        b[i] = i + 1 < k ? q.L.beta[i] : 0.0;
    }
    __syncthreads();
    // Gershgorin interval of T, and T scaled by a power of two into [-1, 1]
    double lo = INFINITY, hi = -INFINITY;
    for (int i = lane; i < k; i += 64) {
        const double rad = fabs(b[i]) + (i > 0 ? fabs(b[i - 1]) : 0.0);
        lo = fmin(lo, a[i] - rad);
        hi = fmax(hi, a[i] + rad);
    }
    lo = wave_min(lo);
    hi = wave_max(hi);
    const double top = fmax(fabs(lo), fabs(hi));
    const int ex = top > 0.0 && top <= 1.7976931348623157e308 ? __builtin_amdgcn_frexp_exp(top) : 0;
    lo = ldexp(lo, -ex);
    hi = ldexp(hi, -ex);
    __syncthreads();
    if ((int)threadIdx.x < k + 8) {   // k <= 128 < kFinalNT
        const int i = threadIdx.x;
        a[i] = i < k ? ldexp(a[i], -ex) : 2.0;
        const double bi = i > 0 && i < k ? ldexp(b[i - 1], -ex) : 0.0;
        b2[i] = bi * bi;
    }
    __syncthreads();
    // first half: smallest x with count(x) >= 1 (theta_min in [lo, hi]); second: count(x) >= k
    const int half = threadIdx.x / (kFinalNT / 2), idx = threadIdx.x % (kFinalNT / 2);
    const int need = half == 0 ? 1 : k;
#pragma unroll 1
    for (int round = 0; round < kRounds; ++round) {
        const double x = lo + (hi - lo) * ((double)(idx + 1) * (1.0 / kWays));
        const uint64_t under = __ballot(sturm_count(a, b2, k, x) < need);
        if (lane == 0) below[round & 1][wave] = __popcll(under);
        __syncthreads();
        int first = 0;   // points still below: the end lies between points first - 1 and first
#pragma unroll
        for (int w = 0; w < kFinalNT / 128; ++w) first += below[round & 1][half * (kFinalNT / 128) + w];
        const double xl = first == 0 ? lo : lo + (hi - lo) * ((double)first * (1.0 / kWays));
        const double xh = first == kWays - 1 ? hi : lo + (hi - lo) * ((double)(first + 1) * (1.0 / kWays));
        lo = xl;
        hi = xh;
    }
    if (idx == 0) theta[half] = ldexp(half == 0 ? lo : hi, ex);   // outer side of the final interval
    __syncthreads();
    if (threadIdx.x == 0) {
        const double g_lo = q.s->emin, g_hi = q.s->emax;
        double e_lo = theta[0] - r_last, e_hi = theta[1] + r_last;
        const double pad = r.margin * (e_hi - e_lo);
        e_lo = fmax(e_lo - pad, g_lo);
        e_hi = fmin(e_hi + pad, g_hi);
        if (!(e_lo <= e_hi)) {
            e_lo = g_lo;
            e_hi = g_hi;
        }
        q.s->emin = e_lo;
        q.s->emax = e_hi;
    }
}

}  // namespace

int64_t lanczos_work_doubles(int64_t n, int steps) {
    const int64_t nbv = blocks_of(n, kSlice), nbr = blocks_of(n, kRows);
    return 2 * (int64_t)steps * n + n + nbr + 2 * 2 * (int64_t)steps * nbv + nbv + 4 * (int64_t)steps + 1;
}

// pv and pz are read and rewritten by different work-groups of one update: two halves in turn
__host__ __device__ LanczosWork lanczos_layout(double* base, int64_t n, int steps) {
    const int64_t nbv = blocks_of(n, kSlice), nbr = blocks_of(n, kRows);
    LanczosWork L;
    double* p = base;
    L.V = p;
    p += (int64_t)steps * n;
    L.Z = p;
    p += (int64_t)steps * n;
    L.w = p;
    p += n;
    L.pa = p;
    p += nbr;
    L.pv = p;
    p += 2 * (int64_t)steps * nbv;
    L.pz = p;
    p += 2 * (int64_t)steps * nbv;
    L.pn = p;
    p += nbv;
    L.g = p;
    p += 2 * (int64_t)steps;
    L.alpha = p;
    p += steps;
    L.beta = p;
    p += steps;
    L.state = reinterpret_cast<int32_t*>(p);   // two int32 in one double
    return L;
}

hipError_t launch_lanczos_run(const LanczosRun& r, int count, hipStream_t st) {
    if (r.steps < 1 || r.steps > kMaxLanczosSteps || count < 1 || count > 65535 || r.nmax < 1) return hipErrorInvalidValue;
    if (r.stride < lanczos_work_doubles(r.nmax, r.steps)) return hipErrorInvalidValue;
    const int nbv = (int)blocks_of(r.nmax, kSlice), nbr = (int)blocks_of(r.nmax, kRows);
    const int steps = (int)(r.nmax < r.steps ? r.nmax : r.steps);
    hipLaunchKernelGGL(k_lz_init, dim3(nbv, count), dim3(kSlice), 0, st, r);
    for (int j = 0; j < steps; ++j) {
        hipLaunchKernelGGL(k_lz_step, dim3(nbr, count), dim3(kNT), 0, st, r, j);
        hipLaunchKernelGGL(k_lz_update, dim3(nbv, count), dim3(kUpdateNT), 0, st, r, j);
    }
    hipLaunchKernelGGL(k_lz_final, dim3(1, count), dim3(kFinalNT), 0, st, r);
    return hipGetLastError();
}

hipError_t launch_lanczos(const double* H, int64_t n, int64_t ldh, int steps, double margin, uint64_t seed,
                          double* work, DevScalars* s, hipStream_t st) {
    if (steps < 1 || steps > kMaxLanczosSteps || steps > n) return hipErrorInvalidValue;
    LanczosRun r{};
    r.H = H;
    r.n = n;
    r.ldh = ldh;
    r.s = s;
    r.base = work;
    r.stride = lanczos_work_doubles(n, steps);
    r.nmax = n;
    r.steps = steps;
    r.margin = margin;
    r.seed = seed;
    return launch_lanczos_run(r, 1, st);
}

}  // namespace chebdm
