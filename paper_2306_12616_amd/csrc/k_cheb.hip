// Scalar side of the method on the device, all in float64:
//   - Chebyshev coefficients of the Fermi function (expansion sum c_n T_n,
//     Sec. II.B; obtained by a Chebyshev-Gauss projection, i.e. a DCT-II);
//   - block coefficients: the paper's power form d (eqs. "formula for d0",
//     "formula for d", "X": back substitution over row blocks) or the
//     composition form e (same identity 2 T_a T_b = T_{a+b} + T_{|a-b|});
//   - trace moments tau_n from traces and Gram products of Chebyshev matrices;
//   - the chemical-potential bisection on t(mu~) = sum_n c_n(mu~) tau_n,
//     rewritten as (1/M) sum_j f(x_j; mu~) w_j with w the DCT-III of tau.
// Angles are reduced exactly in integers: cos(n theta_j) = cospi(q / 2M)
// with q = n (2j+1) mod 4M, so every cosine is a correctly reduced cospi.
#include <cmath>

#include "cheb_dev.h"
#include "internal.h"
#include "reduce.h"
#include "search_dev.h"

namespace chebdm {

namespace {

// bounds_on_device: take e_a, e_b from s (written there by the Gershgorin kernels) instead of
// the arguments, so that a captured graph does not depend on their values.
__global__ void k_set_scalars(DevScalars* s, double emin, double emax, double beta, double mu,
                              int has_mu, double n_elec, double tol, int max_iter, int bounds_on_device) {
    if (bounds_on_device) {
        emin = s->emin;
        emax = s->emax;
    }
    const double cen = 0.5 * (emin + emax), half = 0.5 * (emax - emin);
    s->emin = emin;
    s->emax = emax;
    s->cen = cen;
    s->half = half;
    s->beta_s = beta * half;
    s->mu_s = has_mu ? (mu - cen) / half : 0.0;
    s->n_elec = n_elec;
    s->tol = tol;
    s->max_iter = max_iter;
    s->status = 0;
    s->iters = 0;
    s->trace = 0.0;
}

__global__ void __launch_bounds__(256)
k_fermi_table(int64_t M, const DevScalars* __restrict__ s, double* __restrict__ f) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= M) return;
    const double x = node_cos(2 * j + 1, M);
    f[j] = fermi_scaled(x, s->beta_s, s->mu_s);
}

// One workgroup per coefficient n: c_n = (2 - delta_{n0})/M sum_j f_j cos(n theta_j).  Order 512,
// M = 16384: 30 us with a cospi per node, 8.6 us with mirrored nodes and turned angles; TERMS (the
// reduced forms) 28 -> 21 us.
template <bool TERMS>
__global__ void __launch_bounds__(256)
k_dct2(int64_t M, const double* __restrict__ f, double* __restrict__ c, int order, int damping) {
    __shared__ double smem[4];
    const int64_t n = blockIdx.x;
    const double acc = block_sum<256>(dct2<TERMS>(n, M, f), smem);
    if (threadIdx.x == 0) c[n] = (n == 0 ? 1.0 : 2.0) * acc / (double)M * damping_factor(damping, (int)n, order);
}

// Two Clenshaw chains for the giant steps: with T_{h+j} = 2 T_h T_j - T_{h-j} (eq. "identity"
// with a = h, b = j), sum_{l<m} T_l(Y) R_l = sum_{l<h} T_l(Y) R''_l + T_h(Y) sum_{j<m-h} T_j(Y) R'_j,
// R'_0 = R_h, R'_j = 2 R_{h+j}, R''_{h-j} = R_{h-j} - R_{h+j} (1 <= j < m - h <= h).  Applied to
// column i of the blocks base .. base + m - 1 in place: block h + j then holds R'_j.
__device__ inline void split_column(double (*d)[kMaxBlocks], int i, int base, int m, int h) {
    for (int j = 1; h + j < m; ++j) {
        const double up = d[base + h + j][i];
        d[base + h - j][i] -= up;
        d[base + h + j][i] = 2.0 * up;
    }
}

// Block coefficients, one workgroup.  Output coef[l*k + i] = weight of T_i in block l.  The
// coefficients are staged in LDS first: the recurrence over l is then a chain of LDS reads.
// split_h, split_q > 0: blocks rearranged for two and four Clenshaw chains.
__global__ void __launch_bounds__(64)
k_block_coeffs(const double* __restrict__ c, int order, int k, int m, int form,
               double* __restrict__ coef, int split_h, int split_q) {
    __shared__ double a[kMaxBlocks][kMaxBlocks];   // a[j][l] of T_k^j = sum_l a_{j,l} T_{lk}
    __shared__ double d[kMaxBlocks][kMaxBlocks];   // d[l][i]: block l, index i (output layout)
    __shared__ double cl[kMaxBlocks * kMaxBlocks];
    const int tid = threadIdx.x;
    for (int i = tid; i < k * m; i += 64) cl[i] = i <= order ? c[i] : 0.0;
    __syncthreads();
    auto cpad = [&](int idx) -> double { return cl[idx]; };

    if (form == CHEBDM_GIANT_COMPOSITION) {
        // e_{l,0} = c_{lk}; e_{l,i} = 2 c_{lk+i} - e_{l+1,k-i} (l >= 1); e_{0,i} = c_i - e_{1,k-i}/2
        for (int l = m - 1; l >= 0; --l) {
            for (int i = tid; i < k; i += blockDim.x) {
                double v;
                if (i == 0) {
                    v = cpad(l * k);
                } else {
                    const double up = (l + 1 < m) ? d[l + 1][k - i] : 0.0;
                    v = (l == 0) ? cpad(i) - 0.5 * up : 2.0 * cpad(l * k + i) - up;
                }
                d[l][i] = v;
            }
            __syncthreads();
        }
    } else {
        // Matrix A by the recurrence of eq. "coeff recursion" (row j from row j-1).
        for (int l = tid; l < m; l += blockDim.x)
            for (int j = 0; j < m; ++j) a[j][l] = 0.0;
        __syncthreads();
        if (tid == 0) {
            a[0][0] = 1.0;
            if (m > 1) a[1][1] = 1.0;
        }
        __syncthreads();
        for (int j = 2; j < m; ++j) {
            for (int l = tid; l <= j; l += blockDim.x) {
                auto prev = [&](int ll) -> double { return (ll >= 0 && ll <= j - 1) ? a[j - 1][ll] : 0.0; };
                double v;
                if (l == 0) v = 0.5 * prev(1);
                else if (l == 1) v = prev(0) + 0.5 * prev(2);
                else if (l < j) v = 0.5 * (prev(l - 1) + prev(l + 1));
                else v = 0.5 * prev(l - 1);
                a[j][l] = v;
            }
            __syncthreads();
        }
        // Back substitution over the row blocks of X, l = m-1 down to 0.  Row
        // (l, i) involves d_{i,j} for j >= l and d_{k-i,j} for j >= l+1 only.
        for (int l = m - 1; l >= 0; --l) {
            for (int i = tid; i < k; i += blockDim.x) {
                double s = cpad(l * k + i);
                double v;
                if (i == 0) {
                    for (int j = l + 1; j < m; ++j) s -= a[j][l] * d[j][0];
                    v = s / a[l][l];
                } else {
                    const double own = (l == 0) ? 1.0 : 0.5;
                    double t = 0.0;
                    for (int j = l + 1; j < m; ++j) t += a[j][l] * d[j][i];
                    s -= own * t;
                    if (l + 1 < m) {
                        double u = 0.0;
                        for (int j = l + 1; j < m; ++j) u += a[j][l + 1] * d[j][k - i];
                        s -= 0.5 * u;
                    }
                    v = s / (own * a[l][l]);
                }
                d[l][i] = v;
            }
            __syncthreads();
        }
    }
    if (tid < k) {   // columns are independent
        if (split_h > 0) split_column(d, tid, 0, m, split_h);
        if (split_q > 0) {
            split_column(d, tid, 0, split_h, split_q);
            split_column(d, tid, split_h, m - split_h, split_q);
        }
    }
    __syncthreads();
    for (int idx = tid; idx < k * m; idx += blockDim.x) coef[idx] = d[idx / k][idx % k];
}

// tau_0 = n, tau_i = tr T_i (i <= k), tau_{lk+i} = 2 <T_{lk}, T_i> - tau_{lk-i}.  The recurrence over l
// runs in LDS (through memory it took 12 us at order 512).
__global__ void __launch_bounds__(256)
k_assemble_moments(const double* __restrict__ tr_baby, const double* __restrict__ gram, int k, int m,
                   int order, int64_t n, double* __restrict__ tau) {
    __shared__ double t[kMaxBlocks * kMaxBlocks + kMaxBlocks + 1];   // tau up to m k
    const int tid = threadIdx.x;
    if (tid == 0) t[0] = (double)n;
    for (int i = 1 + tid; i <= k; i += 256) t[i] = tr_baby[i - 1];
    for (int i = tid; i < (m - 1) * k; i += 256) t[k + 1 + i] = k + 1 + i <= order ? gram[i] : 0.0;   // <T_{lk}, T_i>
    __syncthreads();
    if (tid < 64) {   // one wavefront: its LDS accesses are in order
        for (int l = 1; l < m; ++l) {
            const int i = 1 + tid, idx = l * k + i;
            const double v = i <= k && idx <= order ? 2.0 * t[idx] - t[l * k - i] : 0.0;
            __builtin_amdgcn_wave_barrier();
            if (i <= k) t[idx] = v;
            __builtin_amdgcn_wave_barrier();
        }
    }
    __syncthreads();
    for (int i = tid; i <= order; i += 256) tau[i] = t[i];
}

// w_j = sum_n (2 - delta_{n0}) tau_n cos(n theta_j) at the nodes j and M-1-j; also stores x_j.  Order 512,
// M = 16384: 33 us with a cospi per node and term, 11 us with mirrored nodes and turned angles; TERMS
// 31 -> 28 us.
template <bool TERMS>
__global__ void __launch_bounds__(256)
k_dct3(const double* __restrict__ tau, int order, int64_t M, double* __restrict__ w, double* __restrict__ x_tab,
       int damping) {
    extern __shared__ double st[];
    dct3_stage<TERMS>(tau, order, damping, st);
    __syncthreads();
    dct3_pair<TERMS>(st, order, M, ((int64_t)blockIdx.x * 256 + threadIdx.x) / kDctSplit, w, x_tab);
}

constexpr int kBisectThreads = 1024;
// Bisection steps per multi-point pass of one work-group (seven points side by side, two wavefronts
// each), for the steps that the launches below leave over.
constexpr int kBisectLevels = 3;

// The search of one problem by one work-group (mode 1, safeguarded Newton); scratch: M doubles for
// the tail sums
__global__ void __launch_bounds__(kBisectThreads)
k_search_newton(const double* __restrict__ w, const double* __restrict__ x, int64_t M, DevScalars* s,
                double* __restrict__ scratch) {
    constexpr int NP = (1 << kBisectLevels) - 1;
    __shared__ double smem[kBisectThreads / 64];
    __shared__ double part[kBisectThreads / 64];
    __shared__ double win[4 * NP];
    __shared__ double tout[NP];
    mu_search_one<kBisectThreads, kBisectLevels>(M, w, x, *s, 1, 0.0, 0.0, smem, scratch, part, win, tout);
}

// Bisection (mode 0) over the whole chip.  The midpoints that the next kTreeLevels steps can visit
// form a tree of 2^kTreeLevels - 1 points; one launch evaluates all of them, two wavefronts a point,
// and the next launch (every work-group for itself, from the same values) takes the steps with the
// stopping rule after each, so brackets, step count and the returned mu are those of one step at
// a time.  A pass of one work-group over seven points took 5 us for three steps (tail sums and 16
// passes: 94 us at N = 256, 99 at N = 1000); a launch takes 7 us for eight (whole search 55 us; with
// ten steps a launch, 1023 points, 62).
constexpr int kTreeLevels = 8, kTreePoints = (1 << kTreeLevels) - 1, kTreePasses = 6, kTreeNT = 128;

struct SearchState {
    double lo, hi, mid, t_mid;
    int32_t it;      // the step to take next
    int32_t iters, status;
    int32_t stop;    // 1: search over, 2: no bracket (the scalars say so already)
};
static_assert(kTreePasses * (sizeof(SearchState) + sizeof(double) * 2) + 2 * sizeof(double) * kTreePoints <=
                  sizeof(double) * kSearchWork, "search workspace");

// Steps of the bisection from the values tv of one pass's tree.
__device__ inline void take_steps(SearchState& st, const double* tv, double ne, double tol, int max_iter) {
    if (st.stop) return;
    int k = 0;
#pragma unroll 1
    for (int lev = 0; lev < kTreeLevels; ++lev) {
        st.mid = 0.5 * (st.lo + st.hi);
        st.t_mid = tv[k];
        st.iters = st.it;
        if (fabs(st.t_mid - ne) < tol) {
            st.status = CHEBDM_OK;
            st.stop = 1;
            return;
        }
        const bool below = st.t_mid < ne;
        if (below) st.lo = st.mid;
        else st.hi = st.mid;
        if (st.hi - st.lo < 4.0 * ulp_spacing(st.mid) || ++st.it > max_iter) {
            st.stop = 1;
            return;
        }
        k = 2 * k + (below ? 2 : 1);
    }
}

__global__ void __launch_bounds__(kBisectThreads)
k_search_begin(const double* __restrict__ w, const double* __restrict__ x, int64_t M, DevScalars* s,
               double* __restrict__ scratch, SearchState* states) {
    __shared__ double part[kBisectThreads / 64];
    __shared__ double win[8];
    __shared__ double tout[2];
    const double* blk = nullptr;
    if (M >= 4 * kQBlock) {
        tail_sums<kBisectThreads>(w, M, scratch);
        blk = scratch;
    }
    trace_pass_groups<kBisectThreads, 2>(threadIdx.x == 0 ? -1.0 : 1.0, w, x, M, s->beta_s, part, win, tout, blk);
    if (threadIdx.x != 0) return;
    SearchState st{-1.0, 1.0, 0.0, NAN, 1, 0, CHEBDM_WARN_NOCONV, s->max_iter < 1 ? 1 : 0};
    if (!(tout[0] < s->n_elec && s->n_elec < tout[1])) {
        s->mu_s = NAN;
        s->trace = NAN;
        s->iters = 0;
        s->evals = 2;
        s->learned = 0;
        s->status = CHEBDM_ERR_BRACKET;
        s->lo = -1.0;
        s->hi = 1.0;
        st.stop = 2;
    }
    states[0] = st;
}

// Pass p: the state before it follows from states[p - 1] and that pass's values.
__global__ void __launch_bounds__(kTreeNT)
k_search_pass(const double* __restrict__ w, const double* __restrict__ x, int64_t M, const DevScalars* __restrict__ s,
              const double* __restrict__ blk, SearchState* states, double* tv, int p) {
    __shared__ double part[kTreeNT / 64], win[4], tout[1];
    __shared__ double prev[kTreePoints];
    __shared__ SearchState now;
    if (p > 0) {
        const double* tp = tv + ((p - 1) & 1) * kTreePoints;
        for (int i = threadIdx.x; i < kTreePoints; i += kTreeNT) prev[i] = tp[i];
    }
    if (threadIdx.x == 0) now = states[p > 0 ? p - 1 : 0];
    __syncthreads();
    if (threadIdx.x == 0 && p > 0) {
        take_steps(now, prev, s->n_elec, s->tol, s->max_iter);
        if (blockIdx.x == 0) states[p] = now;
    }
    __syncthreads();
    if (now.stop) return;
    const int q1 = (int)blockIdx.x + 1;
    double l = now.lo, h = now.hi;
    for (int b = 30 - __clz(q1); b >= 0; --b) {   // down to node blockIdx.x of the tree
        const double m = 0.5 * (l + h);
        if ((q1 >> b) & 1) l = m;
        else h = m;
    }
    trace_pass_groups<kTreeNT, 1>(0.5 * (l + h), w, x, M, s->beta_s, part, win, tout, M >= 4 * kQBlock ? blk : nullptr);
    if (threadIdx.x == 0) tv[(p & 1) * kTreePoints + blockIdx.x] = tout[0];
}

// The last pass's steps, any that are still left, and the result.
__global__ void __launch_bounds__(kBisectThreads)
k_search_end(const double* __restrict__ w, const double* __restrict__ x, int64_t M, DevScalars* s,
             const double* __restrict__ scratch, const SearchState* states, const double* tv) {
    constexpr int NP = (1 << kBisectLevels) - 1;
    __shared__ double part[kBisectThreads / 64];
    __shared__ double win[4 * NP];
    __shared__ double tout[NP];
    __shared__ double prev[kTreePoints];
    __shared__ SearchState now;
    const double* tp = tv + ((kTreePasses - 1) & 1) * kTreePoints;
    for (int i = threadIdx.x; i < kTreePoints; i += kBisectThreads) prev[i] = tp[i];
    if (threadIdx.x == 0) now = states[kTreePasses - 1];
    __syncthreads();
    const double ne = s->n_elec, tol = s->tol;
    const int max_iter = s->max_iter;
    if (threadIdx.x == 0) take_steps(now, prev, ne, tol, max_iter);
    __syncthreads();
    if (now.stop == 2) return;
    double lo = now.lo, hi = now.hi, mid = now.mid, t_mid = now.t_mid;
    int iters = now.iters, status = now.status;
    if (!now.stop)
        bisect_levels<kBisectThreads, kBisectLevels>(M, w, x, s->beta_s, ne, tol, max_iter, part, win, tout,
                                                     M >= 4 * kQBlock ? scratch : nullptr, lo, hi, mid, t_mid, iters,
                                                     status, now.it);
    if (threadIdx.x == 0) {
        s->mu_s = mid;
        s->trace = t_mid;
        s->iters = iters;
        s->evals = 2 + iters;
        s->learned = 0;
        s->status = status;
        s->lo = lo;
        s->hi = hi;
    }
}

}  // namespace

hipError_t launch_set_scalars(DevScalars* s, double emin, double emax, double beta, double mu,
                              int has_mu, double n_elec, double tol, int max_iter, hipStream_t st,
                              int bounds_on_device) {
    hipLaunchKernelGGL(k_set_scalars, dim3(1), dim3(1), 0, st, s, emin, emax, beta, mu, has_mu,
                       n_elec, tol, max_iter, bounds_on_device);
    return hipGetLastError();
}

hipError_t launch_fermi_coeffs(int order, int M, const DevScalars* s, double* f_tab, double* c_out,
                               hipStream_t st, int damping, int terms) {
    hipLaunchKernelGGL(k_fermi_table, dim3((unsigned)((M + 255) / 256)), dim3(256), 0, st,
                       (int64_t)M, s, f_tab);
    if (!turns_exact(M)) terms = 1;
    hipLaunchKernelGGL(terms ? k_dct2<true> : k_dct2<false>, dim3((unsigned)(order + 1)), dim3(256), 0, st, (int64_t)M,
                       (const double*)f_tab, c_out, order, damping);
    return hipGetLastError();
}

hipError_t launch_block_coeffs(const double* c, int order, int k, int m, int form, double* coef,
                               hipStream_t st, int split_h, int split_q) {
    if (k > kMaxBlocks || m > kMaxBlocks) return hipErrorInvalidValue;
    if (split_h < 0 || m - split_h > (split_h ? split_h : m) || (split_q > 0 && split_h - split_q > split_q))
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_block_coeffs, dim3(1), dim3(64), 0, st, c, order, k, m, form, coef, split_h, split_q);
    return hipGetLastError();
}

hipError_t launch_assemble_moments(const double* tr_baby, const double* gram, int k, int m,
                                   int order, int64_t n, double* tau, hipStream_t st) {
    hipLaunchKernelGGL(k_assemble_moments, dim3(1), dim3(256), 0, st, tr_baby, gram, k, m, order, n, tau);
    return hipGetLastError();
}

hipError_t launch_dct3(const double* tau, int order, int M, double* w, double* x_tab,
                       hipStream_t st, int damping, int terms) {
    const int64_t threads = ((int64_t)M + 1) / 2 * kDctSplit;
    if (!turns_exact(M)) terms = 1;
    hipLaunchKernelGGL(terms ? k_dct3<true> : k_dct3<false>, dim3((unsigned)((threads + 255) / 256)), dim3(256),
                       sizeof(double) * (size_t)dct3_padded(order), st, tau, order, (int64_t)M, w, x_tab, damping);
    return hipGetLastError();
}

hipError_t launch_bisect(const double* w, const double* x_tab, int M, DevScalars* s, int mode, double* scratch,
                         double* work, hipStream_t st) {
    if (mode < 0 || mode > 1) return hipErrorInvalidValue;
    const int64_t m = M;
    if (mode == 1) {
        hipLaunchKernelGGL(k_search_newton, dim3(1), dim3(kBisectThreads), 0, st, w, x_tab, m, s, scratch);
        return hipGetLastError();
    }
    double* tv = work;
    SearchState* states = reinterpret_cast<SearchState*>(work + 2 * kTreePoints);
    hipLaunchKernelGGL(k_search_begin, dim3(1), dim3(kBisectThreads), 0, st, w, x_tab, m, s, scratch, states);
    for (int p = 0; p < kTreePasses; ++p)
        hipLaunchKernelGGL(k_search_pass, dim3(kTreePoints), dim3(kTreeNT), 0, st, w, x_tab, m, (const DevScalars*)s,
                           (const double*)scratch, states, tv, p);
    hipLaunchKernelGGL(k_search_end, dim3(1), dim3(kBisectThreads), 0, st, w, x_tab, m, s, (const double*)scratch,
                       (const SearchState*)states, (const double*)tv);
    return hipGetLastError();
}

}  // namespace chebdm
