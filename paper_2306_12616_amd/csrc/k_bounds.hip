// Spectral bounds, the spectrum map H -> H~, and traces.
//
// Bounds: Gershgorin discs (the paper asks for the lowest and highest
// eigenvalues e_a, e_b, Sec. II.B, without naming a method).  Since H is
// symmetric, the absolute row sums equal the absolute column sums, so each
// thread owns one column and walks down rows: a wavefront reads 512
// contiguous bytes per row (coalesced), and row chunks are split across
// workgroups.  Partial sums land in a [split][column] buffer and one
// workgroup folds them in a fixed order, so the result is deterministic.
#include <cmath>

#include "internal.h"
#include "reduce.h"

namespace chebdm {

namespace {

constexpr int kColsPerBlock = 256;

// SPREAD: also the columns' sums of squares off the diagonal, after the absolute sums in `partial`
// (the pass reads H from memory either way).
template <bool SPREAD>
__global__ void __launch_bounds__(kColsPerBlock)
k_gersh_partial(const double* __restrict__ H, int64_t n, int64_t ldh, int64_t rows_per_split,
                double* __restrict__ partial) {
    const int64_t j = (int64_t)blockIdx.x * kColsPerBlock + threadIdx.x;
    if (j >= n) return;
    const int64_t i0 = (int64_t)blockIdx.y * rows_per_split;
    const int64_t i1 = i0 + rows_per_split < n ? i0 + rows_per_split : n;
    double s = 0.0, q = 0.0;
    const double* p = H + i0 * ldh + j;
#pragma unroll 8
    for (int64_t i = i0; i < i1; ++i, p += ldh) {
        const double h = fabs(*p), v = (i == j) ? 0.0 : h;   // the load without a condition
        s += v;
        if constexpr (SPREAD) q = fma(v, v, q);
    }
    partial[(int64_t)blockIdx.y * n + j] = s;
    if constexpr (SPREAD) partial[((int64_t)gridDim.y + blockIdx.y) * n + j] = q;
}

constexpr int kColThreads = 256;

// Sums of a column's split partials in order (sixteen loads of each in flight; one load per addition
// took 20 us at N = 2000): absolute values and, for SPREAD, squares.
template <bool SPREAD>
__device__ __forceinline__ void split_sums(const double* __restrict__ partial, int64_t n, int nsplit, int64_t j,
                                           double& r, double& q) {
    const double* squares = partial + (int64_t)nsplit * n;
    r = q = 0.0;
    int sp = 0;
    for (; sp + 16 <= nsplit; sp += 16) {
        double v[16], w[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            v[u] = partial[(int64_t)(sp + u) * n + j];
            if constexpr (SPREAD) w[u] = squares[(int64_t)(sp + u) * n + j];
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            r += v[u];
            if constexpr (SPREAD) q += w[u];
        }
    }
    for (; sp < nsplit; ++sp) {
        r += partial[(int64_t)sp * n + j];
        if constexpr (SPREAD) q += squares[(int64_t)sp * n + j];
    }
}

// What the columns' sums give, per column or over a set of them.
struct Discs {
    double lo = INFINITY, hi = -INFINITY, bad = 0.0, spread = INFINITY, radius = INFINITY;
};

// Column j: r_j = sum |h_ij| off the diagonal, the disc [d - r_j, d + r_j] with d = H[j][j].
template <bool SPREAD>
__device__ __forceinline__ Discs column_disc(const double* __restrict__ H, int64_t n, int64_t ldh,
                                             const double* __restrict__ partial, int nsplit, int64_t j) {
    Discs c;
    const double d = H[j * ldh + j];
    double r, q;
    split_sums<SPREAD>(partial, n, nsplit, j, r, q);
    if (!isfinite(r) || !isfinite(d)) c.bad = 1.0;
    c.lo = d - r;
    c.hi = d + r;
    if constexpr (SPREAD) {
        // zero where the sums leave the float64 range (a spread is at most 1 up to rounding)
        const double v = r * r / ((double)(n - 1) * q);
        c.spread = q >= 1e-290 && v < 2.0 ? v : 0.0;
        c.radius = r >= 0.0 ? r : 0.0;
    }
    return c;
}

template <int NT, bool SPREAD>
__device__ __forceinline__ void reduce_discs(Discs& c, double* smem) {
    c.bad = block_sum<NT>(c.bad, smem);
    c.lo = block_min<NT>(c.lo, smem);
    c.hi = block_max<NT>(c.hi, smem);
    if constexpr (SPREAD) {
        c.spread = block_min<NT>(c.spread, smem);
        c.radius = block_min<NT>(c.radius, smem);
    }
}

// Per work-group of columns: min, max, a non-finite flag and the spread's minima, written to out[5][nb].
template <bool SPREAD>
__global__ void __launch_bounds__(kColThreads)
k_gersh_cols(const double* __restrict__ H, int64_t n, int64_t ldh, const double* __restrict__ partial, int nsplit,
             double* __restrict__ out, int nb) {
    __shared__ double smem[kColThreads / 64];
    const int64_t j = (int64_t)blockIdx.x * kColThreads + threadIdx.x;
    Discs c;
    if (j < n) c = column_disc<SPREAD>(H, n, ldh, partial, nsplit, j);
    reduce_discs<kColThreads, SPREAD>(c, smem);
    if (threadIdx.x == 0) {
        out[blockIdx.x] = c.lo;
        out[nb + blockIdx.x] = c.hi;
        out[2 * nb + blockIdx.x] = c.bad;
        if constexpr (SPREAD) {
            out[3 * nb + blockIdx.x] = c.spread;
            out[4 * nb + blockIdx.x] = c.radius;
        }
    }
}

// The bounds into the scalars, and into their host mirror where one is given.
template <bool SPREAD>
__device__ __forceinline__ void put_bounds(DevScalars* s, const Discs& c) {
    if (!s) return;
    s->emin = c.lo;
    s->emax = c.hi;
    s->nonfinite = c.bad > 0.0 ? 1 : 0;
    if constexpr (SPREAD) {
        s->spread = c.spread;
        s->radius = c.radius;
    }
}

// Up to kOneFold columns: columns and result in one launch.
constexpr int kOneFold = 1024;

template <bool SPREAD>
__global__ void __launch_bounds__(kOneFold)
k_gersh_fold(const double* __restrict__ H, int64_t n, int64_t ldh, const double* __restrict__ partial, int nsplit,
             DevScalars* s, DevScalars* h_s) {
    __shared__ double smem[kOneFold / 64];
    Discs c;
    if ((int)threadIdx.x < n) c = column_disc<SPREAD>(H, n, ldh, partial, nsplit, threadIdx.x);
    reduce_discs<kOneFold, SPREAD>(c, smem);
    if (threadIdx.x == 0) {
        put_bounds<SPREAD>(s, c);
        put_bounds<SPREAD>(h_s, c);
    }
}

constexpr int kFinalThreads = 256;

template <bool SPREAD>
__global__ void __launch_bounds__(kFinalThreads)
k_gersh_final(const double* __restrict__ part, int nb, DevScalars* s, DevScalars* h_s) {
    __shared__ double smem[kFinalThreads / 64];
    Discs c;
    for (int b = threadIdx.x; b < nb; b += kFinalThreads) {
        c.lo = fmin(c.lo, part[b]);
        c.hi = fmax(c.hi, part[nb + b]);
        c.bad += part[2 * nb + b];
        if constexpr (SPREAD) {
            c.spread = fmin(c.spread, part[3 * nb + b]);
            c.radius = fmin(c.radius, part[4 * nb + b]);
        }
    }
    reduce_discs<kFinalThreads, SPREAD>(c, smem);
    if (threadIdx.x == 0) {
        put_bounds<SPREAD>(s, c);
        put_bounds<SPREAD>(h_s, c);
    }
}

template <bool SPREAD>
void gershgorin(const double* H, int64_t n, int64_t ldh, double* partial, int64_t nsplit, int64_t rows_per_split,
                DevScalars* s, DevScalars* h_s, hipStream_t st) {
    const int64_t col_blocks = (n + kColsPerBlock - 1) / kColsPerBlock, nb = (n + kColThreads - 1) / kColThreads;
    double* part2 = partial + (SPREAD ? 2 : 1) * nsplit * n;
    hipLaunchKernelGGL(k_gersh_partial<SPREAD>, dim3((unsigned)col_blocks, (unsigned)nsplit), dim3(kColsPerBlock), 0, st,
                       H, n, ldh, rows_per_split, partial);
    if (n <= kOneFold) {
        hipLaunchKernelGGL(k_gersh_fold<SPREAD>, dim3(1), dim3(kOneFold), 0, st, H, n, ldh, (const double*)partial,
                           (int)nsplit, s, h_s);
        return;
    }
    hipLaunchKernelGGL(k_gersh_cols<SPREAD>, dim3((unsigned)nb), dim3(kColThreads), 0, st, H, n, ldh,
                       (const double*)partial, (int)nsplit, part2, (int)nb);
    hipLaunchKernelGGL(k_gersh_final<SPREAD>, dim3(1), dim3(kFinalThreads), 0, st, (const double*)part2, (int)nb, s, h_s);
}

// T_1 = H~ = (H - cen I) / half; only the n x n part is written.
template <typename T>
__global__ void __launch_bounds__(256)
k_shift(const double* __restrict__ H, int64_t n, int64_t ldh, const DevScalars* __restrict__ s,
        T* __restrict__ out, int64_t ldw) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t i = blockIdx.y;
    if (j >= n) return;
    const double cen = s->cen, half = s->half;
    const double h = H[i * ldh + j];
    out[i * ldw + j] = (T)((i == j ? h - cen : h) / half);
}

template <typename T>
__global__ void __launch_bounds__(256)
k_traces(const T* __restrict__ base, int64_t stride, int64_t n, int64_t ld, double* __restrict__ out) {
    __shared__ double smem[4];
    const T* a = base + (int64_t)blockIdx.x * stride;
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) acc += (double)a[i * ld + i];
    acc = block_sum<256>(acc, smem);
    if (threadIdx.x == 0) out[blockIdx.x] = acc;
}

// D = value * I on the n x n block (the degenerate spectrum e_a = e_b).
__global__ void __launch_bounds__(256)
k_fill_identity(double* __restrict__ D, int64_t n, int64_t ldd, double value) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t i = blockIdx.y;
    if (j >= n) return;
    D[i * ldd + j] = (i == j) ? value : 0.0;
}

// D = (double) src on the n x n block.
template <typename T>
__global__ void __launch_bounds__(256)
k_copy_out(const T* __restrict__ src, int64_t ld, int64_t n, double* __restrict__ D, int64_t ldd) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t i = blockIdx.y;
    if (j >= n) return;
    D[i * ldd + j] = (double)src[i * ld + j];
}

// D != nullptr: tr D first, into *trD.
__global__ void __launch_bounds__(256)
k_publish(const double* __restrict__ s, double* __restrict__ trD, const double* __restrict__ D, int64_t n, int64_t ldd,
          const double* __restrict__ extra, int count, double* h_s, double* h_trD, double* h_extra) {
    __shared__ double smem[4];
    const int t = threadIdx.x;
    if (t < (int)(sizeof(DevScalars) / sizeof(double))) h_s[t] = s[t];
    for (int i = t; i < count; i += 256) h_extra[i] = extra[i];
    if (D) {
        double acc = 0.0;
        for (int64_t i = t; i < n; i += 256) acc += D[i * ldd + i];
        acc = block_sum<256>(acc, smem);
        if (t == 0) *trD = *h_trD = acc;
    }
}

}  // namespace

hipError_t launch_publish(const DevScalars* s, double* trD, const double* D, int64_t n, int64_t ldd,
                          const double* extra, int count, DevScalars* h_s, double* h_trD, double* h_extra,
                          hipStream_t st) {
    static_assert(sizeof(DevScalars) % sizeof(double) == 0, "copied as doubles");
    hipLaunchKernelGGL(k_publish, dim3(1), dim3(256), 0, st, reinterpret_cast<const double*>(s), trD, D, n, ldd, extra,
                       count, reinterpret_cast<double*>(h_s), h_trD, h_extra);
    return hipGetLastError();
}

hipError_t launch_fill_identity(double* D, int64_t n, int64_t ldd, double value, hipStream_t st) {
    hipLaunchKernelGGL(k_fill_identity, dim3((unsigned)((n + 255) / 256), (unsigned)n), dim3(256), 0, st, D,
                       n, ldd, value);
    return hipGetLastError();
}

hipError_t launch_copy_out(const void* src, int is_f64, int64_t ld, int64_t n, double* D, int64_t ldd,
                           hipStream_t st) {
    dim3 grid((unsigned)((n + 255) / 256), (unsigned)n);
    if (is_f64)
        hipLaunchKernelGGL(k_copy_out<double>, grid, dim3(256), 0, st, (const double*)src, ld, n, D, ldd);
    else
        hipLaunchKernelGGL(k_copy_out<float>, grid, dim3(256), 0, st, (const float*)src, ld, n, D, ldd);
    return hipGetLastError();
}

hipError_t launch_gershgorin(const double* H, int64_t n, int64_t ldh, double* partial,
                             int64_t partial_cap, DevScalars* s, hipStream_t st, DevScalars* h_s, bool with_spread) {
    const int64_t col_blocks = (n + kColsPerBlock - 1) / kColsPerBlock;
    int64_t nsplit = (2048 + col_blocks - 1) / col_blocks;
    const int64_t max_split = (n + 31) / 32;
    if (nsplit > max_split) nsplit = max_split;
    if (nsplit < 1) nsplit = 1;
    const int64_t nb = (n + kColThreads - 1) / kColThreads, per = with_spread ? 2 * n : n;
    while (nsplit > 1 && nsplit * per + 5 * nb > partial_cap) nsplit >>= 1;
    if (nsplit * per + 5 * nb > partial_cap) return hipErrorInvalidValue;
    const int64_t rows_per_split = (n + nsplit - 1) / nsplit;
    nsplit = (n + rows_per_split - 1) / rows_per_split;
    if (with_spread) gershgorin<true>(H, n, ldh, partial, nsplit, rows_per_split, s, h_s, st);
    else gershgorin<false>(H, n, ldh, partial, nsplit, rows_per_split, s, h_s, st);
    return hipGetLastError();
}

hipError_t launch_shift(const double* H, int64_t n, int64_t ldh, const DevScalars* s, void* T1,
                        int64_t ldw, int prec, hipStream_t st) {
    dim3 grid((unsigned)((n + 255) / 256), (unsigned)n);
    if (prec == CHEBDM_FP64)
        hipLaunchKernelGGL(k_shift<double>, grid, dim3(256), 0, st, H, n, ldh, s, (double*)T1, ldw);
    else
        hipLaunchKernelGGL(k_shift<float>, grid, dim3(256), 0, st, H, n, ldh, s, (float*)T1, ldw);
    return hipGetLastError();
}

hipError_t launch_traces(const void* base, int64_t stride, int count, int64_t n, int64_t ld,
                         int is_f64, double* out, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    if (is_f64)
        hipLaunchKernelGGL(k_traces<double>, dim3(count), dim3(256), 0, st, (const double*)base,
                           stride, n, ld, out);
    else
        hipLaunchKernelGGL(k_traces<float>, dim3(count), dim3(256), 0, st, (const float*)base,
                           stride, n, ld, out);
    return hipGetLastError();
}

}  // namespace chebdm
