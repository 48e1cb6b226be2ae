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

__global__ void __launch_bounds__(kColsPerBlock)
k_gersh_partial(const double* __restrict__ H, int64_t n, int64_t ldh, int64_t rows_per_split,
                double* __restrict__ partial) {
    const int64_t j = (int64_t)blockIdx.x * kColsPerBlock + threadIdx.x;
    if (j >= n) return;
    const int64_t i0 = (int64_t)blockIdx.y * rows_per_split;
    const int64_t i1 = i0 + rows_per_split < n ? i0 + rows_per_split : n;
    double s = 0.0;
    const double* p = H + i0 * ldh + j;
#pragma unroll 8
    for (int64_t i = i0; i < i1; ++i, p += ldh) {
        const double v = fabs(*p);
        s += (i == j) ? 0.0 : v;
    }
    partial[(int64_t)blockIdx.y * n + j] = s;
}

constexpr int kColThreads = 256;

// Column j: r_j = sum of the split partials in order (sixteen loads in flight; one load per addition
// took 20 us at N = 2000), the disc [d - r_j, d + r_j] with d = H[j][j].
__device__ __forceinline__ void column_disc(const double* __restrict__ H, int64_t n, int64_t ldh,
                                            const double* __restrict__ partial, int nsplit, int64_t j, double& lo,
                                            double& hi, double& bad) {
    double r = 0.0;
    const double d = H[j * ldh + j];
    int sp = 0;
    for (; sp + 16 <= nsplit; sp += 16) {
        double v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = partial[(int64_t)(sp + u) * n + j];
#pragma unroll
        for (int u = 0; u < 16; ++u) r += v[u];
    }
    for (; sp < nsplit; ++sp) r += partial[(int64_t)sp * n + j];
    if (!isfinite(r) || !isfinite(d)) bad = 1.0;
    lo = d - r;
    hi = d + r;
}

// Per work-group of columns: min, max and a non-finite flag, written to out[3][nb].
__global__ void __launch_bounds__(kColThreads)
k_gersh_cols(const double* __restrict__ H, int64_t n, int64_t ldh, const double* __restrict__ partial, int nsplit,
             double* __restrict__ out, int nb) {
    __shared__ double smem[kColThreads / 64];
    const int64_t j = (int64_t)blockIdx.x * kColThreads + threadIdx.x;
    double lo = INFINITY, hi = -INFINITY, bad = 0.0;
    if (j < n) column_disc(H, n, ldh, partial, nsplit, j, lo, hi, bad);
    bad = block_sum<kColThreads>(bad, smem);
    lo = block_min<kColThreads>(lo, smem);
    hi = block_max<kColThreads>(hi, smem);
    if (threadIdx.x == 0) {
        out[blockIdx.x] = lo;
        out[nb + blockIdx.x] = hi;
        out[2 * nb + blockIdx.x] = bad;
    }
}

// The bounds into the scalars, and into their host mirror where one is given.
__device__ __forceinline__ void put_bounds(DevScalars* s, double lo, double hi, int bad) {
    if (!s) return;
    s->emin = lo;
    s->emax = hi;
    s->nonfinite = bad;
}

// Up to kOneFold columns: columns and result in one launch.
constexpr int kOneFold = 1024;

__global__ void __launch_bounds__(kOneFold)
k_gersh_fold(const double* __restrict__ H, int64_t n, int64_t ldh, const double* __restrict__ partial, int nsplit,
             DevScalars* s, DevScalars* h_s) {
    __shared__ double smem[kOneFold / 64];
    double lo = INFINITY, hi = -INFINITY, bad = 0.0;
    if ((int)threadIdx.x < n) column_disc(H, n, ldh, partial, nsplit, threadIdx.x, lo, hi, bad);
    bad = block_sum<kOneFold>(bad, smem);
    lo = block_min<kOneFold>(lo, smem);
    hi = block_max<kOneFold>(hi, smem);
    if (threadIdx.x == 0) {
        put_bounds(s, lo, hi, bad > 0.0 ? 1 : 0);
        put_bounds(h_s, lo, hi, bad > 0.0 ? 1 : 0);
    }
}

constexpr int kFinalThreads = 256;

__global__ void __launch_bounds__(kFinalThreads)
k_gersh_final(const double* __restrict__ part, int nb, DevScalars* s, DevScalars* h_s) {
    __shared__ double smem[kFinalThreads / 64];
    double lo = INFINITY, hi = -INFINITY, bad = 0.0;
    for (int b = threadIdx.x; b < nb; b += kFinalThreads) {
        lo = fmin(lo, part[b]);
        hi = fmax(hi, part[nb + b]);
        bad += part[2 * nb + b];
    }
    bad = block_sum<kFinalThreads>(bad, smem);
    lo = block_min<kFinalThreads>(lo, smem);
    hi = block_max<kFinalThreads>(hi, smem);
    if (threadIdx.x == 0) {
        put_bounds(s, lo, hi, bad > 0.0 ? 1 : 0);
        put_bounds(h_s, lo, hi, bad > 0.0 ? 1 : 0);
    }
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
                             int64_t partial_cap, DevScalars* s, hipStream_t st, DevScalars* h_s) {
    const int64_t col_blocks = (n + kColsPerBlock - 1) / kColsPerBlock;
    int64_t nsplit = (2048 + col_blocks - 1) / col_blocks;
    const int64_t max_split = (n + 31) / 32;
    if (nsplit > max_split) nsplit = max_split;
    if (nsplit < 1) nsplit = 1;
    const int64_t nb = (n + kColThreads - 1) / kColThreads;
    while (nsplit > 1 && nsplit * n + 3 * nb > partial_cap) nsplit >>= 1;
    if (nsplit * n + 3 * nb > partial_cap) return hipErrorInvalidValue;
    const int64_t rows_per_split = (n + nsplit - 1) / nsplit;
    nsplit = (n + rows_per_split - 1) / rows_per_split;
    double* part2 = partial + nsplit * n;
    hipLaunchKernelGGL(k_gersh_partial, dim3((unsigned)col_blocks, (unsigned)nsplit), dim3(kColsPerBlock),
                       0, st, H, n, ldh, rows_per_split, partial);
    if (n <= kOneFold) {
        hipLaunchKernelGGL(k_gersh_fold, dim3(1), dim3(kOneFold), 0, st, H, n, ldh, (const double*)partial, (int)nsplit,
                           s, h_s);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_gersh_cols, dim3((unsigned)nb), dim3(kColThreads), 0, st, H, n, ldh,
                       (const double*)partial, (int)nsplit, part2, (int)nb);
    hipLaunchKernelGGL(k_gersh_final, dim3(1), dim3(kFinalThreads), 0, st, (const double*)part2, (int)nb, s,
                       h_s);
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
