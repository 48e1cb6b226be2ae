// The density as one sum of products, D = R_0 + sum_{l=1}^{m-1} T_{lk} R_l, float64.
//
// Where the call has the ladder T_{lk} (the mu search's moments need it), the giant steps need no
// recurrence: the m - 1 products are one contraction of length (m - 1) n, whose K units go out side by
// side in one launch, with one epilogue.  The chains of giant steps were eight launches of up to four
// products of one length, none of which fills the chip below N ~ 1400.
//
// A work-group takes a tile of 32 to 64 rows and one of S slices of the contraction, shared by its four
// wavefronts (parts added in LDS); the second launch adds the slices in order, R_0 last, and stores
// (i, j) and (j, i).  Slice s belongs to XCD s mod 8 (work-groups are dealt to the XCDs round-robin): an
// XCD then reads its own eighth of the matrices instead of all of them.  Operands are symmetric and read
// along rows as in k_gemm.hip, two register stages.
#include "internal.h"

namespace chebdm {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

constexpr int kWaves = 4, kXcds = 8;

__device__ __forceinline__ void tile_at(int t, int ntile, int& ti, int& tj) {
    ti = 0;
    while (t >= ntile - ti) t -= ntile - ti++;
    tj = ti + t;
}

// T, R: T_k and R_1, the next ladder matrix and block `stride` elements on each.
template <int F, int OCC>
__global__ void __launch_bounds__(64 * kWaves, OCC)
k_sum_slices(const double* __restrict__ T, const double* __restrict__ R, int64_t stride, int64_t ld, int64_t units,
             int nchunk, int ntile, int ntri, int S, double* __restrict__ part) {
    constexpr int kTile = 16 * F, kRow = kTile + 1, kTileOuts = kTile * kTile;
    __shared__ double red[kWaves][kTile * kRow];
    const int lane = threadIdx.x % 64, w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int g = (int)blockIdx.x / kXcds, s = g / ntri * kXcds + (int)blockIdx.x % kXcds, t = g % ntri;
    int ti, tj;
    tile_at(t, ntile, ti, tj);
    const int64_t lane_off = (int64_t)(lane % 16) * ld + 4 * (lane / 16);
    const double* A = T + (int64_t)ti * kTile * ld + lane_off;
    const double* B = R + (int64_t)tj * kTile * ld + lane_off;
    const int64_t part_of = (int64_t)s * kWaves + w, parts = (int64_t)S * kWaves;
    const int64_t u0 = units * part_of / parts, count = units * (part_of + 1) / parts - u0;
    int c = (int)(u0 % nchunk);
    int64_t off = u0 / nchunk * stride + 16 * c;
    struct Stage {
        f64x2 a[F][2], b[F][2];   // [16-row block][half of the lane's four k]
    };
    auto load = [&](Stage& x) {
#pragma unroll
        for (int r = 0; r < F; ++r)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                x.a[r][h] = *(const f64x2*)(A + off + (int64_t)r * 16 * ld + 2 * h);
                x.b[r][h] = *(const f64x2*)(B + off + (int64_t)r * 16 * ld + 2 * h);
            }
    };
    auto next = [&] {
        off += 16;
        if (++c == nchunk) {
            c = 0;
            off += stride - 16 * (int64_t)nchunk;
        }
    };
    f64x4 acc[F][F] = {};
    auto mul = [&](const Stage& x) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int r = 0; r < F; ++r)
#pragma unroll
                for (int q = 0; q < F; ++q)
                    acc[r][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(x.a[r][k / 2][k % 2], x.b[q][k / 2][k % 2],
                                                                     acc[r][q], 0, 0, 0);
    };
    if (count > 0) {   // the last refill re-reads the final chunk
        Stage x, y;
        load(x);
        int64_t i = 0;
        for (; i + 2 <= count; i += 2) {
            next();
            load(y);
            mul(x);
            if (i + 2 < count) next();
            load(x);
            mul(y);
        }
        if (i < count) mul(x);
    }
    // D[i][j] of a 16 x 16 block is register i / 4 of lane j + 16 (i mod 4)
#pragma unroll
    for (int r = 0; r < F; ++r)
#pragma unroll
        for (int q = 0; q < F; ++q)
#pragma unroll
            for (int x = 0; x < 4; ++x)
                red[w][(16 * r + 4 * x + lane / 16) * kRow + 16 * q + lane % 16] = acc[r][q][x];
    __syncthreads();
    double* out = part + ((int64_t)s * ntri + t) * kTileOuts;
#pragma unroll
    for (int h = 0; h < kTileOuts / (64 * kWaves); ++h) {
        const int e = threadIdx.x + 64 * kWaves * h, at = e / kTile * kRow + e % kTile;
        out[e] = ((red[0][at] + red[1][at]) + red[2][at]) + red[3][at];
    }
}

// Eight rows of a tile a work-group, a thread an element; the slices' sum in order, eight loads
// in flight.
constexpr int kFixRows = 8;

template <int F>
__global__ void __launch_bounds__(kFixRows * 16 * F)
k_sum_fix(const double* __restrict__ part, int S, int ntile, int ntri, const double* __restrict__ R0, int n, int64_t ld,
          double* __restrict__ D, int64_t ldd) {
    constexpr int kTile = 16 * F, kRow = kTile + 1, kTileOuts = kTile * kTile;
    __shared__ double out[kFixRows][kRow];
    const int t = (int)blockIdx.x / (kTile / kFixRows), rows = (int)blockIdx.x % (kTile / kFixRows) * kFixRows;
    int ti, tj;
    tile_at(t, ntile, ti, tj);
    const int i0 = ti * kTile + rows, j0 = tj * kTile;
    {
        const int i = (int)threadIdx.x / kTile, j = (int)threadIdx.x % kTile;
        const double r0 = R0[(int64_t)(i0 + i) * ld + j0 + j];
        const double* p = part + (int64_t)t * kTileOuts + rows * kTile + threadIdx.x;
        double sum = 0.0;
        for (int s = 0; s < S; s += kXcds) {   // S is a multiple of 8
            double v[kXcds];
#pragma unroll
            for (int u = 0; u < kXcds; ++u) v[u] = p[(int64_t)(s + u) * ntri * kTileOuts];
#pragma unroll
            for (int u = 0; u < kXcds; ++u) sum += v[u];
        }
        sum += r0;
        out[i][j] = sum;
        if (i0 + i <= j0 + j && j0 + j < n) D[(int64_t)(i0 + i) * ldd + j0 + j] = sum;
    }
    __syncthreads();
    const int i = (int)threadIdx.x % kFixRows, j = (int)threadIdx.x / kFixRows;
    if (i0 + i < j0 + j && j0 + j < n) D[(int64_t)(j0 + j) * ldd + i0 + i] = out[i][j];
}

// Slices: about OCC wavefronts a SIMD, at least four chunks of 16 a wavefront, parts within the scratch.
template <int F, int OCC>
hipError_t launch(const double* T, const double* R, int64_t stride, int prods, const double* R0, int64_t n, int64_t ld,
                  double* D, int64_t ldd, double* part, size_t part_bytes, hipStream_t st) {
    constexpr int kTile = 16 * F;
    const int ntile = (int)((n + kTile - 1) / kTile), nchunk = (int)((n + 15) / 16);
    if (n < 1 || prods < 1 || !part || (int64_t)ntile * kTile > ld || ld % 2 != 0) return hipErrorInvalidValue;
    const int64_t ntri = (int64_t)ntile * (ntile + 1) / 2, units = (int64_t)prods * nchunk;
    int64_t S = 1024 * OCC / (kWaves * ntri);
    if (S > units / (4 * kWaves)) S = units / (4 * kWaves);
    S = (S + kXcds / 2) / kXcds * kXcds;
    if (S < kXcds) S = kXcds;
    const int64_t fit = (int64_t)(part_bytes / (ntri * kTile * kTile * sizeof(double))) / kXcds * kXcds;
    if (S > fit) S = fit;
    if (S < kXcds) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_sum_slices<F, OCC>), dim3((unsigned)(ntri * S)), dim3(64 * kWaves), 0, st, T, R, stride, ld,
                       units, nchunk, ntile, (int)ntri, (int)S, part);
    hipLaunchKernelGGL(k_sum_fix<F>, dim3((unsigned)(ntri * (kTile / kFixRows))), dim3(kFixRows * kTile), 0, st,
                       (const double*)part, (int)S, ntile, (int)ntri, R0, (int)n, ld, D, ldd);
    return hipGetLastError();
}

}  // namespace

// 48-tiles from N = 560 (the matrices' padding has to hold their last one, else 64-tiles): fewer operand
// bytes per product; below, 32-tiles, of which more wavefronts fit a SIMD.  mu search and D of order 512
// with chains / 32- / 48- / 64-tiles, us: N = 400 495 / 428 / 436 / 429, 500 673 / 590 / 597 / 600, 600 792 /
// 713 / 697 / 702, 700 958 / 928 / 895 / 930, 800 1330 / 1271 / 1181 / 1185, 1000 1805 / 1905 / 1727 / 1755, 1100
// 2285 / 2440 / 2178 / 2248, 1300 (chains on the int8 units) 3228 / 3651 / 3303 / 3315.
hipError_t launch_product_sum(const double* T, const double* R, int64_t stride, int prods, const double* R0, int64_t n,
                              int64_t ld, double* D, int64_t ldd, void* scratch, size_t scratch_bytes, hipStream_t st) {
    double* part = static_cast<double*>(scratch);
    if (n <= 560) return launch<2, 4>(T, R, stride, prods, R0, n, ld, D, ldd, part, scratch_bytes, st);
    if ((n + 47) / 48 * 48 <= ld) return launch<3, 2>(T, R, stride, prods, R0, n, ld, D, ldd, part, scratch_bytes, st);
    return launch<4, 1>(T, R, stride, prods, R0, n, ld, D, ldd, part, scratch_bytes, st);
}

}  // namespace chebdm
