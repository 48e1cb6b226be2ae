// The density as one sum of products, D = R_0 + sum_{l=1}^{m-1} T_{lk} R_l, float64.
//
// Where the call has the ladder T_{lk} (the mu search's moments need it), the giant steps need no
// recurrence: the m - 1 products are one contraction of length (m - 1) n, whose K units go out side by
// side in one launch, with one epilogue.  The chains of giant steps were eight launches of up to four
// products of one length, none of which fills the chip below N ~ 1400.
//
// Up to N = 700 a work-group takes a tile of 32 or 48 rows and one of S slices of the contraction, shared by its four
// wavefronts (parts added in LDS); the second launch adds the slices in order, R_0 last, and stores
// (i, j) and (j, i).  Slice s belongs to XCD s mod 8 (work-groups are dealt to the XCDs round-robin): an
// XCD then reads its own eighth of the matrices instead of all of them.  Operands are symmetric and read
// along rows as in k_gemm.hip, two register stages.
#include "internal.h"
#include "lds_copy.h"

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

// ------------------------------------------------------------------------- larger matrices: LDS, ranges
//
// 96 x 96 tiles of four 48 x 48 wavefronts that share their operands through LDS: half the L2 bytes of four
// separate 48-tiles, which ran at the rate of L2 (7-8 TB/s; N = 1000: 523 us, 442 with ranges).  Every XCD
// has an eighth of the contraction; its tiles times chunks go to G work-groups in equal contiguous ranges,
// two work-groups a CU, so that there is no last round.  A piece (range r of tile t) leaves its part at
// index r + t, which grows by one at every range and tile border; k_range_fix adds a tile's pieces in order.
constexpr int kBig = 96, kHalf = 48, kStages = 3, kCopies = 6;
constexpr int kPart = kBig * kBig;              // doubles of a piece: wavefront, 36 registers, lane
constexpr int kStageBytes = 4 * kCopies * 1024;

struct Ranges {   // of one XCD
    int64_t first, units, total;   // first unit, units of a tile, tiles times units
};
__device__ __forceinline__ Ranges ranges_of(int64_t units, int ntri, int xcd) {
    const int64_t lo = units * xcd / kXcds, cnt = units * (xcd + 1) / kXcds - lo;
    return {lo, cnt, cnt * ntri};
}

__global__ void __launch_bounds__(64 * kWaves, 2)
k_range_parts(const double* __restrict__ T, const double* __restrict__ R, int64_t stride, int n, int64_t ld,
              int64_t units, int nchunk, int ntile, int ntri, int G, double* __restrict__ part) {
    __shared__ __attribute__((aligned(1024))) char lds[kStages * kStageBytes];
    const int lane = threadIdx.x % 64, w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int xcd = (int)blockIdx.x % kXcds, r = (int)blockIdx.x / kXcds;
    const Ranges g = ranges_of(units, ntri, xcd);
    const int64_t end = g.total * (r + 1) / G;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
    const uint32_t ldsw = __builtin_amdgcn_readfirstlane(lds0 + w * kCopies * 1024);
    const int wm = w % 2, wn = w / 2;
    const double* M = w < 2 ? T : R;   // wavefronts 0, 1 copy the A rows, 2, 3 the B rows
    for (int64_t pos = g.total * r / G; pos < end;) {
        const int t = (int)(pos / g.units);
        const int64_t u = pos - (int64_t)t * g.units;
        const int count = (int)(end - pos < g.units - u ? end - pos : g.units - u);
        pos += count;
        int ti, tj;
        tile_at(t, ntile, ti, tj);
        // copy q of this wavefront: half q % 2 of the 16 x 16 block of rows 48 (w % 2) + 16 (q / 2); rows past
        // the matrix repeat its last one (their outputs are not stored)
        uint32_t voff[kCopies];
#pragma unroll
        for (int q = 0; q < kCopies; ++q) {
            int64_t row = (int64_t)(w < 2 ? ti : tj) * kBig + wm * kHalf + q / 2 * 16 + lane % 16;
            if (row >= n) row = n - 1;
            voff[q] = (uint32_t)((row * ld + 4 * (lane / 16) + 2 * (q % 2)) * (int64_t)sizeof(double));
        }
        int c = (int)((g.first + u) % nchunk);
        int64_t off = (g.first + u) / nchunk * stride + 16 * c;
        auto issue = [&](int k) {
            const uint32_t l = ldsw + (uint32_t)(k % kStages) * kStageBytes;
#pragma unroll
            for (int q = 0; q < kCopies; ++q) copy_1k(l + q * 1024, voff[q], M + off);
            off += 16;
            if (++c == nchunk) {
                c = 0;
                off += stride - 16 * (int64_t)nchunk;
            }
        };
        const int i0 = ti * kBig + wm * kHalf, j0 = tj * kBig + wn * kHalf;
        const bool live = i0 < j0 + kHalf && i0 < n && j0 < n;   // reaches the diagonal and the matrix
        f64x4 acc[3][3] = {};
        issue(0);
        if (count > 1) issue(1);
        for (int k = 0; k < count; ++k) {
            if (k + 1 < count) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(kCopies) : "memory");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (k + 2 < count) issue(k + 2);
            if (!live) continue;
            const char* st = lds + (k % kStages) * kStageBytes + lane * 16;
            f64x2 a[3][2], b[3][2];
#pragma unroll
            for (int f = 0; f < 3; ++f)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    a[f][h] = *(const f64x2*)(st + (wm * kCopies + 2 * f + h) * 1024);
                    b[f][h] = *(const f64x2*)(st + ((2 + wn) * kCopies + 2 * f + h) * 1024);
                }
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int f = 0; f < 3; ++f)
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        acc[f][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[f][s / 2][s % 2], b[q][s / 2][s % 2],
                                                                         acc[f][q], 0, 0, 0);
        }
        if (live) {
            double* out = part + ((int64_t)xcd * (G + ntri) + r + t) * kPart + w * (kPart / 4) + lane;
#pragma unroll
            for (int f = 0; f < 3; ++f)
#pragma unroll
                for (int q = 0; q < 3; ++q)
#pragma unroll
                    for (int x = 0; x < 4; ++x) out[((f * 3 + q) * 4 + x) * 64] = acc[f][q][x];
        }
        // the next piece's copies overwrite stages that are still read, and count their own arrivals
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    }
}

// One work-group per 16 x 48 band f of a tile's wavefront block.
__global__ void __launch_bounds__(256)
k_range_fix(const double* __restrict__ part, int n, int64_t ld, int64_t units, int ntile, int ntri, int G,
            const double* __restrict__ R0, double* __restrict__ D, int64_t ldd) {
    __shared__ double out[16][kHalf + 1];
    const int t = (int)blockIdx.x / 12, w = (int)blockIdx.x % 12 / 3, f = (int)blockIdx.x % 3;
    int ti, tj;
    tile_at(t, ntile, ti, tj);
    const int i0 = ti * kBig + w % 2 * kHalf + f * 16, j0 = tj * kBig + w / 2 * kHalf;
    if (i0 - f * 16 >= j0 + kHalf || i0 >= n || j0 >= n) return;
    // element 256 e + thread of the band: register (q, x) = (.. / 4, .. % 4) of lane .. % 64
    double sum[3] = {0.0, 0.0, 0.0}, r0[3];
    int row[3], col[3];
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        const int reg = (256 * e + (int)threadIdx.x) / 64, lane = threadIdx.x % 64;
        row[e] = 4 * (reg % 4) + lane / 16;
        col[e] = 16 * (reg / 4) + lane % 16;
        const bool in = i0 + row[e] < n && j0 + col[e] < n;
        r0[e] = in ? R0[(int64_t)(i0 + row[e]) * ld + j0 + col[e]] : 0.0;
    }
    for (int xcd = 0; xcd < kXcds; ++xcd) {
        const Ranges g = ranges_of(units, ntri, xcd);
        if (g.units == 0) continue;
        // ranges that hold the tile's first and last unit: the largest r with total r / G <= position
        const int64_t first = t * g.units, last = first + g.units - 1;
        const int ra = (int)(((first + 1) * G + g.total - 1) / g.total - 1);
        const int rb = (int)(((last + 1) * G + g.total - 1) / g.total - 1);
        const double* p = part + ((int64_t)xcd * (G + ntri) + t) * kPart + w * (kPart / 4) + f * 12 * 64 + threadIdx.x;
        for (int r = ra; r <= rb; r += 4) {
            double v[4][3];
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int e = 0; e < 3; ++e) v[k][e] = p[(int64_t)(r + k <= rb ? r + k : rb) * kPart + 256 * e];
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int e = 0; e < 3; ++e) sum[e] += r + k <= rb ? v[k][e] : 0.0;
        }
    }
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        const double v = sum[e] + r0[e];
        const int i = i0 + row[e], j = j0 + col[e];
        out[row[e]][col[e]] = v;
        if (i <= j && j < n) D[(int64_t)i * ldd + j] = v;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        const int at = 256 * e + (int)threadIdx.x, i = at % 16, j = at / 16;
        if (i0 + i < j0 + j && j0 + j < n) D[(int64_t)(j0 + j) * ldd + i0 + i] = out[i][j];
    }
}

hipError_t launch_ranges(const double* T, const double* R, int64_t stride, int prods, const double* R0, int64_t n,
                         int64_t ld, double* D, int64_t ldd, double* part, size_t part_bytes, hipStream_t st) {
    const int ntile = (int)((n + kBig - 1) / kBig), nchunk = (int)((n + 15) / 16);
    // 32-bit byte offsets inside a matrix, matrices and rows 16-byte aligned
    if (n < 1 || prods < 1 || !part || (int64_t)nchunk * 16 > ld || ld % 2 != 0 || ld * ld * 8 > (int64_t)1 << 31)
        return hipErrorInvalidValue;
    const int ntri = ntile * (ntile + 1) / 2;
    const int64_t units = (int64_t)prods * nchunk;
    // 64 ranges an XCD (two work-groups on each of its 32 CUs) of at least eight chunks
    int64_t G = units * ntri / (8 * kXcds);
    if (G > 64) G = 64;
    if (G < 1) G = 1;
    if ((int64_t)(part_bytes / (kXcds * kPart * sizeof(double))) < G + ntri) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_range_parts, dim3((unsigned)(kXcds * G)), dim3(64 * kWaves), 0, st, T, R, stride, (int)n, ld,
                       units, nchunk, ntile, ntri, (int)G, part);
    hipLaunchKernelGGL(k_range_fix, dim3((unsigned)(12 * ntri)), dim3(256), 0, st, (const double*)part, (int)n, ld,
                       units, ntile, ntri, (int)G, R0, D, ldd);
    return hipGetLastError();
}

}  // namespace

// 32-tiles up to N = 560, of which more wavefronts fit a SIMD; 48-tiles to 700 (where the matrices' padding
// holds their last one), fewer operand bytes per product; then the ranges of 96-tiles, whose padding
// and pieces cost more below.  mu search and D of order 512 with chains / 32- / 48-tiles / ranges, us: N = 400
// 495 / 428 / 436 / -, 500 673 / 588 / 597 / -, 600 792 / 713 / 685 / 699, 700 958 / 928 / 876 / 870, 800 1330 / 1271 /
// 1172 / 1160, 1000 1805 / 1905 / 1671 / 1629, 1100 2285 / 2440 / 2135 / 2058; chains on the int8 units / ranges, 1200
// 2612 / 2513, 1340 3208 / 3091, order 2000 6375 / 6333.
hipError_t launch_product_sum(const double* T, const double* R, int64_t stride, int prods, const double* R0, int64_t n,
                              int64_t ld, double* D, int64_t ldd, void* scratch, size_t scratch_bytes, hipStream_t st) {
    double* part = static_cast<double*>(scratch);
    if (n > 700) return launch_ranges(T, R, stride, prods, R0, n, ld, D, ldd, part, scratch_bytes, st);
    if (n > 560 && (n + 47) / 48 * 48 <= ld)
        return launch<3, 2>(T, R, stride, prods, R0, n, ld, D, ldd, part, scratch_bytes, st);
    return launch<2, 4>(T, R, stride, prods, R0, n, ld, D, ldd, part, scratch_bytes, st);
}

}  // namespace chebdm
