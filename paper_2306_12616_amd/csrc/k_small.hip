// Float64 products of small matrices.
//
// Below N ~ 500 a launch of the tiles of k_gemm.hip is a chain of latencies (16-19 us at N = 256 and
// 333 for work of about 1 us): each wavefront streams its K range through two register stages, and
// the epilogue loads its addends at the end.  Here a work-group owns a 32 x 32 or 16 x 16 tile and its eight
// wavefronts share K in chunks of 16; every operand load of a wavefront and the epilogue's C and E
// go out before the first MFMA, so a product costs one round of loads, a few MFMAs, one LDS sum over
// the wavefronts and the stores.  As in k_gemm.hip both operands are symmetric and read along rows
// (lane l: row l % 16, k = 16 c + 4 (l / 16) + s for the s-th MFMA of chunk c), only tiles on and
// above the diagonal are computed, and every value is stored at (i, j) and (j, i).  The workspace
// matrices are zero outside the n x n block, so nothing is predicated but the stores.
// Measured, whole calls: mu search + D N = 256 order 128 438 -> 285 us, fixed mu N = 333 order 200
// 362 -> 206.
#include "internal.h"

namespace chebdm {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

constexpr int kWaves = 8;

// F x F blocks of 16 x 16; MAXC: chunks of 16 a wavefront may own, n <= 128 MAXC.
template <int F, int MAXC>
__global__ void __launch_bounds__(64 * kWaves)
k_gemm_small(const GemmBatch<double> batch, int n, int64_t ld, int ntile, int nchunk) {
    constexpr int kTile = 16 * F, kRow = kTile + 1;   // LDS row padded for the transposed read
    constexpr int NT = 64 * kWaves, OUTS = (kTile * kTile + NT - 1) / NT;
    __shared__ double red[kWaves][kTile * kRow];
    const GemmDesc<double>& d = batch.d[blockIdx.y];
    const int lane = threadIdx.x % 64, w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    int ti = 0, t = blockIdx.x;
    while (t >= ntile - ti) t -= ntile - ti++;
    const int tj = ti + t, i0 = ti * kTile, j0 = tj * kTile;
    const int64_t lane_off = (int64_t)(lane % 16) * ld + 4 * (lane / 16);
    const double* A = d.A + (int64_t)i0 * ld + lane_off;
    const double* B = d.B + (int64_t)j0 * ld + lane_off;
    f64x2 a[MAXC][F][2], b[MAXC][F][2];   // [chunk][16-row block][half of the lane's four k]
#pragma unroll
    for (int u = 0; u < MAXC; ++u) {
        const int c = w + kWaves * u;
        if (c < nchunk) {
#pragma unroll
            for (int r = 0; r < F; ++r)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    a[u][r][h] = *(const f64x2*)(A + (int64_t)r * 16 * ld + 16 * c + 2 * h);
                    b[u][r][h] = *(const f64x2*)(B + (int64_t)r * 16 * ld + 16 * c + 2 * h);
                }
        }
    }
    // the outputs this thread finishes (with 16 x 16 tiles the second half of the threads has none),
    // and their addends
    double add[OUTS];
#pragma unroll
    for (int h = 0; h < OUTS; ++h) {
        const int e = (threadIdx.x + NT * h) % (kTile * kTile);
        const int64_t at = (int64_t)(i0 + e / kTile) * ld + j0 + e % kTile;
        const double c = d.C ? d.C[at] : 0.0, g = d.E ? d.E[at] : 0.0;
        add[h] = fma(d.beta, c, d.gamma * g);
        if (i0 + e / kTile == j0 + e % kTile) add[h] += d.delta;
    }
    f64x4 acc[F][F] = {};
#pragma unroll
    for (int u = 0; u < MAXC; ++u) {
        if (w + kWaves * u < nchunk) {
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int r = 0; r < F; ++r)
#pragma unroll
                    for (int q = 0; q < F; ++q)
                        acc[r][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u][r][s / 2][s % 2], b[u][q][s / 2][s % 2],
                                                                         acc[r][q], 0, 0, 0);
        }
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
    double* Out = static_cast<double*>(d.Out);
#pragma unroll
    for (int h = 0; h < OUTS; ++h) {
        const int e = threadIdx.x + NT * h, i = e / kTile, j = e % kTile, at = i * kRow + j;
        if (e >= kTile * kTile) break;
        double s = red[0][at];
#pragma unroll
        for (int q = 1; q < kWaves; ++q) s += red[q][at];
        s = fma(d.alpha, s, add[h]);
        red[0][at] = s;   // only this thread has read it
        if (i0 + i <= j0 + j && j0 + j < n) Out[(int64_t)(i0 + i) * d.ld_out + j0 + j] = s;
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < OUTS; ++h) {
        const int e = threadIdx.x + NT * h, j = e / kTile, i = e % kTile;
        if (e >= kTile * kTile) break;
        if (i0 + i < j0 + j && j0 + j < n) Out[(int64_t)(j0 + j) * d.ld_out + i0 + i] = red[0][i * kRow + j];
    }
}

}  // namespace

namespace {

constexpr int64_t kMaxN = 16 * kWaves * 6;

int64_t tiles(int64_t n, int64_t edge) {
    const int64_t nt = (n + edge - 1) / edge;
    return nt * (nt + 1) / 2;
}

template <int F>
hipError_t launch(const GemmBatch<double>& b, int64_t n, int64_t ld, hipStream_t st) {
    const int nchunk = (int)((n + 15) / 16), ntile = (int)((n + 16 * F - 1) / (16 * F));
    if (nchunk * 16 > ld || ntile * 16 * F > ld) return hipErrorInvalidValue;
    const dim3 grid((unsigned)tiles(n, 16 * F), (unsigned)b.count), block(64 * kWaves);
#define SMALL(MAXC) hipLaunchKernelGGL((k_gemm_small<F, MAXC>), grid, block, 0, st, b, (int)n, ld, ntile, nchunk)
    if (n <= 128) SMALL(1);
    else if (n <= 256) SMALL(2);
    else if (n <= 384) SMALL(3);
    else if (n <= 512) SMALL(4);
    else SMALL(6);
#undef SMALL
    return hipGetLastError();
}

}  // namespace

// One round of work-groups of 32-tiles (a CU holds one or two).  Past it the larger tiles of
// k_gemm.hip re-use their operands more: mu search + D of order 200 at N = 512 (136 tiles) 593 us
// without this kernel, 532 with launches of up to two products on it, 571 with all; at N = 600 (190)
// 619, 599 and 656; fixed mu of order 512, one product a launch: N = 700 (253 tiles) 933 -> 765,
// N = 768 (300 tiles, two rounds) 994 -> 1221.
bool gemm_small_pays(int64_t n, int count) { return n <= kMaxN && tiles(n, 32) * count <= 280; }

// 16-tiles up to two a CU: a work-group's operand rows come in through one CU, so half as many rows a
// work-group take less time as long as idle CUs take the others.  Fixed mu of order 512 with
// 32-tiles and with 16-tiles: N = 64 215 -> 180 us, N = 256 (136 tiles of 16) 336 -> 256, N = 450
// (435) 485 -> 430, N = 512 (528) 538 -> 568.
hipError_t launch_gemm_small(const GemmBatch<double>& b, int64_t n, int64_t ld, hipStream_t st) {
    if (n < 1 || n > kMaxN || b.count < 1) return hipErrorInvalidValue;
    return tiles(n, 16) * b.count <= 480 ? launch<1>(b, n, ld, st) : launch<2>(b, n, ld, st);
}

}  // namespace chebdm
