// Learned chemical potential: the small network 64 -> 256 -> 256 -> 1 (ReLU,
// float32) that maps Chebyshev trace moments to mu~, trained on the GPU with
// these kernels.
//
// Every layer is local to a batch row except the weight gradients, so a pass is one launch over
// blocks of 16 rows (forward, loss, and the hidden layers' dZ), and the backward pass one more for
// all the weight gradients.  The products run on v_mfma_f32_16x16x4f32 (float32 inputs and sums);
// every sum has a fixed order: deterministic.  A minibatch is launch- and latency-bound: 256 rows
// are 16 work-groups, whose two 16 x 256 x 256 products take about 3.4 us each on one CU.
// Measured at 256 rows, forward + backward + Adam: 513 us with one SIMT kernel per layer, column sum
// and mask (13 launches), 58 us with these four (16 forward, 22 + 18 backward, 4 Adam).
#include "internal.h"
#include "reduce.h"

namespace chebdm {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// parameter offsets (floats)
constexpr int MLP_IN = 64, MLP_H = 256;
constexpr int64_t OFF_W1 = 0, OFF_B1 = OFF_W1 + MLP_H * MLP_IN, OFF_W2 = OFF_B1 + MLP_H,
                  OFF_B2 = OFF_W2 + MLP_H * MLP_H, OFF_W3 = OFF_B2 + MLP_H, OFF_B3 = OFF_W3 + MLP_H,
                  MLP_NPARAM = OFF_B3 + 1;

constexpr int RB = 16;            // batch rows of a work-group
constexpr int LDA = MLP_H + 4;    // LDS row of the activations (floats): 16-byte aligned, banks shifted by row

// Four floats; VEC: p is 16-byte aligned.
template <bool VEC>
__device__ __forceinline__ f32x4 load4(const float* p) {
    if constexpr (VEC) return *(const f32x4*)p;
    return (f32x4){p[0], p[1], p[2], p[3]};
}

// acc += A B for one 16 x 16 tile, K in chunks of 16: lane l holds row (column) l % 16 and
// k = 16 c + 4 (l / 16) + s of A (B); A from LDS rows, B from registers.  Two accumulators halve
// the chain of dependent MFMAs.
template <int CHUNKS>
__device__ __forceinline__ f32x4 tile_mm(const float* a_row, const f32x4* b) {
    f32x4 e = {0.0f, 0.0f, 0.0f, 0.0f}, o = e;
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
        const f32x4 a = *(const f32x4*)(a_row + 16 * c);
        e = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0], b[c][0], e, 0, 0, 0);
        o = __builtin_amdgcn_mfma_f32_16x16x4f32(a[1], b[c][1], o, 0, 0, 0);
        e = __builtin_amdgcn_mfma_f32_16x16x4f32(a[2], b[c][2], e, 0, 0, 0);
        o = __builtin_amdgcn_mfma_f32_16x16x4f32(a[3], b[c][3], o, 0, 0, 0);
    }
    return e + o;
}

// Sum over the 16 lanes of a row, in every lane (DPP row rotations).
template <int N>
__device__ __forceinline__ float row_ror(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 + N, 0xf, 0xf, true));
}
__device__ __forceinline__ float row_sum(float x) {
    x += row_ror<8>(x);
    x += row_ror<4>(x);
    x += row_ror<2>(x);
    return x + row_ror<1>(x);
}

// 16 wavefronts, one 16-column tile of a hidden layer each.  The weights of both layers are
// loaded before the first product needs them.  BWD: also A1, A2, dZ2 = dy w3 (A2 > 0),
// dZ1 = (dZ2 W2) (A1 > 0) to memory, dy = 2 (y - t) / Bn and the block's sum of (y - t)^2.
template <bool BWD, bool VEC>
__global__ void __launch_bounds__(1024)
k_mlp_rows(int Bn, const float* __restrict__ w, const float* __restrict__ X, const float* __restrict__ t,
           float* __restrict__ y, float* __restrict__ A1, float* __restrict__ A2, float* __restrict__ dZ2,
           float* __restrict__ dZ1, float* __restrict__ dy, double* __restrict__ loss_part) {
    __shared__ __attribute__((aligned(16))) float xs[RB][MLP_IN + 4];
    __shared__ __attribute__((aligned(16))) float hs[2][RB][LDA];
    __shared__ float part[16][RB];
    __shared__ float dys[RB];
    const int lane = threadIdx.x % 64, wv = threadIdx.x / 64, c = lane % 16, g = lane / 16;
    const int b0 = blockIdx.x * RB, col = wv * 16 + c;
    f32x4 w1[4], w2[16];
#pragma unroll
    for (int q = 0; q < 4; ++q) w1[q] = load4<VEC>(w + OFF_W1 + col * MLP_IN + 16 * q + 4 * g);
#pragma unroll
    for (int q = 0; q < 16; ++q) w2[q] = load4<VEC>(w + OFF_W2 + col * MLP_H + 16 * q + 4 * g);
    const float bias1 = w[OFF_B1 + col], bias2 = w[OFF_B2 + col], w3 = w[OFF_W3 + col];
    {
        const int r = threadIdx.x / MLP_IN, i = threadIdx.x % MLP_IN;   // 1024 = RB x MLP_IN
        xs[r][i] = b0 + r < Bn ? X[(size_t)(b0 + r) * MLP_IN + i] : 0.0f;
    }
    __syncthreads();
    // the result's lane l holds rows 4 (l / 16) + r of column l % 16
    f32x4 z = tile_mm<4>(&xs[c][4 * g], w1);
    float a1[4], a2[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        a1[r] = fmaxf(z[r] + bias1, 0.0f);
        hs[0][4 * g + r][col] = a1[r];
        if (BWD && b0 + 4 * g + r < Bn) A1[(size_t)(b0 + 4 * g + r) * MLP_H + col] = a1[r];
    }
    __syncthreads();
    z = tile_mm<16>(&hs[0][c][4 * g], w2);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        a2[r] = fmaxf(z[r] + bias2, 0.0f);
        if (BWD && b0 + 4 * g + r < Bn) A2[(size_t)(b0 + 4 * g + r) * MLP_H + col] = a2[r];
        const float s = row_sum(a2[r] * w3);
        if (c == 0) part[wv][4 * g + r] = s;
    }
    if constexpr (BWD) {   // B of the dZ1 product: W2 by columns
#pragma unroll
        for (int q = 0; q < 16; ++q)
#pragma unroll
            for (int s = 0; s < 4; ++s) w2[q][s] = w[OFF_W2 + (16 * q + 4 * g + s) * MLP_H + col];
    }
    __syncthreads();
    if (threadIdx.x < RB) {
        const int r = threadIdx.x;
        float v = w[OFF_B3];
        for (int q = 0; q < 16; ++q) v += part[q][r];
        const bool in = b0 + r < Bn;
        if (in) y[b0 + r] = v;
        if constexpr (BWD) {
            const float d = in ? v - t[b0 + r] : 0.0f;
            const float dv = 2.0f * d / (float)Bn;
            dys[r] = dv;
            if (in) dy[b0 + r] = dv;
            double s = (double)d * (double)d;
            for (int o = 8; o; o >>= 1) s += __shfl_xor(s, o);
            if (r == 0) loss_part[blockIdx.x] = s;
        }
    }
    if constexpr (BWD) {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float d = a2[r] > 0.0f ? dys[4 * g + r] * w3 : 0.0f;
            hs[1][4 * g + r][col] = d;
            if (b0 + 4 * g + r < Bn) dZ2[(size_t)(b0 + 4 * g + r) * MLP_H + col] = d;
        }
        __syncthreads();
        z = tile_mm<16>(&hs[1][c][4 * g], w2);
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (b0 + 4 * g + r < Bn) dZ1[(size_t)(b0 + 4 * g + r) * MLP_H + col] = a1[r] > 0.0f ? z[r] : 0.0f;
    }
}

// Weight gradients, one wavefront per work-group: items 0..255 are the 16 x 16 tiles of
// gW2 = dZ2^T A1, then 64 of gW1 = dZ1^T X, 16 of gw3 = A2^T dy (16 entries each), and one for
// gb3 and the loss.  The bias gradients are the column sums of dZ, taken by the first tile of
// each tile row from the operand it reads anyway.  The batch is the K dimension; the next
// 64 rows are loaded ahead of the MFMAs of the current ones.
constexpr int kGradItems = 256 + 64 + 16 + 1;

__global__ void __launch_bounds__(64)
k_mlp_grads(int Bn, const float* __restrict__ X, const float* __restrict__ A1, const float* __restrict__ A2,
            const float* __restrict__ dZ2, const float* __restrict__ dZ1, const float* __restrict__ dy,
            const double* __restrict__ loss_part, float* __restrict__ grad, float* __restrict__ loss) {
    const int lane = threadIdx.x, c = lane % 16, g = lane / 16;
    int it = blockIdx.x;
    if (it < 320) {
        const bool second = it < 256;
        const int nt = second ? 16 : 4, ld = second ? MLP_H : MLP_IN;
        if (!second) it -= 256;
        const int ti = it / nt, tj = it % nt;
        const float* P = (second ? dZ2 : dZ1) + ti * 16 + c;
        const float* Q = (second ? A1 : X) + tj * 16 + c;
        f32x4 e = {0.0f, 0.0f, 0.0f, 0.0f}, o = e;
        float sum = 0.0f;
        float p[2][16], q[2][16];
        auto load = [&](int b, float* pp, float* qq) {
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int bb = b + 4 * u + g;
                const bool in = bb < Bn;
                pp[u] = in ? P[(size_t)bb * MLP_H] : 0.0f;
                qq[u] = in ? Q[(size_t)bb * ld] : 0.0f;
            }
        };
        auto mul = [&](const float* pp, const float* qq) {
#pragma unroll
            for (int u = 0; u < 16; u += 2) {
                e = __builtin_amdgcn_mfma_f32_16x16x4f32(pp[u], qq[u], e, 0, 0, 0);
                o = __builtin_amdgcn_mfma_f32_16x16x4f32(pp[u + 1], qq[u + 1], o, 0, 0, 0);
                sum += pp[u] + pp[u + 1];
            }
        };
        load(0, p[0], q[0]);
        for (int b = 0; b < Bn; b += 128) {
            load(b + 64, p[1], q[1]);
            mul(p[0], q[0]);
            load(b + 128, p[0], q[0]);
            mul(p[1], q[1]);
        }
        float* G = grad + (second ? OFF_W2 : OFF_W1) + (size_t)(ti * 16 + 4 * g) * ld + tj * 16 + c;
#pragma unroll
        for (int r = 0; r < 4; ++r) G[(size_t)r * ld] = e[r] + o[r];
        if (tj == 0) {
            sum += __shfl_xor(sum, 16);
            sum += __shfl_xor(sum, 32);
            if (g == 0) grad[(second ? OFF_B2 : OFF_B1) + ti * 16 + c] = sum;
        }
    } else if (it < 336) {
        const float* P = A2 + (it - 320) * 16 + c;
        float sum = 0.0f;
        for (int b = g; b < Bn; b += 4) sum = fmaf(P[(size_t)b * MLP_H], dy[b], sum);
        sum += __shfl_xor(sum, 16);
        sum += __shfl_xor(sum, 32);
        if (g == 0) grad[OFF_W3 + (it - 320) * 16 + c] = sum;
    } else {
        float sum = 0.0f;
        for (int b = lane; b < Bn; b += 64) sum += dy[b];
        double ls = 0.0;
        for (int b = lane; b < (Bn + RB - 1) / RB; b += 64) ls += loss_part[b];
        for (int o = 32; o; o >>= 1) {
            sum += __shfl_xor(sum, o);
            ls += __shfl_xor(ls, o);
        }
        if (lane == 0) {
            grad[OFF_B3] = sum;
            *loss = (float)(ls / Bn);
        }
    }
}

__global__ void __launch_bounds__(256)
k_mlp_adam(int n, float* __restrict__ w, const float* __restrict__ g, float* __restrict__ m, float* __restrict__ v,
           float lr, float b1, float b2, float eps, float bc1, float bc2) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    w[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
}

// float4 loads of the weights where the caller's vector is 16-byte aligned (the layers' offsets are
// multiples of four floats)
template <bool BWD, class... Args>
hipError_t rows(hipStream_t st, int Bn, const float* w, Args... args) {
    const dim3 grid((unsigned)((Bn + RB - 1) / RB));
    if ((uintptr_t)w % 16 == 0)
        hipLaunchKernelGGL((k_mlp_rows<BWD, true>), grid, dim3(1024), 0, st, Bn, w, args...);
    else
        hipLaunchKernelGGL((k_mlp_rows<BWD, false>), grid, dim3(1024), 0, st, Bn, w, args...);
    return hipGetLastError();
}

}  // namespace

int64_t mlp_nparams() { return MLP_NPARAM; }

hipError_t launch_mlp_forward(const float* w, const float* X, int Bn, float* y, hipStream_t st) {
    return rows<false>(st, Bn, w, X, (const float*)nullptr, y, (float*)nullptr, (float*)nullptr, (float*)nullptr,
                       (float*)nullptr, (float*)nullptr, (double*)nullptr);
}

// work: loss sums of the row blocks (double), then A1, A2, dZ2, dZ1 (B x 256 each), y (B), dy (B)
hipError_t launch_mlp_backward(const float* w, const float* X, const float* t, int Bn, float* g, float* work,
                               float* loss, hipStream_t st) {
    double* lp = reinterpret_cast<double*>(work);
    float* A1 = work + 2 * (((int64_t)Bn + RB - 1) / RB);
    float* A2 = A1 + (size_t)Bn * MLP_H;
    float* dZ2 = A2 + (size_t)Bn * MLP_H;
    float* dZ1 = dZ2 + (size_t)Bn * MLP_H;
    float* y = dZ1 + (size_t)Bn * MLP_H;
    float* dy = y + Bn;
    hipError_t e;
    if ((e = rows<true>(st, Bn, w, X, t, y, A1, A2, dZ2, dZ1, dy, lp))) return e;
    hipLaunchKernelGGL(k_mlp_grads, dim3(kGradItems), dim3(64), 0, st, Bn, X, (const float*)A1, (const float*)A2,
                       (const float*)dZ2, (const float*)dZ1, (const float*)dy, (const double*)lp, g, loss);
    return hipGetLastError();
}

hipError_t launch_mlp_adam(float* w, const float* g, float* m, float* v, int64_t n, float lr, float b1, float b2,
                           float eps, float bc1, float bc2, hipStream_t st) {
    hipLaunchKernelGGL(k_mlp_adam, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (int)n, w, g, m, v, lr, b1,
                       b2, eps, bc1, bc2);
    return hipGetLastError();
}

}  // namespace chebdm
