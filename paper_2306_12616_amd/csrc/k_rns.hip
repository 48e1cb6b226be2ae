// Float64 matrix products on the int8 MFMA units, by residue arithmetic.
//
// The float64 MFMA unit of gfx950 has a peak of 78.6 TFLOP/s and the product kernels of
// k_gemm.hip already run at 82-85 % of it at N = 4000; the int8 unit has 64 times that peak.
// A product of two matrices of integers below 2^57 is a sum below 2^114, so it is determined by
// its residues modulo coprime moduli whose product P exceeds 2^115 (Chinese remainder theorem),
// and modulo p <= 256 both operands are int8 matrices.  This is the integer modular technique of
// the "Ozaki scheme II" (Ozaki, Uchino, Imamura, 2025); the code is written from the mathematics:
//
//   scale   row r of an operand (symmetric, so also column r) gets the power of two 2^e_r above its
//           2-norm (a Chebyshev matrix of a spectrum known to lie in [-1, 1] has none above 1: e_r = 0
//           without a pass over it); q = rint(x 2^(57 - e_r)), so every row of q has 2-norm <= 2^57 and by
//           Cauchy-Schwarz every entry of a product stays below 2^114.
//   split   15 residue planes q mod p_m (int8), laid out as the MFMA operand fragments.
//   gemm    one int8 product per modulus, exact in int32; the epilogue reduces mod p_m to a byte.
//   join    CRT: value / P = sum_m r_m frac(inv_m / p_m) mod 1 in fixed point with 72 fraction
//           bits, then the product's float64 epilogue Out = alpha AB + beta C + gamma E + delta I.
//
// Everything between the two roundings (of q, 2^-58 of the row's norm, and of the joined value to
// float64) is exact, so a product's error is 2^-57-ish |row of A| |row of B|, below the rounding
// a float64 accumulation over K collects (measured against 113-bit sums, n = 4000, entries
// N(0, 1/n): 1.8e-16 against 5.5e-15).  A row that holds NaN or Inf gets a NaN scale and gives NaN
// in its whole row and column, as its dot products do.
//
// As in k_gemm.hip only tiles on and above the diagonal are computed and every value is stored
// at (i, j) and (j, i), so outputs stay exactly symmetric.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "internal.h"
#include "lds_copy.h"

namespace chebdm {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int NM = kRnsModuli;
constexpr int kBits = 57;
// Pairwise coprime, product 2^116.5 (> 2^115: sums below 2^114 of either sign, with 1.5 bits to
// spare: rows of norm 1 + rounding at e_r = 0 are far inside them).  Besides 256, whose residues wrap in a byte by themselves, none is above 237: the
// rounded quotient of the one-step reduction in the gemm is then close enough to keep the
// residue inside a byte up to K = 5120 (see reduce()).
constexpr int kMod[NM] = {256, 237, 235, 233, 229, 227, 223, 221, 217, 211, 209, 199, 197, 193, 191};
constexpr int64_t kOneStepK = 5120;

struct Tab {
    int p[16];
    float inv[16];
    uint32_t wlo[16], whi[16];   // balanced residues of 256^j and 2^30 256^j, j = 0..3, packed int8
    uint32_t crt[9][4];          // digit b (base 256, balanced, most significant first) of frac(inv_m / p_m)
    double p_hi, p_lo;           // P 2^-114 = p_hi + p_lo
};

constexpr uint32_t pack4(const int* d) {
    return (uint32_t)(d[0] & 255) | ((uint32_t)(d[1] & 255) << 8) | ((uint32_t)(d[2] & 255) << 16) |
           ((uint32_t)(d[3] & 255) << 24);
}
constexpr int balanced(unsigned long long x, int p) {
    const int r = (int)(x % (unsigned)p);
    return r >= (p + 1) / 2 ? r - p : r;
}

constexpr Tab make_tab() {
    Tab t{};
    unsigned __int128 P = 1;
    for (int i = 0; i < NM; ++i) P *= (unsigned)kMod[i];
    int dig[9][16] = {};
    for (int i = 0; i < NM; ++i) {
        const int p = kMod[i];
        t.p[i] = p;
        t.inv[i] = 1.0f / (float)p;
        int lo[4] = {}, hi[4] = {};
        for (int j = 0; j < 4; ++j) {
            lo[j] = balanced(1ull << (8 * j), p);
            hi[j] = balanced(1ull << (30 + 8 * j), p);
        }
        t.wlo[i] = pack4(lo);
        t.whi[i] = pack4(hi);
        int m = 1, inv = 1;   // inv = (P / p)^-1 mod p
        for (int j = 0; j < NM; ++j)
            if (j != i) m = m * (kMod[j] % p) % p;
        while (m * inv % p != 1) ++inv;
        unsigned __int128 c = ((((unsigned __int128)inv) << 72) + (unsigned)(p / 2)) / (unsigned)p;
        for (int b = 8; b >= 0; --b) {   // the carry out of the top digit is a whole number: dropped (mod 1)
            int x = (int)(c & 255);
            c >>= 8;
            if (x >= 128) {
                x -= 256;
                c += 1;
            }
            dig[b][i] = x;
        }
    }
    for (int b = 0; b < 9; ++b)
        for (int q = 0; q < 4; ++q) t.crt[b][q] = pack4(&dig[b][4 * q]);
    const double scale = 1.0 / 1298074214633706907132624082305024.0;   // 2^-110
    t.p_hi = (double)(unsigned long long)(P >> 64) * 18446744073709551616.0 * scale / 16.0;
    t.p_lo = (double)(unsigned long long)P * scale / 16.0;
    return t;
}
__constant__ const Tab kTab = make_tab();

constexpr float kMagic = 12582912.0f;   // 1.5 * 2^23: adding it rounds to an integer

// a mod p as a byte (low 8 bits of the result).  q = rint(a / p) comes out of a float32 fma with
// the magic number; its bits' low 24 are 2^22 + q, and p 2^22 vanishes in the low byte, so
// mad24(bits, -p, a) has the byte of a - p q.  |a - p q| <= p (1/2 + err), err = the float32
// rounding of a and of 1 / p: for K <= 5120 (|a| <= 118^2 K) at most 0.035, so the residue stays
// below 127.5 for p <= 237; p = 256 needs no bound.  Longer sums reduce twice.
template <bool TWICE>
__device__ __forceinline__ uint32_t reduce(int a, float inv, int np) {
    if constexpr (TWICE) {
        const float q = fmaf((float)a, inv, kMagic) - kMagic;
        a += np * (int)q;
    }
    const uint32_t qb = __float_as_uint(fmaf((float)a, inv, kMagic));
    return (uint32_t)(__mul24((int)qb, np) + a);
}

__device__ __forceinline__ uint32_t low_bytes(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
    const uint32_t x = __builtin_amdgcn_perm(b, a, 0x0c0c0400), y = __builtin_amdgcn_perm(d, c, 0x0c0c0400);
    return x | (y << 16);
}

__device__ __forceinline__ int xcd_order(int lin, int total) {
    const int q = total / 8, r = total % 8;
    const int x = lin % 8, slot = lin / 8;
    return x * q + (x < r ? x : r) + slot;
}

// Tile t of the BM x BN tiles (BM = R BN) that reach the diagonal or lie above it, in groups of
// kGroup tile rows, column by column inside a group: work-groups that run together then share
// about kGroup row panels and few column panels in their XCD's L2 (128-tiles, N = 4000: 504 us
// row by row, 457 in groups of 4).
constexpr int kGroup = 4;
template <int R>
__device__ __forceinline__ void tile_rc(int t, int ntr, int ntc, int& ti, int& tj) {
    ti = tj = 0;
    for (int r0 = 0; r0 < ntr; r0 += kGroup) {
        const int rows = ntr - r0 < kGroup ? ntr - r0 : kGroup;
        const int cnt = rows * ntc - R * (rows * r0 + rows * (rows - 1) / 2);
        if (t >= cnt) {
            t -= cnt;
            continue;
        }
        for (int v = 1; v < rows; ++v) {   // columns that only the group's first v rows reach
            if (t < R * v) {
                ti = r0 + t % v;
                tj = R * (r0 + v - 1) + t / v;
                return;
            }
            t -= R * v;
        }
        ti = r0 + t % rows;
        tj = R * (r0 + rows - 1) + t / rows;
        return;
    }
}

// ------------------------------------------------------------------------------ scale and split

struct ScaleArgs {
    const double* A[kRnsGroup];
    double* scale[kRnsGroup];
};
struct SplitArgs {
    const double* A[kRnsGroup];
    int8_t* planes[kRnsGroup];
    const double* scale[kRnsGroup];
};

// One wavefront per row: the power of two above the row's 2-norm.  One pass over the matrix, bound
// by its bytes (N = 2000: 5.3 us each).
__global__ void __launch_bounds__(256) k_rns_scale(const ScaleArgs a, int64_t n, int64_t ld, int64_t rows) {
    const int64_t row = (int64_t)blockIdx.x * 4 + threadIdx.x / 64;
    const int lane = threadIdx.x % 64;
    if (row >= rows) return;
    const double* A = a.A[blockIdx.y] + row * ld;
    double s = 0.0;
    if (row < n)
        for (int64_t j = 2 * lane; j < n; j += 128) {   // the padding up to ld (even) is zero
            const double2 v = *(const double2*)(A + j);
            s = fma(v.x, v.x, s);
            s = fma(v.y, v.y, s);
        }
    for (int o = 32; o; o >>= 1) s += __shfl_xor(s, o);
    double up = 1.0, down = 1.0;
    if (s >= 1e-270 && s <= 1e270) {
        const int e = (ilogb(s) >> 1) + 1;
        up = ldexp(1.0, kBits - e);
        down = ldexp(1.0, e);
    } else if (row < n) {
        // squares near the ends of the float64 range: scale by the largest entry first
        double mx = 0.0;
        int bad = 0;
        for (int64_t j = lane; j < n; j += 64) {
            const double v = fabs(A[j]);
            bad |= !(v <= 1.7976931348623157e308);
            mx = fmax(mx, v);
        }
        for (int o = 32; o; o >>= 1) {
            mx = fmax(mx, __shfl_xor(mx, o));
            bad |= __shfl_xor(bad, o);
        }
        if (bad) {
            up = down = __builtin_nan("");
        } else if (mx > 0.0) {
            const int em = ilogb(mx);
            double t = 0.0;
            for (int64_t j = lane; j < n; j += 64) {
                const double v = ldexp(A[j], -em);
                t = fma(v, v, t);
            }
            for (int o = 32; o; o >>= 1) t += __shfl_xor(t, o);
            int e = em + (ilogb(t) >> 1) + 1;
            if (e < -900) e = -900;   // 2^(57 - e) stays finite; entries below 2^-958 count as zero
            up = ldexp(1.0, kBits - e);
            down = ldexp(1.0, e);
        }
    }
    if (lane == 0) {
        double2* o = (double2*)a.scale[blockIdx.y] + row;
        *o = make_double2(up, down);
    }
}

// Residue planes in fragment order: a chunk is 16 rows x 64 k = 1 KB, lane l of the MFMA operand
// holding row l % 16 and 16 k's.  Which 16 is free as long as both operands agree: byte 2 i + c of
// lane group g is k = 8 i + 2 g + c, so that the four lanes of a row read 64 contiguous bytes.
// The 57-bit integer is cut into q = hi 2^30 + lo and both into balanced base-256 digits; one
// dot product of four digits with the residues of their weights per half gives q mod p + p * small.
__global__ void __launch_bounds__(256) k_rns_split(const SplitArgs a, int64_t n, int64_t ld, int64_t rows, int kt,
                                                   int64_t plane_bytes) {
    const int kb = blockIdx.x * 4 + threadIdx.x / 64, rb = blockIdx.y, lane = threadIdx.x % 64;
    if (kb >= kt) return;
    const int64_t row = (int64_t)rb * 16 + lane % 16;
    const int64_t k0 = (int64_t)kb * 64 + (lane / 16) * 2;
    const double* scale = a.scale[blockIdx.z];
    const double s = scale ? scale[2 * row] : 0x1p57;
    const double* A = a.A[blockIdx.z] + row * ld + k0;
    uint32_t lo[16], hi[16];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        double2 v = {0.0, 0.0};
        if (row < n && k0 + 8 * i < n) v = *(const double2*)(A + 8 * i);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const double x = (c ? v.y : v.x) * s;
            const double h = __builtin_rint(x * 0x1p-30);
            const double l = __builtin_rint(fma(h, -0x1p30, x));
            hi[2 * i + c] = ((uint32_t)(int)h + 0x80808080u) ^ 0x80808080u;
            lo[2 * i + c] = ((uint32_t)(int)l + 0x80808080u) ^ 0x80808080u;
        }
    }
    int8_t* out = a.planes[blockIdx.z] + ((int64_t)rb * kt + kb) * 1024 + lane * 16;
    for (int m = 0; m < NM; ++m) {
        const int wl = (int)kTab.wlo[m], wh = (int)kTab.whi[m], np = -kTab.p[m];
        const float inv = kTab.inv[m];
        v4i w;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int t = __builtin_amdgcn_sdot4((int)lo[4 * q + i], wl, 0, false);
                b[i] = reduce<false>(__builtin_amdgcn_sdot4((int)hi[4 * q + i], wh, t, false), inv, np);
            }
            w[q] = (int)low_bytes(b[0], b[1], b[2], b[3]);
        }
        *(v4i*)(out + (int64_t)m * plane_bytes) = w;
    }
}

// ------------------------------------------------------------------------------ int8 products

struct GemmArgs {
    const int8_t* A[kRnsGroup];
    const int8_t* B[kRnsGroup];
};

// Work-group: WM x WN wavefronts of TM x TN fragments (16 x 16), K in steps of 64, S LDS stages.
// Step k waits for its own copies of stage k, passes the barrier (stage k is then complete and
// everyone has read stage k - 1: its reads end before the wait), starts the copies of stage
// k + S - 1 into the buffer of stage k - 1 and multiplies.  Operands come in fragment order, so
// LDS reads are 16 contiguous bytes a lane: no bank conflicts.  A wavefront whose block lies below
// the diagonal copies for the others and multiplies nothing (the join never reads its residues).
// Bound by the power of the matrix units and by LDS and copy traffic together (N = 4000, one product,
// int8 rate executed: 2.29 POP/s with 128 x 128 tiles, three work-groups a CU, 2.39 with these; the vendor library's
// int8 GEMM at 4096: 2.08; the 128-tile loop without copies 3.3, without LDS reads too 3.6; zero
// operands alone, which switch less, gave 16 %).  The wavefront's 64 x 128 block, against 64 x 64, reads
// a quarter less LDS per product.  mu search and D of order 512, N = 2000 / 2500 / 3000 / 4000 / 4600:
// 256 x 128 tiles of eight 64 x 64 wavefronts (128-tiles at 2000 and 2500) 7.23 / 12.86 / 19.1 / 39.1 /
// 56.9 ms; of four 64 x 128 wavefronts 7.12 / 12.15 / 19.0 / 39.0 / 56.4, and without the blocks below
// the diagonal 7.00 / 12.11 / 18.8 / 38.6 / 55.9.  Four of 128 x 64: 7.18 at 2000, 39.8 at 4000; 256 x 256
// tiles of eight 128 x 64 7.37 and 39.7, of sixteen 64 x 64 7.31 and 38.4.
template <int WM, int WN, int TM, int TN, int S, int OCC, bool TWICE>
__global__ void __launch_bounds__(64 * WM * WN, OCC)
k_rns_gemm(const GemmArgs g, int64_t plane_bytes, int kt, int ntr, int ntc, int ntiles, int8_t* res) {
    constexpr int CH = WM * TM + WN * TN, CW = CH / (WM * WN), STAGE = CH * 1024;
    static_assert(CH % (WM * WN) == 0 && S >= 3 && TM % 4 == 0, "");
    __shared__ __attribute__((aligned(1024))) char lds[S * STAGE];
    const int lane = threadIdx.x % 64, w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int lin = xcd_order((int)blockIdx.x, (int)gridDim.x);
    const int t = lin % ntiles, m = lin / ntiles % NM, z = lin / ntiles / NM;
    int ti, tj;
    tile_rc<WM * TM / (WN * TN)>(t, ntr, ntc, ti, tj);
    const int8_t* src[CW];
#pragma unroll
    for (int c = 0; c < CW; ++c) {
        const int cc = w * CW + c;
        const bool a = cc < WM * TM;
        src[c] = (a ? g.A[z] : g.B[z]) + (int64_t)m * plane_bytes +
                 (int64_t)(a ? ti * WM * TM + cc : tj * WN * TN + (cc - WM * TM)) * kt * 1024;
    }
    const uint32_t voff = lane * 16;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
    const uint32_t ldsw = __builtin_amdgcn_readfirstlane(lds0 + w * CW * 1024);
    auto issue = [&](int k) {
        const uint32_t l = ldsw + (uint32_t)(k % S) * STAGE;
#pragma unroll
        for (int c = 0; c < CW; ++c) copy_1k(l + c * 1024, voff + (uint32_t)k * 1024u, src[c]);
    };
    const int wm = w % WM, wn = w / WM;
    const bool live = (ti * WM + wm) * TM < (tj * WN + wn + 1) * TN;   // not wholly below the diagonal
    v4i acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = (v4i){0, 0, 0, 0};
    const int abase = wm * TM * 1024 + lane * 16, bbase = (WM * TM + wn * TN) * 1024 + lane * 16;
#pragma unroll
    for (int k = 0; k < S - 1; ++k)
        if (k < kt) issue(k);
    for (int k = 0; k < kt; ++k) {
        if (k + S - 2 < kt) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((S - 2) * CW) : "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (k + S - 1 < kt) issue(k + S - 1);
        if (!live) continue;
        const char* st = lds + (k % S) * STAGE;
        v4i a[TM], b[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i) a[i] = *(const v4i*)(st + abase + i * 1024);
#pragma unroll
        for (int j = 0; j < TN; ++j) b[j] = *(const v4i*)(st + bbase + j * 1024);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    if (!live) return;
    // Residues as bytes.  A lane holds rows 4 (l / 16) + r of column l % 16 of each 16 x 16 block;
    // four blocks down make 16 bytes: one 1 KB store per 64 x 16 block of the output.
    const float inv = kTab.inv[m];
    const int np = -kTab.p[m];
    constexpr int RG = WM * TM / 4, CB = WN * TN;
    int8_t* out = res + (((int64_t)z * ntiles + t) * NM + m) * (int64_t)(RG * CB * 1024) + lane * 16;
#pragma unroll
    for (int i = 0; i < TM / 4; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            v4i o;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const v4i v = acc[4 * i + q][j];
                o[q] = (int)low_bytes(reduce<TWICE>(v[0], inv, np), reduce<TWICE>(v[1], inv, np),
                                      reduce<TWICE>(v[2], inv, np), reduce<TWICE>(v[3], inv, np));
            }
            *(v4i*)(out + ((wm * (TM / 4) + i) * CB + (wn * TN + j)) * 1024) = o;
        }
}

// ------------------------------------------------------------------------------ join

struct JoinArgs {
    RnsProduct d[kRnsGroup];
};

// One wavefront per 64 x 16 block: 15 coalesced 16-byte loads a lane hold the residues of 16
// entries, byte permutes gather each entry's 16 residues (the 16th is zero), and dot products of
// four bytes with the CRT constants' digits give the nine digit sums of value / P.  The top four
// are added with wrap-around (mod 1); |value / P| < 1/4, so the rest cannot carry over.
template <int BM, int BN>
__global__ void __launch_bounds__(256)
k_rns_join(const JoinArgs jn, int64_t n, int64_t ld, int ntr, int ntc, int ntiles, const int8_t* res) {
    constexpr int RG = BM / 64, CB = BN / 16, NB = RG * CB / 4;
    const int lane = threadIdx.x % 64;
    const RnsProduct& d = jn.d[blockIdx.y];
    const int t = blockIdx.x / NB, blk = blockIdx.x % NB;
    const int rg = blk / (CB / 4), cb = (blk % (CB / 4)) * 4 + threadIdx.x / 64;
    int ti, tj;
    tile_rc<BM / BN>(t, ntr, ntc, ti, tj);
    const int64_t i0 = (int64_t)ti * BM + rg * 64, j0 = (int64_t)tj * BN + cb * 16;
    if (i0 > j0 + 15 || i0 >= n || j0 >= n) return;
    const int8_t* src = res + (((int64_t)blockIdx.y * ntiles + t) * NM * (RG * CB) + rg * CB + cb) * 1024 + lane * 16;
    v4i r[16];
#pragma unroll
    for (int m = 0; m < NM; ++m) r[m] = *(const v4i*)(src + (int64_t)m * (RG * CB * 1024));
    r[15] = (v4i){0, 0, 0, 0};
    const int64_t j = j0 + lane % 16;
    const bool jin = j < n;
    const double sb = !jin ? 0.0 : d.scale_b ? d.scale_b[2 * j + 1] : 1.0;
    const bool whole = i0 + 63 < j0 && i0 + 63 < n && d.vec;   // off the diagonal, aligned rows
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        uint32_t e[4][4];   // [row][four moduli]
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const uint32_t a = r[4 * g][q], b = r[4 * g + 1][q], c = r[4 * g + 2][q], f = r[4 * g + 3][q];
            const uint32_t ab0 = __builtin_amdgcn_perm(b, a, 0x05010400), ab1 = __builtin_amdgcn_perm(b, a, 0x07030602);
            const uint32_t cf0 = __builtin_amdgcn_perm(f, c, 0x05010400), cf1 = __builtin_amdgcn_perm(f, c, 0x07030602);
            e[0][g] = __builtin_amdgcn_perm(cf0, ab0, 0x05040100);
            e[1][g] = __builtin_amdgcn_perm(cf0, ab0, 0x07060302);
            e[2][g] = __builtin_amdgcn_perm(cf1, ab1, 0x05040100);
            e[3][g] = __builtin_amdgcn_perm(cf1, ab1, 0x07060302);
        }
        const int64_t ib = i0 + q * 16 + (lane / 16) * 4;
        double o[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            int s[9];
#pragma unroll
            for (int b = 0; b < 9; ++b) {
                int v = 0;
#pragma unroll
                for (int g = 0; g < 4; ++g) v = __builtin_amdgcn_sdot4((int)e[x][g], (int)kTab.crt[b][g], v, false);
                s[b] = v;
            }
            const int top = (int)(((uint32_t)s[0] << 24) + ((uint32_t)s[1] << 16) + ((uint32_t)s[2] << 8) + (uint32_t)s[3]);
            const int m1 = s[4] * 256 + s[5], m2 = s[6] * 256 + s[7];
            const double low = fma((double)m1, 0x1p-48, fma((double)m2, 0x1p-64, (double)s[8] * 0x1p-72));
            const double f = fma((double)top, 0x1p-32, low);
            const int64_t i = ib + x;
            o[x] = 0.0;
            if (i < n && jin) {
                const double sa = d.scale_a ? d.scale_a[2 * i + 1] : 1.0;
                double v = d.alpha * (fma(f, kTab.p_hi, f * kTab.p_lo) * sa * sb);
                if (d.C) v = fma(d.beta, d.C[i * ld + j], v);
                if (d.E) v = fma(d.gamma, d.E[i * ld + j], v);
                if (i == j) v += d.delta;
                o[x] = v;
            }
        }
        if (whole) {
            if (jin) {
#pragma unroll
                for (int x = 0; x < 4; ++x) d.Out[(ib + x) * d.ld_out + j] = o[x];
                double2* mo = (double2*)(d.Out + j * d.ld_out + ib);
                mo[0] = make_double2(o[0], o[1]);
                mo[1] = make_double2(o[2], o[3]);
            }
        } else {
#pragma unroll
            for (int x = 0; x < 4; ++x)
                if (ib + x <= j && jin) {   // i <= j < n
                    d.Out[(ib + x) * d.ld_out + j] = o[x];
                    if (ib + x < j) d.Out[j * d.ld_out + ib + x] = o[x];
                }
        }
    }
}

}  // namespace

// 256 x 128 tiles from N = 1536, where their fewer copies outweigh the coarser last round of
// work-groups.  Order 512 with 128-tiles and with these, ms: mu search and D, N = 1400 3.36 and 3.39,
// 1600 4.66 and 4.56, 1800 6.32 and 6.09, 2200 9.65 and 9.15, 2700 15.6 and 14.8, 4000 41.4 and 38.6;
// fixed mu (one product a launch), N = 1400 2.88 and 3.03, 1600 3.66 and 3.68, 1800 4.69 and 4.60,
// 2000 5.36 and 5.45, 2200 6.99 and 6.79, 2900 12.9 and 12.1.
RnsGeom rns_geom(int64_t n) {
    RnsGeom g;
    g.n = n;
    g.big = n >= 1536;
    const int64_t bm = g.big ? 256 : 128, bn = 128;
    g.rows = (n + bm - 1) / bm * bm;
    g.kt = (int)((n + 63) / 64);
    g.plane_bytes = g.rows * g.kt * 64;
    g.set_bytes = g.plane_bytes * NM;
    g.ntr = (int)((n + bm - 1) / bm);
    g.ntc = (int)((n + bn - 1) / bn);
    g.ntiles = 0;
    for (int r = 0; r < g.ntr; ++r) {
        const int c = g.ntc - (int)(bm / bn) * r;
        if (c > 0) g.ntiles += c;
    }
    g.res_bytes = (int64_t)g.ntiles * bm * bn * NM;
    return g;
}

hipError_t launch_rns_scale(const RnsGeom& g, int64_t ld, const double* const* mats, double* const* scale, int count,
                            hipStream_t st) {
    if (count < 1 || count > kRnsGroup || ld < g.n || ld % 2 != 0) return hipErrorInvalidValue;
    ScaleArgs a{};
    for (int i = 0; i < count; ++i) {
        a.A[i] = mats[i];
        a.scale[i] = scale[i];
    }
    hipLaunchKernelGGL(k_rns_scale, dim3((unsigned)((g.rows + 3) / 4), (unsigned)count), dim3(256), 0, st, a, g.n, ld,
                       g.rows);
    return hipGetLastError();
}

hipError_t launch_rns_split(const RnsGeom& g, int64_t ld, const double* const* mats, int8_t* const* planes,
                            const double* const* scale, int count, hipStream_t st) {
    if (count < 1 || count > kRnsGroup || ld < g.n || ld % 2 != 0) return hipErrorInvalidValue;
    SplitArgs a{};
    for (int i = 0; i < count; ++i) {
        a.A[i] = mats[i];
        a.planes[i] = planes[i];
        a.scale[i] = scale[i];
    }
    hipLaunchKernelGGL(k_rns_split, dim3((unsigned)((g.kt + 3) / 4), (unsigned)(g.rows / 16), (unsigned)count),
                       dim3(256), 0, st, a, g.n, ld, g.rows, g.kt, g.plane_bytes);
    return hipGetLastError();
}

hipError_t launch_rns_products(const RnsGeom& g, int64_t ld, const RnsProduct* prods, int count, int8_t* res,
                               hipStream_t st) {
    if (count < 1 || count > kRnsGroup) return hipErrorInvalidValue;
    GemmArgs ga{};
    JoinArgs ja{};
    for (int i = 0; i < count; ++i) {
        ga.A[i] = prods[i].planes_a;
        ga.B[i] = prods[i].planes_b;
        ja.d[i] = prods[i];
        ja.d[i].vec = prods[i].ld_out % 2 == 0 && (uintptr_t)prods[i].Out % 16 == 0;
    }
    const dim3 items((unsigned)(g.ntiles * NM * count));
    const bool twice = (int64_t)g.kt * 64 > kOneStepK;
#define RNS_GEMM(WM, WN, TM, TN, OCC, TW)                                                                       \
    hipLaunchKernelGGL((k_rns_gemm<WM, WN, TM, TN, 3, OCC, TW>), items, dim3(64 * WM * WN), 0, st, ga, g.plane_bytes, \
                       g.kt, g.ntr, g.ntc, g.ntiles, res)
    if (g.big) {
        if (twice) RNS_GEMM(4, 1, 4, 8, 2, true);
        else RNS_GEMM(4, 1, 4, 8, 2, false);
        hipLaunchKernelGGL((k_rns_join<256, 128>), dim3((unsigned)(g.ntiles * 8), (unsigned)count), dim3(256), 0, st, ja,
                           g.n, ld, g.ntr, g.ntc, g.ntiles, (const int8_t*)res);
    } else {
        if (twice) RNS_GEMM(2, 2, 4, 4, 3, true);
        else RNS_GEMM(2, 2, 4, 4, 3, false);
        hipLaunchKernelGGL((k_rns_join<128, 128>), dim3((unsigned)(g.ntiles * 4), (unsigned)count), dim3(256), 0, st, ja,
                           g.n, ld, g.ntr, g.ntc, g.ntiles, (const int8_t*)res);
    }
#undef RNS_GEMM
    return hipGetLastError();
}

}  // namespace chebdm
