// Operators of the operator-granular graph (the granularity of the paper's cost table, Sec. 5.5:
// ConvForward, BNForward, ... are separate managed tensors) for gfx950, bf16 NHWC:
//   training-mode batch normalisation   y = gamma (x - mu_B) / sqrt(var_B + eps) + beta
//   ReLU                                y = max(x, 0)
//   residual add                        y = x + r
// All three are HBM-bound (16 bytes per lane).  Batch normalisation reads x twice (statistics,
// then normalise) and writes y once:
//   bn_stats_kernel     each workgroup sums (x - K_c) and (x - K_c)^2 over its block of rows, per
//                       channel, fp32, K_c = x[0, c] (shifted data: no cancellation when the mean is
//                       far from 0); lanes own 8 channels, the row-parallel lanes of a workgroup are
//                       combined through LDS in row order (all lanes share that work); partial sums to a
//                       scratch buffer
//   bn_finalize_kernel  one thread per channel adds the partials in block order (double), forms
//                       mean, biased variance and a = gamma / sqrt(var + eps)
//   bn_tail_kernel      y = a_c (x - mean_c) + beta_c   (centred first: no cancellation of two large products); where the
//                       segment goes on with the residual add and / or the ReLU of that result, those too, in the same pass
// No atomics: the result is a fixed function of the input (recomputation is bit-identical).
// Backward of the batch normalisation (chain rule through the three lines above, collapsed):
//   gx = a_c (gy - mean(gy)_c - (x - mu_c) S_c / ((var_c + eps) M)),   S_c = sum gy (x - mu_c)
//   dgamma_c = S_c / sqrt(var_c + eps),   dbeta_c = sum gy
// reads x and gy twice and writes gx once, the floor without stored statistics (x has to be read
// for S_c in any case):
//   bn_bwd_stats_kernel     sums of (x - K_c), (x - K_c)^2, gy, gy (x - K_c) per channel and workgroup; where gy is the
//                           gradient that the ReLU before it in the segment leaves, its mask is applied and stored here
//   bn_bwd_finalize_kernel  adds the partials (double), forms a, mu, mean(gy), S/((var + eps) M) and
//                           the two parameter gradients
//   bn_bwd_apply_kernel     gx from x, gy and the four per-channel factors
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"

namespace delta {
namespace ops {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float lo16(uint32_t p) { return __uint_as_float(p << 16); }
__device__ __forceinline__ float hi16(uint32_t p) { return __uint_as_float(p & 0xFFFF0000u); }
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ void unpack8(const u32x4 v, float (&f)[8]) {
    f[0] = lo16(v.x); f[1] = hi16(v.x); f[2] = lo16(v.y); f[3] = hi16(v.y);
    f[4] = lo16(v.z); f[5] = hi16(v.z); f[6] = lo16(v.w); f[7] = hi16(v.w);
}

// g where m > 0, else 0
__device__ __forceinline__ u32x4 keep8(const u32x4 g, const u32x4 m) {
    u32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = keep_where_positive_bf16(g[e], m[e]);
    return o;
}

// NT = blockDim.x threads (256 or 1024): CH = min(chunks, NT) chunk columns per pass, RS = NT / CH rows
// in parallel.  partial: [gridDim.x][2][C] floats.
__global__ __launch_bounds__(1024) void bn_stats_kernel(const unsigned char *x, float *partial, long long M, int C,
                                                       long long rows_per_block, int CH, int RS) {
    extern __shared__ __align__(16) float red[];                 // [RS][CH][16]
    const int chunks = C / 8;
    const int t = threadIdx.x;
    const int ck0 = t % CH, rsub = t / CH;
    const long long r0 = (long long)blockIdx.x * rows_per_block;
    long long r1 = r0 + rows_per_block;
    if (r1 > M) r1 = M;
    for (int cg = 0; cg < chunks; cg += CH) {
        const int ck = cg + ck0;
        const bool live = ck < chunks && rsub < RS;
        float s1[8], s2[8], k[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) s1[e] = s2[e] = 0.f;
        if (live) {
            unpack8(*reinterpret_cast<const u32x4 *>(x + (size_t)ck * 16), k);      // row 0: the shift
            long long r = r0 + rsub;
            for (; r + 3LL * RS < r1; r += 4LL * RS) {            // four rows in flight per lane
                u32x4 raw[4];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    raw[u] = *reinterpret_cast<const u32x4 *>(x + ((size_t)(r + (long long)u * RS) * chunks + ck) * 16);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    float v[8];
                    unpack8(raw[u], v);
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float d = v[e] - k[e];
                        s1[e] += d;
                        s2[e] += d * d;
                    }
                }
            }
            for (; r < r1; r += RS) {
                float v[8];
                unpack8(*reinterpret_cast<const u32x4 *>(x + ((size_t)r * chunks + ck) * 16), v);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float d = v[e] - k[e];
                    s1[e] += d;
                    s2[e] += d * d;
                }
            }
        }
        if (cg) __syncthreads();                                 // the previous pass's reads are done
        if (rsub < RS) {
            float *p = red + ((size_t)rsub * CH + ck0) * 16;
#pragma unroll
            for (int e = 0; e < 8; ++e) { p[e] = s1[e]; p[8 + e] = s2[e]; }
        }
        __syncthreads();
        // every thread adds the RS row-parallel contributions of some of the CH x 16 sums, in row order
        for (int o = t; o < CH * 16; o += (int)blockDim.x) {
            const int c0 = o >> 4, q = o & 15;
            if (cg + c0 >= chunks) continue;
            float a = 0.f;
            for (int j = 0; j < RS; ++j) a += red[(size_t)j * CH * 16 + o];
            partial[((size_t)blockIdx.x * 2 + (q >> 3)) * C + (cg + c0) * 8 + (q & 7)] = a;
        }
    }
}

// ab: [2][C]: a, then the mean.  A workgroup of 1024 threads takes CL = 1 << cl_bits channels (64, or
// 16 when there are few channels, so that more workgroups and shorter chains share the partials):
// thread (channel lane, group g of G = 1024 / CL) adds the partials of blocks g, g + G, ...
// (coalesced over the channels, eight loads in flight), the G groups are then added in order
// through LDS: sixteen threads to a channel, then one.  (One thread per channel with
// all groups: 4.1 us and, with the backward's four sums, 6.9; now 3.4 and 3.8 at 25088 x 512.)
__global__ __launch_bounds__(1024) void bn_finalize_kernel(const unsigned char *x, const float *partial, const float *gamma,
                                                           const float *beta, float *ab, long long M, int C, int blocks,
                                                           float eps, int cl_bits) {
    __shared__ double red[2][1024];                              // [sum][group][channel lane]
    __shared__ double sub[2][8][64];
    const int CL = 1 << cl_bits, G = 1024 >> cl_bits;
    const int cl = threadIdx.x & (CL - 1), grp = threadIdx.x >> cl_bits;
    const int c = blockIdx.x * CL + cl;
    double s1 = 0.0, s2 = 0.0;
    if (c < C) {
        int b = grp;
        for (; b + 7 * G < blocks; b += 8 * G) {
            float p1[8], p2[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                p1[u] = partial[(size_t)(b + G * u) * 2 * C + c];
                p2[u] = partial[(size_t)(b + G * u) * 2 * C + C + c];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) { s1 += (double)p1[u]; s2 += (double)p2[u]; }
        }
        for (; b < blocks; b += G) {
            s1 += (double)partial[(size_t)b * 2 * C + c];
            s2 += (double)partial[(size_t)b * 2 * C + C + c];
        }
    }
    red[0][threadIdx.x] = s1;
    red[1][threadIdx.x] = s2;
    __syncthreads();
    if (grp < 16) {                                              // two sums x eight parts of G / 8 groups each
        const int q = grp & 1, part = grp >> 1, each = G / 8;
        s1 = 0.0;
        for (int g = part * each; g < (part + 1) * each; ++g) s1 += red[q][g * CL + cl];
        sub[q][part][cl] = s1;
    }
    __syncthreads();
    if (grp != 0 || c >= C) return;
    s1 = s2 = 0.0;
#pragma unroll
    for (int part = 0; part < 8; ++part) { s1 += sub[0][part][cl]; s2 += sub[1][part][cl]; }
    const double k = (double)__uint_as_float((uint32_t)reinterpret_cast<const uint16_t *>(x)[c] << 16);
    const double md = s1 / (double)M;
    double var = s2 / (double)M - md * md;
    if (var < 0.0) var = 0.0;
    const double mean = k + md;
    ab[c] = (float)((double)gamma[c] / sqrt(var + (double)eps));
    ab[C + c] = (float)mean;
    (void)beta;
}

// max(v, 0): a negative bf16 has its sign bit set (NaN passes through, as in the fused epilogue)
__device__ __forceinline__ u32x4 relu8(u32x4 v) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const uint32_t lo = v[e] & 0xFFFFu, hi = v[e] >> 16;
        const bool nlo = (lo & 0x8000u) && (lo & 0x7FFFu) <= 0x7F80u;    // negative, not NaN
        const bool nhi = (hi & 0x8000u) && (hi & 0x7FFFu) <= 0x7F80u;
        v[e] = (nlo ? 0u : lo) | ((nhi ? 0u : hi) << 16);
    }
    return v;
}

__device__ __forceinline__ u32x4 add8(const u32x4 a, const u32x4 b) {
    u32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = pack2(lo16(a[e]) + lo16(b[e]), hi16(a[e]) + hi16(b[e]));
    return o;
}

// Element by element, from x: [the normalisation], [+ r], [ReLU], each result rounded to bf16, stored and read on as it is
// stored, so the bits are those of separate passes.  Two pieces in flight per thread.  Bound by memory: 25088 x 512 with all three, five
// tensor passes in 20 us where three launches took 31.6 for seven.  What the run itself has read already leaves past the caches (the
// case of the backward pass too 78.3 -> 76.4 us, 100352 x 512 266 -> 255): only its last result is read next.
template <bool BN, bool ADD, bool RELU>
__global__ __launch_bounds__(256) void bn_tail_kernel(const u32x4 *__restrict__ x, const u32x4 *__restrict__ r, u32x4 *__restrict__ y,
                                                      u32x4 *__restrict__ ya, u32x4 *__restrict__ yr, const float *__restrict__ ab,
                                                      const float *__restrict__ beta, int C, size_t n16) {
    const size_t step = (size_t)gridDim.x * blockDim.x;          // BN: a multiple of C / 8, a thread stays with its channels (11.0 -> 9.8 us at 25088 x 512)
    const size_t first = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    f32x4 a0, a1, m0, m1, b0, b1;
    if constexpr (BN) {
        const int ck = (int)(first % (unsigned)(C / 8));
        a0 = *reinterpret_cast<const f32x4 *>(ab + ck * 8); a1 = *reinterpret_cast<const f32x4 *>(ab + ck * 8 + 4);
        m0 = *reinterpret_cast<const f32x4 *>(ab + C + ck * 8); m1 = *reinterpret_cast<const f32x4 *>(ab + C + ck * 8 + 4);
        b0 = *reinterpret_cast<const f32x4 *>(beta + ck * 8); b1 = *reinterpret_cast<const f32x4 *>(beta + ck * 8 + 4);
    }
    auto finish = [&](size_t i, u32x4 v, const u32x4 rv) {
        if constexpr (BN) {
            float f[8];
            unpack8(v, f);
            v.x = pack2((f[0] - m0.x) * a0.x + b0.x, (f[1] - m0.y) * a0.y + b0.y);
            v.y = pack2((f[2] - m0.z) * a0.z + b0.z, (f[3] - m0.w) * a0.w + b0.w);
            v.z = pack2((f[4] - m1.x) * a1.x + b1.x, (f[5] - m1.y) * a1.y + b1.y);
            v.w = pack2((f[6] - m1.z) * a1.z + b1.z, (f[7] - m1.w) * a1.w + b1.w);
            if constexpr (ADD || RELU) __builtin_nontemporal_store(v, y + i);
            else y[i] = v;
        }
        if constexpr (ADD) {
            v = add8(v, rv);
            if constexpr (RELU) __builtin_nontemporal_store(v, ya + i);
            else ya[i] = v;
        }
        if constexpr (RELU) yr[i] = relu8(v);
    };
    for (size_t i = first; i < n16; i += 2 * step) {
        const size_t j = i + step;
        const bool two = j < n16;
        const u32x4 v0 = x[i], v1 = two ? x[j] : v0;
        u32x4 r0 = {0u, 0u, 0u, 0u}, r1 = r0;
        if constexpr (ADD) { r0 = r[i]; r1 = two ? r[j] : r0; }
        finish(i, v0, r0);
        if (two) finish(j, v1, r1);
    }
}

// Backward statistics.  Same decomposition as bn_stats_kernel; partial: [gridDim.x][4][C] floats
// (sum d, sum d^2, sum g, sum g d with d = x - K_c).  red: [RS][CH][32].
// MASK: g is first set to zero where mask is not > 0, and stored (gm): four tensor passes instead of the five of two launches.
template <bool MASK>
__global__ __launch_bounds__(1024) void bn_bwd_stats_kernel(const unsigned char *x, const unsigned char *g, const unsigned char *mask,
                                                           unsigned char *gm, float *partial, long long M, int C,
                                                           long long rows_per_block, int CH, int RS) {
    extern __shared__ __align__(16) float red[];
    const int chunks = C / 8;
    const int t = threadIdx.x;
    const int ck0 = t % CH, rsub = t / CH;
    const long long r0 = (long long)blockIdx.x * rows_per_block;
    long long r1 = r0 + rows_per_block;
    if (r1 > M) r1 = M;
    for (int cg = 0; cg < chunks; cg += CH) {
        const int ck = cg + ck0;
        const bool live = ck < chunks && rsub < RS;
        float s1[8], s2[8], s3[8], s4[8], k[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) s1[e] = s2[e] = s3[e] = s4[e] = 0.f;
        if (live) {
            unpack8(*reinterpret_cast<const u32x4 *>(x + (size_t)ck * 16), k);
            long long r = r0 + rsub;
            constexpr int kRows = MASK ? 2 : 4;                   // rows of every tensor in flight per lane (128 registers)
            for (; r + (kRows - 1) * (long long)RS < r1; r += kRows * (long long)RS) {
                u32x4 rx[kRows], rg[kRows], rm[kRows];
#pragma unroll
                for (int u = 0; u < kRows; ++u) {
                    const size_t at = ((size_t)(r + (long long)u * RS) * chunks + ck) * 16;
                    rx[u] = *reinterpret_cast<const u32x4 *>(x + at);
                    rg[u] = *reinterpret_cast<const u32x4 *>(g + at);
                    if constexpr (MASK) rm[u] = *reinterpret_cast<const u32x4 *>(mask + at);
                }
                if constexpr (MASK) {
#pragma unroll
                    for (int u = 0; u < kRows; ++u) {
                        rg[u] = keep8(rg[u], rm[u]);
                        *reinterpret_cast<u32x4 *>(gm + ((size_t)(r + (long long)u * RS) * chunks + ck) * 16) = rg[u];
                    }
                }
#pragma unroll
                for (int u = 0; u < kRows; ++u) {
                    float v[8], w[8];
                    unpack8(rx[u], v);
                    unpack8(rg[u], w);
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float d = v[e] - k[e];
                        s1[e] += d;
                        s2[e] += d * d;
                        s3[e] += w[e];
                        s4[e] += w[e] * d;
                    }
                }
            }
            for (; r < r1; r += RS) {
                const size_t at = ((size_t)r * chunks + ck) * 16;
                float v[8], w[8];
                unpack8(*reinterpret_cast<const u32x4 *>(x + at), v);
                u32x4 rg = *reinterpret_cast<const u32x4 *>(g + at);
                if constexpr (MASK) {
                    rg = keep8(rg, *reinterpret_cast<const u32x4 *>(mask + at));
                    *reinterpret_cast<u32x4 *>(gm + at) = rg;
                }
                unpack8(rg, w);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float d = v[e] - k[e];
                    s1[e] += d;
                    s2[e] += d * d;
                    s3[e] += w[e];
                    s4[e] += w[e] * d;
                }
            }
        }
        if (cg) __syncthreads();
        if (rsub < RS) {
            float *p = red + ((size_t)rsub * CH + ck0) * 32;
#pragma unroll
            for (int e = 0; e < 8; ++e) { p[e] = s1[e]; p[8 + e] = s2[e]; p[16 + e] = s3[e]; p[24 + e] = s4[e]; }
        }
        __syncthreads();
        for (int o = t; o < CH * 32; o += (int)blockDim.x) {     // as in bn_stats_kernel
            const int c0 = o >> 5, q = o & 31;
            if (cg + c0 >= chunks) continue;
            float a = 0.f;
            for (int j = 0; j < RS; ++j) a += red[(size_t)j * CH * 32 + o];
            partial[((size_t)blockIdx.x * 4 + (q >> 3)) * C + (cg + c0) * 8 + (q & 7)] = a;
        }
    }
}

// coef: [4][C]: a, mean, mean(gy), S / ((var + eps) M).  gw (may be null): dgamma [C], then dbeta [C].
// Decomposition as in bn_finalize_kernel.
__global__ __launch_bounds__(1024) void bn_bwd_finalize_kernel(const unsigned char *x, const float *partial,
                                                               const float *gamma, float *coef, float *gw, long long M,
                                                               int C, int blocks, float eps, int cl_bits) {
    __shared__ double red[4][1024], sub[4][4][64];
    const int CL = 1 << cl_bits, G = 1024 >> cl_bits;
    const int cl = threadIdx.x & (CL - 1), grp = threadIdx.x >> cl_bits;
    const int c = blockIdx.x * CL + cl;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    if (c < C) {
        int b = grp;
        for (; b + 3 * G < blocks; b += 4 * G) {
            float p[4][4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) p[u][q] = partial[((size_t)(b + G * u) * 4 + q) * C + c];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) s[q] += (double)p[u][q];
        }
        for (; b < blocks; b += G)
#pragma unroll
            for (int q = 0; q < 4; ++q) s[q] += (double)partial[((size_t)b * 4 + q) * C + c];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) red[q][threadIdx.x] = s[q];
    __syncthreads();
    if (grp < 16) {                                              // four sums x four parts of G / 4 groups each
        const int q = grp & 3, part = grp >> 2, each = G / 4;
        double a = 0.0;
        for (int g = part * each; g < (part + 1) * each; ++g) a += red[q][g * CL + cl];
        sub[q][part][cl] = a;
    }
    __syncthreads();
    if (grp != 0 || c >= C) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        s[q] = 0.0;
#pragma unroll
        for (int part = 0; part < 4; ++part) s[q] += sub[q][part][cl];
    }
    const double k = (double)__uint_as_float((uint32_t)reinterpret_cast<const uint16_t *>(x)[c] << 16);
    const double md = s[0] / (double)M;
    double var = s[1] / (double)M - md * md;
    if (var < 0.0) var = 0.0;
    const double ve = var + (double)eps;
    const double S = s[3] - md * s[2];                           // sum gy (x - mean)
    coef[c] = (float)((double)gamma[c] / sqrt(ve));
    coef[C + c] = (float)(k + md);
    coef[2 * C + c] = (float)(s[2] / (double)M);
    coef[3 * C + c] = (float)(S / (ve * (double)M));
    if (gw) {
        gw[c] = (float)(S / sqrt(ve));
        gw[C + c] = (float)s[2];
    }
}

__global__ __launch_bounds__(256) void bn_bwd_apply_kernel(const u32x4 *__restrict__ x, const u32x4 *__restrict__ g,
                                                           u32x4 *__restrict__ gx, const float *__restrict__ coef, int C,
                                                           size_t n16) {
    const size_t step = (size_t)gridDim.x * blockDim.x;          // as in bn_tail_kernel
    const int ck = (int)((blockIdx.x * blockDim.x + threadIdx.x) % (unsigned)(C / 8));
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += step) {
        float v[8], w[8], o[8];
        unpack8(x[i], v);
        unpack8(g[i], w);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const f32x4 a = *reinterpret_cast<const f32x4 *>(coef + ck * 8 + 4 * h);
            const f32x4 m = *reinterpret_cast<const f32x4 *>(coef + C + ck * 8 + 4 * h);
            const f32x4 c1 = *reinterpret_cast<const f32x4 *>(coef + 2 * C + ck * 8 + 4 * h);
            const f32x4 c2 = *reinterpret_cast<const f32x4 *>(coef + 3 * C + ck * 8 + 4 * h);
#pragma unroll
            for (int e = 0; e < 4; ++e) o[4 * h + e] = a[e] * (w[4 * h + e] - c1[e] - (v[4 * h + e] - m[e]) * c2[e]);
        }
        u32x4 r;
        r.x = pack2(o[0], o[1]); r.y = pack2(o[2], o[3]); r.z = pack2(o[4], o[5]); r.w = pack2(o[6], o[7]);
        gx[i] = r;
    }
}

__global__ __launch_bounds__(256) void relu_kernel(const u32x4 *__restrict__ x, u32x4 *__restrict__ y, size_t n16) {
    const size_t step = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += step) y[i] = relu8(x[i]);
}

__global__ __launch_bounds__(256) void add_kernel(const u32x4 *__restrict__ x, const u32x4 *__restrict__ r,
                                                  u32x4 *__restrict__ y, size_t n16) {
    const size_t step = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += step) y[i] = add8(x[i], r[i]);
}

static unsigned stream_blocks(size_t n16) {
    size_t blocks = (n16 + 255) / 256;
    return (unsigned)(blocks > 256 * 16 ? 256 * 16 : blocks);
}
// The same, rounded up so that the grid's threads are a whole number of rows of `chunks` pieces.
static unsigned row_blocks(size_t n16, int chunks) {
    int q = chunks;
    for (int twos = 256; twos > 1 && q % 2 == 0; twos /= 2) q /= 2;
    return (stream_blocks(n16) + q - 1) / q * q;
}

// The last pass over the elements: whatever of normalisation, add and ReLU there is.
static hipError_t launch_tail(const void *x, const ElementwiseTail &t, void *y, const float *ab, const float *beta, int C, size_t n16,
                              hipStream_t stream) {
    const unsigned blocks = y ? row_blocks((n16 + 1) / 2, C / 8) : stream_blocks((n16 + 1) / 2);
    auto run = [&](auto kernel) {
        kernel<<<dim3(blocks), dim3(256), 0, stream>>>(static_cast<const u32x4 *>(x), static_cast<const u32x4 *>(t.r), static_cast<u32x4 *>(y),
                                                       static_cast<u32x4 *>(t.y_add), static_cast<u32x4 *>(t.y_relu), ab, beta, C, n16);
    };
    if (y) {
        if (t.y_add) t.y_relu ? run(bn_tail_kernel<true, true, true>) : run(bn_tail_kernel<true, true, false>);
        else t.y_relu ? run(bn_tail_kernel<true, false, true>) : run(bn_tail_kernel<true, false, false>);
    } else {
        run(bn_tail_kernel<false, true, true>);
    }
    return hipGetLastError();
}

}  // namespace ops

const char *bn_train_check(const void *x, const void *y, const float *gamma, const float *beta, long long M, int C,
                           int bf16) {
    if (!bf16) return "batch normalisation with batch statistics is bf16 only";
    if (M <= 0 || C <= 0 || C % 8 || C > 8192) return "channels must be a multiple of 8, at most 8192";
    if (!x || !y || !gamma || !beta || (((uintptr_t)x | (uintptr_t)y | (uintptr_t)gamma | (uintptr_t)beta) & 15))
        return "pointers must be non-null and 16-byte aligned";
    return nullptr;
}

size_t bn_train_scratch_bytes() { return (size_t)16 << 20; }     // partial sums + the 2 x C factors

// Large tensors take workgroups of 1024 threads, a quarter as many: the same lanes share the rows, and
// the finalize kernel, which runs on a nearly empty chip, reads a quarter of the partial sums.  Half as many where a quarter would leave CUs without one
// and every workgroup at least twelve rounds of its lanes: below that the finalize kernel loses more than the statistics gain.  us with a quarter | half:
// forward and backward, from memory: 100352 x 512 262 | 245, 50176 x 512 137 | 123, 12544 x 1024 95 | 81, 6272 x 1024 59 | 53, 25088 x 512 77 | 74 (in the
// caches 64 | 66); the backward alone at that last size 33 | 35, and with fewer rounds 12544 x 512 24 | 25, 25088 x 256 23 | 25, 100352 x 64 25 | 27.
static void stats_shape(int chunks, long long M, long long &blocks, int &NT, int &CH, int &RS) {
    if (blocks < 256) return;
    NT = 1024;
    const long long half = (blocks + 1) / 2 < 256 ? (blocks + 1) / 2 : 256;
    blocks = (blocks + 3) / 4;
    if (blocks < half && M * chunks >= blocks * (12 * 1024)) blocks = half;
    CH = chunks < NT ? chunks : NT;
    RS = NT / CH;
}

// What the forward needs at most: the 2 x C factors and 64 workgroups' partial sums at C = 8192 (wider
// tensors take fewer workgroups, see the cap below), so that a buffer of this size never changes the
// decomposition - and with it the bits of the result - against a larger one.
size_t bn_train_fwd_scratch_bytes() { return ((size_t)4 << 20) + ((size_t)64 << 10); }

// The per-channel factors of the normalisation, from x alone, at the start of the scratch (device, scratch_bytes >= bn_train_fwd_scratch_bytes()
// bytes, 16-byte aligned): launch_bn_apply reads them there.  Two functions, so that what only the second needs is waited for between them.
hipError_t launch_bn_factors(const void *x, const float *gamma, const float *beta, long long M, int C, float eps, int bf16, void *scratch,
                             size_t scratch_bytes, hipStream_t stream) {
    if (bn_train_check(x, x, gamma, beta, M, C, bf16) || !scratch || ((uintptr_t)scratch & 15) || scratch_bytes < bn_train_fwd_scratch_bytes())
        return hipErrorInvalidValue;
    const int chunks = C / 8;
    int NT = 256;
    int CH = chunks < NT ? chunks : NT;
    int RS = NT / CH;
    float *ab = static_cast<float *>(scratch);                   // [2][C]
    float *partial = ab + 2 * (size_t)C;
    const size_t room = (scratch_bytes - 2 * (size_t)C * 4) / ((size_t)2 * C * 4);
    long long blocks = (M + (long long)RS * 4 - 1) / ((long long)RS * 4);    // at least 4 rows per lane
    // fewer partials for wide tensors: the finalize kernel reads blocks x 2 x C floats
    long long cap = 262144 / C;
    cap = cap < 64 ? 64 : (cap > 2048 ? 2048 : cap);
    if (blocks > cap) blocks = cap;
    if (blocks > (long long)room) blocks = (long long)room;
    if (blocks < 1) return hipErrorInvalidValue;
    stats_shape(chunks, M, blocks, NT, CH, RS);
    const long long rpb = (M + blocks - 1) / blocks;
    blocks = (M + rpb - 1) / rpb;
    const size_t lds = (size_t)RS * CH * 16 * 4;
    static const hipError_t lds_ok = hipFuncSetAttribute(reinterpret_cast<const void *>(ops::bn_stats_kernel),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, 1024 * 16 * 4);
    if (lds_ok != hipSuccess) return lds_ok;
    ops::bn_stats_kernel<<<dim3((unsigned)blocks), dim3((unsigned)NT), lds, stream>>>(static_cast<const unsigned char *>(x), partial,
                                                                            M, C, rpb, CH, RS);
    const int cl_bits = C <= 512 ? 4 : 6;
    ops::bn_finalize_kernel<<<dim3((unsigned)((C + (1 << cl_bits) - 1) >> cl_bits)), dim3(1024), 0, stream>>>(
        static_cast<const unsigned char *>(x), partial, gamma, beta, ab, M, C, (int)blocks, eps, cl_bits);
    return hipGetLastError();
}

// y = the normalisation of x, and the tail's results.  scratch: as launch_bn_factors left it.
hipError_t launch_bn_apply(const void *x, void *y, const float *beta, long long M, int C, int bf16, const ElementwiseTail &tail,
                           const void *scratch, hipStream_t stream) {
    if (bn_train_check(x, y, beta, beta, M, C, bf16) || tail.bad() || !scratch || ((uintptr_t)scratch & 15)) return hipErrorInvalidValue;
    return ops::launch_tail(x, tail, y, static_cast<const float *>(scratch), beta, C, (size_t)M * (C / 8), stream);
}

// Backward of the normalisation.  gw: device fp32 [2][C] (dgamma, dbeta) or null.  Same scratch.
// relu_y / gm: both or neither; gm = gy where relu_y > 0, else 0, is stored and taken in gy's place.
hipError_t launch_bn_train_bwd(const void *x, const void *gy, void *gx, const float *gamma, float *gw, long long M, int C,
                               float eps, int bf16, const void *relu_y, void *gm, void *scratch, hipStream_t stream) {
    if (bn_train_check(x, gx, gamma, gamma, M, C, bf16) || !gy || !relu_y != !gm || (((uintptr_t)relu_y | (uintptr_t)gm) & 15) || ((uintptr_t)gy & 15) || ((uintptr_t)gw & 15) || !scratch ||
        ((uintptr_t)scratch & 15))
        return hipErrorInvalidValue;
    const int chunks = C / 8;
    int NT = 256;
    int CH = chunks < NT ? chunks : NT;
    int RS = NT / CH;
    float *coef = static_cast<float *>(scratch);                 // [4][C]
    float *partial = coef + 4 * (size_t)C;
    const size_t room = (bn_train_scratch_bytes() - 4 * (size_t)C * 4) / ((size_t)4 * C * 4);
    long long blocks = (M + (long long)RS * 4 - 1) / ((long long)RS * 4);
    long long cap = 262144 / C;                                  // 1024 workgroups fill the chip four wavefronts deep
    cap = cap < 64 ? 64 : (cap > 1024 ? 1024 : cap);
    if (blocks > cap) blocks = cap;
    if (blocks > (long long)room) blocks = (long long)room;
    if (blocks < 1) return hipErrorInvalidValue;
    stats_shape(chunks, M, blocks, NT, CH, RS);
    const long long rpb = (M + blocks - 1) / blocks;
    blocks = (M + rpb - 1) / rpb;
    const size_t lds = (size_t)RS * CH * 32 * 4;
    static const hipError_t lds_ok = [] {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(ops::bn_bwd_stats_kernel<false>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 1024 * 32 * 4);
        return e != hipSuccess ? e : hipFuncSetAttribute(reinterpret_cast<const void *>(ops::bn_bwd_stats_kernel<true>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, 1024 * 32 * 4);
    }();
    if (lds_ok != hipSuccess) return lds_ok;
    auto stats = [&](auto kernel) {
        kernel<<<dim3((unsigned)blocks), dim3((unsigned)NT), lds, stream>>>(
            static_cast<const unsigned char *>(x), static_cast<const unsigned char *>(gy), static_cast<const unsigned char *>(relu_y),
            static_cast<unsigned char *>(gm), partial, M, C, rpb, CH, RS);
    };
    gm ? stats(ops::bn_bwd_stats_kernel<true>) : stats(ops::bn_bwd_stats_kernel<false>);
    if (gm) gy = gm;
    const int cl_bits = C <= 512 ? 4 : 6;
    ops::bn_bwd_finalize_kernel<<<dim3((unsigned)((C + (1 << cl_bits) - 1) >> cl_bits)), dim3(1024), 0, stream>>>(
        static_cast<const unsigned char *>(x), partial, gamma, coef, gw, M, C, (int)blocks, eps, cl_bits);
    const size_t n16 = (size_t)M * chunks;
    ops::bn_bwd_apply_kernel<<<dim3(ops::row_blocks(n16, chunks)), dim3(256), 0, stream>>>(
        static_cast<const ops::u32x4 *>(x), static_cast<const ops::u32x4 *>(gy), static_cast<ops::u32x4 *>(gx), coef, C, n16);
    return hipGetLastError();
}

hipError_t launch_relu(const void *x, void *y, size_t bytes, int bf16, hipStream_t stream) {
    if (!bf16 || !x || !y || bytes % 16 || (((uintptr_t)x | (uintptr_t)y) & 15)) return hipErrorInvalidValue;
    if (bytes == 0) return hipSuccess;
    ops::relu_kernel<<<dim3(ops::stream_blocks(bytes / 16)), dim3(256), 0, stream>>>(
        static_cast<const ops::u32x4 *>(x), static_cast<ops::u32x4 *>(y), bytes / 16);
    return hipGetLastError();
}

hipError_t launch_add(const void *x, const void *r, void *y, size_t bytes, int bf16, hipStream_t stream) {
    if (!bf16 || !x || !r || !y || bytes % 16 || (((uintptr_t)x | (uintptr_t)r | (uintptr_t)y) & 15)) return hipErrorInvalidValue;
    if (bytes == 0) return hipSuccess;
    ops::add_kernel<<<dim3(ops::stream_blocks(bytes / 16)), dim3(256), 0, stream>>>(
        static_cast<const ops::u32x4 *>(x), static_cast<const ops::u32x4 *>(r), static_cast<ops::u32x4 *>(y), bytes / 16);
    return hipGetLastError();
}

// ReLU of an add's result, in one pass.
hipError_t launch_add_relu(const void *x, const ElementwiseTail &tail, size_t bytes, int bf16, hipStream_t stream) {
    if (!bf16 || !x || !tail.y_add || !tail.y_relu || tail.bad() || bytes % 16 || ((uintptr_t)x & 15)) return hipErrorInvalidValue;
    if (bytes == 0) return hipSuccess;
    return ops::launch_tail(x, tail, nullptr, nullptr, nullptr, 8, bytes / 16, stream);
}

}  // namespace delta
