// Backward of the fused layer y = relu?(scale_k * conv(x, w) + shift_k (+ res)) for gfx950, bf16.
//
// DELTA's planner follows the tensor accesses of a whole training iteration (Sec. 3,
// Assumptions 1-3: the backward pass reads the stored forward activations, which is why
// released ones must be regenerated or reloaded).  These kernels are that backward pass for the
// bottleneck layers, with frozen batch-norm statistics:
//
//   gpre = gy * [y > 0]                       relu_mask_kernel (also dL/dres)
//   gx   = conv^T(gpre * scale, w)            the forward kernels, run on gpre with the weights
//                                             transposed, flipped and pre-multiplied by scale
//                                             (bwd_weights_kernel)
//   gw[k,r,s,c] = scale_k * sum_m gpre[m,k] * x[m + (r,s), c]      wgrad1x1.hip, wgrad3x3.hip (bf16); wgrad_f32_kernel here
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "kernels.hpp"
#include "wgrad_f32_tile.hpp"

namespace delta {
namespace bwd {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

static constexpr int kOutOfRange = (int)0x80000000;   // outside every buffer descriptor used here

// ---------------------------------------------------------------- gpre = gy * [y > 0]
// 16 bytes per thread, grid-stride.  bf16: y > 0 <=> sign bit clear and not zero (NaN counts as
// "not greater": the forward's ReLU passes NaN through, its gradient is taken as 0).
template <bool BF16>
__global__ __launch_bounds__(256) void relu_mask_kernel(const u32x4 *__restrict__ y, const u32x4 *__restrict__ gy,
                                                        u32x4 *__restrict__ out, size_t n16) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride) {
        const u32x4 a = y[i], g = gy[i];
        u32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if constexpr (BF16) o[e] = keep_where_positive_bf16(g[e], a[e]);
            else o[e] = keep_where_positive_f32(g[e], a[e]);
        }
        out[i] = o;
    }
}

// Strided layers: the masked gradient is written at the input's resolution, out[n, s p, s q, :] =
// gy[n, p, q, :] * [y > 0] and zero everywhere else.  With that tensor the data gradient is again a
// stride-1 convolution and the weight gradient the stride-1 reduction (the zeros contribute
// nothing), at the price of stride^2 times the arithmetic.  One 16-byte piece per thread.
template <bool BF16>
__global__ __launch_bounds__(256) void relu_mask_dilate_kernel(const u32x4 *__restrict__ y, const u32x4 *__restrict__ gy,
                                                               u32x4 *__restrict__ out, int H, int W, int P, int Q,
                                                               int vec_per_pixel, int stride, size_t n16) {
    const size_t step = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += step) {
        const size_t pix = i / vec_per_pixel;
        const int v = (int)(i - pix * vec_per_pixel);
        const int w = (int)(pix % W);
        const size_t rest = pix / W;
        const int h = (int)(rest % H);
        const size_t n = rest / H;
        u32x4 o = {0u, 0u, 0u, 0u};
        const int p = h / stride, q = w / stride;
        if (p * stride == h && q * stride == w && p < P && q < Q) {
            const size_t src = ((n * P + p) * Q + q) * vec_per_pixel + v;
            const u32x4 g = gy[src];
            if (y) {
                const u32x4 a = y[src];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if constexpr (BF16) {
                        const uint32_t lo = a[e] & 0xFFFFu, hi = a[e] >> 16;
                        const bool plo = lo != 0 && lo < 0x7F81u, phi = hi != 0 && hi < 0x7F81u;
                        o[e] = (plo ? (g[e] & 0xFFFFu) : 0u) | (phi ? (g[e] & 0xFFFF0000u) : 0u);
                    } else {
                        o[e] = __uint_as_float(a[e]) > 0.f ? g[e] : 0u;
                    }
                }
            } else {
                o = g;
            }
        }
        out[i] = o;
    }
}

// ---------------------------------------------------------------- strided 1x1 layers, directly
// A 1x1 layer with stride s reads only the pixels (s p, s q) of its input, so both of its
// gradients are stride-1 operations at the OUTPUT's resolution:
//   t = 1x1 data gradient of gpre at P x Q
//   gx[n,h,w,:] = (t[n,h/s,w/s,:] on the grid, else 0) + gx_add, optionally * [x > 0]   spread_add_kernel
// (the weight gradients pick those pixels themselves).  `lanes` threads (a power of two) walk the 16-byte pieces of a pixel, so that its
// coordinates are found once per pixel and by multiplication: with a 64-bit division chain per piece the kernel was bound by that
// arithmetic.  HBM-bound now, 128 x 56 x 56 x 256, 257 MB, beside a weight gradient on the other stream: 82 -> 74 us.
template <bool BF16>
__global__ __launch_bounds__(256) void spread_add_kernel(const u32x4 *__restrict__ t, const u32x4 *__restrict__ add,
                                                         const u32x4 *__restrict__ mask, u32x4 *__restrict__ out, int H,
                                                         int W, int P, int Q, int vec_per_pixel, int stride, int lanes, int npix,
                                                         Divisor dw, Divisor dh, Divisor ds) {
    const int per = 256 / lanes, v0 = threadIdx.x & (lanes - 1);
    for (long long at = (long long)blockIdx.x * per + threadIdx.x / lanes; at < npix; at += (long long)gridDim.x * per) {
        const int pix = (int)at, rest = divide(pix, dw), w = pix - rest * W, n = divide(rest, dh), h = rest - n * H;
        const int p = divide(h, ds), q = divide(w, ds);
        const bool on_grid = (p * stride == h) & (q * stride == w) & (p < P) & (q < Q);
        const size_t ti = (((size_t)n * P + p) * Q + q) * vec_per_pixel;
        for (int v = v0; v < vec_per_pixel; v += lanes) {
            const size_t i = (size_t)pix * vec_per_pixel + v;
            u32x4 o = {0u, 0u, 0u, 0u};
            if (on_grid) o = t[ti + v];
            if (add) {
                const u32x4 a = add[i];
                if (!on_grid) {
                    o = a;                                   // nothing to add to: the bits pass through
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if constexpr (BF16) {
                            const float lo = __uint_as_float(o[e] << 16) + __uint_as_float(a[e] << 16);
                            const float hi = __uint_as_float(o[e] & 0xFFFF0000u) + __uint_as_float(a[e] & 0xFFFF0000u);
                            const f32x2 pr = {lo, hi};
                            o[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pr, bf16x2));
                        } else {
                            o[e] = __float_as_uint(__uint_as_float(o[e]) + __uint_as_float(a[e]));
                        }
                    }
                }
            }
            if (mask) {
                const u32x4 m = mask[i];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if constexpr (BF16) o[e] = keep_where_positive_bf16(o[e], m[e]);
                    else o[e] = keep_where_positive_f32(o[e], m[e]);
                }
            }
            out[i] = o;
        }
    }
}

// ---------------------------------------------------------------- weights for the data gradient
// wt[c][R-1-r][S-1-s][k] = round(w[k][r][s][c] * scale_k): the data gradient is then the forward
// convolution of gpre with wt (stride 1, padding R-1-pad).  One thread per element of wt.
template <bool BF16>
__global__ __launch_bounds__(256) void bwd_weights_kernel(const void *w, const float *scale, void *wt, int K, int R,
                                                          int S, int C) {
    const size_t total = (size_t)K * R * S * C;
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    const int k = (int)(i % K);
    size_t rest = i / K;
    const int s2 = (int)(rest % S); rest /= S;
    const int r2 = (int)(rest % R);
    const int c = (int)(rest / R);
    const size_t src = (((size_t)k * R + (R - 1 - r2)) * S + (S - 1 - s2)) * C + c;
    if constexpr (BF16) {
        const float v = __uint_as_float((uint32_t)static_cast<const uint16_t *>(w)[src] << 16) * scale[k];
        static_cast<__bf16 *>(wt)[i] = (__bf16)v;             // round to nearest even
    } else {
        static_cast<float *>(wt)[i] = static_cast<const float *>(w)[src] * scale[k];
    }
}

// ---------------------------------------------------------------- weight gradient, fp32
// fp32 layers: one workgroup per tap and tile of 16 T x 16 T (k, c), its 16 wavefronts
// sharing the positions, on the fp32 MFMA (16x16x4: exact fp32 products, fp32 sums).  A workgroup holds all
// of a tile's sums, so there is no partial buffer and no workspace: wavefront v takes the v-th run of
// positions and the 16 sums are added in the order of v through LDS (a fixed function of the inputs).  Both operands are
// position-major with the channels contiguous, which is what this MFMA reads (lane l: position l / 16, channel
// T * (l % 16) + i), so they go from memory straight to registers, eight steps of four positions in flight.
// (A thread per (k, c) pair with all positions in one serial chain of multiply-adds through LDS took 94-110 us for a layer of
// 2048 positions.)
// Two forms.  This one takes strided layers and tensors of 2 GiB or more with 64-bit addresses; it is bound by that
// arithmetic, some 40 instructions per MFMA.
// g: [N,H,W,K]; x: [N,XH,XW,C], of which position (h, w) and tap (r, s) read pixel (h stride + r - pad, w stride + s - pad);
// gw: [K][R][R][C].  STRIDED: 1x1 layers with stride > 1 only; the others' pixels are their positions, shifted.
template <int T, bool STRIDED>
__global__ __launch_bounds__(1024) void wgrad_f32_kernel(const float *x, const float *g, const float *scale, float *gw,
                                                         int H, int W, int C, int K, int R, int pad, int XH, int XW, int stride,
                                                         long long M) {
    typedef float vec __attribute__((ext_vector_type(T)));
    constexpr int kWaves = 16, kSteps = 8;                       // positions in flight: 4 per step
    __shared__ float part[kWaves][T * T * 256];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, l16 = lane & 15, quad = lane >> 4;
    const int k0 = blockIdx.x * (16 * T), c0 = blockIdx.y * (16 * T), tap = blockIdx.z;
    const int dr = tap / R - pad, ds = tap % R - pad;
    const long long per = ((M + kWaves - 1) / kWaves + 3) / 4 * 4;
    long long m = (long long)wv * per + quad;                    // this lane's position
    const long long end = (long long)(wv + 1) * per < M ? (long long)(wv + 1) * per : M;
    const long long rounds = (per + 4 * kSteps - 1) / (4 * kSteps);
    int w = (int)(m % W), h = (int)((m / W) % H);
    long long n = STRIDED ? m / W / H : 0;
    const float *gp = g + m * K + k0 + T * l16, *xp = x + (STRIDED ? 0 : m + (long long)dr * W + ds) * C + c0 + T * l16;
    f32x4 acc[T][T];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (long long t = 0; t < rounds; ++t) {
        vec gv[kSteps], xv[kSteps];
#pragma unroll
        for (int u = 0; u < kSteps; ++u) {
            // outside: the tensor's first element is read and dropped (no branch around a load)
            const int xh = STRIDED ? h * stride : h + dr, xw = STRIDED ? w * stride : w + ds;
            const bool live = m < end, in = live && (unsigned)xh < (unsigned)XH && (unsigned)xw < (unsigned)XW;
            const vec gr = *reinterpret_cast<const vec *>(live ? gp : g);
            const vec xr = *reinterpret_cast<const vec *>(!in ? x : STRIDED ? xp + ((n * XH + xh) * XW + xw) * (long long)C : xp);
#pragma unroll
            for (int i = 0; i < T; ++i) {
                gv[u][i] = live ? gr[i] : 0.f;
                xv[u][i] = in ? xr[i] : 0.f;
            }
            m += 4; gp += 4 * (long long)K;
            if (!STRIDED) xp += 4 * (long long)C;
            w += 4;
            while (w >= W) {
                w -= W;
                if (++h == H) {
                    h = 0;
                    ++n;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kSteps; ++u)
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int j = 0; j < T; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(gv[u][i], xv[u][j], acc[i][j], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) part[wv][((i * T + j) * 4 + e) * 64 + lane] = acc[i][j][e];
    __syncthreads();
    if (tid >= T * T * 256) return;
    float sum = part[0][tid];
#pragma unroll
    for (int v = 1; v < kWaves; ++v) sum += part[v][tid];
    // lane of this sum: column (c) l % 16, row (k) 4 (l / 16) + e of the tile's (i, j) interleave
    const int k = k0 + T * (4 * quad + (wv & 3)) + (tid >> 8) / T, c = c0 + T * l16 + (tid >> 8) % T;
    gw[((size_t)k * R * R + tap) * C + c] = sum * scale[k];
}

// The form for stride 1 and tensors below 2 GiB (wgrad_f32_tile.hpp).
template <int T, bool TAPS>
__global__ __launch_bounds__(1024) void wgrad_f32_flat_kernel(const float *x, const float *g, const float *scale, float *gw, int H, int W, int C,
                                                              int K, int R, int pad, int M, Divisor dhw, Divisor dw) {
    __shared__ float part[16 * T * T * 256], factors[64];
    wgrad_f32_tile<T, TAPS, 16>(x, g, scale, gw, H, W, C, K, R, pad, M, dhw, dw, blockIdx.x * (16 * T), blockIdx.y * (16 * T), blockIdx.z, threadIdx.x,
                                part, factors);
}

}  // namespace bwd

// ---------------------------------------------------------------- host side

hipError_t launch_relu_mask(const void *y, const void *gy, void *out, size_t bytes, int bf16, hipStream_t stream) {
    if (bytes % 16) return hipErrorInvalidValue;
    const size_t n16 = bytes / 16;
    if (n16 == 0) return hipSuccess;
    size_t blocks = (n16 + 255) / 256;
    if (blocks > 256 * 16) blocks = 256 * 16;
    if (bf16)
        bwd::relu_mask_kernel<true><<<dim3((unsigned)blocks), dim3(256), 0, stream>>>(
            static_cast<const bwd::u32x4 *>(y), static_cast<const bwd::u32x4 *>(gy), static_cast<bwd::u32x4 *>(out), n16);
    else
        bwd::relu_mask_kernel<false><<<dim3((unsigned)blocks), dim3(256), 0, stream>>>(
            static_cast<const bwd::u32x4 *>(y), static_cast<const bwd::u32x4 *>(gy), static_cast<bwd::u32x4 *>(out), n16);
    return hipGetLastError();
}

// y may be null (no ReLU).  out: [N,H,W,K]; gy, y: [N,P,Q,K].
hipError_t launch_relu_mask_dilate(const void *y, const void *gy, void *out, int N, int H, int W, int P, int Q, int K,
                                   int stride, int bf16, hipStream_t stream) {
    const size_t row_bytes = (size_t)K * (bf16 ? 2 : 4);
    if (row_bytes % 16 || stride < 1) return hipErrorInvalidValue;
    const size_t n16 = (size_t)N * H * W * (row_bytes / 16);
    if (n16 == 0) return hipSuccess;
    size_t blocks = (n16 + 255) / 256;
    if (blocks > 256 * 16) blocks = 256 * 16;
    if (bf16)
        bwd::relu_mask_dilate_kernel<true><<<dim3((unsigned)blocks), dim3(256), 0, stream>>>(
            static_cast<const bwd::u32x4 *>(y), static_cast<const bwd::u32x4 *>(gy), static_cast<bwd::u32x4 *>(out), H, W,
            P, Q, (int)(row_bytes / 16), stride, n16);
    else
        bwd::relu_mask_dilate_kernel<false><<<dim3((unsigned)blocks), dim3(256), 0, stream>>>(
            static_cast<const bwd::u32x4 *>(y), static_cast<const bwd::u32x4 *>(gy), static_cast<bwd::u32x4 *>(out), H, W,
            P, Q, (int)(row_bytes / 16), stride, n16);
    return hipGetLastError();
}

// out[N,H,W,C] = t[N,P,Q,C] spread to the pixels (stride p, stride q), zero elsewhere, + add (may
// be null), then zero where mask (may be null) is not > 0.
hipError_t launch_spread_add(const void *t, const void *add, const void *mask, void *out, int N, int H, int W, int P,
                             int Q, int C, int stride, int bf16, hipStream_t stream) {
    const size_t row_bytes = (size_t)C * (bf16 ? 2 : 4);
    if (row_bytes % 16 || stride < 1 || (P - 1) * stride >= H || (Q - 1) * stride >= W) return hipErrorInvalidValue;
    const long long npix = (long long)N * H * W;
    if (npix == 0) return hipSuccess;
    if (npix > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    const int vec = (int)(row_bytes / 16);
    int lanes = 1;
    while (lanes < vec && lanes < 256) lanes *= 2;
    long long blocks = (npix + 256 / lanes - 1) / (256 / lanes);
    if (blocks > 256 * 16) blocks = 256 * 16;
    auto run = [&](auto kernel) {
        kernel<<<dim3((unsigned)blocks), dim3(256), 0, stream>>>(
            static_cast<const bwd::u32x4 *>(t), static_cast<const bwd::u32x4 *>(add), static_cast<const bwd::u32x4 *>(mask),
            static_cast<bwd::u32x4 *>(out), H, W, P, Q, vec, stride, lanes, (int)npix, make_divisor(W), make_divisor(H), make_divisor(stride));
    };
    bf16 ? run(bwd::spread_add_kernel<true>) : run(bwd::spread_add_kernel<false>);
    return hipGetLastError();
}

hipError_t launch_bwd_weights(const void *w, const float *scale, void *wt, int K, int R, int S, int C, int bf16,
                              hipStream_t stream) {
    const size_t total = (size_t)K * R * S * C;
    if (total == 0 || total > 0x7FFFFFFFull) return hipErrorInvalidValue;
    const unsigned blocks = (unsigned)((total + 255) / 256);
    if (bf16) bwd::bwd_weights_kernel<true><<<dim3(blocks), dim3(256), 0, stream>>>(w, scale, wt, K, R, S, C);
    else bwd::bwd_weights_kernel<false><<<dim3(blocks), dim3(256), 0, stream>>>(w, scale, wt, K, R, S, C);
    return hipGetLastError();
}

// ---------------------------------------------------------------- weight gradient: which kernel
// `a`: the layer as its weight gradient sees it - its own geometry for a 1x1 layer of any stride, stride 1 for the rest
// (gpre at the input's resolution); a 3x3 stride-2 layer whose gradient comes at the output's resolution: launch_wgrad_s2.

// Splits of the reduction over `pixels` for each of `tiles` tiles: what minimises pixel_ns * pixels / splits (the workgroups'
// own time) + sums_ns * splits * tiles (writing and re-reading their sums), and at most one workgroup per CU in all.
// For the large layers of a ResNet at batch 128 that is one per CU; a layer of 784 pixels and 16 tiles takes 3 splits, where
// as many as there were chunks spent most of the time on 35 MB of partial sums.
int wgrad_splits(long long pixels, int tiles, double pixel_ns, double sums_ns) {
    const long long best = (long long)(sqrt(pixel_ns * (double)pixels / (sums_ns * tiles)) + 0.5), most = 256 / tiles;
    const long long n = best * 4 < most * 3 ? best : most;       // near one workgroup per CU: exactly that
    return n < 1 ? 1 : (int)n;
}

static const char *wgrad_f32_check(const ConvArgs &a) {
    if (a.R != a.S || (a.R != 1 && a.R != 3) || (a.stride != 1 && a.R != 1) || a.pad != (a.R - 1) / 2)
        return "weight gradient: 1x1 or 3x3, stride 1, same padding only";
    if (a.Cin % 16 || a.Cout % 16) return "weight gradient (fp32): channel counts must be multiples of 16";
    if (a.N < 1 || a.H < 1 || a.W < 1 || a.Cout / 16 > 65535 || a.Cin / 16 > 65535)
        return "weight gradient (fp32): empty or oversized layer";
    return nullptr;
}

const char *wgrad_check(const ConvArgs &a) {
    if (!a.bf16) return wgrad_f32_check(a);
    if (a.R != a.S || (a.R != 1 && a.R != 3) || (a.stride != 1 && a.R != 1) || a.pad != (a.R - 1) / 2)
        return "weight gradient: 1x1 or 3x3, stride 1, same padding only";
    return a.R == 1 ? wgrad1x1_check(a) : wgrad3x3_check(a);
}

// fp32: 32 x 32 tiles where they fill the chip by themselves (half the loads per product), else 16 x 16; 32-bit offsets where stride and
// sizes allow.
static bool wgrad_f32_wide(const ConvArgs &a) {
    return a.Cout % 32 == 0 && a.Cin % 32 == 0 && (long long)(a.Cout / 32) * (a.Cin / 32) * a.R * a.S >= 256;
}
static bool wgrad_f32_flat(const ConvArgs &a) {
    return a.stride == 1 && (long long)a.N * a.P * a.Q * (a.Cin > a.Cout ? a.Cin : a.Cout) * 4 <= 0x7FFFFFFFLL;
}

const char *wgrad_kernel_name(const ConvArgs &a) {
    if (a.bf16) return a.R == 1 ? "wgrad1x1 bf16" : "wgrad3x3 bf16";
    if (wgrad_f32_flat(a)) return wgrad_f32_wide(a) ? "wgrad_f32 32x32, 32-bit offsets" : "wgrad_f32 16x16, 32-bit offsets";
    return wgrad_f32_wide(a) ? "wgrad_f32 32x32, 64-bit addresses" : "wgrad_f32 16x16, 64-bit addresses";
}

size_t wgrad_workspace_bytes(const ConvArgs &a) {
    if (!a.bf16 || wgrad_check(a)) return 0;
    return a.R == 1 ? wgrad1x1_workspace_bytes(a) : wgrad3x3_workspace_bytes(a);
}

// g = gpre [N,P,Q,Cout]; a.x = x, a.scale = scale; gw [Cout][R][S][Cin] fp32; workspace of at least
// wgrad_workspace_bytes(a), 16-byte aligned (none for fp32).
hipError_t launch_wgrad(const ConvArgs &a, const void *g, float *gw, void *workspace, size_t workspace_bytes,
                        hipStream_t stream) {
    if (wgrad_check(a) || !a.x || !a.scale || !g || !gw) return hipErrorInvalidValue;
    if (a.bf16)
        return a.R == 1 ? launch_wgrad1x1(a, g, gw, workspace, workspace_bytes, stream)
                        : launch_wgrad3x3(a, g, gw, workspace, workspace_bytes, stream);
    const int taps = a.R * a.S;
    const bool wide = wgrad_f32_wide(a);
    const long long M = (long long)a.N * a.P * a.Q;
    const float *x = static_cast<const float *>(a.x), *gf = static_cast<const float *>(g);
    const dim3 grid = wide ? dim3(a.Cout / 32, a.Cin / 32, taps) : dim3(a.Cout / 16, a.Cin / 16, taps);
    if (wgrad_f32_flat(a)) {
        auto run = [&](auto kernel) {
            kernel<<<grid, dim3(1024), 0, stream>>>(x, gf, a.scale, gw, a.P, a.Q, a.Cin, a.Cout, a.R, a.pad, (int)M, make_divisor(a.P * a.Q),
                                                    make_divisor(a.Q));
        };
        if (a.R == 1) wide ? run(bwd::wgrad_f32_flat_kernel<2, false>) : run(bwd::wgrad_f32_flat_kernel<1, false>);
        else wide ? run(bwd::wgrad_f32_flat_kernel<2, true>) : run(bwd::wgrad_f32_flat_kernel<1, true>);
        return hipGetLastError();
    }
    auto run = [&](auto kernel) {
        kernel<<<grid, dim3(1024), 0, stream>>>(x, gf, a.scale, gw, a.P, a.Q, a.Cin, a.Cout, a.R, a.pad, a.H, a.W, a.stride, M);
    };
    if (a.stride == 1) wide ? run(bwd::wgrad_f32_kernel<2, false>) : run(bwd::wgrad_f32_kernel<1, false>);
    else wide ? run(bwd::wgrad_f32_kernel<2, true>) : run(bwd::wgrad_f32_kernel<1, true>);
    return hipGetLastError();
}

// The weight gradient of a 3x3 stride-2 pad-1 bf16 layer from dL/d(pre-activation) at the OUTPUT's resolution: where the one-launch
// kernel has a plan, that is up to 51 output columns.  Wider layers spread the gradient out and take the stride-1 kernel.
bool wgrad_s2_applies(const ConvArgs &a) {
    return a.bf16 && a.R == 3 && a.S == 3 && a.stride == 2 && a.pad == 1 && a.Cin % 128 == 0 && a.Cout % 128 == 0 &&
           a.P == (a.H - 1) / 2 + 1 && a.Q == (a.W - 1) / 2 + 1 && !wgrad3x3_check(a);
}

size_t wgrad_s2_workspace_bytes(const ConvArgs &a) {
    return wgrad_s2_applies(a) ? (wgrad3x3_workspace_bytes(a) + 255) / 256 * 256 : 0;
}

hipError_t launch_wgrad_s2(const ConvArgs &a, const void *g, float *gw, void *workspace, size_t workspace_bytes,
                           hipStream_t stream) {
    if (!wgrad_s2_applies(a)) return hipErrorInvalidValue;
    return launch_wgrad3x3(a, g, gw, workspace, workspace_bytes, stream);
}

}  // namespace delta
