// The fp32 weight gradient of stride-1 layers, one tile of (k, c) of one tap: the body of backward.hip's kernel (sixteen wavefronts) and of
// small_backward.hip's (eight).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"

namespace delta {

// The form for stride 1 and tensors below 2 GiB: 32-bit offsets, and buffer loads that return zero for an offset outside the
// tensor, which is where positions past a wavefront's run and taps outside the image point: 8 instructions per MFMA for a 1x1
// layer, about 20 with taps.  Sixteen steps in flight for T = 1 without taps (a run of 128 positions is two round trips; with
// taps eight are better, 9.6 us against 11.3: the address arithmetic of a round runs before its first product).
// Two rounds in flight in two register sets were slower (7 % of a stack of such layers: the address arithmetic doubles).
// 2 x 32 x 32 positions, us by the form with 64-bit addresses -> this one: 64 -> 256 10.0 -> 7.0, 256 -> 64 10.0 -> 9.1, 64 -> 64 10.0 -> 6.5, 3x3
// 64 -> 64 10.0 -> 9.6.
// Two sums and a tree over the wavefronts: 2.1e-7 from 64 bits (norm) at 2048 positions whether 8 or 16 wavefronts share them; 512 -> 512 on 8192
// positions 2.1e-7, with one sum 2.9e-7.
// part: kWaves T T 256 floats of LDS, factors: 64 more.
template <int T, bool TAPS, int kWaves>
__device__ __forceinline__ void wgrad_f32_tile(const float *x, const float *g, const float *scale, float *gw, int H, int W, int C, int K, int R,
                                               int pad, int M, Divisor dhw, Divisor dw, int k0, int c0, int tap, int tid, float *part,
                                               float *factors) {
    typedef uint32_t uvec __attribute__((ext_vector_type(T)));
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    constexpr int kOutOfRange = (int)0x80000000;                 // outside both buffer descriptors
    constexpr int kSteps = T == 1 && !TAPS ? 16 : 8;
    const int lane = tid & 63, l16 = lane & 15, quad = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (wv == 0) {                                               // scale of the tile's channels, straight into LDS
        typedef __attribute__((address_space(3))) float *lptr_t;
        load_lds_b32(scale + k0 + (lane & (16 * T - 1)), (uint32_t)(uintptr_t)(lptr_t)factors);
    }
    const int dr = TAPS ? tap / R - pad : 0, ds = TAPS ? tap % R - pad : 0;
    const int per = ((M + kWaves - 1) / kWaves + 3) / 4 * 4;
    const int first = wv * per, end = first + per < M ? first + per : M;
    const __amdgpu_buffer_rsrc_t grsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(g), 0, (int)((size_t)M * K * 4), 0x00020000);
    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(x), 0, (int)((size_t)M * C * 4), 0x00020000);
    auto fetch = [&](__amdgpu_buffer_rsrc_t r, uint32_t off) {
        if constexpr (T == 1) return uvec{__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0)};
        else return __builtin_bit_cast(uvec, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0));
    };
    int m = first + quad, h = 0, w = 0;                          // this lane's position
    if constexpr (TAPS) {
        const int rest = m - divide(m, dhw) * (H * W);
        h = divide(rest, dw);
        w = rest - h * W;
    }
    const int hstep = 4 / W % H, wstep = 4 % W;                  // four positions on: at most one carry each
    uint32_t goff = ((uint32_t)m * (uint32_t)K + (uint32_t)(k0 + T * l16)) * 4u;
    uint32_t xoff = ((uint32_t)(m + dr * W + ds) * (uint32_t)C + (uint32_t)(c0 + T * l16)) * 4u;
    // Two sums half as long instead of one: of every other step, in registers of their own - or, where those would be the ones that the steps in
    // flight need (16 wavefronts, T = 2: the compiler then fetched each step when it was used, 512 -> 512 on 8192 positions 55 -> 69 us), of the
    // first half of the run, which waits in this wavefront's part of the LDS.
    constexpr int kSums = T == 2 && kWaves == 16 ? 1 : 2;
    f32x4 acc[kSums][T][T];
#pragma unroll
    for (int u = 0; u < kSums; ++u)
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
            for (int j = 0; j < T; ++j) acc[u][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    float *mine = part + wv * (T * T * 256) + lane;
    int m0 = first, stop = kSums == 2 || end <= first ? end : first + (end - first) / 2 / (4 * kSteps) * (4 * kSteps);
    for (;;) {
        for (; m0 < stop; m0 += 4 * kSteps) {
            uvec gv[kSteps], xv[kSteps];
#pragma unroll
            for (int u = 0; u < kSteps; ++u) {
                bool in = m < end;
                if constexpr (TAPS) in = in & ((unsigned)(h + dr) < (unsigned)H) & ((unsigned)(w + ds) < (unsigned)W);
                gv[u] = fetch(grsrc, in ? goff : (uint32_t)kOutOfRange);        // both zero: no Inf of one meets a zero of the other
                xv[u] = fetch(xrsrc, in ? xoff : (uint32_t)kOutOfRange);
                m += 4;
                goff += (uint32_t)K * 16u;
                xoff += (uint32_t)C * 16u;
                if constexpr (TAPS) {
                    w += wstep;
                    const bool carry = w >= W;
                    w -= carry ? W : 0;
                    h += hstep + (carry ? 1 : 0);
                    h -= h >= H ? H : 0;
                }
            }
#pragma unroll
            for (int u = 0; u < kSteps; ++u)
#pragma unroll
                for (int i = 0; i < T; ++i)
#pragma unroll
                    for (int j = 0; j < T; ++j)
                        acc[u % kSums][i][j] =
                            __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(gv[u][i]), __uint_as_float(xv[u][j]), acc[u % kSums][i][j], 0, 0, 0);
        }
        if (kSums == 2 || stop == end) break;
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
            for (int j = 0; j < T; ++j) {
#pragma unroll
                for (int e = 0; e < 4; ++e) mine[((i * T + j) * 4 + e) * 64] = acc[0][i][j][e];
                acc[0][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        stop = end;
    }
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float *at = mine + ((i * T + j) * 4 + e) * 64;
                *at = acc[0][i][j][e] + (kSums == 2 ? acc[kSums - 1][i][j][e] : end > first ? *at : 0.f);
            }
    if (wv == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
#pragma unroll
    for (int at = tid; at < T * T * 256; at += kWaves * 64) {
        float level[kWaves];                                     // in pairs: fewer roundings of the whole sum
#pragma unroll
        for (int v = 0; v < kWaves; ++v) level[v] = part[v * (T * T * 256) + at];
#pragma unroll
        for (int n = kWaves / 2; n; n /= 2)
#pragma unroll
            for (int v = 0; v < n; ++v) level[v] += level[v + n];
        // lane of this sum: column (c) l % 16, row (k) 4 (l / 16) + e of the tile's (i, j) interleave
        const int kl = T * (4 * quad + ((at >> 6) & 3)) + (at >> 8) / T, k = k0 + kl, c = c0 + T * l16 + (at >> 8) % T;
        gw[((size_t)k * R * R + tap) * C + c] = level[0] * factors[kl];
    }
}

}  // namespace delta
