// Backward of the layers around the bottleneck stack (bf16): max pooling, global average
// pooling, the classifier and the cross-entropy loss.  With backward.hip they make the backward
// half of a ResNet training iteration, the pass whose accesses to stored activations DELTA's
// planner follows (Sec. 3, Assumptions 1-3).  All of them are memory-bound and small next to the
// convolutions; they are written for bytes per thread and coalescing, not for the matrix cores.
// Nothing here uses atomics: every output element is produced by exactly one thread, in a fixed
// order of additions.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "kernels.hpp"

namespace delta {
namespace bops {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

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
__device__ __forceinline__ u32x4 pack8(const float (&f)[8]) {
    u32x4 o;
    o.x = pack2(f[0], f[1]); o.y = pack2(f[2], f[3]); o.z = pack2(f[4], f[5]); o.w = pack2(f[6], f[7]);
    return o;
}

// ---------------------------------------------------------------- max pooling
// A workgroup owns an 8 x 8 tile of INPUT pixels and 64 channels (8 chunks of 8), in three steps:
//  1. copy every pixel that a window touching the tile can reach (the tile plus R-1 / S-1 pixels
//     on each side) into LDS, and the gradients of those windows with them (one global round trip
//     for both; step 3 then reads each window's gradient from LDS instead of once per pixel);
//  2. one thread per (window, chunk): scan the window in the forward's order (r, then s, padding
//     skipped) and record, per channel, the position r*S + s of the first maximal element as
//     one byte (255: none) - each window is scanned once, not once per pixel it covers;
//  3. one thread per (pixel, chunk): for each of the at most ceil(R/stride) x ceil(S/stride)
//     windows containing the pixel, add the window's gradient where the recorded position is
//     the pixel's.  Sums in window order (p, then q), fp32.
// Every loop has a uniform trip count and selects instead of branches: a per-element `if`
// compiled to a branch per element and ran ten times slower.  The kernel is bound by its vector
// arithmetic (about 3300 wavefront instructions per tile): XCD-aware tile numbering and trip counts
// made uniform per wavefront by pixel parity class both left its time unchanged; scanning only the
// windows that can touch the tile (5 x 5 instead of 6 x 6 for the 3 x 3 stride-2 pool) took 16 % off.
static constexpr int kPoolTile = 8, kPoolChunks = 8;

// windows p with a pixel in kPoolTile consecutive rows: stride * p - pad in [h0 - R + 1, h0 + kPoolTile - 1],
// an interval of length kPoolTile + R - 2
__host__ __device__ inline int pool_windows_max(int R, int stride) { return (kPoolTile + R - 2) / stride + 1; }

__global__ __launch_bounds__(256) void maxpool_bwd_kernel(PoolArgs a, const void *gy, void *gx, int tiles_w, int tiles_h,
                                                          int mask_x) {
    extern __shared__ __align__(16) unsigned char plds[];
    const int chunks = a.C / 8, cgroups = (chunks + kPoolChunks - 1) / kPoolChunks;
    int blk = blockIdx.x;
    const int cg = blk % cgroups; blk /= cgroups;
    const int tw = blk % tiles_w; blk /= tiles_w;
    const int th = blk % tiles_h;
    const int n = blk / tiles_h;
    const int h0 = th * kPoolTile, w0 = tw * kPoolTile;
    const int LH = kPoolTile + 2 * (a.R - 1), LW = kPoolTile + 2 * (a.S - 1);
    const int NWH = pool_windows_max(a.R, a.stride), NWW = pool_windows_max(a.S, a.stride);
    unsigned char *arg = plds + (size_t)LH * LW * kPoolChunks * 16;      // [NWH][NWW][chunk] x 8 bytes
    unsigned char *gys = arg + (size_t)NWH * NWW * kPoolChunks * 8;      // [NWH][NWW][chunk] x 16 bytes
    const unsigned char *xg = static_cast<const unsigned char *>(a.x);
    const unsigned char *gg = static_cast<const unsigned char *>(gy);
    // windows that contain a pixel of the tile: p in [pw0, pw0 + NWH) clipped to the image (likewise q)
    int pw0 = h0 + a.pad - a.R + 1;
    pw0 = pw0 <= 0 ? 0 : (pw0 + a.stride - 1) / a.stride;
    int qw0 = w0 + a.pad - a.S + 1;
    qw0 = qw0 <= 0 ? 0 : (qw0 + a.stride - 1) / a.stride;
    // step 1: LDS pixel (lh, lw) = image pixel (h0 - (R-1) + lh, w0 - (S-1) + lw); outside the image: zeros, unused
    for (int i = threadIdx.x; i < LH * LW * kPoolChunks; i += 256) {
        const int c = i % kPoolChunks, pix = i / kPoolChunks;
        const int lh = pix / LW, lw = pix - lh * LW;
        const int hh = h0 - (a.R - 1) + lh, ww = w0 - (a.S - 1) + lw, ck = cg * kPoolChunks + c;
        u32x4 v = {0u, 0u, 0u, 0u};
        if ((unsigned)hh < (unsigned)a.H && (unsigned)ww < (unsigned)a.W && ck < chunks)
            v = *reinterpret_cast<const u32x4 *>(xg + ((((size_t)n * a.H + hh) * a.W + ww) * chunks + ck) * 16);
        *reinterpret_cast<u32x4 *>(plds + (size_t)i * 16) = v;
    }
    for (int i = threadIdx.x; i < NWH * NWW * kPoolChunks; i += 256) {
        const int c = i % kPoolChunks, win = i / kPoolChunks;
        const int p = pw0 + win / NWW, q = qw0 + win % NWW, ck = cg * kPoolChunks + c;
        u32x4 v = {0u, 0u, 0u, 0u};
        if (p < a.P && q < a.Q && ck < chunks)
            v = *reinterpret_cast<const u32x4 *>(gg + ((((size_t)n * a.P + p) * a.Q + q) * chunks + ck) * 16);
        *reinterpret_cast<u32x4 *>(gys + (size_t)i * 16) = v;
    }
    __syncthreads();
    // step 2
    for (int i = threadIdx.x; i < NWH * NWW * kPoolChunks; i += 256) {
        const int c = i % kPoolChunks, win = i / kPoolChunks;
        const int wp = win / NWW, wq = win - wp * NWW;
        const int hb = (pw0 + wp) * a.stride - a.pad, wb = (qw0 + wq) * a.stride - a.pad;
        float m[8];
        uint32_t idx[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) { m[e] = -INFINITY; idx[e] = 255u; }
#pragma unroll
        for (int r = 0; r < a.R; ++r)
#pragma unroll
            for (int s = 0; s < a.S; ++s) {
                const int hh = hb + r, ww = wb + s;
                const bool inside = (unsigned)hh < (unsigned)a.H && (unsigned)ww < (unsigned)a.W;
                // windows beyond the tile's reach (or the image) are never consulted: clamp their reads
                int lh = hh - h0 + a.R - 1, lw = ww - w0 + a.S - 1;
                lh = lh < 0 ? 0 : (lh > LH - 1 ? LH - 1 : lh);
                lw = lw < 0 ? 0 : (lw > LW - 1 ? LW - 1 : lw);
                float v[8];
                unpack8(*reinterpret_cast<const u32x4 *>(plds + ((size_t)(lh * LW + lw) * kPoolChunks + c) * 16), v);
                const uint32_t pos = (uint32_t)(r * a.S + s);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const bool take = inside && v[e] > m[e];
                    m[e] = take ? v[e] : m[e];
                    idx[e] = take ? pos : idx[e];
                }
            }
        u32x2 o;
        o.x = idx[0] | (idx[1] << 8) | (idx[2] << 16) | (idx[3] << 24);
        o.y = idx[4] | (idx[5] << 8) | (idx[6] << 16) | (idx[7] << 24);
        *reinterpret_cast<u32x2 *>(arg + (size_t)i * 8) = o;
    }
    __syncthreads();
    // step 3
    const int np = (a.R + a.stride - 1) / a.stride, nq = (a.S + a.stride - 1) / a.stride;
    for (int i = threadIdx.x; i < kPoolTile * kPoolTile * kPoolChunks; i += 256) {
        const int c = i % kPoolChunks, pix = i / kPoolChunks;
        const int h = h0 + pix / kPoolTile, w = w0 + pix % kPoolTile, ck = cg * kPoolChunks + c;
        const bool owned = h < a.H && w < a.W && ck < chunks;
        int p_lo = h + a.pad - a.R + 1;
        p_lo = p_lo <= 0 ? 0 : (p_lo + a.stride - 1) / a.stride;
        int p_hi = (h + a.pad) / a.stride;
        if (p_hi > a.P - 1) p_hi = a.P - 1;
        int q_lo = w + a.pad - a.S + 1;
        q_lo = q_lo <= 0 ? 0 : (q_lo + a.stride - 1) / a.stride;
        int q_hi = (w + a.pad) / a.stride;
        if (q_hi > a.Q - 1) q_hi = a.Q - 1;
        float acc[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = 0.f;
#pragma unroll
        for (int dp = np - 1; dp >= 0; --dp)                       // ascending p, then q: the order of the sums
#pragma unroll
            for (int dq = nq - 1; dq >= 0; --dq) {
                const int p = p_hi - dp, q = q_hi - dq;
                const bool live = owned && p >= p_lo && q >= q_lo;  // this pixel lies in window (p, q)
                // clamped to the windows steps 1 and 2 covered: the LDS reads stay in bounds
                const int pc = p < pw0 ? pw0 : (p > pw0 + NWH - 1 ? pw0 + NWH - 1 : p);
                const int qc = q < qw0 ? qw0 : (q > qw0 + NWW - 1 ? qw0 + NWW - 1 : q);
                const size_t slot = (size_t)((pc - pw0) * NWW + (qc - qw0)) * kPoolChunks + c;
                const u32x2 am = *reinterpret_cast<const u32x2 *>(arg + slot * 8);
                float g[8];
                unpack8(*reinterpret_cast<const u32x4 *>(gys + slot * 16), g);
                const uint32_t my = (uint32_t)((h - (p * a.stride - a.pad)) * a.S + (w - (q * a.stride - a.pad)));
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const uint32_t pos = ((e < 4 ? am.x : am.y) >> (8 * (e & 3))) & 0xFFu;
                    acc[e] += (live && pos == my) ? g[e] : 0.f;
                }
            }
        if (owned) {
            u32x4 o = pack8(acc);
            if (mask_x) {                                           // also the ReLU mask of x's producer: x is its output
                const int lh = h - h0 + a.R - 1, lw = w - w0 + a.S - 1;
                const u32x4 xv = *reinterpret_cast<const u32x4 *>(plds + ((size_t)(lh * LW + lw) * kPoolChunks + c) * 16);
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = keep_where_positive_bf16(o[e], xv[e]);
            }
            *reinterpret_cast<u32x4 *>(static_cast<unsigned char *>(gx) +
                                       ((((size_t)n * a.H + h) * a.W + w) * chunks + ck) * 16) = o;
        }
    }
}

// The ResNet pool (3 x 3, stride 2, padding 1), packed.  The three steps are those of maxpool_bwd_kernel on 8 x 16 pixels x 64
// channels, but everything that can works on two channels per instruction: the general kernel is bound by its vector
// arithmetic (about 50 instructions per input element and 64 lanes), this one by HBM.
//  1. A staged value becomes a signed 16-bit integer t of the same order: its magnitude, negated where the sign is set (-0 and +0
//     meet at 0; -inf is -0x7F80 and a negative NaN lies below it; a positive NaN, found by an OR over the piece, and a
//     pixel outside the image become -0x8000).
//  2. Window scan: the maximum over r, s of (t << 16 | 8 - position) is the value and its first position at once, two
//     positions per max3.  Nothing wins that is not above -inf, as with a comparison against a running maximum.  The
//     position is stored one-hot, 16 bits per channel.
//  3. A thread owns 2 x 2 pixels and 8 channels: with a stride of 2 they have 1, 2, 2 and 4 windows, nine contributions
//     where a pixel at a time has up to sixteen.  A contribution is gy masked by its position's bit (two shifts and an
//     AND for two channels); only pixels with several windows go through fp32, summed in window order (p, then q).
//     (The sign of a zero is the one difference: a gradient of -0 stays -0.)
// 8 x 16 pixels: a tile stages 11 x 19 for its 128, and 38 KB of LDS leave room for four workgroups on a CU.
// 128 x 112 x 112 x 64, 462 MB: 182 us by the general kernel with its loops unrolled for this window, 102 us (4.5 TB/s) here;
// a copy of 1 GiB reaches 4.7 TB/s.
static constexpr int kPackTH = 8, kPackTW = 16, kPackLH = kPackTH + 3, kPackLW = kPackTW + 3;
static constexpr int kPackWH = kPackTH / 2 + 1, kPackWW = kPackTW / 2 + 1;
typedef short s16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pk_ashr15(uint32_t v) { return __builtin_bit_cast(uint32_t, __builtin_bit_cast(s16x2, v) >> (short)15); }
__device__ __forceinline__ uint32_t pk_sub(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, (s16x2)(__builtin_bit_cast(s16x2, a) - __builtin_bit_cast(s16x2, b)));
}
template <int BIT>
__device__ __forceinline__ uint32_t pk_bit_mask(uint32_t onehot) {       // 0xFFFF in the halves whose bit BIT is set
    return pk_ashr15(__builtin_bit_cast(uint32_t, (s16x2)(__builtin_bit_cast(s16x2, onehot) << (short)(15 - BIT))));
}
template <int R, int S>
__device__ __forceinline__ u32x4 taken(const u32x4 g, const u32x4 onehot) {      // gy where the window's maximum is position (R, S)
    u32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = g[e] & pk_bit_mask<R * 3 + S>(onehot[e]);
    return o;
}

__global__ __launch_bounds__(256) void maxpool_bwd_packed_kernel(PoolArgs a, const void *gy, void *gx, int tiles_w, int tiles_h, int mask_x) {
    __shared__ __align__(16) u32x4 ts[kPackLH * kPackLW * kPoolChunks], hot[kPackWH * kPackWW * kPoolChunks], gys[kPackWH * kPackWW * kPoolChunks];
    const int chunks = a.C / 8, cgroups = (chunks + kPoolChunks - 1) / kPoolChunks;
    // each XCD (blockIdx % 8) takes a contiguous run of tiles: the rows neighbouring tiles share are fetched into one L2
    unsigned blk;
    {
        const unsigned nb = gridDim.x, per = nb >> 3, rem = nb & 7u, xcd = blockIdx.x & 7u, idx = blockIdx.x >> 3;
        blk = xcd < rem ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
    }
    const int cg = (int)(blk % cgroups); blk /= cgroups;
    const int tw = (int)(blk % tiles_w); blk /= tiles_w;
    const int th = (int)(blk % tiles_h), n = (int)(blk / tiles_h);
    const int h0 = th * kPackTH, w0 = tw * kPackTW, p0 = h0 / 2, q0 = w0 / 2;
    const int c = threadIdx.x % kPoolChunks, ck = cg * kPoolChunks + c, first = threadIdx.x / kPoolChunks;
    const bool has = ck < chunks;
    const u32x4 *xg = static_cast<const u32x4 *>(a.x) + (size_t)n * a.H * a.W * chunks + (has ? ck : 0);
    const u32x4 *gg = static_cast<const u32x4 *>(gy) + (size_t)n * a.P * a.Q * chunks + (has ? ck : 0);
    // ---- step 1: LDS pixel (lh, lw) = image pixel (h0 - 1 + lh, w0 - 1 + lw)
    constexpr int kStep = 256 / kPoolChunks, kPix = (kPackLH * kPackLW + kStep - 1) / kStep, kWin = (kPackWH * kPackWW + kStep - 1) / kStep;
    u32x4 xv[kPix], gv[kWin];
#pragma unroll
    for (int i = 0; i < kPix; ++i) {
        const int pix = first + i * kStep, lh = pix / kPackLW, lw = pix - lh * kPackLW, hh = h0 - 1 + lh, ww = w0 - 1 + lw;
        const bool in = ((unsigned)hh < (unsigned)a.H) & ((unsigned)ww < (unsigned)a.W);
        xv[i] = xg[in ? (size_t)(hh * a.W + ww) * chunks : 0];
    }
#pragma unroll
    for (int i = 0; i < kWin; ++i) {
        const int win = first + i * kStep, p = p0 + win / kPackWW, q = q0 + win % kPackWW;
        gv[i] = gg[(p < a.P) & (q < a.Q) ? (size_t)(p * a.Q + q) * chunks : 0];
    }
#pragma unroll
    for (int i = 0; i < kPix; ++i) {
        const int pix = first + i * kStep, lh = pix / kPackLW, lw = pix - lh * kPackLW, hh = h0 - 1 + lh, ww = w0 - 1 + lw;
        const bool in = ((unsigned)hh < (unsigned)a.H) & ((unsigned)ww < (unsigned)a.W);
        u32x4 t;
        uint32_t nan = 0u;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t v = xv[i][e], mag = v & 0x7FFF7FFFu, sign = pk_ashr15(v);
            t[e] = pk_sub(mag ^ sign, sign);
            nan |= mag + 0x007F007Fu;                            // the top bit of a half: its magnitude is beyond infinity's
        }
        if (nan & 0x80008000u) {                                 // rare: no NaN wins
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t bad = pk_ashr15((xv[i][e] & 0x7FFF7FFFu) + 0x007F007Fu);
                t[e] = (t[e] & ~bad) | (0x80008000u & bad);
            }
        }
        if (pix < kPackLH * kPackLW) ts[pix * kPoolChunks + c] = in ? t : u32x4{0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u};
    }
#pragma unroll
    for (int i = 0; i < kWin; ++i) {
        const int win = first + i * kStep;
        if (win < kPackWH * kPackWW) gys[win * kPoolChunks + c] = gv[i];
    }
    __syncthreads();
    // ---- step 2
    for (int win = first; win < kPackWH * kPackWW; win += kStep) {
        const int wp = win / kPackWW, wq = win - wp * kPackWW;
        const bool real = (p0 + wp < a.P) & (q0 + wq < a.Q);
        int m[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) m[e] = (int)0x80000000;
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                const u32x4 v = ts[((2 * wp + r) * kPackLW + 2 * wq + s) * kPoolChunks + c];
                const uint32_t rank = 8 - (r * 3 + s);           // of equal values the first position wins
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int lo = (int)((v[e] << 16) | rank), hi = (int)((v[e] & 0xFFFF0000u) | rank);
                    m[2 * e] = m[2 * e] > lo ? m[2 * e] : lo;
                    m[2 * e + 1] = m[2 * e + 1] > hi ? m[2 * e + 1] : hi;
                }
            }
        u32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t lo = real && m[2 * e] >= (int)0x80810000 ? 1u << (8 - (m[2 * e] & 15)) : 0u;          // above -inf
            const uint32_t hi = real && m[2 * e + 1] >= (int)0x80810000 ? 0x10000u << (8 - (m[2 * e + 1] & 15)) : 0u;
            o[e] = lo | hi;
        }
        hot[win * kPoolChunks + c] = o;
    }
    __syncthreads();
    // ---- step 3
    static_assert((kPackTH / 2) * (kPackTW / 2) == kStep, "one 2 x 2 block of pixels per thread");
    const int i = first / (kPackTW / 2), j = first % (kPackTW / 2);
    const int w00 = (i * kPackWW + j) * kPoolChunks + c;
    const u32x4 g00 = gys[w00], g01 = gys[w00 + kPoolChunks], g10 = gys[w00 + kPackWW * kPoolChunks], g11 = gys[w00 + (kPackWW + 1) * kPoolChunks];
    const u32x4 k00 = hot[w00], k01 = hot[w00 + kPoolChunks], k10 = hot[w00 + kPackWW * kPoolChunks], k11 = hot[w00 + (kPackWW + 1) * kPoolChunks];
    u32x4 o[4];                                                  // pixels (2i, 2j), (2i, 2j + 1), (2i + 1, 2j), (2i + 1, 2j + 1)
    o[0] = taken<1, 1>(g00, k00);
    const u32x4 a1 = taken<1, 2>(g00, k00), b1 = taken<1, 0>(g01, k01), a2 = taken<2, 1>(g00, k00), b2 = taken<0, 1>(g10, k10);
    const u32x4 a3 = taken<2, 2>(g00, k00), b3 = taken<2, 0>(g01, k01), c3 = taken<0, 2>(g10, k10), d3 = taken<0, 0>(g11, k11);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        o[1][e] = pack2(lo16(a1[e]) + lo16(b1[e]), hi16(a1[e]) + hi16(b1[e]));
        o[2][e] = pack2(lo16(a2[e]) + lo16(b2[e]), hi16(a2[e]) + hi16(b2[e]));
        o[3][e] = pack2(((lo16(a3[e]) + lo16(b3[e])) + lo16(c3[e])) + lo16(d3[e]), ((hi16(a3[e]) + hi16(b3[e])) + hi16(c3[e])) + hi16(d3[e]));
    }
    u32x4 *out = static_cast<u32x4 *>(gx) + (size_t)n * a.H * a.W * chunks + ck;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int lh = 2 * i + (u >> 1), lw = 2 * j + (u & 1), h = h0 + lh, w = w0 + lw;
        if (mask_x) {                                            // also the ReLU mask of x's producer: x is its output
            const u32x4 t = ts[((lh + 1) * kPackLW + lw + 1) * kPoolChunks + c];
#pragma unroll
            for (int e = 0; e < 4; ++e) o[u][e] &= pk_ashr15(pk_sub(0u, t[e])) & ~pk_ashr15(t[e]);       // t > 0
        }
        if (has && h < a.H && w < a.W) out[(size_t)(h * a.W + w) * chunks] = o[u];
    }
}

// ---------------------------------------------------------------- global average pooling
// gx[n,h,w,c] = gy[n,c] / (H W); one thread per 8 channels of one input pixel.
__global__ __launch_bounds__(256) void avgpool_bwd_kernel(const void *gy, void *gx, int HW, int chunks, long long total) {
    const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    const int ck = (int)(idx % chunks);
    const long long n = idx / chunks / HW;
    float g[8];
    unpack8(*reinterpret_cast<const u32x4 *>(static_cast<const unsigned char *>(gy) + ((size_t)n * chunks + ck) * 16), g);
    const float inv = 1.0f / (float)HW;
#pragma unroll
    for (int e = 0; e < 8; ++e) g[e] *= inv;
    *reinterpret_cast<u32x4 *>(static_cast<unsigned char *>(gx) + (size_t)idx * 16) = pack8(g);
}

// ---------------------------------------------------------------- cross-entropy
// dL/dz[i,k] = (softmax(z_i)[k] - [k == label_i]) / N.  One wavefront per image; fixed reduction trees.
// HELD: the image's logits in registers, PER_LANE 16-byte pieces of 8 classes per lane, read once and written once
// (classes a multiple of 8, at most PER_LANE * 512); else three passes over the row, a class per lane and step.
// 128 images of 1000 classes, latency-bound: 12 us with three passes of 2-byte loads, 4 held (kernel trace).
template <int PER_LANE>
__global__ __launch_bounds__(256) void softmax_ce_bwd_held_kernel(const uint16_t *logits, const long long *labels, int N,
                                                                  int classes, uint16_t *gz) {
    const int lane = threadIdx.x & 63;
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= N) return;
    const int pieces = classes / 8;
    const u32x4 *z = reinterpret_cast<const u32x4 *>(logits + (size_t)i * classes);
    const long long lab = labels[i];
    float v[PER_LANE][8], mx = -INFINITY;
#pragma unroll
    for (int p = 0; p < PER_LANE; ++p) {
        const bool in = lane + 64 * p < pieces;
        unpack8(z[in ? lane + 64 * p : 0], v[p]);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            v[p][e] = in ? v[p][e] : -INFINITY;
            mx = fmaxf(mx, v[p][e]);
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    float se = 0.f;
#pragma unroll
    for (int p = 0; p < PER_LANE; ++p)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const bool in = lane + 64 * p < pieces;              // past the row: no term, whatever the maximum is
            v[p][e] = __expf(v[p][e] - mx);
            se += in ? v[p][e] : 0.f;
        }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) se += __shfl_xor(se, o);
    const float inv = 1.0f / se, invn = 1.0f / (float)N;
    const bool bad = lab < 0 || lab >= classes;                  // a bad label cannot pass unnoticed
#pragma unroll
    for (int p = 0; p < PER_LANE; ++p) {
        if (lane + 64 * p >= pieces) continue;
        float g[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            g[e] = v[p][e] * inv - ((lane + 64 * p) * 8 + e == lab ? 1.0f : 0.0f);
            g[e] = bad ? __builtin_nanf("") : g[e] * invn;
        }
        reinterpret_cast<u32x4 *>(gz + (size_t)i * classes)[lane + 64 * p] = pack8(g);
    }
}

__global__ __launch_bounds__(256) void softmax_ce_bwd_kernel(const uint16_t *logits, const long long *labels, int N,
                                                             int classes, uint16_t *gz) {
    const int lane = threadIdx.x & 63;
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= N) return;
    const uint16_t *z = logits + (size_t)i * classes;
    float mx = -INFINITY;
    for (int c = lane; c < classes; c += 64) mx = fmaxf(mx, __uint_as_float((uint32_t)z[c] << 16));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    float se = 0.f;
    for (int c = lane; c < classes; c += 64) se += __expf(__uint_as_float((uint32_t)z[c] << 16) - mx);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) se += __shfl_xor(se, o);
    const float inv = 1.0f / se, invn = 1.0f / (float)N;
    const long long lab = labels[i];
    for (int c = lane; c < classes; c += 64) {
        float g = __expf(__uint_as_float((uint32_t)z[c] << 16) - mx) * inv;
        if (c == lab) g -= 1.0f;
        if (lab < 0 || lab >= classes) g = __builtin_nanf("");     // a bad label cannot pass unnoticed
        gz[(size_t)i * classes + c] = __builtin_bit_cast(uint16_t, (__bf16)(g * invn));
    }
}

// ---------------------------------------------------------------- classifier z = x w^T + bias
//   gx[n][c] = sum_k gy[n][k] * scale_k * w[k][c]          gw[k][c] = scale_k * sum_n gy[n][k] * x[n][c], then sum_n gy[n][k]
// Both are small products (0.5 GFLOP for 128 images, 2048 -> 1000) whose operands all sit in the L2; neither reads the other, and one launch
// runs the tiles of both side by side.  Eight wavefronts to a tile of gx split its reduction, and their sums meet in LDS in a fixed tree; operands
// whose reduction index is the row in memory go through LDS and come back transposed (ds_read_b64_tr_b16).
//  * gw: 64 x 128 of (k, c), bf16 MFMAs (exact products, fp32 sums): 128 images of both operands in LDS, and a wavefront owns 32 x 32, so that no sums
//    meet and nothing but the operands goes through LDS; the tiles of c = 0 also add gy up for the bias.  (64 x 64, the eight wavefronts with 16
//    images each and their sums in LDS: 512 workgroups beside gx's 256 where the chip holds 512.)  The sums are the same eight in both, of every eighth
//    step of 16 images, added as a tree.  Four sums of every fourth step are longer chains: distance from float64 over the norm 3.98e-8 | 3.97e-8
//    (these) at 128 images, 6.07 | 5.65 at 512, 7.63 | 6.62 at 1024, 14.7 | 10.6 at 4096.
//  * gx: 32 images x 32 channels.  gy * scale keeps its 32 bits: it is split into three bf16 parts (8 + 8 + 8 bits, exact), each of
//    which multiplies w.
// What bounds it is the chain of launch, two round trips and a combine.  On the fp32 MFMA, which takes neither splitting nor transposing, the
// 128 images took 18.8 us (two launches of 12 before that), a third of it MFMA issue.  2048 -> 1000, one launch after the other, us, 64 x 64 tiles | this:
// 3 images 6.9 | 6.6, 64 8.9 | 7.2, 128 11.4 | 7.7, 256 16.8 | 14.9, 512 27 | 24, 1024 48 | 44, 4096 269 | 168.  (141 registers and more, one workgroup to a CU instead
// of two: 6.4, 7.1, 9.5, 15.3, 27, 51, 201.)
static constexpr int kDensePitch = 128;                          // bytes of a staged row of 64 channels
__device__ __forceinline__ int dense_flip(int row) { return (row >> 1) & 1; }    // which way a row's two 64-byte halves lie (see wgrad1x1.hip)

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef s16x4 __attribute__((address_space(3))) * dense_lds_ptr;
__device__ __forceinline__ s16x8 dense_tr_read(const unsigned char *p, int four_rows) {
    return __builtin_shufflevector(__builtin_amdgcn_ds_read_tr16_b64_v4i16((dense_lds_ptr)p),
                                   __builtin_amdgcn_ds_read_tr16_b64_v4i16((dense_lds_ptr)(p + four_rows)), 0, 1, 2, 3, 4, 5, 6, 7);
}
// One wavefront's LDS instructions execute in order; this only keeps the compiler from moving them.
__device__ __forceinline__ void dense_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// smem: 50 KB.  FEW: at most 128 images, a step to a sum.  Otherwise the images come in groups of 32, every fourth group in turn (0, 4, 8, .., then
// 1, 5, ..), so that two of the eight sums at a time are in registers: 128 of those are what two workgroups to a CU leave.
template <bool FEW>
__device__ __forceinline__ void dense_bwd_weight(const uint16_t *gy, const uint16_t *x, const float *scale, float *gw, int N, int Cin, int Cout,
                                                 unsigned block, unsigned char *smem) {
    constexpr int kImages = 128, kBlock = kImages * kDensePitch; // images in LDS at once; bytes of a block: 64 channels of them
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cblocks = (Cin + 127) / 128, k0 = (int)(block / cblocks) * 64, c0 = (int)(block % cblocks) * 128;
    // a thread fetches 16 bytes of rows tid / 8 and 64 + tid / 8 of three blocks: gy, then x twice (channel counts are multiples of 8)
    const int row = tid >> 3, seg = tid & 7;
    unsigned char *put = smem + row * kDensePitch + (((seg >> 2) ^ dense_flip(row)) << 6) + (seg & 3) * 16;    // row + 64: the same flip
    const int groups = (N + 31) / 32;
    const int end0 = (groups + 3) / 4, end1 = end0 + (groups + 2) / 4, end2 = end1 + (groups + 1) / 4;       // places where three of the four classes end
    auto class_of = [&](int place) { return place < end0 ? 0 : place < end1 ? 1 : place < end2 ? 2 : 3; };
    auto group_at = [&](int place) {
        if (FEW) return place;
        const int q = class_of(place);
        return 4 * (place - (q == 0 ? 0 : q == 1 ? end0 : q == 2 ? end1 : end2)) + q;
    };
    u32x4 in[6];
    auto fetch = [&](int at) {                                   // the groups in places at .. at + 3
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            const int place = at + (wv >> 2) + 2 * (i & 1), n0 = place < groups ? 32 * group_at(place) : N;
            const int ch = (i < 2 ? k0 : c0 + 64 * (i / 2 - 1)) + seg * 8, C = i < 2 ? Cout : Cin;
            in[i] = n0 + (row & 31) < N && ch < C ? *reinterpret_cast<const u32x4 *>((i < 2 ? gy : x) + (size_t)n0 * C + (unsigned)((row & 31) * C + ch))
                                                  : u32x4{0u, 0u, 0u, 0u};
        }
    };
    fetch(0);
    // this wavefront's 32 x 32: classes k0 + 32 kq .., channels c0 + 32 cq ..
    const int kq = wv & 1, cq = wv >> 1, half = lane >> 5, l32 = lane & 31;
    const int k = k0 + 32 * kq + 4 * half, c = c0 + 32 * cq + l32;
    const int srow = 8 * half + ((lane & 15) >> 2), scol = 32 * ((lane >> 4) & 1) + 8 * (lane & 3);
    const unsigned char *gget = smem + srow * kDensePitch + ((kq ^ dense_flip(srow)) << 6) + scol;             // row + 4, row + 16: the same flip
    const unsigned char *xget = smem + (1 + (cq >> 1)) * kBlock + srow * kDensePitch + (((cq & 1) ^ dense_flip(srow)) << 6) + scol;
    auto multiply = [&](int step, f32x16 &acc) {                 // rows past the last image are zeros of both
        const int at = 16 * step * kDensePitch;
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, dense_tr_read(gget + at, 4 * kDensePitch)),
                                                      __builtin_bit_cast(bf16x8, dense_tr_read(xget + at, 4 * kDensePitch)), acc, 0, 0, 0);
    };
    auto store = [&] {
#pragma unroll
        for (int i = 0; i < 6; ++i) *reinterpret_cast<u32x4 *>(put + (i >> 1) * kBlock + (i & 1) * (64 * kDensePitch)) = in[i];
        __syncthreads();
    };
    f32x4 sc[4];
    auto fetch_scale = [&] {
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) sc[e4] = k + 8 * e4 < Cout ? *reinterpret_cast<const f32x4 *>(scale + k + 8 * e4) : f32x4{0.f, 0.f, 0.f, 0.f};
    };
    f32x16 sum[2];                                               // of the first four of the eight sums, of the others
    const f32x16 none = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float bias = 0.f, biases = 0.f;                              // of class k0 + tid % 64, every eighth image; one sum to 128 images, then one to a class of groups
    const unsigned char *bget = smem + wv * kDensePitch + (((lane >> 5) ^ dense_flip(wv)) << 6) + (lane & 31) * 2;     // row + 8: the same flip
    auto add_bias = [&](int r) { bias += __uint_as_float((uint32_t)*reinterpret_cast<const uint16_t *>(bget + r * kDensePitch) << 16); };
    if constexpr (FEW) {
        fetch_scale();
        store();
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            f32x16 acc[2] = {none, none};
            if (32 * j < N) {
                multiply(2 * j, acc[0]);
                multiply(2 * j + 1, acc[1]);
            }
            if (j & 1) sum[j >> 1] += acc[0] + acc[1];
            else sum[j >> 1] = acc[0] + acc[1];
        }
        if (c0 == 0)
            for (int r = 0; r < N; r += 8) add_bias(r);
    } else {
        f32x16 acc[2] = {none, none};
        sum[0] = sum[1] = none;
        for (int at = 0; at < groups; at += 4) {
            if (at) __syncthreads();                             // the images before are read
            store();
            if (at + 4 < groups) fetch(at + 4);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int place = at + j, q = class_of(place);
                if (place >= groups) break;
                multiply(2 * j, acc[0]);
                multiply(2 * j + 1, acc[1]);
                if (c0 == 0)
#pragma unroll
                    for (int r = 32 * j; r < 32 * j + 32; r += 8) add_bias(r);
                if (place + 1 == groups || class_of(place + 1) != q) {
                    sum[q >> 1] += acc[0] + acc[1];
                    acc[0] = acc[1] = none;
                    biases += bias;
                    bias = 0.f;
                }
            }
        }
        fetch_scale();
    }
    // lane: column (c) l % 32, rows (k) 8 e4 + 4 (l / 32) + e of a 32 x 32 tile in register 4 e4 + e
    if (c < Cin) {
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4)
            if (k + 8 * e4 < Cout)                               // four classes, inside or outside together
#pragma unroll
                for (int e = 0; e < 4; ++e) gw[(size_t)(k + 8 * e4 + e) * Cin + c] = (sum[0][4 * e4 + e] + sum[1][4 * e4 + e]) * sc[e4][e];
    }
    if (c0 == 0) {                                               // the bias: eight threads to a class
        float *part = reinterpret_cast<float *>(smem + 3 * kBlock);
        part[tid] = bias += biases;
        __syncthreads();
        if (tid < 64 && k0 + tid < Cout) {
            for (int v = 1; v < 8; ++v) bias += part[v * 64 + tid];
            gw[(size_t)Cout * Cin + k0 + tid] = bias;
        }
    }
}

// KW wavefronts (thread `tid` of KW * 64) to a tile; smem: LDS of `each` bytes per wavefront.  A tile past the last stores nothing.
template <int KW>
__device__ __forceinline__ void dense_bwd_data(const uint16_t *gy, const uint16_t *w, const float *scale, uint16_t *gx, int N, int Cin, int Cout,
                                               unsigned block, int tid, unsigned char *smem, int each) {
    const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, half = lane >> 5;
    const unsigned cblocks = (Cin + 31) / 32, n0 = block / cblocks * 32;
    const int c0 = (int)(block % cblocks) * 32;
    // a step is 32 classes: w's rows (64 bytes of 32 channels) through LDS, gy and scale straight into the MFMA's layout (image l % 32, classes
    // 16 q + 8 (l / 32) .. + 7)
    const int row = lane >> 2, seg = lane & 3;
    const bool cin = c0 + seg * 8 < Cin;
    const uint16_t *gp = gy + (size_t)(n0 + l32 < (unsigned)N ? n0 + l32 : N - 1) * Cout;      // past the last image: that image, not stored
    unsigned char *stg = smem + wv * each;
    unsigned char *put = stg + row * 64 + seg * 16;
    const unsigned char *get = stg + (8 * half + ((lane & 15) >> 2)) * 64 + 32 * ((lane >> 4) & 1) + 8 * (lane & 3);
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    u32x4 wb[2], gb[2];
    f32x4 sb[2][2];
    const u32x4 zero = {0u, 0u, 0u, 0u};
    const __amdgpu_buffer_rsrc_t srsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(scale), 0, Cout * 4, 0x00020000);
    auto fetch = [&](int k0) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int kr = k0 + 16 * u + row, kg = k0 + 16 * u + 8 * half;           // Cout is a multiple of 8
            wb[u] = kr < Cout && cin ? *reinterpret_cast<const u32x4 *>(w + (size_t)kr * Cin + c0 + seg * 8) : zero;
            const bool in = kg < Cout;
            gb[u] = in ? *reinterpret_cast<const u32x4 *>(gp + kg) : zero;
#pragma unroll
            for (int q = 0; q < 2; ++q)                          // past the last class both factors are zero
                sb[u][q] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(srsrc, (kg + 4 * q) * 4, 0, 0));
        }
    };
    fetch(32 * wv);
    for (int k0 = 32 * wv; k0 < Cout; k0 += 32 * KW) {
        dense_fence();
#pragma unroll
        for (int u = 0; u < 2; ++u) *reinterpret_cast<u32x4 *>(put + u * 1024) = wb[u];
        u32x4 parts[2][3];
        uint32_t rest = 0u;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int p = 0; p < 4; ++p) {                        // two classes at a time
                uint32_t bits[2][3];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const float v = (h ? hi16(gb[u][p]) : lo16(gb[u][p])) * sb[u][p >> 1][2 * (p & 1) + h];
                    bits[h][0] = __float_as_uint(v) & 0xFFFF0000u;                                       // cut off, not rounded: never overflows
                    const float r1 = v - __uint_as_float(bits[h][0]);                                    // exact, and so is the next
                    bits[h][1] = __float_as_uint(r1) & 0xFFFF0000u;
                    bits[h][2] = __float_as_uint(r1 - __uint_as_float(bits[h][1]));
                    if ((bits[h][0] & 0x7F800000u) == 0x7F800000u) bits[h][1] = bits[h][2] = 0u;         // an Inf or NaN is its first part
                    rest |= bits[h][1] | bits[h][2];
                }
#pragma unroll
                for (int q = 0; q < 3; ++q) parts[u][q][p] = bits[0][q] >> 16 | (bits[1][q] & 0xFFFF0000u);
            }
        const bool split = __any(rest != 0u);                    // scale = 1: gy is its own first part
        fetch(k0 + 32 * KW);
        dense_fence();
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const bf16x8 wf = __builtin_bit_cast(bf16x8, dense_tr_read(get + u * 1024, 4 * 64));
            if (split) {                                         // the small parts first
                u32x4 fin = __builtin_bit_cast(u32x4, wf);       // an infinite weight meets the first part alone: a small one may be a zero
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    if ((fin[p] & 0x7F80u) == 0x7F80u) fin[p] &= 0xFFFF0000u;
                    if ((fin[p] & 0x7F800000u) == 0x7F800000u) fin[p] &= 0xFFFFu;
                }
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fin), __builtin_bit_cast(bf16x8, parts[u][2]), acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fin), __builtin_bit_cast(bf16x8, parts[u][1]), acc, 0, 0, 0);
            }
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, __builtin_bit_cast(bf16x8, parts[u][0]), acc, 0, 0, 0);
        }
    }
    // lane: image l % 32, channels 8 rb + 4 (l / 32) + e in register 4 rb + e
    dense_fence();
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
        *reinterpret_cast<f32x4 *>(stg + l32 * 144 + (8 * rb + 4 * half) * 4) = f32x4{acc[4 * rb], acc[4 * rb + 1], acc[4 * rb + 2], acc[4 * rb + 3]};
    __syncthreads();
#pragma unroll
    for (int at = tid; at < 256; at += KW * 64) {
        const unsigned n = n0 + (at >> 3);
        const int c = c0 + 4 * (at & 7);
        if (n >= (unsigned)N || c >= Cin) continue;
        f32x4 part[KW];
#pragma unroll
        for (int v = 0; v < KW; ++v) part[v] = *reinterpret_cast<const f32x4 *>(smem + v * each + (at >> 3) * 144 + (at & 7) * 16);
#pragma unroll
        for (int half_of = 1; half_of < KW; half_of *= 2)        // neighbours first: ((0 + 1) + (2 + 3)) + ...
#pragma unroll
            for (int v = 0; v < KW; v += 2 * half_of) part[v] += part[v + half_of];
        *reinterpret_cast<u32x2 *>(gx + (size_t)n * Cin + c) = u32x2{pack2(part[0].x, part[0].y), pack2(part[0].z, part[0].w)};
    }
}

// The first `data_blocks` workgroups tiles of gx, whose reductions are longer, the others tiles of gw.  With few classes a tile of gx has steps for KW
// of the eight wavefronts, and a workgroup takes 8 / KW tiles.  gx alone, us with eight to a tile | this: 4096 x 768, 8 classes 13.0 | 5.3,
// 4096 x 2048, 40 classes 34 | 15; up to 512 tiles eight are better: 128 x 512, 32 classes 3.0 | 3.5, 512 x 768, 24 classes 3.4 | 3.7.
template <int KW, bool WEIGHT, bool FEW>
__global__ __launch_bounds__(512) void dense_bwd_kernel(const uint16_t *gy, const uint16_t *w, const uint16_t *x, const float *scale,
                                                        uint16_t *gx, float *gw, int N, int Cin, int Cout, unsigned data_blocks) {
    constexpr int kEach = WEIGHT ? 8192 : 32 * 144;          // gw's 50 KB or less: registers hold two workgroups to a CU, LDS too
    __shared__ __align__(16) unsigned char smem[8 * kEach];
    if (!WEIGHT || blockIdx.x < data_blocks) {
        const int group = __builtin_amdgcn_readfirstlane(threadIdx.x / (KW * 64));
        dense_bwd_data<KW>(gy, w, scale, gx, N, Cin, Cout, blockIdx.x * (8 / KW) + group, threadIdx.x & (KW * 64 - 1), smem + group * KW * kEach, kEach);
    } else {
        dense_bwd_weight<FEW>(gy, x, scale, gw, N, Cin, Cout, blockIdx.x - data_blocks, smem);
    }
}

}  // namespace bops

hipError_t launch_maxpool_bwd(const PoolArgs &a, const void *gy, void *gx, int mask_x, hipStream_t stream) {
    if (pool_check(a, false) || !a.bf16 || !gy || !gx) return hipErrorInvalidValue;
    if (a.R == 3 && a.S == 3 && a.stride == 2 && a.pad == 1) {
        const int th = (a.H + bops::kPackTH - 1) / bops::kPackTH, tw = (a.W + bops::kPackTW - 1) / bops::kPackTW;
        const long long tiles = (long long)a.N * th * tw * ((a.C / 8 + bops::kPoolChunks - 1) / bops::kPoolChunks);
        if (tiles > 0x7FFFFFFFLL) return hipErrorInvalidValue;
        bops::maxpool_bwd_packed_kernel<<<dim3((unsigned)tiles), dim3(256), 0, stream>>>(a, gy, gx, tw, th, mask_x);
        return hipGetLastError();
    }
    const int tiles_h = (a.H + bops::kPoolTile - 1) / bops::kPoolTile, tiles_w = (a.W + bops::kPoolTile - 1) / bops::kPoolTile;
    const int cgroups = (a.C / 8 + bops::kPoolChunks - 1) / bops::kPoolChunks;
    const long long blocks = (long long)a.N * tiles_h * tiles_w * cgroups;
    if (a.R * a.S > 255) return hipErrorInvalidValue;                   // window positions are recorded as bytes
    const size_t lds = (size_t)(bops::kPoolTile + 2 * (a.R - 1)) * (bops::kPoolTile + 2 * (a.S - 1)) * bops::kPoolChunks * 16 +
                       (size_t)bops::pool_windows_max(a.R, a.stride) * bops::pool_windows_max(a.S, a.stride) * bops::kPoolChunks * (8 + 16);
    if (blocks <= 0 || blocks > 0x7FFFFFFFLL || lds > 64 * 1024) return hipErrorInvalidValue;
    bops::maxpool_bwd_kernel<<<dim3((unsigned)blocks), dim3(256), lds, stream>>>(a, gy, gx, tiles_w, tiles_h, mask_x);
    return hipGetLastError();
}

hipError_t launch_avgpool_bwd(const PoolArgs &a, const void *gy, void *gx, hipStream_t stream) {
    if (pool_check(a, true) || !a.bf16 || !gy || !gx) return hipErrorInvalidValue;
    const long long total = (long long)a.N * a.H * a.W * (a.C / 8);
    const long long blocks = (total + 255) / 256;
    if (blocks <= 0 || blocks > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    bops::avgpool_bwd_kernel<<<dim3((unsigned)blocks), dim3(256), 0, stream>>>(gy, gx, a.H * a.W, a.C / 8, total);
    return hipGetLastError();
}

hipError_t launch_softmax_ce_bwd(const void *logits, const void *labels, int N, int classes, void *gz, hipStream_t stream) {
    if (!logits || !labels || !gz || N <= 0 || classes <= 0) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((N + 3) / 4)), block(256);
    const auto *z = static_cast<const uint16_t *>(logits);
    const auto *lab = static_cast<const long long *>(labels);
    auto *out = static_cast<uint16_t *>(gz);
    const bool pieces = classes % 8 == 0 && !(((uintptr_t)logits | (uintptr_t)gz) & 15);
    if (pieces && classes <= 512) bops::softmax_ce_bwd_held_kernel<1><<<grid, block, 0, stream>>>(z, lab, N, classes, out);
    else if (pieces && classes <= 1024) bops::softmax_ce_bwd_held_kernel<2><<<grid, block, 0, stream>>>(z, lab, N, classes, out);
    else bops::softmax_ce_bwd_kernel<<<grid, block, 0, stream>>>(z, lab, N, classes, out);
    return hipGetLastError();
}

// Classifier: x [N][Cin], w [Cout][Cin] bf16, gy [N][Cout] bf16; gx [N][Cin] bf16 (or null),
// gw fp32 [Cout*Cin + Cout] (weights, then bias; or null).  Cin and Cout multiples of 8, pointers 16-byte aligned.
hipError_t launch_dense_bwd(const void *x, const void *w, const float *scale, const void *gy, void *gx, float *gw,
                            int N, int Cin, int Cout, hipStream_t stream) {
    if (!w || !scale || !gy || N <= 0 || Cin <= 0 || Cout <= 0 || Cin % 8 || Cout % 8) return hipErrorInvalidValue;
    if (((uintptr_t)x | (uintptr_t)w | (uintptr_t)scale | (uintptr_t)gy | (uintptr_t)gx | (uintptr_t)gw) & 15) return hipErrorInvalidValue;
    if (gw && !x) return hipErrorInvalidValue;
    const long long tiles = ((long long)N + 31) / 32 * ((Cin + 31) / 32);
    // wavefronts to a tile of gx: those that have a step of 32 classes; all eight where every tile finds its place at once (they share the store)
    const int kw = tiles <= 512 ? 8 : Cout <= 32 ? 1 : Cout <= 64 ? 2 : Cout <= 128 ? 4 : 8;
    const long long data = gx ? (tiles + 8 / kw - 1) / (8 / kw) : 0, weight = gw ? ((long long)Cout + 63) / 64 * ((Cin + 127) / 128) : 0;
    if (tiles > 0x7FFFFFFFLL || data + weight > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    if (data + weight == 0) return hipSuccess;
    auto run = [&](auto kernel) {
        kernel<<<dim3((unsigned)(data + weight)), dim3(512), 0, stream>>>(static_cast<const uint16_t *>(gy), static_cast<const uint16_t *>(w),
                                                                         static_cast<const uint16_t *>(x), scale, static_cast<uint16_t *>(gx), gw, N,
                                                                         Cin, Cout, (unsigned)data);
    };
    const bool few = N <= 128;
#define DELTA_DENSE(KW) \
    (!gw ? run(bops::dense_bwd_kernel<KW, false, false>) : few ? run(bops::dense_bwd_kernel<KW, true, true>) : run(bops::dense_bwd_kernel<KW, true, false>))
    kw == 1 ? DELTA_DENSE(1) : kw == 2 ? DELTA_DENSE(2) : kw == 4 ? DELTA_DENSE(4) : DELTA_DENSE(8);
#undef DELTA_DENSE
    return hipGetLastError();
}

}  // namespace delta
