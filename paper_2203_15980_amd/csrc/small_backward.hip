// Both gradients of a convolution that cannot fill the chip, in one launch, for gfx950, bf16 and fp32:
//   gx = conv(gpre, wt) (+ gx_add) (* [x > 0])          the data gradient as a forward convolution of gpre (see backward.hip)
//   gw[k,r,s,c] = scale_k * sum_m gpre[m,k] * x[m + (r,s), c]
//
// On a few images every kernel of a backward pass is a chain of launch, round trips to memory and one combine: 6 to 11 us whether
// 30 or 300 workgroups run it, and the two gradients of a layer (with the bf16 weight gradient's partial sums and their
// reduction: three such chains) ran one after the other although neither reads the other.  Here the first workgroups
// of a grid compute tiles of gw, the others tiles of gx:
//  * gx: conv_tile (splitk_tile.hpp), eight wavefronts to a 32 x 32 tile, or two tiles of four for short reductions;
//  * gw: a workgroup owns 32 TW x 32 TW of (k, c) of one tap and ALL its positions, eight wavefronts take steps of 32 / TW positions
//    in turn and their sums meet in LDS in a fixed tree: no partial sums in memory, no second launch, a fixed
//    function of the inputs.  bf16: a step's rows go through registers into LDS that only this wavefront uses and come back
//    transposed (ds_read_b64_tr_b16, as in wgrad1x1.hip).  fp32: wgrad_f32_tile.hpp.
//  * positions past the end and taps outside the image are offsets outside the buffer descriptors, of BOTH operands: they load
//    zeros, and no Inf of one meets a zero of the other.
// Backward of a bottleneck, us before -> now: conv4_x on 1 / 4 / 8 images of 14 x 14 53 -> 23, 64 -> 33, 79 -> 51; conv3_x on 1 / 4 images of 28 x 28 53 -> 23,
// 76 -> 42; conv5_x on 1 / 8 images of 7 x 7 63 -> 34, 81 -> 55; three fp32 bottlenecks on 2 x 32 x 32 152 -> 103.
// small_backward_applies says where the line lies and what both sides measured.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <type_traits>

#include "kernels.hpp"
#include "splitk_tile.hpp"
#include "wgrad_f32_tile.hpp"

namespace delta {
namespace smallb {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

static constexpr int kOutOfRange = (int)0x80000000;              // outside every buffer descriptor used here
static constexpr int kLds = 8 * splitk::kWaveLds;

struct WeightArgs {
    const void *x, *g;                   // [N,XH,XW,C], [M,K]
    const float *scale;
    float *gw;                           // [K][R][R][C]
    int M, C, K, R, pad, stride, P, Q, XH, XW;       // M = N P Q positions, each reading pixel (stride p + r - pad, stride q + s - pad)
    uint32_t xbytes;
    int ctiles, blocks;                  // tiles along c; workgroups in all (tap fastest, then c, then k)
    Divisor pq, q, taps, dct;
};

// bf16: 32 TW x 32 TW of (k, c) of one tap.  PLAIN: 1x1, stride 1 - position m reads pixel m.
template <int TW, bool PLAIN>
__device__ __forceinline__ void weight_tile(const WeightArgs &a, int k0, int c0, int tap, int tid, unsigned char *smem, float *factors) {
    constexpr int kRows = 16 / TW, kStep = 2 * kRows;            // rows of 64 TW bytes per load instruction; positions of a step: two of those
    constexpr int kPitch = 64 * TW, kAhead = 2;                  // steps in flight (128 registers: two workgroups to a CU)
    const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (wv == 0) {                                               // scale of the tile's channels, straight into LDS
        typedef __attribute__((address_space(3))) float *lptr_t;
        load_lds_b32(a.scale + k0 + (lane & (32 * TW - 1)), (uint32_t)(uintptr_t)(lptr_t)factors);
    }
    const __amdgpu_buffer_rsrc_t grsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.g), 0, (int)((uint32_t)a.M * (uint32_t)a.K * 2u), 0x00020000);
    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.x), 0, (int)a.xbytes, 0x00020000);
    const int row = lane / (4 * TW), seg = lane % (4 * TW);
    const int dr = PLAIN ? 0 : tap / a.R - a.pad, ds = PLAIN ? 0 : tap % a.R - a.pad;
    const uint32_t gcol = (uint32_t)k0 * 2u + seg * 16u, xcol = (uint32_t)c0 * 2u + seg * 16u;
    u32x4 gb[kAhead][2], xb[kAhead][2];
    int step = wv;
    auto fetch = [&](u32x4 (&gd)[2], u32x4 (&xd)[2]) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int m = step * kStep + kRows * i + row;
            bool in = m < a.M;
            int pixel = m;
            if constexpr (!PLAIN) {
                const int n = divide(m, a.pq), pq = m - n * (a.P * a.Q), p = divide(pq, a.q), q = pq - p * a.Q;
                const int h = p * a.stride + dr, w = q * a.stride + ds;
                in = in & ((unsigned)h < (unsigned)a.XH) & ((unsigned)w < (unsigned)a.XW);
                pixel = (n * a.XH + h) * a.XW + w;
            }
            gd[i] = __builtin_amdgcn_raw_buffer_load_b128(grsrc, in ? (int)((uint32_t)m * (uint32_t)a.K * 2u + gcol) : kOutOfRange, 0, 0);
            xd[i] = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, in ? (int)((uint32_t)pixel * (uint32_t)a.C * 2u + xcol) : kOutOfRange, 0, 0);
        }
        step += 8;
    };
    // LDS rows as they lie in memory; of 128-byte rows bit 1 of the row number flips the 64-byte halves, so that the four rows a
    // transposing read touches lie in four quarters of the banks
    auto flip = [](int r) { return TW == 1 ? 0 : (r >> 1) & 1; };
    unsigned char *stg = smem + wv * splitk::kWaveLds;
    unsigned char *put = stg + row * kPitch + (((seg >> 2) ^ flip(row)) << 6) + (seg & 3) * 16;       // rows + multiples of 4: the same flip
    const int srow = 8 * (lane >> 5) + ((lane & 15) >> 2), scol = 32 * ((lane >> 4) & 1) + 8 * (lane & 3);
    typedef s16x4 __attribute__((address_space(3))) * lds_ptr;
    auto tr_read = [&](const unsigned char *p) { return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p)); };
    // Four sums in turn for the narrow tile, added at the end: a wavefront may add 1024 products to one, and the splits of the kernels that
    // larger layers take are shorter (one sum: 1.4 to 1.8 times their distance from 64 bits)
    constexpr int kSums = TW == 1 ? 4 : 1;
    f32x16 acc[kSums][TW][TW];
#pragma unroll
    for (int u = 0; u < kSums; ++u)
#pragma unroll
        for (int i = 0; i < TW; ++i)
#pragma unroll
            for (int j = 0; j < TW; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[u][i][j][e] = 0.f;
    const int steps = (a.M + kStep - 1) / kStep, mine = (steps - wv + 7) / 8;
#pragma unroll
    for (int u = 0; u < kAhead; ++u) fetch(gb[u], xb[u]);
    for (int t = 0; t < mine; t += kAhead) {                     // a last partial round runs on zeros
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            splitk::wave_lds_fence();
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                *reinterpret_cast<u32x4 *>(put + i * 1024) = gb[u][i];
                *reinterpret_cast<u32x4 *>(put + 2048 + i * 1024) = xb[u][i];
            }
            fetch(gb[u], xb[u]);
            splitk::wave_lds_fence();
#pragma unroll
            for (int q = 0; q < kStep / 16; ++q) {
                const int sum = kSums == 1 ? 0 : u * 2 + q;
                s16x8 gf[TW], xf[TW];
#pragma unroll
                for (int h = 0; h < TW; ++h) {
                    const unsigned char *p = stg + (16 * q + srow) * kPitch + ((h ^ flip(srow)) << 6) + scol;
                    gf[h] = __builtin_shufflevector(tr_read(p), tr_read(p + 4 * kPitch), 0, 1, 2, 3, 4, 5, 6, 7);
                    p += 2048;
                    xf[h] = __builtin_shufflevector(tr_read(p), tr_read(p + 4 * kPitch), 0, 1, 2, 3, 4, 5, 6, 7);
                }
#pragma unroll
                for (int i = 0; i < TW; ++i)
#pragma unroll
                    for (int j = 0; j < TW; ++j)
                        acc[sum][i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, gf[i]), __builtin_bit_cast(bf16x8, xf[j]),
                                                                                 acc[sum][i][j], 0, 0, 0);
            }
        }
    }
    // ---- the eight sums of each 32 x 32 tile, two tiles at a time: lane l holds c l % 32 and k 8 e4 + 4 (l / 32) + e in register 4 e4 + e
    constexpr int kPer = TW == 1 ? 1 : 2;
    const int taps = a.R * a.R;
#pragma unroll
    for (int at = 0; at < TW * TW; at += kPer) {
        if (at) __syncthreads();                                 // the sums before are read
        splitk::wave_lds_fence();
#pragma unroll
        for (int u = 0; u < kPer; ++u)
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4) {
                f32x16 v = acc[0][(at + u) / TW][(at + u) % TW];
                if constexpr (kSums == 4) v = (v + acc[1][0][0]) + (acc[2][0][0] + acc[3][0][0]);
                *reinterpret_cast<f32x4 *>(stg + u * 4096 + e4 * 1024 + lane * 16) = f32x4{v[4 * e4], v[4 * e4 + 1], v[4 * e4 + 2], v[4 * e4 + 3]};
            }
        if (at == 0 && wv == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid < kPer * 256) {
            f32x4 part[8];
#pragma unroll
            for (int v = 0; v < 8; ++v) part[v] = *reinterpret_cast<const f32x4 *>(smem + v * splitk::kWaveLds + tid * 16);
            const f32x4 sum = ((part[0] + part[1]) + (part[2] + part[3])) + ((part[4] + part[5]) + (part[6] + part[7]));
            const int tile = at + (tid >> 8), e4 = (tid >> 6) & 3;
            const int kl = 32 * (tile / TW) + 8 * e4 + 4 * (lane >> 5), k = k0 + kl, c = c0 + 32 * (tile % TW) + (lane & 31);
            const f32x4 sc = *reinterpret_cast<const f32x4 *>(factors + kl);
#pragma unroll
            for (int e = 0; e < 4; ++e) a.gw[((size_t)(k + e) * taps + tap) * a.C + c] = sum[e] * sc[e];
        }
    }
}

// KW: wavefronts to a tile of gx.  TW: tile of gw, 32 TW (bf16) or 16 TW (fp32) of k and c.
template <bool BF16, int KW, int TW, bool PLAIN>
__global__ __launch_bounds__(512) void small_backward_kernel(ConvArgs da, int tiles_m, int tiles_n, int pixels_first, splitk::Divisors inv,
                                                             WeightArgs w) {
    __shared__ __align__(16) unsigned char smem[kLds];
    __shared__ __align__(16) float factors[128];
    const int tid = threadIdx.x;
    if ((int)blockIdx.x < w.blocks) {
        const int logical = (int)splitk::xcd_run(blockIdx.x, w.blocks);
        const int at = divide(logical, w.taps), tap = logical - at * (w.R * w.R), kt = divide(at, w.dct), ct = at - kt * w.ctiles;
        if constexpr (BF16)
            weight_tile<TW, PLAIN>(w, kt * 32 * TW, ct * 32 * TW, tap, tid, smem, factors);
        else
            wgrad_f32_tile<TW, !PLAIN, 8>(static_cast<const float *>(w.x), static_cast<const float *>(w.g), w.scale, w.gw, w.P, w.Q, w.C, w.K, w.R,
                                          w.pad, w.M, w.pq, w.q, kt * 16 * TW, ct * 16 * TW, tap, tid, reinterpret_cast<float *>(smem), factors);
        return;
    }
    constexpr int kGroups = 8 / KW;                              // tiles of gx to a workgroup
    const int group = __builtin_amdgcn_readfirstlane(tid / (KW * 64));
    const unsigned logical = splitk::xcd_run(blockIdx.x - w.blocks, gridDim.x - w.blocks) * kGroups + group;
    splitk::conv_tile<BF16, KW, 2, BF16 && !PLAIN>(da, tiles_m, tiles_n, pixels_first, inv, logical, tid & (KW * 64 - 1), smem + group * KW * splitk::kWaveLds,
                                   factors + group * 64);
}

template <bool BF16, int KW, int TW, bool PLAIN>
hipError_t launch(const ConvArgs &da, const WeightArgs &w, hipStream_t stream) {
    const int tiles_m = (da.M + splitk::kTile - 1) / splitk::kTile, tiles_n = (da.Cout + splitk::kTile - 1) / splitk::kTile;
    const unsigned data = ((unsigned)tiles_m * (unsigned)tiles_n + 8 / KW - 1) / (8 / KW);
    small_backward_kernel<BF16, KW, TW, PLAIN><<<dim3(w.blocks + data), dim3(512), 0, stream>>>(da, tiles_m, tiles_n, splitk::weights_larger(da),
                                                                                                  splitk::divisors_of(da), w);
    return hipGetLastError();
}

long long steps_of(const ConvArgs &a) { return (long long)a.R * a.S * a.Cin * (a.bf16 ? 2 : 4) / splitk::kStepBytes; }

}  // namespace smallb

// da: the data gradient (launch_conv's or launch_conv_scatter's arguments), or null: the weight gradient alone.  fa: the layer as its weight
// gradient sees it (launch_wgrad's arguments, or a 3x3 stride-2 layer's own geometry).
bool small_backward_applies(const ConvArgs *da, const ConvArgs &fa) {
    const long long es = fa.bf16 ? 2 : 4, M = (long long)fa.N * fa.P * fa.Q;
    if (fa.R != fa.S || (fa.R != 1 && fa.R != 3) || fa.pad != fa.R / 2) return false;
    const int step = fa.bf16 ? 64 : 16;
    if (fa.Cin % step || fa.Cout % step || (!fa.bf16 && fa.stride != 1)) return false;
    // 32-bit offsets from the tensors' own starts, with room for the rows past the last position that a step may name
    if ((long long)fa.N * fa.H * fa.W * fa.Cin * es > 0x7FFFFFFFLL || (M + 512) * fa.Cout * es > 0x7FFFFFFFLL) return false;
    if (da && (da->bf16 != fa.bf16 || da->R > 8 || da->S > 8 || (long long)da->N * da->H * da->W * da->Cin * es > 0x7FFFFFFFLL)) return false;
    // Where the line lies, measured as us per layer in a segment of such layers: two or three launches | this one.
    //   fp32 (2 images, 1x1 64 -> 256 | 256 -> 64 | 3x3 64 -> 64): M = 512 11 9.8 12 | 7.2 7.1 8.2; M = 2048 13 13 17 | 7.5 10.6 13.7; M = 8192 33 45 39 | 24 26 33.
    //   8192 keeps the sums as short as the sixteen wavefronts' of the other route.  Beyond that the number of 32 x 32 tiles of gx counts, here in
    //   brackets: on a full chip the 128 x 128 tiles of the other route load a quarter per product, all the more where a tile's wavefronts have a step or two each.
    //     2 steps of the reduction   2048 -> 64   M = 8192 [16384] 138 | 127
    //     4    1024 -> 128  M = 2048 [2048] 39 | 25   8192 [8192] 90 | 86     512 -> 128  M = 6144 [3072] 45 | 43   8192 [4096] 50 | 55
    //          2048 -> 128  M = 1024 [2048] 29 | 24   1536 [3072] 32 | 37   4096 [8192] 61 | 84
    //     8    512 -> 256   M = 3072 [1536] 48 | 35   4096 [2048] 43 | 44   1024 -> 256  M = 1536 [1536] 40 | 35   2048 [2048] 42 | 44   4096 [4096] 50 | 83
    //     16   512 -> 512   M = 4096 [2048] 65 | 54   6144 [3072] 70 | 79   2048 -> 512  M = 1024 [2048] 59 | 56   1536 [3072] 68 | 82   8192 [16384] 317 | 445
    //     64   512 -> 2048  M = 4096 [2048] 180 | 173   6144 [3072] 230 | 256     144 (3x3)  512 -> 512  M = 4096 [2048] 421 | 389   6144 [3072] 565 | 581
    //   Where some hundred tiles leave a ragged last round the lines are not exact: 256 -> 1024 M = 2048 [512] 28 | 31, 128 -> 2048 M = 3072 [384] 39 | 48.
    if (!fa.bf16) {
        const long long steps = da ? smallb::steps_of(*da) : 0, line = steps >= 8 && steps < 16 ? 1536 : 2048;
        return M <= 8192 && (steps < 4 || splitk::tiles_of(*da) <= line);
    }
    //   bf16: a workgroup walks all positions of its tile of gw, about 2 us per 1000 up to some 8000, beyond which it waits for memory:
    //     1x1 64 -> 256  M = 3136 14.5 | 7.5   6272 15.7 | 11   12544 17.6 | 28     3x3 64 -> 64  M = 6272 20 | 15   12544 23 | 25
    //   With few tiles of gw the other route has many short splits: at M = 6272 it is nearer to 64 bits (9.2e-8 | 9.6e-8 of the norm, 8.6 | 8.0
    //   at 3136); with 64 tiles the two are level at 6400 and 8192 is past it (1.02e-7 | 1.05e-7).
    //   below that the sum of both parts' work is what counts, here in ns with the number of 32 x 32 tiles of gx and gw in it:
    //     1x1 256 -> 1024  M = 196 14 | 6.3   1568 20 | 14   3136 26 | 18   4704 31 | 25 (23 by the formula)   6272 32 | 31 (30)
    //     1x1 512 -> 128   M = 784 15 | 6.3   3136 22 | 12   6272 27 | 22 (21)   12544 32 | 41
    //     1x1 2048 -> 512  M = 49 15 | 6.8    392 22 | 15    784 31 | 23 (21)    1176 31 | 32 (27)    1568 30 | 40 (35)
    //     3x3 256 -> 256   M = 196 20 | 7.9   784 25 | 11    1568 32 | 16 (18)   3136 38 | 24 (28)    6272 45 | 42 (49)
    //     3x3 512 -> 512   M = 49 27 | 16     392 32 | 23 (17)   784 41 | 26 (27)   1568 47 | 44 (46)
    //   From 1 GFLOP on the left side is two streams and the host's 30 us for them; the lines at 26 (1x1) and 38 (3x3) leave out what is not
    //   clearly faster.
    const double gx = da ? (double)splitk::tiles_of(*da) * (8. + (double)smallb::steps_of(*da)) : 0.;
    const double tiles = (double)(fa.Cout / 32) * (fa.Cin / 32) * (fa.R * fa.S), gw = tiles * ((double)M / 32);
    // A strided layer's other launch (spread_add; dgrad3x3_s2, 20 us) already hides a weight gradient on the second stream:
    //     1x1 256 -> 512  M = 784 19 | 11   3136 26 | 19   4704 30 | 26   6272 30 | 32     512 -> 1024  M = 2352 30 | 25   1024 -> 2048  M = 588 32 | 26
    //     3x3 128 -> 128  M = 784 27 | 18   3136 33 | 22   4704 32 | 26   6272 33 | 34     256 -> 256  M = 1568 33 | 29 (11)   512 -> 512  M = 588 37 | 45 (13)
    const int most = tiles < 64 ? 4096 : fa.stride > 1 ? 5000 : 6400;
    const double ns = 7000. + 0.4 * gx + 0.13 * gw;
    if (M > most || ns > (!da ? 11000. : fa.R == 3 ? 38000. : 26000.)) return false;
    //   The sum is right for tiles of gx that have the chip to themselves a few times over; with more of them it promises too little, and the other
    //   route's larger tiles load less (stride 1 | 2, number of tiles of gx in brackets, other route | this one):
    //     8 to 15 steps   1x1 2048 -> 512  M = 784 [1600] 26 | 23, 35 | 29     768 -> 512  M = 2156 [1632] 26 | 26, 29 | 33   2744 [2064] 28 | 32, 30 | 40
    //                     1x1 1024 -> 640  M = 1568 [1568] 31 | 22, 35 | 29    512 -> 512  M = 3528 [1776] 26 | 28, 29 | 35
    //     1 to 4          1x1 1024 -> 64   M = 3920 [3936] 23 | 20, 30 | 31    4704 [4704] 19 | 24, 32 | 36     2048 -> 256  M = 1568 [3136] 33 | 22, 34 | 32
    //     9, 18, 36       3x3 512 -> 64    M = 4704 [2352] 34 | 33   5488 [2752] 35 | 38     512 -> 128  M = 3528 [1776] 39 | 36 (34)   3920 [1968] 36 | 41 (37)
    //                     3x3 512 -> 256   M = 2156 [1088] 37 | 41 (36)     256 -> 256  M = 3920 [984] 43 | 37 (33)
    if (!da || (fa.R == 3 && fa.stride > 1)) return true;        // (one class of a strided layer's gx: a quarter of its pixels, faster up to the lines above)
    const long long line = fa.R == 3 ? (ns > 35000. ? 1024 : 2560) : smallb::steps_of(*da) >= 8 ? 1600 : 4096;
    return splitk::tiles_of(*da) <= line;
}

const char *small_backward_name(const ConvArgs &fa) { return fa.bf16 ? "small_backward bf16" : "small_backward f32"; }

// g = gpre [N,P,Q,Cout]; gw fp32 [Cout][R][S][Cin]; fa with x and scale.
hipError_t launch_small_backward(const ConvArgs *data, const ConvArgs &fa, const void *g, float *gw, hipStream_t stream) {
    if ((data && (data->oy_s ? conv_scatter_check(*data) : conv_check(*data))) || !small_backward_applies(data, fa) || !g || !gw || !fa.x ||
        !fa.scale || ((uintptr_t)g | (uintptr_t)fa.x) & 15)
        return hipErrorInvalidValue;
    ConvArgs da;
    memset(&da, 0, sizeof da);
    if (data) da = *data;
    if (!da.oy_s) { da.wR = da.R; da.wS = da.S; da.w_r0 = da.w_s0 = 0; da.w_step = 1; }
    const int taps = fa.R * fa.R, unit = fa.bf16 ? 32 : 16;
    const long long tiles = (long long)(fa.Cout / unit) * (fa.Cin / unit) * taps;
    // The wider tile of gw, half the loads per product, where the narrow ones would be more than two workgroups to a CU anyway (3x3 256 -> 256 on
    // 1568 pixels 18 -> 15 us, 512 -> 512 on 588 31 -> 23).  In bf16 it has registers for one sum only: up to 2000 pixels, beyond which that is further
    // from 64 bits than the kernels it replaces (3x3 256 -> 256 on 2352 1.00e-7 against 0.95e-7; four sums 0.75e-7).
    const int tw = tiles >= 512 && (!fa.bf16 || fa.M <= 2000) && fa.Cout % (2 * unit) == 0 && fa.Cin % (2 * unit) == 0 ? 2 : 1;
    smallb::WeightArgs w;
    w.x = fa.x; w.g = g; w.scale = fa.scale; w.gw = gw;
    w.M = fa.N * fa.P * fa.Q; w.C = fa.Cin; w.K = fa.Cout; w.R = fa.R; w.pad = fa.pad; w.stride = fa.stride;
    w.P = fa.P; w.Q = fa.Q; w.XH = fa.H; w.XW = fa.W;
    w.xbytes = (uint32_t)((long long)fa.N * fa.H * fa.W * fa.Cin * (fa.bf16 ? 2 : 4));
    w.ctiles = fa.Cin / (unit * tw);
    w.blocks = (int)(tiles / (tw * tw));
    w.pq = make_divisor(fa.P * fa.Q); w.q = make_divisor(fa.Q); w.taps = make_divisor(taps); w.dct = make_divisor(w.ctiles);
    const bool plain = fa.R == 1 && fa.stride == 1, longer = !data || smallb::steps_of(da) >= 8;
    auto pick = [&](auto bf16, auto kw, auto t) {
        return plain ? smallb::launch<decltype(bf16)::value, decltype(kw)::value, decltype(t)::value, true>(da, w, stream)
                     : smallb::launch<decltype(bf16)::value, decltype(kw)::value, decltype(t)::value, false>(da, w, stream);
    };
    auto by_tile = [&](auto bf16, auto kw) {
        return tw == 2 ? pick(bf16, kw, std::integral_constant<int, 2>()) : pick(bf16, kw, std::integral_constant<int, 1>());
    };
    auto by_length = [&](auto bf16) {
        return longer ? by_tile(bf16, std::integral_constant<int, 8>()) : by_tile(bf16, std::integral_constant<int, 4>());
    };
    return fa.bf16 ? by_length(std::true_type()) : by_length(std::false_type());
}

}  // namespace delta
