// Weight gradient of the 1x1 layers (any stride, no padding) for gfx950, bf16:
//   gw[k,c] = scale_k * sum_m gpre[m,k] * x[m,c]
// with m over the output's pixels; for a stride, x[m] is the input pixel under output pixel m.  Part of the backward
// pass whose accesses to stored activations DELTA's planner follows (Sec. 3, Assumptions 1-3).
//
// A "TN" product: both operands are stored pixel-major, the reduction index is the pixel.  Tiles are staged in LDS as they
// lie in memory (pixel rows x channels) and turned into MFMA operands by gfx950's transposing LDS read
// (ds_read_b64_tr_b16: 16 lanes point at 4 rows of 16 channels, each gets one channel's 4 values along the rows).
//  * A workgroup owns 64 KT x 64 CT of (k, c), 8 wavefronts (two on every SIMD): KT * CT tiles of 64 x 64 with QS = 8 /
//    (KT * CT) wavefronts on each, which share a slice's 16-pixel steps; their sums meet in LDS at the end.
//  * What bounds it is the delivery of the operands (64-128 FLOP per byte): slices of 64 or 128 pixels go from memory
//    straight into LDS (global_load_lds, no registers, no store instructions) through a ring of S slices, S - 1 of
//    them in flight per CU (80-120 KB), one barrier per slice.  Through registers with one chunk in flight and two
//    barriers per chunk the same tiles waited for every chunk.  Alone, with the reduction and the launches: 512 -> 2048 on
//    256 x 7 x 7 61 -> 46 us, 256 -> 1024 on 128 x 14 x 14 42 -> 33, 256 -> 512 stride 2 on 128 x 56 x 56 92 -> 52; 64 -> 256 on
//    32 x 56 x 56 is 14.5 us of kernel for 64 MB: bound by HBM.
//  * A strided layer's pixels are picked by the address each lane fetches; they used to be gathered by a kernel of their own.
//  * Workgroups are persistent over slices (split s takes slices s, s + nsplit, ...) and write their sums, in accumulator
//    order, to a partial buffer; wgrad_reduce_kernel adds them in the order of the splits.  No atomics: a fixed function of
//    the inputs.
// Rows past the last pixel are fetched from the last pixel and overwritten with zeros in LDS before they are read.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"

namespace delta {
namespace wg1 {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct Args {
    const unsigned char *x, *g;     // [N,H,W,C], [M,K] bf16
    float *partial;                 // [nsplit][tiles][KT * CT][4 tiles][4][64 lanes] f32x4
    int M, C, K, nslices, nsplit;
    int H, W, P, Q, stride;         // STRIDED only
    Divisor pq, q;                  // P Q, Q
};

template <int KT, int CT> struct Shape {
    static constexpr int kTiles = KT * CT, kQS = 8 / kTiles, kPixels = kTiles == 4 ? 64 : 128;   // of a slice
    static constexpr int kG = kPixels * KT * 128, kX = kPixels * CT * 128;                       // bytes of a slice
    static constexpr int kSlice = kG + kX, kStages = 160 * 1024 / kSlice < 4 ? 160 * 1024 / kSlice : 4;
    static constexpr int kGL = kG / 8192, kXL = kX / 8192, kLoads = kGL + kXL;                   // 1 KB loads per wavefront
    static constexpr int kSums = (kQS - 1) * kTiles * 16384;
    static constexpr int kLds = kStages * kSlice > kSums ? kStages * kSlice : kSums;
};

// Which way the 64-byte groups of LDS row `row` are permuted, so that the four consecutive rows a transposing read touches
// at one column lie in four different quarters of the 64 banks: rows of 128 bytes lie two to a 256-byte line, so
// bit 1 of the row number flips the group; wider rows start a line each and the low two bits flip it.
template <int TW>
__device__ __forceinline__ int swizzle(int row) { return TW == 1 ? (row >> 1) & 1 : row & 3; }

template <int KT, int CT, bool STRIDED>
__global__ __launch_bounds__(512) void wgrad1x1_kernel(Args a) {
    using T = Shape<KT, CT>;
    constexpr int GP = KT * 128, XP = CT * 128, S = T::kStages, QS = T::kQS;
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int base = wv % T::kTiles, qs = wv / T::kTiles, kw = base % KT, cw = base / KT;
    const int ktiles = a.K / (64 * KT), kt = blockIdx.y % ktiles, ct = blockIdx.y / ktiles;

    // ---- direct loads: one fills 1 KB of a slice, i.e. 8 / KT (8 / CT) rows; LDS slot s of row r holds segment s with its
    // 64-byte group permuted: the direct load fixes where a lane's 16 bytes land, so the permutation is applied to the
    // address each lane fetches
    int grow[T::kGL], xrow[T::kXL];
    uint32_t gseg[T::kGL], xseg[T::kXL];
#pragma unroll
    for (int i = 0; i < T::kGL; ++i) {
        const int b = (wv * T::kGL + i) * 1024 + lane * 16, s = (b % GP) >> 4;
        grow[i] = b / GP;
        gseg[i] = (uint32_t)(kt * GP + (((s >> 2) ^ swizzle<KT>(grow[i])) << 6) + (s & 3) * 16);
    }
#pragma unroll
    for (int i = 0; i < T::kXL; ++i) {
        const int b = (wv * T::kXL + i) * 1024 + lane * 16, s = (b % XP) >> 4;
        xrow[i] = b / XP;
        xseg[i] = (uint32_t)(ct * XP + (((s >> 2) ^ swizzle<CT>(xrow[i])) << 6) + (s & 3) * 16);
    }
    typedef __attribute__((address_space(3))) unsigned char *lptr_t;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)smem;
    // The waits for these loads are inline assembly as they are: the compiler does not track what a direct load writes.
    auto fetch = [&](int slice, int buf) {
        const int m0 = slice * T::kPixels, last = a.M - 1 - m0;  // rows past the last pixel: that pixel
        const uint32_t sb = lds0 + (uint32_t)(buf * T::kSlice + wv * T::kGL * 1024);
#pragma unroll
        for (int i = 0; i < T::kGL; ++i) {
            const int row = grow[i] < last ? grow[i] : last;
            const uint32_t off = (uint32_t)(m0 + row) * (uint32_t)a.K * 2u + gseg[i];
            load_lds_b128(a.g, off, sb + i * 1024);
        }
        const uint32_t sx = lds0 + (uint32_t)(buf * T::kSlice + T::kG + wv * T::kXL * 1024);
#pragma unroll
        for (int i = 0; i < T::kXL; ++i) {
            int m = m0 + (xrow[i] < last ? xrow[i] : last);
            if constexpr (STRIDED) {
                const int n = divide(m, a.pq), pq = m - n * (a.P * a.Q), p = divide(pq, a.q), q = pq - p * a.Q;
                m = (n * a.H + p * a.stride) * a.W + q * a.stride;
                load_lds_b128(a.x + (size_t)m * a.C * 2 + xseg[i], sx + i * 1024);       // x may be 2 GiB or more
            } else {
                load_lds_b128(a.x, (uint32_t)m * (uint32_t)a.C * 2u + xseg[i], sx + i * 1024);
            }
        }
    };
    // direct loads complete in order: "at most n later slices outstanding" is vmcnt(n * loads per slice)
    auto wait_slices = [&](int later) {
        if (later <= 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        else if (later == 1) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(T::kLoads) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * T::kLoads) : "memory");
    };

    // ---- transposing reads: a lane supplies row 8 (lane / 32) + (lane % 16) / 4 (+ 4) of a 16-pixel step and channels
    // 16 ((lane / 16) % 2) + 4 (lane % 4) .. + 3 of a 32-channel half; adding multiples of 4 to the row keeps its swizzle
    const int srow = 8 * (lane >> 5) + ((lane & 15) >> 2), scol = 32 * ((lane >> 4) & 1) + 8 * (lane & 3);
    int goff[2], xoff[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        goff[t] = srow * GP + (((kw * 2 + t) ^ swizzle<KT>(srow)) << 6) + scol;
        xoff[t] = T::kG + srow * XP + (((cw * 2 + t) ^ swizzle<CT>(srow)) << 6) + scol;
    }
    typedef s16x4 __attribute__((address_space(3))) * lds_ptr;
    auto tr_read = [&](const unsigned char *p) { return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p)); };

    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    const int mine = (a.nslices - (int)blockIdx.x + a.nsplit - 1) / a.nsplit;
    auto slice_of = [&](int t) { return (int)blockIdx.x + t * a.nsplit; };
#pragma unroll
    for (int t = 0; t < S - 1; ++t)
        if (t < mine) fetch(slice_of(t), t);
    for (int t = 0, buf = 0; t < mine; ++t) {
        wait_slices(mine - 1 - t < S - 2 ? mine - 1 - t : S - 2);        // this wavefront's part of slice t has landed
        __syncthreads();                                                 // everyone's has; the buffer of slice t - 1 is free
        const int nbuf = buf == 0 ? S - 1 : buf - 1;
        if (t + S - 1 < mine) fetch(slice_of(t + S - 1), nbuf);
        unsigned char *sl = smem + buf * T::kSlice;
        const int valid = a.M - slice_of(t) * T::kPixels;
        if (valid < T::kPixels) {                                        // the last slice of all: rows past the last pixel
            for (int i = tid; i < T::kSlice / 16; i += 512) {
                const int row = i * 16 < T::kG ? i * 16 / GP : (i * 16 - T::kG) / XP;
                if (row >= valid) *reinterpret_cast<u32x4 *>(sl + i * 16) = u32x4{0u, 0u, 0u, 0u};
            }
            __syncthreads();
        }
#pragma unroll
        for (int q = 0; q < T::kPixels / (16 * QS); ++q) {
            const int q0 = 16 * (qs + q * QS);
            s16x8 af[2], bf[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                af[h] = __builtin_shufflevector(tr_read(sl + q0 * GP + goff[h]), tr_read(sl + (q0 + 4) * GP + goff[h]), 0, 1, 2, 3, 4, 5, 6, 7);
                bf[h] = __builtin_shufflevector(tr_read(sl + q0 * XP + xoff[h]), tr_read(sl + (q0 + 4) * XP + xoff[h]), 0, 1, 2, 3, 4, 5, 6, 7);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, af[i]), __builtin_bit_cast(bf16x8, bf[j]),
                                                                        acc[i][j], 0, 0, 0);
        }
        buf = buf + 1 == S ? 0 : buf + 1;
    }

    // ---- the QS sums of a tile, added in the order of qs
    f32x4 sum[16];                                               // [i][j][e4]
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const f32x16 &v = acc[k >> 3][(k >> 2) & 1];
        sum[k] = f32x4{v[4 * (k & 3)], v[4 * (k & 3) + 1], v[4 * (k & 3) + 2], v[4 * (k & 3) + 3]};
    }
    if constexpr (QS > 1) {
        __syncthreads();                                         // the ring is dead
        f32x4 *red = reinterpret_cast<f32x4 *>(smem) + lane;     // [QS - 1][tiles][16][64]
        if (qs) {
#pragma unroll
            for (int k = 0; k < 16; ++k) red[((qs - 1) * T::kTiles + base) * 1024 + k * 64] = sum[k];
        }
        __syncthreads();
        if (qs) return;
#pragma unroll
        for (int g = 0; g < QS - 1; ++g)
#pragma unroll
            for (int k = 0; k < 16; ++k) sum[k] += red[(g * T::kTiles + base) * 1024 + k * 64];
    }
    f32x4 *out = reinterpret_cast<f32x4 *>(a.partial) + (((size_t)blockIdx.x * gridDim.y + blockIdx.y) * T::kTiles + base) * 1024 + lane;
#pragma unroll
    for (int k = 0; k < 16; ++k) out[k * 64] = sum[k];
}

// gw[k][c] = scale_k * sum over the splits of the partial sums, in a fixed order.  64 consecutive f32x4 of the blob (one per
// lane) are shared by G wavefronts (wavefront g adds splits g, g + G, ..., four loads in flight), whose G sums are then
// added in a fixed tree; a workgroup of 8 wavefronts takes 8 / G groups.  G follows the number of splits (about
// four loads per lane): with few splits (the wide layers: 4 or 16) every wavefront still has loads to issue, with many
// (256) the loads of a group are spread over the whole workgroup.  (Splitting a wavefront's lanes over four splits as
// well makes this kernel faster alone, 4 us at best, and the backward pass 3 % slower: beside the data-gradient
// stream its time is mostly waiting for free CUs, and more workgroups wait more.)  The accumulator layout of a 32x32 tile
// is: lane l holds column l % 32 and rows 8 e4 + 4 (l / 32) + e in register 4 e4 + e, so a thread's four sums go to
// four k rows of one c, and consecutive lanes write consecutive c.
template <int G>
__global__ __launch_bounds__(512) void wgrad_reduce_kernel(const float *partial, const float *scale, float *gw, int K, int C, int kt_w,
                                                           int ct_w, int nsplit) {
    __shared__ f32x4 part[8][64];
    const int ktiles = K / (64 * kt_w), pairs = kt_w * ct_w;
    const size_t per_split = (size_t)(K / 64) * (C / 64) * 1024;  // f32x4 of one split
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, grp = wave % G;
    const size_t idx = ((size_t)blockIdx.x * (8 / G) + wave / G) * 64 + lane;
    const f32x4 *src = reinterpret_cast<const f32x4 *>(partial) + idx;
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    int sp = grp;
    for (; sp + 3 * G < nsplit; sp += 4 * G) {                   // four independent loads in flight
        const f32x4 v0 = src[(size_t)sp * per_split], v1 = src[(size_t)(sp + G) * per_split];
        const f32x4 v2 = src[(size_t)(sp + 2 * G) * per_split], v3 = src[(size_t)(sp + 3 * G) * per_split];
        sum += (v0 + v1) + (v2 + v3);                            // in pairs: fewer roundings of the whole sum
    }
    for (; sp < nsplit; sp += G) sum += src[(size_t)sp * per_split];
    if constexpr (G > 1) {
        part[wave][lane] = sum;
        __syncthreads();
        if (grp != 0) return;
        f32x4 level[G];
#pragma unroll
        for (int g = 0; g < G; ++g) level[g] = part[wave + g][lane];
#pragma unroll
        for (int n = G / 2; n; n /= 2)
#pragma unroll
            for (int g = 0; g < n; ++g) level[g] += level[g + n];
        sum = level[0];
    }
    // idx = (((tile * pairs + pair) * 4 + quadrant) * 4 + e4) * 64 + lane
    const int i = (int)(idx >> 6), e4 = i & 3, quadrant = (i >> 2) & 3, pair = (i >> 4) % pairs, tile = (i >> 4) / pairs;
    const int c = ((tile / ktiles) * ct_w + pair / kt_w) * 64 + (quadrant & 1) * 32 + (lane & 31);
    const int k0 = ((tile % ktiles) * kt_w + pair % kt_w) * 64 + (quadrant >> 1) * 32 + 8 * e4 + 4 * (lane >> 5);
#pragma unroll
    for (int e = 0; e < 4; ++e) gw[(size_t)(k0 + e) * C + c] = sum[e] * scale[k0 + e];
}

// A workgroup's time per pixel, and what one more split of a 128 x 128 tile costs: its 64 KB written and read back.
static constexpr double kPixelNs = 5.5, kSumsNs = 24.;

struct Plan { int kt, ct, tiles, pixels, nslices, nsplit; };

// nullptr and a filled plan, or the reason the kernel does not apply.  `a`: the forward layer's own geometry.
const char *plan_for(const ConvArgs &a, Plan &p) {
    if (!a.bf16 || a.R != 1 || a.S != 1 || a.pad != 0 || a.stride < 1) return "weight gradient: 1x1, no padding, bf16";
    if (a.Cin % 64 || a.Cout % 64) return "weight gradient: channel counts must be multiples of 64";
    if ((unsigned long long)a.M * a.Cin * 2ull >= 0x7FFFFFFFull || (unsigned long long)a.M * a.Cout * 2ull >= 0x7FFFFFFFull)
        return "weight gradient: tensors of 2 GiB or more";
    if ((long long)a.N * a.H * a.W > 0x7FFFFFFFLL) return "weight gradient: too many pixels";
    // 128 x 128 where both channel counts allow, else four tiles along the one that does
    p.kt = a.Cout % 128 == 0 ? 2 : 1;
    p.ct = a.Cin % 128 == 0 ? 2 : 1;
    if (p.kt == 2 && p.ct == 1 && a.Cout % 256 == 0) p.kt = 4;
    if (p.ct == 2 && p.kt == 1 && a.Cin % 256 == 0) p.ct = 4;
    p.tiles = (a.Cout / (64 * p.kt)) * (a.Cin / (64 * p.ct));
    p.pixels = p.kt * p.ct == 4 ? 64 : 128;
    p.nslices = (a.M + p.pixels - 1) / p.pixels;
    p.nsplit = wgrad_splits(a.M, p.tiles, kPixelNs, kSumsNs * p.kt * p.ct / 4);
    if (p.nsplit > p.nslices) p.nsplit = p.nslices;
    return nullptr;
}

template <int KT, int CT, bool STRIDED>
hipError_t launch(const Args &w, const Plan &p, hipStream_t stream) {
    static bool raised = false;
    if (!raised) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&wgrad1x1_kernel<KT, CT, STRIDED>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, Shape<KT, CT>::kLds);
        if (e != hipSuccess) return e;
        raised = true;
    }
    wgrad1x1_kernel<KT, CT, STRIDED><<<dim3(p.nsplit, p.tiles), dim3(512), Shape<KT, CT>::kLds, stream>>>(w);
    return hipGetLastError();
}

template <int KT, int CT>
hipError_t launch(const Args &w, const Plan &p, bool strided, hipStream_t stream) {
    return strided ? launch<KT, CT, true>(w, p, stream) : launch<KT, CT, false>(w, p, stream);
}

}  // namespace wg1

const char *wgrad1x1_check(const ConvArgs &a) {
    wg1::Plan p;
    return wg1::plan_for(a, p);
}

size_t wgrad1x1_workspace_bytes(const ConvArgs &a) {
    wg1::Plan p;
    return wg1::plan_for(a, p) ? 0 : (size_t)p.nsplit * p.tiles * p.kt * p.ct * 16384;
}

// a: the forward layer's own geometry with a.x = x and a.scale = scale; g = gpre [M][Cout]; gw fp32 [Cout][Cin]; workspace
// of at least wgrad1x1_workspace_bytes(a), 16-byte aligned.
hipError_t launch_wgrad1x1(const ConvArgs &a, const void *g, float *gw, void *workspace, size_t workspace_bytes, hipStream_t stream) {
    wg1::Plan p;
    if (wg1::plan_for(a, p) || !g || !gw || !workspace || !a.x || !a.scale || workspace_bytes < wgrad1x1_workspace_bytes(a) ||
        ((uintptr_t)workspace | (uintptr_t)g | (uintptr_t)a.x) & 15)
        return hipErrorInvalidValue;
    wg1::Args w;
    w.x = static_cast<const unsigned char *>(a.x); w.g = static_cast<const unsigned char *>(g);
    w.partial = static_cast<float *>(workspace);
    w.M = a.M; w.C = a.Cin; w.K = a.Cout; w.nslices = p.nslices; w.nsplit = p.nsplit;
    w.H = a.H; w.W = a.W; w.P = a.P; w.Q = a.Q; w.stride = a.stride;
    w.pq = make_divisor((uint32_t)(a.P * a.Q)); w.q = make_divisor((uint32_t)a.Q);
    const bool strided = a.stride != 1;
    hipError_t e;
    switch (p.kt * 10 + p.ct) {
    case 11: e = wg1::launch<1, 1>(w, p, strided, stream); break;
    case 12: e = wg1::launch<1, 2>(w, p, strided, stream); break;
    case 14: e = wg1::launch<1, 4>(w, p, strided, stream); break;
    case 21: e = wg1::launch<2, 1>(w, p, strided, stream); break;
    case 22: e = wg1::launch<2, 2>(w, p, strided, stream); break;
    case 41: e = wg1::launch<4, 1>(w, p, strided, stream); break;
    default: return hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
    return launch_wgrad1x1_reduce(w.partial, a.scale, gw, a.Cout, a.Cin, p.kt, p.ct, p.nsplit, stream);
}

// Partial sums of `nsplit` splits, [nsplit][K C / (4096 kt ct)][kt ct][4 tiles][4][64 lanes] f32x4 (wgrad1x1_kernel's layout): gw = scale * their sum.
hipError_t launch_wgrad1x1_reduce(const float *partial, const float *scale, float *gw, int K, int C, int kt, int ct, int nsplit, hipStream_t stream) {
    const size_t groups = (size_t)(K / 64) * (C / 64) * 16;
    const int G = nsplit <= 4 ? 1 : nsplit <= 8 ? 2 : nsplit <= 16 ? 4 : 8;
    const dim3 grid((unsigned)(groups / (8 / G))), block(512);
    auto run = [&](auto kernel) { kernel<<<grid, block, 0, stream>>>(partial, scale, gw, K, C, kt, ct, nsplit); };
    switch (G) {
    case 1: run(wg1::wgrad_reduce_kernel<1>); break;
    case 2: run(wg1::wgrad_reduce_kernel<2>); break;
    case 4: run(wg1::wgrad_reduce_kernel<4>); break;
    default: run(wg1::wgrad_reduce_kernel<8>); break;
    }
    return hipGetLastError();
}

}  // namespace delta
