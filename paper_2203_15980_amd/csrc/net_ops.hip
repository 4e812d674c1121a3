// The operators of a ResNet that are not bottleneck convolutions: the 7x7 stem, max
// pooling, global average pooling and the mean softmax cross-entropy.  DELTA regenerates
// them like any other operator output (Sec. 5.5 lists PoolingForward among the tensors that
// are released and recomputed), so they go through delta_recompute_segment as well.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"

namespace delta {

typedef __bf16 bf16x8_s __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_s __attribute__((ext_vector_type(2)));
typedef float f32x2_s __attribute__((ext_vector_type(2)));
typedef float f32x16_s __attribute__((ext_vector_type(16)));
typedef float f32x4_s __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_s __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_s __attribute__((ext_vector_type(2)));

namespace {
__device__ __forceinline__ uint32_t pack2s(float lo, float hi) {
    const f32x2_s v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_s));
}
__device__ __forceinline__ float blo(uint32_t p) { return __uint_as_float(p << 16); }
__device__ __forceinline__ float bhi(uint32_t p) { return __uint_as_float(p & 0xFFFF0000u); }
}  // namespace

// ------------------------------------------------------------------------------ stem
// 7x7, stride 2, pad 3, Cin = 3, Cout = 64, bf16.  Implicit GEMM on the matrix cores with the
// reduction axis laid out as (r, s, c padded to 4): for a fixed kernel row r the 7 taps x 4
// channels of one output pixel are 28 contiguous elements of the input patch once its
// pixels are padded from 3 to 4 channels, starting at a 16-byte boundary (stride 2 x 4
// channels x 2 bytes).  Each row is rounded up to 32 elements -- the extra tap and the
// fourth channel carry zero weights -- so K = 7 x 32 = 224, fourteen 32x32x16 steps.
//
// The layer is bound by its 128 bytes of output per pixel (24.5 input bytes, 224 MFMA steps per
// 32 pixels), so the kernel is built around the memory side:
//  * a workgroup (4 wavefronts, two workgroups per CU) owns 8 output rows x 112 output columns at
//    a time and is persistent over such tiles; the 21 x 240 input pixels a tile needs are whole
//    16-byte-aligned runs of the image rows when the image width is a multiple of 8: a thread
//    fetches 8 pixels (48 bytes) with three 16-byte loads and writes them to LDS as 8 padded
//    pixels.  The next tile's pixels are requested before the current tile is multiplied and wait
//    in registers.  (Other widths take one pixel per thread and step.)
//  * the rearranged weights live in registers (112 per lane) for the whole launch, so the inner
//    loop is one 16-byte LDS read per two MFMAs;
//  * a wavefront finishes 32 pixels (2 rows x 16 columns) at a time through a private fp32 LDS tile
//    that turns channel-major accumulators into pixel rows; scale, shift, ReLU and the rounding
//    happen on the row side, where a lane's 8 channels are the same for every pixel (16 registers
//    instead of 32 LDS reads per 32 pixels), and stores are whole 128-byte lines.
static constexpr int kStemRO = 8, kStemCQ = 112;              // output rows x columns of a tile
static constexpr int kStemPRows = 2 * kStemRO + 5;             // 21 input rows
static constexpr int kStemGroups = (2 * kStemCQ + 16) / 8;     // 30 groups of 8 input pixels per row
// input pixel w of a tile whose first output column is q0 sits at position w - 2 q0 + 11 of its row:
// groups start at position 3, the taps of output column q at position 2 (q - q0) + 8 (16-byte aligned)
static constexpr int kStemPPitch = (3 + 8 * kStemGroups + 1) * 8;   // 1952 bytes
static constexpr int kStemPatch = kStemPRows * kStemPPitch;          // 40992 bytes
static constexpr int kStemTasks = kStemPRows * kStemGroups;          // 630 groups per tile
static constexpr int kStemTPitch = 64 * 4 + 16;                      // fp32 row of 64 channels + pad
static constexpr int kStemLds = kStemPatch + 4 * 32 * kStemTPitch;
static_assert(64 * (7 * 64 + 16) <= kStemPatch, "the weights are staged in the patch buffer first");

__global__ __launch_bounds__(256, 2) void stem7x7_kernel(ConvArgs a, int tiles_p, int tiles_q, int ntiles, int aligned) {
    __shared__ __align__(16) unsigned char lds[kStemLds];
    unsigned char *patch = lds;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int l32 = lane & 31, half = lane >> 5;
    unsigned char *ttile = lds + kStemPatch + wv * (32 * kStemTPitch);
    const uint16_t *wg = static_cast<const uint16_t *>(a.w);
    const uint16_t *xg = static_cast<const uint16_t *>(a.x);

    // ---- weights: wl[k][r][s*4 + c] = w[k][r][s][c], zero for s = 7 or c = 3; through LDS (the patch
    // buffer, not yet in use) into registers: wreg[r][hh][u] = 8 elements 16 hh + 8 half .. of row r of
    // output channel 32 u + l32
    {
        constexpr int WP = 7 * 64 + 16;
        for (int e = tid; e < 64 * 7 * 32; e += 256) {
            const int k = e / 224, rem = e - k * 224;
            const int r = rem >> 5, el = rem & 31;
            const int s = el >> 2, c = el & 3;
            uint16_t v = 0;
            if (s < 7 && c < 3) v = wg[((k * 7 + r) * 7 + s) * 3 + c];
            *reinterpret_cast<uint16_t *>(patch + k * WP + r * 64 + el * 2) = v;
        }
    }
    __syncthreads();
    u32x4_s wreg[7][2][2];
    {
        constexpr int WP = 7 * 64 + 16;
        const unsigned char *wrow = patch + l32 * WP + half * 16;
#pragma unroll
        for (int r = 0; r < 7; ++r)
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                wreg[r][hh][0] = *reinterpret_cast<const u32x4_s *>(wrow + r * 64 + hh * 32);
                wreg[r][hh][1] = *reinterpret_cast<const u32x4_s *>(wrow + 32 * WP + r * 64 + hh * 32);
            }
    }
    const int trow = lane >> 3, tseg = lane & 7;
    float sc[8], sh[8];                             // of channels 8 tseg .. + 8, the ones this lane finishes
    {
        const f32x4_s s0 = *reinterpret_cast<const f32x4_s *>(a.scale + tseg * 8), s1 = *reinterpret_cast<const f32x4_s *>(a.scale + tseg * 8 + 4);
        const f32x4_s h0 = *reinterpret_cast<const f32x4_s *>(a.shift + tseg * 8), h1 = *reinterpret_cast<const f32x4_s *>(a.shift + tseg * 8 + 4);
        sc[0] = s0.x; sc[1] = s0.y; sc[2] = s0.z; sc[3] = s0.w; sc[4] = s1.x; sc[5] = s1.y; sc[6] = s1.z; sc[7] = s1.w;
        sh[0] = h0.x; sh[1] = h0.y; sh[2] = h0.z; sh[3] = h0.w; sh[4] = h1.x; sh[5] = h1.y; sh[6] = h1.z; sh[7] = h1.w;
    }

    // ---- input staging.  Aligned form: task (row i, group g) = 8 pixels, three per thread and tile.
    u32x4_s pre[3][3];
    auto tile_origin = [&](int tile, int &n, int &p0, int &q0) {
        n = tile / (tiles_p * tiles_q);
        const int t2 = tile - n * tiles_p * tiles_q;
        p0 = (t2 / tiles_q) * kStemRO;
        q0 = (t2 % tiles_q) * kStemCQ;
    };
    // Every thread issues its three loads unconditionally (pieces outside the image or past the task list
    // read the first bytes of the image instead and are zeroed when they are written to LDS): nothing
    // depends on the loaded registers until then, so the loads stay in flight under the MFMAs.
    uint32_t pre_ok = 0;
    auto request = [&](int tile) {                   // aligned form only
        int n, p0, q0;
        tile_origin(tile, n, p0, q0);
        pre_ok = 0;
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const int idx = tid + 256 * t;
            const int i = idx / kStemGroups, g = idx - i * kStemGroups;
            const int h = 2 * p0 - 3 + i, w0 = 2 * q0 - 8 + 8 * g;
            const bool ok = idx < kStemTasks && (unsigned)h < (unsigned)a.H && w0 >= 0 && w0 + 8 <= a.W;
            pre_ok |= ok ? 1u << t : 0u;
            const u32x4_s *src = reinterpret_cast<const u32x4_s *>(xg + ((size_t)((size_t)n * a.H + (ok ? h : 0)) * a.W + (ok ? w0 : 0)) * 3);
#pragma unroll
            for (int q = 0; q < 3; ++q) pre[t][q] = src[q];
        }
    };
    auto deposit = [&]() {                           // 24 bf16 = 8 pixels x 3 channels -> 8 x (3 channels + 0)
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const int idx = tid + 256 * t;
            if (idx >= kStemTasks) continue;
            const int i = idx / kStemGroups, g = idx - i * kStemGroups;
            const uint32_t keep = (pre_ok >> t) & 1u ? 0xFFFFFFFFu : 0u;
            const uint32_t d[12] = {pre[t][0].x & keep, pre[t][0].y & keep, pre[t][0].z & keep, pre[t][0].w & keep,
                                    pre[t][1].x & keep, pre[t][1].y & keep, pre[t][1].z & keep, pre[t][1].w & keep,
                                    pre[t][2].x & keep, pre[t][2].y & keep, pre[t][2].z & keep, pre[t][2].w & keep};
            unsigned char *dst = patch + i * kStemPPitch + (3 + 8 * g) * 8;
#pragma unroll
            for (int px = 0; px < 8; ++px) {
                // elements 3 px, 3 px + 1, 3 px + 2 of the 24
                const int e0 = 3 * px;
                uint32_t lo, hi;
                if (e0 & 1) {                        // starts in the upper half of a dword
                    lo = (d[e0 >> 1] >> 16) | (d[(e0 >> 1) + 1] << 16);
                    hi = d[(e0 >> 1) + 1] >> 16;
                } else {
                    lo = d[e0 >> 1];
                    hi = d[(e0 >> 1) + 1] & 0xFFFFu;
                }
                *reinterpret_cast<u32x2_s *>(dst + px * 8) = u32x2_s{lo, hi};
            }
        }
    };
    auto stage_any = [&](int tile) {                 // any width: one pixel per thread and step
        int n, p0, q0;
        tile_origin(tile, n, p0, q0);
        constexpr int COLS = 8 * kStemGroups;
        for (int e = tid; e < kStemPRows * COLS; e += 256) {
            const int i = e / COLS, j = e - i * COLS;
            const int h = 2 * p0 - 3 + i, w = 2 * q0 - 8 + j;
            u32x2_s v = {0u, 0u};
            if ((unsigned)h < (unsigned)a.H && (unsigned)w < (unsigned)a.W) {
                const uint16_t *px = xg + ((size_t)((size_t)n * a.H + h) * a.W + w) * 3;
                v.x = (uint32_t)px[0] | ((uint32_t)px[1] << 16);
                v.y = (uint32_t)px[2];
            }
            *reinterpret_cast<u32x2_s *>(patch + i * kStemPPitch + (3 + j) * 8) = v;
        }
    };

    int tile = blockIdx.x;
    if (aligned && tile < ntiles) request(tile);
    for (; tile < ntiles; tile += gridDim.x) {
        int n, p0, q0;
        tile_origin(tile, n, p0, q0);
        __syncthreads();                             // the previous tile's patch (or the weights) is no longer read
        if (aligned) deposit(); else stage_any(tile);
        __syncthreads();
        if (aligned && tile + (int)gridDim.x < ntiles) request(tile + gridDim.x);   // in flight under the MFMAs

        // ---- 28 units of 2 rows x 16 columns, seven per wavefront
        for (int j = 0; j < 7; ++j) {
            const int unit = wv + 4 * j, ur = unit / 7, uc = unit - ur * 7;
            if (p0 + 2 * ur >= a.P || q0 + 16 * uc >= a.Q) continue;          // the same for the whole wavefront
            const int prow = 2 * ur + (l32 >> 4), pcol = 16 * uc + (l32 & 15);
            f32x16_s acc[2];
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[u][e] = 0.f;
            const unsigned char *xrow = patch + (2 * prow) * kStemPPitch + pcol * 16 + 64 + half * 16;
            // the pixel operand of step k + 4 is requested before step k is multiplied (a ring of four):
            // with two wavefronts per SIMD one read ahead does not cover the LDS latency
            u32x4_s xq[4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                xq[k] = *reinterpret_cast<const u32x4_s *>(xrow + (k >> 1) * kStemPPitch + (k & 1) * 32);
            __builtin_amdgcn_sched_barrier(0);       // (the scheduler would otherwise pull the reads back to one step ahead)
#pragma unroll
            for (int k = 0; k < 14; ++k) {
                const u32x4_s xb = xq[k & 3];
                if (k + 4 < 14)
                    xq[k & 3] = *reinterpret_cast<const u32x4_s *>(xrow + ((k + 4) >> 1) * kStemPPitch + ((k + 4) & 1) * 32);
                acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_s, wreg[k >> 1][k & 1][0]),
                                                                 __builtin_bit_cast(bf16x8_s, xb), acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_s, wreg[k >> 1][k & 1][1]),
                                                                 __builtin_bit_cast(bf16x8_s, xb), acc[1], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            // acc[u][4 rb + e] = channel 32 u + 8 rb + 4 half + e of pixel l32 -> fp32 rows in the private tile
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int rb = 0; rb < 4; ++rb) {
                    const f32x4_s v = {acc[u][4 * rb], acc[u][4 * rb + 1], acc[u][4 * rb + 2], acc[u][4 * rb + 3]};
                    *reinterpret_cast<f32x4_s *>(ttile + l32 * kStemTPitch + (u * 32 + 8 * rb + 4 * half) * 4) = v;
                }
            // (LDS instructions of one wavefront execute in order; the fences only keep the compiler from
            // moving accesses across the exchange)
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int pr = trow + 8 * t;         // pixel of the unit: row pr / 16, column pr % 16
                const f32x4_s f0 = *reinterpret_cast<const f32x4_s *>(ttile + pr * kStemTPitch + tseg * 32);
                const f32x4_s f1 = *reinterpret_cast<const f32x4_s *>(ttile + pr * kStemTPitch + tseg * 32 + 16);
                float o[8] = {f0.x, f0.y, f0.z, f0.w, f1.x, f1.y, f1.z, f1.w};
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = o[e] * sc[e] + sh[e];
                if (a.relu) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) o[e] = o[e] < 0.f ? 0.f : o[e];
                }
                u32x4_s o4;
                o4.x = pack2s(o[0], o[1]); o4.y = pack2s(o[2], o[3]);
                o4.z = pack2s(o[4], o[5]); o4.w = pack2s(o[6], o[7]);
                const int p = p0 + 2 * ur + (pr >> 4), q = q0 + 16 * uc + (pr & 15);
                if (p < a.P && q < a.Q)
                    *reinterpret_cast<u32x4_s *>(static_cast<unsigned char *>(a.y) +
                                                 ((size_t)((size_t)n * a.P + p) * a.Q + q) * 128 + tseg * 16) = o4;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    }
}

bool stem_applies(const ConvArgs &a) {
    return a.bf16 && a.R == 7 && a.S == 7 && a.stride == 2 && a.pad == 3 && a.Cin == 3 && a.Cout == 64 && !a.res;
}

const char *stem_check(const ConvArgs &a) {
    if (a.N <= 0 || a.H <= 0 || a.W <= 0) return "non-positive dimension";
    if (a.P != (a.H + 6 - 7) / 2 + 1 || a.Q != (a.W + 6 - 7) / 2 + 1 || a.P <= 0 || a.Q <= 0)
        return "inconsistent output size";
    if ((long long)a.N * a.P * a.Q != a.M || (long long)a.N * a.H * a.W > 0x7FFFFFFFLL) return "bad M";
    if (!a.x || !a.w || !a.y || !a.scale || !a.shift) return "null pointer";
    if (((uintptr_t)a.y | (uintptr_t)a.scale | (uintptr_t)a.shift) & 15) return "pointers must be 16-byte aligned";
    if (((uintptr_t)a.x | (uintptr_t)a.w) & 1) return "pointers must be 2-byte aligned";
    return nullptr;
}

hipError_t launch_stem(const ConvArgs &a, hipStream_t stream) {
    if (!stem_applies(a) || stem_check(a)) return hipErrorInvalidValue;
    const int tiles_p = (a.P + kStemRO - 1) / kStemRO, tiles_q = (a.Q + kStemCQ - 1) / kStemCQ;
    const long long ntiles = (long long)a.N * tiles_p * tiles_q;
    if (ntiles <= 0 || ntiles > 0x3FFFFFFFLL) return hipErrorInvalidValue;
    const int grid = (int)(ntiles < 512 ? ntiles : 512);            // two workgroups per CU
    // whole 16-byte runs of 8 pixels: rows start 16-byte aligned when the width is a multiple of 8
    const int aligned = a.W % 8 == 0 && ((uintptr_t)a.x & 15) == 0;
    stem7x7_kernel<<<dim3(grid), dim3(256), 0, stream>>>(a, tiles_p, tiles_q, (int)ntiles, aligned);
    return hipGetLastError();
}

// --------------------------------------------------------------------------- pooling

// One thread: 16 bytes of channels (8 bf16 or 4 fp32) of one output pixel.  Bound by memory: a window of 3 x 3 (W3) has its nine loads in flight at once,
// those outside the image repeated from its edge, which is in the window too: 128 x 112 x 112 x 64, stride 2 66.9 -> 52.8 us, 4.9 TB/s.  Other windows
// load one piece after the other.
template <bool BF16, bool W3>
__global__ __launch_bounds__(256) void maxpool_kernel(PoolArgs a, long long total) {
    // Workgroups are dealt round-robin to the 8 XCDs; each XCD takes a contiguous range of outputs, so
    // that the input rows two neighbouring output rows share are fetched into one L2, once (with
    // neighbouring output rows on different XCDs the 3 x 3 stride-2 pool fetched 1.5 x its input).
    const unsigned nb = gridDim.x, per = nb >> 3, rem = nb & 7u;
    const unsigned xcd = blockIdx.x & 7u, slot = blockIdx.x >> 3;
    const unsigned logical = xcd < rem ? xcd * (per + 1) + slot : rem * (per + 1) + (xcd - rem) * per + slot;
    const long long idx = (long long)logical * 256 + threadIdx.x;
    if (idx >= total) return;
    constexpr int CPT = BF16 ? 8 : 4;
    const int chunks = a.C / CPT;
    const int ck = (int)(idx % chunks);
    long long pix = idx / chunks;
    const int q = (int)(pix % a.Q);
    pix /= a.Q;
    const int p = (int)(pix % a.P);
    const int n = (int)(pix / a.P);
    float m[CPT];
#pragma unroll
    for (int e = 0; e < CPT; ++e) m[e] = -INFINITY;
    const unsigned char *xg = static_cast<const unsigned char *>(a.x);
    auto take = [&](const u32x4_s v) {
        if constexpr (BF16) {
            m[0] = fmaxf(m[0], blo(v.x)); m[1] = fmaxf(m[1], bhi(v.x));
            m[2] = fmaxf(m[2], blo(v.y)); m[3] = fmaxf(m[3], bhi(v.y));
            m[4] = fmaxf(m[4], blo(v.z)); m[5] = fmaxf(m[5], bhi(v.z));
            m[6] = fmaxf(m[6], blo(v.w)); m[7] = fmaxf(m[7], bhi(v.w));
        } else {
            m[0] = fmaxf(m[0], __uint_as_float(v.x)); m[1] = fmaxf(m[1], __uint_as_float(v.y));
            m[2] = fmaxf(m[2], __uint_as_float(v.z)); m[3] = fmaxf(m[3], __uint_as_float(v.w));
        }
    };
    if constexpr (W3) {
        u32x4_s v[9];
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            int h = p * a.stride + t / 3 - a.pad, w = q * a.stride + t % 3 - a.pad;
            h = h < 0 ? 0 : h < a.H ? h : a.H - 1;
            w = w < 0 ? 0 : w < a.W ? w : a.W - 1;
            v[t] = *reinterpret_cast<const u32x4_s *>(xg + (((size_t)((size_t)n * a.H + h) * a.W + w) * chunks + ck) * 16);
        }
#pragma unroll
        for (int t = 0; t < 9; ++t) take(v[t]);
    } else {
        for (int r = 0; r < a.R; ++r) {
            const int h = p * a.stride + r - a.pad;
            if ((unsigned)h >= (unsigned)a.H) continue;
            for (int s = 0; s < a.S; ++s) {
                const int w = q * a.stride + s - a.pad;
                if ((unsigned)w >= (unsigned)a.W) continue;
                take(*reinterpret_cast<const u32x4_s *>(xg + (((size_t)((size_t)n * a.H + h) * a.W + w) * chunks + ck) * 16));
            }
        }
    }
    u32x4_s o;
    if constexpr (BF16) {
        o.x = pack2s(m[0], m[1]); o.y = pack2s(m[2], m[3]); o.z = pack2s(m[4], m[5]); o.w = pack2s(m[6], m[7]);
    } else {
        o.x = __float_as_uint(m[0]); o.y = __float_as_uint(m[1]); o.z = __float_as_uint(m[2]); o.w = __float_as_uint(m[3]);
    }
    *reinterpret_cast<u32x4_s *>(static_cast<unsigned char *>(a.y) + (size_t)idx * 16) = o;
}

// Global average.  G wavefronts of a workgroup's eight share 64 (image, 16 bytes of channels) pairs, one per lane: wavefront g
// takes pixels g, g + G, ..., four of its loads are in flight, and the G fp32 sums are
// added in the order of g through LDS.  HBM-bound: 128 x 7 x 7 x 2048 is 25.7 MB; with one thread per pair walking all
// pixels the launch was 512 wavefronts and 17 us, with eight per pair 6.6.  Up to 16 pixels a wavefront has too little to do for
// that: one per pair.  bf16, us, one | eight wavefronts: 2^20 pairs of 1 pixel 6.1 | 17.4, 4 pixels 14.0 | 22.0, 9 pixels
// 25.6 | 29.7, 16 pixels 42.8 | 45.8, 25 pixels 80 | 75, 49 pixels 151 | 141; 2^16 pairs of 9 pixels 5.0 | 4.6 (both the launch), 25
// pixels 6.0 | 5.0.
template <bool BF16, int G>
__global__ __launch_bounds__(512) void avgpool_kernel(PoolArgs a, long long total) {
    constexpr int CPT = BF16 ? 8 : 4;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, g = wv % G;
    const long long idx = ((long long)blockIdx.x * (8 / G) + wv / G) * 64 + lane;
    const int chunks = a.C / CPT, hw = a.H * a.W;
    float s[CPT];
#pragma unroll
    for (int e = 0; e < CPT; ++e) s[e] = 0.f;
    if (idx < total) {
        const int ck = (int)(idx % chunks), n = (int)(idx / chunks);
        const u32x4_s *xg = static_cast<const u32x4_s *>(a.x) + (size_t)n * hw * chunks + ck;
#pragma unroll 4
        for (int i = g; i < hw; i += G) {
            const u32x4_s v = xg[(size_t)i * chunks];
            if constexpr (BF16) {
                s[0] += blo(v.x); s[1] += bhi(v.x); s[2] += blo(v.y); s[3] += bhi(v.y);
                s[4] += blo(v.z); s[5] += bhi(v.z); s[6] += blo(v.w); s[7] += bhi(v.w);
            } else {
                s[0] += __uint_as_float(v.x); s[1] += __uint_as_float(v.y);
                s[2] += __uint_as_float(v.z); s[3] += __uint_as_float(v.w);
            }
        }
    }
    if constexpr (G > 1) {
        __shared__ float part[8][64][CPT + 1];
#pragma unroll
        for (int e = 0; e < CPT; ++e) part[wv][lane][e] = s[e];
        __syncthreads();
        if (g != 0) return;
#pragma unroll
        for (int k = 1; k < G; ++k)
#pragma unroll
            for (int e = 0; e < CPT; ++e) s[e] += part[wv + k][lane][e];
    }
    if (idx >= total) return;
    const float inv = 1.0f / (float)hw;
    u32x4_s o;
    if constexpr (BF16) {
        o.x = pack2s(s[0] * inv, s[1] * inv); o.y = pack2s(s[2] * inv, s[3] * inv);
        o.z = pack2s(s[4] * inv, s[5] * inv); o.w = pack2s(s[6] * inv, s[7] * inv);
    } else {
        o.x = __float_as_uint(s[0] * inv); o.y = __float_as_uint(s[1] * inv);
        o.z = __float_as_uint(s[2] * inv); o.w = __float_as_uint(s[3] * inv);
    }
    *reinterpret_cast<u32x4_s *>(static_cast<unsigned char *>(a.y) + (size_t)idx * 16) = o;
}

const char *pool_check(const PoolArgs &a, bool global_avg) {
    const int cpt = a.bf16 ? 8 : 4;
    if (a.N <= 0 || a.H <= 0 || a.W <= 0 || a.C <= 0) return "non-positive dimension";
    if (a.C % cpt) return "channels must be a multiple of 8 (bf16) or 4 (fp32)";
    if (!a.x || !a.y || (((uintptr_t)a.x | (uintptr_t)a.y) & 15)) return "pointers must be non-null and 16-byte aligned";
    if ((long long)a.N * a.H * a.W > 0x7FFFFFFFLL) return "input too large";
    if (!global_avg) {
        if (a.R <= 0 || a.S <= 0 || a.stride <= 0 || a.pad < 0 || a.pad >= a.R || a.pad >= a.S)
            return "bad window (padding must be smaller than the window)";
        if (a.P != (a.H + 2 * a.pad - a.R) / a.stride + 1 || a.Q != (a.W + 2 * a.pad - a.S) / a.stride + 1 ||
            a.P <= 0 || a.Q <= 0)
            return "inconsistent output size";
    }
    return nullptr;
}

hipError_t launch_maxpool(const PoolArgs &a, hipStream_t stream) {
    if (pool_check(a, false)) return hipErrorInvalidValue;
    const long long total = (long long)a.N * a.P * a.Q * (a.C / (a.bf16 ? 8 : 4));
    const long long blocks = (total + 255) / 256;
    if (blocks > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks), block(256);
    const bool w3 = a.R == 3 && a.S == 3;
    if (a.bf16 && w3) maxpool_kernel<true, true><<<grid, block, 0, stream>>>(a, total);
    else if (a.bf16) maxpool_kernel<true, false><<<grid, block, 0, stream>>>(a, total);
    else if (w3) maxpool_kernel<false, true><<<grid, block, 0, stream>>>(a, total);
    else maxpool_kernel<false, false><<<grid, block, 0, stream>>>(a, total);
    return hipGetLastError();
}

hipError_t launch_avgpool(const PoolArgs &a, hipStream_t stream) {
    if (pool_check(a, true)) return hipErrorInvalidValue;
    const long long total = (long long)a.N * (a.C / (a.bf16 ? 8 : 4));
    auto run = [&](auto kernel, int G) {
        const long long pairs = 64 * (8 / G), blocks = (total + pairs - 1) / pairs;
        if (blocks > 0x7FFFFFFFLL) return hipErrorInvalidValue;
        kernel<<<dim3((unsigned)blocks), dim3(512), 0, stream>>>(a, total);
        return hipGetLastError();
    };
    if ((long long)a.H * a.W <= 16) return a.bf16 ? run(avgpool_kernel<true, 1>, 1) : run(avgpool_kernel<false, 1>, 1);
    return a.bf16 ? run(avgpool_kernel<true, 8>, 8) : run(avgpool_kernel<false, 8>, 8);
}

// ------------------------------------------------------------------------------ loss
// Mean over images of logsumexp(z_i) - z_i[label_i].  One workgroup of 16 wavefronts: the result is one float,
// and what the launch costs is the latency of its loads and reductions.  PIECES (bf16 rows of whole 16-byte pieces, up to 1024
// classes): a wavefront holds four images at once, two pieces per lane and image, so that each logit is read once and the
// images' reduction trees interleave.  ELEMENTS (other rows of 257 to 1024 classes): a lane holds classes lane, lane + 64, ...
// of two images (four spill).  REREAD (up to 256 classes, or more than 1024): an image at a time, the row read twice.  128 images,
// us, REREAD | ELEMENTS: fp32 127 classes 9.9 | 13, 250 12.8 | 12.9, 310 14.5 | 13.0, 1000 34 | 13; bf16 127 10.2 | 14.1,
// 250 13.6 | 14.0, 310 15.4 | 14.0, 1001 35 | 14; bf16 1000 in pieces 12.5.  Fixed
// reduction trees and a fixed image -> wavefront map: the result does not depend on timing.
// A label outside [0, classes) makes the result NaN, so that it cannot pass unnoticed.
template <bool BF16>
__device__ __forceinline__ float logit_at(const void *logits, size_t idx) {
    return BF16 ? __uint_as_float((uint32_t)static_cast<const uint16_t *>(logits)[idx] << 16)
                : static_cast<const float *>(logits)[idx];
}

enum LossForm { REREAD, ELEMENTS, PIECES };

template <bool BF16, LossForm FORM>
__global__ __launch_bounds__(1024) void softmax_ce_kernel(const void *logits, const long long *labels, int N,
                                                          int classes, float *out) {
    constexpr int WAVES = 16, IMGS = FORM == PIECES ? 4 : 2;
    __shared__ float part[WAVES];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    float total = 0.f;
    auto logit_of_label = [&](int i) {
        const long long lab = labels[i];
        return lab >= 0 && lab < classes ? logit_at<BF16>(logits, (size_t)i * classes + lab) : __builtin_nanf("");
    };
    if constexpr (FORM != REREAD) {
        const int pieces = classes / 8;
        auto live = [&](int k) { return FORM == PIECES ? lane + 64 * (k >> 3) < pieces : lane + 64 * k < classes; };
        for (int i0 = wv * IMGS; i0 < N; i0 += WAVES * IMGS) {
            u32x4_s v[IMGS][2];
            float held[IMGS][16];
            float zl[IMGS], mx[IMGS], se[IMGS];
#pragma unroll
            for (int u = 0; u < IMGS; ++u) {
                const int i = i0 + u < N ? i0 + u : N - 1;        // past the last image: read again, not counted
                if constexpr (FORM == PIECES) {
                    const u32x4_s *z = reinterpret_cast<const u32x4_s *>(static_cast<const uint16_t *>(logits) + (size_t)i * classes);
#pragma unroll
                    for (int p = 0; p < 2; ++p) v[u][p] = z[lane + 64 * p < pieces ? lane + 64 * p : 0];
                } else {
#pragma unroll
                    for (int k = 0; k < 16; ++k) held[u][k] = logit_at<BF16>(logits, (size_t)i * classes + (live(k) ? lane + 64 * k : 0));
                }
                zl[u] = logit_of_label(i);
            }
            auto at = [&](int u, int k) {                        // value k of the lane's 16, -inf past the row
                if constexpr (FORM == PIECES) {
                    const u32x4_s q = v[u][k >> 3];
                    const uint32_t w = q[(k & 7) >> 1];
                    return live(k) ? ((k & 1) ? bhi(w) : blo(w)) : -INFINITY;
                } else {
                    return live(k) ? held[u][k] : -INFINITY;
                }
            };
#pragma unroll
            for (int u = 0; u < IMGS; ++u) {
                mx[u] = -INFINITY;
#pragma unroll
                for (int k = 0; k < 16; ++k) mx[u] = fmaxf(mx[u], at(u, k));
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1)
#pragma unroll
                for (int u = 0; u < IMGS; ++u) mx[u] = fmaxf(mx[u], __shfl_xor(mx[u], o));
#pragma unroll
            for (int u = 0; u < IMGS; ++u) {
                se[u] = 0.f;
#pragma unroll
                for (int k = 0; k < 16; ++k) se[u] += live(k) ? __expf(at(u, k) - mx[u]) : 0.f;
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1)
#pragma unroll
                for (int u = 0; u < IMGS; ++u) se[u] += __shfl_xor(se[u], o);
#pragma unroll
            for (int u = 0; u < IMGS; ++u)
                if (i0 + u < N) total += (mx[u] + __logf(se[u])) - zl[u];
        }
    } else {
        for (int i = wv; i < N; i += WAVES) {
            float mx = -INFINITY;
            for (int c = lane; c < classes; c += 64) mx = fmaxf(mx, logit_at<BF16>(logits, (size_t)i * classes + c));
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
            float se = 0.f;
            for (int c = lane; c < classes; c += 64) se += __expf(logit_at<BF16>(logits, (size_t)i * classes + c) - mx);
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) se += __shfl_xor(se, o);
            total += (mx + __logf(se)) - logit_of_label(i);
        }
    }
    if (lane == 0) part[wv] = total;
    __syncthreads();
    if (threadIdx.x == 0) {
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) sum += part[w];
        out[0] = sum / (float)N;
    }
}

// The same over several workgroups: a wavefront per image, and the workgroup that finishes last adds the images'
// losses, every 256th to a thread, then a tree (fixed, whichever workgroup it is).  `losses`: N floats, `done`: a
// counter that is zero between launches - the last workgroup leaves it so.  Losses and counter pass between XCDs, whose L2s know nothing of
// each other: device-scope stores, loads and counter.  us, one workgroup | this, 1000
// classes: 17 images 4.7 | 5.4, 32 5.2 | 5.4, 64 7.2 | 6.2, 128 11.9 | 6.7, 256 22 | 8.7, 1024 79 | 22, 4096 342 | 78: from 33 images on.
__global__ __launch_bounds__(256) void softmax_ce_wide_kernel(const void *logits, const long long *labels, int N, int classes, float *out,
                                                              float *losses, unsigned *done) {
    __shared__ bool last;
    __shared__ float part[4];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, i = blockIdx.x * 4 + wv, pieces = classes / 8;
    if (i < N) {
        const u32x4_s *z = reinterpret_cast<const u32x4_s *>(static_cast<const uint16_t *>(logits) + (size_t)i * classes);
        u32x4_s v[2];
#pragma unroll
        for (int p = 0; p < 2; ++p) v[p] = z[lane + 64 * p < pieces ? lane + 64 * p : 0];
        const long long lab = labels[i];
        const float zl = lab >= 0 && lab < classes ? logit_at<true>(logits, (size_t)i * classes + lab) : __builtin_nanf("");
        float mx = -INFINITY, se = 0.f;
        auto at = [&](int k) {
            const uint32_t w = v[k >> 3][(k & 7) >> 1];
            return lane + 64 * (k >> 3) < pieces ? ((k & 1) ? bhi(w) : blo(w)) : -INFINITY;
        };
#pragma unroll
        for (int k = 0; k < 16; ++k) mx = fmaxf(mx, at(k));
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
#pragma unroll
        for (int k = 0; k < 16; ++k) se += lane + 64 * (k >> 3) < pieces ? __expf(at(k) - mx) : 0.f;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) se += __shfl_xor(se, o);
        if (lane == 0) __hip_atomic_store(losses + i, (mx + __logf(se)) - zl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) last = __hip_atomic_fetch_add(done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
    __syncthreads();
    if (!last) return;
    __threadfence();
    float sum[4] = {0.f, 0.f, 0.f, 0.f};                         // four losses in flight per lane
    for (int k = threadIdx.x; k < N; k += 4 * 256) {
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = k + 256 * u < N ? __hip_atomic_load(losses + k + 256 * u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.f;
#pragma unroll
        for (int u = 0; u < 4; ++u) sum[u] += v[u];
    }
    sum[0] = (sum[0] + sum[1]) + (sum[2] + sum[3]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum[0] += __shfl_xor(sum[0], o);
    if (lane == 0) part[wv] = sum[0];
    __syncthreads();
    if (threadIdx.x == 0) {
        out[0] = ((part[0] + part[1]) + (part[2] + part[3])) / (float)N;
        __hip_atomic_store(done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Whether launch_softmax_ce takes scratch, and how much: the counter, then the images' losses.
size_t softmax_ce_scratch_bytes(int N, int classes, int bf16) {
    return bf16 && classes % 8 == 0 && classes <= 1024 && N > 32 && N <= kLossImages ? 256 + (size_t)N * 4 : 0;
}

// scratch: softmax_ce_scratch_bytes of it, its first four bytes zero, one launch at a time; or null: one workgroup.
hipError_t launch_softmax_ce(const void *logits, const void *labels, int N, int classes, int bf16, float *out, void *scratch,
                             hipStream_t stream) {
    if (!logits || !labels || !out || N <= 0 || classes <= 0) return hipErrorInvalidValue;
    if (scratch && softmax_ce_scratch_bytes(N, classes, bf16) && !((uintptr_t)logits & 15)) {
        softmax_ce_wide_kernel<<<dim3((N + 3) / 4), dim3(256), 0, stream>>>(logits, static_cast<const long long *>(labels), N, classes, out,
                                                                           reinterpret_cast<float *>(static_cast<unsigned char *>(scratch) + 256),
                                                                           static_cast<unsigned *>(scratch));
        return hipGetLastError();
    }
    const auto *lab = static_cast<const long long *>(labels);
    auto run = [&](auto kernel) { kernel<<<dim3(1), dim3(1024), 0, stream>>>(logits, lab, N, classes, out); };
    const bool held = classes > 256 && classes <= 1024;
    if (bf16 && classes % 8 == 0 && classes <= 1024 && !((uintptr_t)logits & 15)) run(softmax_ce_kernel<true, PIECES>);
    else if (bf16) held ? run(softmax_ce_kernel<true, ELEMENTS>) : run(softmax_ce_kernel<true, REREAD>);
    else held ? run(softmax_ce_kernel<false, ELEMENTS>) : run(softmax_ce_kernel<false, REREAD>);
    return hipGetLastError();
}

}  // namespace delta
