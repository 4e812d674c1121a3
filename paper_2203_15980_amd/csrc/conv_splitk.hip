// Convolutions and linear layers that cannot fill the chip, for gfx950:
// y = act(scale_k * conv(x, w) + shift_k (+ res)) (* [mask > 0]), bf16 or fp32.
//
// DELTA's Recompute action (Sec. 3, Table 1) on a few images, one short sequence or a late stage's 7 x 7
// feature maps: the tiled kernels then run a handful of workgroups, each walking its whole reduction
// alone - about 0.4-0.8 us per 128 bytes of the reduction axis, whatever the rest of the chip does
// (3x3 256 -> 256 on 3 x 13 x 17 pixels: 12 workgroups, 28 us).  Such a launch is bound by latency, not
// by bandwidth or the matrix cores, so this kernel shortens the chain instead of feeding it better:
//  * small tiles, 32 pixels x 32 channels per workgroup, so that the same layer is 168 workgroups;
//  * the KW wavefronts of a workgroup share ONE tile and split its reduction: wavefront v takes the 128-byte
//    steps v, v + KW, ... of the (tap, input channel) axis, and the KW sums are added in the order of v
//    through LDS at the end (fixed order: the result is a fixed function of the inputs);
//  * each wavefront stages its own steps: eight lanes fetch one 128-byte row (32 pixel rows and 32 weight rows a
//    step, two steps in flight in registers), write them to LDS that only this wavefront uses and read its
//    32x32 MFMA operands back, so the main loop has no barrier.  Loading the operands straight from memory in
//    the MFMA's own layout (lane = row) needs no LDS at all, but its lanes' 16-byte pieces lie in 64 different
//    lines and the load unit then moves 13 bytes a cycle and CU: 2048 -> 512 at M = 784 20 us that way;
//  * padding taps, pixels past M, channels past Cout and steps past the end are offsets outside the buffer
//    descriptors, which load zeros, as in conv_igemm.hip;
//  * residual and mask are requested before the first step, scale and shift before the sums meet.
// Operands are re-read from the L1 / L2 by every tile that needs them (64 FLOP per byte loaded), which
// is what ends the kernel's range: see splitk_applies for where the lines lie and what both sides measured.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"

namespace delta {
namespace splitk {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

static constexpr int kOutOfRange = (int)0x80000000;     // outside every buffer descriptor used here
static constexpr int kTile = 32;                        // pixels and channels of a workgroup's tile
static constexpr int kPitch = kTile + 4;                // floats per pixel row of a wavefront's sums
static constexpr int kStepBytes = 128;                  // of the reduction axis, per step and row
static constexpr int kWaveLds = 2 * kTile * kStepBytes; // one step's rows; later the wavefront's sums
static_assert(kTile * kPitch * 4 <= kWaveLds, "the sums reuse the staging rows");

__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

__device__ __forceinline__ void wave_lds_fence() {
    // LDS instructions of one wavefront execute in order; this only stops the compiler from moving
    // accesses across the point where lanes exchange data through LDS.
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One 16-byte piece of both operands -> MFMAs.
template <bool BF16>
__device__ __forceinline__ void mma(const u32x4 w, const u32x4 x, f32x16 &acc) {
    if constexpr (BF16) {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x), acc, 0, 0, 0);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(w[e]), __uint_as_float(x[e]), acc, 0, 0, 0);
    }
}

struct Divisors { Divisor pq, q, cs, s; };

// wR, wS, w_r0, w_s0, w_step of `a` are filled by the launcher for every form (see ConvArgs).
// AHEAD: steps in flight per wavefront.
template <bool BF16, int KW, int AHEAD>
__global__ __launch_bounds__(KW * 64) void conv_splitk_kernel(ConvArgs a, int tiles_m, int tiles_n, int pixels_first,
                                                              Divisors inv) {
    constexpr int ES = BF16 ? 2 : 4;
    __shared__ __align__(16) unsigned char smem[KW * kWaveLds];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    // contiguous runs of tiles per XCD (blockIdx % 8); the axis that walks fastest is the one whose operand is
    // smaller, so that an XCD reads its share of the larger one once
    unsigned logical;
    {
        const unsigned nb = gridDim.x, per = nb >> 3, rem = nb & 7u;
        const unsigned xcd = blockIdx.x & 7u, idx = blockIdx.x >> 3;
        logical = xcd < rem ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
    }
    const int tm = pixels_first ? (int)(logical % tiles_m) : (int)(logical / tiles_n);
    const int tn = pixels_first ? (int)(logical / tiles_m) : (int)(logical % tiles_n);
    const int m0 = tm * kTile, n0 = tn * kTile;

    // ---- epilogue operands of this thread: pixel m0 + tid / 8, channels n0 + 4 * (tid % 8) .. + 3
    const int PQ = a.P * a.Q;
    const int em = m0 + (tid >> 3), ec = n0 + 4 * (tid & 7);
    const bool finishes = tid < 256 && em < a.M && ec < a.Cout;
    size_t eoff = 0;
    u32x4 eres = {0u, 0u, 0u, 0u}, emask = {0u, 0u, 0u, 0u};
    if (finishes) {
        size_t pixel = (size_t)em;
        if (a.oy_s) {
            const int n = divide(em, inv.pq), pq = em - n * PQ;
            const int p = divide(pq, inv.q), q = pq - p * a.Q;
            pixel = ((size_t)n * a.OH + (p * a.oy_s + a.oy_a)) * a.OW + (q * a.oy_s + a.oy_b);
        }
        eoff = (pixel * a.Cout + ec) * ES;
        auto read4 = [&](const void *p) {
            const unsigned char *s = static_cast<const unsigned char *>(p) + eoff;
            if constexpr (BF16) {
                const u32x2 v = *reinterpret_cast<const u32x2 *>(s);
                return u32x4{v.x, v.y, 0u, 0u};
            } else {
                return *reinterpret_cast<const u32x4 *>(s);
            }
        };
        if (a.res) eres = read4(a.res);
        if (a.mask) emask = read4(a.mask);
    }

    // ---- the rows this lane fetches: pixels and channels lane / 8 + 8 i of the tile, 16-byte segment lane % 8
    const int lrow = lane >> 3, seg = lane & 7;
    const int cin_bytes = a.Cin * ES;
    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<void *>(a.x), 0, a.N * a.H * a.W * cin_bytes, 0x00020000);
    const int wrow = a.wR * a.wS * cin_bytes;
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.w), 0, a.Cout * wrow, 0x00020000);
    int xoff[4], woff[4];
    unsigned inside[4];            // bit r: row r of the pixel's window lies inside the image; bit 16 + s: column s
    const int taps = a.R * a.S;
    auto span = [](int first, int window, int image) {           // the window positions i with 0 <= first + i < image
        const int lo = first < 0 ? -first : 0, hi = image - first < window ? image - first : window;
        return hi > lo ? (1u << hi) - (1u << lo) : 0u;
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int m = m0 + 8 * i + lrow;
        const int n = divide(m, inv.pq), pq = m - n * PQ;
        const int p = divide(pq, inv.q), q = pq - p * a.Q;
        const int h0 = p * a.stride - a.pad, w0 = q * a.stride - a.pad;
        xoff[i] = ((n * a.H + h0) * a.W + w0) * cin_bytes + seg * 16;
        inside[i] = m < a.M ? span(h0, a.R, a.H) | span(w0, a.S, a.W) << 16 : 0u;
        const int k = n0 + 8 * i + lrow;
        woff[i] = k < a.Cout ? k * wrow + seg * 16 : kOutOfRange;       // adding a tap's offset leaves it out of range
    }
    // ---- this wavefront's steps wv, wv + KW, ...: step j is 128-byte piece j % cs_per_tap of tap j / cs_per_tap.
    // A step past the end sets the offsets' top bit: nothing in a step is conditional, so the compiler counts the loads in flight instead
    // of waiting for all of them
    const int cs_per_tap = cin_bytes / kStepBytes;
    const int mine = (taps * cs_per_tap - wv + KW - 1) / KW;
    int step = wv;
    u32x4 xb[AHEAD][4], wb[AHEAD][4];
    auto fetch = [&](u32x4 (&xd)[4], u32x4 (&wd)[4]) {
        const int tap = divide(step, inv.cs), cs = step - tap * cs_per_tap;
        const int r = divide(tap, inv.s), s = tap - r * a.S;
        const int past = (taps - 1 - tap) & kOutOfRange;
        const int xadd = (r * a.W + s) * cin_bytes + cs * kStepBytes;
        const int wadd = ((a.w_r0 + r * a.w_step) * a.wS + a.w_s0 + s * a.w_step) * cin_bytes + cs * kStepBytes;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool ok = (inside[i] >> (r & 15)) & (inside[i] >> (16 + (s & 15))) & 1u;
            xd[i] = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, (ok ? xoff[i] + xadd : kOutOfRange) | past, 0, 0);
            wd[i] = __builtin_amdgcn_raw_buffer_load_b128(wrsrc, (woff[i] + wadd) | past, 0, 0);
        }
        step += KW;
    };
    // staging rows: 32 of x, then 32 of w; segment s of row r lies in slot s ^ (r % 8), so that the 32 lanes that
    // read one segment of 32 rows spread over the banks
    unsigned char *stg = smem + wv * kWaveLds;
    unsigned char *put = stg + lrow * kStepBytes + ((seg ^ lrow) << 4);        // rows lrow + 8 i: the same swizzle
    const unsigned char *get = stg + l32 * kStepBytes;
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) fetch(xb[u], wb[u]);
    for (int t = 0; t < mine; t += AHEAD) {                      // a last partial round runs on zeros
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            wave_lds_fence();                                    // the reads of the step before are done
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                *reinterpret_cast<u32x4 *>(put + i * (8 * kStepBytes)) = xb[u][i];
                *reinterpret_cast<u32x4 *>(put + (kTile + 8 * i) * kStepBytes) = wb[u][i];
            }
            fetch(xb[u], wb[u]);
            wave_lds_fence();
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int slot = ((2 * j + half) ^ (l32 & 7)) << 4;
                const u32x4 xf = *reinterpret_cast<const u32x4 *>(get + slot);
                const u32x4 wf = *reinterpret_cast<const u32x4 *>(get + kTile * kStepBytes + slot);
                mma<BF16>(wf, xf, acc);
            }
        }
    }
    // acc: pixel l % 32, channels 8 rb + 4 (l / 32) + e in register 4 rb + e
    wave_lds_fence();
    float *part = reinterpret_cast<float *>(stg);
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) {
        const f32x4 v = {acc[4 * rb], acc[4 * rb + 1], acc[4 * rb + 2], acc[4 * rb + 3]};
        *reinterpret_cast<f32x4 *>(part + l32 * kPitch + 8 * rb + 4 * half) = v;
    }
    f32x4 esc = {0.f, 0.f, 0.f, 0.f}, esh = {0.f, 0.f, 0.f, 0.f};
    if (finishes) {                                              // only now: two workgroups of 8 wavefronts fit a CU with 128 registers
        esc = *reinterpret_cast<const f32x4 *>(a.scale + ec);
        esh = *reinterpret_cast<const f32x4 *>(a.shift + ec);
    }
    __syncthreads();
    if (!finishes) return;
    const unsigned char *sum0 = smem + ((tid >> 3) * kPitch + 4 * (tid & 7)) * 4;
    f32x4 v = *reinterpret_cast<const f32x4 *>(sum0);
#pragma unroll
    for (int k = 1; k < KW; ++k) v += *reinterpret_cast<const f32x4 *>(sum0 + k * kWaveLds);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = v[e] * esc[e] + esh[e];
    if (a.res) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            v[e] += __uint_as_float(!BF16 ? eres[e] : (e & 1) ? eres[e >> 1] & 0xFFFF0000u : eres[e >> 1] << 16);
    }
    if (a.relu == 1) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = v[e] < 0.f ? 0.f : v[e];      // NaN stays NaN
    } else if (a.relu == 2) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = gelu_erf(v[e]);
    }
    unsigned char *y = static_cast<unsigned char *>(a.y) + eoff;
    if constexpr (BF16) {
        u32x2 o = {pack2(v[0], v[1]), pack2(v[2], v[3])};
        if (a.mask) o = u32x2{keep_where_positive_bf16(o.x, emask[0]), keep_where_positive_bf16(o.y, emask[1])};
        *reinterpret_cast<u32x2 *>(y) = o;
    } else {
        u32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            o[e] = __float_as_uint(v[e]);
            if (a.mask) o[e] = keep_where_positive_f32(o[e], emask[e]);
        }
        *reinterpret_cast<u32x4 *>(y) = o;
    }
}

template <bool BF16, int KW, int AHEAD>
hipError_t launch(const ConvArgs &a, hipStream_t stream) {
    const int tiles_m = (a.M + kTile - 1) / kTile, tiles_n = (a.Cout + kTile - 1) / kTile;
    const long long xbytes = (long long)a.N * a.H * a.W * a.Cin, wbytes = (long long)a.Cout * a.R * a.S * a.Cin;
    conv_splitk_kernel<BF16, KW, AHEAD><<<dim3((unsigned)tiles_m * (unsigned)tiles_n), dim3(KW * 64), 0, stream>>>(
        a, tiles_m, tiles_n, wbytes > xbytes,
        Divisors{make_divisor(a.P * a.Q), make_divisor(a.Q), make_divisor(a.Cin * (BF16 ? 2 : 4) / kStepBytes), make_divisor(a.S)});
    return hipGetLastError();
}

long long tiles_of(const ConvArgs &a) {
    return (((long long)a.M + kTile - 1) / kTile) * ((a.Cout + kTile - 1) / kTile);
}

}  // namespace splitk

bool conv_splitk_applies(const ConvArgs &a) {
    const long long es = a.bf16 ? 2 : 4;
    if (a.R > 8 || a.S > 8) return false;                        // a bit per window row and column
    if (a.bf16 && a.R == 3 && a.Cin == 64 && a.Cout == 64) return false;   // the block kernel's middle layer: its bits
    // 32-bit offsets from the tensors' own starts
    if ((long long)a.N * a.H * a.W * a.Cin * es > 0x7FFFFFFFLL) return false;
    const long long steps = (long long)a.R * a.S * a.Cin * es / splitk::kStepBytes;
    // Where the line lies.  A tiled kernel that does not fill the chip takes about 4.5 + 0.55 us per 128-byte step of
    // the reduction however small the output; this one about 4.5 us + (3 + 0.37 steps) ns per tile.  Measured (us, tiled
    // kernel | this one; the number of 32 x 32 tiles in brackets):
    //   3x3 256 -> 256 (36 steps)  M = 784 [200] 24.8 | 7.5   1568 [392] 24.9 | 12   3136 [784] 24.9 | 20   6272 [1568] 25.1 | 32
    //   2048 -> 512 (32 steps)     M = 784 [400] 20.5 | 10    1568 [784] 20.7 | 17   3136 [1568] 21.0 | 26
    //   3072 -> 768 (48 steps)     M = 196 [168] 27.9 | 8.4   784 [600] 28.4 | 18    1568 [1176] 28.6 | 30
    //   768 -> 768 (12 steps)      M = 196 [168] 10.9 | 6.0   784 [600] 11.1 | 10.6  1568 [1176] 11.2 | 15
    //   256 -> 1024 (4 steps)      M = 196 [224] 8.6 | 4.9    656 [656] 8.6 | 6.6    1000 [1000] 8.7 | 7.6    1568 [1568] 8.9 | 11
    //   448 -> 512 (7 steps)       M = 640 [320] 11 | 5.7     1280 [640] 11 | 6.8
    //   512 -> 512 (8 steps)       M = 960 [480] 9.7 | 7.5    1040 [528] 9.8 | 9.9 (eight wavefronts to a tile: a second round)
    //   fp32 3x3 64 -> 64 (18)     M = 3136 [196] 27 | 8.0    6272 [392] 27 | 14     12544 [784] 27 | 23
    //   fp32 256 -> 64 (8)         M = 3136 [196] 15 | 7.0    6272 [392] 15 | 10     12544 [784] 15 | 18
    // bf16 layers of three to seven steps have the tiled convolution kernel on the other side; from eight on the GEMM.
    const long long line = steps >= 24 || (a.bf16 && steps >= 3 && steps < 8) ? 1024 : a.bf16 && steps == 8 ? 512 : 640;
    return splitk::tiles_of(a) <= line;
}

const char *conv_splitk_kernel_name(const ConvArgs &a) {
    return a.bf16 ? "conv_splitk bf16 32x32 (reduction split over the workgroup's wavefronts)"
                  : "conv_splitk f32 32x32 (reduction split over the workgroup's wavefronts)";
}

hipError_t launch_conv_splitk(const ConvArgs &a_in, hipStream_t stream) {
    if ((a_in.oy_s ? conv_scatter_check(a_in) : conv_check(a_in)) || !conv_splitk_applies(a_in)) return hipErrorInvalidValue;
    ConvArgs a = a_in;
    if (!a.oy_s) { a.wR = a.R; a.wS = a.S; a.w_r0 = a.w_s0 = 0; a.w_step = 1; }
    const long long steps = (long long)a.R * a.S * a.Cin * (a.bf16 ? 2 : 4) / splitk::kStepBytes;
    if (steps >= 8) return a.bf16 ? splitk::launch<true, 8, 2>(a, stream) : splitk::launch<false, 8, 2>(a, stream);
    return a.bf16 ? splitk::launch<true, 4, 2>(a, stream) : splitk::launch<false, 4, 2>(a, stream);
}

}  // namespace delta
