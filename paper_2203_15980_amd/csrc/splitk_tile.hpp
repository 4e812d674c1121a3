// One 32 x 32 tile of a convolution with its reduction split over wavefronts: the body of conv_splitk.hip's kernel, and of
// small_backward.hip's, which runs it beside a weight gradient.  What bounds it and why it is built this way stands in conv_splitk.hip.
#pragma once
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

struct Divisors { Divisor pq, q, cs, s, tiles; };      // tiles: along the axis that walks fastest

// Contiguous runs of tiles per XCD (workgroup number % 8): the tile of workgroup `block` of `blocks`.
__device__ __forceinline__ unsigned xcd_run(unsigned block, unsigned blocks) {
    const unsigned per = blocks >> 3, rem = blocks & 7u, xcd = block & 7u, idx = block >> 3;
    return xcd < rem ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
}

// Tile `logical` of the output by KW wavefronts (thread `tid` of KW * 64, smem: KW * kWaveLds bytes of their own, factors: 256 more); a number
// past the last tile computes nothing.  The axis that walks fastest is the one whose operand is smaller, so that an XCD reads its share of the
// larger one once.  One barrier, which the whole workgroup has to reach.
// wR, wS, w_r0, w_s0, w_step of `a` are filled by the launcher for every form (see ConvArgs).
// AHEAD: steps in flight per wavefront.  SPREAD: `a` may ask for the spread form.
template <bool BF16, int KW, int AHEAD, bool SPREAD>
__device__ __forceinline__ void conv_tile(const ConvArgs &a, int tiles_m, int tiles_n, int pixels_first, const Divisors &inv,
                                          unsigned logical, int tid, unsigned char *smem, float *factors) {
    constexpr int ES = BF16 ? 2 : 4;
    const int lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int slow = divide((int)logical, inv.tiles), fast = (int)logical - slow * (pixels_first ? tiles_m : tiles_n);
    const int tm = pixels_first ? fast : slow, tn = pixels_first ? slow : fast;
    const int m0 = tm * kTile, n0 = tn * kTile;

    // scale, then shift of the tile's 32 channels: straight into LDS, where they need no register until the end
    if (wv == 0) {
        const int c = n0 + l32 < a.Cout ? n0 + l32 : a.Cout - 1;
        typedef __attribute__((address_space(3))) float *lptr_t;
        load_lds_b32((half ? a.shift : a.scale) + c, (uint32_t)(uintptr_t)(lptr_t)factors);
    }
    // ---- epilogue operands of this thread: pixel m0 + tid / 8, channels n0 + 4 * (tid % 8) .. + 3
    const int PQ = a.P * a.Q;
    const int em = m0 + (tid >> 3), ec = n0 + 4 * (tid & 7);
    const bool finishes = tid < 256 && em < a.M && ec < a.Cout;
    size_t eoff = 0;
    int erows = 1, ecols = 1;          // spread form: rows and columns of the pixel's block
    u32x4 eres = {0u, 0u, 0u, 0u}, emask = {0u, 0u, 0u, 0u};
    if (finishes) {
        size_t pixel = (size_t)em;
        if (a.oy_s) {
            const int n = divide(em, inv.pq), pq = em - n * PQ;
            const int p = divide(pq, inv.q), q = pq - p * a.Q;
            pixel = ((size_t)n * a.OH + (p * a.oy_s + a.oy_a)) * a.OW + (q * a.oy_s + a.oy_b);
            if (SPREAD && a.spread) {
                erows = a.OH - p * a.oy_s < a.oy_s ? a.OH - p * a.oy_s : a.oy_s;
                ecols = a.OW - q * a.oy_s < a.oy_s ? a.OW - q * a.oy_s : a.oy_s;
            }
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
    if (wv == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // the factors, long since
    __syncthreads();
    if (!finishes) return;
    const f32x4 esc = *reinterpret_cast<const f32x4 *>(factors + 4 * (tid & 7)), esh = *reinterpret_cast<const f32x4 *>(factors + 32 + 4 * (tid & 7));
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
    if (SPREAD && a.spread)
        for (int at = 1; at < erows * ecols; ++at) {
            const int dy = at / ecols, dx = at - dy * ecols;
            unsigned char *z = y + ((size_t)dy * a.OW + dx) * a.Cout * ES;
            if constexpr (BF16) *reinterpret_cast<u32x2 *>(z) = u32x2{0u, 0u};
            else *reinterpret_cast<u32x4 *>(z) = u32x4{0u, 0u, 0u, 0u};
        }
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

inline long long tiles_of(const ConvArgs &a) {
    return (((long long)a.M + kTile - 1) / kTile) * ((a.Cout + kTile - 1) / kTile);
}
inline bool weights_larger(const ConvArgs &a) { return (long long)a.Cout * a.R * a.S * a.Cin > (long long)a.N * a.H * a.W * a.Cin; }
inline Divisors divisors_of(const ConvArgs &a) {
    return Divisors{make_divisor(a.P * a.Q), make_divisor(a.Q), make_divisor(a.Cin * (a.bf16 ? 2 : 4) / kStepBytes), make_divisor(a.S),
                    make_divisor(((weights_larger(a) ? a.M : a.Cout) + kTile - 1) / kTile)};
}

}  // namespace splitk
}  // namespace delta
