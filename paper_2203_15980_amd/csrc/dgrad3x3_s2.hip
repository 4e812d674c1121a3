// Data gradient of a 3x3, stride 2, padding 1 layer (bf16) in one launch, for gfx950.
//
// Input pixel (2i + a, 2j + b) receives from the taps of its parity class alone: 1, 2, 2 and 4 of the nine, at gradient
// pixels (i, j) .. (i + 1, j + 1).  Four launches, one per class, read the gradient four times and re-read every output line
// (a class owns every other pixel of a row); the work itself is bound by the lines of gx and of the mask, 2 x N H W C.
// So one workgroup makes all four classes of 64 gradient pixels x 128 channels:
//  - its 4 wavefronts take 32 channels each and hold 4 classes x 64 pixels x 32 channels in 128 accumulator registers;
//  - pixels are numbered through the whole batch, so a tile's four neighbourhoods are one contiguous run of 65 + Q
//    gradient rows, staged once per 64 of the K channels in two buffers; a neighbour beyond the image is a row of zeros in LDS;
//  - the nine taps are nine steps, ordered by the neighbour they read (4, 2, 2, 1): a step needs new weights only, 32 rows
//    that are the wavefront's own, in a ring of three slots filled two steps ahead by direct loads.  Nothing is
//    waited for with a barrier but the gradient rows, once per nine steps;
//  - D[channel][pixel], turned through LDS into whole 256-byte lines of channels for the mask and the store.
// 74 KB of LDS up to Q = 31 and 256 registers leave two workgroups on a CU: one stores while the other multiplies.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"

namespace delta {
namespace dg3 {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

struct Args {
    const unsigned char *g, *w, *res, *mask;    // gy [M,K]; weights [C,3,3,K], taps flipped; [N,H,W,C] or nullptr
    unsigned char *out;                         // [N,H,W,C]
    int M, K, C, H, W, P, Q;
    int rows;                                   // gradient rows staged per chunk: 65 + Q rounded up to 32
    int ctiles;                                 // C / 128
    Divisor pq, q;                              // P Q, Q
};

static constexpr int kTile = 64, kSlot = 4096, kRing = 4 * 3 * kSlot, kMaxLoads = 7;
static constexpr int kMaxQ = kMaxLoads * 32 - kTile - 1;

// Step t: the neighbour it reads (bit 1: the row below, bit 0: the column to the right), the class it adds to (2 a + b)
// and its tap in the flipped weights.
__host__ __device__ constexpr int neighbour(int t) { return t < 4 ? 0 : t < 6 ? 1 : t < 8 ? 2 : 3; }
__host__ __device__ constexpr int class_of(int t) { constexpr int c[9] = {0, 1, 2, 3, 1, 3, 2, 3, 3}; return c[t]; }
__host__ __device__ constexpr int tap_of(int t) { constexpr int f[9] = {4, 3, 1, 0, 5, 2, 7, 6, 8}; return f[t]; }

__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

__global__ __launch_bounds__(256, 2) void dgrad3x3_s2_kernel(Args a) {
    extern __shared__ __align__(128) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    // each XCD (blockIdx % 8) takes a contiguous run of tiles: the channel tiles of a pixel tile and the rows neighbouring
    // tiles share are fetched into one L2
    unsigned blk;
    {
        const unsigned nb = gridDim.x, per = nb >> 3, rem = nb & 7u, xcd = blockIdx.x & 7u, idx = blockIdx.x >> 3;
        blk = xcd < rem ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
    }
    const int ct = (int)(blk % (unsigned)a.ctiles), m0 = (int)(blk / (unsigned)a.ctiles) * kTile;
    const int nloads = a.rows >> 5, gbytes = (a.rows + 1) * 128, nchunks = a.K >> 6;
    typedef __attribute__((address_space(3))) unsigned char *lptr_t;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)smem;

    // ---- direct loads: one fills 8 rows of 128 bytes; slot s of row r holds piece s ^ (r % 8)
    const uint32_t seg = (uint32_t)(((lane & 7) ^ (lane >> 3)) * 16), pitch = (uint32_t)a.K * 2u;
    const unsigned char *g0 = a.g + (size_t)m0 * pitch;
    const int last = a.M - 1 - m0;
    auto fetch_rows = [&](int chunk, int i) {                    // rows 32 i + 8 wv + lane / 8 of the chunk
        int row = 32 * i + 8 * wv + (lane >> 3);
        const uint32_t dst = lds0 + (uint32_t)(kRing + (chunk & 1) * gbytes + (32 * i + 8 * wv) * 128);
        row = row < last ? row : last;                           // past the last pixel: that pixel, never looked at
        const uint32_t off = (uint32_t)row * pitch + (uint32_t)chunk * 128u + seg;
        load_lds_b128(g0, off, dst);
    };
    const uint32_t wbase = (uint32_t)(ct * 128 + wv * 32 + (lane >> 3)) * 9u * pitch + seg;
    auto fetch_taps = [&](int chunk, int tap, int slot) {        // this wavefront's 32 channels of one tap
        const uint32_t dst = lds0 + (uint32_t)((wv * 3 + slot) * kSlot);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t off = wbase + (uint32_t)(i * 72 + tap) * pitch + (uint32_t)chunk * 128u;
            load_lds_b128(a.w, off, dst + i * 1024);
        }
    };
    // direct loads complete in order: all but the newest `newer` are done
    auto wait_loads = [&](int newer) {
        if (newer == 10) asm volatile("s_waitcnt vmcnt(10)" ::: "memory");
        else if (newer == 9) asm volatile("s_waitcnt vmcnt(9)" ::: "memory");
        else if (newer == 8) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        else if (newer == 4) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };

    // ---- where this lane's pixels (m0 + 32 u + lane % 32) and their neighbours lie in a staged chunk: the byte of piece 0;
    // piece 2 k lies at that byte ^ 32 k
    uint32_t at[4][2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int r = 32 * u + l32, m = m0 + r, rest = m - divide(m, a.pq) * (a.P * a.Q), p = divide(rest, a.q), q = rest - p * a.Q;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const bool in = (!(d & 1) | (q + 1 < a.Q)) & (!(d & 2) | (p + 1 < a.P));
            const int row = in ? r + (d & 1) + (d >> 1) * a.Q : a.rows;          // the last row of a buffer holds zeros
            at[d][u] = (uint32_t)(kRing + row * 128 + ((half ^ (row & 7)) << 4));
        }
    }
    const uint32_t wat = (uint32_t)(wv * 3 * kSlot + l32 * 128 + ((half ^ (l32 & 7)) << 4));

    f32x16 acc[4][2];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[c][u][e] = 0.f;

    if (tid < 16) {
        const u32x4 zero = {0u, 0u, 0u, 0u};
        *reinterpret_cast<u32x4 *>(smem + kRing + (tid >> 3) * gbytes + a.rows * 128 + (tid & 7) * 16) = zero;
    }
    for (int i = 0; i < nloads; ++i) fetch_rows(0, i);
    fetch_taps(0, tap_of(0), 0);
    fetch_taps(0, tap_of(1), 1);
    wait_loads(8);
    for (int chunk = 0; chunk < nchunks; ++chunk) {
        // every wavefront's rows of this chunk have landed (each has waited for its own) and nobody reads the other buffer
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        const bool more = chunk + 1 < nchunks;
        const int ahead = more ? nloads : 0;
        const uint32_t gb = (uint32_t)((chunk & 1) * gbytes);
        bf16x8 b[2][4];
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the slot about to be filled has been read
            if (t < ahead) fetch_rows(chunk + 1, t);
            if (t < 7) fetch_taps(chunk, tap_of(t + 2), (t + 2) % 3);
            else if (more) fetch_taps(chunk + 1, tap_of(t - 7), (t + 2) % 3);
            // newer than this step's weights: those of the two steps that follow and the rows requested with them
            wait_loads(t < 7 || more ? 8 + (t < ahead) + (t > 0 && t - 1 < ahead) : t == 7 ? 4 : 0);
            if (t == 0 || neighbour(t) != neighbour(t - 1)) {
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        b[u][k] = *reinterpret_cast<const bf16x8 *>(smem + ((at[neighbour(t)][u] ^ (uint32_t)(32 * k)) + gb));
            }
            bf16x8 w[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) w[k] = *reinterpret_cast<const bf16x8 *>(smem + ((wat ^ (uint32_t)(32 * k)) + (t % 3) * kSlot));
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    acc[class_of(t)][u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[k], b[u][k], acc[class_of(t)][u], 0, 0, 0);
        }
    }
    // ---- a thread's 16 output pieces: piece tid % 16 of pixels tid / 16 + 16 v, in each class
    const int piece = tid & 15;
    size_t off[4];
    bool live[4][4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int m = m0 + 16 * v + (tid >> 4);
        const int n = divide(m, a.pq), rest = m - n * (a.P * a.Q), p = divide(rest, a.q), q = rest - p * a.Q;
        off[v] = (((size_t)n * a.H + 2 * p) * a.W + 2 * q) * a.C * 2 + (size_t)ct * 256 + piece * 16;
#pragma unroll
        for (int c = 0; c < 4; ++c) live[v][c] = (m < a.M) & (2 * p + (c >> 1) < a.H) & (2 * q + (c & 1) < a.W);
    }
    auto class_off = [&](int c) { return ((size_t)(c >> 1) * a.W + (c & 1)) * a.C * 2; };
    u32x4 mv[4][4];
    if (a.mask) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) mv[c][v] = *reinterpret_cast<const u32x4 *>(a.mask + (live[v][c] ? off[v] + class_off(c) : 0));
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");              // nobody reads operands any more
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int px = 32 * u + l32;
        size_t roff = 0;
        int h = 0, w = 0;
        bool in = false;
        if (a.res) {
            const int m = m0 + px, n = divide(m, a.pq), rest = m - n * (a.P * a.Q), p = divide(rest, a.q), q = rest - p * a.Q;
            h = 2 * p; w = 2 * q; in = m < a.M;
            roff = (((size_t)n * a.H + h) * a.W + w) * a.C * 2 + (size_t)ct * 256 + wv * 64 + half * 8;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j) {                        // channels 32 wv + 8 j + 4 half .. + 3
                float f[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) f[e] = acc[c][u][4 * j + e];
                if (a.res) {
                    u32x2 r = {0u, 0u};
                    if (in & (h + (c >> 1) < a.H) & (w + (c & 1) < a.W)) r = *reinterpret_cast<const u32x2 *>(a.res + roff + class_off(c) + j * 16);
                    f[0] += __uint_as_float(r.x << 16); f[1] += __uint_as_float(r.x & 0xFFFF0000u);
                    f[2] += __uint_as_float(r.y << 16); f[3] += __uint_as_float(r.y & 0xFFFF0000u);
                }
                const u32x2 o = {pack2(f[0], f[1]), pack2(f[2], f[3])};
                *reinterpret_cast<u32x2 *>(smem + (c * kTile + px) * 256 + (((4 * wv + j) ^ (px & 15)) << 4) + half * 8) = o;
            }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int px = 16 * v + (tid >> 4);
            u32x4 o = *reinterpret_cast<const u32x4 *>(smem + (c * kTile + px) * 256 + ((piece ^ (px & 15)) << 4));
            if (a.mask) {
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = keep_where_positive_bf16(o[e], mv[c][v][e]);
            }
            if (live[v][c]) *reinterpret_cast<u32x4 *>(a.out + off[v] + class_off(c)) = o;
        }
}

}  // namespace dg3

// `a`: the four classes' common arguments: x = gy [N,H=P,W=Q,Cin=K], w the flipped weights [Cout,3,3,Cin], res, mask and y
// [N,OH,OW,Cout].  One launch costs 10 us plus 18 us per 512 of K while its tiles do not fill the chip; four launches with
// their reductions split cost 21 to 25 us then, whatever K is, and lose from 40 tiles on.  56 x 56 x 128, 28 x 28 x 256 and 14 x 14 x 512, us for four
// launches -> one:  batch 1: 21 -> 13, 23 -> 18, 25 -> 28;  8: 44 -> 14, 29 -> 19, 26 -> 29 (28 tiles);
// 16: 45 -> 15, 56 -> 19, 33 -> 29 (52 tiles);  32: 52 -> 20, 59 -> 21, 73 -> 30;  128: 124 -> 62 (3.7 TB/s), 87 -> 53, 90 -> 46.
// From 32 output columns on the staged rows leave one workgroup to a CU, which is still the better side.  gx of 128 channels, gradient of 128 | 512
// with gx of 512: batch 1 of 64 x 64 44 -> 14 | 87 -> 30, of 318 x 318 53 -> 29 | 215 -> 193; batch 8 of 160 x 160 68 -> 52 | 396 -> 382;
// batch 64 of 64 x 64 76 -> 55 | 468 -> 475, batch 32 of 112 x 112 122 -> 87 | 716 -> 731 (even).
bool dgrad_s2_applies(const ConvArgs &a) {
    if (!a.bf16 || a.Cout % 128 || a.Cin % 64 || a.W > dg3::kMaxQ) return false;
    const long long tiles = ((long long)a.N * a.H * a.W + dg3::kTile - 1) / dg3::kTile * (a.Cout / 128);
    return a.Cin <= 384 || tiles >= 40;
}

hipError_t launch_dgrad_s2(const ConvArgs &a, hipStream_t stream) {
    if (!dgrad_s2_applies(a) || a.H != (a.OH - 1) / 2 + 1 || a.W != (a.OW - 1) / 2 + 1) return hipErrorInvalidValue;
    dg3::Args k;
    k.g = static_cast<const unsigned char *>(a.x); k.w = static_cast<const unsigned char *>(a.w);
    k.res = static_cast<const unsigned char *>(a.res); k.mask = static_cast<const unsigned char *>(a.mask);
    k.out = static_cast<unsigned char *>(a.y);
    k.M = a.N * a.H * a.W; k.K = a.Cin; k.C = a.Cout; k.H = a.OH; k.W = a.OW; k.P = a.H; k.Q = a.W;
    k.rows = (dg3::kTile + 1 + a.W + 31) / 32 * 32;
    k.ctiles = a.Cout / 128;
    k.pq = make_divisor((uint32_t)(a.H * a.W)); k.q = make_divisor((uint32_t)a.W);
    const long long blocks = ((long long)k.M + dg3::kTile - 1) / dg3::kTile * k.ctiles;
    if (blocks > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    const size_t lds = dg3::kRing + 2 * (size_t)(k.rows + 1) * 128;
    static const hipError_t big = hipFuncSetAttribute(reinterpret_cast<const void *>(dg3::dgrad3x3_s2_kernel),
                                                      hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (big != hipSuccess) return big;
    dg3::dgrad3x3_s2_kernel<<<dim3((unsigned)blocks), dim3(256), lds, stream>>>(k);
    return hipGetLastError();
}

}  // namespace delta
