// Weight gradient of the 3x3 layers (stride 1 and stride 2, padding 1) for gfx950, bf16:
//   gw[k,r,s,c] = scale_k * sum_m gpre[m,k] * x[pixel of m shifted by (r,s)][c]
// part of the backward pass whose accesses to stored activations DELTA's planner follows (Sec. 3, Assumptions 1-3).
//
// The reduction index is the output pixel and both operands are stored pixel-major, so tiles are staged in LDS
// as they lie in memory (pixel rows x 64 channels) and turned into MFMA operands by gfx950's transposing LDS read
// (ds_read_b64_tr_b16; see wgrad1x1.hip for the lane layout).
//
// One list of padded pixels.  The images of the batch are stacked into one list of rows with ONE zero row
// after each image, and every row gets ONE zero pixel at its end: the zero at the end of row p is also the pixel left
// of row p + 1, the zero row below image n also the row above image n + 1.  In that list a tap is a constant offset,
// no operand is masked, and a chunk is any run of rows - several 7 x 7 images or part of a 56 x 56 one.  For a stride of
// 2 the list runs over the OUTPUT's pixels and x is staged as its four parity classes (input pixel (2i + a, 2j + b) is
// pixel (i, j) of class (a, b)): tap r reads class a = 1 at row p - 1 (r = 0), a = 0 at row p (r = 1), a = 1 at row p (r = 2),
// likewise for s, so the nine taps are again constant offsets and the layer takes nine taps' work, once.
//
// A workgroup owns 64 x 64 (k, c) and all nine taps: 12 wavefronts, three on every SIMD, as 3 (window row r) x 2
// (32 channels of x) x 2 (halves of a chunk's 16-pixel steps).  A wavefront's three taps of one window row read x at three
// neighbouring offsets, so it reads twelve pixels once and takes the taps out of them by shifting registers (stride 2:
// nine of one class for s = 0 and 2, eight of another for s = 1): 1.2 (1.5) transposing reads per MFMA where a wavefront
// per tap and 64 x 64 tile took 2.0, on 9 wavefronts that left three of four SIMDs a third idle.
// Chunks move through two LDS buffers with one barrier each: while chunk t is multiplied, chunk t + 1 travels in registers.
// The two wavefronts of a pair are added through LDS, the workgroups' sums go to a partial buffer in accumulator
// order and wgrad3x3_reduce_kernel adds them in the order of the splits.  No atomics: a fixed function of the inputs.
// Alone, with the reduction and the launches (a wavefront per tap, chunks of one image, strided layers as four launches | this):
// 512 -> 512 on 256 x 7 x 7 143 | 83 us, 128 -> 128 on 128 x 28 x 28 59 | 54; stride 2, 128 -> 128 on 128 x 56 x 56 121 | 64, 512 -> 512 on
// 128 x 14 x 14 147 | 67.  The kernel alone does 740 - 860 TFLOP/s of the layer's own work at stride 1, 600 at stride 2 (kernel trace),
// with the matrix cores busy 0.44 - 0.57 and 0.35 of the time; what is left is their idle time at a
// chunk's barrier and the padding pixels (1.04 of the work at 56 x 56, 1.31 at 7 x 7).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"

namespace delta {
namespace wg3 {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

static constexpr int kOutOfRange = (int)0x80000000;     // outside every buffer descriptor used here
static constexpr int kThreads = 768, kPairs = 6;        // wavefronts that own sums: 3 window rows x 2 channel halves
static constexpr int kRow = 128;                        // bytes of one pixel's 64 channels
static constexpr int kQuads = kPairs * 3 * 2 * 4 * 64;  // f32x4 of one workgroup's sums
static constexpr int kMaxRows = 640;                    // staged pixel rows of one buffer: two fill the 160 KB
template <int STRIDE> struct Pieces {                   // staged 16-byte pieces per thread, gradient and x; pixels of a chunk
    static constexpr int G = STRIDE == 1 ? 3 : 1, X = STRIDE == 1 ? 4 : 5, kPixels = STRIDE == 1 ? 256 : 64;
};

struct Args {
    const void *x, *g;              // [N,H,W,C], [N,P,Q,K]
    float *partial;                 // [nsplit][tiles][kPairs][3 taps][2][4][64 lanes] f32x4
    int N, H, W, C, K, P, Q;
    int pitch;                      // Q + 1: pixels of a list row
    int rows, RH, QN, XN;           // list rows in all, of a chunk; list pixels of a chunk (a multiple of 32); staged rows of x (of a class)
    int per, nsplit;                // list rows of a split: split s takes rows s * per .. and walks them in chunks
    Divisor image;                  // P + 1: list rows of an image
};

template <int STRIDE>
__global__ __launch_bounds__(kThreads) void wgrad3x3_kernel(Args a) {
    constexpr int GP = Pieces<STRIDE>::G, XP = Pieces<STRIDE>::X, PLANES = STRIDE == 1 ? 1 : 4;
    extern __shared__ __align__(16) unsigned char smem[];        // two buffers: [QN] gradient rows, [PLANES][XN] rows of x
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = wv % 3, ch = (wv / 3) & 1, qs = wv / kPairs;
    const int ktiles = a.K / 64, kt = blockIdx.y % ktiles, ct = blockIdx.y / ktiles;
    const int pitch = a.pitch, buffer = (a.QN + PLANES * a.XN) * kRow;

    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.x), 0, a.N * a.H * a.W * a.C * 2, 0x00020000);
    const __amdgpu_buffer_rsrc_t grsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.g), 0, a.N * a.P * a.Q * a.K * 2, 0x00020000);

    // ---- what this thread stages: piece i is segment tid % 8 of LDS row tid / 8 + 96 i.  Per piece, relative to the chunk:
    // list row (high half) and column (low half; past the image: always zero) in one register, since 12 wavefronts leave a
    // lane 168 of them and the sums take 96
    const int seg = tid & 7;
    int gat[GP], xat[XP];
#pragma unroll
    for (int i = 0; i < GP; ++i) {
        const int q = (tid >> 3) + 96 * i, row = q / pitch;
        gat[i] = row * 0x10000 + (q < a.RH * pitch ? q - row * pitch : 0xFFFF);
    }
#pragma unroll
    for (int i = 0; i < XP; ++i) {
        const int f = (tid >> 3) + 96 * i, plane = f / a.XN, j = f - plane * a.XN;     // row j of a class: list pixel j - pitch - 1
        const int l = j + pitch - 1;                                                   // plus two rows, so that it is not negative
        int row = l / pitch - 2, col = l - (l / pitch) * pitch;
        if (STRIDE == 2) { row = 2 * row + (plane >> 1); col = 2 * col + (plane & 1); }
        xat[i] = row * 0x10000 + (f < PLANES * a.XN ? col : 0xFFFF);
    }
    u32x4 gb[GP], xb[XP];
    const int rows = a.rows, RH = a.RH, H = a.H, W = a.W, P = a.P, Q = a.Q, K2 = a.K * 2, C2 = a.C * 2;
    const uint32_t mul = a.image.mul, shift = a.image.shift;     // P + 1 >= 2: never the identity
    const int gbase = kt * 128 + seg * 16, xbase = ct * 128 + seg * 16;
    const int first = blockIdx.x * a.per, end = first + a.per < rows ? first + a.per : rows;
    auto fetch = [&](int R0) {                                   // rows from R0; gradient rows past the split's end: zeros.  No branches: see conv_igemm.hip
#pragma unroll
        for (int i = 0; i < GP; ++i) {
            const int R = R0 + (gat[i] >> 16), col = gat[i] & 0xFFFF;
            const int n = (int)(__umulhi((uint32_t)R, mul) >> shift), p = R - n * (P + 1);
            const bool ok = (R < end) & (p < P) & (col < Q);
            const int off = ((n * P + p) * Q + col) * K2 + gbase;
            gb[i] = __builtin_amdgcn_raw_buffer_load_b128(grsrc, ok ? off : kOutOfRange, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < XP; ++i) {
            const int row = xat[i] >> 16, col = xat[i] & 0xFFFF, R = R0 + (STRIDE == 2 ? row >> 1 : row);
            const int n = (int)(__umulhi((uint32_t)R, mul) >> shift), p = R - n * (P + 1);
            const int h = STRIDE == 2 ? 2 * p + (row & 1) : p;
            // p == P is the zero row: 2 P and 2 P + 1 lie past the image as well, a stride of 1 has H == P
            const bool ok = ((uint32_t)R < (uint32_t)rows) & (h < H) & (col < W);
            const int off = ((n * H + h) * W + col) * C2 + xbase;
            xb[i] = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, ok ? off : kOutOfRange, 0, 0);
        }
    };
    // The two 64-byte groups of a row are swapped by bit 1 of the row's number, so that the four consecutive rows a
    // transposing read touches at one column lie in four different quarters of the banks.  96 rows on, the bit is the same.
    const int put = (tid >> 3) * kRow + ((((seg >> 2) ^ (tid >> 4)) & 1) << 6) + (seg & 3) * 16;
    auto stage = [&](int buf) {
        unsigned char *gs = smem + buf * buffer, *xs = gs + a.QN * kRow;
#pragma unroll
        for (int i = 0; i < GP; ++i)
            if ((tid >> 3) + 96 * i < a.QN) *reinterpret_cast<u32x4 *>(gs + put + i * (96 * kRow)) = gb[i];
#pragma unroll
        for (int i = 0; i < XP; ++i)
            if ((tid >> 3) + 96 * i < PLANES * a.XN) *reinterpret_cast<u32x4 *>(xs + put + i * (96 * kRow)) = xb[i];
    };

    // ---- transposing reads: a lane supplies row 8 (lane / 32) + (lane % 16) / 4 (+ 4) of a 16-pixel step and channels
    // 16 ((lane / 16) % 2) + 4 (lane % 4) .. + 3; it receives channel lane % 32 of its 32, pixels 8 (lane / 32) .. + 7
    const int srow = 8 * (lane >> 5) + ((lane & 15) >> 2), scol = 32 * ((lane >> 4) & 1) + 8 * (lane & 3);
    typedef s16x4 __attribute__((address_space(3))) * lds_ptr;
    auto tr_read = [&](const unsigned char *p) { return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p))); };
    int goff[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) goff[t] = srow * kRow + (((t ^ (srow >> 1)) & 1) << 6) + scol;
    // rows of x: stride 1, taps s = 0..2 from offset r * pitch; stride 2, class (r != 1, 1) at the offset of s = 0 and class
    // (r != 1, 0) at that of s = 1
    const int xo = STRIDE == 1 ? r * pitch + srow : (r == 1 ? 1 : 3) * a.XN + (r ? pitch : 0) + srow;
    const int xo1 = (r == 1 ? 0 : 2) * a.XN + (r ? pitch : 0) + srow + 1;
    const int xoff = xo * kRow + (((ch ^ (xo >> 1)) & 1) << 6) + scol, xoff1 = xo1 * kRow + (((ch ^ (xo1 >> 1)) & 1) << 6) + scol;

    f32x16 acc[3][2];
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[s][t][e] = 0.f;

    int R0 = first;
    fetch(R0);
    stage(0);
    fetch(R0 + RH);
    for (int buf = 0; R0 < end; R0 += RH, buf ^= 1) {
        __syncthreads();                                         // buffer buf is written, the other one no longer read
        stage(buf ^ 1);
        fetch(R0 + 2 * RH);
        const unsigned char *gs = smem + buf * buffer, *xs = gs + a.QN * kRow;
        const int pixels = end - R0 < RH ? (end - R0) * pitch : a.QN;            // the split's last chunk may be shorter
        for (int q0 = 16 * qs; q0 < pixels; q0 += 32) {
            u32x4 gf[2], xf[3];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const u32x2 lo = tr_read(gs + q0 * kRow + goff[t]), hi = tr_read(gs + (q0 + 4) * kRow + goff[t]);
                gf[t] = u32x4{lo.x, lo.y, hi.x, hi.y};
            }
            const u32x2 d0 = tr_read(xs + q0 * kRow + xoff), d1 = tr_read(xs + (q0 + 4) * kRow + xoff), d2 = tr_read(xs + (q0 + 8) * kRow + xoff);
            xf[0] = u32x4{d0.x, d0.y, d1.x, d1.y};
            const u32x4 one = {__builtin_amdgcn_alignbit(d0.y, d0.x, 16), __builtin_amdgcn_alignbit(d1.x, d0.y, 16),
                               __builtin_amdgcn_alignbit(d1.y, d1.x, 16), __builtin_amdgcn_alignbit(d2.x, d1.y, 16)};   // one pixel on
            if constexpr (STRIDE == 1) {
                xf[1] = one;
                xf[2] = u32x4{d0.y, d1.x, d1.y, d2.x};
            } else {
                const u32x2 e0 = tr_read(xs + q0 * kRow + xoff1), e1 = tr_read(xs + (q0 + 4) * kRow + xoff1);
                xf[1] = u32x4{e0.x, e0.y, e1.x, e1.y};
                xf[2] = one;
            }
#pragma unroll
            for (int s = 0; s < 3; ++s)
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    acc[s][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, gf[t]), __builtin_bit_cast(bf16x8, xf[s]),
                                                                        acc[s][t], 0, 0, 0);
        }
    }
    // ---- a pair's two sums meet in LDS, then leave in accumulator order
    __syncthreads();                                             // the staged chunks are dead
    f32x4 *red = reinterpret_cast<f32x4 *>(smem) + (size_t)(wv % kPairs) * (kQuads / kPairs) + lane;
    if (qs) {
#pragma unroll
        for (int i = 0; i < 24; ++i) {
            const f32x16 &v = acc[i / 8][(i / 4) & 1];
            red[i * 64] = f32x4{v[4 * (i & 3)], v[4 * (i & 3) + 1], v[4 * (i & 3) + 2], v[4 * (i & 3) + 3]};
        }
    }
    __syncthreads();
    if (qs) return;
    f32x4 *out = reinterpret_cast<f32x4 *>(a.partial) + ((size_t)blockIdx.x * gridDim.y + blockIdx.y) * kQuads + (size_t)wv * (kQuads / kPairs) + lane;
#pragma unroll
    for (int i = 0; i < 24; ++i) {
        const f32x16 &v = acc[i / 8][(i / 4) & 1];
        out[i * 64] = red[i * 64] + f32x4{v[4 * (i & 3)], v[4 * (i & 3) + 1], v[4 * (i & 3) + 2], v[4 * (i & 3) + 3]};
    }
}

// gw[k][r][s][c] = scale_k * sum over the splits of the partial sums.  64 consecutive f32x4 are shared by G wavefronts
// (wavefront g adds splits g, g + G, ..., four loads in flight), whose G sums are added in the order of g.
template <int G>
__global__ __launch_bounds__(512) void wgrad3x3_reduce_kernel(const float *partial, const float *scale, float *gw, int K, int C, int nsplit) {
    __shared__ f32x4 part[8][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, grp = wave % G;
    const int ktiles = K / 64;
    const size_t per_split = (size_t)ktiles * (C / 64) * kQuads;
    const size_t idx = ((size_t)blockIdx.x * (8 / G) + wave / G) * 64 + lane;
    const f32x4 *src = reinterpret_cast<const f32x4 *>(partial) + idx;
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    int sp = grp;
    for (; sp + 3 * G < nsplit; sp += 4 * G) {
        const f32x4 v0 = src[(size_t)sp * per_split], v1 = src[(size_t)(sp + G) * per_split];
        const f32x4 v2 = src[(size_t)(sp + 2 * G) * per_split], v3 = src[(size_t)(sp + 3 * G) * per_split];
        sum += v0; sum += v1; sum += v2; sum += v3;
    }
    for (; sp < nsplit; sp += G) sum += src[(size_t)sp * per_split];
    if constexpr (G > 1) {
        part[wave][lane] = sum;
        __syncthreads();
        if (grp != 0) return;
#pragma unroll
        for (int g = 1; g < G; ++g) sum += part[wave + g][lane];
    }
    // idx = (((tile * kPairs + pair) * 3 + s) * 2 + t) * 4 + e4) * 64 + lane; accumulator layout: column (c) lane % 32, rows (k)
    // 8 e4 + 4 (lane / 32) + e
    const int i = (int)(idx >> 6), e4 = i & 3, t = (i >> 2) & 1, s = (i >> 3) % 3, pair = (i / 24) % kPairs, tile = i / (24 * kPairs);
    const int r = pair % 3, c = (tile / ktiles) * 64 + (pair / 3) * 32 + (lane & 31);
    const int k0 = (tile % ktiles) * 64 + t * 32 + 8 * e4 + 4 * (lane >> 5);
#pragma unroll
    for (int e = 0; e < 4; ++e) gw[((size_t)(k0 + e) * 9 + r * 3 + s) * C + c] = sum[e] * scale[k0 + e];
}

// A workgroup's time per list pixel, and what one more split costs per tile: its 147 KB written and read back.
static constexpr double kPixelNs = 7.5, kSumsNs = 53.;

struct Plan { int rh, qn, xn, rows, per, nsplit, tiles; size_t lds; };

// nullptr and a filled plan, or the reason the kernel does not apply.  `a`: the forward layer's own geometry.
const char *plan_for(const ConvArgs &a, Plan &p) {
    if (!a.bf16 || a.R != 3 || a.S != 3 || a.pad != 1 || (a.stride != 1 && a.stride != 2)) return "weight gradient: 3x3, stride 1 or 2, padding 1, bf16";
    if (a.Cin % 64 || a.Cout % 64) return "weight gradient: channel counts must be multiples of 64";
    const int P = (a.H - 1) / a.stride + 1, Q = (a.W - 1) / a.stride + 1, pitch = Q + 1;
    if ((unsigned long long)a.N * a.H * a.W * a.Cin * 2ull >= 0x7FFFFFFFull || (unsigned long long)a.N * P * Q * a.Cout * 2ull >= 0x7FFFFFFFull)
        return "weight gradient: tensors of 2 GiB or more";
    const long long rows = (long long)a.N * (P + 1);
    if (rows > 0x70000000LL) return "weight gradient: too many rows";
    p.rows = (int)rows;
    p.tiles = (a.Cin / 64) * (a.Cout / 64);
    const int planes = a.stride == 1 ? 1 : 4, xmost = 96 * (a.stride == 1 ? wg3::Pieces<1>::X : wg3::Pieces<2>::X);
    p.nsplit = wgrad_splits(rows * pitch, p.tiles, kPixelNs, kSumsNs);
    // a chunk is as many rows as make 256 (64) pixels at most, and a split's chunks are of one height
    const long long most = (a.stride == 1 ? wg3::Pieces<1>::kPixels : wg3::Pieces<2>::kPixels) / pitch;
    const long long per = (rows + p.nsplit - 1) / p.nsplit, chunks = most > 1 ? (per + most - 1) / most : per;
    long long rh = (per + chunks - 1) / chunks;
    for (;; --rh) {
        p.rh = (int)rh;
        p.qn = (int)(rh * pitch + 31) / 32 * 32;
        p.xn = p.qn + (a.stride == 1 ? 2 * pitch : pitch) + 4;     // + 4: what a step reads beyond its last tap
        if (p.qn <= 96 * (a.stride == 1 ? wg3::Pieces<1>::G : wg3::Pieces<2>::G) && planes * p.xn <= xmost && p.qn + planes * p.xn <= kMaxRows) break;
        if (rh == 1) return "weight gradient: image row too wide for one chunk";
    }
    p.per = (int)per;
    p.nsplit = (int)((rows + per - 1) / per);
    p.lds = 2 * (size_t)(p.qn + planes * p.xn) * kRow;
    if (p.lds < kQuads * sizeof(f32x4)) p.lds = kQuads * sizeof(f32x4);
    return nullptr;
}

template <int STRIDE>
hipError_t launch(const Args &w, const Plan &p, hipStream_t stream) {
    static bool raised = false;
    if (!raised) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&wgrad3x3_kernel<STRIDE>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           160 * 1024);
        if (e != hipSuccess) return e;
        raised = true;
    }
    wgrad3x3_kernel<STRIDE><<<dim3(p.nsplit, p.tiles), dim3(kThreads), p.lds, stream>>>(w);
    return hipGetLastError();
}

}  // namespace wg3

const char *wgrad3x3_check(const ConvArgs &a) {
    wg3::Plan p;
    return wg3::plan_for(a, p);
}

size_t wgrad3x3_workspace_bytes(const ConvArgs &a) {
    wg3::Plan p;
    return wg3::plan_for(a, p) ? 0 : (size_t)p.nsplit * p.tiles * wg3::kQuads * sizeof(wg3::f32x4);
}

// a: the forward layer's geometry with a.x = x and a.scale = scale; g = gpre at the OUTPUT's resolution; gw fp32
// [Cout][3][3][Cin]; workspace of at least wgrad3x3_workspace_bytes(a), 16-byte aligned.
hipError_t launch_wgrad3x3(const ConvArgs &a, const void *g, float *gw, void *workspace, size_t workspace_bytes, hipStream_t stream) {
    wg3::Plan p;
    if (wg3::plan_for(a, p) || !g || !gw || !workspace || !a.x || !a.scale || workspace_bytes < wgrad3x3_workspace_bytes(a) ||
        ((uintptr_t)workspace | (uintptr_t)g | (uintptr_t)a.x) & 15)
        return hipErrorInvalidValue;
    wg3::Args w;
    w.x = a.x; w.g = g; w.partial = static_cast<float *>(workspace);
    w.N = a.N; w.H = a.H; w.W = a.W; w.C = a.Cin; w.K = a.Cout;
    w.P = (a.H - 1) / a.stride + 1; w.Q = (a.W - 1) / a.stride + 1;
    w.pitch = w.Q + 1;
    w.rows = p.rows; w.RH = p.rh; w.QN = p.qn; w.XN = p.xn; w.per = p.per; w.nsplit = p.nsplit;
    w.image = make_divisor((uint32_t)(w.P + 1));
    const hipError_t e = a.stride == 1 ? wg3::launch<1>(w, p, stream) : wg3::launch<2>(w, p, stream);
    if (e != hipSuccess) return e;
    const size_t groups = (size_t)p.tiles * wg3::kQuads / 64;
    // wavefronts per group of 64 sums: about four splits each
    const int G = p.nsplit <= 4 ? 1 : p.nsplit <= 8 ? 2 : p.nsplit <= 16 ? 4 : 8;
    const dim3 grid((unsigned)(groups / (8 / G)));
    switch (G) {
    case 1: wg3::wgrad3x3_reduce_kernel<1><<<grid, dim3(512), 0, stream>>>(w.partial, a.scale, gw, a.Cout, a.Cin, p.nsplit); break;
    case 2: wg3::wgrad3x3_reduce_kernel<2><<<grid, dim3(512), 0, stream>>>(w.partial, a.scale, gw, a.Cout, a.Cin, p.nsplit); break;
    case 4: wg3::wgrad3x3_reduce_kernel<4><<<grid, dim3(512), 0, stream>>>(w.partial, a.scale, gw, a.Cout, a.Cin, p.nsplit); break;
    default: wg3::wgrad3x3_reduce_kernel<8><<<grid, dim3(512), 0, stream>>>(w.partial, a.scale, gw, a.Cout, a.Cin, p.nsplit); break;
    }
    return hipGetLastError();
}

}  // namespace delta
