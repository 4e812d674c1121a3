// Both gradients of a 1x1 stride-1 layer whose weights are small, in one pass over its tensors, for gfx950, bf16:
//   gx[m,c] = (sum_k gpre[m,k] * wt[c,k] (+ gx_add[m,c])) (* [x[m,c] > 0])
//   gw[k,c] = scale_k * sum_m gpre[m,k] * x[m,c]
//
// These layers are bound by memory (28-100 FLOP per byte): as two kernels they read gpre and x twice (x a second time as the ReLU
// mask), 141 bytes where 77 do for 64 -> 256 channels and 231 where 167 do for 256 -> 64 with gx_add.  Here a workgroup holds
// everything that belongs to one run of pixels at once:
//  * a workgroup owns all K = 64 KT channels of gpre and 64 CT channels of x, and is persistent over chunks of P pixels (worker w takes
//    chunks w, w + workers, ...); a layer of more channels is several slices of C, the slices of a worker on one XCD, where
//    they share gpre in the L2;
//  * a chunk's rows of gpre, x and gx_add go from memory straight into LDS (global_load_lds) through a ring of S chunks, S - 1 of them in
//    flight per CU (48-120 KB): that is what keeps the memory busy while the chunk before is multiplied (0.5 us of a chunk's 2.5);
//  * gw: as in wgrad1x1.hip, transposing LDS reads, sums in registers for the whole launch (at most 64 a lane), partial sums to the workspace
//    in that kernel's layout, whose reduction adds them in the order of the workers and applies scale;
//  * gx: 16x16x32 MFMAs with the wavefront's rows of wt in registers for the whole launch (8-64), gpre from LDS; the epilogue finds gx_add
//    and the mask in LDS too, leaves bf16 rows there (in gx_add's place where there is one) and the rows leave as whole lines;
//  * LDS rows: the 64-byte groups of a row are permuted by the row's low bits, the 16-byte pieces of a group by the next two, so that the four
//    rows a transposing read touches and the sixteen a gx read touches spread over the banks; the direct load fixes where a lane's
//    16 bytes land, so the permutation is applied to the address each lane fetches;
//  * EVEN: gx_add has values at pixels of even row and column only (a stride-2 layer's data gradient, just stored): the loads of the others go to a few
//    zero pixels of the tensor, in an image by the worker's number, which the caches hold, so that a quarter of the tensor is read;
//  * rows past the last pixel are fetched from the last pixel and overwritten with zeros in LDS before they are read;
//  * OWN: a layer with a ReLU of its own brings gy and y, whose rows have one buffer: gpre = gy * [y > 0] replaces gy in LDS and leaves for memory on
//    the way, instead of in a launch before this one that reads both and whose result is read again.
// Backward of three conv2_x bottlenecks on 32 x 56 x 56 440 -> 346 us, of conv3_x's first on 128 x 56 x 56 610 -> 551, of its others on 128 x 28 x 28 322 -> 278.
// joint1x1_applies says where the line lies and what both sides measured.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "kernels.hpp"

namespace delta {
namespace joint {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

struct Args {
    const unsigned char *g, *x, *add, *wt;       // [M,K], [M,C], [M,C] (ADD), [C,K]
    unsigned char *gx;                           // [M,C]
    float *partial;                              // [workers][slices][KT CT][4 tiles][4][64 lanes] f32x4
    int M, C, nchunks, workers, slices, mask;
    const unsigned char *y;                      // OWN: g is gy, and gpre = gy * [y > 0] is made here
    unsigned char *gpre;                         // [M,K] both
    int N, H, W, zeros;                          // EVEN: images, their rows and columns; how many zero pixels stand for all, less one (1, 2, .. 16 less one)
    Divisor dw, dh;
};

// What is added to gx: nothing; a tensor; a tensor whose pixels of odd row or column are known to be zeros.
enum Add { NONE, ALL, EVEN };

template <int KT, int CT, int ADD, bool OWN> struct Shape {
    static constexpr int kPixels = KT + 2 * CT <= 6 && !OWN ? 64 : 32;            // of a chunk
    static constexpr int kG = kPixels * KT * 128, kX = kPixels * CT * 128;        // bytes
    static constexpr int kSlice = kG + kX * (ADD ? 2 : 1), kOut = ADD ? 0 : kX;   // of a chunk; of the separate output tile
    static constexpr int kY = OWN ? kG : 0;                                       // y's rows, one buffer of them
    static constexpr int kFit = (160 * 1024 - kOut - kY) / kSlice, kStages = kFit < 4 ? kFit : 4;
    static constexpr int kBlocks = kSlice / 1024, kLoads = (kBlocks + 7) / 8;     // 1 KB loads of a chunk; per wavefront
    static constexpr int kStores = (kX + 8191) / 8192;                           // 16-byte stores of gx per thread that has any
    static constexpr int kMasks = kY / 8192;                                     // 16-byte pieces of gpre (and of y) per thread
    // 32 x 32 tiles of gw: NK x NC, on WK x WC wavefronts (QS of them on each, sharing a chunk's pixels)
    static constexpr int NK = 2 * KT, NC = 2 * CT;
    static constexpr int WC = NC >= 8 ? 8 : NK >= 8 && NC == 2 ? 1 : NK == 2 && NC == 4 ? 4 : 2;
    static constexpr int WK = NC >= 8 ? 1 : NK >= 8 && NC == 2 ? 8 : NK == 2 ? 2 : 4;
    static constexpr int QS = 8 / (WK * WC), TK = NK / WK, TC = NC / WC;
    // gx: slabs of 16 channels, SW to a wavefront, PG wavefronts share a slab's pixels
    static constexpr int kSlabs = 4 * CT, SW = kSlabs > 8 ? kSlabs / 8 : 1, kGroups = kSlabs < 8 ? kSlabs : 8;
    static constexpr int PG = 8 / kGroups, kPT = kPixels / 16 / PG;
    static constexpr int kSums = QS > 1 ? (QS - 1) * WK * WC * TK * TC * 4096 : 0;
    static constexpr int kRing = kStages * kSlice + kOut + kY, kLds = kRing > kSums ? kRing : kSums;
    static_assert(kStages >= 3 && kLds <= 160 * 1024 && kSlice % 1024 == 0 && (kStages - 2) * kLoads + (kStages - 1) * (kStores + kMasks) <= 63, "LDS, vmcnt");
    static_assert(!OWN || (!ADD && kY % 8192 == 0), "a whole number of pieces to a thread");
};

// How the 64-byte groups of a row of T * 128 bytes are permuted, and the 16-byte pieces of a group.
template <int T> __device__ __forceinline__ int group_flip(int row) { return T == 1 ? (row >> 1) & 1 : row & 3; }
__device__ __forceinline__ int piece_flip(int row) { return (row >> 2) & 3; }
template <int T> __device__ __forceinline__ int lds_at(int row, int group, int piece) {
    return row * (T * 128) + ((group ^ group_flip<T>(row)) << 6) + ((piece ^ piece_flip(row)) << 4);
}

__device__ __forceinline__ float lo16(uint32_t p) { return __uint_as_float(p << 16); }
__device__ __forceinline__ float hi16(uint32_t p) { return __uint_as_float(p & 0xFFFF0000u); }
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
// The workgroup meets; LDS is in order, and what travels between memory and LDS or memory stays in flight.
__device__ __forceinline__ void meet() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

template <int KT, int CT, int ADD, bool OWN>
__global__ __launch_bounds__(512) void joint1x1_kernel(Args a) {
    using T = Shape<KT, CT, ADD, OWN>;
    constexpr int S = T::kStages, P = T::kPixels, XP = CT * 128, L = T::kLoads;
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, quad = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int xcd = blockIdx.x & 7, rest = blockIdx.x >> 3, worker = rest / a.slices * 8 + xcd, slice = rest % a.slices;
    if (worker >= a.workers) return;                             // the whole workgroup
    const uint32_t krow = KT * 128, crow = (uint32_t)a.C * 2u, c0 = (uint32_t)slice * XP;

    // ---- direct loads: 1 KB blocks of a chunk, gpre's rows, then x's, then gx_add's; the last wavefronts may repeat the last block
    const unsigned char *base[L];
    int row[L];
    uint32_t seg[L], pitch[L], dst[L];
    bool even[L];
#pragma unroll
    for (int i = 0; i < L; ++i) {
        const int n = wv * L + i < T::kBlocks ? wv * L + i : T::kBlocks - 1, b = n * 1024 + lane * 16;
        dst[i] = (uint32_t)n * 1024u;
        even[i] = ADD == EVEN && n * 1024 >= T::kG + T::kX;
        if (n * 1024 < T::kG) {
            row[i] = b / (KT * 128);
            const int slot = b % (KT * 128) >> 4;
            base[i] = a.g;
            pitch[i] = krow;
            seg[i] = (uint32_t)((((slot >> 2) ^ group_flip<KT>(row[i])) << 6) + (((slot & 3) ^ piece_flip(row[i])) << 4));
        } else {
            const bool second = ADD && n * 1024 >= T::kG + T::kX;
            const int bx = b - T::kG - (second ? T::kX : 0);
            row[i] = bx / XP;
            const int slot = bx % XP >> 4;
            base[i] = second ? a.add : a.x;
            pitch[i] = crow;
            seg[i] = c0 + (uint32_t)((((slot >> 2) ^ group_flip<CT>(row[i])) << 6) + (((slot & 3) ^ piece_flip(row[i])) << 4));
        }
    }
    typedef __attribute__((address_space(3))) unsigned char *lptr_t;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)smem;
    const int zero0 = ADD == EVEN ? worker % a.N * a.H * a.W + 1 : 0;   // pixel 1 of an image: as many sets of lines as images, spread over the workers
    auto fetch = [&](int chunk, int buf) {
        const int m0 = chunk * P, last = a.M - 1 - m0;           // rows past the last pixel: that pixel
#pragma unroll
        for (int i = 0; i < L; ++i) {
            int m = m0 + (row[i] < last ? row[i] : last);
            if (ADD == EVEN && even[i]) {
                const int t = divide(m, a.dw), w = m - t * a.W, h = t - divide(t, a.dh) * a.H;
                if ((h | w) & 1) m = zero0 + 2 * (row[i] & a.zeros);
            }
            load_lds_b128(base[i], (uint32_t)m * pitch[i] + seg[i], lds0 + (uint32_t)(buf * T::kSlice) + dst[i]);
        }
    };
    // OWN: y's rows of a chunk, laid out as gpre's, a thread's pieces 512 apart; they have one buffer, free as soon as the chunk before is masked
    unsigned char *ybuf = smem + S * T::kSlice + T::kOut;
    auto fetch_y = [&](int chunk) {
        if constexpr (OWN) {
            const int m0 = chunk * P, last = a.M - 1 - m0;
#pragma unroll
            for (int i = 0; i < T::kMasks; ++i) {
                const int at = (tid + 512 * i) * 16, r = at / (KT * 128), slot = at % (KT * 128) >> 4;
                const uint32_t where = (uint32_t)((((slot >> 2) ^ group_flip<KT>(r)) << 6) + (((slot & 3) ^ piece_flip(r)) << 4));
                load_lds_b128(a.y, (uint32_t)(m0 + (r < last ? r : last)) * krow + where,
                              lds0 + (uint32_t)(S * T::kSlice + T::kOut + wv * 1024 + i * 8192));
            }
        }
    };
    // Loads and stores complete in order: a chunk has landed when at most the later chunks' loads and the stores issued since are under way.
    const bool stores = wv * 1024 < T::kX;                       // this wavefront stores rows of gx (kStores times a chunk)
    const bool masks = OWN && slice == 0;                        // the first slice stores gpre (kMasks times a chunk)
    auto wait_for = [&](int later, int stored, auto each) {
#pragma unroll
        for (int r = 0; r <= S - 2; ++r)
#pragma unroll
            for (int s = 0; s <= S - 1; ++s)
                if (later == r && stored == s) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(r * L + s * decltype(each)::value) : "memory");
    };
    auto wait_chunk = [&](int t, int mine) {
        if constexpr (OWN) {
            // y of chunk t was the first thing asked for after chunk t - 1 was masked; behind it came chunk t + S - 2 and that chunk's stores
            const bool steady = t + S - 2 < mine;
            if (t == 0) wait_for(steady ? S - 2 : 0, 0, std::integral_constant<int, 0>());
            else if (masks && stores) wait_for(steady, steady, std::integral_constant<int, T::kStores + T::kMasks>());
            else if (masks) wait_for(steady, steady, std::integral_constant<int, T::kMasks>());
            else if (stores) wait_for(steady, steady, std::integral_constant<int, T::kStores>());
            else wait_for(steady, 0, std::integral_constant<int, 0>());
        } else {
            const int later = mine - 1 - t < S - 2 ? mine - 1 - t : S - 2;
            wait_for(later, !stores ? 0 : t < S - 1 ? t : S - 1, std::integral_constant<int, T::kStores>());
        }
    };

    // ---- gw: transposing reads.  A lane supplies row 8 (lane / 32) + (lane % 16) / 4 (+ 4) of a 16-pixel step and channels
    // 16 ((lane / 16) % 2) + 4 (lane % 4) .. + 3 of a 32-channel group
    const int base_tile = wv % (T::WK * T::WC), qs = wv / (T::WK * T::WC), kw = base_tile % T::WK, cw = base_tile / T::WK;
    const int srow = 8 * (lane >> 5) + (l16 >> 2), spiece = 2 * (quad & 1) + ((lane & 3) >> 1), sbyte = 8 * (lane & 1);
    int goff[2][T::TK], xoff[2][T::TC];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int i = 0; i < T::TK; ++i) goff[h][i] = lds_at<KT>(srow + 4 * h, kw * T::TK + i, spiece) + sbyte;
#pragma unroll
        for (int j = 0; j < T::TC; ++j) xoff[h][j] = T::kG + lds_at<CT>(srow + 4 * h, cw * T::TC + j, spiece) + sbyte;
    }
    typedef s16x4 __attribute__((address_space(3))) * lds_ptr;
    auto tr_read = [&](const unsigned char *p) { return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p)); };
    f32x16 acc[T::TK][T::TC];
#pragma unroll
    for (int i = 0; i < T::TK; ++i)
#pragma unroll
        for (int j = 0; j < T::TC; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    const int mine = (a.nchunks - worker + a.workers - 1) / a.workers;
    auto chunk_of = [&](int t) { return worker + t * a.workers; };
    fetch(chunk_of(0), 0);                                       // workers <= nchunks: everyone has one

    // ---- this wavefront's rows of wt, for the whole launch, behind the first chunk: slab s, 32 channels of k per step, lane: c l16, k 8 quad .. + 7
    constexpr int kSteps = KT * 2;
    const int sg = wv % T::kGroups, pg = wv / T::kGroups;
    u32x4 wt[T::SW][kSteps];
#pragma unroll
    for (int s = 0; s < T::SW; ++s)
#pragma unroll
        for (int q = 0; q < kSteps; ++q)
            wt[s][q] = *reinterpret_cast<const u32x4 *>(a.wt + (size_t)(c0 / 2 + (sg * T::SW + s) * 16 + l16) * krow + q * 64 + quad * 16);
    // Waited for here: the compiler would wait for them in the loop, and for everything else that is under way with them.
#pragma unroll
    for (int s = 0; s < T::SW; ++s)
#pragma unroll
        for (int q = 0; q < kSteps; ++q) asm volatile("" : "+v"(wt[s][q]));

    if constexpr (OWN) fetch_y(chunk_of(0));
#pragma unroll
    for (int t = 1; t < S - 1; ++t)
        if (t < mine) fetch(chunk_of(t), t);
    for (int t = 0, buf = 0; t < mine; ++t) {
        wait_chunk(t, mine);                                     // this wavefront's part of chunk t has landed
        meet();                                                  // everyone's has; the buffer of chunk t - 1 is free
        auto ahead = [&] {
            if (t + S - 1 < mine) fetch(chunk_of(t + S - 1), buf == 0 ? S - 1 : buf - 1);
        };
        if constexpr (!OWN) ahead();
        unsigned char *sl = smem + buf * T::kSlice;
        const int m0 = chunk_of(t) * P, valid = a.M - m0;
        if (valid < P) {                                         // the last chunk of all: rows past the last pixel
            for (int i = tid; i < (T::kG + T::kX) / 16; i += 512) {
                const int r = i * 16 < T::kG ? i * 16 / (KT * 128) : (i * 16 - T::kG) / XP;
                if (r >= valid) *reinterpret_cast<u32x4 *>(sl + i * 16) = u32x4{0u, 0u, 0u, 0u};
            }
            meet();
        }
        if constexpr (OWN) {                                     // gpre = gy * [y > 0], in place and to memory
            u32x4 o[T::kMasks];
#pragma unroll
            for (int i = 0; i < T::kMasks; ++i) {
                const int at = (tid + 512 * i) * 16;
                const u32x4 gv = *reinterpret_cast<const u32x4 *>(sl + at), yv = *reinterpret_cast<const u32x4 *>(ybuf + at);
#pragma unroll
                for (int e = 0; e < 4; ++e) o[i][e] = keep_where_positive_bf16(gv[e], yv[e]);
                *reinterpret_cast<u32x4 *>(sl + at) = o[i];
            }
            meet();
            if (t + 1 < mine) fetch_y(chunk_of(t + 1));
            ahead();
            if (masks) {
#pragma unroll
                for (int i = 0; i < T::kMasks; ++i) {
                    const int at = (tid + 512 * i) * 16, r = at / (KT * 128), slot = at % (KT * 128) >> 4;
                    const uint32_t where = (uint32_t)((((slot >> 2) ^ group_flip<KT>(r)) << 6) + (((slot & 3) ^ piece_flip(r)) << 4));
                    if (r < valid) *reinterpret_cast<u32x4 *>(a.gpre + (size_t)(m0 + r) * krow + where) = o[i];
                }
            }
        }
        // ---- gw
#pragma unroll
        for (int q = 0; q < P / (16 * T::QS); ++q) {
            const int r0 = 16 * (qs + q * T::QS);
            s16x8 gf[T::TK], xf[T::TC];
#pragma unroll
            for (int i = 0; i < T::TK; ++i)
                gf[i] = __builtin_shufflevector(tr_read(sl + r0 * (KT * 128) + goff[0][i]), tr_read(sl + r0 * (KT * 128) + goff[1][i]), 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
            for (int j = 0; j < T::TC; ++j)
                xf[j] = __builtin_shufflevector(tr_read(sl + r0 * XP + xoff[0][j]), tr_read(sl + r0 * XP + xoff[1][j]), 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
            for (int i = 0; i < T::TK; ++i)
#pragma unroll
                for (int j = 0; j < T::TC; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, gf[i]), __builtin_bit_cast(bf16x8, xf[j]),
                                                                        acc[i][j], 0, 0, 0);
        }
        // ---- gx: lane holds pixel l16 and channels 4 quad .. + 3 of a 16 x 16 tile
        unsigned char *out = ADD ? sl + T::kG + T::kX : smem + S * T::kSlice;
#pragma unroll
        for (int u = 0; u < T::kPT; ++u) {
            const int r = (pg * T::kPT + u) * 16 + l16;
            f32x4 v[T::SW];
#pragma unroll
            for (int s = 0; s < T::SW; ++s) v[s] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < kSteps; ++q) {
                const u32x4 gv = *reinterpret_cast<const u32x4 *>(sl + lds_at<KT>(r, q, quad));
#pragma unroll
                for (int s = 0; s < T::SW; ++s)
                    v[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wt[s][q]), __builtin_bit_cast(bf16x8, gv), v[s], 0, 0, 0);
            }
#pragma unroll
            for (int s = 0; s < T::SW; ++s) {
                const int slab = sg * T::SW + s, at = lds_at<CT>(r, slab >> 1, (slab & 1) * 2 + (quad >> 1)) + 8 * (quad & 1);
                if constexpr (ADD) {
                    const u32x2 ad = *reinterpret_cast<const u32x2 *>(out + at);
                    v[s][0] += lo16(ad.x); v[s][1] += hi16(ad.x); v[s][2] += lo16(ad.y); v[s][3] += hi16(ad.y);
                }
                u32x2 o = {pack2(v[s][0], v[s][1]), pack2(v[s][2], v[s][3])};
                if (a.mask) {
                    const u32x2 xm = *reinterpret_cast<const u32x2 *>(sl + T::kG + at);
                    o = u32x2{keep_where_positive_bf16(o.x, xm.x), keep_where_positive_bf16(o.y, xm.y)};
                }
                *reinterpret_cast<u32x2 *>(out + at) = o;
            }
        }
        meet();
        if (stores) {
#pragma unroll
            for (int j = 0; j < T::kStores; ++j) {
                const int i = tid + 512 * j, r = i / (XP / 16), s = i % (XP / 16);
                const u32x4 o = *reinterpret_cast<const u32x4 *>(out + lds_at<CT>(r, s >> 2, s & 3));
                if (r < valid) *reinterpret_cast<u32x4 *>(a.gx + (size_t)(m0 + r) * crow + c0 + s * 16) = o;
            }
        }
        buf = buf + 1 == S ? 0 : buf + 1;
    }

    // ---- the sums; lane: column (c) l % 32, rows (k) 8 e4 + 4 (l / 32) + e in register 4 e4 + e, as in wgrad1x1.hip
    if constexpr (T::QS > 1) {                                   // one tile to a wavefront: those of the first QS - 1 others through LDS
        static_assert(T::QS <= 2 && T::TK * T::TC == 1, "two wavefronts to a tile");
        __syncthreads();
        f32x4 *red = reinterpret_cast<f32x4 *>(smem) + base_tile * 256 + lane;
        if (qs) {
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4) red[e4 * 64] = f32x4{acc[0][0][4 * e4], acc[0][0][4 * e4 + 1], acc[0][0][4 * e4 + 2], acc[0][0][4 * e4 + 3]};
        }
        __syncthreads();
        if (qs) return;
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[0][0][4 * e4 + e] += red[e4 * 64][e];
    }
    f32x4 *sums = reinterpret_cast<f32x4 *>(a.partial) + ((size_t)worker * a.slices + slice) * (KT * CT) * 1024 + lane;
#pragma unroll
    for (int i = 0; i < T::TK; ++i)
#pragma unroll
        for (int j = 0; j < T::TC; ++j) {
            const int k32 = kw * T::TK + i, c32 = cw * T::TC + j;
            f32x4 *tile = sums + ((size_t)((k32 >> 1) + KT * (c32 >> 1)) * 16 + ((k32 & 1) * 2 + (c32 & 1)) * 4) * 64;
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4) tile[e4 * 64] = f32x4{acc[i][j][4 * e4], acc[i][j][4 * e4 + 1], acc[i][j][4 * e4 + 2], acc[i][j][4 * e4 + 3]};
        }
}

struct Plan { int kt, ct, slices, pixels, nchunks, workers; };

// `fa`: the layer, 1x1 stride 1.
bool plan_for(const ConvArgs &fa, Plan &p) {
    if (!fa.bf16 || fa.R != 1 || fa.S != 1 || fa.stride != 1 || fa.pad != 0 || fa.Cin % 64 || fa.Cout % 64) return false;
    const int kt = fa.Cout / 64;
    if (kt != 1 && kt != 2 && kt != 4 && kt != 8) return false;
    if ((long long)fa.M * fa.Cin * 2 > 0x7FFFFFFFLL || (long long)fa.M * fa.Cout * 2 > 0x7FFFFFFFLL) return false;
    int ct = 8 / kt < 4 ? 8 / kt : 4;
    while (fa.Cin % (64 * ct)) ct /= 2;
    p.kt = kt; p.ct = ct; p.slices = fa.Cin / (64 * ct);
    p.pixels = kt + 2 * ct <= 6 ? 64 : 32;
    p.nchunks = (fa.M + p.pixels - 1) / p.pixels;
    // One workgroup per CU, and no more of them than have as many chunks as the longest; at least two chunks (three of 32 pixels) to a worker,
    // whose partial sums cost as much as a chunk (us with one | two | three: 64 -> 256 on 12544 pixels 17.0 | 14.3 | 14.5, 64 -> 64
    // 10.1 | 9.4 | 9.9, 256 -> 64 16.9 | 17.1 | 15.6, 128 -> 256 23.1 | 23.6 | 20.7).
    // All slices of a worker are on its XCD, whose 32 CUs hold 32 / slices workers: one worker more on any of them is a second round for the whole launch
    // (us with 256 / slices workers, this, and two kernels: 768 -> 256 on 26950 pixels 75, 47, 55; 448 -> 256 on 159936 239, 143, 167; 1280 -> 128 on 68992
    // 189, 131, 168).
    const int most = p.slices > 32 ? 8 : 32 / p.slices * 8, least = p.pixels == 64 ? 2 : 3;
    int each = (p.nchunks + most - 1) / most;
    if (each < least) each = least;
    p.workers = (p.nchunks + each - 1) / each;
    return true;
}

template <int KT, int CT, int ADD, bool OWN>
hipError_t launch(const Args &w, hipStream_t stream) {
    using T = Shape<KT, CT, ADD, OWN>;
    static bool raised = false;
    if (!raised) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&joint1x1_kernel<KT, CT, ADD, OWN>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, T::kLds);
        if (e != hipSuccess) return e;
        raised = true;
    }
    joint1x1_kernel<KT, CT, ADD, OWN><<<dim3((unsigned)((w.workers + 7) / 8 * 8 * w.slices)), dim3(512), T::kLds, stream>>>(w);
    return hipGetLastError();
}

}  // namespace joint

// Where the line lies, measured as us per layer in a segment of such layers, two kernels on two streams (one stream below 1 GFLOP) | this one with its
// reduction, without | with gx_add:
//   64 -> 256   M = 6272 15.6 | 12.7    12544 17.2 | 14.3    50176 28 | 19    100352 37 | 24    401408 101 | 64
//   256 -> 64   M = 6272 18.5 19.4 | 12.9 13.6    25088 25 26 | 20 19    100352 40 48 | 32 36    401408 143 188 | 90 129
//   64 -> 64    M = 6272 14 14 | 8.9 9.1    100352 26 28 | 17 18         128 -> 128  M = 5488 16 17 | 12 12    100352 33 35 | 25 27
//   256 -> 128  M = 6272 21 23 | 17 18    50176 31 33 | 28 30    401408 174 212 | 108 144
//   512 -> 128  M = 7840 26 25 | 24 23    25088 46 48 | 28 30    100352 79 99 | 59 73      1024 -> 256  M = 6272 31 32 | 29 28    25088 53 57 | 52 55
//   64 -> 512   M = 7840 18.7 | 20.1    12544 22.2 | 21.7    100352 46 | 37      128 -> 512  M = 7840 25 | 26    25088 27 | 26    100352 51 | 53, which as part
//   of a bottleneck's backward pass still wins (282 us with this layer on two kernels, 278 with it here)
//   512 -> 256  M = 25088 39 43 | 36 37; but 512 -> 512, 1024 -> 512 and 2048 -> 512 on 12544 and 25088 pixels 31 to 77 | 37 to 90: with 512 gradient
//   channels a slice holds 64 input channels, and from four slices on gpre's way through the L2 to each of them is what it costs.
// small_backward.hip comes first: it takes the smaller layers by its own price, to 4096 or 6400 pixels at most.  Below 4000 pixels (9000 with 512 gradient
// channels) what it leaves goes to two kernels.  Both lines lie higher than they have to: 1024 -> 256 on 3332 to 3920 pixels 32 | 24 to 27, 128 -> 512 on
// 7840 and 8624 32 | 25 to 27, but 128 -> 512 on 7056 21.5 | 23.7 and 64 -> 512 on 7056 and 8624 18.4 21.5 | 20.0 22.3 (one stream, below 1 GFLOP).
bool joint1x1_applies(const ConvArgs &fa) {
    joint::Plan p;
    return joint::plan_for(fa, p) && (p.kt == 8 ? p.slices <= 2 && fa.M >= 9000 : p.slices <= 8 && fa.M >= 4000);
}

size_t joint1x1_workspace_bytes(const ConvArgs &fa) {
    joint::Plan p;
    return joint1x1_applies(fa) && joint::plan_for(fa, p) ? (size_t)p.workers * p.slices * p.kt * p.ct * 16384 : 0;
}

// The widest gradient to the fewest input channels, where gpre is most of what a launch moves.  us with its reduction, the mask's launch before it | on the way:
// 64 -> 256 on 401408 pixels 180 | 135, 100352 54 | 45, 34000 28.6 | 25.4, 14000 19.7 | 18.6, 9000 17.0 | 16.7, but 6000 15.7 | 15.8, 4100 14.3 | 14.6;
// 128 -> 512 on 100352 112 | 91, 34000 52 | 44, 14000 33.6 | 29.8, 9050 27.1 | 26.7; 64 -> 512 on 34000 45 | 39, 14000 28.2 | 25.7, 11000 24.3 | 23.8, but 10500
// 24.1 | 24.2, 9050 23.4 | 24.3.  Every slice reads gy and y and masks them again, of which the first stores gpre: with three (192 -> 256) 60000 pixels
// 50.3 | 49.6 and 25088 29.7 | 28.6, but 18000 24.0 | 24.9, 16000 22.8 | 24.2, 11000 22.1 | 22.5; five (320 -> 256) on 25088 36.3 | 40.2, 100352 96 | 113,
// seven (448 -> 256) 43 | 52, 122 | 161.  128 -> 512 keeps three chunks of gy and x and one of y in 144 KB: chunks of 16 pixels in four buffers 113 us (half the
// work per barrier), of 32 with y in two 109.
bool joint1x1_masks(const ConvArgs &da, const ConvArgs &fa) {
    joint::Plan p;
    if (!joint1x1_applies(fa) || !joint::plan_for(fa, p) || p.ct != 1 || da.res) return false;
    return p.kt == 4 ? p.slices == 1 && fa.M >= 7000 : p.kt == 8 && (p.slices == 2 || (p.slices == 1 && fa.M >= 11000));
}

// From here on a gx_add that is zeros but for its pixels of even row and column is read at those pixels only; the loads of the others take zeros that
// the caches hold.  Block of a strided layer, 256 channels to 128, us, all of gx_add read | this: on 128 x 56 x 56 475 | 455, 96 376 | 365, 64 280 | 274, but
// 40 209.5 | 211.2 and 24 155 | 156, where the caches still hold the tensor; 256 to 64 (strided 1x1, 3x3 and this layer) 353 | 333, 288 | 272, 64 197 | 197.  In several slices it never pays: 512 to 256 on 128 x 28 x 28 372 | 377, on
// 64 x 56 x 56 650 | 660.
constexpr size_t kEvenBytes = (size_t)96 << 20;

// gpre, where it is not null: g is gy and gpre = gy * [y > 0] is made and stored here (joint1x1_masks).
// da: the data gradient's convolution, complete (its mask, where there is one, is x); fa: the layer, with x and scale; g = gpre; gw fp32
// [Cout][Cin]; workspace of joint1x1_workspace_bytes(fa), 16-byte aligned.
hipError_t launch_joint1x1(const ConvArgs &da, const ConvArgs &fa, const void *g, const void *y, void *gpre, float *gw, void *workspace,
                           size_t workspace_bytes, bool add_even, hipStream_t stream) {
    joint::Plan p;
    if (!joint1x1_applies(fa) || !joint::plan_for(fa, p) || !g || !gw || !workspace || !fa.x || !fa.scale || !da.w || !da.y ||
        (da.mask && da.mask != fa.x) || da.x != g || da.M != fa.M || da.Cin != fa.Cout || da.Cout != fa.Cin || da.oy_s || da.relu ||
        workspace_bytes < joint1x1_workspace_bytes(fa) || !y != !gpre || (gpre && (!joint1x1_masks(da, fa) || gpre == g || gpre == y)) ||
        (((uintptr_t)g | (uintptr_t)fa.x | (uintptr_t)da.w | (uintptr_t)da.y | (uintptr_t)da.res | (uintptr_t)workspace |
          (uintptr_t)y | (uintptr_t)gpre) & 15))
        return hipErrorInvalidValue;
    joint::Args w;
    w.g = static_cast<const unsigned char *>(g); w.x = static_cast<const unsigned char *>(fa.x); w.add = static_cast<const unsigned char *>(da.res);
    w.wt = static_cast<const unsigned char *>(da.w); w.gx = static_cast<unsigned char *>(da.y); w.partial = static_cast<float *>(workspace);
    w.M = fa.M; w.C = fa.Cin; w.nchunks = p.nchunks; w.workers = p.workers; w.slices = p.slices; w.mask = da.mask != nullptr;
    w.N = fa.N; w.H = fa.H; w.W = fa.W; w.dw = make_divisor((uint32_t)fa.W); w.dh = make_divisor((uint32_t)fa.H);
    w.zeros = 0;                                                 // pixels 1, 3, .. of the first row (of the first column, if there is one column)
    while (w.zeros < 15 && 1 + 2 * (2 * w.zeros + 1) < fa.W) w.zeros = 2 * w.zeros + 1;
    w.y = static_cast<const unsigned char *>(y); w.gpre = static_cast<unsigned char *>(gpre);
    hipError_t e;
    if (gpre) {                                                  // chunks of 32 pixels, as many workers or fewer
        const int chunks = (fa.M + 31) / 32, each = (chunks + p.workers - 1) / p.workers;
        w.nchunks = chunks;
        w.workers = p.workers = (chunks + each - 1) / each;
        e = p.kt == 4 ? joint::launch<4, 1, joint::NONE, true>(w, stream) : joint::launch<8, 1, joint::NONE, true>(w, stream);
    } else if (add_even && da.res && p.ct == 4 && p.slices == 1 && (size_t)fa.M * fa.Cin * 2 >= kEvenBytes) {
        e = p.kt == 1 ? joint::launch<1, 4, joint::EVEN, false>(w, stream) : joint::launch<2, 4, joint::EVEN, false>(w, stream);
    } else
    switch (p.kt * 10 + p.ct) {
#define DELTA_JOINT(KT, CT) \
    case KT * 10 + CT: e = da.res ? joint::launch<KT, CT, joint::ALL, false>(w, stream) : joint::launch<KT, CT, joint::NONE, false>(w, stream); break;
    DELTA_JOINT(1, 1) DELTA_JOINT(1, 2) DELTA_JOINT(1, 4) DELTA_JOINT(2, 1) DELTA_JOINT(2, 2) DELTA_JOINT(2, 4)
    DELTA_JOINT(4, 1) DELTA_JOINT(4, 2) DELTA_JOINT(8, 1)
#undef DELTA_JOINT
    default: return hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
    return launch_wgrad1x1_reduce(w.partial, fa.scale, gw, fa.Cout, fa.Cin, p.kt, p.ct, p.workers, stream);
}

}  // namespace delta
