// Internal launchers of the HIP kernels (conv_igemm.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace delta {

struct ConvArgs {
    const void *x;        // [N,H,W,Cin]
    const void *w;        // [Cout,R,S,Cin]
    const void *res;      // [N,P,Q,Cout] or nullptr
    const void *mask;     // [N,P,Q,Cout] or nullptr: y is stored as 0 where mask is not > 0 (after residual and ReLU)
    void *y;              // [N,P,Q,Cout]
    const float *scale;   // [Cout]
    const float *shift;   // [Cout]
    int N, H, W, Cin, Cout, R, S, stride, pad, P, Q, M;
    int relu;             // 0: none, 1: ReLU, 2: GELU (erf form; tiled kernel only)
    // (the next three share four bytes: kernels take this structure by value, and eight bytes more were 0.02 to 0.04 us of the smallest launches, 5 to 8 us)
    short bf16;           // 1: bf16 storage, fp32 accumulate; 0: fp32
    // With the scattered form of a 1x1 layer: the pixels of the oy_s x oy_s block that starts at an output pixel, inside the image and not
    // written themselves, are stored as zeros (launch_conv_spread: a strided 1x1 layer's data gradient in one pass).
    unsigned char spread = 0;
    // Another stream's kernels run beside this launch (a weight gradient, most of them one workgroup to a CU): tail_pieces.
    unsigned char shared = 0;
    // Scattered form (launch_conv_scatter only; the data gradient of a strided layer, one parity
    // class of input pixels at a time).  oy_s > 0: output pixel (n, p, q) is stored at pixel
    // (n, p * oy_s + oy_a, q * oy_s + oy_b) of an [N, OH, OW, Cout] tensor; res and mask are read
    // there; P and Q are the caller's (a tap that leaves the input reads zeros); the R x S taps are
    // taps (w_r0 + r * w_step, w_s0 + s * w_step) of a weight tensor [Cout, wR, wS, Cin].
    int oy_s = 0, oy_a = 0, oy_b = 0, OH = 0, OW = 0;
    int wR = 0, wS = 0, w_r0 = 0, w_s0 = 0, w_step = 1;
};

// Division by a launch constant as a multiplication, exact for 0 <= n < 2^31: with 2^(s-1) < d <= 2^s and mul = ceil(2^(31+s) / d),
// floor(n mul / 2^(31+s)) == floor(n / d), because mul d exceeds 2^(31+s) by less than d <= 2^s.  mul 0 stands for d = 1.
struct Divisor { uint32_t mul, shift; };
inline Divisor make_divisor(uint32_t d) {
    if (d <= 1) return Divisor{0u, 0u};
    uint32_t s = 1;
    while (s < 32 && (1ull << s) < d) ++s;
    return Divisor{(uint32_t)(((1ull << (31 + s)) + d - 1) / d), s - 1};
}
__device__ __forceinline__ int divide(int n, Divisor d) { return d.mul ? (int)(__umulhi((uint32_t)n, d.mul) >> d.shift) : n; }

// 16 bytes per lane from memory straight into LDS: lane l's land at byte `lds` + 16 l, `lds` the same for the whole wavefront.  Inline
// assembly, because the compiler does not track what a direct load writes; whoever uses it waits with s_waitcnt vmcnt
// (direct loads complete in order).  The load reads M0, and the hardware needs one wait state between the scalar write of
// M0 and such a load; the compiler inserts none inside an asm block, hence the s_nop.
__device__ __forceinline__ void load_lds_b128(const unsigned char *at, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                 :: "v"(at), "s"(__builtin_amdgcn_readfirstlane(lds)) : "memory", "m0");
}
// The same from `off` bytes past a base that is the same for the whole wavefront.
__device__ __forceinline__ void load_lds_b128(const unsigned char *base, uint32_t off, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(off), "s"(base), "s"(__builtin_amdgcn_readfirstlane(lds)) : "memory", "m0");
}

// 4 bytes per lane: lane l's land at byte `lds` + 4 l.
__device__ __forceinline__ void load_lds_b32(const void *at, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off"
                 :: "v"(at), "s"(__builtin_amdgcn_readfirstlane(lds)) : "memory", "m0");
}

// The test behind every ReLU mask of the backward pass.  bf16: greater than zero <=> sign bit clear,
// not zero and not NaN.  Returns the bits of `v` (two bf16 values) with the halves cleared whose
// half of `m` fails it.
__device__ __forceinline__ uint32_t keep_where_positive_bf16(uint32_t v, uint32_t m) {
    const uint32_t lo = m & 0xFFFFu, hi = m >> 16;
    const bool plo = lo != 0 && lo < 0x7F81u;          // positive, finite or +inf
    const bool phi = hi != 0 && hi < 0x7F81u;
    return (plo ? (v & 0xFFFFu) : 0u) | (phi ? (v & 0xFFFF0000u) : 0u);
}
__device__ __forceinline__ uint32_t keep_where_positive_f32(uint32_t v, uint32_t m) {
    return __uint_as_float(m) > 0.f ? v : 0u;
}

// GELU in its erf form, v/2 (1 + erf(v / sqrt 2)).  1 + erf(x) = erfc(-x): for x < 0 it is
// erfc(|x|), for x >= 0 it is 2 - erfc(x), and erfc(|x|) = poly(t) exp(-x^2), t = 1/(1 + p |x|)
// (Abramowitz & Stegun 7.1.26, absolute error 1.5e-7) - no cancellation in the negative tail, one
// exp and one reciprocal per element instead of the library erff's branches.
__device__ __forceinline__ float gelu_erf(float v) {
    const float x = fabsf(v) * 0.70710678118654752f;
    const float t = __builtin_amdgcn_rcpf(1.0f + 0.3275911f * x);
    const float poly = t * (0.254829592f + t * (-0.284496736f + t * (1.421413741f + t * (-1.453152027f + t * 1.061405429f))));
    const float c = poly * __builtin_amdgcn_exp2f(-x * x * 1.4426950408889634f);   // erfc(|x|)
    return 0.5f * v * (v < 0.f ? c : 2.0f - c);
}

// nullptr when the kernel supports the shape, else the reason.
const char *conv_check(const ConvArgs &a);
const char *conv_kernel_name(const ConvArgs &a);
hipError_t launch_conv(const ConvArgs &a, hipStream_t stream);
// In how many pieces the tiles past the last whole round of the 256 CUs go out (1: whole), for a kernel that can cut a tile in up to `most`: as many as leave a
// CU at most one.  Whole where another stream's work fills such a round.  conv_pieces: of the kernel that launch_conv takes.
inline int tail_pieces(const ConvArgs &a, long long tiles, int most) {
    const int rest = (int)(tiles % 256);
    if (tiles <= 256 || !rest || a.spread || a.shared) return 1;
    while (rest * most > 256) most /= 2;
    return most;
}
int conv3x3_halo_pieces(const ConvArgs &a);
int gemm_nt_pieces(const ConvArgs &a);
int conv_pieces(const ConvArgs &a);
const char *conv_scatter_check(const ConvArgs &a);
const char *conv_scatter_kernel_name(const ConvArgs &a);
hipError_t launch_conv_scatter(const ConvArgs &a, hipStream_t stream);
// A stride-1 1x1 layer stored at the pixels (stride p, stride q) of an [N, OH, OW, Cout] tensor, zeros between (no residual, no mask)
bool conv_spread_applies(const ConvArgs &a, int stride, int OH, int OW);
void as_spread(ConvArgs &a, int stride, int OH, int OW);
hipError_t launch_conv_spread(const ConvArgs &a, hipStream_t stream);
bool dgrad_s2_applies(const ConvArgs &a);
hipError_t launch_dgrad_s2(const ConvArgs &a, hipStream_t stream);
// conv_splitk.hip: layers with too little output to fill the chip, the reduction split over a workgroup's wavefronts
bool conv_splitk_applies(const ConvArgs &a);
const char *conv_splitk_kernel_name(const ConvArgs &a);
hipError_t launch_conv_splitk(const ConvArgs &a, hipStream_t stream);
// conv1x1.hip: streaming kernel for bf16 1x1 convolutions whose weights fit LDS
bool conv1x1_stream_applies(const ConvArgs &a);
hipError_t launch_conv1x1_stream(const ConvArgs &a, hipStream_t stream);
// gemm_nt.hip: bf16 1x1 stride-1 layers with a long reduction axis as a 256 x 256-tiled GEMM
bool gemm_nt_applies(const ConvArgs &a);
const char *gemm_nt_kernel_name(const ConvArgs &a);   // with the tile the launch will use
hipError_t launch_gemm_nt(const ConvArgs &a, hipStream_t stream);
// conv3x3_halo.hip: bf16 3x3 stride-1 kernel that keeps the input halo of a pixel tile in LDS
bool conv3x3_halo_applies(const ConvArgs &a);
const char *conv3x3_halo_kernel_name(const ConvArgs &a);
hipError_t launch_conv3x3_halo(const ConvArgs &a, hipStream_t stream);
// conv3x3_c64.hip: bf16 3x3 stride-1 64 -> 64 channels, persistent workgroups with all nine taps resident in LDS
bool conv3x3_c64_applies(const ConvArgs &a);
hipError_t launch_conv3x3_c64(const ConvArgs &a, hipStream_t stream);
// bottleneck_block.hip: one identity bottleneck of conv2_x (1x1 256 -> 64, 3x3 64 -> 64, 1x1 64 -> 256 + x,
// ReLU after each, bf16) in a single launch; a1 / a2 / out may each be null (not stored)
struct BlockArgs {
    const void *x;                       // [M, 256] block input, also the shortcut ([M, 64] with a projection shortcut)
    void *a1, *a2, *out;                 // [M, 64], [M, 64], [M, 256]
    const void *w1, *w2, *w3;            // [64][256] ([64][64]), [64][3][3][64], [256][64]
    const float *s1, *h1, *s2, *h2, *s3, *h3;   // folded batch-norm scale / shift of the three layers
    int N, H, W, M;
    // projection shortcut (the first block of the stage): sc = ssc * (wsc . x) + hsc, added to the third layer
    int proj;
    const void *wsc;                     // [256][64]
    const float *ssc, *hsc;
    void *sc;                            // [M, 256] or nullptr: not stored
};
const char *bottleneck_block_check(const BlockArgs &a);
hipError_t launch_bottleneck_block(const BlockArgs &a, hipStream_t stream);
// attention.hip: fused multi-head self-attention, head dimension 64, bf16.  qkv [N,S,3*64*heads], ctx [N,S,64*heads]
const char *attention_check(const void *qkv, const void *ctx, int N, int S, int heads, int bf16);
int attention_waves(int N, int S, int heads);       // wavefronts (of 32 queries) per workgroup
hipError_t launch_attention(const void *qkv, void *ctx, int N, int S, int heads, int bf16, hipStream_t stream);
// transformer_ops.hip: layer normalisation over the last axis of [rows, C], bf16
const char *layernorm_check(const void *x, const void *y, const float *gamma, const float *beta, long long rows, int C,
                            int bf16);
hipError_t launch_layernorm(const void *x, void *y, const float *gamma, const float *beta, long long rows, int C,
                            float eps, int bf16, hipStream_t stream);
// opgranular_ops.hip: training-mode batch normalisation over [M, C] (bf16), ReLU, residual add
const char *bn_train_check(const void *x, const void *y, const float *gamma, const float *beta, long long M, int C,
                           int bf16);
size_t bn_train_scratch_bytes();
size_t bn_train_fwd_scratch_bytes();      // what the forward alone needs of it (any C up to 8192)
// What a segment does next with the result, element by element: y_add = result + r, y_relu = ReLU of that (or of the result).  Null: not there.
struct ElementwiseTail {
    const void *r = nullptr;
    void *y_add = nullptr, *y_relu = nullptr;
    bool bad() const { return !r != !y_add || (((uintptr_t)r | (uintptr_t)y_add | (uintptr_t)y_relu) & 15); }
};
hipError_t launch_bn_factors(const void *x, const float *gamma, const float *beta, long long M, int C, float eps, int bf16, void *scratch,
                             size_t scratch_bytes, hipStream_t stream);
hipError_t launch_bn_apply(const void *x, void *y, const float *beta, long long M, int C, int bf16, const ElementwiseTail &tail,
                           const void *scratch, hipStream_t stream);
hipError_t launch_bn_train_bwd(const void *x, const void *gy, void *gx, const float *gamma, float *gw, long long M, int C,
                               float eps, int bf16, const void *relu_y, void *gm, void *scratch, hipStream_t stream);
hipError_t launch_add_relu(const void *x, const ElementwiseTail &tail, size_t bytes, int bf16, hipStream_t stream);
hipError_t launch_relu(const void *x, void *y, size_t bytes, int bf16, hipStream_t stream);
hipError_t launch_add(const void *x, const void *r, void *y, size_t bytes, int bf16, hipStream_t stream);
// net_ops.hip: ResNet stem (7x7, stride 2, pad 3, 3 -> 64 channels, bf16), pooling, loss
bool stem_applies(const ConvArgs &a);
const char *stem_check(const ConvArgs &a);
hipError_t launch_stem(const ConvArgs &a, hipStream_t stream);
// stem_wgrad.hip: weight gradient of the stem
size_t stem_wgrad_workspace_bytes(const ConvArgs &a);
hipError_t launch_stem_wgrad(const ConvArgs &a, const void *g, float *gw, void *workspace, size_t workspace_bytes,
                             hipStream_t stream);

struct PoolArgs {
    const void *x;   // [N,H,W,C]
    void *y;         // [N,P,Q,C] (max) or [N,C] (global average)
    int N, H, W, C, R, S, stride, pad, P, Q;
    int bf16;
};
const char *pool_check(const PoolArgs &a, bool global_avg);
hipError_t launch_maxpool(const PoolArgs &a, hipStream_t stream);
hipError_t launch_avgpool(const PoolArgs &a, hipStream_t stream);
constexpr int kLossImages = 16384;          // most images whose losses the scratch of launch_softmax_ce holds (256 + 4 bytes each)
size_t softmax_ce_scratch_bytes(int N, int classes, int bf16);
hipError_t launch_softmax_ce(const void *logits, const void *labels, int N, int classes, int bf16, float *out, void *scratch,
                             hipStream_t stream);

// backward.hip: backward of the fused layer (bf16 weight gradient; data gradient through the
// forward kernels with transformed weights)
hipError_t launch_relu_mask(const void *y, const void *gy, void *out, size_t bytes, int bf16, hipStream_t stream);
hipError_t launch_relu_mask_dilate(const void *y, const void *gy, void *out, int N, int H, int W, int P, int Q, int K,
                                   int stride, int bf16, hipStream_t stream);
hipError_t launch_spread_add(const void *t, const void *add, const void *mask, void *out, int N, int H, int W, int P,
                             int Q, int C, int stride, int bf16, hipStream_t stream);
hipError_t launch_bwd_weights(const void *w, const float *scale, void *wt, int K, int R, int S, int C, int bf16,
                              hipStream_t stream);
const char *wgrad_check(const ConvArgs &a);            // nullptr when a weight-gradient kernel applies
const char *wgrad_kernel_name(const ConvArgs &a);
size_t wgrad_workspace_bytes(const ConvArgs &a);
// 3x3 stride-2 pad-1 layers, from the gradient at the output's resolution (a.x = x at the input's resolution, a.H, a.W,
// a.P, a.Q the layer's own)
bool wgrad_s2_applies(const ConvArgs &a);
size_t wgrad_s2_workspace_bytes(const ConvArgs &a);
hipError_t launch_wgrad_s2(const ConvArgs &a, const void *g, float *gw, void *workspace, size_t workspace_bytes,
                           hipStream_t stream);
hipError_t launch_wgrad(const ConvArgs &a, const void *g, float *gw, void *workspace, size_t workspace_bytes,
                        hipStream_t stream);

// wgrad1x1.hip, wgrad3x3.hip: the bf16 weight gradients (the layer's own geometry; g at the output's resolution)
int wgrad_splits(long long pixels, int tiles, double pixel_ns, double sums_ns);
const char *wgrad1x1_check(const ConvArgs &a);
size_t wgrad1x1_workspace_bytes(const ConvArgs &a);
hipError_t launch_wgrad1x1(const ConvArgs &a, const void *g, float *gw, void *workspace, size_t workspace_bytes, hipStream_t stream);
hipError_t launch_wgrad1x1_reduce(const float *partial, const float *scale, float *gw, int K, int C, int kt, int ct, int nsplit, hipStream_t stream);
const char *wgrad3x3_check(const ConvArgs &a);
size_t wgrad3x3_workspace_bytes(const ConvArgs &a);
hipError_t launch_wgrad3x3(const ConvArgs &a, const void *g, float *gw, void *workspace, size_t workspace_bytes, hipStream_t stream);

// joint1x1.hip: both gradients of a 1x1 stride-1 bf16 layer in one pass over its tensors (da: the data gradient's convolution, fa: the layer;
// add_even: da.res is known to hold zeros at every pixel of odd row or column)
bool joint1x1_applies(const ConvArgs &fa);
size_t joint1x1_workspace_bytes(const ConvArgs &fa);
bool joint1x1_masks(const ConvArgs &da, const ConvArgs &fa);     // whether it can make gpre = gy * [y > 0] on the way
hipError_t launch_joint1x1(const ConvArgs &da, const ConvArgs &fa, const void *g, const void *y, void *gpre, float *gw, void *workspace,
                           size_t workspace_bytes, bool add_even, hipStream_t stream);
// small_backward.hip: both gradients of a layer that cannot fill the chip in one launch (da: the data gradient's convolution
// or null for the weight gradient alone, fa: the layer as
// launch_wgrad or launch_wgrad_s2 takes it)
bool small_backward_applies(const ConvArgs *da, const ConvArgs &fa);
const char *small_backward_name(const ConvArgs &fa);
hipError_t launch_small_backward(const ConvArgs *da, const ConvArgs &fa, const void *g, float *gw, hipStream_t stream);

// backward_ops.hip: backward of pooling, the classifier and the loss (bf16)
// mask_x: gx is also multiplied by [x > 0] (the ReLU mask of the layer that produced the pool's input)
hipError_t launch_maxpool_bwd(const PoolArgs &a, const void *gy, void *gx, int mask_x, hipStream_t stream);
hipError_t launch_avgpool_bwd(const PoolArgs &a, const void *gy, void *gx, hipStream_t stream);
hipError_t launch_softmax_ce_bwd(const void *logits, const void *labels, int N, int classes, void *gz, hipStream_t stream);
hipError_t launch_dense_bwd(const void *x, const void *w, const float *scale, const void *gy, void *gx, float *gw,
                            int N, int Cin, int Cout, hipStream_t stream);

hipError_t launch_bn_fold(const float *gamma, const float *beta, const float *mean, const float *var,
                          float eps, unsigned C, float *scale, float *shift, hipStream_t stream);
hipError_t launch_copy(const void *src, void *dst, size_t bytes, hipStream_t stream);
hipError_t launch_mfma_probe(float *out, int iters, int blocks, hipStream_t stream);

}  // namespace delta
