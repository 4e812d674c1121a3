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
//  * residual and mask are requested before the first step, scale and shift too, straight into LDS: requested where they are needed they
//    were one more round trip to memory at the end (three fp32 bottlenecks, 21 launches with it: 177 -> 173 us; an encoder layer of 1 x 77, four: 41.4 -> 40.1).
// Operands are re-read from the L1 / L2 by every tile that needs them (64 FLOP per byte loaded), which
// is what ends the kernel's range: see splitk_applies for where the lines lie and what both sides measured.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"
#include "splitk_tile.hpp"

namespace delta {
namespace splitk {

template <bool BF16, int KW, int AHEAD, bool SPREAD>
__global__ __launch_bounds__(KW * 64) void conv_splitk_kernel(ConvArgs a, int tiles_m, int tiles_n, int pixels_first,
                                                              Divisors inv) {
    __shared__ __align__(16) unsigned char smem[KW * kWaveLds];
    __shared__ __align__(16) float factors[64];
    conv_tile<BF16, KW, AHEAD, SPREAD>(a, tiles_m, tiles_n, pixels_first, inv, xcd_run(blockIdx.x, gridDim.x), threadIdx.x, smem, factors);
}

template <bool BF16, int KW, int AHEAD>
hipError_t launch(const ConvArgs &a, hipStream_t stream) {
    const int tiles_m = (a.M + kTile - 1) / kTile, tiles_n = (a.Cout + kTile - 1) / kTile;
    const dim3 grid((unsigned)tiles_m * (unsigned)tiles_n), block(KW * 64);
    if (a.spread) conv_splitk_kernel<BF16, KW, AHEAD, true><<<grid, block, 0, stream>>>(a, tiles_m, tiles_n, weights_larger(a), divisors_of(a));
    else conv_splitk_kernel<BF16, KW, AHEAD, false><<<grid, block, 0, stream>>>(a, tiles_m, tiles_n, weights_larger(a), divisors_of(a));
    return hipGetLastError();
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
