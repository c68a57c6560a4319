// What the two contraction kernels' epilogues have in common.
#pragma once

#include "dgq_internal.h"

namespace dgq {

// GELU(t) = t * Phi(t).  Phi through the rational approximation 7.1.26 of Abramowitz and
// Stegun for erfc: with z = |t| / sqrt 2 and u = 1 / (1 + p z),
//     erfc(z) = (a1 u + a2 u^2 + a3 u^3 + a4 u^4 + a5 u^5) exp(-z^2),   |error| <= 1.5e-7,
// so Phi(t) = erfc(z) / 2 for t < 0 (no cancellation in the lower tail) and 1 - erfc(z) / 2
// otherwise: absolute error of Phi below 1e-7 plus fp32 rounding, at a third of the
// instructions of the library erf (which made the fused epilogue slower than the plain one).
__device__ inline float gelu(float t) {
    const float z = fabsf(t) * 0.70710678118654752f;
    const float u = __builtin_amdgcn_rcpf(fmaf(0.3275911f, z, 1.0f));
    float pl = fmaf(1.061405429f, u, -1.453152027f);
    pl = fmaf(pl, u, 1.421413741f);
    pl = fmaf(pl, u, -0.284496736f);
    pl = fmaf(pl, u, 0.254829592f);
    pl = pl * u;
    // exp(-z^2) = 2^(-t^2 / 2 * log2 e)
    const float e = __builtin_amdgcn_exp2f(t * t * -0.72134752044448170f);
    const float half_erfc = 0.5f * pl * e;
    const float phi = t < 0.0f ? half_erfc : 1.0f - half_erfc;
    return t * phi;
}

// The 3 x 3 convolution's gathered taps (stride 1, zero padding 1).  `codes` holds three
// copies of the map's code tensor, copy c at codes + c * copy_bytes: copy 1 is the map itself,
// copy 0 / copy 2 hold in row r the code row of the pixel to the left / right of r (the code of
// the value 0 where the image ends).  Tap t = 3 (dy + 1) + (dx + 1) of a 16-row (32-row) block
// of output pixels is then the block dy image rows further in copy dx + 1 -- contiguous 1 KiB
// pieces, one per chunk, as for a linear layer -- or, outside the image, a block of the code of 0
// (fill: one 1 KiB block per chunk).  Needs the image width to be a multiple of the rows of a
// block.  The K' order is tap-major, K' = 9 K'_map.
struct ConvGather {
    int32_t w_blocks = 0;    // image width / rows per code block
    int32_t height = 0;      // image height
    int32_t chunks = 0;      // chunks per tap (K'_map / 64)
    int64_t copy_bytes = 0;  // bytes of one copy of the code tensor
    const int8_t *fill = nullptr;
};

// What the choice of a contraction kernel depends on.
struct LinearShape {
    int64_t rows, out_channels;
    int32_t n_chunks, n_groups;
    int gated;         // 0, 1 gated epilogue, 2 gated and requantized
    bool conv, multi;  // gathered taps, more than two pixel classes
};

// Tile of the ring kernel (k2_linear.hip): 0 64 x 64, 1 64 x 128 behind four stages, 2 64 x 128 behind three, 3 128 x 128.
int ring_shape(const LinearShape &s);

// The contraction for launches the chip is not full of (k2_direct.hip): the block of outputs per wavefront (0: 16 x 16, 1: 16 x
// 32, 2: 32 x 32; gated 32 x 16), or -1 where the ring kernel is the faster one.
int direct_block(const LinearShape &s);
// arguments as for launch_linear, cv for a gathered convolution
hipError_t launch_linear_direct(int block, const Groups &g, const Weight &w, const int8_t *codes,
                                const uint8_t *row_class, int64_t rows, float *y, int geglu,
                                uint8_t *rq_cls, const ConvGather *cv, int32_t *acc_dump,
                                hipStream_t st);

}  // namespace dgq
