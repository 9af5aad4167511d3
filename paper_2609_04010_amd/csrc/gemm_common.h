// Device helpers shared by the GEMM kernels.
#pragma once

#include "kernels.h"
#include "mfma.h"

namespace dd {

// gelu_tanh(x) = 0.5 x (1 + tanh(y)) = x / (1 + exp(-2y)), y = sqrt(2/pi) (x + 0.044715 x^3), with
// exp(-2y) = 2^(x (a + b x^2)), a = -2 sqrt(2/pi) log2(e), b = 0.044715 a: five VALU operations plus
// v_exp_f32 and v_rcp_f32 (about 1 ulp each; the result is rounded to bf16 afterwards)
DD_DEV float gelu_tanh(float x) {
    const float e = __builtin_amdgcn_exp2f(x * fmaf(x * x, -0.1029432395800235f, -2.302208198144325f));
    return x * __builtin_amdgcn_rcpf(1.0f + e);
}

// the same for fp32 results
DD_DEV float gelu_tanh_f32(float x) {
    return 0.5f * x * (1.0f + tanhf(0.7978845608028654f * (x + 0.044715f * x * x * x)));
}

constexpr int BK = 64;   // K depth of an operand tile

// EPI_GATE row factor of output row m (m % gate_period is in range for any m, clamped rows too)
DD_DEV float gate_row_scale(const GemmArgs& g, int m) {
    if (!g.gate) return g.gate_scale;
    return g.gate[m % g.gate_period] != 0 ? g.gate_scale : 0.f;
}

// Tiles of the ring kernel (k_gemm_ring.hip): 128 x 128 (four stages, one workgroup of eight
// wavefronts per CU), 64 x 64 with four stages (two workgroups of four wavefronts per CU) or three
// stages (three per CU), 32 x 32 with K over the four wavefronts, and (fp32) 32 x 64 with K over two
// pairs of wavefronts, and 128 x 192 with three stages (one workgroup of eight wavefronts per CU)
enum RingTile { RING_128 = 0, RING_64_DEEP = TILE_TAIL, RING_64 = 2, RING_32K = TILE_32K, RING_32X64 = 12,
                RING_128X192 = 13 };
void launch_gemm_ring(int dtype, RingTile tile, int epi, const GemmArgs& g, hipStream_t s);
double gemm_ring_us(RingTile tile, int64_t M, int64_t N, int64_t K, int splits, int cus);

}  // namespace dd
