// What the two bf16 matrix-product kernels share (the 256 x 256 tiles of jv_encoder.hip and the
// smaller tiles of jv_gemm_tiles.hip): the function behind GELU, the tile shapes, and the launchers of the latter.
#pragma once

#include "jv_common.h"
#include "jv_mfma.h"

namespace jv {

typedef __attribute__((address_space(3))) void lds_void;

// gelu(x) = x Phi(x), Phi the standard normal distribution function.  The epilogues read
// Phi from a table in LDS (kPhiSteps intervals on [-6, 6], linear interpolation: absolute error
// below 5e-6; outside the range Phi is 0 or 1 to 1e-9) that every workgroup builds for itself
// from  Phi(x) = 1 - erfc(x / sqrt 2) / 2,  erfc(z) = (a1 t + ... + a5 t^5) exp(-z^2),
// t = 1 / (1 + p z), z >= 0  (Abramowitz-Stegun 7.1.26, absolute error 1.5e-7).
constexpr int kPhiSteps = 1024;
constexpr float kPhiLo = -6.0f, kPhiStep = 12.0f / kPhiSteps;
__device__ inline float normal_cdf(float x) {
    const float z = fabsf(x) * 0.70710678118654752f;
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, z, 1.0f));
    const float poly = t * fmaf(t, fmaf(t, fmaf(t, fmaf(t, 1.061405429f, -1.453152027f), 1.421413741f),
                                        -0.284496736f), 0.254829592f);
    const float half_erfc = 0.5f * poly * __builtin_amdgcn_exp2f(-1.4426950408889634f * z * z);
    return x < 0.f ? half_erfc : 1.0f - half_erfc;
}

// table[2 i] = Phi(x_i), table[2 i + 1] = Phi(x_i+1) - Phi(x_i), x_i = kPhiLo + i kPhiStep, i < kPhiSteps; filled by
// `threads` threads, kPhiSteps / threads consecutive entries each.
__device__ inline void phi_table_fill(float *table, int tid, int threads) {
    const int n = kPhiSteps / threads;
    float p0 = normal_cdf(kPhiLo + (float)(tid * n) * kPhiStep);
    for (int i = tid * n; i < (tid + 1) * n; ++i) {
        const float p1 = normal_cdf(kPhiLo + (float)(i + 1) * kPhiStep);
        *(float2 *)(table + 2 * i) = float2{p0, p1 - p0};
        p0 = p1;
    }
}
__device__ inline float gelu_from_table(float x, const float *table) {
    const float t = __builtin_amdgcn_fmed3f(fmaf(x, 1.0f / kPhiStep, -kPhiLo / kPhiStep), 0.0f,
                                            (float)kPhiSteps - 0.004f);
    const float2 pd = *(const float2 *)(table + 2 * (unsigned)t);
    return x * fmaf(__builtin_amdgcn_fractf(t), pd.y, pd.x);
}

// Tile shapes (tokens x features): the kernel of jv_encoder.hip, then those of jv_gemm_tiles.hip
// (128 x 128 in two forms: a deep operand ring with one workgroup per compute unit, a short one
// with two).
enum GemmTile { kTile256x256 = 0, kTile256x128, kTile128x128Deep, kTile128x128, kTile64x128, kTile64x64, kTile256x192, kGemmTileShapes };

// y = epilogue(a w^T + bias) on tiles of shape `tile`, K split over k_split workgroups per tile
// (1: none; above 1 only with the plain epilogue and fp32 output: part p writes its sums
// y_split * p elements behind y).  Shapes and pointers as gemm_forward has checked them.
jv_status gemm_tiles_forward(GemmTile tile, int k_split, long long y_split, const void *a, const void *w,
                             const float *bias, const void *residual, void *y, int M, int N, int K, int lda,
                             int epi, bool out_bf16, hipStream_t stream);

// y = (((part 0 + part 1) + ...) + bias) + residual, K summed in `parts` parts of equal length, on
// tiles of kTile256x128, kTile128x128Deep or kTile64x128.
jv_status gemm_residual_parts(GemmTile tile, int parts, const void *a, const void *w, const float *bias, const void *residual, void *y,
                              int M, int N, int K, bool out_bf16, hipStream_t stream);

}  // namespace jv
