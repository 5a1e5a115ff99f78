// What the solves of gka_solve_f32.hip and gka_solve_wide.hip have in common, whatever their products are made of: the masks and the
// end of the chunk-wise Frobenius norm
//
//   ||H_c||^2 = zeta_c^2 ||H_[n]||^2 + sum_{j<=c} m[j,c]^2 w_j,
//   w_j = 2 (zeta_j k_j^T H_[n] k_j + sum_{i<j} m[i,j] G_ij^2) / beta_j + G_jj^2,  G = K K^T
//
// (Section 4.2.1; the folded three-term expansion, see gka_chunk_solve.hip). Tokens sit on the N dimension: lane (n, kg) =
// (lane & 15, lane >> 4) holds rows 4 kg .. + 3 of token n of a tile.
#pragma once
#include "gka_device.hpp"
#include "gka_kernels.hpp"

namespace gka {

__device__ __forceinline__ f32x4 zero4() { return f32x4{0.0f, 0.0f, 0.0f, 0.0f}; }

// beta_j M[j,c] for rows j = 16 jt + 4 kg + r and the column c; strict: j < c. Lane j holds Gall = log2 zeta_j and ball = beta_j.
template <bool GATED>
__device__ __forceinline__ f32x4 mask_rows(float Gall, float ball, int kg, int jt, int c, bool strict)
{
    const float Gc = __shfl(Gall, c, 64);
    f32x4 m;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int j = 16 * jt + 4 * kg + r;
        float x = __builtin_amdgcn_exp2f(Gc - __shfl(Gall, j, 64));
        if constexpr (GATED) x *= __shfl(ball, j, 64);
        m[r] = (strict ? j < c : j <= c) ? x : 0.0f;
    }
    return m;
}

// Scratch of the norm in LDS.
template <int NW>
struct NormScratch {
    static constexpr size_t bytes = (2 * NW + 6) * 64 * 4;
    float *sA;                                         // [NW][64] k_j^T H k_j, a wave's rows
    float *sB;                                         // [4][64]  sum of m[i,j] G_ij^2 over a tile of i
    float *sDg;                                        // [64]     G_jj^2
    float *sW;                                         // [64]     w_j
    float *sF;                                         // [NW][64] sum of m[j,c]^2 w_j over a wave's share of j
    __device__ __forceinline__ explicit NormScratch(void *lds)
        : sA((float *)lds), sB(sA + NW * 64), sDg(sB + 4 * 64), sW(sDg + 64), sF(sW + 64) {}
};

// From sA, sB and sDg of the JT key tiles in sight to sF: lane c of wave w adds up its share of m[j,c]^2 w_j (all waves of the
// workgroup).
template <int NW, bool GATED>
__device__ __forceinline__ void sum_norm_terms(const NormScratch<NW> &s, int tid, int w, int JT, float Gall, float ball)
{
    const int lane = tid & 63;
    lds_barrier();
    if (tid < 16 * JT) {                               // (the first wave: lane j = token j)
        float as = 0.0f, bs = 0.0f;
#pragma unroll
        for (int i = 0; i < NW; ++i) as += s.sA[i * 64 + tid];
        for (int i = 0; i <= tid >> 4; ++i) bs += s.sB[i * 64 + tid];
        const float cross = 2.0f * (exp2f(Gall) * as + bs);
        s.sW[tid] = GATED ? (ball > 0.0f ? cross / ball + s.sDg[tid] : 0.0f) : cross + s.sDg[tid];
    }
    lds_barrier();
    float f = 0.0f;                                    // lane c = token c; keys dealt out over the waves
#pragma unroll
    for (int i = 0; i < 64 / NW; ++i) {
        const int j = i * NW + w;
        if (j < 16 * JT) {
            float m = __builtin_amdgcn_exp2f(Gall - lane_value(Gall, j));
            if constexpr (GATED) m *= lane_value(ball, j);
            m = j <= lane ? m : 0.0f;
            f += m * m * s.sW[j];
        }
    }
    s.sF[w * 64 + lane] = f;
    lds_barrier();
}

}  // namespace gka
