// Per-chunk solve with float32 products (v_mfma_f32_16x16x4_f32): chunk-wise Frobenius norms (Section 4.2.1), Algorithm
// 1 on all tokens of the chunk at once and the readout of Eq. (CH), for d = 64, 128 and 256, float32 or bf16 tensors.
// The mathematics is that of gka_chunk_solve.hip (bf16 products), whose header derives the split
//
//   (H_c x_c) = zeta_c (H_[n] x_c) + sum_{j<=c} M[j,c] k_j (k_j . x_c)
//
// and the residual form of the recurrence. What differs is the shape: a float32 product takes sixteen times the matrix
// pipe's time of a bf16 one, so everything here serves the pipe.
//   * A workgroup takes TT = 1 or 2 tiles of 16 tokens of one chunk (4 / TT workgroups per chunk). Wave w owns the feature
//     rows 16 RT w .. of every vector, for all of the workgroup's tokens: no product is computed twice, and the state's
//     rows of a wave stay in its registers for all passes (RT D / 4 registers; a pass reads no state from memory or LDS).
//   * Tokens sit on the N dimension: lane (n, kg) = (lane & 15, lane >> 4) holds rows 4 kg .. + 3 of token n of a tile,
//     so per-token scalars are per-lane scalars. Vectors cross waves through LDS rows [token][feature]; a lane reads
//     four consecutive features 16 s + 4 kg .. + 3 at once and uses them in four products (the contraction index is
//     enumerated in that order by both operands).
//   * Key products P = K delta^T are dealt out by 16 x 16 tiles (causal ones only) over the waves ahead of the state
//     product, which does not need them: the barrier that publishes P waits for no one.
// Bound: the matrix pipe (157 TFLOP/s in float32). Measured, microseconds per forward pass, against 32 x 32 x 2 products
// with two waves per token block that each formed all of P, H_[n] in LDS, one workgroup per chunk: d = 64, 1 pair x 256
// tokens 62 -> 32; d = 64, 64 x 1024 205 -> 163; d = 128, 16 x 1500 309 -> 197; d = 128, 64 x 1024 664 -> 436
// (98 TFLOP/s). d = 256, 32 x 1024 float32 tensors against the token-by-token kernel: 16220 -> 724, of which this kernel 600 (the
// matrix pipe busy 75 % of it); bf16 tensors there: gka_solve_wide.hip. Registers: capped at 128 up to d = 128 (four waves per SIMD), at 256 at d = 256 (two). With
// TT = 2 that spills: d = 128 3 (bf16 tensors), 14 (float32), 12 to 29 with the variants or two right-hand sides; d = 256
// 15 (bf16), 31 (float32), up to 57 with the variants; d = 64 16 with the variants of float32 tensors. With TT = 1 none.
#include "gka_solve_shared.hpp"

namespace gka {

template <int D, int TT>
struct SolveF32Shape {
    static constexpr int NW = D == 64 ? 4 : 8;         // waves
    static constexpr int NTHR = 64 * NW;
    static constexpr int RT = D / (16 * NW);           // row tiles of 16 features per wave
    static constexpr int KS = D / 16;                  // steps of 16 features (four products) of a contraction
    static constexpr int TB = 4 / TT;                  // workgroups per chunk
    static constexpr int NUNITS = TT == 2 ? 7 : 4;   // causal (key tile, token tile) pairs, at most
    static constexpr int MAXU = (NUNITS + NW - 1) / NW;             // ... per wave
    static constexpr size_t k_bytes = (size_t)kChunk * (D + 4) * 4;
    static constexpr size_t x_bytes = (size_t)16 * TT * (D + 4) * 4;
    static constexpr size_t p_bytes = (size_t)16 * TT * (kChunk + 4) * 4;
    static constexpr size_t lds_bytes = k_bytes + x_bytes + p_bytes;
    static_assert(NormScratch<NW>::bytes <= x_bytes, "the scratch of the norm fits the operand rows");
};

// float4 index of columns 4 c4 .. + 3 of a row in a tile of rows of W floats. Rows are padded by 16 bytes: sixteen rows at
// the same columns, or four rows' sixteen columns, fall into different banks, and every access of a lane is an
// immediate offset from one address (an XOR swizzle made the compiler keep fifty addresses in registers: 162 of them
// at d = 128 with TT = 2, one workgroup per CU).
template <int W>
__device__ __forceinline__ int row4(int row, int c4) { return row * (W / 4 + 1) + c4; }
template <int W>
__device__ __forceinline__ int row1(int row, int col) { return row * (W + 4) + col; }

__device__ __forceinline__ f32x4 mma4(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
// sum over the four lanes that hold the rows of one token
__device__ __forceinline__ float sum_kg(float x)
{
    x += __shfl_xor(x, 16, 64);
    return x + __shfl_xor(x, 32, 64);
}

// MODE as in gka_chunk_solve.hip: 0 plain, 1 (GATED) with the layer's variants, 2 (DUAL) solve only for two right-hand
// sides one after the other (the backward pass).
template <class IO, int D, int TT, int MODE>
__device__ __forceinline__ void solve_f32_body(const SolveArgs &a)
{
    typedef SolveF32Shape<D, TT> SH;
    constexpr bool GATED = MODE != 0, DUAL = MODE == 2;
    constexpr int NW = SH::NW, NTHR = SH::NTHR, RT = SH::RT, KS = SH::KS, TB = SH::TB, MAXU = SH::MAXU;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    f32x4 *sK = (f32x4 *)smem;                         // k rows (later v rows) of the chunk, [64][D]
    f32x4 *sX = (f32x4 *)(smem + SH::k_bytes);         // operand rows [16 TT][D]
    f32x4 *sP = (f32x4 *)(smem + SH::k_bytes + SH::x_bytes);   // masked key products [16 TT][64]
    // scratch of the norm, in the operand rows
    const NormScratch<NW> norm(sX);

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, kg = lane >> 4;
    // the later token tiles of a chunk see more keys: their workgroups start first. Consecutive workgroups take the
    // same chunk of consecutive pairs (in the [B,T,H,d] layout the heads of a token are adjacent).
    const int per_tb = a.n_pairs * a.n_chunks;
    const int tb = TB - 1 - a.skip_blocks - (int)blockIdx.x / per_tb;
    const int within = (int)blockIdx.x % per_tb;
    const int pair = within % a.n_pairs, chunk_local = within / a.n_pairs;
    const int chunk = a.chunk0 + chunk_local;
    const int b = (a.pair0 + pair) / a.H, h = (a.pair0 + pair) % a.H;
    const int64_t chunk_id = (int64_t)chunk_local * a.n_pairs + pair;
    const int64_t base_bh = (int64_t)b * a.stride_b + (int64_t)h * a.stride_h;
    const int64_t gate_base = (int64_t)b * a.T * a.H + h;
    const int tok0 = chunk * kChunk;
    if (tok0 + 16 * TT * tb >= a.T) return;            // (whole workgroup) only padding
    const int JT = TT * (tb + 1);                      // key tiles in sight
    const bool solve = !(GATED && !DUAL && a.readout_only);
    const bool stated = chunk > 0 || a.init_states;    // else H_[n] = U_[n] = 0: nothing to read or multiply

    // ---------------- requests: gates, k rows, state rows, q ----------------
    const int64_t gate_at = gate_base + (int64_t)min(tok0 + lane, a.T - 1) * a.H;
    const float gm = a.gate[gate_at];
    float ball = 1.0f;                                 // lane j: write gate beta_j
    if constexpr (GATED) {
        const float raw = (a.beta ? a.beta : a.gate)[gate_at];
        ball = a.beta ? raw : 1.0f;
    }
    constexpr int RPI = NTHR / (D / 4), NP = kChunk / RPI;      // rows per sweep of the workgroup, sweeps
    typename IO::raw4 rows[NP];
    auto load_rows = [&](const void *x) {
#pragma unroll
        for (int i = 0; i < NP; ++i)
            if (i * RPI < 16 * JT)
                rows[i] = IO::load_raw4(x, base_bh + (int64_t)min(tok0 + i * RPI + tid / (D / 4), a.T - 1) * a.stride_t +
                                               4 * (tid % (D / 4)));
    };
    auto store_rows = [&]() {                          // rows beyond the sequence are zero
#pragma unroll
        for (int i = 0; i < NP; ++i)
            if (i * RPI < 16 * JT) {
                const int row = i * RPI + tid / (D / 4);
                f32x4 x = IO::cvt4(rows[i]);
                if (tok0 + row >= a.T) x = zero4();
                sK[row4<D>(row, tid % (D / 4))] = x;
            }
    };
    load_rows(a.k);
    // A fragments of this wave's rows of a state: element [16 rt + n][16 s + 4 kg + e] of the state in sreg[rt][s][e]
    f32x4 sreg[RT][KS];
    auto load_state = [&](const void *ws) {
        const f32x4 *src = (const f32x4 *)ws + chunk_id * (D * D / 4) + (int64_t)w * RT * KS * 64 + lane;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int s = 0; s < KS; ++s) sreg[rt][s] = stated ? src[(rt * KS + s) * 64] : zero4();
    };
    int c_loc[TT];                                     // this lane's tokens
    int64_t tok_off[TT];
    bool valid[TT];
    f32x4 qv[RT][TT];
    float lam[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
        c_loc[tt] = 16 * (TT * tb + tt) + n;
        valid[tt] = tok0 + c_loc[tt] < a.T;
        const int tok = min(tok0 + c_loc[tt], a.T - 1);
        tok_off[tt] = base_bh + (int64_t)tok * a.stride_t + 16 * RT * w + 4 * kg;
        lam[tt] = ((!GATED || a.lambda) ? a.lambda : a.gate)[gate_base + (int64_t)tok * a.H];
    }
    auto load_q = [&](const void *x, int rt, int tt) {
        const f32x4 v = IO::load4(x, tok_off[tt] + 16 * rt);
        return valid[tt] ? v : zero4();
    };
    auto load_rhs = [&]() {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) qv[rt][tt] = load_q(a.q, rt, tt);
    };
    if constexpr (D != 256) load_rhs();                // (d = 256: the norm needs the registers)
    float hn2 = 0.0f;
    if (solve) {
        load_state(a.ws_H);
        constexpr int NHN = (D / 32) * (D / 32);       // partial sums of ||H_[n]||^2
        if (stated) hn2 = wave_sum(lane < NHN ? a.ws_hn[chunk_id * NHN + lane] : 0.0f);
    }

    // ---------------- decays (Section 4.2.1; log-space form of Appendix B.2, base 2) ----------------
    const float Gall = wave_inclusive_scan((tok0 + lane < a.T) ? log2_gate(gm) : 0.0f, lane);
    float zeta[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) zeta[tt] = exp2f(__shfl(Gall, c_loc[tt], 64));
    auto mask4 = [&](int jt, int c, bool strict) { return mask_rows<GATED>(Gall, ball, kg, jt, c, strict); };
    // this wave's (key tile, token tile) pairs of the masked key products
    int unit_j[MAXU], unit_t[MAXU];                    // token tile TT: no such pair
    f32x4 unit_m[MAXU];
#pragma unroll
    for (int i = 0; i < MAXU; ++i) {
        int u = i * NW + w, tt = 0, len = TT * tb + 1;
        while (tt < TT && u >= len) { u -= len; ++tt; ++len; }
        unit_j[i] = u;
        unit_t[i] = tt;
        unit_m[i] = tt < TT ? mask4(u, 16 * (TT * tb + tt) + n, false) : zero4();
    }
    store_rows();
    lds_barrier();

    // [16 rows of K, tile jt] x [16 rows of X, tile xt]^T over all features
    auto key_product = [&](int jt, const f32x4 *X, int xt) {
        f32x4 c0 = zero4(), c1 = zero4();              // two chains of dependent products
#pragma unroll 4
        for (int s = 0; s < KS; ++s) {
            const f32x4 ka = sK[row4<D>(16 * jt + n, 4 * s + kg)], xb = X[row4<D>(16 * xt + n, 4 * s + kg)];
            c0 = mma4(ka[0], xb[0], c0);
            c1 = mma4(ka[1], xb[1], c1);
            c0 = mma4(ka[2], xb[2], c0);
            c1 = mma4(ka[3], xb[3], c1);
        }
        return c0 + c1;
    };

    // ---------------- chunk-wise Frobenius norm (gka_solve_shared.hpp) ----------------
    float fro[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) fro[tt] = 0.0f;
    if (solve) {
        for (int jt = 0; jt < JT; ++jt) {
            float part = 0.0f;
            if (stated) {
                f32x4 acc[RT];
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) acc[rt] = zero4();
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    const f32x4 kb = sK[row4<D>(16 * jt + n, 4 * s + kg)];
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int rt = 0; rt < RT; ++rt) acc[rt] = mma4(sreg[rt][s][e], kb[e], acc[rt]);
                }
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    const f32x4 kr = sK[row4<D>(16 * jt + n, 4 * (RT * w + rt) + kg)];
#pragma unroll
                    for (int r = 0; r < 4; ++r) part += acc[rt][r] * kr[r];
                }
                part = sum_kg(part);
            }
            if (kg == 0) norm.sA[w * 64 + 16 * jt + n] = part;
        }
        for (int u0 = w; u0 < JT * (JT + 1) / 2; u0 += NW) {
            int it = u0, jt = 0;
            while (it > jt) { ++jt; it -= jt; }        // tile it <= jt of the lower triangle, row by row
            const f32x4 G = key_product(it, sK, jt);
            const f32x4 m = mask4(it, 16 * jt + n, true);
            float bp = 0.0f, dp = 0.0f;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float g2 = G[r] * G[r];
                bp += m[r] * g2;
                dp += (4 * kg + r == n) ? g2 : 0.0f;
            }
            bp = sum_kg(bp);
            dp = sum_kg(dp);
            if (kg == 0) {
                norm.sB[it * 64 + 16 * jt + n] = bp;
                if (it == jt) norm.sDg[16 * jt + n] = dp;
            }
        }
        sum_norm_terms<NW, GATED>(norm, tid, w, JT, Gall, ball);
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            float fs = 0.0f;
#pragma unroll
            for (int i = 0; i < NW; ++i) fs += norm.sF[i * 64 + c_loc[tt]];
            fro[tt] = sqrtf(fmaxf(zeta[tt] * zeta[tt] * hn2 + fs, 0.0f));
            if (a.fro_out && valid[tt] && w == 0 && kg == 0)
                a.fro_out[gate_base + (int64_t)(tok0 + c_loc[tt]) * a.H] = fro[tt];
        }
        lds_barrier();                                 // the scratch becomes the operand rows
    }

    // ---------------- Chebyshev iteration (Algorithm 1), residual form ----------------
    if constexpr (D == 256) load_rhs();
    float s0[TT], rho2[TT], omega[TT];
    f32x4 xi[RT][TT], dl[RT][TT], gS[RT][TT], gI[RT][TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
        if (GATED && !a.lambda) lam[tt] = a.lambda_scale * fro[tt];     // Section 4.1: lambda_t = a ||H_t||_F
        if (!valid[tt] || !solve) lam[tt] = 1.0f;
        const float L = fro[tt] + lam[tt], mu = lam[tt];                // Section 4.1
        s0[tt] = 2.0f / (L + mu);
        const float rho = (L - mu) / (L + mu);
        rho2[tt] = rho * rho;
        omega[tt] = 2.0f;
    }
    auto publish = [&](const f32x4 (&x)[RT][TT]) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) sX[row4<D>(16 * tt + n, 4 * (RT * w + rt) + kg)] = x[rt][tt];
    };
    // acc += S X^T for this wave's rows of the state in sreg
    auto state_product = [&](f32x4 (&acc)[RT][TT]) {
        if (!stated) return;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            f32x4 xb[TT];
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) xb[tt] = sX[row4<D>(16 * tt + n, 4 * s + kg)];
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int tt = 0; tt < TT; ++tt) acc[rt][tt] = mma4(sreg[rt][s][e], xb[tt][e], acc[rt][tt]);
        }
    };
    auto masked_key_products = [&]() {
#pragma unroll
        for (int i = 0; i < MAXU; ++i)
            if (unit_t[i] < TT)
                sP[row4<kChunk>(16 * unit_t[i] + n, 4 * unit_j[i] + kg)] =
                    key_product(unit_j[i], sX, unit_t[i]) * unit_m[i];
    };
    // acc += A^T (P o M) for this wave's rows, A = the rows in sK
    auto intra_product = [&](f32x4 (&acc)[RT][TT]) {
        const float *rowsf = (const float *)sK;
#pragma unroll
        for (int jt = 0; jt < 4; ++jt) {
            if (jt >= JT) break;
            float at[RT][4];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int e = 0; e < 4; ++e) at[rt][e] = rowsf[row1<D>(16 * jt + 4 * kg + e, 16 * (RT * w + rt) + n)];
#pragma unroll
            for (int tt = 0; tt < TT; ++tt)
                if (jt <= TT * tb + tt) {
                    const f32x4 pb = sP[row4<kChunk>(16 * tt + n, 4 * jt + kg)];
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int rt = 0; rt < RT; ++rt) acc[rt][tt] = mma4(at[rt][e], pb[e], acc[rt][tt]);
                }
        }
    };
    for (int rhs = 0; rhs < (DUAL ? 2 : 1); ++rhs) {
    if (DUAL && rhs == 1) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) {
                qv[rt][tt] = load_q(a.q2, rt, tt) + load_q(a.q2_lo, rt, tt);
                omega[tt] = 2.0f;
            }
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            gS[rt][tt] = zero4();
            gI[rt][tt] = -qv[rt][tt];
            dl[rt][tt] = xi[rt][tt] = s0[tt] * qv[rt][tt];              // xi_0 = 2 q / (L + mu)
        }
    for (int it = 0; it < a.n_iter; ++it) {
        publish(dl);
        lds_barrier();                                 // delta visible; the masked products of the last pass are used up
        masked_key_products();
        state_product(gS);
        lds_barrier();
        intra_product(gI);
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            omega[tt] = 4.0f / (4.0f - rho2[tt] * omega[tt]);           // weight schedule
            const float cm = omega[tt] - 1.0f, cs = -omega[tt] * s0[tt];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float res = zeta[tt] * gS[rt][tt][r] + gI[rt][tt][r] + lam[tt] * xi[rt][tt][r];   // -r_{i-1}
                    dl[rt][tt][r] = cm * dl[rt][tt][r] + cs * res;
                    xi[rt][tt][r] += dl[rt][tt][r];
                }
        }
    }
    if (GATED && a.xhat_out) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int tt = 0; tt < TT; ++tt)
                if (valid[tt]) {
                    const int64_t e = (gate_base + (int64_t)(tok0 + c_loc[tt]) * a.H) * D + 16 * (RT * w + rt) + 4 * kg;
                    *(f32x4 *)((DUAL && rhs == 1 ? a.xhat2_out : a.xhat_out) + e) = xi[rt][tt];
                    if constexpr (DUAL)
                        store_value_remainder(rhs == 0 ? a.xhat_hi : a.xhat2_hi, rhs == 0 ? a.xhat_lo : nullptr, e, xi[rt][tt]);
                }
    }
    }                                                  // (right-hand sides)
    if constexpr (DUAL) return;

    // ---------------- readout y_c = zeta_c U_[n] x_c + sum_{j<=c} m[j,c] v_j (k_j . x_c) ----------------
    if (GATED && a.solve_only) return;                 // (whole workgroup)
    load_state(a.ws_U);
    load_rows(a.v);
    if (GATED && a.alpha) {                            // alpha-connection (Section 4.3)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            const float al = a.alpha[gate_base + (int64_t)min(tok0 + c_loc[tt], a.T - 1) * a.H];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) xi[rt][tt] = al * xi[rt][tt] + (1.0f - al) * load_q(a.q, rt, tt);
        }
    }
    publish(xi);
    lds_barrier();
    masked_key_products();
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) gS[rt][tt] = zero4();
    state_product(gS);
    lds_barrier();                                     // every wave is done with the keys
    store_rows();
    lds_barrier();
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) gS[rt][tt] *= zeta[tt];
    intra_product(gS);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
            if (valid[tt])
                IO::store4(a.o, tok_off[tt] + 16 * rt, gS[rt][tt][0], gS[rt][tt][1], gS[rt][tt][2], gS[rt][tt][3]);
}

template <class IO, int D, int TT, int MODE>
__global__ __launch_bounds__((SolveF32Shape<D, TT>::NTHR)) __attribute__((amdgpu_waves_per_eu(D == 256 ? 2 : 4))) void
solve_f32_kernel(SolveArgs a)
{
    solve_f32_body<IO, D, TT, MODE>(a);
}

template <class IO, int D, int TT, int MODE>
static hipError_t launch_solve_f32_t(const SolveArgs &a, hipStream_t stream)
{
    typedef SolveF32Shape<D, TT> SH;
    auto kern = solve_f32_kernel<IO, D, TT, MODE>;
    // (set once per kernel instantiation and device, not per launch)
    static bool attr_set_on[64] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64 || !attr_set_on[dev]) {
        e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)SH::lds_bytes);
        if (e != hipSuccess) return e;
        if (dev >= 0 && dev < 64) attr_set_on[dev] = true;
    }
    // A workgroup reads the rows of k and v of its chunk up to its own tokens. Outputs that replace them: the token blocks of a
    // chunk one launch after the other, the last ones first.
    const bool over_rows = !a.solve_only && (a.o == a.v || a.o == a.k);
    const int blocks = over_rows ? 1 : SH::TB;
    SolveArgs args = a;
    for (args.skip_blocks = 0; args.skip_blocks < SH::TB; args.skip_blocks += blocks) {
        hipLaunchKernelGGL(kern, dim3((unsigned)(a.n_pairs * a.n_chunks * blocks)), dim3(SH::NTHR), SH::lds_bytes, stream, args);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <class IO, int D, int MODE>
static hipError_t launch_solve_f32_d(const SolveArgs &a, hipStream_t stream)
{
    // Tokens per workgroup (16 TT): small workgroups spread a small problem over the chip, large ones repeat less of the
    // norm and share operand reads. Measured (whole forward pass, microseconds, TT = 1 / 2): d = 64: 64 chunks 35 / 46,
    // 256 chunks 62 / 64, 512 chunks 112 / 104; d = 128: 20 chunks 49 / 71, 160 chunks 102 / 112, 256 chunks 141 / 129,
    // 1024 chunks 472 / 436; d = 256: 20 chunks 119 / 181, 88 chunks 210 / 209, 160 chunks 240 / 227, 512 chunks 834 / 724.
    // (TT = 4 at d = 128, 1024 chunks: 460; at d = 256 the state rows leave no registers for it.)
    const int64_t chunks = (int64_t)a.n_pairs * a.n_chunks;
    // (gka_solve_wide.hip: one round of workgroups either way up to 64 and 128 chunks. Whole forward pass, TT = 1 / 2: 20 chunks
    // 57 / 79, 64 chunks 68 / 91, 88 chunks 114 / 100, 128 chunks 106 / 93, 160 chunks 136 / 133, 512 chunks 399 / 347; with
    // float32 products 119, 134, 210, 193, 228, 717)
    if (solve_wide_takes(a, D, std::is_same<IO, IOBF16>::value)) return launch_solve_wide(a, chunks <= 64 ? 1 : 2, stream);
    if (chunks <= (D == 256 ? 96 : 192)) return launch_solve_f32_t<IO, D, 1, MODE>(a, stream);
    return launch_solve_f32_t<IO, D, 2, MODE>(a, stream);
}

template <class IO, int D>
static hipError_t launch_solve_f32_g(const SolveArgs &a, hipStream_t stream)
{
    if constexpr (D != 256) {
        if (a.q2) return launch_solve_f32_d<IO, D, 2>(a, stream);
    }
    if (a.beta || a.alpha || !a.lambda || a.xhat_out) return launch_solve_f32_d<IO, D, 1>(a, stream);
    return launch_solve_f32_d<IO, D, 0>(a, stream);
}

hipError_t launch_solve_f32(const SolveArgs &a, int d, bool io_bf16, hipStream_t stream)
{
    if (io_bf16) {
        if (d == 256) return launch_solve_f32_g<IOBF16, 256>(a, stream);
        if (d == 128) return launch_solve_f32_g<IOBF16, 128>(a, stream);
        return launch_solve_f32_g<IOBF16, 64>(a, stream);
    }
    if (d == 256) return launch_solve_f32_g<IOF32, 256>(a, stream);
    if (d == 128) return launch_solve_f32_g<IOF32, 128>(a, stream);
    return launch_solve_f32_g<IOF32, 64>(a, stream);
}

}  // namespace gka
