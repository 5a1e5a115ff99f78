// Per-chunk solve and readout at d = 256 for bf16 tensors: the work of gka_solve_f32.hip (whose header has the mathematics and
// the division of the work: TT tiles of 16 tokens of a chunk per workgroup, wave w owns feature rows 32 w .., the state's rows of
// a wave in its registers, vectors cross waves through LDS) with every float32 product replaced by products of 16-bit pieces
// that keep float32's precision, at an eighth to a fifth of the matrix pipe's time:
//   * states and vectors as two binary16 pieces, x s = hi + lo with a power of two s (22 bits of the largest element's scale and
//     of what is not much smaller; else within 2^-34 of the largest, 2^-29 for the updates): S x ~ Sh xh + Sl xh + Sh xl, what is left out is
//     2^-22 of the product, less than the rounding of a float32 sum of 256 terms. s is chosen per row of a state (largest
//     element to [2^9, 2^10); per wave, for its 32 rows, small rows beside large ones kept few digits), per token for the
//     solve's updates (largest element of the first to [2^4, 2^5): the passes may grow them, see kMaxPasses and kRescaleAbove)
//     and once more for the readout's operand.
//   * keys are one binary16 piece with a power of two per key for K x (two products; largest element to [2^14, 2^15): exact down to
//     2^-31 of it, below that within 2^-39 of it), and bf16 as stored for K^T (P o M) and V^T (P o M), whose other operand, the
//     masked products, is cut into three bf16 pieces (24 bits).
// Operands of all contractions over features sit in LDS as fragments of v_mfma_f32_16x16x32: lane (n, kg) = (lane & 15,
// lane >> 4), eight values, slot p <-> feature 32 s + 16 (p / 4) + 4 kg + p % 4. A wave's rows of a vector are one such
// fragment.
// Measured, 32 pairs x 1024 tokens, 10 passes, us: this kernel 299 in place of 610 with float32 products, the whole forward pass
// (with the state pass on pieces too) 724 -> 381; 4 pairs x 300 tokens 119 -> 57. Two thirds of a workgroup's time are its
// states on their way from memory (512 KiB, nothing beside it on the CU) and what surrounds the passes; a pass is 7.4 k
// cycles, of which the matrix pipe needs 4.4 k and LDS 3.2 k. Against the oracle: the solve's result 3.4e-7 -> 2.2e-7 (2-norm;
// 2.9e-6 both with lambda a hundredth), ||H_t||_F 3.5e-7 -> 2.5e-7, the output its own rounding both.
#include "gka_solve_shared.hpp"

namespace gka {

namespace {

constexpr int kWideD = 256, kWideWaves = 8, kWideThreads = 64 * kWideWaves;
constexpr int kSteps = kWideD / 32;                      // steps of 32 features of a contraction
constexpr int kRowStride = kWideD + MmaBF16::kRowPad;    // elements of a row of the tile that is read transposed

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));

template <int TT>
struct WideShape {
    static constexpr int TB = 4 / TT;                    // workgroups per chunk
    static constexpr int NUNITS = TT == 2 ? 7 : 4;       // causal (key tile, token tile) pairs, at most (one per wave)
    static constexpr size_t k_bytes = (size_t)4 * kSteps * 64 * 16;               // keys, binary16 fragments [jt][s][lane]
    static constexpr size_t row_bytes = (size_t)kChunk * kRowStride * 2;          // k rows, later v rows, bf16
    static constexpr size_t x_bytes = (size_t)TT * 2 * kSteps * 64 * 16;          // operand fragments [tt][hi, lo][s][lane]
    static constexpr size_t p_bytes = (size_t)TT * 2 * 3 * 64 * 16;               // masked products [tt][jb][piece][lane]
    static constexpr size_t tab_bytes = (kChunk + 2 * kWideWaves * 16 * TT + kWideD + 2 * 16 * TT) * 4;  // scales of keys, maxima of tokens, scales of state rows, flags
    static constexpr size_t lds_bytes = k_bytes + row_bytes + x_bytes + p_bytes + tab_bytes;
    static_assert(NormScratch<kWideWaves>::bytes <= x_bytes, "the scratch of the norm fits the operand fragments");
};

__device__ __forceinline__ f32x4 mma_h(f16x8 a, f16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x4 mma_b(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
// largest over the four lanes that hold the rows of one token
__device__ __forceinline__ float max_kg(float x)
{
    x = fmaxf(x, __shfl_xor(x, 16, 64));
    return fmaxf(x, __shfl_xor(x, 32, 64));
}
__device__ __forceinline__ float wave_max(float x)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x = fmaxf(x, __shfl_xor(x, off, 64));
    return x;
}
// The power of two that brings x > 0 into [2^e, 2^(e + 1)), as far as it and its inverse are normal (1 for x = 0).
__device__ __forceinline__ int scale_exponent(float x, int e)
{
    const int ex = (int)((__float_as_uint(x) >> 23) & 255u) - 127;
    return x > 0.0f ? max(-126, min(126, e - ex)) : 0;
}
__device__ __forceinline__ float pow2(int e) { return __uint_as_float((uint32_t)(e + 127) << 23); }
// eight values as two binary16 pieces
__device__ __forceinline__ void split_f16(f32x4 a, f32x4 b, f16x8 &hi, f16x8 &lo)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        hi[e] = (_Float16)a[e];
        hi[4 + e] = (_Float16)b[e];
        lo[e] = (_Float16)(a[e] - (float)hi[e]);
        lo[4 + e] = (_Float16)(b[e] - (float)hi[4 + e]);
    }
}
__device__ __forceinline__ u16x4 bits4(f32x4 x)
{
    return u16x4{f32_to_bf16_bits(x[0]), f32_to_bf16_bits(x[1]), f32_to_bf16_bits(x[2]), f32_to_bf16_bits(x[3])};
}

}  // namespace

// Passes up to which the updates stay in range: with the spectrum in [mu, L] the residuals never exceed the right-hand side in
// the 2-norm, so delta_i = (omega_i - 1) delta_{i-1} + omega_i 2 / (L + mu) r_{i-1}, omega_i < 2, is at most (2 i + 1) |delta_0|, at
// most 16 (2 i + 1) of its largest element, which is below 2^5: 2^9 (2 i + 1) < 65504.
constexpr int kMaxPasses = 60;
// A token whose update has an element above this in a pass has the next one scaled down by 2^kRescale. Systems of the layer hardly get
// there; from an initial state that is not positive semidefinite the updates grow, in the 2-norm at most sevenfold in a pass (A delta
// is at most (L + lambda) |delta|, the step 2 / (L + mu), omega < 2), in their largest element at most 16 times as much: below
// 2^9 * 112 < 65504, and by less than 2^kRescale.
constexpr float kRescaleAbove = 0x1p9f;
constexpr int kRescale = 8;

// GATED: the layer's variants (write gate, alpha-connection, lambda_t = a ||H_t||_F) and the solve's result as an output. GIVEN: the
// sequence starts from given states, which nobody has looked at: updates that grow are scaled down. (32 pairs x 1024 tokens 366 -> 373
// us with it; from zero states every H_t is positive semidefinite.)
template <int TT, bool GATED, bool GIVEN>
__global__ __launch_bounds__(kWideThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void solve_wide_kernel(SolveArgs a)
{
    typedef WideShape<TT> SH;
    typedef IOBF16 IO;
    constexpr int NW = kWideWaves, TB = SH::TB;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    f16x8 *sK = (f16x8 *)smem;
    uint16_t *sRow = (uint16_t *)(smem + SH::k_bytes);
    f16x8 *sX = (f16x8 *)(smem + SH::k_bytes + SH::row_bytes);
    bf16x8 *sP = (bf16x8 *)(smem + SH::k_bytes + SH::row_bytes + SH::x_bytes);
    float *sKs = (float *)((unsigned char *)sP + SH::p_bytes);                    // [64]
    float *sMax = sKs + kChunk;                                                   // [updates, readout][NW][16 TT]
    // scratch of the norm, in the operand fragments
    const NormScratch<NW> norm(sX);
    const PaddedRows at{kRowStride};

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, kg = lane >> 4;
    float *sScale = sMax + 2 * NW * 16 * TT + 32 * w;    // [NW][32] inverse scales of this wave's rows of a state
    int *sGrown = (int *)(sMax + 2 * NW * 16 * TT + kWideD);                      // [even, odd pass][16 TT] update above kRescaleAbove
    if (GIVEN && tid < 2 * 16 * TT) sGrown[tid] = 0;
    // The workgroups of a chunk read the same 512 KiB of states. They get block indices equal modulo 8, next to each other: the
    // same XCD, whose L2 then serves all but the first, at about the same time. (All of one token block before the next:
    // states read from HBM once for each,
    // 32 pairs x 1024 tokens 426 us per forward pass instead of 409; U_[n]'s lines asked for during the passes: 428.) Within a chunk the later tokens, which see more keys, come first.
    const int n_all = a.n_pairs * a.n_chunks, blocks = a.skip_blocks < 0 ? TB : 1;
    const int group = (int)blockIdx.x / (8 * blocks), in_group = min(8, n_all - 8 * group);
    const int rest = (int)blockIdx.x - group * 8 * blocks;
    const int tb = TB - 1 - max(a.skip_blocks, 0) - rest / in_group;
    const int within = 8 * group + rest % in_group;
    const int pair = within % a.n_pairs, chunk_local = within / a.n_pairs;
    const int chunk = a.chunk0 + chunk_local;
    const int b = (a.pair0 + pair) / a.H, h = (a.pair0 + pair) % a.H;
    const int64_t chunk_id = (int64_t)chunk_local * a.n_pairs + pair;
    const int64_t base_bh = (int64_t)b * a.stride_b + (int64_t)h * a.stride_h;
    const int64_t gate_base = (int64_t)b * a.T * a.H + h;
    const int tok0 = chunk * kChunk;
    if (tok0 + 16 * TT * tb >= a.T) return;              // (whole workgroup) only padding
    const int JT = TT * (tb + 1), JB = (JT + 1) / 2;     // key tiles in sight, and pairs of them
    const bool stated = chunk > 0 || a.init_states;      // else H_[n] = U_[n] = 0: nothing to read or multiply

    // ---------------- requests: gates, k rows, state rows ----------------
    const int64_t gate_at = gate_base + (int64_t)min(tok0 + lane, a.T - 1) * a.H;
    const float gm = a.gate[gate_at];
    float ball = 1.0f;                                   // lane j: write gate beta_j
    if constexpr (GATED) {
        const float raw = (a.beta ? a.beta : a.gate)[gate_at];
        ball = a.beta ? raw : 1.0f;
    }
    // row i NW + w of the chunk by wave w, four features 4 lane .. per lane
    constexpr int NP = kChunk / NW;
    IO::raw4 rows[NP];
    auto load_rows = [&](const void *x) {
#pragma unroll
        for (int i = 0; i < NP; ++i)
            if (i * NW < 16 * JT)
                rows[i] = IO::load_raw4(x, base_bh + (int64_t)min(tok0 + i * NW + w, a.T - 1) * a.stride_t + 4 * lane);
    };
    auto store_rows = [&]() {                            // (rows beyond the sequence and the key tiles in sight are zero)
#pragma unroll
        for (int i = 0; i < NP; ++i)
            if (i * NW < 32 * JB) {
                const bool live = i * NW < 16 * JT && tok0 + i * NW + w < a.T;
                *(u16x4 *)(sRow + at(i * NW + w, 4 * lane)) = live ? rows[i] : u16x4{0, 0, 0, 0};
            }
    };
    load_rows(a.k);
    // this wave's rows of a state as A fragments: element [32 w + 16 rt + n][32 s + 16 (p / 4) + 4 kg + p % 4] times the scale
    f16x8 shi[2][kSteps], slo[2][kSteps];
    // inverse scales of rows 32 w + 16 rt + 4 kg .. (from LDS wherever they are needed: no registers for them across the passes)
    auto state_scale = [&](int rt) { return *(const f32x4 *)(sScale + 16 * rt + 4 * kg); };
    auto load_state = [&](const void *ws) {
        if (!stated) return;
        const f32x4 *src = (const f32x4 *)ws + chunk_id * (kWideD * kWideD / 4) + (int64_t)w * 2 * 16 * 64 + lane;
        f32x4 x[2][2 * kSteps];
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int s = 0; s < 2 * kSteps; ++s) x[rt][s] = src[(rt * 2 * kSteps + s) * 64];
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) {
            float m = 0.0f;
#pragma unroll
            for (int s = 0; s < 2 * kSteps; ++s)
#pragma unroll
                for (int e = 0; e < 4; ++e) m = fmaxf(m, fabsf(x[rt][s][e]));
            const int sexp = scale_exponent(max_kg(m), 9);
            const float sc = pow2(sexp);
#pragma unroll
            for (int s = 0; s < kSteps; ++s) split_f16(sc * x[rt][2 * s], sc * x[rt][2 * s + 1], shi[rt][s], slo[rt][s]);
            sScale[16 * rt + n] = pow2(-sexp);           // (the same from the four lanes of a row)
        }
    };
    sScale[lane & 31] = 1.0f;
    load_state(a.ws_H);
    int c_loc[TT];                                       // this lane's tokens
    int64_t tok_off[TT];
    bool valid[TT];
    float lam[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
        c_loc[tt] = 16 * (TT * tb + tt) + n;
        valid[tt] = tok0 + c_loc[tt] < a.T;
        const int tok = min(tok0 + c_loc[tt], a.T - 1);
        tok_off[tt] = base_bh + (int64_t)tok * a.stride_t + 32 * w + 4 * kg;
        lam[tt] = ((!GATED || a.lambda) ? a.lambda : a.gate)[gate_base + (int64_t)tok * a.H];
    }
    auto load_q = [&](int rt, int tt) {
        const f32x4 v = IO::load4(a.q, tok_off[tt] + 16 * rt);
        return valid[tt] ? v : zero4();
    };
    float hn2 = 0.0f;
    if (stated) hn2 = wave_sum(a.ws_hn[chunk_id * 64 + lane]);                    // 8 x 8 partial sums of ||H_[n]||^2

    // ---------------- decays (Section 4.2.1; log-space form of Appendix B.2, base 2) ----------------
    const float Gall = wave_inclusive_scan((tok0 + lane < a.T) ? log2_gate(gm) : 0.0f, lane);
    float zeta[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) zeta[tt] = exp2f(__shfl(Gall, c_loc[tt], 64));
    auto mask4 = [&](int jt, int c, bool strict) { return mask_rows<GATED>(Gall, ball, kg, jt, c, strict); };
    // this wave's (key tile, token tile) pair of the masked key products (token tile TT: none)
    int unit_j, unit_t = 0;
    f32x4 unit_m;
    {
        int u = w, len = TT * tb + 1;
        while (unit_t < TT && u >= len) { u -= len; ++unit_t; ++len; }
        unit_j = u;
        unit_m = unit_t < TT ? mask4(u, 16 * (TT * tb + unit_t) + n, false) : zero4();
    }
    // keys to LDS: bf16 rows, and binary16 fragments with a power of two per key (largest element to [2^14, 2^15): sums of 256
    // products with the updates' 2^16 stay below 2^40)
    store_rows();
#pragma unroll
    for (int i = 0; i < NP; ++i)
        if (i * NW < 16 * JT) {
            const int row = i * NW + w;
            f32x4 x = IO::cvt4(rows[i]);
            if (tok0 + row >= a.T) x = zero4();
            const int e = scale_exponent(wave_max(fmaxf(fmaxf(fabsf(x[0]), fabsf(x[1])), fmaxf(fabsf(x[2]), fabsf(x[3])))), 14);
            const float sc = pow2(e);
            f16x4 y;
#pragma unroll
            for (int r = 0; r < 4; ++r) y[r] = (_Float16)(sc * x[r]);
            // features 4 lane ..: step lane / 8, half (lane / 4) % 2 of the fragment, kg = lane % 4
            *((f16x4 *)(sK + ((row >> 4) * kSteps + (lane >> 3)) * 64 + 16 * (lane & 3) + (row & 15)) + ((lane >> 2) & 1)) = y;
            if (lane == 0) sKs[row] = pow2(-e);
        }
    for (int i = tid; i < (int)(SH::p_bytes / 16); i += kWideThreads)             // (tiles beyond a token's own stay zero)
        *(f32x4 *)(sP + i) = zero4();
    lds_barrier();

    // [16 keys, tile jt] x X^T over all features, X as NX pieces of fragments `step` apart
    auto key_product = [&](int jt, const f16x8 *X, auto piecesc) {
        constexpr int NX = decltype(piecesc)::value;
        f32x4 c[2] = {zero4(), zero4()};                 // two chains of dependent products
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
            const f16x8 ka = sK[(jt * kSteps + s) * 64 + lane];
#pragma unroll
            for (int x = 0; x < NX; ++x) c[(s * NX + x) & 1] = mma_h(ka, X[(x * kSteps + s) * 64 + lane], c[(s * NX + x) & 1]);
        }
        return c[0] + c[1];
    };
    typedef std::integral_constant<int, 1> One;
    typedef std::integral_constant<int, 2> Two;

    // ---------------- chunk-wise Frobenius norm (gka_solve_shared.hpp) ----------------
    float fro[TT];
    {
        for (int jt = 0; jt < JT; ++jt) {
            float part = 0.0f;
            const float ksj = sKs[16 * jt + n];          // (column n: key 16 jt + n)
            if (stated) {
                f32x4 acc[2] = {zero4(), zero4()};
#pragma unroll
                for (int s = 0; s < kSteps; ++s) {
                    const f16x8 kb = sK[(jt * kSteps + s) * 64 + lane];
#pragma unroll
                    for (int rt = 0; rt < 2; ++rt) {
                        acc[rt] = mma_h(shi[rt][s], kb, acc[rt]);
                        acc[rt] = mma_h(slo[rt][s], kb, acc[rt]);
                    }
                }
                const f16x8 kr = sK[(jt * kSteps + w) * 64 + lane];               // this wave's features of the keys
#pragma unroll
                for (int rt = 0; rt < 2; ++rt) {
                    acc[rt] *= state_scale(rt);
#pragma unroll
                    for (int r = 0; r < 4; ++r) part += acc[rt][r] * (float)kr[4 * rt + r];
                }
                part = sum_over_kg(part) * ksj * ksj;
            }
            if (kg == 0) norm.sA[w * 64 + 16 * jt + n] = part;
        }
        for (int u0 = w; u0 < JT * (JT + 1) / 2; u0 += NW) {
            int it = u0, jt = 0;
            while (it > jt) { ++jt; it -= jt; }          // tile it <= jt of the lower triangle, row by row
            const f32x4 G = key_product(it, sK + jt * kSteps * 64, One());
            const f32x4 m = mask4(it, 16 * jt + n, true), ksi = *(const f32x4 *)(sKs + 16 * it + 4 * kg);
            const float ksj = sKs[16 * jt + n];
            float bp = 0.0f, dp = 0.0f;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float g = G[r] * ksi[r] * ksj, g2 = g * g;
                bp += m[r] * g2;
                dp += (4 * kg + r == n) ? g2 : 0.0f;
            }
            bp = sum_over_kg(bp);
            dp = sum_over_kg(dp);
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
    }

    // ---------------- Chebyshev iteration (Algorithm 1), residual form ----------------
    float s0[TT], rho2[TT], omega[TT];
    f32x4 xi[2][TT], dl[2][TT], gS[2][TT], gI[2][TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
        if (GATED && !a.lambda) lam[tt] = a.lambda_scale * fro[tt];               // Section 4.1: lambda_t = a ||H_t||_F
        if (!valid[tt]) lam[tt] = 1.0f;
        const float L = fro[tt] + lam[tt], mu = lam[tt];                          // Section 4.1
        s0[tt] = 2.0f / (L + mu);
        const float rho = (L - mu) / (L + mu);
        rho2[tt] = rho * rho;
        omega[tt] = 2.0f;
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) {
            const f32x4 q = load_q(rt, tt);
            gS[rt][tt] = zero4();
            gI[rt][tt] = -q;
            dl[rt][tt] = xi[rt][tt] = s0[tt] * q;                                 // xi_0 = 2 q / (L + mu)
        }
    }
    // the exponents that bring the largest elements of vectors of this lane's tokens to [2^e, 2^(e + 1)) (all waves together)
    int xexp[TT];
    auto token_scales = [&](const f32x4 (&x)[2][TT], int e, float *table) {
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            float m = 0.0f;
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                for (int r = 0; r < 4; ++r) m = fmaxf(m, fabsf(x[rt][tt][r]));
            m = max_kg(m);
            if (kg == 0) table[w * 16 * TT + 16 * tt + n] = m;
        }
        lds_barrier();
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            float m = 0.0f;
#pragma unroll
            for (int i = 0; i < NW; ++i) m = fmaxf(m, table[i * 16 * TT + 16 * tt + n]);
            xexp[tt] = scale_exponent(m, e);
        }
    };
    auto publish = [&](const f32x4 (&x)[2][TT]) {
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            const float sc = pow2(xexp[tt]);
            f16x8 hi, lo;
            split_f16(sc * x[0][tt], sc * x[1][tt], hi, lo);
            sX[((tt * 2 + 0) * kSteps + w) * 64 + lane] = hi;
            sX[((tt * 2 + 1) * kSteps + w) * 64 + lane] = lo;
        }
    };
    // acc += S X^T (times both scales) for this wave's rows
    auto state_product = [&](f32x4 (&acc)[2][TT]) {
        if (!stated) return;
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
            f16x8 xh[TT], xl[TT];
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) {
                xh[tt] = sX[((tt * 2 + 0) * kSteps + s) * 64 + lane];
                xl[tt] = sX[((tt * 2 + 1) * kSteps + s) * 64 + lane];
            }
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                for (int tt = 0; tt < TT; ++tt) acc[rt][tt] = mma_h(shi[rt][s], xh[tt], acc[rt][tt]);
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                for (int tt = 0; tt < TT; ++tt) acc[rt][tt] = mma_h(slo[rt][s], xh[tt], acc[rt][tt]);
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                for (int tt = 0; tt < TT; ++tt) acc[rt][tt] = mma_h(shi[rt][s], xl[tt], acc[rt][tt]);
        }
    };
    const f32x4 unit_ks = unit_t < TT ? *(const f32x4 *)(sKs + 16 * unit_j + 4 * kg) : zero4();
    auto masked_key_products = [&]() {
        if (unit_t >= TT) return;
        int e = xexp[0];
#pragma unroll
        for (int tt = 1; tt < TT; ++tt) e = unit_t == tt ? xexp[tt] : e;
        f32x4 v = key_product(unit_j, sX + unit_t * 2 * kSteps * 64, Two()) * unit_m * (pow2(-e) * unit_ks);
#pragma unroll
        for (int piece = 0; piece < 3; ++piece) {
            const u16x4 bits = bits4(v);
            *((u16x4 *)(sP + ((unit_t * 2 + (unit_j >> 1)) * 3 + piece) * 64 + lane) + (unit_j & 1)) = bits;
            v -= IOBF16::cvt4(bits);
        }
    };
    // acc += A^T (P o M) for this wave's rows, A = the rows in sRow
    auto intra_product = [&](f32x4 (&acc)[2][TT]) {
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
            if (jb >= JB) break;
            bf16x8 at_[2];
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
                at_[rt] = gather_transposed_bf16(sRow, at, 32 * w + 16 * rt, lane, 32 * jb + 4 * kg, 32 * jb + 16 + 4 * kg);
#pragma unroll
            for (int tt = 0; tt < TT; ++tt)
#pragma unroll
                for (int piece = 0; piece < 3; ++piece) {
                    const bf16x8 pb = sP[((tt * 2 + jb) * 3 + piece) * 64 + lane];
#pragma unroll
                    for (int rt = 0; rt < 2; ++rt) acc[rt][tt] = mma_b(at_[rt], pb, acc[rt][tt]);
                }
        }
    };
    token_scales(dl, 4, sMax);                                 // (its barrier: the norm's scratch is free for the operands)
    float zs[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) zs[tt] = zeta[tt] * pow2(-xexp[tt]);
    for (int it = 0; it < a.n_iter; ++it) {
        publish(dl);
        int *flags = sGrown + (it & 1) * 16 * TT + n;
        if constexpr (GIVEN) {
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) {
                float largest = 0.0f;
#pragma unroll
                for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) largest = fmaxf(largest, fabsf(dl[rt][tt][r]));
                if (largest * pow2(xexp[tt]) > kRescaleAbove) flags[16 * tt] = 1;
            }
        }
        lds_barrier();                                   // delta visible; the masked products of the last pass are used up
        int grown[TT] = {};
        if constexpr (GIVEN) {
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) grown[tt] = flags[16 * tt];
        }
        masked_key_products();
        state_product(gS);
        lds_barrier();
        if (GIVEN && w == 0 && kg == 0) {                // (everybody has read them; they are written again two barriers from here)
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) flags[16 * tt] = 0;
        }
        intra_product(gI);
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            omega[tt] = 4.0f / (4.0f - rho2[tt] * omega[tt]);                     // weight schedule
            const float cm = omega[tt] - 1.0f, cs = -omega[tt] * s0[tt];
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) {
                const f32x4 zsr = zs[tt] * state_scale(rt);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float res = zsr[r] * gS[rt][tt][r] + gI[rt][tt][r] + lam[tt] * xi[rt][tt][r];   // -r_{i-1}
                    dl[rt][tt][r] = cm * dl[rt][tt][r] + cs * res;
                    xi[rt][tt][r] += dl[rt][tt][r];
                }
            }
        }
        if constexpr (GIVEN) {
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) {
                const int down = xexp[tt] > kRescale - 126 && grown[tt] ? kRescale : 0;
                xexp[tt] -= down;
                zs[tt] *= pow2(down);
#pragma unroll
                for (int rt = 0; rt < 2; ++rt) gS[rt][tt] *= pow2(-down);
            }
        }
    }
    if (GATED && a.xhat_out) {
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int tt = 0; tt < TT; ++tt)
                if (valid[tt])
                    *(f32x4 *)(a.xhat_out + (gate_base + (int64_t)(tok0 + c_loc[tt]) * a.H) * kWideD + 32 * w + 16 * rt + 4 * kg) =
                        xi[rt][tt];
    }

    // ---------------- readout y_c = zeta_c U_[n] x_c + sum_{j<=c} m[j,c] v_j (k_j . x_c) ----------------
    load_state(a.ws_U);
    load_rows(a.v);
    if (GATED && a.alpha) {                              // alpha-connection (Section 4.3)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            const float al = a.alpha[gate_base + (int64_t)min(tok0 + c_loc[tt], a.T - 1) * a.H];
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) xi[rt][tt] = al * xi[rt][tt] + (1.0f - al) * load_q(rt, tt);
        }
    }
    token_scales(xi, 9, sMax + NW * 16 * TT);                                 // (its barrier: every wave is done with the operands of the last pass
    publish(xi);                                         // and with the keys' transposed rows)
    store_rows();
    lds_barrier();
    masked_key_products();
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) gS[rt][tt] = zero4();
    state_product(gS);
    lds_barrier();
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) gS[rt][tt] *= zeta[tt] * pow2(-xexp[tt]) * state_scale(rt);
    intra_product(gS);
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
            if (valid[tt])
                IO::store4(a.o, tok_off[tt] + 16 * rt, gS[rt][tt][0], gS[rt][tt][1], gS[rt][tt][2], gS[rt][tt][3]);
}

template <int TT, bool GATED, bool GIVEN>
static hipError_t launch_solve_wide_t(const SolveArgs &a, hipStream_t stream)
{
    typedef WideShape<TT> SH;
    static bool lds_raised[kMaxLdsDevices] = {};
    hipError_t e = raise_lds_limits(lds_raised, {{(const void *)solve_wide_kernel<TT, GATED, GIVEN>, SH::lds_bytes}});
    if (e != hipSuccess) return e;
    // (outputs that replace rows of k or v: the token blocks of a chunk one launch after the other, as in gka_solve_f32.hip)
    const bool over_rows = a.o == a.v || a.o == a.k;
    SolveArgs args = a;
    for (args.skip_blocks = over_rows ? 0 : -1; args.skip_blocks < (over_rows ? SH::TB : 0); ++args.skip_blocks) {
        hipLaunchKernelGGL((solve_wide_kernel<TT, GATED, GIVEN>), dim3((unsigned)(a.n_pairs * a.n_chunks * (over_rows ? 1 : SH::TB))),
                           dim3(kWideThreads), SH::lds_bytes, stream, args);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

bool solve_wide_takes(const SolveArgs &a, int d, bool io_bf16)
{
    return a.pieces && d == kWideD && io_bf16 && a.n_iter <= kMaxPasses;
}

hipError_t launch_solve_wide(const SolveArgs &a, int tiles, hipStream_t stream)
{
    const bool gated = a.beta || a.alpha || !a.lambda || a.xhat_out;
    if (a.init_states) {
        if (tiles == 2) return gated ? launch_solve_wide_t<2, true, true>(a, stream) : launch_solve_wide_t<2, false, true>(a, stream);
        return gated ? launch_solve_wide_t<1, true, true>(a, stream) : launch_solve_wide_t<1, false, true>(a, stream);
    }
    if (tiles == 2) return gated ? launch_solve_wide_t<2, true, false>(a, stream) : launch_solve_wide_t<2, false, false>(a, stream);
    return gated ? launch_solve_wide_t<1, true, false>(a, stream) : launch_solve_wide_t<1, false, false>(a, stream);
}

}  // namespace gka
