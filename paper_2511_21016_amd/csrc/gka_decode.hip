// Recurrent steps of Eq. (CH) per (sequence, head) pair: state update (with the optional write gate), ||H_t||_F,
// Algorithm 1 with the matrix held in registers, readout (with the optional alpha-connection). One workgroup per pair;
// all arithmetic fp32. The states are read once, advanced by a.T tokens in registers and written once, so the state
// traffic of a call does not grow with the number of tokens. The same kernel is gka_forward's recurrent path (any
// number of tokens, separate initial and final states, ||H_t||_F and the solve's result as optional outputs), the
// only one for float32 tensors at the head dimensions 16 and 32 and for sequences of up to 128 tokens at 256.
//
// Layout. NW waves; wave w owns D / NW rows of both states. Lane (rg, cg) = (lane / 8, lane % 8) of a wave holds, of the R
// rows D / NW w + 8 rr + rg (rr < R = D / (8 NW)), the float4 pieces cg + 8 i (i < D / 32): eight lanes read a whole
// 128-byte line, a wave's pieces i = 0, 1, .. eight whole rows, and i is the 32-column block. A product S x is formed by
// rows: a lane takes the D / 8 components of x under its pieces from LDS (D / 32 reads of 16 bytes, one line per wave),
// and the R partial sums are added over the eight lanes of a row by three DPP moves that also deal the rows out, so
// that every lane ends up with one complete row sum (lanes whose cg differs in bit 1 only with the same one). That
// lane then owns the row's component of xi, delta and the residual: a pass is one LDS write, one barrier, D / 32 LDS
// reads, the multiply-adds and three DPP steps. Barriers order LDS only: the stores of the advanced states drain
// while the token is solved.
// What bounds it: few pairs, the latency of that chain (about 0.25 us per pass; d = 128, 32 pairs 8.4 us); many pairs, HBM for
// single tokens (d = 128, 8192 pairs, 10 passes: 376 us for 2.16 GB, 5.7 TB/s), and the vector units for several tokens
// per call (4 tokens of 1536 pairs, block-lower H: 105 us).
#include "gka_device.hpp"
#include "gka_kernels.hpp"

namespace gka {

template <int D, int NW_>
struct DecodeShape {
    static constexpr int NW = NW_, NTHR = 64 * NW;
    static constexpr int R = D / (8 * NW), NI = D / 32;      // rows and float4 pieces per row of a lane
    static_assert(R * 8 * NW == D && (R == 1 || R == 2 || R == 4), "every lane holds R whole rows' pieces");
    static constexpr bool STREAM_U = D == 256;               // H fills the registers
    static constexpr int G = R == 4 ? 2 : 1;                 // groups of rows whose ||.||^2 is summed apart
};

// The sums over the eight lanes cg of R row sums each: this lane's share is row 8 rr + rg with rr = row_share<R>(lane).
template <int R>
__device__ __forceinline__ int row_share(int lane)
{
    return R == 4 ? ((lane >> 1) & 2) | (lane & 1) : R == 2 ? (lane >> 2) & 1 : 0;
}
template <int R>
__device__ __forceinline__ float sum_rows(const float (&p)[R], int lane)
{
    auto dpp = [](float x, auto ctrl) {
        return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), decltype(ctrl)::value, 0xF,
                                                                  0xF, true));
    };
    constexpr std::integral_constant<int, 0x141> half_mirror;     // lane cg <-> 7 - cg
    constexpr std::integral_constant<int, 0xB1> xor1;             // quad_perm [1,0,3,2]
    constexpr std::integral_constant<int, 0x4E> xor2;             // quad_perm [2,3,0,1]
    const bool b2 = lane & 4, b0 = lane & 1;
    float t;
    if constexpr (R == 4) {
        // rows 2 b2, 2 b2 + 1 stay, the others go to the mirror lane; then row b0 of the two stays
        const float k0 = b2 ? p[2] : p[0], k1 = b2 ? p[3] : p[1];
        const float a0 = k0 + dpp(b2 ? p[0] : p[2], half_mirror), a1 = k1 + dpp(b2 ? p[1] : p[3], half_mirror);
        t = (b0 ? a1 : a0) + dpp(b0 ? a0 : a1, xor1);
    } else if constexpr (R == 2) {
        t = (b2 ? p[1] : p[0]) + dpp(b2 ? p[0] : p[1], half_mirror);
        t += dpp(t, xor1);
    } else {
        t = p[0] + dpp(p[0], half_mirror);
        t += dpp(t, xor1);
    }
    return t + dpp(t, xor2);
}

// MULTI = false: the single-step kernel, a.T == 1 known at compile time.
// LOWER: of H_in / H_state only the 32 x 32 blocks on and below the block diagonal are read and written; the blocks
// above are rebuilt in registers from their mirror images (through LDS, once per call), so the arithmetic is the same.
// STREAM: U is streamed (as always at d = 256) although it would fit: each piece is read, advanced, used for the
// readout and written back after the solve. For single tokens of many pairs: fewer registers, four workgroups per CU.
template <class IO, int D, int NW, bool MULTI, bool LOWER, bool STREAM>
__global__ __launch_bounds__(64 * NW)
void decode_step_kernel(DecodeArgs a)
{
    typedef DecodeShape<D, NW> SH;
    const int T = MULTI ? a.T : 1;
    constexpr int NTHR = SH::NTHR, R = SH::R, NI = SH::NI, C4 = D / 4;
    constexpr bool STREAM_U = SH::STREAM_U || STREAM;
    static_assert(!STREAM || !MULTI, "U is streamed once per token: at d < 256 only where a call is one token");
    const int t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int rg = lane >> 3, cg = lane & 7;
    const int pair = blockIdx.x;

    __shared__ __attribute__((aligned(16))) float s_in[3][D];     // q, k, v of the token
    __shared__ __attribute__((aligned(16))) float s_x[2][D];      // operand of the product (delta_i or xhat), alternating
    // ||H||^2 by groups of 16 rows (R >= 2): the order of the sum does not depend on NW, single and multi-token calls
    // stay bit-identical
    constexpr int G = SH::G;
    __shared__ float s_red[NW * G];

    const int row0 = w * (D / NW) + rg;                           // row 8 rr + row0
    const int my = 8 * row_share<R>(lane) + row0;                 // the component this lane owns in the solve
    const bool writer = !(lane & 2) && (R == 4 || !(lane & 1)) && (R != 1 || !(lane & 4));   // one of the lanes that own it
    const int64_t state_off = (int64_t)pair * D * D + (int64_t)row0 * D + 4 * cg;
    auto piece = [&](int rr, int i) { return 8 * rr * D + 32 * i; };   // its offset from the lane's base
    const float *Hin = a.H_in ? a.H_in + state_off : nullptr;      // nullptr: zero initial states
    const float *Uin = a.U_in ? a.U_in + state_off : nullptr;
    float *Hs = a.H_state ? a.H_state + state_off : nullptr;       // nullptr: the final states are not wanted
    float *Us = a.U_state ? a.U_state + state_off : nullptr;
    const int b = pair / a.H, h = pair - b * a.H;

    // a token's q, k, v (one component per thread, the three arrays dealt out over the threads) and scalars, fetched
    // while the token before it is solved
    constexpr int NIN = (3 * D + NTHR - 1) / NTHR;
    struct TokenIn { float x[NIN], gamma, beta, alpha, lam; };
    auto fetch = [&](int tok) {
        TokenIn in;
        const int64_t bth = ((int64_t)b * T + tok) * a.H + h;      // [B,T,H] index of the token
        const int64_t at = b * a.stride_b + tok * a.stride_t + h * a.stride_h;   // its row of q, k, v, o
#pragma unroll
        for (int i = 0; i < NIN; ++i) {
            const int e = i * NTHR + t, which = min(e / D, 2);
            in.x[i] = IO::load(which == 0 ? a.q : which == 1 ? a.k : a.v, at + e % D);
        }
        in.gamma = a.gate[bth];
        in.beta = a.beta ? a.beta[bth] : 1.0f;                     // write gate (Remark in Section 4.1)
        in.alpha = a.alpha ? a.alpha[bth] : 1.0f;                  // alpha-connection (Section 4.3)
        in.lam = a.lambda ? a.lambda[bth] : 0.0f;
        return in;
    };
    TokenIn next = fetch(0);

    f32x4 hreg[R][NI], ureg[STREAM_U ? 1 : R][NI];
    // row block of the lane's row 8 rr + row0 (a wave's eight rows lie in one 32-row block)
    auto held = [&](int rr, int i) { return !LOWER || i <= (w * (D / NW) + 8 * rr) / 32; };
#pragma unroll
    for (int rr = 0; rr < R; ++rr)
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            hreg[rr][i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            if (Hin && held(rr, i)) hreg[rr][i] = __builtin_nontemporal_load((const f32x4 *)(Hin + piece(rr, i)));
        }
    if constexpr (!STREAM_U) {
#pragma unroll
        for (int rr = 0; rr < R; ++rr)
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                ureg[rr][i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                if (Uin) ureg[rr][i] = __builtin_nontemporal_load((const f32x4 *)(Uin + piece(rr, i)));
            }
    }
    // the first row's pieces of a streamed U are on their way during the solve
    f32x4 upre[STREAM ? NI : 1];
    if constexpr (STREAM) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            upre[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            if (Uin) upre[i] = __builtin_nontemporal_load((const f32x4 *)(Uin + piece(0, i)));
        }
    }
    if constexpr (LOWER) {
        constexpr int NOFF = NI * (NI - 1) / 2;
        // the blocks below the diagonal, block (bi, bj) at bi (bi - 1) / 2 + bj
        __shared__ __attribute__((aligned(16))) float s_tr[NOFF][32][36];
#pragma unroll
        for (int rr = 0; rr < R; ++rr)
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int bi = (w * (D / NW) + 8 * rr) / 32, row = 8 * rr + row0;
                if (i < bi) *(f32x4 *)&s_tr[bi * (bi - 1) / 2 + i][row % 32][4 * cg] = hreg[rr][i];
            }
        lds_barrier();
#pragma unroll
        for (int rr = 0; rr < R; ++rr)
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int bi = (w * (D / NW) + 8 * rr) / 32, row = 8 * rr + row0;
                if (i > bi) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) hreg[rr][i][e] = s_tr[i * (i - 1) / 2 + bi][4 * cg + e][row % 32];
                }
            }
    }
    // H is written in full where the caller of the forward pass wants the final state (valid under either layout)
    auto stored = [&](int rr, int i) { return held(rr, i) || a.h_out_full; };
    // the components of a vector in LDS under this lane's pieces i
    auto columns = [&](const float *x, int i) { return *(const f32x4 *)(x + 4 * cg + 32 * i); };
    auto row_sums = [&](const f32x4 (&acc)[R]) {
        float p[R];
#pragma unroll
        for (int rr = 0; rr < R; ++rr) p[rr] = (acc[rr][0] + acc[rr][1]) + (acc[rr][2] + acc[rr][3]);
        return sum_rows<R>(p, lane);
    };
    for (int tok = 0; tok < T; ++tok) {
        const int64_t bth = ((int64_t)b * T + tok) * a.H + h;
        const int64_t at = b * a.stride_b + tok * a.stride_t + h * a.stride_h;
        // addresses of state pieces are recomputed per token (hoisted out of the loop they would take registers that the
        // states need)
        int voff = 0;
        if constexpr (MULTI || STREAM_U) asm volatile("" : "+v"(voff));
        const TokenIn in = next;
#pragma unroll
        for (int i = 0; i < NIN; ++i)
            if (i * NTHR + t < 3 * D) (&s_in[0][0])[i * NTHR + t] = in.x[i];
        const float gamma = in.gamma, beta = in.beta, alpha = in.alpha;
        lds_barrier();
        if constexpr (MULTI) next = fetch(min(tok + 1, T - 1));

        // ---- state update (Eq. (CH)) and ||H_t||_F^2
        const float qr = s_in[0][my];
        float kr[R], vr[R], ss[G] = {};
#pragma unroll
        for (int rr = 0; rr < R; ++rr) {
            kr[rr] = s_in[1][8 * rr + row0];
            vr[rr] = beta * s_in[2][8 * rr + row0];
        }
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const f32x4 kc = columns(s_in[1], i);
#pragma unroll
            for (int rr = 0; rr < R; ++rr) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // beta (k_i k_j): the product of the two k components first, so that both mirror images of an
                    // element get the same bits
                    hreg[rr][i][e] = gamma * hreg[rr][i][e] + beta * (kr[rr] * kc[e]);
                    // (the multiply-add written out: held or streamed, U gets the same bits)
                    if constexpr (!STREAM_U) ureg[rr][i][e] = __builtin_fmaf(gamma, ureg[rr][i][e], vr[rr] * kc[e]);
                    ss[G * rr / R] += hreg[rr][i][e] * hreg[rr][i][e];
                }
            }
        }
        if (tok == T - 1) {                      // the stores drain while the last token is solved
#pragma unroll
            for (int rr = 0; rr < R; ++rr)
#pragma unroll
                for (int i = 0; i < NI; ++i) {
                    if (Hs && stored(rr, i)) __builtin_nontemporal_store(hreg[rr][i], (f32x4 *)(Hs + voff + piece(rr, i)));
                    if constexpr (!STREAM_U) {
                        if (Us) __builtin_nontemporal_store(ureg[rr][i], (f32x4 *)(Us + voff + piece(rr, i)));
                    }
                }
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const float total = wave_inclusive_scan(ss[g], lane);
            if (lane == 63) s_red[w * G + g] = total;
        }
        lds_barrier();
        float fro2 = 0.0f;
#pragma unroll
        for (int i = 0; i < NW * G; ++i) fro2 += s_red[i];
        const float fro = sqrtf(fro2);
        const float lam = a.lambda ? in.lam : a.lambda_scale * fro;          // Section 4.1: lambda_t = a ||H_t||_F
        if (a.fro_out && t == 0) a.fro_out[bth] = fro;

        // ---- Algorithm 1 in residual form
        const float L = fro + lam, mu = lam;
        const float s0 = 2.0f / (L + mu);
        const float rho = (L - mu) / (L + mu);
        const float rho2 = rho * rho;
        float xi = s0 * qr, dl = xi, rs = qr;
        float omega = 2.0f;
        int buf = 0;
        for (int it = 0; it < a.n_iter; ++it) {
            // (the buffer of the pass before last: every wave has read it before it passed the last barrier)
            if (writer) s_x[buf][my] = dl;
            omega = 4.0f / (4.0f - rho2 * omega);
            lds_barrier();
            f32x4 acc[R];                          // (four chains per row)
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const f32x4 xc = columns(s_x[buf], i);
#pragma unroll
                for (int rr = 0; rr < R; ++rr)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc[rr][e] = i == 0 ? hreg[rr][i][e] * xc[e] : acc[rr][e] + hreg[rr][i][e] * xc[e];
            }
            const float hx = row_sums(acc);
            rs -= hx + lam * dl;
            dl = (omega - 1.0f) * dl + omega * s0 * rs;
            xi += dl;
            buf ^= 1;
        }

        // ---- readout y = U (alpha xhat + (1 - alpha) q)
        if (writer) {
            s_x[buf][my] = alpha * xi + (1.0f - alpha) * qr;
            if (a.xhat_out) a.xhat_out[bth * D + my] = xi;
        }
        lds_barrier();
        f32x4 acc[R];
#pragma unroll
        for (int rr = 0; rr < R; ++rr) acc[rr] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (STREAM_U) {
            // four pieces at a time: read, advanced, used and written back. From the caller's initial state at the first
            // token, afterwards what this same lane stored at the previous token. A zero initial state: a single token reads
            // nothing (d = 256, one token of 256 pairs: 21.1 us, 32.2 with the loads replaced by zeros), by a branch around
            // the whole walk over U (branches around the loads leave one of them in flight). With several tokens a branch
            // makes the compiler spill 92 registers: there the loads go to a few rows of the final state, the same for all
            // waves, and zeros take their place.
            const bool zero = tok == 0 && !Uin;
            const float *Usrc = (zero ? Us - row0 * D : tok > 0 ? Us : Uin) + voff;
            enum { FROM_ZERO, LOADED, FROM_MEMORY };
            auto four_pieces = [&](int rr, int i0, auto from) {
                constexpr int FROM = decltype(from)::value;
                if constexpr (SH::STREAM_U) __builtin_amdgcn_sched_barrier(0);   // (d = 256: no room for more at once)
                const float vs = beta * s_in[2][8 * rr + row0];
                f32x4 u[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const f32x4 *src = (const f32x4 *)(Usrc + piece(rr, i0 + i));
                    if constexpr (FROM == FROM_ZERO) u[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                    else if constexpr (FROM == LOADED) u[i] = upre[i0 + i];
                    else if constexpr (MULTI) u[i] = *src;
                    else u[i] = __builtin_nontemporal_load(src);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const f32x4 kc = columns(s_in[1], i0 + i), xc = columns(s_x[buf], i0 + i);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        u[i][e] = __builtin_fmaf(gamma, MULTI && zero ? 0.0f : u[i][e], vs * kc[e]);
                        acc[rr][e] += u[i][e] * xc[e];
                    }
                    f32x4 *dst = (f32x4 *)(Us + voff + piece(rr, i0 + i));
                    if constexpr (MULTI) *dst = u[i];
                    else __builtin_nontemporal_store(u[i], dst);
                }
            };
            auto all_pieces = [&](auto first, auto from) {
                if constexpr (STREAM) {            // (no condition on rr around the loads: it costs them their non-temporal
                    static_assert(NI == 4);        // hint, d = 128, 8192 pairs 388 us instead of 380)
                    four_pieces(0, 0, first);
                }
#pragma unroll
                for (int rr = STREAM; rr < R; ++rr)
#pragma unroll
                    for (int i0 = 0; i0 < NI; i0 += 4) four_pieces(rr, i0, from);
            };
            constexpr std::integral_constant<int, FROM_ZERO> zeros;
            constexpr std::integral_constant<int, LOADED> loaded;
            constexpr std::integral_constant<int, FROM_MEMORY> memory;
            if constexpr (MULTI) {
#pragma unroll
                for (int rr = 0; rr < R; ++rr)
#pragma unroll
                    for (int i0 = 0; i0 < NI; i0 += 4) four_pieces(rr, i0, memory);
            } else if (zero) {
                all_pieces(zeros, zeros);
            } else {
                all_pieces(loaded, memory);
            }
        } else {
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const f32x4 xc = columns(s_x[buf], i);
#pragma unroll
                for (int rr = 0; rr < R; ++rr)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[rr][e] += ureg[rr][i][e] * xc[e];
            }
        }
        const float y = row_sums(acc);
        if (writer) IO::store1(a.o, at + my, y);
        // (the next token overwrites s_in, and two of its barriers later s_x: every wave must be done with s_in)
        if constexpr (MULTI) lds_barrier();
    }
}

// Head dimension 16 (the vision models of Appendix L: many pairs, short sequences): one wave per pair and no LDS. A
// state is 64 float4 pieces, lane l holds columns 4 (l % 4) .. + 3 of row l / 4 of H and of U; per-component
// quantities of the solve (xi, delta, residual) live in the four lanes of the component's row. A product H x is taken
// row-wise: the lane's four elements times the four components of x it needs (fetched from the lanes that hold them by
// lane shuffles), then a sum over the four lanes of the row. Four pairs share a workgroup only to fill it; the waves
// never synchronise. The arithmetic is that of decode_step_kernel in another order of summation.
template <class IO>
__global__ __launch_bounds__(256) void decode_step_kernel_d16(DecodeArgs a, int n_pairs)
{
    constexpr int D = 16;
    const int lane = threadIdx.x & 63;
    const int pair = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (pair >= n_pairs) return;                 // (wave-uniform)
    const int r = lane >> 2, c4 = lane & 3;
    const int T = a.T;
    const int64_t state_off = (int64_t)pair * D * D + lane * 4;
    const int b = pair / a.H, h = pair - b * a.H;
    f32x4 hreg = {0.0f, 0.0f, 0.0f, 0.0f}, ureg = {0.0f, 0.0f, 0.0f, 0.0f};
    if (a.H_in) hreg = *(const f32x4 *)(a.H_in + state_off);
    if (a.U_in) ureg = *(const f32x4 *)(a.U_in + state_off);
    // the components 4 c4 .. 4 c4 + 3 of a vector whose component i is held by the lanes of row i
    auto my_columns = [&](float x, float (&out)[4]) {
#pragma unroll
        for (int e = 0; e < 4; ++e) out[e] = __shfl(x, (4 * c4 + e) * 4, 64);
    };
    // sum over the four lanes of a row (a quad): two cross-lane moves within quads
    auto row_sum = [&](float x) {
        x += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0xB1, 0xF, 0xF, true));   // quad_perm [1,0,3,2]
        x += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x4E, 0xF, 0xF, true));   // quad_perm [2,3,0,1]
        return x;
    };
    // inputs of a token are fetched while the token before it is solved
    struct TokenIn { float q, k, v, gamma, beta, alpha, lam; };
    auto fetch = [&](int tok) {
        const int64_t bth = ((int64_t)b * T + tok) * a.H + h;
        const int64_t row0 = b * a.stride_b + tok * a.stride_t + h * a.stride_h;
        TokenIn t;
        t.q = IO::load(a.q, row0 + r);
        t.k = IO::load(a.k, row0 + r);
        t.v = IO::load(a.v, row0 + r);
        t.gamma = a.gate[bth];
        t.beta = a.beta ? a.beta[bth] : 1.0f;
        t.alpha = a.alpha ? a.alpha[bth] : 1.0f;
        t.lam = a.lambda ? a.lambda[bth] : 0.0f;
        return t;
    };
    TokenIn next = fetch(0);
    for (int tok = 0; tok < T; ++tok) {
        const int64_t bth = ((int64_t)b * T + tok) * a.H + h;
        const int64_t row0 = b * a.stride_b + tok * a.stride_t + h * a.stride_h;
        const TokenIn in = next;
        next = fetch(min(tok + 1, T - 1));
        const float qr = in.q, kr = in.k, vr = in.v, gamma = in.gamma, beta = in.beta, alpha = in.alpha;
        float kc[4];
        my_columns(kr, kc);
        // ---- state update (Eq. (CH)) and ||H_t||_F
        float ss = 0.0f;
        const float bv = beta * vr;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            hreg[e] = gamma * hreg[e] + beta * (kr * kc[e]);
            ureg[e] = gamma * ureg[e] + bv * kc[e];
            ss += hreg[e] * hreg[e];
        }
        const float fro = sqrtf(wave_sum(ss));
        const float lam = a.lambda ? in.lam : a.lambda_scale * fro;          // Section 4.1: lambda_t = a ||H_t||_F
        if (a.fro_out && lane == 0) a.fro_out[bth] = fro;
        // ---- Algorithm 1 in residual form, component r in the four lanes of row r
        // (the kernel is bound by its instruction count: reciprocals by the hardware instruction, 1 ulp)
        const float L = fro + lam, mu = lam;
        const float rcp = __builtin_amdgcn_rcpf(L + mu);
        const float s0 = 2.0f * rcp;
        const float rho = (L - mu) * rcp;
        const float rho2 = rho * rho;
        float xi = s0 * qr, dl = xi, rs = qr, omega = 2.0f;
        for (int i = 0; i < a.n_iter; ++i) {
            float xc[4];
            my_columns(dl, xc);
            const float hx = row_sum(hreg[0] * xc[0] + hreg[1] * xc[1] + hreg[2] * xc[2] + hreg[3] * xc[3]);
            omega = 4.0f * __builtin_amdgcn_rcpf(4.0f - rho2 * omega);
            rs -= hx + lam * dl;
            dl = (omega - 1.0f) * dl + (omega * s0) * rs;
            xi += dl;
        }
        if (a.xhat_out && c4 == 0) a.xhat_out[bth * D + r] = xi;
        // ---- readout y = U (alpha xhat + (1 - alpha) q)
        float xc[4];
        my_columns(alpha * xi + (1.0f - alpha) * qr, xc);
        const float y = row_sum(ureg[0] * xc[0] + ureg[1] * xc[1] + ureg[2] * xc[2] + ureg[3] * xc[3]);
        if (c4 == 0) IO::store1(a.o, row0 + r, y);
    }
    if (a.H_state) *(f32x4 *)(a.H_state + state_off) = hreg;
    if (a.U_state) *(f32x4 *)(a.U_state + state_off) = ureg;
}

// Single tokens at d = 128: up to this many pairs one workgroup per CU is all there is, and eight waves that hold both
// states finish a token's chain sooner; above it several workgroups of four waves share a CU, which holding U would not
// let them (us, held with eight waves / streamed with four, full H: 64 pairs 10.0 / 11.7, 192 11.7 / 12.9, 256 12.8 / 14.3,
// 288 19.4 / 17.8, 512 23.8 / 23.3, 1024 50.5 / 47.4, 8192 383 / 377; H on and below the block diagonal: 256 11.8 / 13.9,
// 288 17.0 / 16.9, 1024 42.1 / 38.5, 2048 80.1 / 78.4, 8192 309 / 318; 384 pairs of full H 20.9 / 19.9).
constexpr int kDecodeHoldPairs = 256;

template <class IO, int D, int NW, bool MULTI, bool LOWER, bool STREAM = false>
static void launch_nw(const DecodeArgs &a, int n_pairs, hipStream_t stream)
{
    hipLaunchKernelGGL((decode_step_kernel<IO, D, NW, MULTI, LOWER, STREAM>), dim3((unsigned)n_pairs), dim3(64 * NW), 0,
                       stream, a);
}

template <class IO, int D, bool MULTI, bool LOWER>
static void launch_one(const DecodeArgs &a, int n_pairs, hipStream_t stream)
{
    if constexpr (D == 256) {
        launch_nw<IO, D, 16, MULTI, LOWER>(a, n_pairs, stream);
    } else if constexpr (D == 128) {
        if constexpr (!MULTI) {
            if (a.U_state && n_pairs > kDecodeHoldPairs) {
                launch_nw<IO, D, 4, MULTI, LOWER, true>(a, n_pairs, stream);
                return;
            }
        }
        launch_nw<IO, D, 8, MULTI, LOWER>(a, n_pairs, stream);
    } else {
        launch_nw<IO, D, 4, MULTI, LOWER>(a, n_pairs, stream);
    }
}

template <class IO, bool MULTI>
static void launch_decode(const DecodeArgs &a, int n_pairs, int d, hipStream_t stream)
{
    // (up to d = 32 the state is a single 32 x 32 block: both layouts are the full one)
    if (a.h_lower_blocks && d >= 64) {
        if (d == 128) launch_one<IO, 128, MULTI, true>(a, n_pairs, stream);
        else launch_one<IO, 64, MULTI, true>(a, n_pairs, stream);
        return;
    }
    switch (d) {
    case 16:
        hipLaunchKernelGGL((decode_step_kernel_d16<IO>), dim3((unsigned)((n_pairs + 3) / 4)), dim3(256), 0, stream, a,
                           n_pairs);
        break;
    case 32: launch_one<IO, 32, MULTI, false>(a, n_pairs, stream); break;
    case 64: launch_one<IO, 64, MULTI, false>(a, n_pairs, stream); break;
    case 128: launch_one<IO, 128, MULTI, false>(a, n_pairs, stream); break;
    default: launch_one<IO, 256, MULTI, false>(a, n_pairs, stream); break;
    }
}

// d in {16, 32, 64, 128, 256}; the block-lower layout of H only up to d = 128; d = 256 needs U_state (checked by the
// callers).
hipError_t launch_decode_step(const DecodeArgs &a, int n_pairs, int d, bool io_bf16, hipStream_t stream)
{
    if (d != 16 && d != 32 && d != 64 && d != 128 && d != 256) return hipErrorInvalidValue;
    if ((a.h_lower_blocks && d == 256) || (d == 256 && !a.U_state)) return hipErrorInvalidValue;
    if (io_bf16) {
        if (a.T == 1) launch_decode<IOBF16, false>(a, n_pairs, d, stream);
        else launch_decode<IOBF16, true>(a, n_pairs, d, stream);
    } else {
        if (a.T == 1) launch_decode<IOF32, false>(a, n_pairs, d, stream);
        else launch_decode<IOF32, true>(a, n_pairs, d, stream);
    }
    return hipGetLastError();
}

}  // namespace gka
