// Chunk-wise forward pass (Section 4.2.1) for head dimensions up to 32, bf16 tensors and operands, float32 accumulation:
//   * the layer itself at d = 16 (the vision models of Appendix L) and d = 32: Eq. (CH), its Frobenius norm, Algorithm 1
//     and the readout y_t = U_t xhat_t;
//   * the solve of latent sketching (appendix "Latent Sketching for Approximate Solutions") in d_s <= 32 sketched
//     dimensions, z_t = CH(S H_t S^T + lambda_t I, S q_t, r), on the sketched keys and queries (no values, no readout).
// At these sizes a state is one or four accumulator tiles of the matrix instructions, and a contraction over the features
// a single step. Every operand of a pass of Algorithm 1 then lives in registers: a pass touches no memory at all.
//   small_walk_kernel: a wave walks the sequence of a (batch, head) pair, or a segment of it, 16 tokens at a time with the
//      states in registers; the 16 tokens sit on the output lanes of the products (per-token scalars are per-lane
//      scalars): chunk-wise Frobenius norm, all passes in residual form, the readout, then the states after the tile.
// Where pairs are few and sequences long, two launches before it compute the states before every chunk of 64 tokens:
//   1. small_chunk_delta_kernel: per chunk, Delta H = sum_j w_j k_j k_j^T and Delta U = sum_j w_j v_j k_j^T (w_j: decay
//      from token j to the chunk's end, times the write gate) and the chunk's log2 decay; one wave per chunk.
//   2. small_state_scan_kernel: per pair, the states before every chunk, S_[n+1] = zeta_n S_[n] + Delta_n (elementwise
//      in float32, one float4 per thread and state, sixteen chunks in flight), from the caller's initial states if
//      given; the states after the last chunk are the final states.
// The arithmetic of the walk is that of the 128-dimensional kernels: the token's system is taken divided by its zeta_c,
//   g / zeta_c = H_[n] xi + K^T ((M / zeta_c) o (K xi)) - q / zeta_c,
//   delta' = (omega - 1) delta - omega s0 (zeta_c (g / zeta_c) + lambda xi'),  xi' = xi + delta,
// with bf16 operands (K, the update delta, the masked products; H_[n] as value + remainder) and float32 accumulation; in
// the readout U_[n] and xhat enter as bf16 value + remainder.
//
// Fragment conventions (v_mfma_f32_16x16x32_bf16, lane l = 16 kg + n): an accumulator tile holds rows 4 kg + r
// (r = 0..3) of column n; an operand fragment holds eight contraction values of row (A) or column (B) n. Two
// accumulator tiles of the same columns convert in place into one B fragment, slot s <-> index 16 (s / 4) + 4 kg + s % 4
// of the 32 the fragment covers ("slot order"); every A fragment enumerates its contraction index in that order.
#include "gka_device.hpp"
#include "gka_kernels.hpp"

namespace gka {

namespace {

constexpr int kDs = 32;                    // features of a sketched row that are computed
constexpr int kRowPad = 8;                 // padding of an LDS row of keys or values, 2-byte elements
constexpr float kMinZeta = 0x1p-60f;       // floor of zeta_c where the system is divided by it
// How the walks are cut (us per forward pass, bf16, r = 10):
// * One walk per pair, without the two launches that compute the states before every chunk: with many pairs, which fill
//   the SIMDs (d = 16, 6144 pairs x 197 tokens 98 against 140 chunk by chunk, 2400 x 400 98 and 98, 1200 x 785 143 and 96;
//   d = 32, 3072 x 300 137 and 240, 1024 x 400 84 and 103, 768 x 785 162 and 150), and with up to two chunks (d = 16,
//   768 x 100: 17 against 19).
// * Up to chunk_workgroups chunks in all the four waves of a workgroup take a chunk (d = 16, 192 x 500, 1536 chunks: 21.8
//   against 22.9 with two waves that advance over each other's tiles, 576 x 197, 2304 chunks: 24.5 and 25.6 with one wave,
//   768 x 250, 3072: 31.3 and 29.6; d = 32, 256 x 400, 1792 chunks: 37.2 and 40.5, 576 x 197, 2304 chunks: 43.1 and 41.7).
// * Where such a sequence is short it is walked from its start all the same, in one launch, by a wave per tile that advances
//   the states over the tiles before its own without solving them (d = 16, 13 tiles, 48 pairs: 11.4 against 12.3 by chunks,
//   96 pairs 13.0 and 12.7, 10 tiles, 192 pairs 12.1 and 13.6, 256 pairs 14.3 and 14.1, 16 tiles, 48 pairs 13.0 and 12.3 to
//   14.4 (what three launches take of the host, which varies), 96 pairs 15.7 and 12.7, 19 tiles, 4 pairs 14.2 and 12.4
//   to 16.6; d = 32, 10 tiles, 288 pairs 23.8 and 26.6, 13 tiles,
//   96 pairs 20.5 and 19.2): few_walk_work bounds pairs x tiles^3, which these turning points have in common.
template <int D>
struct WalkRule {
    static constexpr int many_pairs = D == 16 ? 2048 : 1024;
    static constexpr int short_chunks = 2;
    static constexpr int chunk_workgroups = D == 16 ? 2560 : 2048;
    static constexpr int few_walk_tiles = D == 16 ? 20 : 10, few_walk_work = D == 16 ? 1 << 18 : 360000;
};
constexpr int kTileWaveChunks = 1024;      // up to this many chunks in all a walk from the start has a wave per tile
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 mma16(bf16x8 a, bf16x8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 zero4() { return f32x4{0.0f, 0.0f, 0.0f, 0.0f}; }
__device__ __forceinline__ bf16x8 pack8(f32x4 lo, f32x4 hi)
{
    bf16x8 f;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        f[p] = (__bf16)lo[p];
        f[4 + p] = (__bf16)hi[p];
    }
    return f;
}
__device__ __forceinline__ void unpack8(bf16x8 f, f32x4 &lo, f32x4 &hi)
{
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        lo[p] = (float)f[p];
        hi[p] = (float)f[4 + p];
    }
}
// rounded value and what the rounding left over, both as fragments
__device__ __forceinline__ void split8(f32x4 lo, f32x4 hi, bf16x8 &val, bf16x8 &rem)
{
    val = pack8(lo, hi);
    f32x4 bl, bh;
    unpack8(val, bl, bh);
    rem = pack8(lo - bl, hi - bh);
}
// The lane's number, formed anew wherever it is asked for: values derived from it are then not kept (or spilled)
// across the code in between.
__device__ __forceinline__ int fresh_lane()
{
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
}
__device__ __forceinline__ int64_t row_offset(const SmallArgs &a, int b, int h, int tok)
{
    return b * a.stride_b + (int64_t)min(tok, a.T - 1) * a.stride_t + h * a.stride_h;
}
// The chunk's 64 rows of x into a wave's LDS tile, 16 bytes at a time. Rows past the end of the sequence repeat the last
// one (finite values that only meet zero weights).
template <int D>
__device__ __forceinline__ void stage_rows(const SmallArgs &a, const void *x, uint16_t *rows, int b, int h, int tok0,
                                           int lane)
{
    constexpr int PPR = D / 8;                 // pieces of 16 bytes per row
    u32x4 v[PPR];
#pragma unroll
    for (int i = 0; i < PPR; ++i) {
        const int piece = i * 64 + lane;
        v[i] = *(const u32x4 *)((const uint16_t *)x + row_offset(a, b, h, tok0 + piece / PPR) + 8 * (piece % PPR));
    }
#pragma unroll
    for (int i = 0; i < PPR; ++i) {
        const int piece = i * 64 + lane;
        *(u32x4 *)(rows + (piece / PPR) * (D + kRowPad) + 8 * (piece % PPR)) = v[i];
    }
}

}  // namespace

// ---- 1. chunk deltas ---------------------------------------------------------------------------------------------
// One wave per chunk (four chunks of consecutive pairs per workgroup). Delta H tile (fi, fj) = sum over the chunk's keys
// of K^T[fi] (w o K)[fj]: A = features x keys, B = keys x features, both gathered column-wise from the LDS tile of key
// rows; stored transposed (Delta H is symmetric up to the rounding of w o K), so that a lane holds four consecutive
// elements of a row. Delta U^T tile (fi, fj) = K^T[fi] (w o V)[fj], stored transposed likewise: row-major Delta U.
// REM: the weighted rows enter as bf16 value + remainder (the states are then as exact as those of a walk from the start; half as
// long again where chunks are many).
template <bool WITH_U, int D, bool REM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 8))) void small_chunk_delta_kernel(SmallArgs a)
{
    constexpr int NF = D / 16;                 // feature tiles that exist; a state is stored as D x D
    const PaddedRows at = {D + kRowPad};
    __shared__ __attribute__((aligned(16))) uint16_t s_k[4][64 * (D + kRowPad)];
    __shared__ __attribute__((aligned(16))) uint16_t s_v[WITH_U ? 4 : 1][WITH_U ? 64 * (D + kRowPad) : 8];
    __shared__ __attribute__((aligned(16))) float s_w[4][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int n = lane & 15, kg = lane >> 4;
    const int64_t unit_raw = (int64_t)blockIdx.x * 4 + w;
    const int64_t n_units = (int64_t)a.n_pairs * a.n_chunks;
    const bool live = unit_raw < n_units;
    const int64_t unit = live ? unit_raw : n_units - 1;     // a dead wave repeats the last chunk and stores nothing
    const int pair = (int)(unit % a.n_pairs), chunk = (int)(unit / a.n_pairs);
    const int b = pair / a.H, h = pair % a.H;
    const int tok0 = chunk * kChunk;
    stage_rows<D>(a, a.k, s_k[w], b, h, tok0, lane);
    if constexpr (WITH_U) stage_rows<D>(a, a.v, s_v[w], b, h, tok0, lane);
    const bool valid = tok0 + lane < a.T;
    const int64_t gi = (b * (int64_t)a.T + min(tok0 + lane, a.T - 1)) * a.H + h;
    const float G = wave_inclusive_scan(valid ? log2_gate(a.gate[gi]) : 0.0f, lane);
    const float Gt = lane_value(G, 63);
    const float beta = a.beta ? a.beta[gi] : 1.0f;
    s_w[w][lane] = valid ? exp2f(Gt - G) * beta : 0.0f;
    __syncthreads();
    f32x4 accH[2][2] = {{zero4(), zero4()}, {zero4(), zero4()}}, accU[2][2] = {{zero4(), zero4()}, {zero4(), zero4()}};
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const f32x4 w0 = *(const f32x4 *)&s_w[w][32 * ks + 4 * kg], w1 = *(const f32x4 *)&s_w[w][32 * ks + 16 + 4 * kg];
        bf16x8 kt[2], wk[2], wk_rem[2], wv[2], wv_rem[2];
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            f32x4 lo, hi;
            kt[f] = gather_transposed_bf16(s_k[w], at, 16 * f, lane, 32 * ks + 4 * kg, 32 * ks + 16 + 4 * kg);
            unpack8(kt[f], lo, hi);
            split8(lo * w0, hi * w1, wk[f], wk_rem[f]);
            if constexpr (WITH_U) {
                unpack8(gather_transposed_bf16(s_v[w], at, 16 * f, lane, 32 * ks + 4 * kg, 32 * ks + 16 + 4 * kg), lo,
                        hi);
                split8(lo * w0, hi * w1, wv[f], wv_rem[f]);
            }
        }
#pragma unroll
        for (int fi = 0; fi < NF; ++fi)
#pragma unroll
            for (int fj = 0; fj < NF; ++fj) {
                if constexpr (REM) accH[fi][fj] = mma16(kt[fi], wk_rem[fj], accH[fi][fj]);
                accH[fi][fj] = mma16(kt[fi], wk[fj], accH[fi][fj]);
                if constexpr (WITH_U && REM) accU[fi][fj] = mma16(kt[fi], wv_rem[fj], accU[fi][fj]);
                if constexpr (WITH_U) accU[fi][fj] = mma16(kt[fi], wv[fj], accU[fi][fj]);
            }
    }
    if (live) {
        const int64_t at = (pair * (int64_t)a.n_chunks + chunk) * (D * D);
#pragma unroll
        for (int fi = 0; fi < NF; ++fi)
#pragma unroll
            for (int fj = 0; fj < NF; ++fj) {
                *(f32x4 *)(a.dH + at + (16 * fj + n) * D + 16 * fi + 4 * kg) = accH[fi][fj];
                if constexpr (WITH_U) *(f32x4 *)(a.dU + at + (16 * fj + n) * D + 16 * fi + 4 * kg) = accU[fi][fj];
            }
        if (lane == 0) a.chunk_log2_decay[pair * (int64_t)a.n_chunks + chunk] = Gt;
    }
}

// ---- 2. states before every chunk --------------------------------------------------------------------------------
// One workgroup per pair, thread t: elements 4 t .. 4 t + 3 of the D x D states (row-major, as the caller's initial
// and final states).
template <bool WITH_U, int D>
__global__ __launch_bounds__(D * D / 4) void small_state_scan_kernel(SmallArgs a)
{
    constexpr int kAhead = WITH_U ? 8 : 16;
    constexpr int SS = D * D;
    const int pair = blockIdx.x, t = threadIdx.x;
    const int64_t base = pair * (int64_t)a.n_chunks * SS + 4 * t;
    const float *decay = a.chunk_log2_decay + pair * (int64_t)a.n_chunks;
    const int64_t ext = (int64_t)pair * SS + 4 * t;          // this piece in the caller's states
    f32x4 H = zero4(), U = zero4();
    if (a.H_init) H = *(const f32x4 *)(a.H_init + ext);
    if (WITH_U && a.U_init) U = *(const f32x4 *)(a.U_init + ext);
    for (int c0 = 0; c0 < a.n_chunks; c0 += kAhead) {
        f32x4 dh[kAhead], du[WITH_U ? kAhead : 1];
        float z[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
            const int c = min(c0 + i, a.n_chunks - 1);
            dh[i] = *(const f32x4 *)(a.dH + base + (int64_t)c * SS);
            if constexpr (WITH_U) du[i] = *(const f32x4 *)(a.dU + base + (int64_t)c * SS);
            z[i] = decay[c];
        }
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
            if (c0 + i < a.n_chunks) {
                const float zeta = exp2f(z[i]);
                *(f32x4 *)(a.sH + base + (int64_t)(c0 + i) * SS) = H;
                H = zeta * H + dh[i];
                if constexpr (WITH_U) {
                    *(f32x4 *)(a.sU + base + (int64_t)(c0 + i) * SS) = U;
                    U = zeta * U + du[i];
                }
            }
        }
    }
    if (a.H_final) *(f32x4 *)(a.H_final + ext) = H;
    if (WITH_U && a.U_final) *(f32x4 *)(a.U_final + ext) = U;
}

// ---- 3. walk: solve and readout ----------------------------------------------------------------------------------
namespace {

// The per-token inputs of a tile as a lane (n, kg) holds them: token n of the tile, features 4 kg .. of each block of 16.
template <bool WITH_U, int NF>
struct TileRows {
    u16x4 k[NF], q[NF], v[WITH_U ? NF : 1];
    float gate, lam, beta, alpha;
};
// Wave-uniform bases and lane offsets in bytes (a row of the tile is at most 15 stride_t away): 32 bits, but for packed
// tensors of 2^23 heads and more.
template <bool FAR>
using RowOffset = std::conditional_t<FAR, uint64_t, uint32_t>;
inline bool far_rows(const SmallArgs &a) { return 2 * (15 * (uint64_t)a.stride_t + kDs) > 0xffffffffu; }
template <bool WITH_U, int NF, bool FAR>
__device__ __forceinline__ TileRows<WITH_U, NF> fetch_tile(const SmallArgs &a, int b, int h, int tile, int n, int kg)
{
    TileRows<WITH_U, NF> in;
    const int64_t base = b * a.stride_b + 16 * (int64_t)tile * a.stride_t + h * a.stride_h;
    const int64_t ti = (b * (int64_t)a.T + 16 * tile) * a.H + h;
    const uint32_t i = min(n, a.T - 1 - 16 * tile);          // (rows past the end repeat the last one)
    const RowOffset<FAR> at = 2 * (i * (RowOffset<FAR>)a.stride_t + 4 * kg);
    const uint32_t at_t = 4 * (i * (uint32_t)a.H);
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        in.k[f] = *(const u16x4 *)((const char *)((const uint16_t *)a.k + base + 16 * f) + at);
        in.q[f] = *(const u16x4 *)((const char *)((const uint16_t *)a.q + base + 16 * f) + at);
        if constexpr (WITH_U) in.v[f] = *(const u16x4 *)((const char *)((const uint16_t *)a.v + base + 16 * f) + at);
    }
    in.gate = *(const float *)((const char *)(a.gate + ti) + at_t);
    in.lam = a.lambda ? *(const float *)((const char *)(a.lambda + ti) + at_t) : 0.0f;
    in.beta = a.beta ? *(const float *)((const char *)(a.beta + ti) + at_t) : 1.0f;
    in.alpha = WITH_U && a.alpha ? *(const float *)((const char *)(a.alpha + ti) + at_t) : 1.0f;
    return in;
}

// fragment halves: a fragment of 32 contraction values is two runs of four per lane
__device__ __forceinline__ bf16x8 join(u16x4 lo, u16x4 hi)
{
    const u16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
}
__device__ __forceinline__ u16x4 pack4(f32x4 x)
{
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    bf16x4 v;
#pragma unroll
    for (int p = 0; p < 4; ++p) v[p] = (__bf16)x[p];
    u32x2 b = __builtin_bit_cast(u32x2, v);
    asm("" : "+v"(b));                         // (two conversions of pairs: seen through, they become four and merges)
    return __builtin_bit_cast(u16x4, b);
}
// rounded value and what the rounding left over
__device__ __forceinline__ void split4(f32x4 x, u16x4 &val, u16x4 &rem)
{
    val = pack4(x);
    rem = pack4(x - IOBF16::cvt4(val));
}

// Products, c + X Y. An operand of 16 contraction values is one run of four per lane, which is also how an accumulator
// tile packs: 16 features take the 16-deep product. With 32 features everything is 32-deep, also over the tile's 16 keys
// (their second half of the slots is empty or carries a remainder): a 16-deep product that accumulates onto the result
// of a 32-deep one a few instructions earlier has read its accumulator before it was written.
template <int NF>
struct Products {                              // NF = 2
    static __device__ __forceinline__ f32x4 features(const u16x4 (&x)[2], const u16x4 (&y)[2], f32x4 c)
    {
        return mma16(join(x[0], x[1]), join(y[0], y[1]), c);
    }
    static __device__ __forceinline__ f32x4 keys(u16x4 x, u16x4 y, f32x4 c)
    {
        return mma16(join(x, x), join(y, u16x4{0, 0, 0, 0}), c);
    }
    static __device__ __forceinline__ f32x4 keys(u16x4 x, u16x4 val, u16x4 rem, f32x4 c)
    {
        return mma16(join(x, x), join(val, rem), c);
    }
};
template <>
struct Products<1> {
    static __device__ __forceinline__ f32x4 keys(u16x4 x, u16x4 y, f32x4 c)
    {
        typedef short s16x4 __attribute__((ext_vector_type(4)));
        return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, x), __builtin_bit_cast(s16x4, y), c, 0, 0,
                                                         0);
    }
    static __device__ __forceinline__ f32x4 keys(u16x4 x, u16x4 val, u16x4 rem, f32x4 c)
    {
        return keys(x, rem, keys(x, val, c));
    }
    static __device__ __forceinline__ f32x4 features(const u16x4 (&x)[1], const u16x4 (&y)[1], f32x4 c)
    {
        return keys(x[0], y[0], c);
    }
};

// sum over the 16 lanes of a row, inclusive prefix
__device__ __forceinline__ float row_inclusive_scan(float x)
{
    auto add = [](float v, auto ctrl) {
        return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value, 0xf, 0xf,
                                                              false));
    };
    x = add(x, std::integral_constant<int, 0x111>{});
    x = add(x, std::integral_constant<int, 0x112>{});
    x = add(x, std::integral_constant<int, 0x114>{});
    return add(x, std::integral_constant<int, 0x118>{});
}
// LDS that only one wave writes and reads: its accesses keep their order in the LDS queue, the compiler has to as well
__device__ __forceinline__ void wave_lds_order() { asm volatile("" ::: "memory"); }

}  // namespace

// One wave per (pair, segment of the sequence, part of the segment): it walks tiles of 16 tokens with H and U^T in
// accumulator tiles. A tile's solve needs its own 16 keys and nothing else of the sequence but the states before it: a pass
// has one key product, 4 masked elements per lane and 1 + 2 .. products for the gradient (with the four token tiles of a
// chunk of 64 solved against the state before the chunk, up to four key tiles and 16 masked elements). By symmetry an
// accumulator tile of H is the A operand of the solve, and U^T that of the readout: no transposition. H, U, x and the
// weighted rows enter products as bf16 value + remainder: the matrix pipe is idle most of the time. Bounded by instruction
// issue (36 vector instructions of a wave per pass at d = 16, some 300 per tile around them) and, where waves are few, by
// the chain of dependent products (0.11 us per pass, 1 us per tile). No barrier: LDS holds a wave's own 16 rows, for the
// transposed reads, and per-token scalars. d = 16, 6144 pairs x 197 tokens: 235 us for the whole forward pass with states
// per chunk of 64 in memory and four key tiles, 98 us now; d = 32, 3072 x 300: 306 and 138 us.
// Registers: 68 per lane at d = 16 (seven waves per SIMD; 6144 pairs fill six), at d = 32 110 without and 138 with the readout.
// WALK_FAR: 64-bit row offsets. WALK_CHUNK: the four waves of a workgroup take the four tiles of one chunk, each from the states
// before the chunk, which it advances over the tiles before its own from rows that the four waves have put into LDS (one
// barrier). With a wave per tile that fetched those rows itself, memory was waited for at every tile: d = 32, 144 pairs x 300
// tokens 32.3 us per forward pass, 23.2 now; sketched solve of 64 x 1000 tokens 65.0 and 56.2. (Four waves that solve against
// the state before the chunk, up to four key tiles per pass, are as fast, 22.5 and 58.0, but round the masked products of 64
// keys: 2.85e-3 from float64 instead of 2.60e-3.)
enum { WALK_NEAR, WALK_FAR, WALK_CHUNK };
template <bool WITH_U, int D, int MODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 16 ? 6 : WITH_U ? 3 : 4, 8)))
void small_walk_kernel(SmallArgs a)
{
    constexpr int NF = D / 16;                 // feature tiles
    constexpr bool FAR = MODE == WALK_FAR, CHUNK = MODE == WALK_CHUNK;
    typedef Products<NF> MM;
    __shared__ __attribute__((aligned(16))) uint16_t s_k[4][NF * 256];
    __shared__ __attribute__((aligned(16))) uint16_t s_v[4][WITH_U ? NF * 256 : 8];
    __shared__ __attribute__((aligned(16))) float s_tab[4][3 * 16];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // consecutive waves (CHUNK: workgroups): the same segment of consecutive pairs (adjacent memory in the [B,T,H,d] layout)
    const unsigned unit = CHUNK ? blockIdx.x : blockIdx.x * 4 + w;
    if (!CHUNK && unit >= (unsigned)a.n_pairs * a.n_segs * a.n_subs) return;
    const int pair = unit % (unsigned)a.n_pairs, part = unit / (unsigned)a.n_pairs;
    const int seg = CHUNK ? part : part / a.n_subs, sub = CHUNK ? w : part - seg * a.n_subs;
    const int b = pair / a.H, h = pair % a.H;
    // the states are known at tile_begin; tiles from solve_begin on are this wave's
    const int seg_tiles = a.seg_chunks * (kChunk / 16), n_tiles = (a.T + 15) / 16;
    const int sub_tiles = CHUNK ? 1 : seg_tiles / a.n_subs;
    const int tile_begin = seg * seg_tiles, solve_begin = tile_begin + sub * sub_tiles;
    const int tile_end = min(solve_begin + sub_tiles, n_tiles);
    if (!CHUNK && solve_begin >= n_tiles) return;
    const bool finishes = !CHUNK && a.whole && tile_end == n_tiles;
    uint16_t *rows = s_k[w], *vrows = s_v[w];
    float *Gtab = s_tab[w], *Btab = Gtab + 16, *Wtab = Gtab + 32;
    // a tile's rows and scalars into the wave's LDS; returns the decays before its tokens
    auto publish = [&](const TileRows<WITH_U, NF> &in, int tile, int n, int kg) {
        const bool valid = 16 * tile + n < a.T;
        const float G = row_inclusive_scan(valid ? log2_gate(in.gate) : 0.0f);
        if (kg == 0) {
            Gtab[n] = G;
            Btab[n] = valid ? in.beta : 0.0f;  // (tokens past the end weigh nothing)
        }
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            *(u16x4 *)(rows + f * 256 + 16 * n + 4 * kg) = in.k[f];
            if constexpr (WITH_U) *(u16x4 *)(vrows + f * 256 + 16 * n + 4 * kg) = in.v[f];
        }
        return G;
    };
    const PaddedRows at = {16};                // tiles of 16 rows x 16 features

    // ---- states before the segment: accumulator tile (fi, fj) holds S[16 fj + n][16 fi + 4 kg + r]
    f32x4 H[NF][NF], U[NF][NF];
    TileRows<WITH_U, NF> next;
    {
        const int lane = fresh_lane(), n = lane & 15, kg = lane >> 4;
        const bool first = !CHUNK && a.whole;
        const int64_t s0 = first ? (int64_t)pair * (D * D) : (pair * (int64_t)a.n_chunks + seg * a.seg_chunks) * (D * D);
        const float *Hs = first ? a.H_init : a.sH, *Us = first ? a.U_init : a.sU;
#pragma unroll
        for (int fi = 0; fi < NF; ++fi)
#pragma unroll
            for (int fj = 0; fj < NF; ++fj) {
                const int64_t e = s0 + (16 * fj + n) * D + 16 * fi + 4 * kg;
                H[fi][fj] = Hs ? *(const f32x4 *)(Hs + e) : zero4();
                U[fi][fj] = WITH_U && Us ? *(const f32x4 *)(Us + e) : zero4();
            }
        next = fetch_tile<WITH_U, NF, FAR>(a, b, h, CHUNK ? min(solve_begin, n_tiles - 1) : tile_begin, n, kg);
        if constexpr (CHUNK) {
            publish(next, solve_begin, n, kg);
            __syncthreads();
            if (solve_begin >= n_tiles) return;              // (none of the wave's tokens exists)
        }
    }
    for (int tile = tile_begin; tile < tile_end; ++tile) {
        // (lane-derived values formed anew in every tile: kept over the loop they would be spilled)
        const int lane = fresh_lane(), n = lane & 15, kg = lane >> 4;
        const TileRows<WITH_U, NF> in = next;                // (CHUNK: of the wave's own tile, the last of its loop)
        if constexpr (!CHUNK) next = fetch_tile<WITH_U, NF, FAR>(a, b, h, min(tile + 1, tile_end - 1), n, kg);
        const bool valid = 16 * tile + n < a.T;
        const int64_t ti0 = (b * (int64_t)a.T + 16 * tile) * a.H + h;    // the tile's first token in [B,T,H]

        // ---- per-token scalars and rows through LDS
        float Gc;
        if constexpr (CHUNK) {
            rows = s_k[tile - tile_begin];
            vrows = s_v[tile - tile_begin];
            Gtab = s_tab[tile - tile_begin];
            Btab = Gtab + 16;
            Gc = Gtab[n];
        } else {
            Gc = publish(in, tile, n, kg);
        }
        const float Gt = lane_value(Gc, 15);
        const float beta_c = valid ? in.beta : 0.0f;
        wave_lds_order();
        const f32x4 Gj = *(const f32x4 *)(Gtab + 4 * kg), bj = *(const f32x4 *)(Btab + 4 * kg);
        u16x4 kT[NF];                          // column 16 f + n of the keys 4 kg .. 4 kg + 3
#pragma unroll
        for (int f = 0; f < NF; ++f) kT[f] = transposed_run(rows + f * 256, at, lane, 4 * kg);
        // decay mask of Section 4.2.1 (log-space form of Appendix B.2, base 2) with the write gate folded in:
        // m[j,c] = 2^(G_c - G_j) beta_j for j <= c; lane element r <-> key j = 4 kg + r
        if (tile >= solve_begin) {
            // (hardware exp2 here and below: decays under 2^-126 are flushed to zero)
            float zeta = __builtin_amdgcn_exp2f(Gc);
            f32x4 decay;
#pragma unroll
            for (int r = 0; r < 4; ++r) decay[r] = (4 * kg + r <= n) ? __builtin_amdgcn_exp2f(Gc - Gj[r]) : 0.0f;
            f32x4 m = decay * bj;

            // ---- H as A operand, value and remainder
            u16x4 Hv[NF][NF], Hr[NF][NF];          // [row block][contraction block]
            float hn2 = 0.0f;
#pragma unroll
            for (int fo = 0; fo < NF; ++fo)
#pragma unroll
                for (int fi = 0; fi < NF; ++fi) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) hn2 += H[fi][fo][r] * H[fi][fo][r];
                    split4(H[fi][fo], Hv[fo][fi], Hr[fo][fi]);
                }

            // ---- Frobenius norm at every token (Section 4.2.1, the double sum folded by M[i,c] M[j,c] = M[j,c]^2 M[i,j]):
            //   ||H_c||^2 = zeta_c^2 ||H_[n]||^2 + sum_{j<=c} M[j,c]^2 w_j,
            //   w_j = beta_j (2 (zeta_j k_j^T H_[n] k_j + sum_{i<=j} m[i,j] G_ij^2) - beta_j G_jj^2)
            // (G = K K^T; M the decays without the write gate: no division by a gate, which may be as small as it likes)
            float fro;
            {
                float w_part = 0.0f, diag = 0.0f;
#pragma unroll
                for (int fo = 0; fo < NF; ++fo) {
                    const f32x4 hk = MM::features(Hr[fo], in.k, MM::features(Hv[fo], in.k, zero4()));
                    const f32x4 kc = IOBF16::cvt4(in.k[fo]);
#pragma unroll
                    for (int r = 0; r < 4; ++r) w_part += hk[r] * kc[r];
                }
                w_part *= zeta;
                const f32x4 G = MM::features(in.k, in.k, zero4());
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float g2 = G[r] * G[r];
                    w_part += m[r] * g2;
                    diag = 4 * kg + r == n ? g2 : diag;
                }
                const float wc = beta_c * sum_over_kg(2.0f * w_part - beta_c * diag);
                if (kg == 0) Wtab[n] = wc;
                wave_lds_order();
                const f32x4 wv = *(const f32x4 *)(Wtab + 4 * kg);
                float f = 0.0f;
#pragma unroll
                for (int r = 0; r < 4; ++r) f += decay[r] * decay[r] * wv[r];
                hn2 = lane_value(wave_inclusive_scan(hn2, lane), 63);
                // (the hardware's root takes a denormal argument for zero: the norm of a state below 1e-19)
                const float fro2 = fmaxf(zeta * zeta * hn2 + sum_over_kg(f), 0.0f);
                const bool tiny = fro2 < 0x1p-96f;
                fro = __builtin_amdgcn_sqrtf(tiny ? 0x1p64f * fro2 : fro2) * (tiny ? 0x1p-32f : 1.0f);
            }
            if (a.fro_out && valid && kg == 0) (a.fro_out + ti0)[(uint32_t)n * a.H] = fro;
            const float lam = a.lambda ? in.lam : a.lambda_scale * fro;      // Section 4.1: lambda_t = a ||H_t||_F

            // ---- Algorithm 1 in residual form; Section 4.1: L = ||H_t||_F + lambda_t, mu = lambda_t
            const float L = fro + lam, mu = lam;
            const float rcp = __builtin_amdgcn_rcpf(L + mu);
            const float s0 = 2.0f * rcp;
            const float rho = (L - mu) * rcp, rho2 = rho * rho;
            zeta = fmaxf(zeta, kMinZeta);
            const float rz = __builtin_amdgcn_rcpf(zeta);
            m *= rz;
            f32x4 xi[NF], dl[NF], gn[NF];
#pragma unroll
            for (int fo = 0; fo < NF; ++fo) {
                const f32x4 qv = IOBF16::cvt4(in.q[fo]);         // (columns of tokens past the end go nowhere)
                xi[fo] = zero4();
                dl[fo] = s0 * qv;
                gn[fo] = -rz * qv;
            }
            // weight schedule omega' = 4 / (4 - rho^2 omega) as wr = omega / 4
            float wr = 0.5f;
            const float w_rho = -4.0f * rho2, w_g = -4.0f * s0 * zeta, w_x = -4.0f * s0 * lam;
            for (int it = 0; it < a.n_iter; ++it) {
                wr = __builtin_amdgcn_rcpf(4.0f + w_rho * wr);
                const float cm = 4.0f * wr - 1.0f, ncs = w_g * wr, ncl = w_x * wr;
                u16x4 d[NF];
#pragma unroll
                for (int fo = 0; fo < NF; ++fo) d[fo] = pack4(dl[fo]);
                const u16x4 p = pack4(MM::features(in.k, d, zero4()) * m);
#pragma unroll
                for (int fo = 0; fo < NF; ++fo) {
                    gn[fo] = MM::features(Hr[fo], d, MM::features(Hv[fo], d, gn[fo]));
                    gn[fo] = MM::keys(kT[fo], p, gn[fo]);
                }
#pragma unroll
                for (int fo = 0; fo < NF; ++fo) {
                    xi[fo] += dl[fo];
                    dl[fo] = cm * dl[fo] + ncs * gn[fo] + ncl * xi[fo];
                }
            }
            f32x4 x[NF];
#pragma unroll
            for (int fo = 0; fo < NF; ++fo) x[fo] = xi[fo] + dl[fo];
            if (a.xhat_out && valid) {
                float *z = a.xhat_out + ti0 * a.xhat_row + (int64_t)n * a.H * a.xhat_row;
#pragma unroll
                for (int fo = 0; fo < NF; ++fo) {
                    *(f32x4 *)(z + 16 * fo + 4 * kg) = x[fo];
                    if (!WITH_U && a.xhat_zero_upper)            // (a reader of 64 stored features)
                        *(f32x4 *)(z + kDs + 16 * fo + 4 * kg) = zero4();
                }
            }
            // the next tile's rows are awaited here, where they have had the passes to arrive: behind the conditional store of
            // the outputs the wait would be for that store too
            if constexpr (!CHUNK) {
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    asm volatile("" : "+v"(next.k[f]), "+v"(next.q[f]));
                    if constexpr (WITH_U) asm volatile("" : "+v"(next.v[f]));
                }
                asm volatile("" : "+v"(next.gate), "+v"(next.lam), "+v"(next.beta), "+v"(next.alpha));
            }
            if constexpr (WITH_U) {
                // ---- readout y_c = zeta_c U_[n] x_c + sum_{j<=c} m[j,c] v_j (k_j . x_c), x = alpha xhat + (1 - alpha) q
                // (Section 4.3), formed with the mask divided by zeta_c and multiplied by zeta_c at the end
                if (a.alpha) {
#pragma unroll
                    for (int fo = 0; fo < NF; ++fo) x[fo] = in.alpha * x[fo] + (1.0f - in.alpha) * IOBF16::cvt4(in.q[fo]);
                }
                u16x4 xv[NF], xr[NF];
#pragma unroll
                for (int fo = 0; fo < NF; ++fo) split4(x[fo], xv[fo], xr[fo]);
                const u16x4 p = pack4(MM::features(in.k, xr, MM::features(in.k, xv, zero4())) * m);
#pragma unroll
                for (int fo = 0; fo < NF; ++fo) {
                    u16x4 Uv[NF], Ur[NF];
#pragma unroll
                    for (int fi = 0; fi < NF; ++fi) split4(U[fi][fo], Uv[fi], Ur[fi]);
                    f32x4 y = MM::features(Uv, xr, MM::features(Ur, xv, MM::features(Uv, xv, zero4())));
                    const u16x4 vT = transposed_run(vrows + fo * 256, at, lane, 4 * kg);
                    y = zeta * MM::keys(vT, p, y);
                    if (valid) {
                        const int64_t base = b * a.stride_b + 16 * (int64_t)tile * a.stride_t + h * a.stride_h;
                        char *o = (char *)((uint16_t *)a.o + base + 16 * fo);
                        IOBF16::store4(o + 2 * ((RowOffset<FAR>)n * (RowOffset<FAR>)a.stride_t + 4 * kg), 0, y[0], y[1], y[2], y[3]);
                    }
                }
            }
        }
        if (tile + 1 == tile_end && !finishes) break;
        // ---- states after the tile: H <- zeta_T H + K^T (w o K), U^T <- zeta_T U^T + K^T (w o V)
        wave_lds_order();                      // (scalars and rows are read again: registers are short during the passes)
        const float zt = __builtin_amdgcn_exp2f(Gt);
        f32x4 wj;                              // weights of the keys 4 kg + r in the states after the tile
#pragma unroll
        for (int r = 0; r < 4; ++r) wj[r] = __builtin_amdgcn_exp2f(Gt - Gtab[4 * kg + r]) * Btab[4 * kg + r];
#pragma unroll
        for (int fj = 0; fj < NF; ++fj) {
            u16x4 wkv, wkr;
            split4(IOBF16::cvt4(kT[fj]) * wj, wkv, wkr);
#pragma unroll
            for (int fi = 0; fi < NF; ++fi) H[fi][fj] = MM::keys(kT[fi], wkv, wkr, zt * H[fi][fj]);
            if constexpr (WITH_U) {
                split4(IOBF16::cvt4(transposed_run(vrows + fj * 256, at, lane, 4 * kg)) * wj, wkv, wkr);
#pragma unroll
                for (int fi = 0; fi < NF; ++fi) U[fi][fj] = MM::keys(kT[fi], wkv, wkr, zt * U[fi][fj]);
            }
        }
        wave_lds_order();                      // the next tile's rows replace these
    }
    // (with several segments the scan has written the final states)
    if (finishes && a.H_final) {
        const int lane = fresh_lane(), n = lane & 15, kg = lane >> 4;
#pragma unroll
        for (int fi = 0; fi < NF; ++fi)
#pragma unroll
            for (int fj = 0; fj < NF; ++fj) {
                const int64_t e = (int64_t)pair * (D * D) + (16 * fj + n) * D + 16 * fi + 4 * kg;
                *(f32x4 *)(a.H_final + e) = H[fi][fj];
                if (WITH_U) *(f32x4 *)(a.U_final + e) = U[fi][fj];
            }
    }
}

namespace {
size_t state_array_bytes(int n_pairs, int n_chunks, int d)
{
    return ((size_t)n_pairs * n_chunks * d * d * sizeof(float) + 255) & ~(size_t)255;
}
template <bool WITH_U, int D>
void launch_all(SmallArgs a, hipStream_t stream)
{
    const int64_t n_units = (int64_t)a.n_pairs * a.n_chunks;
    typedef WalkRule<D> Rule;
    const bool tile_waves = n_units <= kTileWaveChunks;
    const int64_t n_tiles = (a.T + 15) / 16;
    // (final states in the buffers of the initial ones: not where several waves of a pair would start from the initial states
    // while one of them writes the final ones; the scan reads and writes each of their elements in one thread)
    const bool in_place = a.H_final && (a.H_final == a.H_init || a.U_final == a.U_init);
    const bool whole = !(tile_waves && in_place) &&
                       (a.n_pairs >= Rule::many_pairs || a.n_chunks <= Rule::short_chunks ||
                        (tile_waves && n_tiles <= Rule::few_walk_tiles &&
                         a.n_pairs * n_tiles * n_tiles * n_tiles <= Rule::few_walk_work));
    a.whole = whole;
    a.seg_chunks = whole ? a.n_chunks : 1;
    a.n_segs = whole ? 1 : a.n_chunks;
    // (outputs that replace the rows of k or v: no wave advances the states over tiles that another one solves)
    const bool over_rows = a.o && (a.o == a.k || a.o == a.v);
    a.n_subs = whole && tile_waves && !over_rows ? a.seg_chunks * (kChunk / 16) : 1;
    const bool by_chunk = !whole && n_units <= Rule::chunk_workgroups;
    if (!whole) {
        const dim3 grid((unsigned)((n_units + 3) / 4));
        if (by_chunk) hipLaunchKernelGGL((small_chunk_delta_kernel<WITH_U, D, true>), grid, dim3(256), 0, stream, a);
        else hipLaunchKernelGGL((small_chunk_delta_kernel<WITH_U, D, false>), grid, dim3(256), 0, stream, a);
        hipLaunchKernelGGL((small_state_scan_kernel<WITH_U, D>), dim3((unsigned)a.n_pairs), dim3(D * D / 4), 0, stream, a);
    }
    if (by_chunk) {
        hipLaunchKernelGGL((small_walk_kernel<WITH_U, D, WALK_CHUNK>), dim3((unsigned)n_units), dim3(256), 0, stream, a);
        return;
    }
    const int64_t n_waves = (int64_t)a.n_pairs * a.n_segs * a.n_subs;
    const dim3 grid((unsigned)((n_waves + 3) / 4));
    if (far_rows(a)) hipLaunchKernelGGL((small_walk_kernel<WITH_U, D, WALK_FAR>), grid, dim3(256), 0, stream, a);
    else hipLaunchKernelGGL((small_walk_kernel<WITH_U, D, WALK_NEAR>), grid, dim3(256), 0, stream, a);
}
}  // namespace

// d: 16 or 32, the head dimension (32 for the solve of latent sketching)
size_t small_dim_workspace_bytes(int n_pairs, int n_chunks, int d, bool with_readout)
{
    const size_t decays = ((size_t)n_pairs * n_chunks * sizeof(float) + 255) & ~(size_t)255;
    return (with_readout ? 4 : 2) * state_array_bytes(n_pairs, n_chunks, d) + decays;
}

// `workspace`: small_dim_workspace_bytes(n_pairs, n_chunks, a.d, a.v != nullptr) bytes, 256-byte aligned.
hipError_t launch_small_dim_forward(SmallArgs a, void *workspace, hipStream_t stream)
{
    if (a.n_pairs < 1 || a.n_chunks < 1 || a.T < 1 || (a.d != 16 && a.d != 32)) return hipErrorInvalidValue;
    if ((int64_t)a.n_pairs * a.n_chunks > 0x7fffffff / 4) return hipErrorInvalidValue;
    const bool with_u = a.v != nullptr;
    if (with_u != (a.o != nullptr)) return hipErrorInvalidValue;
    if (!with_u && (a.alpha || a.U_init || a.U_final || a.d != 32)) return hipErrorInvalidValue;
    const size_t per_array = state_array_bytes(a.n_pairs, a.n_chunks, a.d);
    unsigned char *ws = (unsigned char *)workspace;
    a.dH = (float *)ws;
    a.sH = (float *)(ws + per_array);
    a.dU = with_u ? (float *)(ws + 2 * per_array) : nullptr;
    a.sU = with_u ? (float *)(ws + 3 * per_array) : nullptr;
    a.chunk_log2_decay = (float *)(ws + (with_u ? 4 : 2) * per_array);
    if (!with_u) launch_all<false, 32>(a, stream);
    else if (a.d == 32) launch_all<true, 32>(a, stream);
    else launch_all<true, 16>(a, stream);
    return hipGetLastError();
}

}  // namespace gka
