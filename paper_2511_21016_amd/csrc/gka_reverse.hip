// Reverse recurrences of the backward pass (Section 4.2.2, Eq. (Ai) and its counterpart for U), bf16 tensors, all in one
// walk over the sequence from its last token to its first. With
//   S_t = sum_{s>=t} M[t,s] (p_s x_s^T + x_s p_s^T)   (A_t + A_t^T),   Ubar_t = sum_{s>=t} M[t,s] dy_s xt_s^T,
// (no write gate inside them) it forms, per token,
//   dk_t = beta_t (Ubar_t^T v_t - S_t k_t),   dv_t = beta_t Ubar_t k_t,   kd_t = k_t . dk_t / beta_t,   vd_t = v_t . Ubar_t k_t.
// x and xt arrive as bf16 value + remainder, p, dy, k, v in bf16; products of the states, of the masked intra-chunk
// products and of the weighted rows take value + remainder operands (kept from the readouts this replaces: the gate
// gradient is a long cumulative sum of differences of these outputs, and only rounding of the stored tensors, common
// to all of them, cancels in it).
//
// One workgroup walks a segment of a pair's chunks; D / 16 waves. Wave w owns rows 16 w .. + 15 of -S, Ubar and Ubar^T as
// 16 x 16 accumulator tiles: tile jb holds element [16 w + n][16 jb + 4 kg + r] on lane (n, kg) = (lane & 15, lane >> 4),
// register r, so two neighbouring tiles convert in place into an A fragment of v_mfma_f32_16x16x32_bf16. Tokens sit on
// the N dimension. The rows of a chunk are staged in LDS once (32-byte granules XOR-swizzled with the row number: row
// reads and transpose reads without conflicts) and feed every product: two of the four readouts that this kernel
// replaces read k, x and p, the other two k, v, dy and xt, and each wrote 4 bytes per element for an elementwise
// kernel that combined them. PART selects the recurrences: 3 both in one walk (xt = x, i.e. no alpha-connection), 1 -S_t k_t
// only, 2 the Ubar parts, added to what the call before left in dk (with an alpha-connection the rows of x and of xt do
// not fit in LDS together).
//
// Bound by neither pipe: one workgroup per CU (its LDS), two waves per SIMD at d = 128 and one at d = 64, whose loads, LDS
// exchanges and barriers do not cover each other. 64 pairs x 4096 tokens, d = 128: 75 us for the segments' summaries and 246
// for the walk. (With the rows of the next chunk fetched into registers behind the output stores, 48 of them, 44 spilled:
// 80 + 352, a fifth of it spent where those loads were issued; copies straight into LDS without the touch of the next chunk's
// lines: 268.) With an alpha-connection, 64 pairs x 2000 tokens: part 1 (two chunks' tiles) 33 + 70, part 2 27 + 117. All
// variants fit in 231 registers without spills.
#include "gka_device.hpp"
#include "gka_kernels.hpp"

namespace gka {

namespace {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef MmaBF16::frag frag;

template <int D, int PART>
struct ReverseShape {
    static constexpr bool DO_S = PART & 1, DO_U = PART & 2;
    static constexpr int NW = D / 16, NT = 64 * NW;
    static constexpr int NTILE = D / 16;               // accumulator tiles of a wave's rows of a state
    static constexpr int KS = D / 32;                  // contraction steps over the features
    // staged tensors: k, x, x_lo | xt, xt_lo, then p (S) and dy, v (U)
    static constexpr int N_TENSORS = 3 + DO_S + 2 * DO_U;
    static constexpr int N_SUMMARY = 2 + DO_S + DO_U;  // ... of the summary launch: no queries k, v
    static constexpr int N_MATS = DO_S + DO_U + 1;     // masked key products: x . k (both), p . k (S), dy . v (U)
    static constexpr size_t tile_elems = (size_t)kChunk * D;
    static constexpr int UNITS = 6;                    // causal (token tile, pair of key tiles)
    static constexpr size_t p_bytes = (size_t)N_MATS * UNITS * 2 * 64 * 16;   // value and remainder
    static constexpr size_t tab_bytes = (2 + 2 * NW) * kChunk * 4;            // G, weights; partial dots
    // Two chunks' tiles where they fit (d = 64; -S_t k_t alone at d = 128), so that a chunk's copies have a whole chunk's work
    // to land in; else one, whose tiles are filled again as they fall free.
    static constexpr size_t lds_main(bool two) { return (two ? 2 : 1) * N_TENSORS * tile_elems * 2 + p_bytes + tab_bytes; }
    static constexpr bool TWO_FITS = lds_main(true) <= 160 * 1024;
    // (one recurrence at d = 64) two workgroups on a CU with one chunk's tiles each
    static constexpr bool TWO_GROUPS = NT == 256 && TWO_FITS && 2 * lds_main(false) <= 160 * 1024;
    static constexpr size_t lds_summary = 2 * N_SUMMARY * tile_elems * 2 + NW * kChunk * 4;   // two chunks; the waves' weights
    // a copy instruction of a wave moves 1 KiB: ROWS rows; two instructions per wave and tensor
    static constexpr int ROWS = 512 / D, COPIES = kChunk / ROWS / NW;
    typedef SwizzledRows<D * 2, 2> Rows;
};

__device__ __forceinline__ f32x4 mma16(frag a, frag b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// x as bf16 value and bf16 remainder
__device__ __forceinline__ void split8(const float (&x)[8], frag &hi, frag &lo)
{
    hi = MmaBF16::pack(x);
    float back[8];
    MmaBF16::unpack(hi, back);
#pragma unroll
    for (int e = 0; e < 8; ++e) back[e] = x[e] - back[e];
    lo = MmaBF16::pack(back);
}
__device__ __forceinline__ frag negate(frag x)
{
    u32x4_t u = __builtin_bit_cast(u32x4_t, x);
#pragma unroll
    for (int i = 0; i < 4; ++i) u[i] ^= 0x80008000u;
    return __builtin_bit_cast(frag, u);
}

}  // namespace

// Units of the masked key products that wave w takes. d = 128 with all three matrices: waves 0-5 one of [0] and one other, waves
// 6 and 7 three others each; else one after the other.
template <int D, int PART>
__device__ __forceinline__ int reverse_units(int w)
{
    typedef ReverseShape<D, PART> SH;
    if (D == 128 && SH::N_MATS == 3) return w < 6 ? 2 : 3;
    return (SH::N_MATS * SH::UNITS - w + SH::NW - 1) / SH::NW;
}
template <int D, int PART>
__device__ __forceinline__ int reverse_unit(int w, int i)
{
    typedef ReverseShape<D, PART> SH;
    if (D == 128 && SH::N_MATS == 3) return w < 6 ? w + SH::UNITS * i : SH::UNITS + 6 + 3 * (w - 6) + i;
    return w + SH::NW * i;
}

// TWO: two chunks' tiles in LDS.
template <int D, int PART, bool SUMMARY, bool TWO>
__global__ __launch_bounds__(4 * D) __attribute__((amdgpu_waves_per_eu(2))) void reverse_kernel(ReverseArgs a)
{
    typedef ReverseShape<D, PART> SH;
    typedef typename SH::Rows Rows;
    constexpr bool DO_S = SH::DO_S, DO_U = SH::DO_U;
    constexpr int NW = SH::NW, NT = SH::NT, NTILE = SH::NTILE, KS = SH::KS, UNITS = SH::UNITS;
    constexpr int NTEN = SUMMARY ? SH::N_SUMMARY : SH::N_TENSORS;
    constexpr Rows at;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    uint16_t *tiles = (uint16_t *)smem;
    // (order: x, x_lo, then p, dy, then the queries k, v)
    uint16_t *sX = tiles, *sXL = tiles + SH::tile_elems;
    uint16_t *sPr = tiles + 2 * SH::tile_elems;                                // p (S)
    uint16_t *sDY = tiles + (2 + DO_S) * SH::tile_elems;                       // dy (U)
    uint16_t *sK = tiles + (2 + DO_S + DO_U) * SH::tile_elems;
    uint16_t *sV = tiles + (3 + DO_S + DO_U) * SH::tile_elems;
    constexpr int TOUCH = TWO ? 0 : ((2 + DO_S + DO_U) * kChunk * D * 2 / 128 + NT - 1) / NT;
    frag *sP = (frag *)(tiles + (TWO ? 2 : 1) * NTEN * SH::tile_elems);
    float *sG = (float *)((unsigned char *)sP + SH::p_bytes);
    float *sW = sG + kChunk;
    float *sDot = sW + kChunk;                                                 // [2][NW][64]

    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    int lane = tid & 63, n = lane & 15, kg = lane >> 4;
    const int pair = blockIdx.x % a.n_pairs, seg = blockIdx.x / a.n_pairs;
    const int b = pair / a.H, h = pair % a.H;
    const int64_t row_stride = (int64_t)a.H * D;
    const int64_t base = ((int64_t)b * a.T * a.H + h) * D;                     // packed [B,T,H,D]
    const int64_t gate_base = (int64_t)b * a.T * a.H + h;
    const int n_chunks = (a.T + kChunk - 1) / kChunk;
    const int chunk_begin = seg * a.seg_len, chunk_end = min(chunk_begin + a.seg_len, n_chunks);
    if (chunk_begin >= chunk_end) return;              // (whole workgroup)
    // token tau of the walk -> token of the tensors
    auto tensor_token = [&](int tau) { return a.T - 1 - min(tau, a.T - 1); };

    // ---- states at the start of the segment: -S, Ubar, Ubar^T
    f32x4 st_s[DO_S ? NTILE : 1], st_u[DO_U ? NTILE : 1], st_t[DO_U && !SUMMARY ? NTILE : 1];
    constexpr int N_STATES = DO_S + DO_U;
    auto summary_tile = [&](int sg, int which, int row_tile, int jb) {
        return a.seg_buf + ((((int64_t)(pair * a.n_segs + sg) * N_STATES + which) * NW + row_tile) * NTILE + jb) * 256;
    };
#pragma unroll
    for (int jb = 0; jb < NTILE; ++jb) {
        const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (DO_S) st_s[jb] = zero;
        if constexpr (DO_U) st_u[jb] = zero;
        if constexpr (DO_U && !SUMMARY) st_t[jb] = zero;
    }
    if constexpr (!SUMMARY) {
        for (int sg = 0; sg < seg; ++sg) {
            const float decay = exp2f(a.seg_logdecay[pair * a.n_segs + sg]);
#pragma unroll
            for (int jb = 0; jb < NTILE; ++jb) {
                if constexpr (DO_S) {
                    const float *t = summary_tile(sg, 0, w, jb);
#pragma unroll
                    for (int r = 0; r < 4; ++r) st_s[jb][r] = decay * st_s[jb][r] + t[r * 64 + lane];
                }
                if constexpr (DO_U) {
                    const float *t = summary_tile(sg, DO_S, w, jb);
#pragma unroll
                    for (int r = 0; r < 4; ++r) st_u[jb][r] = decay * st_u[jb][r] + t[r * 64 + lane];
                    // Ubar^T[16 w + n][16 jb + 4 kg + r] = Ubar[16 jb + 4 kg + r][16 w + n]: tile (jb, w), lane
                    // (4 kg + r, n / 4), register n % 4
                    const f32x4 tt = *(const f32x4 *)(summary_tile(sg, DO_S, jb, w) + (n & 3) * 64 + 16 * (n >> 2) + 4 * kg);
                    st_t[jb] = decay * st_t[jb] + tt;
                }
            }
        }
    }

    // ---- rows of a chunk: direct copies global -> LDS (no staging registers: 48 for six tensors, which spilled and, read a chunk
    // ahead behind the output stores, held every wave up for a fifth of the walk). The lane picks the 16 source bytes that belong
    // at its place of the swizzled row. The compiler does not track these copies: they are awaited before the barrier that
    // hands their tiles over.
    auto source = [&](int i) {
        if (i < 2) return i == 0 ? a.x : a.x_lo;
        if (i < 2 + DO_S + DO_U) return DO_S && i == 2 ? a.p : a.dy;
        return i == 2 + DO_S + DO_U ? a.k : a.v;
    };
    const uint32_t tiles_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)tiles;
    auto copy_rows = [&](int first, int last, int c, int buffer) {
        constexpr int PER_ROW = 64 / SH::ROWS;           // 16-byte pieces of a row
#pragma unroll
        for (int j = 0; j < SH::COPIES; ++j) {
            const int idx = j * NW + w, row0 = idx * SH::ROWS;
            const int row = row0 + lane / PER_ROW;
            // (one uniform base per instruction, 32-bit offsets within its rows)
            const int t_low = max(a.T - 1 - (c * kChunk + row0 + SH::ROWS - 1), 0);
            const int64_t at0 = base + t_low * row_stride;
            const int off = (int)((uint32_t)(tensor_token(c * kChunk + row) - t_low) * (uint32_t)row_stride * 2u) +
                            (((lane % PER_ROW) * 16) ^ ((row & Rows::kMask) << 5));
#pragma unroll
            for (int i = 0; i < NTEN; ++i)
                if (i >= first && i < last)
                    async_copy16_to_lds_untracked(tiles_addr + ((buffer * NTEN + i) * (uint32_t)SH::tile_elems + idx * 512) * 2,
                                                  raw_buffer_words((const uint16_t *)source(i) + at0), off);
        }
    };
    auto gate_of = [&](int c) {                          // gate'_tau = gate_{T - tau}
        const int tau = min(c * kChunk + lane, a.T - 1);
        return tau == 0 ? 1.0f : a.gate[gate_base + (int64_t)(a.T - tau) * a.H];
    };
    // decays of a chunk, lane j: token j: G_j, the weight of token j in the states after the chunk
    float G = 0.0f, wj = 0.0f;
    auto scan = [&](int c, float gate) {
        const bool valid = c * kChunk + lane < a.T;
        G = wave_inclusive_scan(valid ? log2_gate(gate) : 0.0f, lane);
        wj = valid ? exp2f(lane_value(G, 63) - G) : 0.0f;
    };
    // operand fragment of row 16 t + n of a tile: features 32 ks + 4 kg .. + 3 and 16 further
    auto row_frag = [&](const uint16_t *tile, int t, int ks) {
        const u32x2_t lo = *(const u32x2_t *)(tile + at(16 * t + n, 32 * ks + 4 * kg));
        const u32x2_t hi = *(const u32x2_t *)(tile + at(16 * t + n, 32 * ks + 16 + 4 * kg));
        const u32x4_t u = {lo[0], lo[1], hi[0], hi[1]};
        return __builtin_bit_cast(frag, u);
    };
    // transposed: feature 16 jb + n, tokens 32 m + 4 kg .. + 3 and 16 further
    auto col_frag = [&](const uint16_t *tile, int jb, int m) {
        return gather_transposed_bf16(tile, at, 16 * jb, lane, 32 * m + 4 * kg, 32 * m + 16 + 4 * kg);
    };

    float Gseg = 0.0f;
    float gate_next = gate_of(chunk_begin);
    copy_rows(0, NTEN, chunk_begin, 0);
    for (int c = chunk_begin; c < chunk_end; ++c) {
        // (the lane index passes through an opaque copy in every chunk: addresses formed from it are not kept in registers
        // across the loop)
        lane = tid & 63;
        asm volatile("" : "+v"(lane));
        n = lane & 15;
        kg = lane >> 4;
        // ---- decays of the chunk (every wave for itself)
        const bool valid = c * kChunk + lane < a.T;
        scan(c, gate_next);
        const float Gtot = lane_value(G, 63);
        Gseg += Gtot;
        const int buffer = TWO ? (c - chunk_begin) & 1 : 0;
        if constexpr (TWO) {
            sX = tiles + (size_t)buffer * NTEN * SH::tile_elems;
            sXL = sX + SH::tile_elems;
            sPr = sX + 2 * SH::tile_elems;
            sDY = sX + (2 + DO_S) * SH::tile_elems;
            sK = sX + (2 + DO_S + DO_U) * SH::tile_elems;
            sV = sX + (3 + DO_S + DO_U) * SH::tile_elems;
        }
        if constexpr (SUMMARY) {
            sW = (float *)sP + w * kChunk;             // (of its own for every wave)
            sW[lane] = wj;
        } else if (w == 0) {
            sG[lane] = G;
            sW[lane] = wj;
        }
        wait_vector_memory_but<0>();                   // this wave's copies have landed
        lds_barrier();                                 // ... and everybody's; the table is complete
        gate_next = gate_of(c + 1);
        // One set of tiles: the next chunk's lines of the tensors that can only be copied at the end of this one are asked for now,
        // a word of each, so that the copies find them in L2.
        uint32_t touched[TOUCH > 0 ? TOUCH : 1];
        if constexpr (TOUCH > 0) {
            constexpr int LINES = kChunk * D * 2 / 128;  // of a tensor
#pragma unroll
            for (int j = 0; j < TOUCH; ++j) {
                const int line = min(j * NT + tid, (2 + DO_S + DO_U) * LINES - 1);
                const int i = line / LINES, row = line % LINES / (D * 2 / 128), part = line % (D * 2 / 128);
                const int tok = tensor_token(min((c + 1) * kChunk + row, chunk_end * kChunk - 1));
                const uint16_t *src = (const uint16_t *)(i < 2 ? (i == 0 ? a.x : a.x_lo) : DO_S && i == 2 ? a.p : a.dy);
                touched[j] = *(const uint32_t *)(src + base + tok * row_stride + part * 64);
            }
        }
        if constexpr (TWO) {
            if (c + 1 < chunk_end) copy_rows(0, NTEN, c + 1, buffer ^ 1);
        }

        // this wave's columns of the row tensors, transposed: A operand of the intra-chunk products and, weighted, B
        // operand of the state updates
        frag xT[2], xlT[2], pT[DO_S ? 2 : 1], dyT[DO_U ? 2 : 1];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            xT[m] = col_frag(sX, w, m);
            xlT[m] = col_frag(sXL, w, m);
            if constexpr (DO_S) pT[m] = col_frag(sPr, w, m);
            if constexpr (DO_U) dyT[m] = col_frag(sDY, w, m);
        }

        if constexpr (!SUMMARY) {
            // ---- masked key products, (token tile tt, key tiles 2 m, 2 m + 1) per unit, dealt out over the waves:
            // [0] x . k, [1] p . k (S), last: dy . v (U)
            // (a unit of [0], two products for every one of the others', counts twice: dealt out so that every wave has the same)
            const int n_units = reverse_units<D, PART>(w);
            for (int i = 0; i < n_units; ++i) {
                const int u0 = reverse_unit<D, PART>(w, i), mat = u0 / UNITS, u = u0 - mat * UNITS;
                const int tt = u < 2 ? u : u < 4 ? 2 : 3, m = u < 2 ? 0 : u & 1;
                const bool is_u = DO_U && mat == SH::N_MATS - 1;
                const uint16_t *keys = mat == 0 ? sX : is_u ? sDY : sPr, *query = is_u ? sV : sK;
                f32x4 acc[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const frag q = row_frag(query, tt, ks);
#pragma unroll
                    for (int t2 = 0; t2 < 2; ++t2) {
                        acc[t2] = mma16(row_frag(keys, 2 * m + t2, ks), q, acc[t2]);
                        if (mat == 0) acc[t2] = mma16(row_frag(sXL, 2 * m + t2, ks), q, acc[t2]);
                    }
                }
                // M[s,t] = exp2(G_t - G_s) for s <= t (Appendix B.2, base 2)
                const float Gt = sG[16 * tt + n];
                float pm[8];
#pragma unroll
                for (int t2 = 0; t2 < 2; ++t2) {
                    const int s0 = 16 * (2 * m + t2) + 4 * kg;
                    const f32x4 Gs = *(const f32x4 *)(sG + s0);
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        pm[4 * t2 + r] = s0 + r <= 16 * tt + n ? acc[t2][r] * __builtin_amdgcn_exp2f(Gt - Gs[r]) : 0.0f;
                }
                frag hi, lo;
                split8(pm, hi, lo);
                sP[((mat * UNITS + u) * 2 + 0) * 64 + lane] = hi;
                sP[((mat * UNITS + u) * 2 + 1) * 64 + lane] = lo;
            }

            // ---- the states' parts: zk = -S k + Ubar^T v, zv = Ubar k
            f32x4 zk[4], zv[DO_U ? 4 : 1];
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) zk[tt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            if constexpr (DO_U) {
#pragma unroll
                for (int tt = 0; tt < 4; ++tt) zv[tt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            }
            auto state_frag = [&](const f32x4 (&st)[NTILE], int m, frag &hi, frag &lo) {
                const float x[8] = {st[2 * m][0], st[2 * m][1], st[2 * m][2], st[2 * m][3],
                                    st[2 * m + 1][0], st[2 * m + 1][1], st[2 * m + 1][2], st[2 * m + 1][3]};
                split8(x, hi, lo);
            };
#pragma unroll
            for (int m = 0; m < KS; ++m) {
                __builtin_amdgcn_sched_barrier(0);
                frag sh, sl, uh, ul, th, tl;
                if constexpr (DO_S) state_frag(st_s, m, sh, sl);
                if constexpr (DO_U) {
                    state_frag(st_u, m, uh, ul);
                    state_frag(st_t, m, th, tl);
                }
#pragma unroll
                for (int tt = 0; tt < 4; ++tt) {
                    const frag kf = row_frag(sK, tt, m);
                    if constexpr (DO_S) {
                        zk[tt] = mma16(sh, kf, zk[tt]);
                        zk[tt] = mma16(sl, kf, zk[tt]);
                    }
                    if constexpr (DO_U) {
                        zv[tt] = mma16(uh, kf, zv[tt]);
                        zv[tt] = mma16(ul, kf, zv[tt]);
                        const frag vf = row_frag(sV, tt, m);
                        zk[tt] = mma16(th, vf, zk[tt]);
                        zk[tt] = mma16(tl, vf, zk[tt]);
                    }
                }
            }
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) {
                const float zt = exp2f(sG[16 * tt + n]);
                zk[tt] *= zt;
                if constexpr (DO_U) zv[tt] *= zt;
            }
            lds_barrier();                             // the masked products are visible
            // ---- intra-chunk parts: zk += xt (dy . v) - p (x . k) - x (p . k), zv += dy (x . k)
#pragma unroll
            for (int u = 0; u < UNITS; ++u) {
                __builtin_amdgcn_sched_barrier(0);
                const int tt = u < 2 ? u : u < 4 ? 2 : 3, m = u < 2 ? 0 : u & 1;
                auto masked = [&](int mat, int part) { return sP[((mat * UNITS + u) * 2 + part) * 64 + lane]; };
                const frag xk_hi = masked(0, 0), xk_lo = masked(0, 1);
                if constexpr (DO_S) {
                    const frag np = negate(pT[m]), nx = negate(xT[m]);
                    const frag pk_hi = masked(1, 0), pk_lo = masked(1, 1);
                    zk[tt] = mma16(np, xk_hi, zk[tt]);
                    zk[tt] = mma16(np, xk_lo, zk[tt]);
                    zk[tt] = mma16(nx, pk_hi, zk[tt]);
                    zk[tt] = mma16(nx, pk_lo, zk[tt]);
                    zk[tt] = mma16(negate(xlT[m]), pk_hi, zk[tt]);
                }
                if constexpr (DO_U) {
                    const frag dv_hi = masked(SH::N_MATS - 1, 0), dv_lo = masked(SH::N_MATS - 1, 1);
                    zk[tt] = mma16(xT[m], dv_hi, zk[tt]);
                    zk[tt] = mma16(xT[m], dv_lo, zk[tt]);
                    zk[tt] = mma16(xlT[m], dv_hi, zk[tt]);
                    zv[tt] = mma16(dyT[m], xk_hi, zv[tt]);
                    zv[tt] = mma16(dyT[m], xk_lo, zv[tt]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            // ---- outputs: lane (n, kg) holds features 16 w + 4 kg .. + 3 of token 16 tt + n
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) {
                const int tau = c * kChunk + 16 * tt + n;
                const bool live = tau < a.T;
                const int tok = tensor_token(tau);
                const int64_t off = base + tok * row_stride + 16 * w + 4 * kg;
                if (PART == 2) zk[tt] += *(const f32x4 *)(a.dk + off);
                if constexpr (DO_U) {
                    const float be = a.beta ? a.beta[gate_base + (int64_t)tok * a.H] : 1.0f;
                    const f32x4 kv = IOBF16::cvt4(*(const u16x4 *)(sK + at(16 * tt + n, 16 * w + 4 * kg)));
                    const f32x4 vv = IOBF16::cvt4(*(const u16x4 *)(sV + at(16 * tt + n, 16 * w + 4 * kg)));
                    float kd = 0.0f, vd = 0.0f;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        kd += kv[r] * zk[tt][r];
                        vd += vv[r] * zv[tt][r];
                    }
                    kd = sum_over_kg(kd);
                    vd = sum_over_kg(vd);
                    if (kg == 0) {
                        sDot[w * kChunk + 16 * tt + n] = kd;
                        sDot[(NW + w) * kChunk + 16 * tt + n] = vd;
                    }
                    if (live) {
                        *(f32x4 *)(a.dk + off) = be * zk[tt];
                        *(f32x4 *)(a.dv + off) = be * zv[tt];
                    }
                } else {
                    if (live) *(f32x4 *)(a.dk + off) = zk[tt];
                }
            }
        }

        if constexpr (TOUCH > 0) {
#pragma unroll
            for (int j = 0; j < TOUCH; ++j) asm volatile("" ::"v"(touched[j]));
        }
        if constexpr (!SUMMARY) {
            lds_barrier();                             // the queries' tiles are free; the partial dots are complete
            if (!TWO && c + 1 < chunk_end) copy_rows(2 + DO_S + DO_U, NTEN, c + 1, 0);
            if constexpr (DO_U) {
                if (w == 0 && valid) {
                    float kd = 0.0f, vd = 0.0f;
#pragma unroll
                    for (int i = 0; i < NW; ++i) {
                        kd += sDot[i * kChunk + lane];
                        vd += sDot[(NW + i) * kChunk + lane];
                    }
                    const int64_t g = gate_base + (int64_t)tensor_token(c * kChunk + lane) * a.H;
                    a.kd[g] = kd;
                    a.vd[g] = vd;
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);

        // ---- state <- zeta_C state + sum of weighted outer products
        const float zetaC = exp2f(Gtot);
        frag wx_hi[2], wx_lo[2], wp_hi[DO_S ? 2 : 1], wp_lo[DO_S ? 2 : 1], wd_hi[DO_U ? 2 : 1], wd_lo[DO_U ? 2 : 1];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const f32x4 w0 = *(const f32x4 *)(sW + 32 * m + 4 * kg), w1 = *(const f32x4 *)(sW + 32 * m + 16 + 4 * kg);
            auto weighted = [&](frag src, frag src_lo, bool has_lo, float sign, frag &hi, frag &lo) {
                float x[8];
                MmaBF16::unpack(src, x);
                if (has_lo) {
                    float x2[8];
                    MmaBF16::unpack(src_lo, x2);
#pragma unroll
                    for (int e = 0; e < 8; ++e) x[e] += x2[e];
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x[e] *= sign * w0[e];
                    x[4 + e] *= sign * w1[e];
                }
                split8(x, hi, lo);
            };
            weighted(xT[m], xlT[m], true, 1.0f, wx_hi[m], wx_lo[m]);
            if constexpr (DO_S) weighted(pT[m], pT[m], false, -1.0f, wp_hi[m], wp_lo[m]);
            if constexpr (DO_U) weighted(dyT[m], dyT[m], false, 1.0f, wd_hi[m], wd_lo[m]);
        }
#pragma unroll
        for (int jb = 0; jb < NTILE; ++jb) {
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (DO_S) st_s[jb] *= zetaC;
            if constexpr (DO_U) st_u[jb] *= zetaC;
            if constexpr (DO_U && !SUMMARY) st_t[jb] *= zetaC;
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const frag xc = col_frag(sX, jb, m), xlc = col_frag(sXL, jb, m);
                if constexpr (DO_S) {
                    const frag pc = col_frag(sPr, jb, m);
                    const frag npc = negate(pc);
                    st_s[jb] = mma16(xc, wp_hi[m], st_s[jb]);
                    st_s[jb] = mma16(xc, wp_lo[m], st_s[jb]);
                    st_s[jb] = mma16(xlc, wp_hi[m], st_s[jb]);
                    st_s[jb] = mma16(npc, wx_hi[m], st_s[jb]);
                    st_s[jb] = mma16(npc, wx_lo[m], st_s[jb]);
                }
                if constexpr (DO_U) {
                    st_u[jb] = mma16(xc, wd_hi[m], st_u[jb]);
                    st_u[jb] = mma16(xc, wd_lo[m], st_u[jb]);
                    st_u[jb] = mma16(xlc, wd_hi[m], st_u[jb]);
                    if constexpr (!SUMMARY) {
                        const frag dc = col_frag(sDY, jb, m);
                        st_t[jb] = mma16(dc, wx_hi[m], st_t[jb]);
                        st_t[jb] = mma16(dc, wx_lo[m], st_t[jb]);
                    }
                }
            }
        }
        if constexpr (!SUMMARY) {
            lds_barrier();                             // the other tiles and the table are free
            if (!TWO && c + 1 < chunk_end) copy_rows(0, 2 + DO_S + DO_U, c + 1, 0);
        }
    }
    wait_all_memory();                                 // no copy into this workgroup's LDS may be in flight when it ends

    if constexpr (SUMMARY) {
#pragma unroll
        for (int jb = 0; jb < NTILE; ++jb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if constexpr (DO_S) summary_tile(seg, 0, w, jb)[r * 64 + lane] = st_s[jb][r];
                if constexpr (DO_U) summary_tile(seg, DO_S, w, jb)[r * 64 + lane] = st_u[jb][r];
            }
        if (tid == 0) a.seg_logdecay[pair * a.n_segs + seg] = Gseg;
    } else if constexpr (DO_U) {
        if (a.fin_xtdy && seg == a.n_segs - 1) {       // sum_t M[0,t] xt_t dy_t^T, row-major
            float *S1 = a.fin_xtdy + (int64_t)pair * D * D + (int64_t)(16 * w + n) * D;
#pragma unroll
            for (int jb = 0; jb < NTILE; ++jb) *(f32x4 *)(S1 + 16 * jb + 4 * kg) = st_t[jb];
        }
    }
}

namespace {
template <int D, int PART>
hipError_t launch_reverse_t(const ReverseArgs &a, hipStream_t stream)
{
    typedef ReverseShape<D, PART> SH;
    // d = 64, one recurrence, more workgroups than CUs: two of them on a CU with one chunk's tiles each. Whole backward pass,
    // two chunks' tiles and one workgroup / this: 257 pairs x 500 tokens 479 / 409 us, 300 x 1000 994 / 854, 1000 x 150 487 / 430; up
    // to a workgroup for each CU two chunks' tiles (256 x 500: 371, 382 with rows fetched into registers).
    constexpr bool ONE = !SH::TWO_FITS || SH::TWO_GROUPS;
    const bool two = SH::TWO_FITS && !(SH::TWO_GROUPS && (int64_t)a.n_pairs * a.n_segs > kComputeUnits);
    static bool lds_raised[kMaxLdsDevices] = {};
    hipError_t e = raise_lds_limits(lds_raised, {{(const void *)reverse_kernel<D, PART, false, SH::TWO_FITS>, SH::lds_main(SH::TWO_FITS)},
                                                 {(const void *)reverse_kernel<D, PART, false, !ONE>, SH::lds_main(!ONE)},
                                                 {(const void *)reverse_kernel<D, PART, true, true>, SH::lds_summary}});
    if (e != hipSuccess) return e;
    if (a.n_segs > 1) {                                // summaries of every segment but the last, from zero states
        hipLaunchKernelGGL((reverse_kernel<D, PART, true, true>), dim3(a.n_pairs * (a.n_segs - 1)), dim3(SH::NT), SH::lds_summary,
                           stream, a);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const dim3 grid(a.n_pairs * a.n_segs), block(SH::NT);
    if (two) hipLaunchKernelGGL((reverse_kernel<D, PART, false, SH::TWO_FITS>), grid, block, SH::lds_main(true), stream, a);
    else hipLaunchKernelGGL((reverse_kernel<D, PART, false, !ONE>), grid, block, SH::lds_main(!ONE), stream, a);
    return hipGetLastError();
}
}  // namespace

size_t reverse_workspace_bytes(int n_pairs, int n_segs, int d)
{
    return (size_t)n_pairs * n_segs * 2 * d * d * sizeof(float) + (size_t)n_pairs * n_segs * sizeof(float);
}

hipError_t launch_reverse(const ReverseArgs &a, int d, int part, hipStream_t stream)
{
    if (d == 128) {
        if (part == 3) return launch_reverse_t<128, 3>(a, stream);
        return part == 1 ? launch_reverse_t<128, 1>(a, stream) : launch_reverse_t<128, 2>(a, stream);
    }
    if (part == 3) return launch_reverse_t<64, 3>(a, stream);
    return part == 1 ? launch_reverse_t<64, 1>(a, stream) : launch_reverse_t<64, 2>(a, stream);
}

}  // namespace gka
